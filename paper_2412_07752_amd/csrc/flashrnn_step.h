// One time step on its own (bf16 I/O, T = 1: token-by-token generation).  The persistent kernels spend a one-step call on bringing a whole head's R
// into the registers of one CU per batch tile; here nothing has to stay anywhere, so a head's units are dealt out over the chip: one workgroup per 16 units
// (all gates) and RB batch rows, whose 256 threads share the contraction.  A thread reads 16 bytes of R at a time, eight units of one gate of one
// contraction row, as they lie in the caller's tensor; products and sums are float32 (bf16 operands, as on the matrix cores).  With few rows R is read
// once, and the call is as long as the latency of a launch, one round of loads and the point-wise function: sLSTM 4 x 192, 1 row 8.7 -> 4.0 us.
#pragma once
#include "flashrnn_kernels.h"

namespace flashrnn {

template <int CELL, int RB>
__global__ __launch_bounds__(256) void step_kernel(const KernelParams p) {
    using CT = CellTraits<CELL>;
    constexpr int G = CT::G, S = CT::S, NC = CT::NC, COLS = 2 * G, KS = 256 / COLS, NI = 8;   // pieces of 8 units per contraction row, rows at a time, rounds in flight
    const uint32_t B = p.B, NH = p.NH, D = p.D, HD = NH * D, blocks = D / 16, tid = threadIdx.x;
    const uint32_t e0 = blockIdx.x % blocks * 16, n = blockIdx.x / blocks % NH, b0 = blockIdx.x / (blocks * NH) * RB;
    __shared__ float part[KS][COLS * 8 + 4][RB];   // (the threads' sums: slice, column)
    if (blockIdx.x == 0 && tid == 0) { p.err[0] = 0; p.err[1] = 0; }   // (as the packing kernel of the other plans)

    // ---- what the point-wise function of this thread's (unit, row) pair needs is requested first: behind the contraction it would be a second round of memory latency
    const uint32_t u = tid % 16, pr = tid / 16, b = b0 + pr, e = e0 + u;
    const bool pair = tid < 16 * RB && b < B;
    float st[S];
    uint32_t wx_bits[G], b_bits[G];
    if (pair) {
#pragma unroll
        for (int s = 0; s < S; ++s) st[s] = p.states0 != nullptr ? p.states0[((size_t)s * B + b) * HD + n * D + e] : 0.0f;
#pragma unroll
        for (int g2 = 0; g2 < G; ++g2) {
            wx_bits[g2] = ((const uint16_t*)p.Wx)[((size_t)b * G + g2) * HD + n * D + e];
            b_bits[g2] = ((const uint16_t*)p.bias)[((size_t)n * G + g2) * D + e];
        }
    }

    const uint32_t ks = tid / COLS, col = tid % COLS, g = col / 2, half = col % 2;
    float acc[RB][8];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[r][j] = 0.0f;
    auto contract = [&](auto state_c) {   // (without initial states R meets zeros, as everywhere: an infinite or NaN weight makes a NaN)
        const uint16_t* R = (const uint16_t*)p.R + (size_t)n * D * G * D + g * D + e0 + half * 8;
        const float* h = p.states0 + n * D;
        for (uint32_t d0 = ks; d0 < D; d0 += KS * NI) {
            i32x4 w[NI];
            float hv[NI][RB];
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const uint32_t d = d0 + i * KS < D ? d0 + i * KS : d0;
                w[i] = *(const i32x4*)(R + (size_t)d * G * D);
#pragma unroll
                for (int r = 0; r < RB; ++r) hv[i][r] = decltype(state_c)::value ? h[(size_t)(b0 + r < B ? b0 + r : B - 1) * HD + d] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                if (d0 + i * KS >= D) break;
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const float x = bf16_bits_to_f32(f32_to_bf16_bits(hv[i][r]));   // (the operand h is rounded to bf16)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        acc[r][2 * j] = fmaf(x, bf16_bits_to_f32((uint32_t)w[i][j] & 0xFFFFu), acc[r][2 * j]);
                        acc[r][2 * j + 1] = fmaf(x, __builtin_bit_cast(float, (uint32_t)w[i][j] & 0xFFFF0000u), acc[r][2 * j + 1]);
                    }
                }
            }
        }
    };
    if (ks < (uint32_t)KS) {
        if (p.states0 != nullptr) contract(std::true_type{});
        else contract(std::false_type{});
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int j = 0; j < 8; ++j) part[ks][col * 8 + j][r] = acc[r][j];
    }
    __syncthreads();
    // the slices' sums: all threads, each a run of them, then the point-wise function of one (unit, row) pair per thread
    constexpr int NV = COLS * 8 * RB, NSL = 256 / NV > 0 ? 256 / NV : 1;   // values, threads per value
    __shared__ float sums[NSL][NV];
    for (uint32_t x = tid; x < (uint32_t)NV * NSL; x += 256) {
        const uint32_t v = x % NV, sl = x / NV, c2 = v / RB, r = v % RB;
        float a = 0.0f;
#pragma unroll
        for (uint32_t k = 0; k < (KS + NSL - 1) / NSL; ++k)
            if (sl + k * NSL < (uint32_t)KS) a += part[sl + k * NSL][c2][r];
        sums[sl][v] = a;
    }
    __syncthreads();
    if (!pair) return;
    float wx[G], yb[G], cv[NC];
#pragma unroll
    for (int s = 0; s < S; ++s) p.states[((size_t)s * B + b) * HD + n * D + e] = st[s];
#pragma unroll
    for (int g2 = 0; g2 < G; ++g2) {
        wx[g2] = bf16_bits_to_f32(wx_bits[g2]);
        yb[g2] = bf16_bits_to_f32(b_bits[g2]);
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl) yb[g2] += sums[sl][(g2 * 16 + u) * RB + pr];
    }
    Cell<CELL, true>::fwd(wx, yb, st, cv);
#pragma unroll
    for (int s = 0; s < S; ++s) p.states[((size_t)(S + s) * B + b) * HD + n * D + e] = st[s];
    if (p.cache != nullptr) store_record<true, CT::RS, NC>(make_rsrc((const char*)p.cache + (size_t)n * D * CT::RS * 2), ((b * HD) + e) * CT::RS * 2, 0, cv);
}

}  // namespace flashrnn
