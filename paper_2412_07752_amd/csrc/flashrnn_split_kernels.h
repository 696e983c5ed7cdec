// Persistent kernels for heads split over the CUs of one XCD (bf16 I/O, heads of up to 1024 units), and for those spread over all XCDs (up to 2048 units).
//
// Backward: every member of a group keeps the gate gradients dg_t of its own units to itself and multiplies them with the columns of R
// that belong to them: a partial dh_{t-1} of the WHOLE head.  What crosses the CUs are these partial sums (float32, added in a fixed
// order by the unit's owner), not the gate gradients: 4 D bytes per row out and in instead of 2 G D bytes in, the matrix
// product needs one CU's 16 UB G contraction elements in LDS instead of all G D, and the hand-over follows the product instead of preceding it.
//
// The waves of a workgroup have roles.  A wave's vector memory operations return in order, so a wave that waits for another CU's words must not
// have a load from HBM in its queue:
//   compute waves   point-wise function, matrix product, exchange; nothing else of theirs touches memory
//   load waves      the inputs of the next steps, straight into LDS, in bursts of several steps: a CU's vector memory path returns all its waves'
//                   loads in order, so a poll behind loads from HBM waits for those whoever issued them; once every few steps that costs little
//                   (sLSTM 8 x 256, 32 rows forward, 2048 steps: loads every step 2.96 ms, every 2 / 4 / 8 / 16 steps 2.41 / 2.19 / 2.11 / 2.05, none at all 1.77)
//   store waves     the outputs of the step, from the LDS rows that the compute waves leave
// They meet at the barriers of a step only.
// (Backward kernels, against the exchange of gate gradients by bwd_kernel: sLSTM 8 x 256, 32 rows, 2048 steps 3.27 -> 1.79 ms, 3 x 256, 16 rows, 1024
// steps 1.59 -> 0.84 ms, LSTM 1 x 768, 128 rows, 1024 steps 6.77 -> 3.25 ms.  Forward kernels, against fwd_kernel: 2.31 -> 1.98 ms, 1.00 -> 0.76, 3.30 -> 2.29.)
#pragma once
#include "flashrnn_kernels.h"

namespace flashrnn {

// All waves of the workgroup; LDS writes in front of it are visible behind it.  (Not __syncthreads(): nothing else is waited for.)
__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N> __device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// ---------------------------------------------------------------------------------------------
// The Jacobian of a step in two parts: factors that do not depend on dh_t, formed while the exchange is on its way, and the few
// multiply-adds behind it.
// ---------------------------------------------------------------------------------------------
template <int CELL> struct PointGrad;
template <> struct PointGrad<CELL_LSTM> {   // k = {o (1 - tanh^2 c), z i (1 - i), c_prev f (1 - f), i (1 - z^2), tanh(c) o (1 - o)}
    static constexpr int NK = 6;
    static __device__ __forceinline__ void factors(const float (&cv)[4], const float (&sc)[2], const float (&sp)[2], float (&k)[NK]) {
        const float i = cv[0], f = cv[1], z = cv[2], o = cv[3], tc = tanh_<true>(sc[1]);
        k[0] = o * (1.0f - tc * tc);
        k[1] = z * i * (1.0f - i);
        k[2] = sp[1] * f * (1.0f - f);
        k[3] = i * (1.0f - z * z);
        k[4] = tc * o * (1.0f - o);
        k[5] = f;
    }
    static __device__ __forceinline__ void apply(const float (&k)[NK], float (&ds)[2], float (&dwx)[4], float (&dg)[4]) {
        const float dh = ds[0], dc = fmaf(dh, k[0], ds[1]);
        dg[0] = dc * k[1]; dg[1] = dc * k[2]; dg[2] = dc * k[3]; dg[3] = dh * k[4];
        dwx[0] = dg[0]; dwx[1] = dg[1]; dwx[2] = dg[2]; dwx[3] = dg[3];
        ds[0] = 0.0f; ds[1] = dc * k[5];
    }
};
template <> struct PointGrad<CELL_SLSTM> {   // k = {o/n, o c/n^2, z, i, c_prev, n_prev, f sig(-f), i (1 - z^2), (c/n) o (1 - o), f}
    static constexpr int NK = 10;
    static __device__ __forceinline__ void factors(const float (&cv)[5], const float (&sc)[4], const float (&sp)[4], float (&k)[NK]) {
        const float inv = fast_rcp(sc[2]), q = sc[1] * inv, o = cv[3], z = cv[2], oi = o * inv;
        k[0] = oi;
        k[1] = oi * q;
        k[2] = z;
        k[3] = cv[0];
        k[4] = sp[1];
        k[5] = sp[2];
        k[6] = cv[1] * cv[4];
        k[7] = cv[0] * (1.0f - z * z);
        k[8] = q * o * (1.0f - o);
        k[9] = cv[1];
    }
    static __device__ __forceinline__ void apply(const float (&k)[NK], float (&ds)[4], float (&dwx)[4], float (&dg)[4]) {
        const float dh = ds[0], dc = fmaf(dh, k[0], ds[1]), dn = fmaf(-dh, k[1], ds[2]);
        dg[0] = fmaf(dc, k[2], dn) * k[3];
        dg[1] = fmaf(dc, k[4], dn * k[5]) * k[6];
        dg[2] = dc * k[7];
        dg[3] = dh * k[8];
        dwx[0] = dg[0]; dwx[1] = dg[1]; dwx[2] = dg[2]; dwx[3] = dg[3];
        ds[0] = 0.0f; ds[1] = dc * k[9]; ds[2] = dn * k[9]; ds[3] = 0.0f;
    }
};
template <> struct PointGrad<CELL_GRU> {   // k = {(1 - z)(1 - cand^2), (h_prev - cand) z (1 - z), k0 yn r (1 - r), k0 r, z}
    static constexpr int NK = 5;
    static __device__ __forceinline__ void factors(const float (&cv)[4], const float (&)[1], const float (&sp)[1], float (&k)[NK]) {
        const float r = cv[0], z = cv[1], cand = cv[2], yn = cv[3];
        k[0] = (1.0f - z) * (1.0f - cand * cand);
        k[1] = (sp[0] - cand) * z * (1.0f - z);
        k[2] = k[0] * yn * r * (1.0f - r);
        k[3] = k[0] * r;
        k[4] = z;
    }
    static __device__ __forceinline__ void apply(const float (&k)[NK], float (&ds)[1], float (&dwx)[3], float (&dg)[3]) {
        const float dh = ds[0];
        dg[0] = dh * k[2]; dg[1] = dh * k[1]; dg[2] = dh * k[3];
        dwx[0] = dg[0]; dwx[1] = dg[1]; dwx[2] = dh * k[0];
        ds[0] = dh * k[4];
    }
};
template <> struct PointGrad<CELL_GRU4> {
    static constexpr int NK = 5;
    static __device__ __forceinline__ void factors(const float (&cv)[4], const float (&)[1], const float (&sp)[1], float (&k)[NK]) {
        const float z = cv[0], r = cv[1], cand = cv[2], tg = cv[3];
        const float pre = (1.0f - z) * (1.0f - cand * cand);
        k[0] = (sp[0] - cand) * z * (1.0f - z);
        k[1] = pre * tg * r * (1.0f - r);
        k[2] = pre;
        k[3] = pre * r * (1.0f - tg * tg);
        k[4] = z;
    }
    static __device__ __forceinline__ void apply(const float (&k)[NK], float (&ds)[1], float (&dwx)[4], float (&dg)[4]) {
        const float dh = ds[0];
#pragma unroll
        for (int g = 0; g < 4; ++g) { dg[g] = dh * k[g]; dwx[g] = dg[g]; }
        ds[0] = dh * k[4];
    }
};
template <> struct PointGrad<CELL_ELMAN> {
    static constexpr int NK = 1;
    static __device__ __forceinline__ void factors(const float (&cv)[1], const float (&)[1], const float (&)[1], float (&k)[NK]) { k[0] = 1.0f - cv[0] * cv[0]; }
    static __device__ __forceinline__ void apply(const float (&k)[NK], float (&ds)[1], float (&dwx)[1], float (&dg)[1]) {
        dg[0] = ds[0] * k[0];
        dwx[0] = dg[0];
        ds[0] = 0.0f;
    }
};

// partial sums of one [16 units] x [BT rows] block: BT / 4 floats per lane (lane (c, quad): unit c; rows quad (+ 4), with 16 rows 4 quad ..)
template <int PP, int AUX = 0> __device__ __forceinline__ void store_part(rsrc_t rs, uint32_t voff, uint32_t soff, const float (&v)[PP]) {
    int x[PP];
#pragma unroll
    for (int i = 0; i < PP; ++i) x[i] = exch_word(__builtin_bit_cast(uint32_t, v[i]));
    // (16 bytes: no scalar offset, see store_io_r)
    if constexpr (PP == 4) __builtin_amdgcn_raw_buffer_store_b128(i32x4{x[0], x[1], x[2], x[3]}, rs, voff + soff, 0, AUX);
    else if constexpr (PP == 2) __builtin_amdgcn_raw_buffer_store_b64(i32x2{x[0], x[1]}, rs, voff, soff, AUX);
    else __builtin_amdgcn_raw_buffer_store_b32(x[0], rs, voff, soff, AUX);
}
template <int PP> __device__ __forceinline__ void clear_part(rsrc_t rs, uint32_t voff, uint32_t soff) {
    constexpr int none = (int)kNoWord;
    if constexpr (PP == 4) __builtin_amdgcn_raw_buffer_store_b128(i32x4{none, none, none, none}, rs, voff + soff, 0, 0);
    else if constexpr (PP == 2) __builtin_amdgcn_raw_buffer_store_b64(i32x2{none, none}, rs, voff, soff, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(none, rs, voff, soff, 0);
}
// The lane index, formed anew: what a group's prologue and epilogue derive from it is not kept in registers through the time loop.
__device__ __forceinline__ int fresh_lane(int lane) {
    asm volatile("" : "+v"(lane));
    return lane;
}
constexpr uint32_t kTrash = 1024;   // bytes at the end of an exchange buffer: blocks that nobody waits for
constexpr int kAuxPoll = (int)(0x80000000u | (unsigned)kAuxAgent);   // (volatile: every round goes to memory again)
template <int PP> __device__ __forceinline__ void poll_part(rsrc_t rs, uint32_t voff, uint32_t soff, uint32_t (&v)[PP]) {
    if constexpr (PP == 4) {
        const i32x4 x = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, kAuxPoll);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (uint32_t)x[i];
    } else if constexpr (PP == 2) {
        const i32x2 x = __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, kAuxPoll);
        v[0] = (uint32_t)x[0]; v[1] = (uint32_t)x[1];
    } else {
        v[0] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, kAuxPoll);
    }
}
// One more look at the words failed: give up?  (spin limit, or another workgroup has given up)
__device__ __forceinline__ bool poll_gives_up(int spins, int spin_limit, int* err) {
    if (spins > spin_limit) {
        __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
    return (spins & 255) == 255 && __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// steps whose inputs are fetched in one burst: two bursts of up to 16 steps fit `room` bytes
constexpr int burst_steps(int slot, int room) { return room >= 32 * slot ? 16 : room >= 16 * slot ? 8 : room >= 8 * slot ? 4 : 2; }

// ---------------------------------------------------------------------------------------------
// Backward
// ---------------------------------------------------------------------------------------------
// UB blocks of 16 units per workgroup, NB output blocks of 16 units per compute wave.
// DIRECT (few members): compute wave w owns unit block w and forms, for every member of the group, the partial sums of that member's
// block w: the words it waits for are those of its own lanes, and the step has one barrier.  Otherwise the D / 16 output blocks are dealt out
// over eight compute waves, the arriving partial sums are added up by all of them (each thread one place of the segment and a fixed subset of the
// producers) and meet in LDS.
template <int CELL, int UB, int NB, int BT, bool DIRECT> struct SplitBwd {
    using CT = CellTraits<CELL>;
    static constexpr int G = CT::G, S = CT::S, NC = CT::NC;
    static constexpr bool SP = BT < 16;
    static constexpr int U = 16 * UB, K = G * U;
    static constexpr int NCW = DIRECT ? UB : 8, NLD = DIRECT ? 3 : 2, NST = DIRECT ? 1 : 2, NW = NCW + NLD + NST;
    static constexpr int NKS = (K + 63) / 64, KTD = (K + 31) / 32;     // steps of the sparse / dense matrix instruction
    static constexpr int HPB = ((SP ? NKS * 64 : KTD * 32) + operand_pad(true, SP)) * 2;   // bytes of an operand row
    static constexpr int NDG = DIRECT ? 2 : 1;                          // operand buffers
    static constexpr int PPV = BT / 4;                                  // floats per lane of a block
    static constexpr int SEG = UB * BT * 64;                            // bytes one member sends another per step
    static constexpr int NPT = UB * BT / 4, PT = DIRECT ? BT / 4 : (NPT + 7) / 8;   // tiles of 16 units x 4 rows: in all, per wave
    static constexpr int SEGC = SEG / 16, NSUB = 512 / SEGC < 8 ? 512 / SEGC : 8, NPC = (NB * 8 / UB + NSUB - 1) / NSUB;
    static constexpr int NBUF = DIRECT ? 4 : 2;
    // inputs of a step in chunks of 16 bytes, each stream rounded up to whole pieces of 64 chunks
    static constexpr int REC = CT::RS * 2, SB0 = cell_uses_h_prev(CELL) ? 0 : 1, NSB = CELL == CELL_SLSTM ? 2 : CELL == CELL_ELMAN ? 0 : 1;
    static constexpr int CR = BT * UB * REC, CS = NSB * BT * 4 * UB, CD = BT * 2 * UB;
    static constexpr int GR = (CR + 63) / 64, GS = (CS + 63) / 64, GD = (CD + 63) / 64, NLJ = (GR + GS + GD + NLD - 1) / NLD;
    static constexpr int SLOT = (GR + GS + GD) * 1024, KB = burst_steps(SLOT, 112 * 1024), RD = 2 * KB;   // steps per burst, slots
    static constexpr int GO = CELL == CELL_GRU ? G + 1 : G, COUT = BT * GO * 2 * UB, NSJ = (COUT + NST * 64 - 1) / (NST * 64);
    static constexpr int DG_BYTES = BT * HPB, IMG_BYTES = CELL == CELL_GRU ? BT * U * 2 : 0;
    static constexpr int IMG_OFF = NDG * DG_BYTES, RING_OFF = (IMG_OFF + NDG * IMG_BYTES + 127) / 128 * 128;
    static constexpr int RED_OFF = RING_OFF + RD * SLOT, SMEM = RED_OFF + (DIRECT ? 0 : NSUB * SEG);
    static constexpr int kCell = CELL, kUB = UB, kBT = BT, kBarriers = DIRECT ? 1 : 2;   // barriers per step
    static __device__ __forceinline__ uint32_t unit0(const KernelParams&, uint32_t member) { return member * U; }   // first unit of a member
};

// position of (row, unit block ub) in an input row of the ring: the blocks of row r are stored r places on, modulo UB, so that the
// rows that one instruction reads lie in different banks
template <int UB> __device__ __forceinline__ uint32_t ring_block(uint32_t ub, uint32_t row) { return (ub + row) % UB; }

// The inputs of a group's steps, by C::NLD waves (wl = 0 ..): piece by piece of 64 chunks of 16 bytes into the ring.
template <class C> struct BwdLoader {
    uint32_t voff[C::NLJ];   // this lane's chunk of piece j of the wave
    __device__ __forceinline__ BwdLoader(const KernelParams& p, uint32_t n, uint32_t q, uint32_t e0, int lane, int wl) {
        constexpr int UB = C::kUB, BT = C::kBT;
        const uint32_t B = p.B, D = p.D, HD = p.NH * D;
#pragma unroll
        for (int j = 0; j < C::NLJ; ++j) {
            const int piece = j * C::NLD + wl;
            voff[j] = 0x80000000u;
            auto place = [&](uint32_t idx, uint32_t rows, uint32_t cpb, uint32_t esz, uint32_t plane) {   // rows of UB blocks of cpb chunks
                const uint32_t cpr = UB * cpb, r = idx / cpr, pos = idx % cpr, row = r % BT;
                const uint32_t blk = (pos / cpb + UB * BT - row) % UB, brow = q * BT + row;
                if (r < rows && brow < B) voff[j] = (r / BT) * plane + (brow * HD + n * D + e0 + blk * 16) * esz + (pos % cpb) * 16;
            };
            if (piece < C::GR) place(piece * 64 + lane, BT, C::REC, C::REC, 0);
            else if (piece < C::GR + C::GS) place((piece - C::GR) * 64 + lane, C::NSB * BT, 4, 4, B * HD * 4);
            else if (piece < C::GR + C::GS + C::GD) place((piece - C::GR - C::GS) * 64 + lane, BT, 2, 2, 0);
        }
    }
    // inputs of the steps s0 .. s0 + KB - 1 (counted from the last one)
    __device__ __forceinline__ void burst(const KernelParams& p, char* smem, int wl, int s0) const {
        const size_t units = (size_t)p.B * p.NH * p.D;
#pragma unroll 1
        for (int s = s0; s < s0 + C::KB && s < p.T; ++s) {
            const size_t t = p.T - 1 - s;
            const rsrc_t rc = make_rsrc((const char*)p.cache + t * (units * C::REC));
            const rsrc_t rst = make_rsrc((const char*)p.states + (t * C::S + C::SB0) * (units * 4));
            const rsrc_t rdh = make_rsrc((const char*)p.dH + t * (units * 2));
            char* to = smem + C::RING_OFF + s % C::RD * C::SLOT + wl * 1024;
#pragma unroll
            for (int j = 0; j < C::NLJ; ++j) {
                const int piece = j * C::NLD + wl;
                if (piece < C::GR + C::GS + C::GD) load_chunk_to_lds(piece < C::GR ? rc : piece < C::GR + C::GS ? rst : rdh, to + j * C::NLD * 1024, voff[j]);
            }
        }
    }
};
// The outputs of a step, by C::NST waves (ws = 0 ..), from the rows of gate gradients in LDS.
template <class C> struct BwdStorer {
    uint32_t voff[C::NSJ], vofn[C::NSJ], loff[C::NSJ];
    bool img[C::NSJ];
    __device__ __forceinline__ BwdStorer(const KernelParams& p, uint32_t n, uint32_t q, uint32_t e0, int lane, int ws) {
        constexpr int CELL = C::kCell, UB = C::kUB, BT = C::kBT;
        constexpr uint32_t kDrop = 0x80000000u;
        const uint32_t B = p.B, D = p.D, HD = p.NH * D;
#pragma unroll
        for (int j = 0; j < C::NSJ; ++j) {
            const uint32_t idx = (j * C::NST + ws) * 64 + lane, cpr = 2 * UB, r = idx / cpr, ch = idx % cpr, g = r % C::GO, row = r / C::GO, brow = q * BT + row;
            const bool in = row < BT && brow < B;
            // (the rows of the matrix operand are dWx_t, but for the GRU's candidate: its input-side gradient has an image of its own, and
            // what the operand holds goes to the buffer of recurrent-side gradients)
            voff[j] = in && g < (uint32_t)C::G ? ((brow * C::G + g) * HD + n * D + e0) * 2 + ch * 16 : kDrop;
            vofn[j] = in && g == (uint32_t)C::G ? (brow * HD + n * D + e0) * 2 + ch * 16 : kDrop;
            img[j] = CELL == CELL_GRU && g == 2;
            loff[j] = row >= BT ? 0u : img[j] ? C::IMG_OFF + row * C::U * 2 + ch * 16 : row * C::HPB + (g == (uint32_t)C::G ? 2u : g) * C::U * 2 + ch * 16;
        }
    }
    // step s (counted from the last one), from operand buffer buf
    __device__ __forceinline__ void store(const KernelParams& p, const char* smem, int s, uint32_t buf) const {
        const size_t units = (size_t)p.B * p.NH * p.D, t = p.T - 1 - s;
        const rsrc_t dwx = make_rsrc((char*)p.dWx + t * (units * (C::G * 2)));
        i32x4 v[C::NSJ];
#pragma unroll
        for (int j = 0; j < C::NSJ; ++j) v[j] = *(const i32x4*)(smem + loff[j] + buf * (C::kCell == CELL_GRU && img[j] ? C::IMG_BYTES : C::DG_BYTES));
#pragma unroll
        for (int j = 0; j < C::NSJ; ++j) {
            __builtin_amdgcn_raw_buffer_store_b128(v[j], dwx, voff[j], 0, 0);
            if constexpr (C::kCell == CELL_GRU) __builtin_amdgcn_raw_buffer_store_b128(v[j], make_rsrc((char*)p.dgn + t * (units * 2)), vofn[j], 0, 0);
        }
    }
};

template <class C>
__device__ __forceinline__ void split_bwd_load(const KernelParams& p, const BlockMap& bm, char* smem, int lane, int wl) {
    for (int gid = bm.gpar; gid < p.NG; gid += p.GPAR) {
        const BwdLoader<C> in(p, gid % p.NH, gid / p.NH, C::unit0(p, bm.member), lane, wl);
        in.burst(p, smem, wl, 0);
        wait_vmem<0>();
        wg_barrier();
        in.burst(p, smem, wl, C::KB);
        for (int s = 0; s < p.T; ++s) {
            // step s + 1 begins a burst: it must be there, and the slots of the burst before are free behind the barrier
            const bool next = (s + 1) % C::KB == 0;
            if (next) wait_vmem<0>();
            wg_barrier();
            if (next) in.burst(p, smem, wl, s + 1 + C::KB);
            if constexpr (C::kBarriers == 2) wg_barrier();
        }
        wait_vmem<0>();
    }
}

template <class C>
__device__ __forceinline__ void split_bwd_store(const KernelParams& p, const BlockMap& bm, char* smem, int lane, int ws) {
    for (int gid = bm.gpar; gid < p.NG; gid += p.GPAR) {
        const BwdStorer<C> out(p, gid % p.NH, gid / p.NH, C::unit0(p, bm.member), lane, ws);
        wg_barrier();
        for (int s = 0; s < p.T; ++s) {
            wg_barrier();
            out.store(p, smem, s, C::NDG == 2 ? (uint32_t)(s & 1) : 0u);
            if constexpr (C::kBarriers == 2) wg_barrier();
        }
    }
}

template <int CELL, int UB, int NB, int BT, bool DIRECT>
__device__ __forceinline__ void split_bwd_compute(const KernelParams& p, const BlockMap& bm, char* smem, int lane, int w) {
    using C = SplitBwd<CELL, UB, NB, BT, DIRECT>;
    using PG = PointGrad<CELL>;
    constexpr int G = C::G, S = C::S, NC = C::NC, PT = C::PT, PPV = C::PPV, U = C::U;
    constexpr bool SP = C::SP;
    constexpr uint32_t kDrop = 0x80000000u;
    const int T = p.T, P = p.P, me = bm.member;
    const uint32_t B = p.B, NH = p.NH, D = p.D, HD = NH * D, m = D / 16;
    const SparseLane<BT == 8 ? 8 : 4> sl(lane);
    const uint32_t c = sl.c, quad = sl.quad;
    const rsrc_t xr = make_rsrc(p.exch);
    const uint32_t xbuf = (uint32_t)p.GPAR * P * P * C::SEG + kTrash, xgroup = (uint32_t)bm.gpar * P * P * C::SEG;
    char* ring = smem + C::RING_OFF;
    char* red = smem + C::RED_OFF;
    bool failed = false;
    FRNN_TRACE_BEGIN();

    // ---- this lane's (unit, row) pairs: tile k covers 16 units x 4 rows.  Via LDS, rows are dealt out so that the lanes of a tile read
    // their words of a block (PPV consecutive floats per lane) from different banks.
    const bool pairs = DIRECT || w < C::NPT;
    uint32_t ub[PT], word[PT], row[PT];
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        const int id = DIRECT ? w * (BT / 4) + k : (pairs ? w : 0) + 8 * k, rr = id % (BT / 4);
        ub[k] = id / (BT / 4);
        word[k] = DIRECT || BT == 4 ? rr : BT == 8 ? (rr + (quad >> 1)) & 1 : (rr + quad) & 3;
        row[k] = BT == 16 ? 4 * quad + word[k] : quad + 4 * word[k];
    }
    // ---- the output blocks of this wave (b = 0 is its own block if DIRECT) and where their partial sums go: segment [receiver][sender], UB blocks.
    // (A wave without a last block forms one all the same and leaves it at the end of the buffer, where nobody looks: no condition in the step.)
    uint32_t out_off[NB], out_blk[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const uint32_t idx = b * 8 + w;
        const bool none = !DIRECT && idx >= m;
        out_blk[b] = DIRECT ? ((uint32_t)(me + b) % NB) * UB + w : none ? 0 : ((uint32_t)me * UB + UB + idx) % m;
        out_off[b] = none ? xbuf - kTrash : xgroup + ((out_blk[b] / UB) * P + me) * C::SEG + (out_blk[b] % UB) * (64 * BT);
    }
    // ---- what this thread waits for.  DIRECT: the words of its own lane from every other member.  Else the 16 bytes at `pos` of the segments
    // of nv senders from sub * npc on: the waves add up what arrives, each thread a fixed run of senders.
    constexpr int NIN = DIRECT ? NB - 1 : C::NPC, IW = DIRECT ? PPV : 4;
    const uint32_t xmine = xgroup + (uint32_t)me * P * C::SEG;
    const uint32_t pos = (uint32_t)(w * 64 + lane) % C::SEGC, sub = (uint32_t)(w * 64 + lane) / C::SEGC;
    const int npc = (P + C::NSUB - 1) / C::NSUB;
    int nv = sub < C::NSUB ? P - (int)sub * npc : 0;
    nv = nv > npc ? npc : nv;
    const uint32_t in_lane = DIRECT ? (uint32_t)(lane * BT) : sub * npc * C::SEG + pos * 16;
    uint32_t in_off[NIN > 0 ? NIN : 1];
#pragma unroll
    for (int j = 0; j < NIN; ++j) in_off[j] = xmine + (DIRECT ? ((uint32_t)(me + NB - 1 - j) % NB) * C::SEG + w * (64 * BT) : j * C::SEG);
    // (the lane offset of sender j, formed anew where it is used: kept from step to step they would take a register each)
    auto in_voff = [&](int j) {
        if constexpr (DIRECT) return in_lane;
        else {
            asm volatile("" : "+v"(nv));
            return j < nv ? in_lane : kDrop;
        }
    };

    for (uint32_t j = w * 64 + lane; j < (uint32_t)(C::NDG * C::DG_BYTES) / 4; j += C::NCW * 64) ((uint32_t*)smem)[j] = 0u;   // (padding of the operand rows)

    int iter = 0;
    for (int gid = bm.gpar; gid < p.NG; gid += p.GPAR, ++iter) {
        const uint32_t n = gid % NH, q = gid / NH, e0 = me * U;
        const uint32_t pl = fresh_lane(lane), pc = pl & 15, pquad = pl >> 4;
        // ---- R: column c = unit of the output block, contraction over this workgroup's gate gradients k = g * U + u, in registers for all steps
        bf16x16 Rs[SP ? NB : 1][SP ? C::NKS : 1];
        bf16x8 Rd[SP ? 1 : NB][SP ? 1 : C::KTD];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint16_t* rrow = (const uint16_t*)p.R + ((size_t)n * D + out_blk[b] * 16 + pc) * G * D + e0;
            auto quads = [&](uint32_t kk) {   // four elements of R from k = kk on (zeros beyond the last gate)
                if constexpr (C::K % (SP ? 64 : 32) == 0) {
                    return *(const i32x2*)(rrow + (kk / U) * D + kk % U);
                } else {
                    const bool in = kk < (uint32_t)C::K;
                    const i32x2 v = *(const i32x2*)(rrow + (in ? (kk / U) * D + kk % U : 0));
                    return in ? v : i32x2{0, 0};
                }
            };
            if constexpr (SP) {
#pragma unroll
                for (int kc = 0; kc < C::NKS; ++kc) {
                    i32x4 piece[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t kk = (2 * kc + h) * 32 + sparse_k(pquad);
                        piece[h] = sparse_piece(quads(kk), quads(kk + 8));
                    }
                    Rs[b][kc] = sparse_dense(piece[0], piece[1]);
                }
            } else {
#pragma unroll
                for (int kt = 0; kt < C::KTD; ++kt) {
                    const uint32_t kk = kt * 32 + pquad * 8;
                    const i32x2 lo = quads(kk), hi = quads(kk + 4);
                    Rd[b][kt] = __builtin_bit_cast(bf16x8, i32x4{lo[0], lo[1], hi[0], hi[1]});
                }
            }
        }
        // ---- pairs: places, carried gradients, states after the last step
        uint32_t l_rec[PT], l_st[PT], l_dh[PT], l_dg[PT];
        // this lane's batch row of tile k, and the place of its value in a plane of states
        auto batch_row = [&](int k, uint32_t ln) {
            const uint32_t qd = ln >> 4, rr = (DIRECT ? w * (BT / 4) + k : (pairs ? w : 0) + 8 * k) % (BT / 4);
            const uint32_t wd = DIRECT || BT == 4 ? rr : BT == 8 ? (rr + (qd >> 1)) & 1 : (rr + qd) & 3;
            return q * BT + (BT == 16 ? 4 * qd + wd : qd + 4 * wd);
        };
        auto state_at = [&](int k, uint32_t ln) {
            const uint32_t brow = batch_row(k, ln);
            return ((brow < B ? brow : B - 1) * HD + n * D + e0 + ub[k] * 16 + (ln & 15)) * 4;
        };
        float ds[PT][S], sc[PT][S], sp[PT][S], kf[PT][PG::NK], dh_ext[PT], dbacc[PT][G];
        const size_t st_step = (size_t)S * B * HD * 4;
        const uint32_t st_state = B * HD * 4;
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const uint32_t g_st = state_at(k, pl);
            const uint32_t rb = row[k] * UB + ring_block<UB>(ub[k], row[k]);
            l_rec[k] = (rb * 16 + c) * C::REC;
            l_st[k] = C::GR * 1024 + (rb * 16 + c) * 4;
            l_dh[k] = (C::GR + C::GS) * 1024 + (rb * 16 + c) * 2;
            l_dg[k] = row[k] * C::HPB + (ub[k] * 16 + c) * 2;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                float v[1] = {0.0f};
                if (p.dlast != nullptr && !(CELL == CELL_SLSTM && s == 3)) load_io_r<false, 1>(make_rsrc(p.dlast), g_st, s * st_state, v);
                ds[k][s] = v[0];
                sp[k][s] = 1.0f;
                float x[1] = {1.0f};
                if (!cell_uses_h_prev(CELL) && s >= C::SB0 && s < C::SB0 + C::NSB) load_io_r<false, 1>(make_rsrc((const char*)p.states + (size_t)T * st_step), g_st, s * st_state, x);
                sc[k][s] = x[0];
            }
#pragma unroll
            for (int g = 0; g < G; ++g) dbacc[k][g] = 0.0f;
        }
        auto take = [&](uint32_t slot) {   // this lane's inputs of a step, and what follows from them alone
            const char* in = ring + slot * C::SLOT;
#pragma unroll
            for (int k = 0; k < PT; ++k) {
                float cv[NC];
                take_record_lds<C::CT::RS, NC>(in + l_rec[k], cv);
#pragma unroll
                for (int s = C::SB0; s < C::SB0 + C::NSB; ++s) sp[k][s] = *(const float*)(in + l_st[k] + (s - C::SB0) * BT * U * 4);
                dh_ext[k] = bf16_bits_to_f32(*(const uint16_t*)(in + l_dh[k]));
                PG::factors(cv, sc[k], sp[k], kf[k]);
                if constexpr (!cell_uses_h_prev(CELL)) {
#pragma unroll
                    for (int s = C::SB0; s < C::SB0 + C::NSB; ++s) sc[k][s] = sp[k][s];
                }
            }
        };
        wg_barrier();   // the first inputs are there, the operand rows are zero
        if (T > 0 && pairs) take(0);
        // (what the prologue has loaded is complete here: the waits of the time loop are for its own operations only)
        pin(ds);
        pin(sc);
        pin(kf);
        pin(dh_ext);

        FRNN_TRACE_RESET();
        uint32_t slot = 0;
        for (int s = 0; s < T; ++s) {
            const uint32_t cnt = (uint32_t)iter * (uint32_t)T + (uint32_t)s;
            const uint32_t buf = cnt % C::NBUF * xbuf;
            char* dg_rows = smem + (C::NDG == 2 ? (s & 1) * C::DG_BYTES : 0);
            // ---- gate gradients of the step into the operand rows
            if (pairs) {
#pragma unroll
                for (int k = 0; k < PT; ++k) {
                    float dwx[G], dg[G];
                    ds[k][0] += dh_ext[k];
                    PG::apply(kf[k], ds[k], dwx, dg);
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        *(uint16_t*)(dg_rows + l_dg[k] + g * U * 2) = (uint16_t)f32_to_bf16_bits(dg[g]);
                        dbacc[k][g] += dg[g];
                    }
                    if constexpr (CELL == CELL_GRU)
                        *(uint16_t*)(smem + C::IMG_OFF + (C::NDG == 2 ? (s & 1) * C::IMG_BYTES : 0) + row[k] * U * 2 + (ub[k] * 16 + c) * 2) = (uint16_t)f32_to_bf16_bits(dwx[2]);
                }
            }
            // (DIRECT: the accumulators are cleared ahead of the barrier, where the wave waits for its LDS writes anyway)
            constexpr int CH = DIRECT ? (NB % 2 == 0 ? NB / 2 : 2) : 2;
            f32x4 a[CH];
#pragma unroll
            for (int x = 0; x < CH; ++x) {
                a[x] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (DIRECT) asm volatile("" : "+v"(a[x]));
            }
            // (two exchange buffers: the words taken back behind the last poll must be gone before anything of this step is published)
            if constexpr (!DIRECT) wait_vmem<0>();
            FRNN_TRACE_MARK(0);
            wg_barrier();
            FRNN_TRACE_MARK(1);
            // ---- partial sums of dh_{t-1}: this workgroup's gate gradients times their columns of R
            bf16x8 gS[SP ? C::NKS : C::KTD];
            if constexpr (SP) {
                lds_sparse_chunk<BT, C::NKS, C::NKS, false, true>(dg_rows + sl.rslot * C::HPB, sl, 0, gS);
            } else {
#pragma unroll
                for (int kt = 0; kt < C::KTD; ++kt) gS[kt] = *(const bf16x8*)(dg_rows + c * C::HPB + kt * 64 + quad * 16);
            }
            // (CH blocks at a time: the matrix instructions of one block depend on each other)
            float own[PPV];
#pragma unroll
            for (int bi = 0; bi < NB; bi += CH) {
                if (bi > 0) {
#pragma unroll
                    for (int x = 0; x < CH; ++x) a[x] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int kc = 0; kc < (SP ? C::NKS : C::KTD); ++kc)
#pragma unroll
                    for (int x = 0; x < CH; ++x)
                        if (bi + x < NB) {
                            const int b = DIRECT ? (bi + x + 1) % NB : bi + x;
                            if constexpr (SP) a[x] = smfmac(gS[kc], Rs[b][kc], a[x], sl.idx);
                            else a[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gS[kc], Rd[b][kc], a[x], 0, 0, 0);
                        }
#pragma unroll
                for (int x = 0; x < CH; ++x)
                    if (bi + x < NB) {
                        const int b = DIRECT ? (bi + x + 1) % NB : bi + x;
                        float v[PPV];
#pragma unroll
                        for (int i = 0; i < PPV; ++i) v[i] = SP ? a[x][(2 * i) & 3] + a[x][(2 * i + 1) & 3] : a[x][i];
                        asm volatile("" : : "v"(a[x]));   // (4-row tiles: nobody gets the two unused registers of an accumulator before the sums are formed)
                        if (DIRECT && b == 0) {
#pragma unroll
                            for (int i = 0; i < PPV; ++i) own[i] = v[i];
                        } else {
                            store_part<PPV>(xr, lane * BT, buf + out_off[b], v);
                        }
                    }
            }
            FRNN_TRACE_MARK(4);
            // ---- the inputs of the next step, while the partial sums travel
            slot = slot + 1 == (uint32_t)C::RD ? 0 : slot + 1;
            if (pairs) take(slot);
            pin(kf);   // (here, not behind the poll)
            pin(dh_ext);
            FRNN_TRACE_MARK(6);
            // ---- the partial sums of this workgroup's units from the other members
            uint32_t got[NIN > 0 ? NIN : 1][IW];
            if (p.spin_limit < 0 && !failed) {   // host-forced failure (tests of the error path): give up without looking
                __hip_atomic_store(p.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                failed = true;
            }
            f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (DIRECT) {
                for (int spins = 0;; ++spins) {
#pragma unroll
                    for (int j = 0; j < NIN; ++j) poll_part<IW>(xr, in_voff(j), buf + in_off[j], got[j]);
                    uint32_t top = 0u;   // (a word out of range reads as zero)
#pragma unroll
                    for (int j = 0; j < NIN; ++j)
#pragma unroll
                        for (int i = 0; i < IW; ++i) top = max(top, got[j][i]);
                    if (__all((int)(top != kNoWord)) || failed) break;
                    if (poll_gives_up(spins, p.spin_limit, p.err)) { failed = true; break; }
                }
            } else {
                // Many senders: one after the other, and those that are there are not looked at again.  (A group's members read all of its partial sums with every look, and what the polls take of the
                // L2's bandwidth the stores of the partial sums wait for: LSTM 1 x 768 backward, 512 steps with 16 rows 727 us against 867 with all senders looked at every time, 256 steps with 64 / 128 rows 524 / 877 and 574 / 1013.
                // Where a wave waits for three to five senders' words of its own lanes, above, all of them at a time are 4 to 7 % faster.)
                // (A member sends its blocks from the next member's on, so the words of the member in front are the first to arrive: downwards, but for 16 rows -- 128 rows 922 us downwards.)
                constexpr bool kDown = BT < 16;
                auto sender = [&](auto j_c) {
                    constexpr int x = decltype(j_c)::value, j0 = kDown ? NIN - 1 - x : x, first = kDown ? 0 : j0, end = kDown ? j0 + 1 : NIN;
                    if constexpr (x < NIN) {
                        for (int spins = 0;; ++spins) {
                            if (x == 0 || spins > 0) {
#pragma unroll
                                for (int j = first; j < end; ++j) poll_part<IW>(xr, in_voff(j), buf + in_off[j], got[j]);
                            }
                            uint32_t top = 0u;   // (a word out of range reads as zero)
#pragma unroll
                            for (int i = 0; i < IW; ++i) top = max(top, got[j0][i]);
                            if (__all((int)(top != kNoWord)) || failed) break;
                            if (poll_gives_up(spins, p.spin_limit, p.err)) { failed = true; break; }
                        }
                    }
                };
                sender(std::integral_constant<int, 0>{});
                sender(std::integral_constant<int, 1>{});
                sender(std::integral_constant<int, 2>{});
                sender(std::integral_constant<int, 3>{});
                sender(std::integral_constant<int, 4>{});
                sender(std::integral_constant<int, 5>{});
                sender(std::integral_constant<int, 6>{});
                sender(std::integral_constant<int, 7>{});
                static_assert(NIN <= 8);
#pragma unroll
                for (int j = 0; j < NIN; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[i] += __builtin_bit_cast(float, got[j][i]);
            }
            // (taken back for the round NBUF later: this workgroup is the only one that looks at these words)
#pragma unroll
            for (int j = 0; j < NIN; ++j) clear_part<IW>(xr, in_voff(j), buf + in_off[j]);
            FRNN_TRACE_MARK(2);
            if constexpr (DIRECT) {
#pragma unroll
                for (int k = 0; k < PT; ++k) {
                    float rec = own[k];
#pragma unroll
                    for (int j = 0; j < NIN; ++j) rec += __builtin_bit_cast(float, got[j][k]);
                    ds[k][0] += fminf(fmaxf(rec, -p.clip), p.clip);   // (Sec. 4.1 clip; +inf = off)
                }
            } else {
                if (sub < C::NSUB) *(f32x4*)(red + sub * C::SEG + pos * 16) = sum;
                wg_barrier();
                FRNN_TRACE_MARK(3);
                if (pairs) {
#pragma unroll
                    for (int k = 0; k < PT; ++k) {
                        const float* r0 = (const float*)(red + ub[k] * (64 * BT)) + lane * PPV + word[k];
                        float part[C::NSUB];
#pragma unroll
                        for (int j = 0; j < C::NSUB; ++j) part[j] = r0[j * (C::SEG / 4)];
                        float rec = part[0];
#pragma unroll
                        for (int j = 1; j < C::NSUB; ++j) rec += part[j];
                        ds[k][0] += fminf(fmaxf(rec, -p.clip), p.clip);
                    }
                }
            }
        }
        // ---- gradients of the initial states, per-row partial sums of db
        const uint32_t el = fresh_lane(lane);
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const uint32_t brow = batch_row(k, el);
            if (pairs && brow < B) {
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const float v[1] = {ds[k][s]};
                    store_io_r<false, 1>(make_rsrc(p.dstates0), state_at(k, el), s * st_state, v);
                }
                float* db = p.db_part + (((size_t)brow * NH + n) * G) * D + e0 + ub[k] * 16 + (el & 15);
#pragma unroll
                for (int g = 0; g < G; ++g) db[(size_t)g * D] = dbacc[k][g] + (p.db_accumulate ? db[(size_t)g * D] : 0.0f);
            }
        }
    }
    FRNN_TRACE_END(p);
}

template <int CELL, int UB, int NB, int BT, bool DIRECT>
__global__ __launch_bounds__((SplitBwd<CELL, UB, NB, BT, DIRECT>::NW * 64)) void split_bwd_kernel(const KernelParams p) {
    using C = SplitBwd<CELL, UB, NB, BT, DIRECT>;
    extern __shared__ __align__(16) char smem[];
    const BlockMap bm(p, true);
    if (!bm.active) return;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w < C::NCW) split_bwd_compute<CELL, UB, NB, BT, DIRECT>(p, bm, smem, lane, w);
    else if (w < C::NCW + C::NLD) split_bwd_load<C>(p, bm, smem, lane, w - C::NCW);
    else split_bwd_store<C>(p, bm, smem, lane, w - C::NCW - C::NLD);
}

// ---------------------------------------------------------------------------------------------
// Backward in two hand-overs: many members
// ---------------------------------------------------------------------------------------------
// With P members each partial sum of every unit has to reach its owner from all of them: 4 D bytes per row out of and into every CU, most of a
// step's time with 16 rows or hundreds of CUs.  Here the members form a mesh of PB = 8 / UB subgroups (s = member % PB) of PA = P / PB members
// (a = member / PB).  A subgroup's members gather each other's gate gradients (bf16 rows of G * U * PA elements) and each forms the partial sums of eight of the
// D / 16 output blocks, those owned by the members with its own a in all subgroups: PB segments of UB blocks, added up by their owners.
// A head spread over the chip has one subgroup per XCD (UB = 1): gate gradients stay inside an XCD's L2, only partial sums of eight blocks
// per member cross the XCDs.
// NCW = 8 compute waves share the subgroup's contraction like those of split_fwd_kernel (wave w polls its KTW k-steps straight into operand registers);
// their sums meet in LDS, where wave w takes up block w.  Kernels that hold 128 registers of R per lane have no waves beside them (OWN_IO): the four
// waves without point-wise work, at least, move inputs and outputs.
// (LSTM 1 x 2048, 16 rows, per step 7.68 -> 2.70 us against the exchange of gate gradients through memory, 1 x 1024 with 16 / 64 / 128 rows 2.61 / 4.81 / 10.4
// -> 1.69 / 2.07 / 4.10.  Bound by the two hand-overs: 22 % and 39 % of a step of 1 x 2048, matrix product and the waves' sums a quarter.)
template <int CELL, int UB, int KTW, int BT> struct MeshBwd {
    static constexpr bool OWN_IO = KTW >= 4;
    using CT = CellTraits<CELL>;
    static constexpr int G = CT::G, S = CT::S, NC = CT::NC;
    static constexpr bool SP = BT < 16;
    static constexpr int U = 16 * UB, GU = G * U, PB = 8 / UB, NBUF = 4;
    static constexpr int NCW = 8, NLD = OWN_IO ? 4 : 2, NST = NLD, NW = OWN_IO ? NCW : NCW + NLD + NST, OB = 8;
    static constexpr int DK = NCW * KTW * 32, XROW = DK * 2;           // exchanged rows of gate gradients
    static constexpr int NKF = KTW / 2, HALF = KTW & 1;
    static constexpr int PPV = BT / 4, SEG = UB * BT * 64;             // floats per lane of a block; bytes one member sends another
    static constexpr int NPT = UB * BT / 4;                            // tiles of 16 units x 4 rows, one per wave
    static_assert(NPT <= NCW);
    static constexpr int REC = CT::RS * 2, SB0 = cell_uses_h_prev(CELL) ? 0 : 1, NSB = CELL == CELL_SLSTM ? 2 : CELL == CELL_ELMAN ? 0 : 1;
    static constexpr int CR = BT * UB * REC, CS = NSB * BT * 4 * UB, CD = BT * 2 * UB;
    static constexpr int GR = (CR + 63) / 64, GS = (CS + 63) / 64, GD = (CD + 63) / 64, NLJ = (GR + GS + GD + NLD - 1) / NLD;
    static constexpr int SLOT = (GR + GS + GD) * 1024;
    static constexpr int GO = CELL == CELL_GRU ? G + 1 : G, COUT = BT * GO * 2 * UB, NSJ = (COUT + NST * 64 - 1) / (NST * 64);
    static constexpr int NDG = 2, HPB = (GU + 16) * 2, DG_BYTES = BT * HPB, IMG_BYTES = CELL == CELL_GRU ? BT * U * 2 : 0;   // dWx on its way out
    static constexpr int IMG_OFF = NDG * DG_BYTES, RING_OFF = (IMG_OFF + NDG * IMG_BYTES + 127) / 128 * 128;
    static constexpr int RED = NCW * OB * 64 * PPV * 4;                // the waves' sums; two buffers, or one and a second barrier per step
    static constexpr int ROOM = 160 * 1024 - RING_OFF, NRED = 2 * RED + 8 * SLOT <= ROOM ? 2 : 1, kBarriers = NRED == 2 ? 1 : 2;
    static constexpr int KB = burst_steps(SLOT, ROOM - NRED * RED < 96 * 1024 ? ROOM - NRED * RED : 96 * 1024), RD = 2 * KB;
    static constexpr int RED_OFF = RING_OFF + RD * SLOT, SMEM = RED_OFF + NRED * RED;
    static constexpr int kCell = CELL, kUB = UB, kBT = BT;
    // the units of a subgroup are consecutive
    static __device__ __forceinline__ uint32_t unit0(const KernelParams& p, uint32_t member) { return ((member % PB) * (p.P / PB) + member / PB) * U; }
    static constexpr size_t exch_bytes(int groups, int P) { return (size_t)NBUF * groups * ((size_t)PB * BT * XROW + (size_t)P * PB * SEG); }
};

template <int CELL, int UB, int KTW, int BT>
__device__ __forceinline__ void mesh_bwd_compute(const KernelParams& p, const BlockMap& bm, char* smem, int lane, int w) {
    using C = MeshBwd<CELL, UB, KTW, BT>;
    using PG = PointGrad<CELL>;
    constexpr int G = C::G, S = C::S, NC = C::NC, PPV = C::PPV, U = C::U, GU = C::GU, PB = C::PB, NKF = C::NKF, HALF = C::HALF;
    constexpr bool SP = C::SP;
    constexpr uint32_t kDrop = 0x80000000u;
    const int T = p.T;
    const uint32_t B = p.B, NH = p.NH, D = p.D, HD = NH * D, PA = p.P / PB, a_me = bm.member / PB, s_me = bm.member % PB, e0 = C::unit0(p, bm.member);
    const uint32_t K2 = GU * PA, k0 = w * KTW * 32;
    const SparseLane<BT == 8 ? 8 : 4> sl(lane);
    const rsrc_t xr = make_rsrc(p.exch);
    // exchange buffers: [round & 3] of the subgroups' rows of gate gradients, then [round & 3] of the segments [receiver][sending subgroup]
    const uint32_t xbuf1 = (uint32_t)p.GPAR * PB * BT * C::XROW, xgroup1 = ((uint32_t)bm.gpar * PB + s_me) * BT * C::XROW;
    const uint32_t xbuf2 = (uint32_t)p.GPAR * p.P * PB * C::SEG, xgroup2 = C::NBUF * xbuf1 + (uint32_t)bm.gpar * p.P * PB * C::SEG;
    char* ring = smem + C::RING_OFF;
    bool failed = false;
    FRNN_TRACE_BEGIN();

    // ---- this lane's (unit, row) pair, if the wave has a tile
    const bool pairs = w < C::NPT;
    const uint32_t ub = pairs ? w / (BT / 4) : 0, rr = pairs ? w % (BT / 4) : 0;
    auto row_of = [&](uint32_t ln) { return BT == 16 ? 4 * (ln >> 4) + rr : (ln >> 4) + 4 * rr; };
    const uint32_t row = row_of(lane), c = lane & 15;
    const uint32_t x1lane = (c & 3) == 0 ? row * C::XROW + (a_me * GU + ub * 16 + c) * 2 : kDrop;   // (the lanes of every fourth unit publish it and the three behind it)
    const uint32_t rb = row * UB + ring_block<UB>(ub, row);
    const uint32_t l_rec = (rb * 16 + c) * C::REC, l_st = C::GR * 1024 + (rb * 16 + c) * 4, l_dh = (C::GR + C::GS) * 1024 + (rb * 16 + c) * 2;
    const uint32_t l_dg = row * C::HPB + (ub * 16 + c) * 2;
    // ---- this lane's operand pieces of the subgroup's rows (as in split_fwd_kernel)
    constexpr int NPC = SP ? NKF + HALF : KTW;
    const uint32_t xrow = (SP ? sl.rslot : c) * C::XROW + k0 * 2 + (SP ? sl.rbyte : sl.quad * 16);
    const bool reads = !(BT == 4 && (c & 2));
    uint32_t k_lane = reads ? k0 + (SP ? sl.rbyte / 2 : sl.quad * 8) : K2;
    auto piece_voff = [&](int j) {
        asm volatile("" : "+v"(k_lane));
        return k_lane + j * (SP ? 64 : 32) < K2 ? xrow + j * (SP ? 128 : 64) : kDrop;
    };
    uint32_t half_off = kDrop;
    if (SP && HALF && reads && k0 + NKF * 64 + sl.rbyte32 / 2 < K2) half_off = sl.rslot * C::XROW + (k0 + NKF * 64) * 2 + sl.rbyte32;
    // ---- block w goes to the member with this a in subgroup w / UB; the words of this wave's tile come from all subgroups
    const uint32_t x2out = xgroup2 + ((a_me * PB + w / UB) * PB + s_me) * C::SEG + (w % UB) * (64 * BT);
    const uint32_t x2in = xgroup2 + (uint32_t)bm.member * PB * C::SEG + ub * (64 * BT) + rr * 4;

    int iter = 0;
    for (int gid = bm.gpar; gid < p.NG; gid += p.GPAR, ++iter) {
        const uint32_t n = gid % NH, q = gid / NH;
        const uint32_t pl = fresh_lane(lane), pc = pl & 15, pquad = pl >> 4;
        const size_t st_step = (size_t)S * B * HD * 4;
        const uint32_t st_state = B * HD * 4;
        auto state_at = [&](uint32_t ln) {
            const uint32_t brow = q * BT + row_of(ln);
            return ((brow < B ? brow : B - 1) * HD + n * D + e0 + ub * 16 + (ln & 15)) * 4;
        };
        float ds[S], sc[S], sp[S], kf[PG::NK], dh_ext = 0.0f, dbacc[G];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            float v[1] = {0.0f}, x[1] = {1.0f};
            if (p.dlast != nullptr && !(CELL == CELL_SLSTM && s == 3)) load_io_r<false, 1>(make_rsrc(p.dlast), state_at(pl), s * st_state, v);
            if (!cell_uses_h_prev(CELL) && s >= C::SB0 && s < C::SB0 + C::NSB) load_io_r<false, 1>(make_rsrc((const char*)p.states + (size_t)T * st_step), state_at(pl), s * st_state, x);
            ds[s] = v[0];
            sc[s] = x[0];
            sp[s] = 1.0f;
        }
#pragma unroll
        for (int k = 0; k < PG::NK; ++k) kf[k] = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g) dbacc[g] = 0.0f;
        pin(ds);
        pin(sc);
        // ---- R: eight output blocks (block b: member a_me of subgroup b / UB), this wave's slice of the subgroup's contraction
        bf16x16 Rs[SP && NKF ? 8 : 1][SP && NKF ? NKF : 1];
        i32x4 Rh[SP && HALF ? 8 : 1];
        bf16x8 Rd[SP ? 1 : 8][SP ? 1 : KTW];
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint32_t d = ((b / UB) * PA + a_me) * U + (b % UB) * 16 + pc;
            const rsrc_t r_row = make_rsrc((const uint16_t*)p.R + (size_t)n * D * G * D);
            auto four = [&](uint32_t k) {   // four elements of column d from k on of this wave's slice (beyond the subgroup's gate gradients out of range: zeros)
                const uint32_t kk = k0 + k, am = kk / GU, rem = kk % GU;
                return __builtin_amdgcn_raw_buffer_load_b64(r_row, kk < K2 ? (d * (G * D) + (rem / U) * D + (s_me * PA + am) * U + rem % U) * 2 : kDrop, 0, 0);
            };
            if constexpr (SP) {
#pragma unroll
                for (int kc = 0; kc < NKF; ++kc) {
                    i32x4 piece[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t k = (2 * kc + h) * 32 + sparse_k(pquad);
                        piece[h] = sparse_piece(four(k), four(k + 8));
                    }
                    Rs[b][kc] = sparse_dense(piece[0], piece[1]);
                }
                if constexpr (HALF) Rh[b] = sparse_piece(four(NKF * 64 + 8 * pquad), four(NKF * 64 + 8 * pquad + 4));
            } else {
#pragma unroll
                for (int kt = 0; kt < KTW; ++kt) {
                    const i32x2 lo = four(kt * 32 + pquad * 8), hi = four(kt * 32 + pquad * 8 + 4);
                    Rd[b][kt] = __builtin_bit_cast(bf16x8, i32x4{lo[0], lo[1], hi[0], hi[1]});
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        auto take = [&](uint32_t slot) {   // this lane's inputs of a step, and what follows from them alone
            const char* in = ring + slot * C::SLOT;
            float cv[NC];
            take_record_lds<C::CT::RS, NC>(in + l_rec, cv);
#pragma unroll
            for (int s = C::SB0; s < C::SB0 + C::NSB; ++s) sp[s] = *(const float*)(in + l_st + (s - C::SB0) * BT * U * 4);
            dh_ext = bf16_bits_to_f32(*(const uint16_t*)(in + l_dh));
            PG::factors(cv, sc, sp, kf);
            if constexpr (!cell_uses_h_prev(CELL)) {
#pragma unroll
                for (int s = C::SB0; s < C::SB0 + C::NSB; ++s) sc[s] = sp[s];
            }
            pin(kf);
        };
        const int wio = w - 4;   // (OWN_IO) this wave among those that move inputs and outputs
        const BwdLoader<C> in(p, n, q, e0, fresh_lane(lane), wio < 0 ? 0 : wio);
        const BwdStorer<C> out_waves(p, n, q, e0, fresh_lane(lane), wio < 0 ? 0 : wio);
        if constexpr (C::OWN_IO) {
            if (wio >= 0) in.burst(p, smem, wio, 0);
            wait_vmem<0>();
        }
        wg_barrier();   // the first inputs are there
        if constexpr (C::OWN_IO) {
            if (wio >= 0) in.burst(p, smem, wio, C::KB);
        }
        if (T > 0 && pairs) take(0);

        FRNN_TRACE_RESET();
        uint32_t slot = 0;
        for (int s = 0; s < T; ++s) {
            const uint32_t cnt = (uint32_t)iter * (uint32_t)T + (uint32_t)s, x1 = (cnt & 3u) * xbuf1 + xgroup1, x2 = (cnt & 3u) * xbuf2;
            // ---- gate gradients of the step: to the subgroup, and into the image of dWx
            if (pairs) {
                float dwx[G], dg[G];
                ds[0] += dh_ext;
                PG::apply(kf, ds, dwx, dg);
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float v[1] = {dg[g]};
                    float v4[4];
                    expand_tile<4, 1, true>(v, v4);
                    store_words(xr, x1lane, x1 + g * (U * 2), i32x2{exch_word(pack_bf16x2(v4[0], v4[1])), exch_word(pack_bf16x2(v4[2], v4[3]))}, false);
                }
                char* out = smem + (s & 1) * C::DG_BYTES;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    *(uint16_t*)(out + l_dg + g * U * 2) = (uint16_t)f32_to_bf16_bits(dg[g]);
                    dbacc[g] += dg[g];
                }
                if constexpr (CELL == CELL_GRU) *(uint16_t*)(smem + C::IMG_OFF + (s & 1) * C::IMG_BYTES + row * U * 2 + (ub * 16 + c) * 2) = (uint16_t)f32_to_bf16_bits(dwx[2]);
            }
            FRNN_TRACE_MARK(0);
            // ---- this wave's slice of the subgroup's gate gradients
            i32x4 raw[NPC];
            if (p.spin_limit < 0 && !failed) {   // host-forced failure (tests of the error path): give up without looking
                __hip_atomic_store(p.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                failed = true;
            }
            for (int spins = 0;; ++spins) {
#pragma unroll
                for (int j = 0; j < NPC; ++j) {
                    if (SP && HALF && j == NKF) {
                        const i32x2 v = __builtin_amdgcn_raw_buffer_load_b64(xr, half_off, x1, kAuxPoll);
                        raw[j] = i32x4{v[0], v[1], 0, 0};
                    } else {
                        raw[j] = __builtin_amdgcn_raw_buffer_load_b128(xr, piece_voff(j), x1, kAuxPoll);
                    }
                }
                uint32_t top = 0u;   // (a word out of range reads as zero)
#pragma unroll
                for (int j = 0; j < NPC; ++j) top = max(top, max(max((uint32_t)raw[j][0], (uint32_t)raw[j][1]), max((uint32_t)raw[j][2], (uint32_t)raw[j][3])));
                if (__all((int)(top != kNoWord)) || failed) break;
                if (poll_gives_up(spins, p.spin_limit, p.err)) { failed = true; break; }
            }
            wait_vmem<0>();   // (also what this wave has taken back, if it had nothing to poll)
            FRNN_TRACE_MARK(2);
            char* red = smem + C::RED_OFF + (C::NRED == 2 ? (s & 1) * C::RED : 0);
            constexpr int CH = KTW >= 4 ? 2 : 4;   // blocks at a time: R leaves no registers for more accumulators
#pragma unroll
            for (int b0 = 0; b0 < 8; b0 += CH) {
                f32x4 a[CH];
#pragma unroll
                for (int x = 0; x < CH; ++x) a[x] = f32x4{0.f, 0.f, 0.f, 0.f};
                // (R leaves no registers for accumulators of the half step's own, as split_fwd_compute has them: it comes first, and the steps of 64 begin when
                // all its sums are there -- four passes, eight instruction slots)
                if constexpr (SP && HALF) {
#pragma unroll
                    for (int x = 0; x < CH; ++x) a[x] = smfmac32(i32x2{raw[NPC - 1][0], raw[NPC - 1][1]}, Rh[b0 + x], a[x], sl.idx);
                    static_assert(CH == 4);
                    asm volatile("s_nop 7" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]));
                }
#pragma unroll
                for (int j = 0; j < (SP ? NKF : KTW); ++j)
#pragma unroll
                    for (int x = 0; x < CH; ++x) {
                        if constexpr (SP) a[x] = smfmac(__builtin_bit_cast(bf16x8, raw[j]), Rs[b0 + x][j], a[x], sl.idx);
                        else a[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, raw[j]), Rd[b0 + x][j], a[x], 0, 0, 0);
                    }
#pragma unroll
                for (int x = 0; x < CH; ++x) {
                    float* o = (float*)(red + ((w * 8 + b0 + x) * 64 + lane) * (PPV * 4));
                    typedef __attribute__((__vector_size__(PPV * sizeof(float)))) float part_t;
                    part_t v;
#pragma unroll
                    for (int i = 0; i < PPV; ++i) v[i] = SP ? a[x][(2 * i) & 3] + a[x][(2 * i + 1) & 3] : a[x][i];
                    *(part_t*)o = v;
                    asm volatile("" : : "v"(a[x]));   // (4-row tiles: nobody gets the two unused registers of an accumulator before the sums are formed)
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            FRNN_TRACE_MARK(4);
            wg_barrier();
            FRNN_TRACE_MARK(1);
            if (pairs) {   // (every member of the subgroup has this round, so all are done with the one before: its words are taken back)
#pragma unroll
                for (int g = 0; g < G; ++g) clear_tile<true>(xr, x1lane, ((cnt + 3u) & 3u) * xbuf1 + xgroup1 + g * (U * 2), false);
            }
            // ---- block w of the eight: the waves' sums, to its owner
            {
                typedef __attribute__((__vector_size__(PPV * sizeof(float)))) float part_t;
                part_t v[8];
#pragma unroll
                for (int x = 0; x < 8; ++x) v[x] = *(const part_t*)(red + ((x * 8 + w) * 64 + lane) * (PPV * 4));
                float sum[PPV];
#pragma unroll
                for (int i = 0; i < PPV; ++i) sum[i] = ((v[0][i] + v[1][i]) + (v[2][i] + v[3][i])) + ((v[4][i] + v[5][i]) + (v[6][i] + v[7][i]));
                if (p.spread) store_part<PPV, kAuxAgent>(xr, lane * BT, x2 + x2out, sum);
                else store_part<PPV>(xr, lane * BT, x2 + x2out, sum);
            }
            if constexpr (C::OWN_IO) {   // (the burst before is complete: every wave has waited for all of its own ahead of the barrier)
                if (wio >= 0) {
                    out_waves.store(p, smem, s, (uint32_t)(s & 1));
                    if ((s + 1) % C::KB == 0) in.burst(p, smem, wio, s + 1 + C::KB);
                }
            }
            if constexpr (C::NRED == 1) wg_barrier();
            FRNN_TRACE_MARK(5);
            slot = slot + 1 == (uint32_t)C::RD ? 0 : slot + 1;
            if (pairs) {
                take(slot);   // the inputs of the next step, while the partial sums travel
                uint32_t got[PB];
                for (int spins = 0;; ++spins) {
#pragma unroll
                    for (int j = 0; j < PB; ++j) got[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(xr, lane * BT, x2 + x2in + j * C::SEG, kAuxPoll);
                    uint32_t top = 0u;
#pragma unroll
                    for (int j = 0; j < PB; ++j) top = max(top, got[j]);
                    if (__all((int)(top != kNoWord)) || failed) break;
                    if (poll_gives_up(spins, p.spin_limit, p.err)) { failed = true; break; }
                }
                // (taken back for the round after the next three: nobody else looks at these words)
#pragma unroll
                for (int j = 0; j < PB; ++j) {
                    if (p.spread) __builtin_amdgcn_raw_buffer_store_b32((int)kNoWord, xr, lane * BT, x2 + x2in + j * C::SEG, kAuxAgent);
                    else __builtin_amdgcn_raw_buffer_store_b32((int)kNoWord, xr, lane * BT, x2 + x2in + j * C::SEG, 0);
                }
                float rec = __builtin_bit_cast(float, got[0]);
#pragma unroll
                for (int j = 1; j < PB; ++j) rec += __builtin_bit_cast(float, got[j]);
                ds[0] += fminf(fmaxf(rec, -p.clip), p.clip);   // (Sec. 4.1 clip; +inf = off)
            }
            FRNN_TRACE_MARK(7);
        }
        // ---- gradients of the initial states, per-row partial sums of db
        const uint32_t el = fresh_lane(lane), brow = q * BT + row_of(el);
        if (pairs && brow < B) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const float v[1] = {ds[s]};
                store_io_r<false, 1>(make_rsrc(p.dstates0), state_at(el), s * st_state, v);
            }
            float* db = p.db_part + (((size_t)brow * NH + n) * G) * D + e0 + ub * 16 + (el & 15);
#pragma unroll
            for (int g = 0; g < G; ++g) db[(size_t)g * D] = dbacc[g] + (p.db_accumulate ? db[(size_t)g * D] : 0.0f);
        }
    }
    FRNN_TRACE_END(p);
}

template <int CELL, int UB, int KTW, int BT>
__global__ __launch_bounds__((MeshBwd<CELL, UB, KTW, BT>::NW * 64)) void mesh_bwd_kernel(const KernelParams p) {
    using C = MeshBwd<CELL, UB, KTW, BT>;
    extern __shared__ __align__(16) char smem[];
    const BlockMap bm(p, true);
    if (!bm.active) return;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (C::OWN_IO || w < C::NCW) mesh_bwd_compute<CELL, UB, KTW, BT>(p, bm, smem, lane, w);
    else if (w < C::NCW + C::NLD) split_bwd_load<C>(p, bm, smem, lane, w - C::NCW);
    else split_bwd_store<C>(p, bm, smem, lane, w - C::NCW - C::NLD);
}

// ---------------------------------------------------------------------------------------------
// Forward
// ---------------------------------------------------------------------------------------------
// UB blocks of 16 units per workgroup.  NCW compute waves share the contraction: wave w takes the k-steps w * KTW .. of h_{t-1} for ALL
// outputs of the workgroup, so it polls its own slice of the exchanged rows straight into the operand registers of its matrix instructions (no LDS
// rows, no barrier between the poll and the product, each word polled once per workgroup); the slices' sums meet in LDS, where the point-wise
// function takes them up.  h is exchanged as in fwd_kernel: rows of bf16 words, four buffers, taken back one round later.
// p.R is the packed forward copy of R: Rt[n][g][e][k], k < D.
// SPREAD: the group's members sit on all XCDs (member % 8 is the XCD).  h goes to memory once; in each XCD every member fetches an equal share of the
// group's rows from there (16 bytes per row and member and lane: BT / 4 waves of the upper four, "relays") and leaves it in a buffer of the XCD's own, which
// all members of that XCD poll in their L2.  (LSTM 1 x 2048, 16 rows 4.57 -> 3.2 us per step, 4 rows 2.5; of a step the way through memory takes a third, the
// XCD's own hand-over a quarter.  An XCD's members own consecutive units: with consecutive units on all XCDs 3.64.)  There are no waves beside the
// eight compute waves, whose upper four move inputs and outputs too.
template <int CELL, int UB, int KTW, int NCW, int BT, bool SPREAD = false> struct SplitFwd {
    using CT = CellTraits<CELL>;
    static constexpr int G = CT::G, S = CT::S, NC = CT::NC;
    static constexpr bool SP = BT < 16;
    static constexpr int U = 16 * UB, NLD = 1, NST = SPREAD ? 4 : NCW == 4 ? 3 : 1, NW = SPREAD ? NCW : NCW + NLD + NST;
    static_assert(!SPREAD || (UB == 1 && NCW == 8));
    static constexpr int DK = NCW * KTW * 32, XROW = DK * 2;
    static constexpr int NKF = KTW / 2, HALF = KTW & 1;                // sparse steps of 64, of 32
    static constexpr int NPT = UB * BT / 4, PW = NPT <= NCW ? NPT : NPT / 2, PT = NPT / PW;   // tiles of 16 units x 4 rows, the waves that take them, tiles each
    static constexpr int GP = G == 3 ? 4 : G;                           // floats per pair of the slices' sums
    // inputs of a step: rows (gate, row) in the ring; outputs: state rows, records
    static constexpr int CW = G * BT * 2 * UB, NLJ = (CW + 64 * NLD - 1) / (64 * NLD), SLOT = NLD * NLJ * 1024;
    static constexpr int REC = CT::RS * 2, CST = S * BT * 4 * UB, CRC = BT * REC * UB;
    static constexpr int GST = (CST + 63) / 64, GRC = (CRC + 63) / 64, NSJ = (GST + GRC + NST - 1) / NST;
    // (row pitches of the output image: the four rows that one instruction writes -- consecutive ones, or with 16 rows every fourth -- lie 64 bytes
    // apart modulo the banks)
    static constexpr int PST = U * 4 + (BT == 16 ? 16 : UB == 1 ? 0 : 64), PRC = U * REC + (BT == 16 ? 16 : UB == 1 ? 0 : 64);
    static constexpr int OUT = S * BT * PST + BT * PRC, RED = NCW * NPT * 64 * GP * 4;
    // (two buffers of the slices' sums where they fit; with one a second barrier per step)
    static constexpr int ROOM = 160 * 1024 - U * GP * 4 - 2 * OUT - 16, NRED = 2 * RED + 8 * SLOT <= ROOM ? 2 : 1;
    static constexpr int KB = burst_steps(SLOT, ROOM - NRED * RED < 64 * 1024 ? ROOM - NRED * RED : 64 * 1024), RD = 2 * KB;   // steps per burst, slots
    static constexpr int BIAS_OFF = RD * SLOT, OUT_OFF = BIAS_OFF + U * GP * 4, RED_OFF = (OUT_OFF + 2 * OUT + 15) / 16 * 16, SMEM = RED_OFF + NRED * RED;
    // unit blocks of a ring row are rotated by the number of the row among those that one instruction reads
    static __host__ __device__ constexpr uint32_t rot(uint32_t row) { return BT == 16 ? row / 4 : row; }
    static constexpr int kUB = UB, kBT = BT;
    // (spread: the units of an XCD's members are consecutive -- where D is a multiple of 512 every cache line of h is written from one XCD)
    static __device__ __forceinline__ uint32_t unit0(const KernelParams& p, uint32_t member) { return SPREAD ? ((member % 8) * (p.P / 8) + member / 8) * U : member * U; }
};

// The inputs of a group's steps, by one wave, into the ring.
template <class C> struct FwdLoader {
    uint32_t voff[C::NLJ];
    __device__ __forceinline__ FwdLoader(const KernelParams& p, uint32_t n, uint32_t q, uint32_t e0, int lane) {
        constexpr int UB = C::kUB, BT = C::kBT;
#pragma unroll
        for (int j = 0; j < C::NLJ; ++j) {
            const uint32_t idx = j * 64 + lane, cpr = 2 * UB, r = idx / cpr, pos = idx % cpr, g = r / BT, row = r % BT, brow = q * BT + row;
            const uint32_t blk = (pos / 2 + UB * BT - C::rot(row)) % UB;
            voff[j] = g < (uint32_t)C::G && brow < (uint32_t)p.B ? ((brow * C::G + g) * (uint32_t)(p.NH * p.D) + n * p.D + e0 + blk * 16) * 2 + (pos & 1) * 16 : 0x80000000u;
        }
    }
    __device__ __forceinline__ void burst(const KernelParams& p, char* smem, int s0) const {   // inputs of the steps s0 .. s0 + KB - 1
        const size_t wx_step = (size_t)p.B * C::G * p.NH * p.D * 2;
#pragma unroll 1
        for (int s = s0; s < s0 + C::KB && s < p.T; ++s) {
            const rsrc_t rs = make_rsrc((const char*)p.Wx + s * wx_step);
#pragma unroll
            for (int j = 0; j < C::NLJ; ++j) load_chunk_to_lds(rs, smem + s % C::RD * C::SLOT + j * 1024, voff[j]);
        }
    }
};
// The outputs of a step, by C::NST waves (ws = 0 ..), from their image in LDS.
template <class C> struct FwdStorer {
    uint32_t voff[C::NSJ], loff[C::NSJ];
    __device__ __forceinline__ FwdStorer(const KernelParams& p, uint32_t n, uint32_t q, uint32_t e0, int lane, int ws) {
        constexpr int UB = C::kUB, BT = C::kBT;
        const uint32_t B = p.B, HD = p.NH * p.D;
#pragma unroll
        for (int j = 0; j < C::NSJ; ++j) {
            const int piece = j * C::NST + ws;
            voff[j] = 0x80000000u;
            loff[j] = C::OUT_OFF;
            auto place = [&](uint32_t idx, uint32_t rows, uint32_t esz, uint32_t plane, uint32_t base, uint32_t pitch) {   // rows of U elements of esz bytes
                const uint32_t cpr = UB * esz, r = idx / cpr, ch = idx % cpr, brow = q * BT + r % BT;
                if (r < rows) {
                    loff[j] = C::OUT_OFF + base + r * pitch + ch * 16;
                    if (brow < B) voff[j] = (r / BT) * plane + (brow * HD + n * p.D + e0) * esz + ch * 16;
                }
            };
            if (piece < C::GST) place(piece * 64 + lane, C::S * BT, 4, B * HD * 4, 0, C::PST);
            else if (p.cache != nullptr && piece < C::GST + C::GRC) place((piece - C::GST) * 64 + lane, BT, C::REC, 0, C::S * BT * C::PST, C::PRC);
        }
    }
    __device__ __forceinline__ void store(const KernelParams& p, const char* smem, int ws, int s) const {   // the outputs of step s
        const size_t units = (size_t)p.B * p.NH * p.D;
        const bool saves = p.cache != nullptr;
        const rsrc_t st = make_rsrc((char*)p.states + (size_t)(s + 1) * C::S * units * 4), ca = make_rsrc((char*)p.cache + (saves ? s : 0) * (units * C::REC));
        i32x4 v[C::NSJ];
#pragma unroll
        for (int j = 0; j < C::NSJ; ++j) v[j] = *(const i32x4*)(smem + loff[j] + (s & 1) * C::OUT);
#pragma unroll
        for (int j = 0; j < C::NSJ; ++j) {
            const bool state = j * C::NST + ws < C::GST;
            if (state || saves) __builtin_amdgcn_raw_buffer_store_b128(v[j], state ? st : ca, voff[j], 0, 0);
        }
    }
};

template <class C>
__device__ __forceinline__ void split_fwd_load(const KernelParams& p, const BlockMap& bm, char* smem, int lane) {
    for (int gid = bm.gpar; gid < p.NG; gid += p.GPAR) {
        const FwdLoader<C> in(p, gid % p.NH, gid / p.NH, C::unit0(p, bm.member), lane);
        in.burst(p, smem, 0);
        wg_barrier();
        wg_barrier();
        for (int s = 0; s < p.T; ++s) {
            const bool next = s % C::KB == 0;    // step s begins a burst: it must be there, and the slots of the burst before are free behind the barrier
            if (next) wait_vmem<0>();
            wg_barrier();
            if (next) in.burst(p, smem, s + C::KB);
            if constexpr (C::NRED == 1) wg_barrier();
        }
        wait_vmem<0>();
        wg_barrier();
    }
}

template <class C>
__device__ __forceinline__ void split_fwd_store(const KernelParams& p, const BlockMap& bm, char* smem, int lane, int ws) {
    for (int gid = bm.gpar; gid < p.NG; gid += p.GPAR) {
        const FwdStorer<C> out(p, gid % p.NH, gid / p.NH, C::unit0(p, bm.member), lane, ws);
        wg_barrier();
        wg_barrier();
        for (int s = 0; s <= p.T; ++s) {
            wg_barrier();
            if (s > 0) out.store(p, smem, ws, s - 1);
            if constexpr (C::NRED == 1) if (s < p.T) wg_barrier();
        }
    }
}

template <int CELL, int UB, int KTW, int NCW, int BT, bool SPREAD>
__device__ __forceinline__ void split_fwd_compute(const KernelParams& p, const BlockMap& bm, char* smem, int lane, int w) {
    using C = SplitFwd<CELL, UB, KTW, NCW, BT, SPREAD>;
    constexpr int G = C::G, S = C::S, NC = C::NC, PT = C::PT, U = C::U, NKF = C::NKF, HALF = C::HALF, GP = C::GP;
    constexpr bool SP = C::SP;
    constexpr uint32_t kDrop = 0x80000000u;
    typedef __attribute__((__vector_size__(GP * sizeof(float)))) float sums_t;
    const int T = p.T, me = bm.member;
    const uint32_t B = p.B, NH = p.NH, D = p.D, HD = NH * D, e0 = C::unit0(p, me);
    const SparseLane<BT == 8 ? 8 : 4> sl(lane);
    const uint32_t c = sl.c, quad = sl.quad, k0 = w * KTW * 32;
    const rsrc_t xr = make_rsrc(p.exch);
    const uint32_t xbuf = (uint32_t)p.GPAR * BT * C::XROW, xgroup = (uint32_t)bm.gpar * BT * C::XROW;
    const uint32_t xnear = SPREAD ? (4u + 4u * (me % 8)) * xbuf : 0u;   // this XCD's own four buffers, behind the common ones
    bool failed = false;
    FRNN_TRACE_BEGIN();

    // ---- this lane's (unit, row) pairs: the same row and unit in PT blocks of units UBK apart
    constexpr uint32_t UBK = UB / PT;
    static_assert(C::PW <= NCW && C::PW % (BT / 4) == 0, "one or two tiles per wave, the second UBK blocks further on");
    const bool pairs = w < C::PW;
    const uint32_t tile = pairs ? w : 0, ub = tile / (BT / 4);
    struct Places { uint32_t xlane, wx, bias, st, rec; };
    auto places_of = [&](uint32_t ln) {
        const uint32_t cc = ln & 15, qd = ln >> 4, row = BT == 16 ? 4 * qd + tile % (BT / 4) : qd + 4 * (tile % (BT / 4));
        Places pl;
        pl.xlane = (cc & 3) == 0 ? row * C::XROW + (e0 + ub * 16 + cc) * 2 : kDrop;   // (the lanes of every fourth unit publish it and the three behind it)
        pl.wx = ((row * UB + (ub + C::rot(row)) % UB) * 16 + cc) * 2;
        pl.bias = C::BIAS_OFF + (ub * 16 + cc) * (GP * 4);
        pl.st = C::OUT_OFF + row * C::PST + (ub * 16 + cc) * 4;
        pl.rec = C::OUT_OFF + S * BT * C::PST + row * C::PRC + (ub * 16 + cc) * C::REC;
        return pl;
    };
    // (kernels whose R leaves few registers form them anew every step)
    constexpr bool kTight = G * UB * KTW >= 44;
    const Places at_once = places_of(lane);
    // ---- this lane's operand pieces inside the exchanged rows.  Out of range read as zeros: beyond the head's units; with 4 rows the operand rows
    // that repeat others (they only reach result registers that nobody uses).
    constexpr int NPC = SP ? NKF + HALF : KTW;
    const uint32_t xrow = (SP ? sl.rslot : c) * C::XROW + k0 * 2 + (SP ? sl.rbyte : quad * 16);
    const bool reads = !(BT == 4 && (c & 2));
    // (the offset of piece j is formed anew where it is used: kept from step to step they would take a register each)
    uint32_t k_lane = k0 + (SP ? sl.rbyte / 2 : quad * 8);   // first contraction element of the lane's piece 0
    if (!reads) k_lane = D;
    auto piece_voff = [&](int j) {
        asm volatile("" : "+v"(k_lane));
        return k_lane + j * (SP ? 64 : 32) < D ? xrow + j * (SP ? 128 : 64) : kDrop;
    };
    uint32_t half_off = kDrop;   // (the last half step, of 32 elements)
    if (SP && HALF && reads && k0 + NKF * 64 + sl.rbyte32 / 2 < D) half_off = sl.rslot * C::XROW + (k0 + NKF * 64) * 2 + sl.rbyte32;

    int iter = 0;
    for (int gid = bm.gpar; gid < p.NG; gid += p.GPAR, ++iter) {
        const uint32_t n = gid % NH, q = gid / NH;
        // ---- bias into LDS, initial states
        wg_barrier();   // (the group before is done with its bias)
        const uint32_t pl = fresh_lane(lane), pc = pl & 15, pquad = pl >> 4;
        for (uint32_t j = w * 64 + pl; j < (uint32_t)U * G; j += NCW * 64) {
            float v[1];
            load_io<true, 1>(p.bias, ((size_t)n * G + j / U) * D + e0 + j % U, v);
            *(float*)(smem + C::BIAS_OFF + (j % U) * (GP * 4) + (j / U) * 4) = v[0];
        }
        float st[PT][S];
        {
            const uint32_t brow = q * BT + (BT == 16 ? 4 * pquad + tile % (BT / 4) : pquad + 4 * (tile % (BT / 4)));
            const uint32_t g_st = ((brow < B ? brow : B - 1) * HD + n * D + e0 + ub * 16 + pc) * 4;
#pragma unroll
            for (int k = 0; k < PT; ++k)
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    float v[1] = {0.0f};
                    if (p.states0 != nullptr) load_io_r<false, 1>(make_rsrc(p.states0), g_st + k * UBK * 64, s * (B * HD * 4), v);
                    st[k][s] = v[0];
                    store_io_r<false, 1>(make_rsrc(p.states), pairs && brow < B ? g_st + k * UBK * 64 : kDrop, s * (B * HD * 4), v);
                }
        }
        auto publish = [&](const Places& pl, int k, uint32_t off, bool real) {
            const float h[1] = {st[k][0]};
            float v4[4];
            expand_tile<4, 1, true>(h, v4);
            store_words(xr, pl.xlane | (real ? 0u : kDrop), off + k * UBK * 32, i32x2{exch_word(pack_bf16x2(v4[0], v4[1])), exch_word(pack_bf16x2(v4[2], v4[3]))}, SPREAD);
        };
        if (pairs && T > 0) {
#pragma unroll
            for (int k = 0; k < PT; ++k) publish(kTight ? places_of(pl) : at_once, k, ((uint32_t)iter * (uint32_t)T & 3u) * xbuf + xgroup, true);
        }
        pin(st);
        // ---- R in registers for all steps (last here: everything above needs registers too): column c = unit of a block, this wave's slice of the contraction
        bf16x16 Rs[SP && NKF ? G * UB : 1][SP && NKF ? NKF : 1];
        i32x4 Rh[SP && HALF ? G * UB : 1];
        bf16x8 Rd[SP ? 1 : G * UB][SP ? 1 : KTW];
        const rsrc_t r_head = make_rsrc((const uint16_t*)p.R + (size_t)n * G * D * D);
#pragma unroll
        for (int x = 0; x < G * UB; ++x) {
            const uint32_t rrow = (((x / UB) * D + e0 + (x % UB) * 16 + pc) * D + k0) * 2;
            auto four = [&](uint32_t k) {   // four elements from k on of this wave's slice (beyond the head's units out of range: zeros)
                return __builtin_amdgcn_raw_buffer_load_b64(r_head, k0 + k < D ? rrow + k * 2 : kDrop, 0, 0);
            };
            if constexpr (SP) {
#pragma unroll
                for (int kc = 0; kc < NKF; ++kc) {
                    i32x4 piece[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t k = (2 * kc + h) * 32 + sparse_k(pquad);
                        piece[h] = sparse_piece(four(k), four(k + 8));
                    }
                    Rs[x][kc] = sparse_dense(piece[0], piece[1]);
                }
                if constexpr (HALF) Rh[x] = sparse_piece(four(NKF * 64 + 8 * pquad), four(NKF * 64 + 8 * pquad + 4));
            } else {
#pragma unroll
                for (int kt = 0; kt < KTW; ++kt) {
                    const i32x2 lo = four(kt * 32 + pquad * 8), hi = four(kt * 32 + pquad * 8 + 4);
                    Rd[x][kt] = __builtin_bit_cast(bf16x8, i32x4{lo[0], lo[1], hi[0], hi[1]});
                }
            }
        }
        // (SPREAD) what the upper four waves do beside their part of the products
        const int wio = SPREAD ? w - 4 : -1;
        const FwdLoader<C> in(p, n, q, e0, pl);
        const FwdStorer<C> out_waves(p, n, q, e0, pl, wio < 0 ? 0 : wio);
        const bool relay = SPREAD && wio >= 0 && wio < BT / 4;
        uint32_t relay_off = 0;
        if constexpr (SPREAD) {
            const uint32_t id = (me / 8) * (BT * 16) + (wio < 0 ? 0 : wio) * 64 + pl, cpr = D / 8;   // chunk of 16 bytes among the group's BT rows of D / 8
            relay_off = id / cpr * C::XROW + id % cpr * 16;
            if (wio == 3) in.burst(p, smem, 0);
        }
        wg_barrier();

        FRNN_TRACE_RESET();
        uint32_t slot = 0;
        for (int s = 0; s < T; ++s) {
            const uint32_t cnt = (uint32_t)iter * (uint32_t)T + (uint32_t)s;
            FRNN_TRACE_MARK(0);
            // (the matrix instructions add to their result registers in place: cleared here, while the words travel, where there are registers for it)
            constexpr bool kEarly = NPC <= 4 && G * UB * (KTW + 4) <= 96;
            f32x4 acc[kEarly ? UB : 1][G];
            if constexpr (kEarly) {
#pragma unroll
                for (int u = 0; u < UB; ++u)
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        acc[u][g] = f32x4{0.f, 0.f, 0.f, 0.f};
                        asm volatile("" : "+v"(acc[u][g]));
                    }
            }
            // ---- this wave's slice of h_{t-1}
            const uint32_t xin = xnear + (cnt & 3u) * xbuf + xgroup;
            if constexpr (SPREAD) {   // the relays: their share of h_{t-1} from memory into the XCD's buffer
                if (relay) {
                    i32x4 v;
                    for (int spins = 0;; ++spins) {
                        v = __builtin_amdgcn_raw_buffer_load_b128(xr, relay_off, (cnt & 3u) * xbuf + xgroup, kAuxPoll);
                        const uint32_t top = max(max((uint32_t)v[0], (uint32_t)v[1]), max((uint32_t)v[2], (uint32_t)v[3]));
                        if (__all((int)(top != kNoWord)) || failed || p.spin_limit < 0) break;
                        if (poll_gives_up(spins, p.spin_limit, p.err)) { failed = true; break; }
                    }
                    __builtin_amdgcn_raw_buffer_store_b128(v, xr, relay_off + xin, 0, 0);
                }
            }
            i32x4 raw[NPC];
            if (p.spin_limit < 0 && !failed) {   // host-forced failure (tests of the error path): give up without looking
                __hip_atomic_store(p.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                failed = true;
            }
            auto look = [&](int j) {
                if (SP && HALF && j == NKF) {
                    const i32x2 v = __builtin_amdgcn_raw_buffer_load_b64(xr, half_off, xin, kAuxPoll);
                    raw[j] = i32x4{v[0], v[1], 0, 0};
                } else {
                    raw[j] = __builtin_amdgcn_raw_buffer_load_b128(xr, piece_voff(j), xin, kAuxPoll);
                }
            };
            // piece `from` (and with `all` the ones behind it too) is there; until then it and the ones behind it are looked at again
            auto wait_for = [&](auto from_c, bool all) {
                constexpr int from = decltype(from_c)::value;
                for (int spins = 0;; ++spins) {
                    if (from == 0 || spins > 0) {
#pragma unroll
                        for (int j = from; j < NPC; ++j) look(j);
                    }
                    uint32_t top = 0u;   // (a word out of range reads as zero)
#pragma unroll
                    for (int j = from; j < NPC; ++j)
                        if (all || j == from) top = max(top, max(max((uint32_t)raw[j][0], (uint32_t)raw[j][1]), max((uint32_t)raw[j][2], (uint32_t)raw[j][3])));
                    if (__all((int)(top != kNoWord)) || failed) break;
                    if (poll_gives_up(spins, p.spin_limit, p.err)) { failed = true; break; }
                }
            };
            auto product = [&](int j, int u, f32x4 (&a)[G], f32x4& ah) {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if constexpr (!SP) a[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, raw[j]), Rd[g * UB + u][j], a[g], 0, 0, 0);
                    else if (HALF && G == 1 && j == NKF) ah = smfmac32(i32x2{raw[j][0], raw[j][1]}, Rh[u], ah, sl.idx);
                    else if (HALF && j == NKF) a[g] = smfmac32(i32x2{raw[j][0], raw[j][1]}, Rh[HALF ? g * UB + u : 0], a[g], sl.idx);
                    else a[g] = smfmac(__builtin_bit_cast(bf16x8, raw[j]), Rs[NKF ? g * UB + u : 0][NKF ? j : 0], a[g], sl.idx);
                }
            };
            const uint32_t rl = kTight ? fresh_lane(lane) : lane;
            char* red = smem + C::RED_OFF + (C::NRED == 2 ? (s & 1) * C::RED : 0);
            auto leave = [&](int u, f32x4 (&a)[G], f32x4& ah) {   // this wave's sums of unit block u
#pragma unroll
                for (int r = 0; r < BT / 4; ++r) {
                    if constexpr (SP && HALF && G == 1) {
                        a[0][(2 * r) & 3] += ah[(2 * r) & 3];
                        a[0][(2 * r + 1) & 3] += ah[(2 * r + 1) & 3];
                    }
                    sums_t v;
#pragma unroll
                    for (int g = 0; g < GP; ++g) v[g] = g >= G ? 0.0f : SP ? a[g < G ? g : 0][(2 * r) & 3] + a[g < G ? g : 0][(2 * r + 1) & 3] : a[g < G ? g : 0][r];
                    *(sums_t*)(red + ((w * C::NPT + u * (BT / 4) + r) * 64 + rl) * (GP * 4)) = v;
                }
                // (4-row tiles use two of an accumulator's registers: nobody else gets the other two before the sums are formed)
#pragma unroll
                for (int g = 0; g < G; ++g) asm volatile("" : : "v"(a[g]));
                if constexpr (SP && HALF && G == 1) asm volatile("" : : "v"(ah));
            };
            // A half step on registers that a step of 64 is still adding to has given wrong sums, and the compiler keeps no distance between the two.  So the
            // sums are read between them, behind the wait for the half step's piece: an empty instruction, for which the compiler lets the matrix
            // instructions finish (they long have: 0.3 % over heads of 288 to 368 and 1280 units; accumulators of its own for the half step 3 %, the same
            // read ahead of the wait 1.6 %).  Elman, with one matrix instruction per piece, has accumulators of its own.
            f32x4 ah[UB];
#pragma unroll
            for (int u = 0; u < UB; ++u) ah[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            static_assert(!(SP && HALF) || kEarly, "the half step's distance rests on the wait in front of it");
            if constexpr (kEarly) {
                // each piece is multiplied as soon as it is there
                auto piece = [&](auto j_c) {
                    constexpr int j = decltype(j_c)::value;
                    if constexpr (j < NPC) {
                        wait_for(j_c, false);
                        if constexpr (SP && HALF && G > 1 && j == NKF) {
#pragma unroll
                            for (int u = 0; u < UB; ++u)
#pragma unroll
                                for (int g = 0; g < G; ++g) asm volatile("" : "+v"(acc[u][g]));
                        }
                        if constexpr (j == NPC - 1) wait_vmem<0>();   // (also what this wave has taken back, if it had nothing to poll)
                        if constexpr (j == 0) FRNN_TRACE_MARK(2);
#pragma unroll
                        for (int u = 0; u < UB; ++u) product(j, u, acc[u], ah[u]);
                    }
                };
                piece(std::integral_constant<int, 0>{});
                piece(std::integral_constant<int, 1>{});
                piece(std::integral_constant<int, 2>{});
                piece(std::integral_constant<int, 3>{});
                static_assert(NPC <= 4);
#pragma unroll
                for (int u = 0; u < UB; ++u) leave(u, acc[u], ah[u]);
            } else {
                wait_for(std::integral_constant<int, 0>{}, true);
                wait_vmem<0>();   // (also what this wave has taken back, if it had nothing to poll)
                FRNN_TRACE_MARK(2);
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    f32x4 a[G];
#pragma unroll
                    for (int g = 0; g < G; ++g) a[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < NPC; ++j) product(j, u, a, ah[u]);
                    leave(u, a, ah[u]);
                    if constexpr (G * UB * KTW >= 44) __builtin_amdgcn_sched_barrier(0);   // (one block's accumulators at a time where R leaves no more registers)
                }
            }
            FRNN_TRACE_MARK(4);
            wg_barrier();
            FRNN_TRACE_MARK(1);
            if constexpr (SPREAD) {
                // (this workgroup has round cnt from every member, so all members of its XCD are done with the round before: the relay takes its words back.
                // The burst before is complete: its wave has waited for everything ahead of the barrier.)
                if (relay) __builtin_amdgcn_raw_buffer_store_b128(i32x4{(int)kNoWord, (int)kNoWord, (int)kNoWord, (int)kNoWord}, xr, relay_off + xnear + ((cnt + 3u) & 3u) * xbuf + xgroup, 0, 0);
                if (wio >= 0 && s > 0) out_waves.store(p, smem, wio, s - 1);
                if (wio == 3 && s % C::KB == 0) in.burst(p, smem, s + C::KB);
            }
            if (pairs) {
                const Places here = kTight ? places_of(fresh_lane(lane)) : at_once;
                // (every member has this round, so every member is done with the one before: its words are taken back)
#pragma unroll
                for (int k = 0; k < PT; ++k) clear_tile<true>(xr, here.xlane, ((cnt + 3u) & 3u) * xbuf + xgroup + k * UBK * 32, SPREAD);
                float yb[PT][G], wx[PT][G], cv[PT][NC];
                auto sums = [&](int k) {
                    sums_t v[4];
                    auto slices = [&](int x0) {
#pragma unroll
                        for (int x = 0; x < 4; ++x)
                            if (x0 + x < NCW) v[x] = *(const sums_t*)(red + (((x0 + x) * C::NPT + w + C::PW * k) * 64 + rl) * (GP * 4));
                    };
                    slices(0);
                    const sums_t b = *(const sums_t*)(smem + here.bias + k * UBK * (16 * GP * 4));
#pragma unroll
                    for (int g = 0; g < G; ++g) wx[k][g] = bf16_bits_to_f32(*(const uint16_t*)(smem + slot * C::SLOT + g * (BT * U * 2) + (here.wx ^ (k * UBK * 32))));
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        yb[k][g] = b[g];
#pragma unroll
                        for (int x = 0; x < 4; ++x) yb[k][g] += v[x][g];
                    }
                    if constexpr (NCW > 4) {
                        slices(4);
#pragma unroll
                        for (int g = 0; g < G; ++g)
#pragma unroll
                            for (int x = 0; x < NCW - 4; ++x) yb[k][g] += v[x][g];
                    }
                };
                if constexpr (C::NRED == 1) {
#pragma unroll
                    for (int k = 0; k < PT; ++k) sums(k);
                    wg_barrier();
                }
#pragma unroll
                for (int k = 0; k < PT; ++k) {
                    if constexpr (C::NRED == 2) sums(k);
                    Cell<CELL, true>::fwd(wx[k], yb[k], st[k], cv[k]);
                    publish(here, k, ((cnt + 1u) & 3u) * xbuf + xgroup, s + 1 < T);
                    if constexpr (kTight && PT > 1) __builtin_amdgcn_sched_barrier(0);
                }
                FRNN_TRACE_MARK(5);
                // ---- states and saved values into the output image: the store waves move them behind the next barrier
                char* out = smem + (s & 1) * C::OUT;
#pragma unroll
                for (int k = 0; k < PT; ++k) {
#pragma unroll
                    for (int x = 0; x < S; ++x) *(float*)(out + here.st + k * UBK * 64 + x * (BT * C::PST)) = st[k][x];
                    if (p.cache != nullptr) {
                        constexpr int NWD = (C::CT::RS + 1) / 2;
                        uint32_t wd[NWD];
                        pack_record<true, C::CT::RS, NC>(cv[k], wd);
                        if constexpr (C::CT::RS == 1) *(uint16_t*)(out + here.rec + k * UBK * 16 * C::REC) = (uint16_t)(wd[0] & 0xFFFFu);
                        else if constexpr (NWD == 2) *(i32x2*)(out + here.rec + k * UBK * 16 * C::REC) = i32x2{(int)wd[0], (int)wd[1]};
                        else *(i32x4*)(out + here.rec + k * UBK * 16 * C::REC) = i32x4{(int)wd[0], (int)wd[1], (int)wd[2], (int)wd[3]};
                    }
                }
            } else if constexpr (C::NRED == 1) {
                wg_barrier();
            }
            slot = slot + 1 == (uint32_t)C::RD ? 0 : slot + 1;
            FRNN_TRACE_MARK(6);
        }
        wg_barrier();   // the last outputs are in their image
        if constexpr (SPREAD) {
            if (wio >= 0 && T > 0) out_waves.store(p, smem, wio, T - 1);
        }
    }
    FRNN_TRACE_END(p);
}

template <int CELL, int UB, int KTW, int NCW, int BT, bool SPREAD = false>
__global__ __launch_bounds__((SplitFwd<CELL, UB, KTW, NCW, BT, SPREAD>::NW * 64)) void split_fwd_kernel(const KernelParams p) {
    using C = SplitFwd<CELL, UB, KTW, NCW, BT, SPREAD>;
    extern __shared__ __align__(16) char smem[];
    const BlockMap bm(p, true);
    if (!bm.active) return;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (SPREAD || w < NCW) split_fwd_compute<CELL, UB, KTW, NCW, BT, SPREAD>(p, bm, smem, lane, w);
    else if (w < NCW + C::NLD) split_fwd_load<C>(p, bm, smem, lane);
    else split_fwd_store<C>(p, bm, smem, lane, w - NCW - C::NLD);
}

}  // namespace flashrnn
