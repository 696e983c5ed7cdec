// Instantiation lists of the persistent kernels.  Included by one translation unit per
// (cell, I/O dtype) with FRNN_CELL, FRNN_G and FRNN_BF16 defined.
//
// Shapes (KT = k-steps per wave, 32 contraction elements per bf16 step, 4 per f32 step):
//   one workgroup per group:   units D <= 32 / 64 / 128 / 192 (bf16) or 16 / 32 / 64 / 128 (f32)
//   several workgroups:        D up to 1024 (bf16) / 256 (f32) inside one XCD, optionally 4 contraction slices;
//                              D up to 2688 (bf16) spread over all XCDs: one block of 16 units and 4 contraction slices
//                              per workgroup, one wave per SIMD with up to 336 registers of R
#pragma once
#include "flashrnn_host.h"
#include "flashrnn_kernels.h"
#include "flashrnn_tile_kernels.h"
#include "flashrnn_split_kernels.h"
#include "flashrnn_recompute.h"
#include "flashrnn_step.h"

namespace flashrnn {

// staged 8-row kernels of heads of more than 128 units (a cell whose kernel does not fit the 168 registers of twelve waves defines 0)
#ifndef FRNN_LONG8_FWD
#define FRNN_LONG8_FWD 1
#endif
#ifndef FRNN_LONG8_BWD
#define FRNN_LONG8_BWD 1
#endif

#define FRNN_F(KT, KS, BT, MULTI, MAXW, EB) \
    {FRNN_CELL, FRNN_BF16, 0, KT, KS, BT, MULTI, MAXW, EB, 0, 0, (const void*)&fwd_kernel<FRNN_CELL, (FRNN_BF16 != 0), KT, KS, BT, (MULTI != 0), MAXW, EB>, 0, 0, 0, 0, 0},
#define FRNN_B(KT, KS, BT, MULTI, MAXW, EB) \
    {FRNN_CELL, FRNN_BF16, 1, (KT) * FRNN_G, KS, BT, MULTI, MAXW, EB, 0, 0, (const void*)&bwd_kernel<FRNN_CELL, (FRNN_BF16 != 0), (KT) * FRNN_G, KS, BT, (MULTI != 0), MAXW, EB>, 0, 0, 0, 0, 0},
// forward and backward share the shape list: the backward contraction axis is G times longer
#define FRNN_FB(KT, KS, BT, MULTI, MAXW) FRNN_F(KT, KS, BT, MULTI, MAXW, 1) FRNN_B(KT, KS, BT, MULTI, MAXW, 1)
// small batch tiles (bf16, one workgroup per group): forward from the dedicated tile kernel
#define FRNN_FT(KT, BT, MAXW) \
    {FRNN_CELL, FRNN_BF16, 0, KT, 1, BT, 0, MAXW, 1, 1, 0, (const void*)&fwd_tile_kernel<FRNN_CELL, KT, BT, MAXW>, 0, 0, 0, 0, 0},
// ... backward: one kernel for heads of exactly KT * 32 units (compile-time LDS layout) and one for the sizes below (two
// kernels, not two paths in one: the backward kernel sits near the register limit of its launch bound, and a spill in either
// path would disqualify both)
#define FRNN_BTL(KT, BT, MAXW) \
    {FRNN_CELL, FRNN_BF16, 1, (KT) * FRNN_G, 1, BT, 0, MAXW, 1, 1, 1, (const void*)&bwd_tile_kernel<FRNN_CELL, (KT) * FRNN_G, BT, MAXW, true>, 0, 0, 0, 0, 0}, \
    {FRNN_CELL, FRNN_BF16, 1, (KT) * FRNN_G, 1, BT, 0, MAXW, 1, 1, 0, (const void*)&bwd_tile_kernel<FRNN_CELL, (KT) * FRNN_G, BT, MAXW, false>, 0, 0, 0, 0, 0},
// ... and, for heads of up to 128 units, two more that request their inputs six steps ahead through registers
// (taken when they will come from HBM; KernelEntry::exact = 2: heads of exactly 32, 64 or 128 units, 3: the sizes below)
#define FRNN_BTLD(KT, BT, MAXW) \
    {FRNN_CELL, FRNN_BF16, 1, (KT) * FRNN_G, 1, BT, 0, MAXW, 1, 1, 2, (const void*)&bwd_tile_kernel<FRNN_CELL, (KT) * FRNN_G, BT, MAXW, true, true>, 0, 0, 0, 0, 0}, \
    {FRNN_CELL, FRNN_BF16, 1, (KT) * FRNN_G, 1, BT, 0, MAXW, 1, 1, 3, (const void*)&bwd_tile_kernel<FRNN_CELL, (KT) * FRNN_G, BT, MAXW, false, true>, 0, 0, 0, 0, 0},
#define FRNN_TILE(KT, BT, MAXW) FRNN_FT(KT, BT, MAXW) FRNN_B(KT, 1, BT, 0, MAXW, 1) FRNN_BTL(KT, BT, MAXW)
// the largest heads: one block of 16 units per workgroup, 4 contraction slices, one wave per SIMD
#define FRNN_FL(KT, BT) FRNN_F(KT, 4, BT, 1, 4, 1)
#define FRNN_BL(KT, BT) FRNN_B(KT, 4, BT, 1, 4, 1)
// EB blocks of 16 units per wave (fewer, fatter waves: the operand is read from LDS once per wave)
#define FRNN_FBE(KT, BT, MAXW, EB) FRNN_F(KT, 1, BT, 0, MAXW, EB) FRNN_B(KT, 1, BT, 0, MAXW, EB)

// heads split over the CUs of an XCD, backward with wave roles: UB blocks of 16 units per workgroup, NB output blocks per compute wave
#define FRNN_SB(UB, NB, BT, DIRECT) \
    {FRNN_CELL, FRNN_BF16, 1, 0, 1, BT, 1, SplitBwd<FRNN_CELL, UB, NB, BT, (DIRECT != 0)>::NW, 1, 0, 0, \
     (const void*)&split_bwd_kernel<FRNN_CELL, UB, NB, BT, (DIRECT != 0)>, UB, NB, DIRECT, SplitBwd<FRNN_CELL, UB, NB, BT, (DIRECT != 0)>::NBUF, SplitBwd<FRNN_CELL, UB, NB, BT, (DIRECT != 0)>::SMEM},
// ... backward in two hand-overs, KTW k-steps for each of eight compute waves
#define FRNN_SM(UB, KTW, BT) \
    {FRNN_CELL, FRNN_BF16, 1, KTW, 8, BT, 1, MeshBwd<FRNN_CELL, UB, KTW, BT>::NW, 1, 0, 0, \
     (const void*)&mesh_bwd_kernel<FRNN_CELL, UB, KTW, BT>, UB, 0, 2, 4, MeshBwd<FRNN_CELL, UB, KTW, BT>::SMEM},
// ... and forward: KTW k-steps for each of NCW compute waves
#define FRNN_SF(UB, KTW, NCW, BT) \
    {FRNN_CELL, FRNN_BF16, 0, KTW, NCW, BT, 1, SplitFwd<FRNN_CELL, UB, KTW, NCW, BT>::NW, 1, 0, 0, \
     (const void*)&split_fwd_kernel<FRNN_CELL, UB, KTW, NCW, BT>, UB, 0, 0, 4, SplitFwd<FRNN_CELL, UB, KTW, NCW, BT>::SMEM},
// ... spread over the XCDs
#define FRNN_SX(KTW, BT) \
    {FRNN_CELL, FRNN_BF16, 0, KTW, 8, BT, 1, 8, 1, 0, 0, (const void*)&split_fwd_kernel<FRNN_CELL, 1, KTW, 8, BT, true>, 1, 0, 3, 4, SplitFwd<FRNN_CELL, 1, KTW, 8, BT, true>::SMEM},

static const KernelEntry kEntries[] = {
#if FRNN_BF16
    FRNN_FB(1, 1, 16, 0, 4) FRNN_TILE(1, 8, 4) FRNN_TILE(1, 4, 4) FRNN_BTLD(1, 8, 4) FRNN_BTLD(1, 4, 4)
    FRNN_FB(2, 1, 16, 0, 4) FRNN_TILE(2, 8, 4) FRNN_TILE(2, 4, 4) FRNN_BTLD(2, 8, 4) FRNN_BTLD(2, 4, 4)
    FRNN_FB(4, 1, 16, 0, 8) FRNN_TILE(4, 8, 8) FRNN_TILE(4, 4, 8) FRNN_BTLD(4, 8, 8) FRNN_BTLD(4, 4, 8)
    FRNN_FB(6, 1, 16, 0, 12) FRNN_B(6, 1, 8, 0, 12, 1) FRNN_TILE(6, 4, 12)
#if FRNN_LONG8_FWD
    FRNN_FT(6, 8, 12)
#endif
#if FRNN_LONG8_BWD
    FRNN_BTL(6, 8, 12)
#endif
    FRNN_FBE(4, 16, 4, 2) FRNN_FBE(4, 8, 4, 2) FRNN_FBE(4, 4, 4, 2)
    FRNN_FBE(6, 16, 4, 3) FRNN_FBE(6, 8, 4, 3) FRNN_FBE(6, 4, 4, 3)
#define FRNN_MULTI_SHAPES(BT) \
    FRNN_FB(2, 1, BT, 1, 4) FRNN_FB(4, 1, BT, 1, 4) FRNN_FB(6, 1, BT, 1, 4) FRNN_FB(1, 4, BT, 1, 4) \
    FRNN_FB(8, 1, BT, 1, 8) FRNN_FB(12, 1, BT, 1, 4) FRNN_FB(16, 1, BT, 1, 4) FRNN_FB(24, 1, BT, 1, 4) \
    FRNN_FB(6, 4, BT, 1, 8) FRNN_FB(8, 4, BT, 1, 8)
    // a head split over workgroups, for batch tiles of 16, 8 and 4 rows (small tiles: more groups, less to exchange)
    FRNN_MULTI_SHAPES(16) FRNN_MULTI_SHAPES(8) FRNN_MULTI_SHAPES(4)
#undef FRNN_MULTI_SHAPES
    // (Elman: one gate's gradients in bf16 are half as much to exchange as partial sums -- 40 steps of 1 x 768 with 6 / 64 rows backward 67 / 88 us, with
    // partial sums 78 / 100, 1 x 1024 74 / 92 and 88 / 111 -- but where few members wait for their own lanes' words, or across the XCDs)
#if FRNN_G > 1
#define FRNN_SPLIT_SHAPES(BT) FRNN_SB(1, 4, BT, 0) FRNN_SB(2, 4, BT, 0) FRNN_SB(2, 6, BT, 0) FRNN_SM(2, 4, BT)
    FRNN_SPLIT_SHAPES(16) FRNN_SPLIT_SHAPES(8) FRNN_SPLIT_SHAPES(4)
#undef FRNN_SPLIT_SHAPES
#endif
    FRNN_SB(4, 5, 8, 1) FRNN_SB(4, 4, 4, 1) FRNN_SB(4, 5, 4, 1) FRNN_SB(4, 6, 4, 1)
#define FRNN_SPLIT_SHAPES(BT) FRNN_SF(1, 2, 4, BT) FRNN_SF(1, 3, 4, BT) FRNN_SF(1, 4, 4, BT) \
    FRNN_SF(2, 3, 4, BT) FRNN_SF(2, 4, 4, BT) FRNN_SF(2, 4, 6, BT)
    FRNN_SPLIT_SHAPES(16) FRNN_SPLIT_SHAPES(8) FRNN_SPLIT_SHAPES(4)
    FRNN_SF(2, 2, 4, 4) FRNN_SF(2, 6, 6, 8) FRNN_SF(2, 6, 6, 4)
    // (four blocks per workgroup at 256 units only: with 192 registers of R, heads of 320 and 384 units, fwd_kernel is 5 to 30 % faster)
    FRNN_SF(4, 2, 4, 4)
#undef FRNN_SPLIT_SHAPES
    FRNN_SM(1, 3, 8) FRNN_SM(1, 3, 4)
#if FRNN_G > 1
    FRNN_SM(1, 4, 8)
#endif
    FRNN_SX(5, 4) FRNN_SX(6, 4) FRNN_SX(8, 4) FRNN_SX(5, 8) FRNN_SX(6, 8) FRNN_SX(8, 8)
    // heads of 1040 .. 2688 units: contraction lengths 1280, 1536, 2048, 2560, 2688.  Forward with all 16 rows of a
    // batch tile where the registers allow, backward (whose point-wise phase holds more values per row) with 8 or 4;
    // the planner takes the largest tile whose kernel neither spills nor overflows the LDS.
    FRNN_FL(10, 16) FRNN_FL(12, 16) FRNN_FL(16, 16) FRNN_FL(20, 16) FRNN_FL(21, 16)
    FRNN_FL(10, 4) FRNN_FL(12, 4) FRNN_FL(16, 4) FRNN_FL(20, 4) FRNN_FL(21, 4)
    FRNN_BL(10, 8) FRNN_BL(12, 8) FRNN_BL(16, 8) FRNN_BL(20, 8) FRNN_BL(21, 8)
    FRNN_BL(10, 4) FRNN_BL(12, 4) FRNN_BL(16, 4) FRNN_BL(20, 4) FRNN_BL(21, 4)
#else
    FRNN_FB(4, 1, 16, 0, 4) FRNN_FB(8, 1, 16, 0, 4) FRNN_FB(16, 1, 16, 0, 4) FRNN_FB(32, 1, 16, 0, 8)
    // small batches: tiles of 4 and 8 rows (a quarter / half of the point-wise work and of the lane-wise traffic per workgroup)
    FRNN_FB(4, 1, 8, 0, 4) FRNN_FB(8, 1, 8, 0, 4) FRNN_FB(16, 1, 8, 0, 4) FRNN_FB(32, 1, 8, 0, 8)
    FRNN_FB(4, 1, 4, 0, 4) FRNN_FB(8, 1, 4, 0, 4) FRNN_FB(12, 1, 4, 0, 4) FRNN_FB(16, 1, 4, 0, 4) FRNN_FB(24, 1, 4, 0, 8) FRNN_FB(32, 1, 4, 0, 8)
    FRNN_FB(16, 1, 16, 1, 4) FRNN_FB(32, 1, 16, 1, 4) FRNN_FB(48, 1, 16, 1, 4) FRNN_FB(64, 1, 16, 1, 4)
    FRNN_FB(8, 4, 16, 1, 4)
    FRNN_FB(48, 1, 4, 1, 4) FRNN_FB(64, 1, 4, 1, 4)
#endif
};

#if FRNN_BF16
// one time step on its own: 1 and 4 rows per workgroup
#define FRNN_ST(RB) {FRNN_CELL, FRNN_BF16, 0, 0, 1, RB, 0, 4, 1, 1, 0, (const void*)&step_kernel<FRNN_CELL, RB>, 0, 0, 0, 0, 0},
static const KernelEntry kStep[] = {FRNN_ST(1) FRNN_ST(4)};
#undef FRNN_ST
#else
static const KernelEntry* const kStep = nullptr;
#endif

inline KernelTable make_table() {
    return KernelTable{kEntries, (int)(sizeof(kEntries) / sizeof(kEntries[0])), (const void*)&recompute_records_kernel<FRNN_CELL, (FRNN_BF16 != 0)>, kStep};
}

#undef FRNN_F
#undef FRNN_B
#undef FRNN_FB
#undef FRNN_FBE
#undef FRNN_FL
#undef FRNN_SB
#undef FRNN_SF
#undef FRNN_SM
#undef FRNN_SX
#undef FRNN_BL
#undef FRNN_FT
#undef FRNN_BTL
#undef FRNN_BTLD
#undef FRNN_TILE

}  // namespace flashrnn
