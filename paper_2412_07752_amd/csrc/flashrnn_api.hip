// C ABI of the library (see include/flashrnn.h): argument checks, launch planning, workspace carving
// and the launches.  No device memory is allocated here.
#include "flashrnn.h"

#include <hip/hip_ext.h>

#include <stdlib.h>
#include <string.h>

#include <mutex>
#include <map>
#include <set>

#include "flashrnn_common.h"
#include "flashrnn_host.h"
#include "flashrnn_recompute.h"
#include "flashrnn_split_kernels.h"

using namespace flashrnn;

namespace {

constexpr int kXcds = 8;            // accelerator dies a workgroup index cycles through
constexpr size_t kAlign = 256;

inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
inline int num_states(int cell) { return cell == FLASHRNN_LSTM ? 2 : cell == FLASHRNN_GRU ? 1 : cell == FLASHRNN_SLSTM ? 4 : cell == FLASHRNN_ELMAN ? 1 : cell == FLASHRNN_GRU4 ? 1 : -1; }
inline int num_gates(int cell) { return cell == FLASHRNN_LSTM ? 4 : cell == FLASHRNN_GRU ? 3 : cell == FLASHRNN_SLSTM ? 4 : cell == FLASHRNN_ELMAN ? 1 : cell == FLASHRNN_GRU4 ? 4 : -1; }
inline int num_cached(int cell) { return cell == FLASHRNN_SLSTM ? 5 : 4; }
inline size_t io_size(int dt) { return dt == FLASHRNN_BF16 ? 2 : 4; }

// The planner's override variables (FLASHRNN_MULTI, _BT, ...) and FLASHRNN_SPIN_LIMIT exist for the tests that force
// every kernel family onto small shapes.  They are looked at only when FLASHRNN_PLAN_OVERRIDES=1 was in the
// environment at the library's first call; otherwise no call touches the environment.
bool overrides_enabled() {
    static const bool on = [] {
        const char* v = getenv("FLASHRNN_PLAN_OVERRIDES");
        return v && *v == '1';
    }();
    return on;
}
int env_int(const char* name, int dflt) {
    if (!overrides_enabled()) return dflt;
    const char* v = getenv(name);
    return (v && *v) ? atoi(v) : dflt;
}

int device_cus() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0) cus = n;
        else cus = 256;  // MI355X
    }
    return cus;
}

KernelTable table_for(int cell, int dt) {
    const bool bf = dt == FLASHRNN_BF16;
    switch (cell) {
        case FLASHRNN_LSTM: return bf ? table_lstm_bf16() : table_lstm_f32();
        case FLASHRNN_GRU: return bf ? table_gru_bf16() : table_gru_f32();
        case FLASHRNN_ELMAN: return bf ? table_elman_bf16() : table_elman_f32();
        case FLASHRNN_GRU4: return bf ? table_gru4_bf16() : table_gru4_f32();
        default: return bf ? table_slstm_bf16() : table_slstm_f32();
    }
}

struct Plan {
    const KernelEntry* e = nullptr;
    int NWU = 0, P = 0, NG = 0, GPAR = 0, grid = 0, block = 0, DK = 0, spread = 0;
    size_t smem = 0, exch_bytes = 0, rpack_bytes = 0;
};

int validate(const flashrnn_desc_t* d) {
    if (!d) return FLASHRNN_ERR_NULL;
    if (num_states(d->cell) < 0 || (d->io_dtype != FLASHRNN_F32 && d->io_dtype != FLASHRNN_BF16)) return FLASHRNN_ERR_SHAPE;
    if (d->T < 0 || d->B <= 0 || d->NH <= 0 || d->D <= 0) return FLASHRNN_ERR_SHAPE;
    if (d->recurrent_grad_clip != d->recurrent_grad_clip) return FLASHRNN_ERR_SHAPE;   // NaN
    if (d->D % 16 != 0) return FLASHRNN_ERR_UNSUPPORTED;
    // The kernels address one time step's slab of every tensor with 32-bit byte offsets below 2^31 (offsets from
    // 2^31 on mean "drop this access"): the largest slabs are the states (S f32 values per unit), the inputs (G values)
    // and the saved-values records.
    const unsigned long long units = (unsigned long long)d->B * d->NH * d->D, e = io_size(d->io_dtype);
    const unsigned long long slab_max = 0x7FFFFFFFull;
    if (units * num_states(d->cell) * 4 > slab_max || units * num_gates(d->cell) * e > slab_max || units * record_slots(d->cell) * e > slab_max)
        return FLASHRNN_ERR_UNSUPPORTED;
    return FLASHRNN_OK;
}

constexpr size_t kLdsBytes = 160 * 1024;   // LDS of one CU
constexpr int kTraceGrid = 512;            // workgroups whose per-phase clock sums a trace build keeps
constexpr size_t kTraceBytes = (size_t)kTraceGrid * kTraceWaves * kTracePhases * 8;

// true if the kernel keeps part of its registers in scratch memory (known once a device is there)
bool kernel_spills(const void* fn) {
    static std::mutex mu;
    static std::map<const void*, bool> seen;
    std::lock_guard<std::mutex> lock(mu);
    auto it = seen.find(fn);
    if (it != seen.end()) return it->second;
    hipFuncAttributes attr;
    bool spills = false;
    if (hipFuncGetAttributes(&attr, fn) == hipSuccess) spills = attr.localSizeBytes > 0;
    else (void)hipGetLastError();
    seen[fn] = spills;
    return spills;
}

// A plan whose groups are split over the CUs of one XCD takes the kernel with wave roles (flashrnn_split_kernels.h) for its batch tile, where
// there is one that needs no more rounds over the groups.
void take_split_kernel(const flashrnn_desc_t* d, int bwd, const KernelTable& tab, int cus, Plan* pl) {
    const int units16 = d->D / 16, cap = cus / kXcds, force_ub = env_int("FLASHRNN_NWU", 0), force_gpar = env_int("FLASHRNN_GPAR", 0);
    auto in_flight = [&](int P) {
        int gpar = pl->spread ? cus / P : kXcds * (cap / P);
        if (gpar > pl->NG) gpar = pl->NG;
        return force_gpar > 0 && force_gpar < gpar ? force_gpar : gpar;
    };
    const int rounds = (pl->NG + pl->GPAR - 1) / pl->GPAR;
    const int mesh = env_int("FLASHRNN_MESH", 0);   // (test hook: 1 prefers the kernels with two hand-overs)
    // Backward: where the members' words fit the lanes of the waves that wait for them, that kernel; then one hand-over of partial sums from
    // everybody to everybody; then (more than 768 units, where R leaves that kernel no registers) two hand-overs over a mesh: us per step of LSTM 1 x 1024
    // with 16 / 64 / 128 rows 1.69 / 2.07 / 4.10, and 2.61 / 4.81 / 10.4 with exchanged gate gradients; 1 x 768 1.58 / 2.00 / 3.49 and 1.56 / 1.84 / 3.17
    // in one hand-over.
    auto kind_rank = [&](const KernelEntry& e) { return e.direct == 1 ? 2 : e.direct == 2 ? (mesh == 1 ? 3 : 0) : 1; };
    const KernelEntry* best = nullptr;
    for (int i = 0; i < tab.count; ++i) {
        const KernelEntry& e = tab.entries[i];
        if (!e.ub || e.bwd != bwd || e.BT != pl->e->BT || units16 % e.ub || (force_ub && !pl->spread && e.ub != force_ub)) continue;
        const int P = units16 / e.ub;
        if (e.smem > (int)kLdsBytes || e.direct == 3) continue;
        if (bwd && e.direct == 2) {
            // (a mesh of 8 / ub subgroups; spread over the chip each XCD is one of its eight)
            if (units16 % 8 || num_gates(d->cell) * d->D * e.ub / 8 > e.KT * e.KS * 32 || (e.ub == 1) != (pl->spread != 0)) continue;
            if (!pl->spread && (d->D > 1024 || P > cap)) continue;
        } else if (pl->spread || P > cap || (bwd ? (e.direct ? P != e.nb : units16 > 8 * e.nb) : e.KT * e.KS * 32 < d->D)) {
            continue;
        }
        if ((pl->NG + in_flight(P) - 1) / in_flight(P) > rounds) continue;
        // backward the wave-direct kernels first, then the most units per workgroup, then the smallest kernel that holds the head; forward
        // the fewest units per workgroup (a step's matrix product and point-wise function shrink with them: sLSTM 3 x 256, 16 rows, 1024 steps 900 / 785 /
        // 733 us with 64 / 32 / 16), then the least padding
        const int rank = kind_rank(e), brank = best ? kind_rank(*best) : 0;
        const bool better = !best ? true : bwd ? (rank != brank ? rank > brank : e.ub != best->ub ? e.ub > best->ub : e.direct == 2 ? e.KT < best->KT : e.nb < best->nb)
                                : (e.ub != best->ub ? e.ub < best->ub : e.KT * e.KS != best->KT * best->KS ? e.KT * e.KS < best->KT * best->KS : e.KS < best->KS);
        if (better && !kernel_spills(e.fn)) best = &e;
    }
    if (!best) return;
    pl->e = best;
    pl->NWU = best->ub;
    pl->P = units16 / best->ub;
    pl->GPAR = in_flight(pl->P);
    pl->grid = (pl->spread ? pl->GPAR : (pl->GPAR + kXcds - 1) / kXcds * kXcds) * pl->P;
    pl->block = 64 * best->maxw;
    pl->DK = d->D;   // (the packed copy of R has no padding)
    pl->smem = best->smem;
    // backward a partial sum of every unit from every member, forward the rows of h
    const size_t xrow = (size_t)best->KT * best->KS * 64;   // bytes of an exchanged row
    if (best->direct == 2) pl->exch_bytes = (size_t)best->nbuf * pl->GPAR * (8 / best->ub) * (best->BT * xrow + (size_t)pl->P * best->ub * best->BT * 64);
    else pl->exch_bytes = (size_t)best->nbuf * (bwd ? (size_t)pl->GPAR * pl->P * units16 * best->BT * 64 + kTrash : (size_t)pl->GPAR * best->BT * xrow);
}

// The forward pass of a head spread over the chip: the kernel whose members fetch h from memory once per XCD, with the smallest batch tile whose groups
// all run at once.  (Groups in rounds, and 16-row tiles, stay with fwd_kernel: LSTM 1 x 2048, 32 rows 4.66 us per step in 16-row tiles there, 6.5 here.)
void take_spread_fwd_kernel(const flashrnn_desc_t* d, const KernelTable& tab, int cus, Plan* pl) {
    const int units16 = d->D / 16, force_bt = env_int("FLASHRNN_BT", 0), force_gpar = env_int("FLASHRNN_GPAR", 0);
    if (units16 % kXcds) return;
    const size_t rpack = (size_t)d->NH * num_gates(d->cell) * d->D * 2;
    for (int BT = 4; BT <= 8; BT *= 2) {
        const KernelEntry* best = nullptr;
        for (int i = 0; i < tab.count; ++i) {
            const KernelEntry& e = tab.entries[i];
            if (e.ub && !e.bwd && e.direct == 3 && e.BT == BT && e.KT * e.KS * 32 >= d->D && e.smem <= (int)kLdsBytes && !kernel_spills(e.fn) && (!best || e.KT < best->KT)) best = &e;
        }
        if (!best || (force_bt && BT != force_bt)) continue;
        const int NG = d->NH * ((d->B + BT - 1) / BT);
        int gpar = cus / units16 < NG ? cus / units16 : NG;
        if (force_gpar > 0 && force_gpar < gpar) gpar = force_gpar;
        else if (gpar < NG) continue;
        // (per step with 4 / 8 / 16 rows, here and with every member polling all rows in memory: LSTM 1 x 1152 2.46 / 2.56 / 2.87 us and 3.31 / 3.30 / 3.32, 1 x 2048
        // 2.68 / 2.95 / 3.38 and 4.72; GRU 1 x 1280 2.40 / 2.51 / 2.93 and 2.85, Elman 2.03 / 2.16 / 2.51 and 2.37: two groups of the smaller cells stay)
        if (num_gates(d->cell) < 4 && d->D <= 1280 && NG > 1 && !force_gpar) continue;
        const size_t exch = (size_t)best->nbuf * gpar * BT * best->KT * best->KS * 64 * (1 + kXcds);   // rows of h: common ones, and each XCD's own
        // (a call that the library's own scratch array can hold stays within it)
        const size_t scratch = FLASHRNN_STATIC_SCRATCH_BYTES, fixed = rpack * d->D + kAlign;
        if (fixed + align_up(exch) > scratch && kAlign + align_up(pl->exch_bytes) + rpack * pl->DK <= scratch) continue;
        pl->e = best; pl->NWU = 1; pl->P = units16; pl->NG = NG; pl->GPAR = gpar; pl->grid = gpar * units16; pl->block = 64 * best->maxw; pl->DK = d->D; pl->smem = best->smem;
        pl->exch_bytes = exch;
        return;
    }
}

// Launch plan.  One workgroup per group whenever the head's R fits one CU's registers with 16 units
// per wave (no cross-CU traffic at all); then small batch tiles spread the point-wise work over more
// CUs.  Otherwise a group is split over P workgroups of one XCD that exchange h / dg every step.
// mode 0: forward call that saves its values, 1: backward call, 2: forward call that saves nothing.
int make_plan(const flashrnn_desc_t* d, int mode, Plan* out) {
    const int bwd = mode == 1 ? 1 : 0;
    const int G = num_gates(d->cell);
    const bool bf = d->io_dtype == FLASHRNN_BF16;
    const int kstep = bf ? 32 : 4;
    const int kdim = bwd ? G * d->D : d->D;
    const int units16 = d->D / 16;
    const KernelTable tab = table_for(d->cell, d->io_dtype);
    const int cus = device_cus();
    const int force_multi = env_int("FLASHRNN_MULTI", -1);   // 1: always split groups, 0: never, 2: always spread over all XCDs
    const int force_bt = env_int("FLASHRNN_BT", 0);
    const int force_nwu = env_int("FLASHRNN_NWU", 0);
    const int force_ks = env_int("FLASHRNN_KS", 0);
    const int force_gpar = env_int("FLASHRNN_GPAR", 0);
    const int force_kind = env_int("FLASHRNN_KIND", -1);     // kernel family (KernelEntry::tile)
    const int force_eb = env_int("FLASHRNN_EB", 0);          // blocks of 16 units per wave (one workgroup per group)      // groups in flight when groups are split (testing the group loop)
    Plan pl;
    // What the backward pass reads and writes per (t, row, unit): saved values, states, dH, dWx.  Beyond the last-level cache
    // (256 MB; the forward pass has just written most of it) its inputs come from HBM, and small heads take the kernels that fetch deeper.
    const double bwd_bytes = ((double)record_slots(d->cell) * io_size(d->io_dtype) + (double)num_states(d->cell) * 4 + (double)(1 + G) * io_size(d->io_dtype)) *
                             (double)d->T * d->B * d->NH * d->D;
    // (measured at 12 x 64, T = 1024: up to 165 MB -- LSTM with 8 rows, sLSTM with 5 -- the direct loads are 10 % faster, from
    // 184 MB on -- LSTM with 9 rows -- the deep fetch is)
    const int deep_mode = bwd ? env_int("FLASHRNN_DEEP_FETCH", bwd_bytes > 172.0 * 1024 * 1024 ? 1 : 0) : 0;   // (2: also where the rules below exclude it)
    const bool deep = deep_mode != 0;

    if (force_multi < 1) {
        // Every (batch tile, kernel) pair that can run the shape gets a cost: rounds of workgroups over the CUs
        // times a relative time per step.  The relative times are measured ones (D = 192 and 128, MI355X): the
        // staged tile kernels run a step of 4 rows in 1.0, of 8 rows in 1.45 to 2.7 (below); the generic kernels, whose
        // lanes access global memory themselves, need about 1.8 / 3.0 / 6.0 for 4 / 8 / 16 rows.  A kernel that
        // spills registers or whose images do not fit the LDS is not a candidate.
        const KernelEntry* best = nullptr;
        double best_cost = 0.0;
        size_t best_smem = 0;
        for (int i = 0; i < tab.count; ++i) {
            const KernelEntry& e = tab.entries[i];
            if (e.bwd != bwd || e.multi || e.ub || e.KS != 1) continue;
            if (force_bt && e.BT != force_bt) continue;
            if (e.KT * kstep < kdim || units16 % e.eb != 0 || e.maxw * e.eb < units16) continue;
            if (force_eb ? e.eb != force_eb : false) continue;
            if (force_kind >= 0 && e.tile != force_kind) continue;
            const int dk = e.KT * kstep, nw = units16 / e.eb;
            const bool exact_only = e.exact == 1 || e.exact == 2;
            if (exact_only && dk != kdim) continue;
            if (e.exact >= 2 && !deep) continue;
            // (heads of 128 units: the deeper fetch pays only once half of the CUs stream -- GRU 8 x 128 with 64 rows backward
            // -6 %, LSTM 6 x 128 with 128 rows -5 %, with 16 rows +10 %)
            if (e.exact >= 2 && deep_mode != 2 && e.maxw > 4 && d->NH * ((d->B + e.BT - 1) / e.BT) < cus / 2) continue;
            // (three and more workgroups per CU: they hide each other's latency and the call runs at the bandwidth of HBM; the
            // direct loads are then 4 to 9 % faster -- 12 x 64 with 512 rows.  Workgroups of one or two waves do so once a time step's saved
            // values exceed 1 MB: LSTM 48 x 16, 512 steps backward with 42 / 85 / 128 rows 242 / 429 / 627 us deep and 406 / 545 / 630 direct, 48 x 32
            // with 64 / 85 rows 428 / 622 and 525 / 562, sLSTM 48 x 32 with 32 / 53 rows 288 / 488 and 422 / 496)
            const bool many = nw <= 2 ? (size_t)d->B * d->NH * d->D * record_slots(d->cell) * 2 > 1000000 : d->NH * ((d->B + e.BT - 1) / e.BT) > 2 * cus;
            if (e.exact >= 2 && deep_mode != 2 && many) continue;
            size_t smem = (size_t)2 * e.BT * (dk + (bf ? 8 : 4)) * (bf ? 2 : 4);
            if (e.tile == 1 && bwd) {
                const int nsb = d->cell == FLASHRNN_SLSTM ? 2 : d->cell == FLASHRNN_ELMAN ? 0 : 1, go = d->cell == FLASHRNN_GRU ? G + 1 : G;
                smem = tile_lds_bwd(e.BT, go, nsb, d->D, dk * 2, record_slots(d->cell) * 2).total;
            } else if (e.tile == 1) {
                smem = tile_lds(e.BT, G, num_states(d->cell), d->D, 64 * nw, dk * 2).total_fwd;
            }
            if (smem > kLdsBytes) continue;
            if (e.tile == 1 && kernel_spills(e.fn)) continue;
            const int ng = d->NH * ((d->B + e.BT - 1) / e.BT);
            // Rounds of workgroups over the CUs.  Small staged workgroups (4 rows, at most 4 waves) share a CU, two and three at a
            // time, and overlap each other's waits: with more groups than CUs their time grows by 0.62 per CU-load of groups, not by
            // whole rounds (forward 12 x 64: 1.38 of a single round's time at 1.125 groups per CU, 1.55 at 1.5, 2.6 at 3).
            const double per_cu = (double)ng / cus;
            // With one or two waves each, several fit on the CU's four SIMDs and the time grows less, until the CU is full (LSTM 48 x 16, 512 steps
            // without saved values with 16 / 32 / 42 / 64 / 85 / 128 rows 112 / 116 / 117 / 160 / 236 / 328 us, 48 x 32 126 / 162 / 165 / 211 / 313 / 424).
            double rounds = (double)((ng + cus - 1) / cus);
            if (e.tile == 1 && e.BT == 4 && nw <= 4 && ng > cus) {
                rounds = nw > 2 ? 0.7 + 0.62 * per_cu : 0.8 + 0.4 * per_cu;
                if (nw <= 2 && rounds < 0.77 * per_cu) rounds = 0.77 * per_cu;
            }
            // (8-row staged tiles, measured at 12 x 64 with 96 to 256 rows: backward 1.3 of a 4-row step, forward 1.65 --
            // 1.25 when the call saves nothing and writes a third of the bytes: 1.48 in one round, 1.12 per round in two.  Heads of 16 and 32 units 1.5 without saved values
            // and backward: 48 x 16 with 24 rows 175 and 258 us against 115 and 208 in 4-row tiles, 48 x 32 with 32 rows 181 and 293 against 162 and 270)
            double rel8 = bwd ? 1.3 : (mode == 2 ? 1.25 : 1.65);
            if (nw <= 2 && mode != 0) rel8 = 1.5;
            // The sLSTM's forward step, whose point-wise function is the longest, 1.5: better than a second 4-row round from 80 units on (12 x 80, 64 steps,
            // 96 rows 57 us against 71 with and without saved values, 12 x 112 without them 59 and 75), until the call streams so much that many small
            // workgroups, with more requests in flight, win again (12 x 80, 256 steps, 100 rows with saved values 313 us against 291,
            // 12 x 112, 128 steps without them 154 and 140).  Heads of 48 and 64 units share a CU in 4-row tiles: with saved values these are slower from 1.05
            // to 1.1 workgroups per CU on (12 x 64, 64 steps, 96 rows 41.4 us against 36.7, 12 x 48 38.2 and 35.8), but for the shortest sequences (12 x 48, 16 steps,
            // 100 rows 13.5 and 15.0), and always better without them (12 x 64, 64 steps, 128 rows 33.8 and 36.8).
            if (d->cell == FLASHRNN_SLSTM && !bwd) {
                const double mb = (double)(G * 2 + 4 * 4 + (mode == 0 ? record_slots(d->cell) * 2 : 0)) * d->T * d->B * d->NH * d->D / 1e6;
                rel8 = 2.7;
                if (nw > 4 && (mode == 0 ? mb < 320 : nw <= 6 || mb < 300)) rel8 = 1.52;
                else if (nw > 2 && nw <= 4 && mode == 0 && mb > 140 && mb < 320) rel8 = nw == 3 ? 1.38 : 1.33;
            }
            // float32: the 4-row kernels, which waste nothing of the 4 x 4 matrix instruction, beat 8 rows everywhere (16 heads, 24 steps, 64 / 128 / 192 rows: LSTM of 64
            // units forward 21 / 30 / 41 us in 4-row and 49 / 50 / 77 in 8-row tiles, backward 43 / 63 / 83 and 62 / 74 / 114; sLSTM of 128
            // units backward, 24 steps with 66 / 96 / 128 rows 146 / 158 / 185 and 177 / 190 / 222, four-gate GRU 136 / 147 / 175 and 163 / 176 / 197).
            // Where workgroups share a CU -- up to four waves, or the few registers of one gate -- also one of 16 rows, up to eight to the CU (LSTM 16 x 32 with 256 rows
            // forward 25 us and 41, 16 x 64 51 and 62, Elman 16 x 128 48 and 57); whole rounds of larger heads lose to it from four on (LSTM 16 x 96 with 256 rows
            // 151 / 254 us and 143 / 240, 16 x 128 166 / 341 and 163 / 298), but for the sLSTM (16 x 96 179 / 256 and 194 / 283, 16 x 128 202 / 352 and 219 / 388).
            double rel = e.tile == 1 ? (e.BT == 4 ? 1.0 : rel8) : (e.BT == 4 ? 1.8 : e.BT == 8 ? 3.0 : 6.0);
            if (!bf) {
                const bool shares = nw <= 4 || G == 1;
                rounds = e.BT == 4 && G == 3 && !bwd && ng > cus ? per_cu : rounds;   // (two workgroups to a CU: the last round need not be a whole one)
                rel = e.BT == 4 ? 1.0 : e.BT == 8 ? 2.9 : nw <= 2 ? 2.4 : nw <= 4 ? 2.8 : G == 1 ? (bwd ? 2.2 : 3.0) : d->cell == FLASHRNN_SLSTM ? 4.3 : 3.3;
                if (e.BT == 4 && shares && ng > cus) {
                    rounds = nw <= 2 ? 0.9 + 0.2 * per_cu : 0.9 + 0.35 * per_cu;
                    const double full = bwd ? 0.75 * per_cu - 0.25 : 0.66 * per_cu;
                    if (nw > 2 && G > 1 && rounds < full) rounds = full;
                }
            }
            if (e.tile == 0) rel *= 1.0 + 0.05 * (e.eb - 1);       // thin waves overlap better
            rel *= bf ? 1.0 + 0.02 * (dk - kdim) / (double)kstep : 1.0 + 0.3 * (dk - kdim) / (double)dk;   // padded k-steps are wasted MFMAs
            if (exact_only) rel *= 0.99;                           // compile-time LDS layout: fewer address instructions
            if (e.exact >= 2) rel *= 0.9;                          // (only a candidate when the inputs come from HBM: -10 % there)
            const double cost = rounds * rel;
            if (!best || cost < best_cost) { best = &e; best_cost = cost; best_smem = smem; }
        }
        if (best) {
            pl.e = best;
            pl.NWU = units16 / best->eb;
            pl.P = 1;
            pl.NG = d->NH * ((d->B + best->BT - 1) / best->BT);
            pl.GPAR = pl.NG;
            pl.grid = pl.NG;
            pl.block = 64 * pl.NWU;
            pl.DK = best->KT * kstep;
            pl.smem = best_smem;
            pl.exch_bytes = 0;
        }
    }
    if (!pl.e && force_multi != 0 && force_multi != 2) {
        // Batch tiles of 16, 8 or 4 rows here too.  A smaller tile means more groups (each with its own workgroups, on its
        // own XCD when there are few) and proportionally less to exchange and less point-wise work per workgroup; the
        // smallest tile whose groups all run at once is taken, else the largest (fewest rounds over the groups) -- of those that come into question.
        const int want_ks = force_ks ? force_ks : (d->D >= 512 ? 4 : 1);
        auto entry_of = [&](int BT) {
            const KernelEntry* best = nullptr;
            for (int spills_ok = 0; spills_ok < 2 && !best; ++spills_ok)   // a kernel that keeps registers in scratch memory only as a last resort
            for (int i = 0; i < tab.count; ++i) {
                const KernelEntry& e = tab.entries[i];
                const int dk = e.KT * e.KS * kstep;
                if (e.bwd != bwd || !e.multi || e.ub || e.BT != BT || dk < kdim) continue;
                if (e.maxw == 4 && e.KS == 4 && e.KT * (bwd ? 1 : G) >= 40) continue;   // the shapes of the spread placement
                if (!spills_ok && kernel_spills(e.fn)) continue;
                // least padding of the contraction axis first, then the wanted number of slices, then the most waves
                const int bdk = best ? best->KT * best->KS * kstep : 0;
                const bool want = e.KS == want_ks, bwant = best && best->KS == want_ks;
                if (!best || dk < bdk || (dk == bdk && (want > bwant || (want == bwant && e.maxw > best->maxw)))) best = &e;
            }
            return best;
        };
        const int bts[3] = {4, 8, 16};
        // Only tiles whose kernels let a group run on the fewest workgroups: where the registers of a larger tile allow
        // four waves per workgroup instead of eight, each group of it takes twice the CUs, and a smaller tile in more rounds is faster (heads of 256
        // units: sLSTM 8 x 256, 256 steps backward, 128 rows 1618 us with 16-row tiles on 4 CUs, 1152 in two rounds of 4-row tiles on 2;
        // LSTM 8 x 256, 128 steps, 256 rows 1485 and, with 8-row tiles, 885; sLSTM forward 1037 and 774).
        // The sLSTM's backward pass holds the most values per row: one round of 16-row tiles is slower there than two of 8-row tiles at every size
        // (128 steps, 4 x 384 with 256 rows 1912 and 1760 us, 4 x 512 with 128 rows 1100 and 977, 1 x 768 1448 and 1208, 2 x 1024 with 64 rows
        // 2083 and 1833; LSTM 1 x 768 with 128 rows 1012 and 1186, GRU 3 x 640 with 80 rows 1280 and 1628, hence for this cell only).
        int usable[3], fewest = 0;
        for (int bi = 0; bi < 3; ++bi) {
            const KernelEntry* e = entry_of(bts[bi]);
            int nwu = e ? e->maxw / e->KS : 0;
            while (nwu > 1 && units16 % nwu) --nwu;
            usable[bi] = nwu > 0 ? units16 / nwu : 0;   // workgroups of a group
            if (usable[bi] && (!fewest || usable[bi] < fewest)) fewest = usable[bi];
        }
        for (int bi = 0; bi < 3; ++bi) usable[bi] = usable[bi] && (!bf || usable[bi] == fewest);   // (float32: not measured)
        if (bf && bwd && d->cell == FLASHRNN_SLSTM && (usable[0] || usable[1])) usable[2] = 0;
        for (int pass = 0; pass < 2 && !pl.e; ++pass) {
            for (int bi = 0; bi < 3 && !pl.e; ++bi) {
                const int BT = pass == 0 ? bts[bi] : bts[2 - bi];
                if (force_bt ? BT != force_bt : !usable[pass == 0 ? bi : 2 - bi]) continue;
                // workgroups of one launch per XCD: all members of a group must be resident at once, at most one per CU
                // where a workgroup takes all registers of its CU.  (A head of 1024 units asks for every CU of an XCD, in both
                // directions: with two CUs kept back the backward pass of such a head fell to one group of 16 rows at 13 us a step.)
                int cap = cus / kXcds;
                const int NG = d->NH * ((d->B + BT - 1) / BT);
                const KernelEntry* best = entry_of(BT);
                if (!best) continue;
                const int nwu_max = best->maxw / best->KS;
                // most workgroups per group (shortest MFMA and point-wise phase per step) that still lets
                // every group run at once; fall back to looping over groups
                const int slots = (NG + kXcds - 1) / kXcds;       // groups per XCD if all run at once
                int chosen = 0;
                // (at least four waves per workgroup where the shape allows: the workgroup polls the group's rows
                // together, and with fewer threads that takes more rounds - measured on D = 256 and 768)
                const int nwu_min = 4 / best->KS > 1 ? 4 / best->KS : 1;
                // Forward: the most workgroups per group that fit (shortest MFMA and point-wise phase; its rows are short to poll).
                // Backward: the fewest -- its exchanged rows are G times longer, and a workgroup with more threads strips them
                // in fewer rounds (measured at D = 256: forward 1.27 / 1.36 / 1.74 ms with 8 / 4 / 2 workgroups per group,
                // backward 2.70 / 2.88 / 2.38 ms).
                for (int p2 = 0; p2 < 2 && !chosen; ++p2) {
                    const int lo = p2 == 0 ? nwu_min : 1;
                    for (int step = 0; step <= nwu_max - lo; ++step) {
                        const int nwu = bwd && !force_nwu ? nwu_max - step : lo + step;
                        if (units16 % nwu) continue;
                        const int P = units16 / nwu;
                        if (force_nwu ? nwu == force_nwu : P * slots <= cap) { chosen = nwu; break; }
                    }
                }
                int gpar = NG;
                if (!chosen && pass == 0 && !force_bt) continue;      // not all groups at once with this tile: try a larger one
                if (!chosen) {
                    // even the fewest workgroups per group do not fit all groups: loop over groups
                    for (int nwu = nwu_max; nwu >= 1 && !chosen; --nwu)
                        if (units16 % nwu == 0 && units16 / nwu <= cap) chosen = nwu;
                    if (!chosen && units16 % nwu_max == 0 && units16 / nwu_max <= cus / kXcds) {
                        // the largest heads need every CU of an XCD for one group (no margin: should a CU be taken, the
                        // waits run into their spin limit and the call reports a timeout)
                        chosen = nwu_max;
                        cap = cus / kXcds;
                    }
                    if (chosen) gpar = kXcds * (cap / (units16 / chosen));
                    if (gpar > NG) gpar = NG;
                }
                if (chosen && force_gpar > 0 && force_gpar < gpar) gpar = force_gpar;
                if (chosen) {
                    pl.e = best;
                    pl.NWU = chosen;
                    pl.P = units16 / chosen;
                    pl.NG = NG;
                    pl.GPAR = gpar;
                    pl.grid = (gpar + kXcds - 1) / kXcds * pl.P * kXcds;
                    pl.block = 64 * chosen * best->KS;
                    pl.DK = best->KT * best->KS * kstep;
                    const int nt = bwd ? 1 : G;
                    // one buffer of BT operand rows (polled once per workgroup and step), then the partial sums of the slices
                    pl.smem = (size_t)BT * (pl.DK + operand_pad(bf, bf && BT < 16)) * (bf ? 2 : 4) + (best->KS > 1 ? (size_t)2 * (best->KS - 1) * chosen * nt * 4 * 64 * 4 : 16);
                    pl.exch_bytes = (size_t)4 * gpar * BT * pl.DK * (bf ? 2 : 4);   // four buffers
                }
            }
        }
    }
    const int split_mode = env_int("FLASHRNN_SPLIT", 1);   // (test hook: 0 no kernels with wave roles, 2 nothing else forward, 3 nothing else backward)
    if (pl.e && pl.e->multi && bf && split_mode != 0) take_split_kernel(d, bwd, tab, cus, &pl);
    if (!pl.e && force_multi != 0 && bf) {
        // Heads beyond what the CUs of one XCD can hold (D > 1024): the group is spread over the CUs of all XCDs, one
        // block of 16 units and 4 contraction slices per workgroup (one wave per SIMD, up to 336 registers of R each),
        // and h / dg cross the XCDs through memory.  The largest batch tile whose kernel neither spills registers nor
        // overflows the LDS; as many groups at once as fit the chip, the rest in turn.  (No CUs are kept back: a head of 2048
        // units takes 128 of them, and two of its groups side by side halve the backward pass.)
        const int budget = cus;
        const int bts[3] = {16, 8, 4};
        for (int spills_ok = 0; spills_ok < 2 && !pl.e; ++spills_ok)   // (a kernel with a few registers in scratch memory only if no tile is free of them)
        for (int bi = 0; bi < 3 && !pl.e; ++bi) {
            const int BT = bts[bi];
            if (force_bt && BT != force_bt) continue;
            const KernelEntry* best = nullptr;
            for (int i = 0; i < tab.count; ++i) {
                const KernelEntry& e = tab.entries[i];
                const int dk = e.KT * e.KS * kstep;
                if (e.bwd != bwd || !e.multi || e.ub || e.BT != BT || e.KS != 4 || e.maxw != 4 || dk < kdim) continue;
                if (!best || dk < best->KT * best->KS * kstep) best = &e;
            }
            if (!best || units16 > budget) continue;
            const int dk = best->KT * best->KS * kstep, nt = bwd ? 1 : G;
            const size_t smem = (size_t)BT * (dk + operand_pad(true, BT < 16)) * 2 + (size_t)2 * 3 * nt * 4 * 64 * 4;
            if (smem > kLdsBytes || (!spills_ok && kernel_spills(best->fn))) continue;
            const int NG = d->NH * ((d->B + BT - 1) / BT);
            int gpar = budget / units16;
            if (gpar > NG) gpar = NG;
            if (force_gpar > 0 && force_gpar < gpar) gpar = force_gpar;
            pl.e = best;
            pl.NWU = 1;
            pl.P = units16;
            pl.NG = NG;
            pl.GPAR = gpar;
            pl.grid = gpar * pl.P;
            pl.block = 64 * 4;
            pl.DK = dk;
            pl.smem = smem;
            pl.exch_bytes = (size_t)4 * gpar * BT * dk * 2;
            pl.spread = 1;
        }
    }
    if (pl.spread && split_mode != 0) {
        if (bwd) take_split_kernel(d, bwd, tab, cus, &pl);
        else take_spread_fwd_kernel(d, tab, cus, &pl);
    }
    if (!pl.e || (split_mode == (bwd ? 3 : 2) && !pl.e->ub)) return FLASHRNN_ERR_UNSUPPORTED;
    pl.rpack_bytes = pl.e->ub && bwd ? 0 : (bwd ? (size_t)d->NH * d->D * pl.DK : (size_t)d->NH * G * d->D * pl.DK) * io_size(d->io_dtype);
    *out = pl;
    return FLASHRNN_OK;
}

// Calls of one time step in bf16 run on a kernel of their own, but for small heads with more than one row and for the larger batches, whose rows share
// what the persistent kernels read of R (us per call, persistent and step: 12 x 64 with 1 / 16 rows 3.7 / 3.8 and 3.1 / 4.4; 8 x 128 with 16 rows 4.9 and 4.3;
// 4 x 192 with 1 / 32 / 128 rows 8.6 / 8.5 / 9.9 and 4.1 / 6.5 / 13.4; 1 x 768 with 1 / 64 / 256 rows 30 / 31 / 46 and 6.9 / 17 / 54).
bool make_step_plan(const flashrnn_desc_t* d, Plan* pl) {
    const KernelEntry* step = table_for(d->cell, d->io_dtype).step;
    if (d->T != 1 || !step || env_int("FLASHRNN_KIND", -1) >= 0 || env_int("FLASHRNN_STEP", 1) == 0) return false;   // (tests of the other kernels)
    const KernelEntry& e = step[d->B == 1 ? 0 : 1];
    const long long tiles = (d->B + e.BT - 1) / e.BT, grid = tiles * d->NH * (d->D / 16);
    if (d->B > 1 && tiles > (d->D <= 64 ? 0 : d->D <= 128 ? 4 : d->D <= 192 ? 8 : 16)) return false;
    // (Every batch tile reads R once more, which the persistent kernels do not: with many heads or rows that is what a call takes.  sLSTM, us step / persistent, and
    // MB that the tiles read: 64 x 80 with 4 / 16 rows 5.5 / 5.6 (3) and 9.7 / 6.0 (13); 24 x 192 with 4 / 32 rows 8.1 / 8.6 (7) and 23.0 / 11.1 (57); 24 x 256 with 8 / 16 / 32
    // rows 14.1 / 21.8 (25), 26.1 / 29.3 (50) and 48.2 / 31.2 (101); 12 x 512 with 8 / 16 rows 23.6 / 31.8 (50) and 43.9 / 31.7 (101); 4 x 1024 with 8 / 32 / 64 rows 23.5 / 35.1
    // (67), 79 / 35 (268) and 196 / 51 (537); one row 64 x 128 5.7 / 5.9 (8.4) and 96 x 128 10.3 / 6.0 (13).  Elman, whose persistent kernels have a gate's work only: 24 x 128 with
    // 2 / 8 rows 3.3 / 3.5 (0.8) and 3.8 / 3.5 (1.6), 32 x 192 3.8 / 4.1 (2.4) and 4.4 / 4.3 (4.7), 24 x 384 with 8 / 12 rows 8.5 / 11.6 (14) and 12.2 / 11.5 (21).)
    const double mb = (double)tiles * d->NH * num_gates(d->cell) * d->D * d->D * 2 / 1e6;
    const int size = d->D <= 128 ? 0 : d->D <= 192 ? 1 : d->D <= 256 ? 2 : d->D <= 512 ? 3 : 4;
    static const double most[3][5] = {{8.5, 9.5, 76, 76, 76}, {4.5, 7.5, 25.2, 50.4, 75.6}, {1.1, 2.5, 16, 18, 26}};   // one row; more; more, one gate
    if (mb > most[d->B == 1 ? 0 : num_gates(d->cell) > 1 ? 1 : 2][size]) return false;
    if (grid > 1 << 20) return false;
    Plan s;
    s.e = &e;
    s.NWU = 1; s.P = d->D / 16; s.NG = (int)(tiles * d->NH); s.GPAR = s.NG; s.grid = (int)grid; s.block = 256;
    *pl = s;
    return true;
}

struct Workspace {
    size_t err_off, exch_off, rpack_off[2] /* forward, backward */, dgn_off, dbpart_off, drpart_off, trace_off, total;
    size_t fwd_total;   // bytes a forward call touches: error words, exchange buffers, the forward copy of R
};

// The plans of a descriptor's calls.
struct Plans {
    Plan fwd, bwd, infer;   // forward call that saves its values, backward call, forward call that saves nothing
    Plan step;              // forward calls of one step whose states do not overlap the initial ones (e == nullptr: they run the plans above)
};

int carve_uncached(const flashrnn_desc_t* d, Workspace* w, Plans* pl) {
    Plan *const pf = &pl->fwd, *const pb = &pl->bwd, *const pfn = &pl->infer;
    int rc = make_plan(d, 0, pf);
    if (rc != FLASHRNN_OK) return rc;
    rc = make_plan(d, 1, pb);
    if (rc != FLASHRNN_OK) return rc;
    // A forward call that saves nothing may take another batch tile of the staged kernels (they use no workspace beyond the
    // error words, so the layout below does not depend on it); everywhere else it runs the plan of the saving call.
    if (make_plan(d, 2, pfn) != FLASHRNN_OK || pfn->e->tile == 0 || pf->e->tile == 0) *pfn = *pf;
    // (a call of one step uses nothing of the layout below but the error words)
    make_step_plan(d, &pl->step);
    const int G = num_gates(d->cell);
    size_t off = 0;
    w->err_off = off; off += kAlign;   // word 0: forward kernels, word 1: backward kernels
    // exchange buffers and packed R of a call: the two directions use the same memory, each with a split of its own
    w->exch_off = off;
    w->rpack_off[0] = off + align_up(pf->exch_bytes);
    w->rpack_off[1] = off + align_up(pb->exch_bytes);
    w->fwd_total = w->rpack_off[0] + align_up(pf->rpack_bytes);
    const size_t bwd_total = w->rpack_off[1] + align_up(pb->rpack_bytes);
    off = w->fwd_total > bwd_total ? w->fwd_total : bwd_total;
    w->dgn_off = off; off += align_up(d->cell == FLASHRNN_GRU ? (size_t)d->T * d->B * d->NH * d->D * io_size(d->io_dtype) : 0);
    const int sk = dr_split_k(d->io_dtype == FLASHRNN_BF16, d->T, d->B, d->NH, d->D, G);
    // partial sums of db: one row per batch row (from the persistent kernel) or per contraction slice (from the dR GEMM)
    w->dbpart_off = off; off += align_up((size_t)(d->B > sk ? d->B : sk) * d->NH * G * d->D * 4);
    w->drpart_off = off;
    off += align_up(sk > 1 ? (size_t)sk * d->NH * d->D * G * d->D * 4 : 0);
    w->trace_off = off;
#ifdef FLASHRNN_TRACE
    off += 2 * kTraceBytes;   // forward, backward
#endif
    w->total = off;
    return FLASHRNN_OK;
}

// Plans and workspace layout of a descriptor.  A thread that calls with the same descriptor again (the usual case:
// forward, backward, forward, ...) gets the last answer back instead of planning anew; the answer depends on the
// descriptor and the device only (and on the override variables, which switch this memo off).
int carve(const flashrnn_desc_t* d, Workspace* w, Plans* pl) {
    struct Memo { bool valid = false; flashrnn_desc_t d; int dev; int rc; Workspace w; Plans pl; };
    static thread_local Memo memo;
    int dev = -1;
    (void)hipGetDevice(&dev);
    flashrnn_desc_t key = *d;
    key.recurrent_grad_clip = 0.0f;   // does not enter the plan
    if (!overrides_enabled() && memo.valid && memo.dev == dev && memcmp(&memo.d, &key, sizeof(key)) == 0) {
        *w = memo.w;
        *pl = memo.pl;
        return memo.rc;
    }
    *pl = Plans();
    const int rc = carve_uncached(d, w, pl);
    memo.valid = true; memo.d = key; memo.dev = dev; memo.rc = rc; memo.w = *w; memo.pl = *pl;
    return rc;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

int prepare_kernel(const Plan& pl) {
    static std::mutex mu;
    static std::set<const void*> done;
    std::lock_guard<std::mutex> lock(mu);
    if (done.count(pl.e->fn)) return FLASHRNN_OK;
    if (hipFuncSetAttribute(pl.e->fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) {
        (void)hipGetLastError();
        if (pl.smem > 64 * 1024) return FLASHRNN_ERR_LAUNCH;
    }
    done.insert(pl.e->fn);
    return FLASHRNN_OK;
}

// optional bracketing of the persistent kernels with HIP events (flashrnn_profile_*)
constexpr int kProfSlots = 256;
struct Profile {
    int stride = 0;            // 0 = off; n = every n-th call per direction carries events
    int seen[2] = {0, 0};
    int count[2] = {0, 0};
    hipEvent_t ev[2][kProfSlots][2] = {};
};
Profile g_prof;
std::mutex g_prof_mu;

int launch_persistent(const Plan& pl, KernelParams& kp, hipStream_t stream) {
    if (prepare_kernel(pl) != FLASHRNN_OK) return FLASHRNN_ERR_LAUNCH;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_prof_mu);
        const int dir = pl.e->bwd;
        if (g_prof.stride > 0 && g_prof.seen[dir]++ % g_prof.stride == 0 && g_prof.count[dir] < kProfSlots) {
            const int i = g_prof.count[dir]++;
            for (int j = 0; j < 2; ++j)
                if (!g_prof.ev[dir][i][j] && hipEventCreate(&g_prof.ev[dir][i][j]) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
            e0 = g_prof.ev[dir][i][0];
            e1 = g_prof.ev[dir][i][1];
        }
    }
    kp.P = pl.P;
    kp.NWU = pl.NWU;
    kp.NG = pl.NG;
    kp.GPAR = pl.GPAR;
    kp.spread = pl.spread;
    kp.spin_limit = env_int("FLASHRNN_SPIN_LIMIT", 1 << 21);
    void* args[] = {&kp};
    if (e0 && e1) {
        // the two events ride on the kernel's own dispatch (start and end time stamps of that dispatch): no extra commands
        // in the stream, so the measurement does not slow the step down
        if (hipExtLaunchKernel(pl.e->fn, dim3(pl.grid), dim3(pl.block), args, pl.smem, stream, e0, e1, 0) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
    } else if (hipLaunchKernel(pl.e->fn, dim3(pl.grid), dim3(pl.block), args, pl.smem, stream) != hipSuccess) {
        return FLASHRNN_ERR_LAUNCH;
    }
    return FLASHRNN_OK;
}

// Scratch memory of flashrnn_fwd_static_scratch: one array per GPU, part of the loaded code object (no allocation call
// ever).  Host code must not use the array's name as an address: the device address is looked up once per device, with
// that device current, and kept.
constexpr size_t kStaticScratchBytes = (size_t)FLASHRNN_STATIC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

void* static_scratch_ptr() {
    static std::mutex mu;
    static void* ptrs[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { (void)hipGetLastError(); return nullptr; }
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { (void)hipGetLastError(); return nullptr; }
        ptrs[dev] = ptr;
    }
    return ptrs[dev];
}

// Forward call on the workspace `workspace`; ws_limit > 0: the workspace is the library's own array of that size and
// only the part a forward call touches has to fit.
int fwd_impl(const flashrnn_desc_t* d, const void* Wx, const void* R, const void* b, const void* states0, void* states,
             void* gate_cache, void* workspace, size_t ws_limit, void* hip_stream) {
    int rc = validate(d);
    if (rc != FLASHRNN_OK) return rc;
    if (!R || !b || !states || (d->T > 0 && !Wx)) return FLASHRNN_ERR_NULL;
    if (!aligned16(Wx) || !aligned16(R) || !aligned16(b) || !aligned16(states0) || !aligned16(states) || !aligned16(gate_cache))
        return FLASHRNN_ERR_UNSUPPORTED;
    Workspace w;
    Plans pl;
    rc = carve(d, &w, &pl);
    if (rc != FLASHRNN_OK) return rc;
    // The one-step kernel's workgroups read h_0 of a whole head while others write states: initial states that lie in `states` itself (but as its
    // slot 0, which gets the same values) go the way of longer sequences, where units that others own come through the exchange or were read before.
    const size_t slab = (size_t)num_states(d->cell) * d->B * d->NH * d->D * 4;
    const uintptr_t s0 = (uintptr_t)states0, out = (uintptr_t)states;
    const bool overlap = states0 && s0 != out && s0 < out + 2 * slab && out < s0 + slab;
    const Plan& pf = pl.step.e && !overlap ? pl.step : gate_cache ? pl.fwd : pl.infer;
    if (!workspace || ((uintptr_t)workspace & (kAlign - 1))) return FLASHRNN_ERR_WORKSPACE;
    if (ws_limit && w.fwd_total > ws_limit) return FLASHRNN_ERR_SCRATCH;
    hipStream_t stream = (hipStream_t)hip_stream;
    char* ws = (char*)workspace;
    const int G = num_gates(d->cell);
    // the exchange buffers start empty (a fill kernel, not a memset: the call may be captured into a graph);
    // both error words are cleared by the packing kernel
    if (pf.exch_bytes && launch_fill(ws + w.exch_off, align_up(pf.exch_bytes), kNoWord, stream) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
    // (the staged forward kernels and the float32 kernels of 4-row tiles on one CU read R as it is and clear the error words themselves)
    const bool r_in_place = pf.e->tile != 0 || (d->io_dtype == FLASHRNN_F32 && pf.e->BT == 4 && !pf.e->multi);
    if (!r_in_place && launch_pack_r(d->io_dtype == FLASHRNN_BF16, false, R, ws + w.rpack_off[0], d->NH, d->D, G, pf.DK, (int*)(ws + w.err_off), stream) != hipSuccess)
        return FLASHRNN_ERR_LAUNCH;
    KernelParams kp;
    memset(&kp, 0, sizeof(kp));
    kp.Wx = Wx; kp.R = r_in_place ? R : (const void*)(ws + w.rpack_off[0]); kp.bias = b; kp.states0 = (const float*)states0; kp.states = (float*)states;
    kp.cache = gate_cache;
    kp.exch = (uint32_t*)(ws + w.exch_off);
    kp.err = (int*)(ws + w.err_off);
    kp.T = d->T; kp.B = d->B; kp.NH = d->NH; kp.D = d->D;
#ifdef FLASHRNN_TRACE
    if (!ws_limit && pf.grid <= kTraceGrid) {
        kp.trace = (unsigned long long*)(ws + w.trace_off);
        if (launch_fill_zero(kp.trace, kTraceBytes, stream) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
    }
#endif
    return launch_persistent(pf, kp, stream);
}

// Workspace of flashrnn_bwd_recompute behind the ordinary one: the records of one window of time steps and two buffers
// for the state gradients carried from window to window.  Windows as equal as whole steps allow, at most 80 MiB of records each (but at least one step): small enough to stay
// in the last-level cache between the kernel that writes them and the one that reads them.  Every window costs three launches and the backward kernel's prologue, 20 us at
// 3 x 256.  Backward with recompute within 64 / 80 / 128 MiB, us: sLSTM 3 x 256, 16 rows, 1024 steps 1115 / 1093 / 1082; LSTM 12 x 64, 64 rows, 1024 steps 862 / 824 / 818; float32 LSTM 4 x 96,
// 64 rows, 512 steps 1015 / 1029 / 991; sLSTM 8 x 256, 32 rows, 512 steps 1223 / 1225 / 1142 (and 48 MiB 1297).
struct RecomputeLayout { size_t window_off, carry_off, total; int window; };
RecomputeLayout recompute_layout(const flashrnn_desc_t* d, size_t base_total) {
    RecomputeLayout rl;
    const size_t units = (size_t)d->B * d->NH * d->D;
    const size_t rec_step = units * record_slots(d->cell) * io_size(d->io_dtype);
    const long long most = (long long)(((size_t)80 << 20) / rec_step), fits = most > 0 ? most : 1;   // steps
    const long long windows = (d->T + fits - 1) / fits;
    long long steps = windows > 0 ? (d->T + windows - 1) / windows : 1;
    const int forced = env_int("FLASHRNN_RECOMPUTE_STEPS", 0);   // (test hook: windows of this many steps)
    if (forced > 0) steps = forced;
    if (steps < 1) steps = 1;
    if (steps > d->T) steps = d->T > 0 ? d->T : 1;
    rl.window = (int)steps;
    rl.window_off = base_total;
    rl.carry_off = rl.window_off + align_up((size_t)steps * rec_step);
    rl.total = rl.carry_off + 2 * align_up((size_t)num_states(d->cell) * units * 4);
    return rl;
}

// Backward call.  Wx == nullptr: the saved values come from gate_cache (flashrnn_bwd).  Otherwise (flashrnn_bwd_recompute)
// they are formed again, a window of time steps at a time, into the window buffer behind the ordinary workspace, and the
// persistent kernel runs window by window from the last step to the first, the gradients of the carried states going from
// one launch to the next through two buffers in the workspace.
int bwd_impl(const flashrnn_desc_t* d, const void* Wx, const void* R, const void* b, const void* states, const void* gate_cache,
             const void* dH, const void* dstates_last, void* dWx, void* dR, void* db, void* dstates0, void* workspace, void* hip_stream) {
    int rc = validate(d);
    if (rc != FLASHRNN_OK) return rc;
    const bool recompute = Wx != nullptr;
    if (!R || !states || !dR || !db || !dstates0 || (d->T > 0 && ((!recompute && !gate_cache) || !dH || !dWx)) || (recompute && !b)) return FLASHRNN_ERR_NULL;
    if (!aligned16(R) || !aligned16(states) || !aligned16(gate_cache) || !aligned16(dH) || !aligned16(dstates_last) ||
        !aligned16(dWx) || !aligned16(dR) || !aligned16(db) || !aligned16(dstates0) || !aligned16(Wx) || !aligned16(b))
        return FLASHRNN_ERR_UNSUPPORTED;
    Workspace w;
    Plans pl;
    rc = carve(d, &w, &pl);
    if (rc != FLASHRNN_OK) return rc;
    const Plan& pb = pl.bwd;
    if (!workspace || ((uintptr_t)workspace & (kAlign - 1))) return FLASHRNN_ERR_WORKSPACE;
    hipStream_t stream = (hipStream_t)hip_stream;
    char* ws = (char*)workspace;
    const int G = num_gates(d->cell), S = num_states(d->cell);
    const bool bf = d->io_dtype == FLASHRNN_BF16;
    const size_t esz = io_size(d->io_dtype);
    // The backward copy of R is R itself, padded along (gate, unit) to the kernel's contraction length: without padding the kernel reads R where it
    // is, and so do the staged kernels and those with wave roles, for whose waits the first fill clears the error word (the packing kernel does for the others that wait).
    const bool r_in_place = pb.e->ub || pb.e->tile || (!pb.e->multi && pb.DK == G * d->D);
    if (!r_in_place && launch_pack_r(bf, true, R, ws + w.rpack_off[1], d->NH, d->D, G, pb.DK, (int*)(ws + w.err_off) + 1, stream) != hipSuccess)
        return FLASHRNN_ERR_LAUNCH;
    const size_t units = (size_t)d->B * d->NH * d->D;
    const size_t st_step = (size_t)S * units * 4, io_step = units * esz, rec_step = units * record_slots(d->cell) * esz;
    const RecomputeLayout rl = recompute_layout(d, w.total);
    const int window = recompute ? rl.window : (d->T > 0 ? d->T : 1);
    // windows from the last step to the first; [r0, r1) are 0-based step indices (step r turns states[r] into states[r + 1])
    for (int r1 = d->T; r1 > 0 || (r1 == 0 && d->T == 0); r1 -= window) {
        const int r0 = r1 - window > 0 ? r1 - window : 0, steps = r1 - r0;
        const bool first = r1 == d->T, last = r0 == 0;
        const void* cache = gate_cache;
        if (recompute && steps > 0) {
            RecomputeParams rp;
            rp.Wx = (const char*)Wx + (size_t)r0 * G * io_step; rp.R = R; rp.bias = b;
            rp.states = (const float*)((const char*)states + (size_t)r0 * st_step);
            rp.cache = ws + rl.window_off; rp.steps = steps; rp.B = d->B; rp.NH = d->NH; rp.D = d->D;
            void* args[] = {&rp};
            const dim3 grid((unsigned)((steps * d->B + recompute_cols(bf) - 1) / recompute_cols(bf)), (unsigned)((d->D + 63) / 64), (unsigned)d->NH);
            if (hipLaunchKernel(table_for(d->cell, d->io_dtype).recompute, grid, dim3(256), args, 0, stream) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
            cache = ws + rl.window_off;
        } else if (!recompute) {
            cache = gate_cache;
        }
        // (where no packing kernel ran, the first fill clears the error word of the waits)
        if (pb.exch_bytes && launch_fill(ws + w.exch_off, align_up(pb.exch_bytes), kNoWord, stream, r_in_place && first ? (int*)(ws + w.err_off) + 1 : nullptr) != hipSuccess)
            return FLASHRNN_ERR_LAUNCH;
        KernelParams kp;
        memset(&kp, 0, sizeof(kp));
        kp.R = r_in_place ? R : (const void*)(ws + w.rpack_off[1]);
        kp.states = (float*)((char*)const_cast<void*>(states) + (size_t)r0 * st_step);
        kp.cache = const_cast<void*>(cache);
        kp.dH = (const char*)dH + (size_t)r0 * io_step;
        kp.dWx = (char*)dWx + (size_t)r0 * G * io_step;
        kp.dgn = ws + w.dgn_off + (size_t)r0 * io_step;
        // carried state gradients: in from the caller (first launch) or from the window after this one, out to the caller
        // (last launch) or to the window before this one; the two carry buffers alternate
        const int flip = ((d->T - r1) / window) & 1;
        kp.dlast = first ? (const float*)dstates_last : (const float*)(ws + rl.carry_off + (size_t)(flip ^ 1) * align_up((size_t)S * units * 4));
        kp.dstates0 = last ? (float*)dstates0 : (float*)(ws + rl.carry_off + (size_t)flip * align_up((size_t)S * units * 4));
        kp.db_accumulate = first ? 0 : 1;
        kp.clip = d->recurrent_grad_clip > 0.0f ? d->recurrent_grad_clip : d->recurrent_grad_clip < 0.0f ? 0.0f : __builtin_inff();
        kp.db_part = (float*)(ws + w.dbpart_off);
        kp.exch = (uint32_t*)(ws + w.exch_off);
        kp.err = (int*)(ws + w.err_off) + 1;   // the forward call's word stays as it is: flashrnn_check reports both
        kp.T = steps; kp.B = d->B; kp.NH = d->NH; kp.D = d->D;
#ifdef FLASHRNN_TRACE
        if (pb.grid <= kTraceGrid && first) {
            kp.trace = (unsigned long long*)(ws + w.trace_off + kTraceBytes);
            if (launch_fill_zero(kp.trace, kTraceBytes, stream) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
        }
#endif
        rc = launch_persistent(pb, kp, stream);
        if (rc != FLASHRNN_OK) return rc;
        if (d->T == 0) break;
    }
    (void)rec_step;
    // db: sum of the per-row partial sums in row order; dR: GEMM over (t, b)
    // (the staged kernels leave db to the GEMM, which reads every gate gradient anyway)
    const size_t nb = (size_t)d->NH * G * d->D;
    const bool db_from_gemm = pb.e->tile != 0;
    if (d->T == 0) {
        if (db_from_gemm) {
            if (launch_fill_zero(db, nb * 4, stream) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
        } else if (launch_sum_slices((const float*)(ws + w.dbpart_off), (float*)db, nb, d->B, nb, stream) != hipSuccess) {
            return FLASHRNN_ERR_LAUNCH;
        }
        if (launch_fill_zero(dR, (size_t)d->NH * d->D * G * d->D * 4, stream) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
        return FLASHRNN_OK;
    }
    if (launch_dr_gemm(bf, (const float*)states, dWx, ws + w.dgn_off, (float*)(ws + w.drpart_off), (float*)dR, d->T, d->B, d->NH, d->D,
                       G, S, d->cell == FLASHRNN_GRU, (float*)(ws + w.dbpart_off), db_from_gemm, (float*)db, stream) != hipSuccess)
        return FLASHRNN_ERR_LAUNCH;
    return FLASHRNN_OK;
}

}  // namespace

extern "C" {

int flashrnn_num_states(int cell) { return num_states(cell); }
int flashrnn_num_gates(int cell) { return num_gates(cell); }

size_t flashrnn_gate_cache_bytes(const flashrnn_desc_t* d) {
    if (validate(d) != FLASHRNN_OK) return 0;
    return (size_t)d->T * d->B * d->NH * d->D * record_slots(d->cell) * io_size(d->io_dtype);
}

size_t flashrnn_workspace_bytes(const flashrnn_desc_t* d) {
    if (validate(d) != FLASHRNN_OK) return 0;
    Workspace w;
    Plans pl;
    if (carve(d, &w, &pl) != FLASHRNN_OK) return 0;
    return w.total;
}

namespace {
// The plan a call runs: which = 0 forward call that saves its values, 1 backward call, 2 forward call that saves nothing.
int plan_of_call(const flashrnn_desc_t* d, int which, Plan* pl) {
    if (which < 0 || which > 2) return FLASHRNN_ERR_SHAPE;
    Workspace w;
    Plans all;
    const int rc = carve(d, &w, &all);
    if (rc != FLASHRNN_OK) return rc;
    *pl = which == 1 ? all.bwd : all.step.e ? all.step : which == 0 ? all.fwd : all.infer;
    return FLASHRNN_OK;
}
}  // namespace

int flashrnn_plan(const flashrnn_desc_t* d, int backward, int* workgroups, int* cus_per_head, int* waves_per_wg) {
    int rc = validate(d);
    if (rc != FLASHRNN_OK) return rc;
    Plan pl;
    rc = plan_of_call(d, backward, &pl);
    if (rc != FLASHRNN_OK) return rc;
    if (workgroups) *workgroups = (pl.GPAR < pl.NG ? pl.GPAR : pl.NG) * pl.P;
    if (cus_per_head) *cus_per_head = pl.P * ((d->B + pl.e->BT - 1) / pl.e->BT);
    if (waves_per_wg) *waves_per_wg = pl.block / 64;
    return FLASHRNN_OK;
}

int flashrnn_plan_kernel(const flashrnn_desc_t* d, int backward, int* staged, int* batch_tile, int* split) {
    int rc = validate(d);
    if (rc != FLASHRNN_OK) return rc;
    Plan pl;
    rc = plan_of_call(d, backward, &pl);
    if (rc != FLASHRNN_OK) return rc;
    if (staged) *staged = pl.e->tile != 0 ? (pl.e->exact >= 2 ? 2 : 1) : 0;
    if (batch_tile) *batch_tile = pl.e->BT;
    if (split) *split = pl.P;
    return FLASHRNN_OK;
}

int flashrnn_fwd(const flashrnn_desc_t* d, const void* Wx, const void* R, const void* b, const void* states0, void* states,
                 void* gate_cache, void* workspace, void* hip_stream) {
    return fwd_impl(d, Wx, R, b, states0, states, gate_cache, workspace, 0, hip_stream);
}

int flashrnn_fwd_static_scratch(const flashrnn_desc_t* d, const void* Wx, const void* R, const void* b, const void* states0,
                                void* states, void* gate_cache, void* hip_stream) {
    const int rc = validate(d);   // argument errors are reported without touching a device
    if (rc != FLASHRNN_OK) return rc;
    void* ws = static_scratch_ptr();
    if (!ws) return FLASHRNN_ERR_LAUNCH;
    return fwd_impl(d, Wx, R, b, states0, states, gate_cache, ws, kStaticScratchBytes, hip_stream);
}

int flashrnn_bwd(const flashrnn_desc_t* d, const void* R, const void* b, const void* states, const void* gate_cache,
                 const void* dH, const void* dstates_last, void* dWx, void* dR, void* db, void* dstates0, void* workspace,
                 void* hip_stream) {
    return bwd_impl(d, nullptr, R, b, states, gate_cache, dH, dstates_last, dWx, dR, db, dstates0, workspace, hip_stream);
}

int flashrnn_bwd_recompute(const flashrnn_desc_t* d, const void* Wx, const void* R, const void* b, const void* states, const void* dH,
                           const void* dstates_last, void* dWx, void* dR, void* db, void* dstates0, void* workspace, void* hip_stream) {
    if (d && validate(d) == FLASHRNN_OK && d->T > 0 && !Wx) return FLASHRNN_ERR_NULL;
    alignas(16) static const char kNoInputs[16] = {0};   // T = 0: nothing to recompute; any non-null, aligned pointer selects the windowed path
    return bwd_impl(d, Wx ? Wx : (d && d->T == 0 ? (const void*)kNoInputs : nullptr), R, b, states, nullptr, dH, dstates_last, dWx, dR, db, dstates0,
                    workspace, hip_stream);
}

size_t flashrnn_recompute_workspace_bytes(const flashrnn_desc_t* d) {
    if (validate(d) != FLASHRNN_OK) return 0;
    Workspace w;
    Plans pl;
    if (carve(d, &w, &pl) != FLASHRNN_OK) return 0;
    return recompute_layout(d, w.total).total;
}

int flashrnn_check(const flashrnn_desc_t* d, const void* workspace, void* hip_stream) {
    if (!workspace) return FLASHRNN_OK;
    if (workspace == FLASHRNN_STATIC_SCRATCH) {
        workspace = static_scratch_ptr();
        if (!workspace) return FLASHRNN_ERR_LAUNCH;
    }
    int flags[2] = {0, 0};
    hipStream_t stream = (hipStream_t)hip_stream;
    bool fwd_waits = true, bwd_waits = true;
    {   // plans without cross-CU waits cannot time out and do not maintain their error word
        Workspace w;
        Plans pl;
        if (d && validate(d) == FLASHRNN_OK && carve(d, &w, &pl) == FLASHRNN_OK) { fwd_waits = pl.fwd.e->multi; bwd_waits = pl.bwd.e->multi; }
        if (!fwd_waits && !bwd_waits) return hipStreamSynchronize(stream) == hipSuccess ? FLASHRNN_OK : FLASHRNN_ERR_LAUNCH;
    }
    if (hipMemcpyAsync(flags, workspace, sizeof(flags), hipMemcpyDeviceToHost, stream) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
    if (hipStreamSynchronize(stream) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
    return ((fwd_waits && flags[0] != 0) || (bwd_waits && flags[1] != 0)) ? FLASHRNN_ERR_TIMEOUT : FLASHRNN_OK;
}

int flashrnn_trace_phases(const flashrnn_desc_t* d, const void* workspace, int backward, double* clocks, int* waves, void* hip_stream) {
#ifdef FLASHRNN_TRACE
    int rc = validate(d);
    if (rc != FLASHRNN_OK) return rc;
    if (!workspace || !clocks) return FLASHRNN_ERR_NULL;
    Workspace w;
    Plans pl;
    rc = carve(d, &w, &pl);
    if (rc != FLASHRNN_OK) return rc;
    static unsigned long long host[kTraceGrid * kTraceWaves * kTracePhases];
    hipStream_t stream = (hipStream_t)hip_stream;
    if (hipMemcpyAsync(host, (const char*)workspace + w.trace_off + (backward ? kTraceBytes : 0), kTraceBytes, hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
        return FLASHRNN_ERR_LAUNCH;
    // mean over the waves that recorded anything
    double sum[kTracePhases] = {0};
    int n = 0;
    for (int i = 0; i < kTraceGrid * kTraceWaves; ++i) {
        unsigned long long tot = 0;
        for (int j = 0; j < kTracePhases; ++j) tot += host[(size_t)i * kTracePhases + j];
        if (tot == 0) continue;
        for (int j = 0; j < kTracePhases; ++j) sum[j] += (double)host[(size_t)i * kTracePhases + j];
        ++n;
    }
    for (int j = 0; j < kTracePhases; ++j) clocks[j] = n ? sum[j] / n : 0.0;
    if (waves) *waves = n;
    return FLASHRNN_OK;
#else
    (void)d; (void)workspace; (void)backward; (void)clocks; (void)waves; (void)hip_stream;
    return FLASHRNN_ERR_UNSUPPORTED;
#endif
}

int flashrnn_profile_enable(int on) {
    std::lock_guard<std::mutex> lock(g_prof_mu);
    g_prof.stride = on > 0 ? on : 0;
    g_prof.seen[0] = g_prof.seen[1] = 0;
    g_prof.count[0] = g_prof.count[1] = 0;
    return FLASHRNN_OK;
}

int flashrnn_profile_kernel_ms(int backward, float* mean_ms, int* launches) {
    std::lock_guard<std::mutex> lock(g_prof_mu);
    const int dir = backward ? 1 : 0;
    double sum = 0.0;
    for (int i = 0; i < g_prof.count[dir]; ++i) {
        float ms = 0.f;
        if (hipEventSynchronize(g_prof.ev[dir][i][1]) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
        if (hipEventElapsedTime(&ms, g_prof.ev[dir][i][0], g_prof.ev[dir][i][1]) != hipSuccess) return FLASHRNN_ERR_LAUNCH;
        sum += ms;
    }
    if (mean_ms) *mean_ms = g_prof.count[dir] ? (float)(sum / g_prof.count[dir]) : 0.f;
    if (launches) *launches = g_prof.count[dir];
    return FLASHRNN_OK;
}

const char* flashrnn_status_string(int status) {
    switch (status) {
        case FLASHRNN_OK: return "ok";
        case FLASHRNN_ERR_NULL: return "a required pointer is NULL";
        case FLASHRNN_ERR_SHAPE: return "invalid shape, cell or dtype";
        case FLASHRNN_ERR_UNSUPPORTED: return "unsupported head size, alignment or dtype combination";
        case FLASHRNN_ERR_WORKSPACE: return "workspace missing or not 256-byte aligned";
        case FLASHRNN_ERR_LAUNCH: return "a HIP call failed";
        case FLASHRNN_ERR_TIMEOUT: return "a cross-CU wait ran into its spin limit";
        case FLASHRNN_ERR_SCRATCH: return "the problem needs more scratch memory than the library's static array holds";
        default: return "unknown status";
    }
}

}  // extern "C"
