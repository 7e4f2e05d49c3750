// The two products of the hot path (Section 3, Algorithms 1 and 2), written for gfx950.
//
// Lane layout ("quad"): four lanes per row, sixteen rows per wave step.  The library's row
// tiles (below) turn every load of a wave step into one contiguous block; read from the
// caller's row layout (four lanes, slots 4k + q) a wave load touches sixteen 32-byte pieces.
//
// Waves walk contiguous chunks of rows, so runs of equal keys (the star of a row in the
// star-ordered pass, the attitude start t in the attitude pass) are accumulated in registers
// (run_step) and reduced over the row groups and written once when they end.
#pragma once

#include "kernels.hpp"

namespace gsr {

constexpr int kQuad = 4;          // lanes per row
constexpr int kStepRows = kWave / kQuad;  // rows per wave step (16)

__device__ __forceinline__ double ld_val(const double* __restrict__ p) {
    return __builtin_nontemporal_load(p);
}
__device__ __forceinline__ double ld_val(const float* __restrict__ p) {
    return (double)__builtin_nontemporal_load(p);
}

// ---------------------------------------------------------------------------------------
// Row tiles: a library-owned copy of the coefficients and indices in which every load
// instruction of a wave step reads one contiguous block (the paper's row layout makes each
// lane's coefficients 4 slots apart, so a wave load would touch sixteen separate 32-byte
// pieces).  A tile holds the kStepRows rows of one wave step.  Lane q of a row's quad holds
// six coefficients, k = 0..5 (tile_slot gives their slots):
//   k = 0, 1, 2 : attitude elements 2q, 2q + 1 and 8 + q of the row's twelve, counted knot by
//                 knot (element e = knot e / 3, axis e % 3: the order of AttCopy)
//   k = 3       : astrometric q
//   k = 4       : astrometric 4 (q = 0), instrumental 4, 5 (q = 1, 2), global (q = 3)
//   k = 5       : instrumental 3, 0, 1, 2 (q = 0..3)
// Storage of a tile ([rg][q][..] = lane-contiguous):
//   binary64 : three 1 KiB groups [rg][q][2]: k = (0, 1), (2, 3), (4, 5)
//   binary32 : a 1 KiB group [rg][q][4] (k = 2..5), then a 512 B group [rg][q][2] (k = 0, 1)
//   indices  : [rg][q][2] int32 = (star, att), (instr0, instr4), (instr1, instr5),
//              (instr2, instr3) for q = 0..3
// The index tile follows the coefficients of the same tile (one stream per wave).  Padding
// rows of the last tile carry zero coefficients and the last row's indices.
constexpr int kTileVals = kStepRows * kPar;  // 384 coefficients per tile
constexpr int kTileIdx = kStepRows * 8;      // 128 int32 per tile
template <typename VT>
constexpr int64_t tile_elems() {  // coefficients, then the index tile, in units of VT
    return kTileVals + kTileIdx * 4 / (int64_t)sizeof(VT);
}

// Slot (0..23, paper order) of coefficient k of lane q.
__host__ __device__ constexpr int tile_slot(int q, int k) {
    if (k < 3) {
        const int e = k < 2 ? 2 * q + k : 8 + q;
        return kAstro + kParAxis * (e % kAxes) + e / kAxes;
    }
    if (k == 3) return q;
    if (k == 4) return q == 0 ? 4 : 20 + q;
    return q == 0 ? 20 : 16 + q;
}

// One row of a wave step as lane q of its quad holds it: the coefficients above, the row's
// star and attitude start, the instrumental index of k = 5 (ia) and of k = 4 (ib, lanes 1, 2).
struct TileRow {
    double e0, e1, e2, as, z, wi;
    int32_t star, att, ia, ib;
};

__device__ __forceinline__ void ld_tile(const double* __restrict__ tiles, int64_t tile, int lane,
                                        TileRow& r) {
    const f64x2* __restrict__ p =
        reinterpret_cast<const f64x2*>(tiles + tile * tile_elems<double>()) + lane;
    const f64x2 a = __builtin_nontemporal_load(p);
    const f64x2 b = __builtin_nontemporal_load(p + kWave);
    const f64x2 c = __builtin_nontemporal_load(p + 2 * kWave);
    r.e0 = a.x;
    r.e1 = a.y;
    r.e2 = b.x;
    r.as = b.y;
    r.z = c.x;
    r.wi = c.y;
}
__device__ __forceinline__ void ld_tile(const float* __restrict__ tiles, int64_t tile, int lane,
                                        TileRow& r) {
    const float* __restrict__ t = tiles + tile * tile_elems<float>();
    const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(t) + lane);
    const f32x2 w = __builtin_nontemporal_load(reinterpret_cast<const f32x2*>(t + 4 * kWave) + lane);
    r.e0 = w.x;
    r.e1 = w.y;
    r.e2 = v.x;
    r.as = v.y;
    r.z = v.z;
    r.wi = v.w;
}

// Index tile of a wave step.
template <typename VT>
__device__ __forceinline__ void ld_tile_idx(const VT* __restrict__ tiles, int64_t tile, int lane,
                                            TileRow& r) {
    const int32_t* itile =
        reinterpret_cast<const int32_t*>(tiles + tile * tile_elems<VT>() + kTileVals);
    const i32x2 v = __builtin_nontemporal_load(reinterpret_cast<const i32x2*>(itile) + lane);
    r.star = __builtin_amdgcn_update_dpp(0, v.x, 0x00, 0xF, 0xF, false);  // quad_perm [0,0,0,0]
    r.att = __builtin_amdgcn_update_dpp(0, v.y, 0x00, 0xF, 0xF, false);
    const int32_t i3 = __builtin_amdgcn_update_dpp(0, v.y, 0xFF, 0xF, 0xF, false);  // [3,3,3,3]
    r.ia = ((lane & 3) == 0) ? i3 : v.x;
    r.ib = v.y;
}

// The caller's arrays, for systems whose row tiles did not fit: lane q of a row's quad takes from
// them what the tiles would have given it (binary32: rounded to nearest, as the tiles are).  A
// wave load then touches sixteen pieces of 32 bytes.
struct RowSrc {
    const double* vals;
    const int32_t *star, *att, *instr;
};
template <typename VT>
__device__ __forceinline__ void ld_row(const RowSrc& a, int64_t row, int q, TileRow& r) {
    const double* __restrict__ v = a.vals + row * kPar;
    auto at = [&](int slot) { return (double)(VT)ld_val(v + slot); };
    const int32_t* __restrict__ in = a.instr + row * kInstr;
    r.e0 = at(tile_slot(q, 0));
    r.e1 = at(tile_slot(q, 1));
    r.e2 = at(tile_slot(q, 2));
    r.as = at(tile_slot(q, 3));
    r.z = at(tile_slot(q, 4));
    r.wi = at(tile_slot(q, 5));
    r.star = a.star[row];
    r.att = a.att[row];
    r.ia = in[q == 0 ? 3 : q - 1];
    r.ib = in[q == 1 || q == 2 ? q + 3 : 3];
}

// A wave step's rows from the tiles, or (ROWS) from the caller's arrays; rows past m repeat the
// last one there.
template <bool ROWS, typename VT>
__device__ __forceinline__ void ld_step(const VT* __restrict__ tiles, const RowSrc& src, int64_t m,
                                        int64_t tile, int lane, TileRow& r) {
    if (ROWS) {
        ld_row<VT>(src, min(tile * kStepRows + lane / kQuad, m - 1), lane % kQuad, r);
    } else {
        ld_tile(tiles, tile, lane, r);
        ld_tile_idx(tiles, tile, lane, r);
    }
}

// Setup: row tiles from the paper's row layout (one thread per tile element).
template <typename VT>
static __global__ void k_make_tiles(int64_t m, int64_t ntiles, const double* __restrict__ vals,
                                    VT* __restrict__ tiles) {
    const int64_t total = ntiles * kTileVals;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        const int64_t tile = e / kTileVals;
        const int o = (int)(e - tile * kTileVals);
        VT* __restrict__ dst = tiles + tile * tile_elems<VT>() + o;
        int lane, k;
        if (sizeof(VT) == 8) {
            lane = (o % (2 * kWave)) / 2;
            k = 2 * (o / (2 * kWave)) + o % 2;
        } else if (o < 4 * kWave) {
            lane = o / 4;
            k = 2 + o % 4;
        } else {
            lane = (o - 4 * kWave) / 2;
            k = (o - 4 * kWave) % 2;
        }
        const int64_t row = tile * kStepRows + lane / kQuad;
        const int slot = tile_slot(lane % kQuad, k);
        *dst = row < m ? (VT)vals[row * kPar + slot] : (VT)0;  // binary32: round to nearest
    }
}

template <typename VT>
static __global__ void k_make_itiles(int64_t m, int64_t ntiles, const int32_t* __restrict__ star,
                                     const int32_t* __restrict__ att,
                                     const int32_t* __restrict__ instr, VT* __restrict__ tiles) {
    const int64_t total = ntiles * kTileIdx;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        const int64_t tile = e / kTileIdx;
        const int o = (int)(e - tile * kTileIdx);
        const int lane = o / 2, h = o % 2, q = lane % kQuad;
        const int64_t row = min(tile * kStepRows + lane / kQuad, m - 1);
        int32_t v;
        if (q == 0) {
            v = h ? att[row] : star[row];
        } else {
            const int k = (q == 1) ? (h ? 4 : 0) : (q == 2) ? (h ? 5 : 1) : (h ? 3 : 2);
            v = instr[row * kInstr + k];
        }
        reinterpret_cast<int32_t*>(tiles + tile * tile_elems<VT>() + kTileVals)[o] = v;
    }
}

// Attitude tiles (the attitude copy): kStepRows rows of 12 attitude coefficients; lane
// (rg, q) needs column t + q of the three axes of row rg: a group [rg][q][2] (axes 0, 1)
// followed by a group [rg][q] (axis 2).  Padding rows are zero.
constexpr int kTileAtt = kStepRows * kAxes * kParAxis;  // 192 coefficients per tile

__device__ __forceinline__ void ld_att_tile(const double* __restrict__ t, int64_t tile, int lane,
                                            double (&va)[kAxes]) {
    const double* __restrict__ b = t + tile * kTileAtt;
    const f64x2 v = __builtin_nontemporal_load(reinterpret_cast<const f64x2*>(b) + lane);
    va[0] = v.x;
    va[1] = v.y;
    va[2] = __builtin_nontemporal_load(b + 2 * kWave + lane);
}
__device__ __forceinline__ void ld_att_tile(const float* __restrict__ t, int64_t tile, int lane,
                                            double (&va)[kAxes]) {
    const float* __restrict__ b = t + tile * kTileAtt;
    const f32x2 v = __builtin_nontemporal_load(reinterpret_cast<const f32x2*>(b) + lane);
    va[0] = v.x;
    va[1] = v.y;
    va[2] = __builtin_nontemporal_load(b + 2 * kWave + lane);
}

// Cross-lane moves of a double with a DPP control (both 32-bit halves).
// quad_perm [1,0,3,2] = 0xB1, [2,3,0,1] = 0x4E; row_ror:4 = 0x124, row_ror:8 = 0x128.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const int lo2 = __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xF, 0xF, false);
    const int hi2 = __builtin_amdgcn_update_dpp(0, hi, CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi2, lo2);
}

// Sum over the four lanes of a quad, result in all four.
__device__ __forceinline__ double quad_sum(double v) {
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    return v;
}

// v[l] + v[l ^ 16] (PAIR = 16) or v[l] + v[l ^ 32] (PAIR = 32) in every lane, with the gfx950
// row swaps (no LDS crossbar): swapping a register with itself yields, in every lane, the
// value of the lower and of the upper partner, added in that order (the same in both lanes).
template <int PAIR>
__device__ __forceinline__ double pair_sum(double v) {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    unsigned l0, l1, h0, h1;
    if (PAIR == 16) {
        const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        l0 = a[0]; l1 = a[1]; h0 = b[0]; h1 = b[1];
    } else {
        const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        l0 = a[0]; l1 = a[1]; h0 = b[0]; h1 = b[1];
    }
    return __hiloint2double((int)h0, (int)l0) + __hiloint2double((int)h1, (int)l1);
}

// Sum over the lanes with the same lane % STRIDE (STRIDE = 1, 2, 4 or 8), result in all of
// them: DPP within each 16-lane row, then the two row swaps across rows.
template <int STRIDE>
__device__ __forceinline__ double group_sum(double v) {
    static_assert(STRIDE == 1 || STRIDE == 2 || STRIDE == 4 || STRIDE == 8, "stride");
    if (STRIDE <= 1) v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
    if (STRIDE <= 2) v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
    if (STRIDE <= 4) v += dpp_f64<0x124>(v);  // row_ror:4
    v += dpp_f64<0x128>(v);                   // row_ror:8
    v = pair_sum<16>(v);
    return pair_sum<32>(v);
}

// Runs of equal keys over the row groups of a wave (lane = STRIDE * group + q; keys sorted
// within the step, -1 for rows that take no part).  acc[] holds each lane's share of the
// open run `ckey`.  A step whose rows all continue the open run only adds; when runs end,
// their sums are reduced over the row groups and passed to flush(key, sums) -- called by
// every lane, with the totals valid in all of them -- and the step's last run stays open.
template <int NV, int STRIDE, typename F>
__device__ __forceinline__ void run_step(int32_t key, const double (&v)[NV], double (&acc)[NV],
                                         int32_t& ckey, F&& flush) {
    const uint64_t valid = __ballot(key >= 0);
    if (valid == 0) return;
    // lane indices below are wave-uniform: read the key with v_readlane (no LDS round trip)
    const int32_t kfirst =
        __builtin_amdgcn_readlane(key, __ffsll((unsigned long long)valid) - 1);
    const int32_t klast = __builtin_amdgcn_readlane(key, 63 - __clzll((unsigned long long)valid));
    if (kfirst == ckey && klast == ckey) {
#pragma unroll
        for (int j = 0; j < NV; ++j) acc[j] += v[j];
        return;
    }
    double red[NV];
    if (ckey >= 0) {  // the open run ends in this step (or ended at its start)
#pragma unroll
        for (int j = 0; j < NV; ++j) red[j] = group_sum<STRIDE>(acc[j] + (key == ckey ? v[j] : 0.0));
        flush(ckey, red);
    }
    auto next_after = [&](int32_t k) {
        const uint64_t gt = __ballot(key > k);
        return (int32_t)__builtin_amdgcn_readlane(key, __ffsll((unsigned long long)gt) - 1);
    };
    int32_t k = (kfirst == ckey) ? next_after(ckey) : kfirst;
    while (k != klast) {  // runs that start and end inside the step
#pragma unroll
        for (int j = 0; j < NV; ++j) red[j] = group_sum<STRIDE>(key == k ? v[j] : 0.0);
        flush(k, red);
        k = next_after(k);
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) acc[j] = (key == klast) ? v[j] : 0.0;
    ckey = klast;
}

// Close the open run at the end of a chunk.
template <int NV, int STRIDE, typename F>
__device__ __forceinline__ void run_close(double (&acc)[NV], int32_t& ckey, F&& flush) {
    if (ckey < 0) return;
    double red[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) red[j] = group_sum<STRIDE>(acc[j]);
    flush(ckey, red);
    ckey = -1;
}

// x[ins0 + c] += sum_b part[b][c] for the n_instr + 1 instrumental and global columns.
// blockIdx.y takes a slice of the blocks; slices meet in one atomic add per column.
static __global__ void k_reduce_partials(int ncols, int nblocks, const double* __restrict__ part,
                                         double* __restrict__ x, const LsqrState* __restrict__ st,
                                         int check_stop) {
    if (check_stop && st->stop) return;
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncols) return;
    const int per = (nblocks + gridDim.y - 1) / gridDim.y;
    const int b0 = blockIdx.y * per, b1 = min(nblocks, b0 + per);
    double s = 0.0;
    for (int b = b0; b < b1; ++b) s += part[(int64_t)b * ncols + c];
    if (gridDim.y == 1) {
        x[c] += s;
    } else if (b0 < b1) {
        atomic_add_f64(x + c, s);
    }
}

// ---------------------------------------------------------------------------------------
// Fused LSQR u-step and star-ordered part of the following v-step (one read of each row):
//   u~[r] = sv (A xt)[r] - alpha su u~[r]            (xt = p o v~, the previous v-step)
//   s[c] += A[r,c] u~[r]   for the astrometric, instrumental and global columns
// s is accumulated unnormalized (1/beta is applied by the vector step once beta is known);
// the attitude columns of s come from k_aprod2_att on the attitude copy.  Block partials:
// sum u~^2 -> partials[block], instrumental/global sums -> part[block][n_instr + 1].
//
// What bounds it: HBM.  A read stream on this GPU loses about a quarter of its rate as soon
// as a few per cent of scattered writes run beside it (streaming the tiles of a 2e7-row
// system: 0.66 ms; with each wave storing its 128 bytes of u~ per step 0.89 ms, whatever the
// store's cache policy; with the same stores collected into bursts of 64 KiB or more per
// block, non-temporal, into an array that is not the one being read: 0.75 ms).  So a block
// takes rounds of consecutive rows, keeps the round's u~ and its finished stars' sums on
// chip, and writes both at the end of the round, all waves together; the old and the new u~
// are two arrays that swap roles every iteration.  Stars that continue into the
// neighbouring wave meet on chip too; only a block's first and last star need atomics (they
// cost as much as the stores: 0.87 -> 1.05 ms with two such stars per wave and round).
// Two forms:
//   k_aprod12     : u~ and the star sums in LDS, beside the block's instrumental sums and the
//                   staged instrumental unknowns (needs room for kRoundLds wave steps: with 20
//                   rows a star n_instr up to about 8,700, with one row a star and its many
//                   slots up to about 3,300).  The block's waves take the round's wave steps in
//                   turn, so that the block reads one contiguous stream, and every lane adds
//                   its products to the star's LDS slot (0.86 ms against 0.89 with a run of
//                   steps per wave and the sums of equal stars reduced over the lanes first);
//   k_aprod12_reg : u~ and the star sums in registers (the LDS is full at n_instr = 10,000, or
//                   several rounds of the LDS form would each be shorter than kRoundLds).  Each
//                   wave takes a run of wave steps; sums of equal stars stay in registers until
//                   the star ends (run_step).
// Attitude operand: xa holds the attitude part of xt knot by knot (three axes of a knot
// together), so a row's twelve elements are 96 contiguous bytes: one or two cache lines
// instead of three to six, two loads per lane instead of three.
// Measured inside a solve: 2e7 rows, n_instr 6,000: 1.12 -> 0.90 to 0.98 ms from process to
// process (4.4 -> 5.0 to 5.5 TB/s of the algorithmic bytes; 0.84 ms launched by itself);
// register form, n_instr 10,000: 2.5e7 rows 1.39 -> 1.21 ms, 2e8 rows 9.67 -> 9.36 ms.
//
// TRANS: the same pass for the transposed operator D A^T (the adjoint solve), where the
// row-space vector is v~:  v~[r] = su (A xt)[r] - beta sv v~[r]  (xt = p o u~), preceded on
// the same rows by the pending update z += f1 w; w = sv v~ - f2 w of the row-space z, w (all
// in place: uin == uout).  Partials then are 4 rows (pstride apart; entries past gridDim
// belong to the constraint rows): sum v~^2, sum z^2, sum z w, sum w^2.
constexpr int kRowBlock = 1024;                   // threads of a row-pass block
constexpr int kRowWaves = kRowBlock / kWave;      // 16 waves, one block per compute unit
constexpr int kRoundRows = kRowWaves * kStepRows; // rows of a round per wave step
constexpr int kRoundLds = 9;       // fewest wave steps per round worth the LDS form
constexpr int kRoundLdsMax = 48;   // most wave steps per round of the LDS form
constexpr int kRegGroups = 8;      // register form: groups of four wave steps per round
constexpr int kRegStars = 2;       // register form: sets of 16 pending stars
constexpr int kRegXch = 5 * kRowWaves + 5 * (kRowWaves + 1) + (kRowWaves + 2) / 2;  // doubles

template <typename VT>
struct RowArgs {
    Geo g;
    const VT* tiles;
    const int32_t* star;
    const double* xx;     // operand
    const double* xa;     // its attitude part, knot by knot
    const double* uin;    // old u~ (TRANS: old v~)
    double* uout;
    double* s;
    const LsqrState* st;
    double* partials;
    double* part;
    double *ww, *zz;      // TRANS: w and z of the row space
    int pstride;
    int tw;               // wave steps per wave and round
    int nsb;              // LDS form: stars with a slot;  register form: 1 = exchange area
};

// The row's dot product, summed over the quad.  IL: the attitude unknowns from xa (knot by
// knot), otherwise from xx.
template <bool IL>
__device__ __forceinline__ double row_dot(const Geo& g, const TileRow& r, int q,
                                          const double* __restrict__ xx,
                                          const double* __restrict__ xa,
                                          const double* __restrict__ xi, double xglob) {
    // every lane issues all its loads before the first use, without branches: a load under a
    // lane condition would wait for the ones before it
    const double* __restrict__ xs = xx + (int64_t)kAstro * r.star;
    const double x0 = xs[q];
    const double x4 = xs[q == 0 ? 4 : q];
    double v0, v1, v2;
    if (IL) {
        typedef f64x2 __attribute__((aligned(8))) f64x2u;
        const double* __restrict__ a = xa + (int64_t)kAxes * r.att;
        const f64x2 v = *reinterpret_cast<const f64x2u*>(a + 2 * q);
        v0 = v.x;
        v1 = v.y;
        v2 = a[8 + q];
    } else {
        // element e of the row: axis e % 3, knot att + e / 3
        const double* __restrict__ a = xx + g.att0 + r.att;
        const int e0 = 2 * q, e1 = 2 * q + 1, e2 = 8 + q;
        v0 = a[(int64_t)(e0 % kAxes) * g.T + e0 / kAxes];
        v1 = a[(int64_t)(e1 % kAxes) * g.T + e1 / kAxes];
        v2 = a[(int64_t)(e2 % kAxes) * g.T + e2 / kAxes];
    }
    const bool two = q == 1 || q == 2;  // lanes with a second instrumental coefficient
    const double wx = xi[r.ia];
    const double wb = xi[two ? r.ib : r.ia];
    const double zx = q == 0 ? x4 : two ? wb : xglob;
    double sum = r.as * x0;
    sum = fma(r.e0, v0, sum);
    sum = fma(r.e1, v1, sum);
    sum = fma(r.e2, v2, sum);
    sum = fma(r.wi, wx, sum);
    sum = fma(r.z, zx, sum);
    return quad_sum(sum);
}

// Ends a branch whose other side does the same to LDS: merged, the two would become one flat
// access, after which every wait for a load is a wait for all of them.
__device__ __forceinline__ void keep_apart() { asm volatile(""); }

// Brings the unknowns of stars s0..s1 (consecutive) near before the first row needs them: one
// line per thread `i`.
__device__ __forceinline__ void touch_stars(const double* __restrict__ xx, int32_t s0, int32_t s1,
                                            int i) {
    const int64_t e = (int64_t)kAstro * s0 + 16 * i;
    double t = 0.0;
    if (e < (int64_t)kAstro * (s1 + 1)) t = xx[e];
    asm volatile("" ::"v"(t));
}

template <typename VT, bool TRANS = false>
static __global__ __launch_bounds__(kRowBlock) void k_aprod12(RowArgs<VT> p) {
    // [n_instr + 1] sums, [n_instr] staged xt, [tw][kRoundRows] u~, [nsb][5] star sums
    extern __shared__ double lds[];
    __shared__ double sh[kRowWaves];
    const LsqrState* __restrict__ st = p.st;
    if (st->stop) return;
    const Geo g = p.g;
    const VT* __restrict__ tiles = p.tiles;
    const int32_t* __restrict__ star = p.star;
    const double* __restrict__ xx = p.xx;
    const double* __restrict__ xa = p.xa;
    const double* uin = p.uin;
    double* uout = p.uout;
    double* __restrict__ s = p.s;
    const double xs = TRANS ? st->su : st->sv;
    const double ys = TRANS ? st->beta * st->sv : st->alpha * st->su;
    const bool pending = TRANS && st->pending;
    const double f1 = st->f1, f2 = st->f2, svo = st->sv;
    const int tw = p.tw, nsb = p.nsb;
    double zsq = 0.0, zw = 0.0, wsq = 0.0;
    double* lsum = lds;  // instrumental and global sums of the block
    double* lxi = lds + g.I + 1;
    double* ubuf = lds + 2 * (int64_t)g.I + 2;  // 16-byte aligned
    double* sbuf = ubuf + tw * kRoundRows;
    for (int k = threadIdx.x; k <= g.I; k += kRowBlock) lsum[k] = 0.0;
    for (int k = threadIdx.x; k < g.I; k += kRowBlock) lxi[k] = xx[g.ins0 + k];
    for (int k = threadIdx.x; k < kAstro * nsb; k += kRowBlock) sbuf[k] = 0.0;
    __syncthreads();
    const double* __restrict__ xi = lxi;  // LDS reads (not flat loads tied to vmcnt)
    const int lane = threadIdx.x % kWave, rg = lane / kQuad, q = lane % kQuad;
    const int w = threadIdx.x / kWave;
    const double xglob = xx[g.glb0];
    const int64_t ntiles = (g.m + kStepRows - 1) / kStepRows;
    const int64_t bt = (int64_t)tw * kRowWaves, nch = (ntiles + bt - 1) / bt;
    double usq = 0.0, gacc = 0.0;
    for (int64_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
        const int64_t R0 = ch * bt * kStepRows, R1 = min(R0 + bt * kStepRows, g.m);
        const int64_t te = min((ch + 1) * bt, ntiles);
        const int32_t S0 = star[R0], S1 = star[R1 - 1];
        const bool shf = R0 > 0 && star[R0 - 1] == S0, shl = R1 < g.m && star[R1] == S1;
        touch_stars(xx, S0, S1, threadIdx.x);
        for (int64_t t = ch * bt + w; t < te; t += kRowWaves) {
            TileRow a;
            ld_tile(tiles, t, lane, a);
            ld_tile_idx(tiles, t, lane, a);
            const int64_t r = t * kStepRows + rg;
            const double uo = uin[min(r, g.m - 1)];
            const double sum = row_dot<true>(g, a, q, xx, xa, xi, xglob);
            const double un = (ys != 0.0) ? xs * sum - ys * uo : xs * sum;
            if (r >= R1) continue;
            if (q == 0) {
                usq = fma(un, un, usq);
                ubuf[r - R0] = un;
            }
            // the star's slot, or (stars past the last slot) straight to s, which is zero
            // there before the pass
            const int o = a.star - S0;
            if ((uint32_t)o < (uint32_t)nsb) {
                atomicAdd(sbuf + kAstro * o + q, a.as * un);
                if (q == 0) atomicAdd(sbuf + kAstro * o + 4, a.z * un);
            } else {
                double* xo = s + (int64_t)kAstro * a.star;
                atomic_add_f64(xo + q, a.as * un);
                if (q == 0) atomic_add_f64(xo + 4, a.z * un);
                keep_apart();
            }
            atomicAdd(lsum + a.ia, a.wi * un);
            if (q == 1 || q == 2) atomicAdd(lsum + a.ib, a.z * un);
            if (q == 3) gacc = fma(a.z, un, gacc);
        }
        __syncthreads();
        // the round's results, written together
        if (TRANS) {
            for (int64_t r = R0 + threadIdx.x; r < R1; r += kRowBlock) {
                if (pending) {  // z, w updated with the old v~ of this row
                    const double wo = p.ww[r];
                    const double zn = fma(f1, wo, p.zz[r]);
                    const double wn = svo * uin[r] - f2 * wo;
                    p.zz[r] = zn;
                    p.ww[r] = wn;
                    zsq = fma(zn, zn, zsq);
                    zw = fma(zn, wn, zw);
                    wsq = fma(wn, wn, wsq);
                }
                uout[r] = ubuf[r - R0];
            }
        } else {
            for (int64_t r = R0 + 2 * threadIdx.x; r < R1; r += 2 * kRowBlock) {
                if (r + 1 < R1)
                    __builtin_nontemporal_store(*reinterpret_cast<const f64x2*>(ubuf + (r - R0)),
                                                reinterpret_cast<f64x2*>(uout + r));
                else
                    uout[r] = ubuf[r - R0];
            }
        }
        const int ne = kAstro * min(S1 - S0 + 1, nsb);
        const int e0 = shf ? kAstro : 0, e1 = (shl && S1 - S0 < nsb) ? ne - kAstro : ne;
        for (int e = threadIdx.x; e < ne; e += kRowBlock) {
            const double v = sbuf[e];
            sbuf[e] = 0.0;
            double* xo = s + (int64_t)kAstro * S0 + e;
            if (e >= e0 && e < e1)  // s is zero before this pass: owned stars are stored
                __builtin_nontemporal_store(v, xo);
            else
                atomic_add_f64(xo, v);
        }
        __syncthreads();
    }
    const double gs = wave_sum(gacc);
    if (lane == 0) atomicAdd(lsum + g.I, gs);
    const double tot = block_sum<kRowBlock>(usq, sh);
    if (threadIdx.x == 0) p.partials[blockIdx.x] = tot;
    if (TRANS) {
        double t2 = block_sum<kRowBlock>(zsq, sh);
        if (threadIdx.x == 0) p.partials[p.pstride + blockIdx.x] = t2;
        t2 = block_sum<kRowBlock>(zw, sh);
        if (threadIdx.x == 0) p.partials[2 * p.pstride + blockIdx.x] = t2;
        t2 = block_sum<kRowBlock>(wsq, sh);
        if (threadIdx.x == 0) p.partials[3 * p.pstride + blockIdx.x] = t2;
    }
    __syncthreads();
    double* dst = p.part + (int64_t)blockIdx.x * (g.I + 1);
    for (int k = threadIdx.x; k <= g.I; k += kRowBlock) dst[k] = lsum[k];
}

// The register form.  Lane (rg, q) keeps u~ of row 16 q + rg of every group of four wave
// steps, and of each finished star's sums the one of its place: star `base + 16 k + rg`
// astrometric q in pv[k], astrometric 4 of star base + 16 q + rg in p5.  A star shared with
// the neighbouring wave goes through the exchange area (nsb = 1; xw: the wave's share of the
// star that continues from the rows before, xch: one slot per wave boundary of the block, the
// star's slot being its first boundary) or, where the LDS has no room for it, to s with
// atomics.
template <typename VT, bool TRANS = false>
static __global__ __launch_bounds__(kRowBlock) void k_aprod12_reg(RowArgs<VT> p) {
    extern __shared__ double lds[];  // [n_instr + 1] sums, [n_instr] staged xt, exchange area
    const LsqrState* __restrict__ st = p.st;
    if (st->stop) return;
    const Geo g = p.g;
    const VT* __restrict__ tiles = p.tiles;
    const int32_t* __restrict__ star = p.star;
    const double* __restrict__ xx = p.xx;
    const double* __restrict__ xa = p.xa;
    const double* uin = p.uin;
    double* uout = p.uout;
    double* __restrict__ s = p.s;
    const double xs = TRANS ? st->su : st->sv;
    const double ys = TRANS ? st->beta * st->sv : st->alpha * st->su;
    const int tw = p.tw;
    const bool xb = p.nsb != 0;
    double zsq = 0.0, zw = 0.0, wsq = 0.0;
    double* lsum = lds;
    double* lxi = lds + g.I + 1;
    double* xw = lds + 2 * (int64_t)g.I + 1;
    double* xch = xw + kAstro * kRowWaves;
    int32_t* bkey = reinterpret_cast<int32_t*>(xch + kAstro * (kRowWaves + 1));
    constexpr int kXch = kAstro * (kRowWaves + 1);
    for (int k = threadIdx.x; k <= g.I; k += kRowBlock) lsum[k] = 0.0;
    for (int k = threadIdx.x; k < g.I; k += kRowBlock) lxi[k] = xx[g.ins0 + k];
    if (xb && threadIdx.x < kXch) xch[threadIdx.x] = 0.0;
    __syncthreads();
    const double* __restrict__ xi = lxi;
    const int lane = threadIdx.x % kWave, rg = lane / kQuad, q = lane % kQuad;
    // in scalar registers, and with it the bounds of the wave's rows and their shared stars: in
    // vector registers they were spilled (12 to 28 bytes per lane)
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const double xglob = xx[g.glb0];
    const int64_t ntiles = (g.m + kStepRows - 1) / kStepRows;
    const int64_t bt = (int64_t)tw * kRowWaves, nch = (ntiles + bt - 1) / bt;
    double usq = 0.0, gacc = 0.0;
    for (int64_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
        const int64_t tb = ch * bt + (int64_t)w * tw, te = min(tb + tw, ntiles);
        const int64_t r_beg = tb * kStepRows, r_end = min(te * kStepRows, g.m);
        int32_t sf = -1, sl = -1;  // stars shared with the rows before and after the wave's
        if (tb < te) {
            const int32_t s0 = star[r_beg], s1 = star[r_end - 1];
            sf = (r_beg > 0 && star[r_beg - 1] == s0) ? s0 : -1;
            sl = (r_end < g.m && star[r_end] == s1) ? s1 : -1;
            touch_stars(xx, s0, s1, lane);
        }
        if (xb && lane == 0) {
            bkey[w] = sf;
            if (w == kRowWaves - 1) bkey[kRowWaves] = sl;
        }
        double pv[kRegStars], p5 = 0.0;
        int32_t base = -1, top = -1;
#pragma unroll
        for (int k = 0; k < kRegStars; ++k) pv[k] = 0.0;
        auto put = [&](int32_t key, int c, double v) {  // one sum of a finished star
            double* xo = s + (int64_t)kAstro * key + c;
            if (key == sl) {
                if (xb) {
                    atomicAdd(xch + kAstro * (w + 1) + c, v);
                } else {
                    atomic_add_f64(xo, v);
                    keep_apart();
                }
            } else {
                *xo = v;  // s is zero before this pass: owned stars are stored
            }
        };
        auto emit = [&]() {
            if (base < 0) return;
#pragma unroll
            for (int k = 0; k < kRegStars; ++k) {
                const int32_t key = base + 16 * k + rg;
                if (key <= top) put(key, q, pv[k]);
                pv[k] = 0.0;
            }
            const int32_t key = base + 16 * q + rg;
            if (q < kRegStars && key <= top) put(key, 4, p5);
            p5 = 0.0;
            base = -1;
        };
        auto flush = [&](int32_t key_, const double (&t)[2]) {
            const int32_t key = __builtin_amdgcn_readfirstlane(key_);
            if (key == sf) {
                if (lane < kAstro) {  // lanes 0..3: t[0]; lane 4, a q = 0 lane: t[1]
                    const double v = lane < 4 ? t[0] : t[1];
                    if (xb) {
                        xw[kAstro * w + lane] = v;
                    } else {
                        atomic_add_f64(s + (int64_t)kAstro * key + lane, v);
                        keep_apart();
                    }
                }
                return;
            }
            if (base >= 0 && key - base >= 16 * kRegStars) emit();
            if (base < 0) base = key;
            top = key;
            const int o = key - base;
            const double t4 = dpp_f64<0x00>(t[1]);  // quad_perm [0,0,0,0]
#pragma unroll
            for (int k = 0; k < kRegStars; ++k) pv[k] = (rg == o - 16 * k) ? t[0] : pv[k];
            p5 = (16 * q + rg == o) ? t4 : p5;
        };
        double acc[2] = {0.0, 0.0};
        int32_t ckey = -1;
        double ub[kRegGroups];
#pragma unroll
        for (int gi = 0; gi < kRegGroups; ++gi) {
            ub[gi] = 0.0;
            const int64_t t0 = tb + 4 * gi;
            if (t0 >= te) continue;
#pragma clang loop unroll(disable)
            for (int sq = 0; sq < 4; ++sq) {
                const int64_t t = t0 + sq;
                if (t >= te) break;
                TileRow a;
                ld_tile(tiles, t, lane, a);
                ld_tile_idx(tiles, t, lane, a);
                const int64_t r = t * kStepRows + rg;
                const double uo = uin[min(r, g.m - 1)];
                const double sum = row_dot<true>(g, a, q, xx, xa, xi, xglob);
                const double un = (ys != 0.0) ? xs * sum - ys * uo : xs * sum;
                int32_t key = -1;
                double v[2] = {0.0, 0.0};
                if (r < r_end) {
                    if (q == 0) usq = fma(un, un, usq);
                    key = a.star;
                    v[0] = a.as * un;
                    v[1] = (q == 0) ? a.z * un : 0.0;
                    atomicAdd(lsum + a.ia, a.wi * un);
                    if (q == 1 || q == 2) atomicAdd(lsum + a.ib, a.z * un);
                    if (q == 3) gacc = fma(a.z, un, gacc);
                }
                ub[gi] = (q == sq) ? un : ub[gi];
                run_step<2, kQuad>(key, v, acc, ckey, flush);
            }
        }
        run_close<2, kQuad>(acc, ckey, flush);
        __syncthreads();
        // the round's results, written together
#pragma unroll
        for (int gi = 0; gi < kRegGroups; ++gi) {
            const int64_t r = (tb + 4 * gi) * kStepRows + kStepRows * q + rg;
            if (r >= r_end) continue;
            if (TRANS) {
                if (st->pending) {  // z, w updated with the old v~ of this row
                    const double wo = p.ww[r];
                    const double zn = fma(st->f1, wo, p.zz[r]);
                    const double wn = st->sv * uin[r] - st->f2 * wo;
                    p.zz[r] = zn;
                    p.ww[r] = wn;
                    zsq = fma(zn, zn, zsq);
                    zw = fma(zn, wn, zw);
                    wsq = fma(wn, wn, wsq);
                }
                uout[r] = ub[gi];
            } else {
                __builtin_nontemporal_store(ub[gi], uout + r);
            }
        }
        emit();
        if (xb) {
            if (sf >= 0 && lane < kAstro) {
                int j = w;  // the star's first boundary in the block
                while (j > 0 && bkey[j - 1] == sf) --j;
                atomicAdd(xch + kAstro * j + lane, xw[kAstro * w + lane]);
            }
            __syncthreads();
            if (threadIdx.x < kXch) {
                const int j = threadIdx.x / kAstro, c = threadIdx.x % kAstro;
                const int32_t key = bkey[j];
                if (key >= 0 && (j == 0 || bkey[j - 1] != key)) {
                    double* xo = s + (int64_t)kAstro * key + c;
                    if (key == bkey[0] || key == bkey[kRowWaves])  // continues in another block
                        atomic_add_f64(xo, xch[threadIdx.x]);
                    else
                        *xo = xch[threadIdx.x];
                }
                xch[threadIdx.x] = 0.0;
            }
            __syncthreads();
        }
    }
    const double gs = wave_sum(gacc);
    if (lane == 0) atomicAdd(lsum + g.I, gs);
    __syncthreads();
    double* sh = lxi;  // the staged unknowns are no longer needed
    const double tot = block_sum<kRowBlock>(usq, sh);
    if (threadIdx.x == 0) p.partials[blockIdx.x] = tot;
    if (TRANS) {
        double t2 = block_sum<kRowBlock>(zsq, sh);
        if (threadIdx.x == 0) p.partials[p.pstride + blockIdx.x] = t2;
        t2 = block_sum<kRowBlock>(zw, sh);
        if (threadIdx.x == 0) p.partials[2 * p.pstride + blockIdx.x] = t2;
        t2 = block_sum<kRowBlock>(wsq, sh);
        if (threadIdx.x == 0) p.partials[3 * p.pstride + blockIdx.x] = t2;
    }
    __syncthreads();
    double* dst = p.part + (int64_t)blockIdx.x * (g.I + 1);
    for (int k = threadIdx.x; k <= g.I; k += kRowBlock) dst[k] = lsum[k];
}

// ---------------------------------------------------------------------------------------
// aprod 1 by itself:  sum_i = sum_k A[i,k] xx[col(i,k)], then
//   A1_ADD   : y[i] += sum_i
//   A1_LSQR  : y[i] = xs sum_i - ys y[i]  with (xs, ys) = (sv, alpha su)   [forward operator]
//   A1_LSQR_T: same with (xs, ys) = (su, beta sv)                           [transposed]
//   A1_RESID : y[i] = b[i] - sum_i
// LSQR modes also write the block partial of sum y[i]^2.  gate (may be NULL): nothing is done
// when *gate is set (a residual of a correction step that will not be taken).
// Rounds as in the fused pass: the round's sums wait in LDS and y is read and written in one
// go at its end (2e7 rows, n_instr 6,000: 1.12 ms with a load and a store of y per wave step,
// 0.85 ms with the round and the knot-by-knot attitude operand).
// IL: xa holds the attitude part of xx knot by knot (AttCopy); otherwise it is gathered from
// xx, three loads per lane.  LDSI: the instrumental part of xx is staged in LDS.
enum { A1_ADD = 0, A1_LSQR = 1, A1_LSQR_T = 2, A1_RESID = 3 };

template <typename VT, int MODE, bool IL, bool LDSI, bool ROWS = false>
static __global__ __launch_bounds__(kRowBlock) void k_aprod1(
    Geo g, const VT* __restrict__ tiles, const int32_t* __restrict__ star,
    const double* __restrict__ xx, const double* __restrict__ xa, double* y,
    const double* __restrict__ b, const LsqrState* __restrict__ st,
    double* __restrict__ partials, int tw, const int32_t* __restrict__ gate, RowSrc src) {
    extern __shared__ double lds[];  // [n_instr] staged unknowns (LDSI), [tw][kRoundRows] sums
    __shared__ double sh[kRowWaves];
    if (gate && *gate) return;
    constexpr bool kLsqr = (MODE == A1_LSQR || MODE == A1_LSQR_T);
    double xs = 1.0, ys = 0.0;
    if (kLsqr) {
        if (st->stop) return;
        xs = MODE == A1_LSQR ? st->sv : st->su;
        ys = MODE == A1_LSQR ? st->alpha * st->su : st->beta * st->sv;
    }
    double* lxi = lds;
    double* ubuf = lds + (LDSI ? (g.I + 1) / 2 * 2 : 0);
    if (LDSI) {
        for (int k = threadIdx.x; k < g.I; k += kRowBlock) lxi[k] = xx[g.ins0 + k];
        __syncthreads();
    }
    const double* __restrict__ xi = LDSI ? lxi : xx + g.ins0;
    const int lane = threadIdx.x % kWave, rg = lane / kQuad, q = lane % kQuad;
    const int w = threadIdx.x / kWave;
    const double xglob = xx[g.glb0];
    const int64_t ntiles = (g.m + kStepRows - 1) / kStepRows;
    const int64_t bt = (int64_t)tw * kRowWaves, nch = (ntiles + bt - 1) / bt;
    double acc = 0.0;
    for (int64_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
        const int64_t R0 = ch * bt * kStepRows, R1 = min(R0 + bt * kStepRows, g.m);
        const int64_t te = min((ch + 1) * bt, ntiles);
        if (tw > 1) touch_stars(xx, star[R0], star[R1 - 1], threadIdx.x);
        const double* yo = MODE == A1_RESID ? b : y;
        const int64_t r1st = R0 + threadIdx.x;  // its old value arrives with the tiles
        const double yo1st = r1st < R1 ? yo[r1st] : 0.0;
        for (int64_t t = ch * bt + w; t < te; t += kRowWaves) {
            TileRow a;
            ld_step<ROWS>(tiles, src, g.m, t, lane, a);
            const double sum = row_dot<IL>(g, a, q, xx, xa, xi, xglob);
            if (q == 0) ubuf[(t - ch * bt) * kStepRows + rg] = sum;
        }
        __syncthreads();
        for (int64_t r = r1st; r < R1; r += kRowBlock) {
            const double sum = ubuf[r - R0], old = r == r1st ? yo1st : yo[r];
            if (MODE == A1_ADD) {
                y[r] = old + sum;
            } else if (MODE == A1_RESID) {
                y[r] = old - sum;
            } else {
                const double u = (ys != 0.0) ? xs * sum - ys * old : xs * sum;
                y[r] = u;
                acc = fma(u, u, acc);
            }
        }
        __syncthreads();
    }
    if (kLsqr) {
        const double tot = block_sum<kRowBlock>(acc, sh);
        if (threadIdx.x == 0) partials[blockIdx.x] = tot;
    }
}

// xa[3 c + axis] = xx[att0 + axis T + c] (AttCopy)
static __global__ void k_att_copy(AttCopy ac, const double* __restrict__ xx) {
    const int64_t n = kAxes * ac.T, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride)
        put_att(ac, ac.att0 + e, xx[ac.att0 + e]);
}

// ---------------------------------------------------------------------------------------
// aprod 2, star-ordered columns (astrometric, instrumental, global) by themselves:
//   x[col(i,k)] += A[i,k] y[i]  (A2_ADD; A2_LSQR / A2_LSQR_T, where y is the unnormalized
//   u~ or v~ and the following vector step applies 1/beta or 1/alpha), or the contribution is
//   A[i,k]^2 (A2_SQ, column norms).  LSQR modes return at once when the stop flag is set; in
//   them and in A2_SQ the target starts at zero, so a star the block owns is stored.
// The fused pass without its dot products: it reads the tiles' second and third groups and
// the indices (binary32: the first group), 2,560 of 3,584 bytes a wave step (2e7 rows: 0.66 ms
// against 1.15 over the caller's rows, of which it fetched every line).  LDSI: the block's
// instrumental sums in LDS; otherwise (n_instr too large) atomics.
enum { A2_ADD = 0, A2_LSQR = 1, A2_LSQR_T = 2, A2_SQ = 3 };

template <int MODE>
__device__ __forceinline__ double contrib(double a, double yy) {
    return MODE == A2_SQ ? a * a : a * yy;
}

template <typename VT, int MODE, bool LDSI, bool ROWS = false>
static __global__ __launch_bounds__(kRowBlock) void k_aprod2_star(
    Geo g, const VT* __restrict__ tiles, const int32_t* __restrict__ star,
    const double* __restrict__ y, double* __restrict__ x, const LsqrState* __restrict__ st,
    double* __restrict__ part, int tw, int nsb, RowSrc src) {
    extern __shared__ double lds[];  // [n_instr + 1] sums (LDSI) or [1] global, [nsb][5] stars
    if ((MODE == A2_LSQR || MODE == A2_LSQR_T) && st->stop) return;
    const int nI = LDSI ? g.I : 0;
    double* lsum = lds;
    double* sbuf = lds + nI + 1;
    for (int k = threadIdx.x; k < nI + 1 + kAstro * nsb; k += kRowBlock) lds[k] = 0.0;
    __syncthreads();
    const int lane = threadIdx.x % kWave, rg = lane / kQuad, q = lane % kQuad;
    const int w = threadIdx.x / kWave;
    const int64_t ntiles = (g.m + kStepRows - 1) / kStepRows;
    const int64_t bt = (int64_t)tw * kRowWaves, nch = (ntiles + bt - 1) / bt;
    double gacc = 0.0;
    for (int64_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
        const int64_t R0 = ch * bt * kStepRows, R1 = min(R0 + bt * kStepRows, g.m);
        const int64_t te = min((ch + 1) * bt, ntiles);
        const int32_t S0 = star[R0], S1 = star[R1 - 1];
        const bool shf = R0 > 0 && star[R0 - 1] == S0, shl = R1 < g.m && star[R1] == S1;
        for (int64_t t = ch * bt + w; t < te; t += kRowWaves) {
            TileRow a;
            ld_step<ROWS>(tiles, src, g.m, t, lane, a);
            const int64_t r = t * kStepRows + rg;
            const double yy = (MODE == A2_SQ) ? 0.0 : y[min(r, g.m - 1)];
            if (r >= R1) continue;
            const double cs = contrib<MODE>(a.as, yy), cz = contrib<MODE>(a.z, yy),
                         ci = contrib<MODE>(a.wi, yy);
            // the star's slot, or (stars past the last slot) straight to x
            const int o = a.star - S0;
            if ((uint32_t)o < (uint32_t)nsb) {
                atomicAdd(sbuf + kAstro * o + q, cs);
                if (q == 0) atomicAdd(sbuf + kAstro * o + 4, cz);
            } else {
                double* xo = x + (int64_t)kAstro * a.star;
                atomic_add_f64(xo + q, cs);
                if (q == 0) atomic_add_f64(xo + 4, cz);
                keep_apart();
            }
            if (LDSI) {
                atomicAdd(lsum + a.ia, ci);
                if (q == 1 || q == 2) atomicAdd(lsum + a.ib, cz);
            } else {
                atomic_add_f64(x + g.ins0 + a.ia, ci);
                if (q == 1 || q == 2) atomic_add_f64(x + g.ins0 + a.ib, cz);
            }
            if (q == 3) gacc += cz;
        }
        __syncthreads();
        const int ne = kAstro * min(S1 - S0 + 1, nsb);
        const int e0 = shf ? kAstro : 0, e1 = (shl && S1 - S0 < nsb) ? ne - kAstro : ne;
        for (int e = threadIdx.x; e < ne; e += kRowBlock) {
            const double v = sbuf[e];
            sbuf[e] = 0.0;
            double* xo = x + (int64_t)kAstro * S0 + e;
            if (e < e0 || e >= e1)
                atomic_add_f64(xo, v);
            else if (MODE == A2_ADD)
                *xo += v;
            else
                __builtin_nontemporal_store(v, xo);
        }
        __syncthreads();
    }
    const double gs = wave_sum(gacc);
    if (lane == 0) atomicAdd(lsum + nI, gs);
    __syncthreads();
    if (LDSI) {
        double* dst = part + (int64_t)blockIdx.x * (nI + 1);
        for (int k = threadIdx.x; k <= nI; k += kRowBlock) dst[k] = lsum[k];
    } else if (threadIdx.x == 0) {
        atomic_add_f64(x + g.glb0, *lsum);
    }
}

// ---------------------------------------------------------------------------------------
// aprod 2, attitude columns, over the library-owned copy of the attitude coefficients in
// the order (group, row slice, t).  The attitude starts are cut into nb buckets of W knots
// and the rows into slices of consecutive rows, dealt round-robin to the dies; group
// G = b kXcd + x holds the rows of bucket b in the slices of die x.  Block G (placed by the
// dispatcher on die G % kXcd) takes group G and sums the columns t + q of its bucket, three
// axes, in LDS; its waves move through the die's slices in step with the die's other blocks,
// so the u~ values they gather at any time come from one slice, which the die's L2 holds.
// The block's sums go to part[G] (kAxes rows of lw = W + kParAxis - 1 columns), added to x by
// k_att_reduce.  Row k of the copy (tile k / kStepRows): attT = A[row_k, 5 + 4 a + j],
// rowT[k] = row_k, tL[k] = att[row_k] - b W; group G is rows seg[G] .. seg[G + 1] - 1.
constexpr int kXcd = 8;  // accelerator dies; the dispatcher places block i on die i % 8
constexpr int kBlockAtt = 512;
constexpr int kAttChunkTiles = 2;  // wave steps per chunk (chunks dealt to the waves in turn)

template <typename VT, int MODE>
static __global__ __launch_bounds__(kBlockAtt) void k_aprod2_att(
    Geo g, const VT* __restrict__ attT, const int32_t* __restrict__ rowT,
    const int32_t* __restrict__ tL, const int64_t* __restrict__ seg, int lw,
    const double* __restrict__ y, double* __restrict__ part, const LsqrState* __restrict__ st) {
    if ((MODE == A2_LSQR || MODE == A2_LSQR_T) && st->stop) return;
    extern __shared__ double acc[];  // [kAxes][lw]
    for (int i = threadIdx.x; i < kAxes * lw; i += blockDim.x) acc[i] = 0.0;
    __syncthreads();
    const int lane = threadIdx.x % kWave, rg = lane / kQuad, q = lane % kQuad;
    const int wave = threadIdx.x / kWave, wpb = blockDim.x / kWave;
    const int64_t lo = seg[blockIdx.x], hi = seg[blockIdx.x + 1];
    if (lo < hi) {
        const int64_t t_beg = lo / kStepRows, t_end = (hi + kStepRows - 1) / kStepRows;
        for (int64_t c0 = t_beg + (int64_t)wave * kAttChunkTiles; c0 < t_end;
             c0 += (int64_t)wpb * kAttChunkTiles) {
            const int64_t c1 = min(c0 + kAttChunkTiles, t_end);
            constexpr int U = 2;  // wave steps loaded before any is added
            for (int64_t tl = c0; tl < c1; tl += U) {
                int32_t col[U];
                double va[U][kAxes], yy[U];
                bool valid[U];
#pragma unroll
                for (int w = 0; w < U; ++w) {
                    const int64_t tile = (tl + w < c1) ? tl + w : c0;
                    const int64_t k = tile * kStepRows + rg;
                    valid[w] = tl + w < c1 && k >= lo && k < hi;
                    const int64_t kk = valid[w] ? k : lo;  // in-bounds stand-in
                    col[w] = tL[kk] + q;
                    yy[w] = (MODE == A2_SQ) ? 0.0 : y[rowT[kk]];
                    ld_att_tile(attT, tile, lane, va[w]);
                }
#pragma unroll
                for (int w = 0; w < U; ++w) {
                    if (!valid[w]) continue;
#pragma unroll
                    for (int ax = 0; ax < kAxes; ++ax)
                        atomicAdd(acc + ax * lw + col[w], contrib<MODE>(va[w][ax], yy[w]));
                }
            }
        }
    }
    __syncthreads();
    double* __restrict__ dst = part + (int64_t)blockIdx.x * kAxes * lw;
    for (int i = threadIdx.x; i < kAxes * lw; i += blockDim.x) dst[i] = acc[i];
}

// x[att0 + a T + c] += the sums of column c over the groups whose bucket covers it: bucket
// c / W of every die and the buckets before it whose columns reach c (the previous one for
// the first kParAxis - 1 columns of a bucket when W >= kParAxis - 1, more when W is smaller).
// check_stop: nothing is done once the LSQR stop flag is set.
static __global__ void k_att_reduce(Geo g, int w, int lw, const double* __restrict__ part,
                                    double* __restrict__ x, const LsqrState* __restrict__ st,
                                    int check_stop) {
    if (check_stop && st->stop) return;
    const int64_t n = (int64_t)kAxes * g.T;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        const int64_t ax = e / g.T, c = e - ax * g.T;
        double sum = 0.0;
        for (int64_t b = c / w; b >= 0 && c - b * w < lw; --b) {
            const double* __restrict__ p = part + (b * kXcd * kAxes + ax) * lw + (c - b * w);
#pragma unroll
            for (int d = 0; d < kXcd; ++d) sum += p[(int64_t)d * kAxes * lw];
        }
        x[g.att0 + e] += sum;
    }
}

// Library-owned attitude copy (the order of k_aprod2_att), as attitude tiles: row k of the
// copy is row rowT[k] of the system; ntiles * kTileAtt elements.
template <typename VT>
static __global__ void k_gather_att(int64_t m, int64_t ntiles, const VT* __restrict__ vals,
                                    const int32_t* __restrict__ rowT, VT* __restrict__ attT) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t total = ntiles * kTileAtt;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        const int64_t tile = e / kTileAtt;
        const int o = (int)(e - tile * kTileAtt);
        const int lane = (o < 2 * kWave) ? o / 2 : o - 2 * kWave;
        const int ax = (o < 2 * kWave) ? o % 2 : 2;
        const int64_t k = tile * kStepRows + lane / kQuad;
        const int j = kParAxis * ax + lane % kQuad;
        attT[e] = k < m ? vals[(int64_t)rowT[k] * kPar + kAstro + j] : (VT)0;
    }
}

static __global__ void k_iota(int64_t m, int32_t* __restrict__ v) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride)
        v[i] = (int32_t)i;
}

// Sort key of row i for the attitude copy: group G = (t / w) kXcd + (slice % kXcd) above the
// slice's number on its die (sbits wide) above t - (t / w) w (tbits wide); slice = i >> shift.
static __global__ void k_att_keys(int64_t m, int shift, int w, int sbits, int tbits,
                                  const int32_t* __restrict__ att, uint64_t* __restrict__ key) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const int64_t slice = i >> shift, t = att[i], b = t / w;
        const uint64_t grp = (uint64_t)(b * kXcd + slice % kXcd);
        key[i] = (((grp << sbits) | (uint64_t)(slice / kXcd)) << tbits) | (uint64_t)(t - b * w);
    }
}

// seg[G] = first position of group G in the sorted keys (G = 0 .. ng; seg[ng] = m).
static __global__ void k_att_seg(int64_t m, int ng, int low_bits, const uint64_t* __restrict__ key,
                                 int64_t* __restrict__ seg) {
    const int grp = blockIdx.x * blockDim.x + threadIdx.x;
    if (grp > ng) return;
    const uint64_t target = (uint64_t)grp << low_bits;
    int64_t lo = 0, hi = m;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (key[mid] < target)
            lo = mid + 1;
        else
            hi = mid;
    }
    seg[grp] = lo;
}

// The column offset in the bucket, t - b w, from each sorted key.
static __global__ void k_att_tl(int64_t m, uint64_t mask, const uint64_t* __restrict__ key,
                                int32_t* __restrict__ tl) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride)
        tl[i] = (int32_t)(key[i] & mask);
}

}  // namespace gsr
