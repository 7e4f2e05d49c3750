// Batched form: n_sys independent systems stored back to back, K right-hand sides each,
// solved together (declarations and contracts in include/gsr.h).
//
// Every (system, right-hand side) pair runs its own PC-LSQR recurrence (LsqrState per
// pair); the matrix of each system is read once per product for all K right-hand sides
// (sparse matrix times K-column block, RHS-minor storage so the K values of one row or
// column form one contiguous 8K-byte piece).
// Work is described by lists of segments that never cross a system boundary:
//   row chunks    (one wave walks a chunk: products, row-space vector steps, partial sums),
//   block chunks  (one block walks a chunk: star-ordered pass of aprod 2, LDS per system),
//   rounds        (one block: the row pass of the solver),
//   attitude chunks (one wave: runs of t-ordered rows),
//   column tiles  (one block: unknown-space vector steps).
// A whole fixed-iteration solve is captured in one hipGraph and launched once.  Round
// length and block size of the row pass are picked per batch shape by timing candidates
// (autotuner).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "gsr_internal.hpp"
#include "products.hpp"

#include <hipcub/hipcub.hpp>

namespace gsr {

struct SysDesc {
    int64_t row0, m;   // rows [row0, row0 + m) of the concatenated arrays
    int64_t col0, n;   // unknowns [col0, col0 + n) of the batched vector
    int64_t att0, ins0, glb0;  // section bases relative to col0
    int64_t n_stars;
    int32_t T, I;
    int32_t chunk0, nchunk;    // row chunks of the system
    int32_t tile0, ntile;      // column tiles of the system
    int32_t round0, nround;    // rounds of the system
    int64_t btile0;            // first row tile of the system (rows padded to whole tiles)
};

struct Seg {
    int64_t e0, e1;  // rows or columns (global)
    int32_t sys, pad;
};

constexpr int kBTileMin = 256, kBTileMax = 2048;  // columns per tile

// Block index renumbered so that the blocks of one die are consecutive: contiguous work
// ranges (one or a few systems) then stay on one die and share its L2.
__device__ __forceinline__ int xcd_block(int b, int G) {
    const int per = G / kXcd, rem = G % kXcd;
    const int x = b % kXcd, i = b / kXcd;
    return x * per + min(x, rem) + i;
}

// ---------------------------------------------------------------------------------------
// products

// Y[r, j] (op)= sum_k A[r,k] X[col0 + col(r,k), j]
template <typename VT, int MODE, int K>
static __global__ __launch_bounds__(256) void k_baprod1(
    const SysDesc* __restrict__ sys, const Seg* __restrict__ chunks, int nchunks,
    const VT* __restrict__ vals, const int32_t* __restrict__ star,
    const int32_t* __restrict__ att, const int32_t* __restrict__ instr,
    const double* __restrict__ X, double* __restrict__ Y, const double* __restrict__ B,
    const LsqrState* __restrict__ st, double* __restrict__ partials) {
    constexpr bool kLsqr = (MODE == A1_LSQR);
    constexpr int RS = kWave / K;  // rows per wave step
    const int lane = threadIdx.x % kWave, rr = lane / K, j = lane % K;
    const int wpb = blockDim.x / kWave;
    for (int ch = blockIdx.x * wpb + threadIdx.x / kWave; ch < nchunks; ch += gridDim.x * wpb) {
        const Seg c = chunks[ch];
        const SysDesc d = sys[c.sys];
        bool live = true;
        double xs = 1.0, ys = 0.0;
        if (kLsqr) {
            const LsqrState* p = st + (int64_t)c.sys * K + j;
            live = !p->stop;
            xs = p->sv;
            ys = p->alpha * p->su;
        }
        const double* __restrict__ Xs = X + d.col0 * K + j;
        double acc = 0.0;
        for (int64_t r0 = c.e0; r0 < c.e1; r0 += RS) {
            const int64_t r = r0 + rr;
            if (!(live && r < c.e1)) continue;
            const VT* __restrict__ row = vals + r * kPar;
            double a[kPar];
#pragma unroll
            for (int k = 0; k < kPar; ++k) a[k] = ld_val(row + k);
            const int32_t s = star[r], t = att[r];
            int32_t ins[kInstr];
#pragma unroll
            for (int k = 0; k < kInstr; ++k) ins[k] = instr[r * kInstr + k];
            double sum = 0.0;
#pragma unroll
            for (int k = 0; k < kAstro; ++k) sum = fma(a[k], Xs[((int64_t)kAstro * s + k) * K], sum);
#pragma unroll
            for (int ax = 0; ax < kAxes; ++ax)
#pragma unroll
                for (int k = 0; k < kParAxis; ++k)
                    sum = fma(a[kAstro + ax * kParAxis + k],
                              Xs[(d.att0 + (int64_t)ax * d.T + t + k) * K], sum);
#pragma unroll
            for (int k = 0; k < kInstr; ++k) sum = fma(a[17 + k], Xs[(d.ins0 + ins[k]) * K], sum);
            sum = fma(a[23], Xs[d.glb0 * K], sum);
            double* yp = Y + r * K + j;
            if (MODE == A1_ADD) {
                *yp += sum;
            } else if (MODE == A1_RESID) {
                *yp = B[r * K + j] - sum;
            } else {
                const double u = (ys != 0.0) ? xs * sum - ys * *yp : xs * sum;
                *yp = u;
                acc = fma(u, u, acc);
            }
        }
        if (kLsqr) {
#pragma unroll
            for (int off = K; off < kWave; off <<= 1) acc += __shfl_xor(acc, off, kWave);
            if (lane < K) partials[(int64_t)ch * K + j] = acc;
        }
    }
}

// Star-ordered pass of X[c, j] += A[r, c] yy[r, j] (astrometric, instrumental, global).
// Block chunks are walked by whole blocks; each wave takes a contiguous sub-range.  The
// instrumental and global sums of the current system live in LDS and are added to X with
// one atomic per (column, j) when the block moves to another system or finishes.
template <int K>
static __global__ __launch_bounds__(512) void k_baprod2_star(
    const SysDesc* __restrict__ sys, const Seg* __restrict__ bchunks, int nbchunks,
    const double* __restrict__ vals, const int32_t* __restrict__ star,
    const int32_t* __restrict__ instr, const double* __restrict__ Y, double* __restrict__ X,
    int max_instr) {
    extern __shared__ double lds[];  // [(max_instr + 1) * K]
    constexpr int RS = kWave / K;
    const int lane = threadIdx.x % kWave, rr = lane / K, j = lane % K;
    const int w = threadIdx.x / kWave, wpb = blockDim.x / kWave;
    const int per = (nbchunks + gridDim.x - 1) / gridDim.x;
    const int bc_beg = xcd_block(blockIdx.x, gridDim.x) * per, bc_end = min(nbchunks, bc_beg + per);
    const int nl = (max_instr + 1) * K;
    for (int e = threadIdx.x; e < nl; e += blockDim.x) lds[e] = 0.0;
    __syncthreads();
    int cur = -1;
    SysDesc d = {};
    double gacc = 0.0;
    auto flush_lds = [&]() {
        const double gs = [&] {
            double v = gacc;
#pragma unroll
            for (int off = K; off < kWave; off <<= 1) v += __shfl_xor(v, off, kWave);
            return v;
        }();
        if (lane < K) atomicAdd(lds + d.I * K + j, gs);
        gacc = 0.0;
        __syncthreads();
        const int ne = (d.I + 1) * K;
        double* xi = X + (d.col0 + d.ins0) * K;  // instrumental then global: contiguous
        for (int e = threadIdx.x; e < ne; e += blockDim.x) {
            const double v = lds[e];
            if (v != 0.0) atomic_add_f64(xi + e, v);
            lds[e] = 0.0;
        }
        __syncthreads();
    };
    for (int bc = bc_beg; bc < bc_end; ++bc) {
        const Seg c = bchunks[bc];
        if (c.sys != cur) {
            if (cur >= 0) flush_lds();
            cur = c.sys;
            d = sys[cur];
        }
        // this wave's contiguous sub-range of the block chunk
        const int64_t len = c.e1 - c.e0;
        const int64_t sub = ((len + wpb - 1) / wpb + RS - 1) / RS * RS;
        const int64_t r_beg = min(c.e1, c.e0 + w * sub), r_end = min(c.e1, r_beg + sub);
        const int64_t sys_end = d.row0 + d.m;
        const int32_t shared_first =
            (r_beg < r_end && r_beg > d.row0 && star[r_beg - 1] == star[r_beg]) ? star[r_beg] : -1;
        const int32_t shared_last =
            (r_beg < r_end && r_end < sys_end && star[r_end] == star[r_end - 1]) ? star[r_end - 1]
                                                                                : -1;
        double* __restrict__ Xa = X + d.col0 * K + j;
        // finished star: the lanes of row group 0 add it
        auto flush = [&](int32_t key, const double (&t)[kAstro]) {
            if (rr != 0) return;
            double* xa = Xa + (int64_t)kAstro * key * K;
            if (key == shared_first || key == shared_last) {
#pragma unroll
                for (int q = 0; q < kAstro; ++q) atomic_add_f64(xa + q * K, t[q]);
            } else {
#pragma unroll
                for (int q = 0; q < kAstro; ++q) xa[q * K] += t[q];
            }
        };
        double acc[kAstro] = {0.0, 0.0, 0.0, 0.0, 0.0};
        int32_t ckey = -1;
        for (int64_t r0 = r_beg; r0 < r_end; r0 += RS) {
            const int64_t r = r0 + rr;
            const bool valid = r < r_end;
            int32_t key = -1;
            double v[kAstro] = {0.0, 0.0, 0.0, 0.0, 0.0};
            if (valid) {
                const double* __restrict__ row = vals + r * kPar;
                key = star[r];
                const double yy = Y[r * K + j];
#pragma unroll
                for (int q = 0; q < kAstro; ++q) v[q] = ld_val(row + q) * yy;
#pragma unroll
                for (int q = 0; q < kInstr; ++q) {
                    const int32_t ic = instr[r * kInstr + q];
                    atomicAdd(lds + ic * K + j, ld_val(row + 17 + q) * yy);
                }
                gacc += ld_val(row + 23) * yy;
            }
            run_step<kAstro, K>(key, v, acc, ckey, flush);
        }
        run_close<kAstro, K>(acc, ckey, flush);
    }
    if (cur >= 0) flush_lds();
}

// The t-ordered attitude copy: the 12 attitude coefficients of each t-ordered row, row after row
// (each system's rows padded to whole tiles, as its row tiles are).
constexpr int kAttRow = kAxes * kParAxis;

static __global__ void k_make_batt_rows(int64_t m, int64_t row0, const double* __restrict__ vals,
                                        const int32_t* __restrict__ rowT,
                                        double* __restrict__ at) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m * kAttRow; e += stride)
        at[e] = vals[(int64_t)rowT[row0 + e / kAttRow] * kPar + kAstro + e % kAttRow];
}

// R consecutive doubles (16-byte pieces when R is even; p then 16-byte aligned).
template <int R>
__device__ __forceinline__ void ld_r(const double* __restrict__ p, double (&o)[R]) {
    if constexpr (R % 2 == 0) {
#pragma unroll
        for (int i = 0; i < R; i += 2) {
            const f64x2 t = *reinterpret_cast<const f64x2*>(p + i);
            o[i] = t.x;
            o[i + 1] = t.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < R; ++i) o[i] = p[i];
    }
}
template <int R>
__device__ __forceinline__ void st_r(double* __restrict__ p, const double (&v)[R]) {
    if constexpr (R % 2 == 0) {
#pragma unroll
        for (int i = 0; i < R; i += 2) *reinterpret_cast<f64x2*>(p + i) = f64x2{v[i], v[i + 1]};
    } else {
#pragma unroll
        for (int i = 0; i < R; ++i) p[i] = v[i];
    }
}

// Column of XT = p o V, the operand of the row pass (the library's own), that holds column c of
// system d: the attitude columns lie knot by knot (the three axes of a knot together), so that a
// row's twelve are one contiguous piece (eight right-hand sides: 768 bytes, 6 to 7 cache lines;
// axis by axis 9, and in planes of two right-hand sides 10).
__device__ __forceinline__ int64_t xt_col(const SysDesc& d, int64_t c) {
    const int64_t t = c - d.att0;
    if (t < 0 || t >= (int64_t)kAxes * d.T) return c;
    const int ax = t >= 2 * (int64_t)d.T ? 2 : t >= d.T ? 1 : 0;
    return d.att0 + kAxes * (t - (int64_t)ax * d.T) + ax;
}

// Batched row pass: for every (row, right-hand side j) of a round
//   U[r, j] = sv_j (A XT)[r, j] - alpha_j su_j U[r, j]   (BR_LSQR; BR_T: U as it is, BR_SQ: the
//   squared coefficients, no U)
// and S += A^T U except the attitude columns, reading each row once.  Sum U^2 per (round, j) ->
// partials.  Pairs that have stopped keep their U and contribute nothing.
// The quad of a row holds its coefficients as in the single-system pass (TileRow).
//   K <= 2 : as there, each lane takes its own columns of the row, for all right-hand sides, and
//            the quad adds up;
//   K >= 4 : each lane takes R = K / 4 right-hand sides and all columns of the row, the
//            coefficients passed round the quad by DPP: a load instruction then reads whole
//            pieces of 16 R bytes per column, and the row's u~ needs no sum over lanes (with the
//            columns split and eight right-hand sides per lane: 1.82 ms against 1.61).
// A round (one entry of `rounds`, consecutive rows of one system) keeps its stars' sums in LDS
// and writes them at its end; with K <= 2 its U too, as the single-system pass does (with K >= 4
// a wave step's U is one piece of 512 bytes or more and is written at once: no slower, and the
// LDS holds longer rounds).  The instrumental sums of the current system stay in LDS until the
// block moves to another system.
// Star sums: a star's rows within the wave step are a contraction (coefficients x rows times
// rows x right-hand sides), taken by the 4 x 4 x 4 binary64 matrix instruction, whose operand
// layout is the one the row's lanes already have: lane l holds coefficient l % 4 of row l / 4,
// in block (l / 4) % 4 and place l / 16 of it, and right-hand side l % 4 of the same row; the
// four blocks are added over the lanes and one lane per sum adds it to the star's LDS slot
// (with every lane adding its own product, sixteen LDS atomics fall on one address, 47 clocks
// per instruction against 9 on separate ones).
// What bounds it with K = 8: the vector memory path.  16 systems of 1.31e7 rows: 1.61 ms
// (2.9 TB/s of the algorithmic bytes); without its LDS work 1.49, without the attitude columns'
// cache misses 1.33, without any gather (BR_T) 0.63.  64 systems of 1.76e6 rows with K = 2: 127
// (coefficients of a whole row in every lane, sums of stars over lanes) -> 98 us.  BR_T against
// the star-ordered pass with 8 row groups per wave: 1.19 -> 0.63 ms.
// Rounds are dealt to the blocks so that each die takes an eighth of them in system order and
// its blocks move through the systems together, sharing each system's columns in the die's L2.
enum { BR_LSQR = 0, BR_T = 1, BR_SQ = 2 };
constexpr int kBRowBlock = 1024;

struct BRowArgs {
    const SysDesc* sys;
    const Seg* rounds;
    int nrounds;
    const double* tiles;
    const int32_t* star;
    const double* XT;
    double *U, *S;
    const LsqrState* st;
    double* partials;
    int I;      // most instrumental columns of a system
    int rows;   // most rows of a round (LDSI or not)
    int nsb;    // stars of a round with a slot
};

// LDS doubles of a block: sums, sums of squares, staged XT, U of the round, star slots.
__host__ __device__ constexpr int64_t brow_fixed(int k, int I, bool ldsi) {
    return (int64_t)k * (I + 1) + k + (k * (I + 1)) % 2 + k % 2 +
           (ldsi ? (int64_t)k * I + (k * I) % 2 : 0);
}

// The value of one lane of each quad (quad_perm [s,s,s,s] = s * 0x55), in all its lanes.
template <int CTRL>
__device__ __forceinline__ int32_t quad_lane(int32_t v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}

// A value that is the same in all lanes of a wave, in scalar registers.
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform(int64_t v) {
    return (int64_t)(uint32_t)uniform((int32_t)v) | (int64_t)uniform((int32_t)(v >> 32)) << 32;
}
__device__ __forceinline__ double uniform(double v) {
    return __hiloint2double(uniform(__double2hiint(v)), uniform(__double2loint(v)));
}

template <int K, int MODE, bool LDSI>
static __global__ __launch_bounds__(kBRowBlock) void k_browpass(BRowArgs p) {
    constexpr int L = K >= 4 ? 4 : 1;  // lanes of a quad that share out the right-hand sides
    constexpr int R = K / L;           // right-hand sides of a lane
    constexpr bool kDot = MODE == BR_LSQR;
    constexpr bool kBurst = kDot && L == 1;
    extern __shared__ double lds[];
    const int li = p.I + 1;
    double* lsum = lds;                             // [I + 1][K]
    double* lusq = lsum + K * li + (K * li) % 2;    // [K]
    double* lxi = lusq + K + K % 2;                 // [I][K]
    double* ubuf = lxi + (LDSI ? K * p.I + (K * p.I) % 2 : 0);  // [rows][K]
    double* sbuf = ubuf + (kBurst ? (int64_t)p.rows * K : 0);  // [nsb][kAstro][K]
    const int lane = threadIdx.x % kWave, rg = lane / kQuad, q = lane % kQuad;
    const int j0 = L == 1 ? 0 : q * R;
    const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    const int ngrp = min((int)gridDim.x, kXcd);
    const int grp = blockIdx.x % ngrp, gi = blockIdx.x / ngrp;
    const int nbg = gridDim.x / ngrp + (grp < (int)gridDim.x % ngrp ? 1 : 0);
    const int rd_beg = (int)((int64_t)p.nrounds * grp / ngrp);
    const int rd_end = (int)((int64_t)p.nrounds * (grp + 1) / ngrp);
    for (int e = threadIdx.x; e < K * li + (K * li) % 2 + K; e += blockDim.x) lds[e] = 0.0;
    for (int e = threadIdx.x; e < kAstro * K * p.nsb; e += blockDim.x) sbuf[e] = 0.0;
    __syncthreads();
    int cur = -1;
    SysDesc d = {};
    auto flush_sums = [&]() {  // instrumental then global columns, contiguous in S
        double* xi = p.S + (d.col0 + d.ins0) * K;
        for (int e = threadIdx.x; e < (d.I + 1) * K; e += blockDim.x) {
            double* l = lsum + (e < d.I * K ? e : e + (p.I - d.I) * K);
            const double v = *l;
            if (v != 0.0) atomic_add_f64(xi + e, v);
            *l = 0.0;
        }
        __syncthreads();
    };
    for (int rd = rd_beg + gi; rd < rd_end; rd += nbg) {
        Seg c = p.rounds[rd];
        c = {uniform(c.e0), uniform(c.e1), uniform(c.sys), 0};
        if (c.sys != cur) {
            if (cur >= 0) flush_sums();
            cur = c.sys;
            const SysDesc t = p.sys[cur];
            d.row0 = uniform(t.row0);
            d.m = uniform(t.m);
            d.col0 = uniform(t.col0);
            d.att0 = uniform(t.att0);
            d.ins0 = uniform(t.ins0);
            d.glb0 = uniform(t.glb0);
            d.I = uniform(t.I);
            d.btile0 = uniform(t.btile0);
            if (kDot && LDSI) {
                const double* xs_i = p.XT + (d.col0 + d.ins0) * K;
                for (int e = threadIdx.x; e < d.I * K; e += blockDim.x) lxi[e] = xs_i[e];
                __syncthreads();
            }
        }
        // this lane's right-hand sides j0 .. j0 + R - 1 (K <= 2: all of them)
        const LsqrState* ps = p.st + (int64_t)cur * K;
        bool live[R], any_live = MODE == BR_SQ;
        double xs[R], ys[R], xglob[R];
#pragma unroll
        for (int j = 0; j < K; ++j) any_live = any_live || !ps[j].stop;
        if (!any_live) continue;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            live[i] = MODE == BR_SQ || !ps[j0 + i].stop;
            if (kDot) {
                xs[i] = ps[j0 + i].sv;
                ys[i] = ps[j0 + i].alpha * ps[j0 + i].su;
                xglob[i] = p.XT[(d.col0 + d.glb0) * K + j0 + i];
            }
        }
        const int64_t R0 = c.e0, R1 = c.e1;
        const int64_t T0 = d.btile0 + (R0 - d.row0) / kStepRows;
        const int nt = (int)((R1 - R0 + kStepRows - 1) / kStepRows);
        const int32_t S0 = uniform(p.star[R0]), S1 = uniform(p.star[R1 - 1]);
        const bool shf = R0 > d.row0 && p.star[R0 - 1] == S0;
        const bool shl = R1 < d.row0 + d.m && p.star[R1] == S1;
        const double* __restrict__ Xs = p.XT + d.col0 * K + j0;
        double usq[R] = {};
        const double* __restrict__ xi = (LDSI ? lxi : p.XT + (d.col0 + d.ins0) * K) + j0;
        for (int t = w; t < nt; t += nw) {
            TileRow a;
            ld_tile(p.tiles, T0 + t, lane, a);
            ld_tile_idx(p.tiles, T0 + t, lane, a);
            const int64_t r = R0 + (int64_t)t * kStepRows + rg;
            const bool valid = r < R1;
            const int32_t s_first = __builtin_amdgcn_readlane(a.star, 0);
            const int32_t s_last = __builtin_amdgcn_readlane(a.star, kWave - 1);
            const bool two = q == 1 || q == 2;  // lanes with a second instrumental coefficient
            const double* xa = Xs + (int64_t)kAstro * a.star * K;
            const double* xt = Xs + (d.att0 + (int64_t)kAxes * a.att) * K;
            double un[R], sum[R];
            if (MODE != BR_SQ) ld_r<R>(p.U + min(r, R1 - 1) * K + j0, un);
            // all loads without branches: a load under a lane condition would wait for the
            // ones before it
            if constexpr (kDot && L == 1) {
                double x0[R], x4[R], e01[2 * R], e2[R], wx[R], wb[R];
                ld_r<R>(xa + q * K, x0);
                ld_r<R>(xa + 4 * K, x4);
                if constexpr (R == 1) {
                    typedef f64x2 __attribute__((aligned(8))) f64x2u;
                    const f64x2 v = *reinterpret_cast<const f64x2u*>(xt + 2 * q);
                    e01[0] = v.x;
                    e01[1] = v.y;
                } else {
                    ld_r<2 * R>(xt + 2 * q * R, e01);
                }
                ld_r<R>(xt + (8 + q) * R, e2);
                __builtin_amdgcn_sched_barrier(0);
                ld_r<R>(xi + a.ia * K, wx);
                ld_r<R>(xi + (two ? a.ib : a.ia) * K, wb);
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    double v = a.as * x0[i];
                    v = fma(a.e0, e01[i], v);
                    v = fma(a.e1, e01[R + i], v);
                    v = fma(a.e2, e2[i], v);
                    v = fma(a.wi, wx[i], v);
                    v = fma(a.z, q == 0 ? x4[i] : two ? wb[i] : xglob[i], v);
                    sum[i] = quad_sum(v);
                }
            }
            int ic[kInstr];      // K >= 4: the row's instrumental columns and coefficients
            double ci[kInstr];
            if constexpr (L == 4) {
                ic[0] = quad_lane<0x00>(a.ia);
                ic[1] = quad_lane<0x55>(a.ia);
                ic[2] = quad_lane<0xAA>(a.ia);
                ic[3] = quad_lane<0xFF>(a.ia);
                ic[4] = quad_lane<0x55>(a.ib);
                ic[5] = quad_lane<0xAA>(a.ib);
                ci[0] = dpp_f64<0x00>(a.wi);
                ci[1] = dpp_f64<0x55>(a.wi);
                ci[2] = dpp_f64<0xAA>(a.wi);
                ci[3] = dpp_f64<0xFF>(a.wi);
                ci[4] = dpp_f64<0x55>(a.z);
                ci[5] = dpp_f64<0xAA>(a.z);
            }
            if constexpr (kDot && L == 4) {
                double x[kAxes * kParAxis + kAstro][R];
#pragma unroll
                for (int e = 0; e < kAxes * kParAxis; ++e) ld_r<R>(xt + e * K, x[e]);
#pragma unroll
                for (int e = 0; e < kAstro; ++e) ld_r<R>(xa + e * K, x[kAxes * kParAxis + e]);
#pragma unroll
                for (int i = 0; i < R; ++i) sum[i] = dpp_f64<0xFF>(a.z) * xglob[i];
#pragma unroll
                for (int k = 0; k < kInstr; ++k) {
                    double v[R];
                    ld_r<R>(xi + ic[k] * K, v);
#pragma unroll
                    for (int i = 0; i < R; ++i) sum[i] = fma(ci[k], v[i], sum[i]);
                }
                auto add = [&](double c, const double (&v)[R]) {
#pragma unroll
                    for (int i = 0; i < R; ++i) sum[i] = fma(c, v[i], sum[i]);
                };
                add(dpp_f64<0x00>(a.e0), x[0]);
                add(dpp_f64<0x00>(a.e1), x[1]);
                add(dpp_f64<0x55>(a.e0), x[2]);
                add(dpp_f64<0x55>(a.e1), x[3]);
                add(dpp_f64<0xAA>(a.e0), x[4]);
                add(dpp_f64<0xAA>(a.e1), x[5]);
                add(dpp_f64<0xFF>(a.e0), x[6]);
                add(dpp_f64<0xFF>(a.e1), x[7]);
                add(dpp_f64<0x00>(a.e2), x[8]);
                add(dpp_f64<0x55>(a.e2), x[9]);
                add(dpp_f64<0xAA>(a.e2), x[10]);
                add(dpp_f64<0xFF>(a.e2), x[11]);
                add(dpp_f64<0x00>(a.as), x[12]);
                add(dpp_f64<0x55>(a.as), x[13]);
                add(dpp_f64<0xAA>(a.as), x[14]);
                add(dpp_f64<0xFF>(a.as), x[15]);
                add(dpp_f64<0x00>(a.z), x[16]);
            }
            if (kDot) {
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const double u = (ys[i] != 0.0) ? xs[i] * sum[i] - ys[i] * un[i]
                                                    : xs[i] * sum[i];
                    un[i] = live[i] ? u : un[i];
                }
                if (kBurst) {
                    if (q == 0) st_r<R>(ubuf + (t * kStepRows + rg) * K, un);
                } else if (valid) {
                    double* up = p.U + r * K + j0;
                    if constexpr (R == 2)
                        __builtin_nontemporal_store(f64x2{un[0], un[1]}, reinterpret_cast<f64x2*>(up));
                    else
                        __builtin_nontemporal_store(un[0], up);
                }
            }
            double ul[R];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                ul[i] = MODE == BR_SQ ? 1.0 : (live[i] && valid) ? un[i] : 0.0;
                if (!kBurst && kDot) usq[i] = fma(ul[i], ul[i], usq[i]);
            }
            if (MODE == BR_SQ) {
                a.as *= a.as;
                a.z *= a.z;
                a.wi *= a.wi;
            }
            if constexpr (L == 4) {
                // odd rows take their right-hand sides in the other order: the lanes of an
                // atomic then spread over all banks
                double* lj = lsum + j0;
                const int odd = R == 2 ? rg & 1 : 0;
                const double u0 = odd ? ul[R - 1] : ul[0], u1 = odd ? ul[0] : ul[R - 1];
#pragma unroll
                for (int k = 0; k < kInstr; ++k) {
                    double* l = lj + ic[k] * K;
                    atomicAdd(l + odd, ci[k] * u0);
                    if (R == 2) atomicAdd(l + (1 - odd), ci[k] * u1);
                }
            } else {
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    atomicAdd(lsum + a.ia * K + i, a.wi * ul[i]);
                    if (two) atomicAdd(lsum + a.ib * K + i, a.z * ul[i]);
                }
            }
            // stars and the global column; lane l of a product of the matrix instruction holds
            // right-hand side jq of coefficient l / 16, in block (l / 4) % 4
#pragma unroll
            for (int i = 0; i < (L == 4 ? R : 1); ++i) {
                const double y = L == 4 ? ul[i] : R == 2 && (q & 1) ? ul[R - 1] : ul[0];
                const int jq = L == 4 ? j0 + i : q, co = lane / 16;
                const bool mine = (lane & 12) == 0 && jq < K;
                for (int32_t cs = s_first;;) {  // each star of the wave step
                    const bool in = a.star == cs;
                    const double ym = in ? y : 0.0;
                    double ta = __builtin_amdgcn_mfma_f64_4x4x4f64(in ? a.as : 0.0, ym, 0.0, 0, 0, 0);
                    double tz = __builtin_amdgcn_mfma_f64_4x4x4f64(in ? a.z : 0.0, ym, 0.0, 0, 0, 0);
                    ta += dpp_f64<0x124>(ta);
                    ta += dpp_f64<0x128>(ta);
                    tz += dpp_f64<0x124>(tz);
                    tz += dpp_f64<0x128>(tz);
                    const int o = cs - S0;
                    if (o < p.nsb) {
                        if (mine) {
                            atomicAdd(sbuf + (kAstro * o + co) * K + jq, ta);
                            if (co == 0) atomicAdd(sbuf + (kAstro * o + 4) * K + jq, tz);
                        }
                    } else {  // past the last slot: straight to S, which is zero there
                        keep_apart();
                        if (mine) {
                            double* xo = p.S + (d.col0 + (int64_t)kAstro * cs) * K + jq;
                            atomic_add_f64(xo + co * K, ta);
                            if (co == 0) atomic_add_f64(xo + 4 * K, tz);
                        }
                        keep_apart();
                    }
                    if (mine && co == 3) atomicAdd(lsum + p.I * K + jq, tz);
                    if (cs == s_last) break;
                    const uint64_t more = __ballot(a.star > cs);
                    cs = __builtin_amdgcn_readlane(a.star, __ffsll((unsigned long long)more) - 1);
                }
            }
        }
        __syncthreads();
        if (kDot && !kBurst) {
#pragma unroll
            for (int i = 0; i < R; ++i) {
#pragma unroll
                for (int off = kQuad; off < kWave; off <<= 1)
                    usq[i] += __shfl_xor(usq[i], off, kWave);
                if (lane < kQuad) atomicAdd(lusq + j0 + i, usq[i]);
            }
        }
        if (kBurst) {  // the round's U in one burst, and its sum of squares
            constexpr int W = K >= 2 ? 2 : 1, P = K / W;
            double acc[W] = {};
            typedef double vec __attribute__((ext_vector_type(W)));
            vec* dst = reinterpret_cast<vec*>(p.U + R0 * K);
            const vec* src = reinterpret_cast<const vec*>(ubuf);
            for (int e = threadIdx.x; e < (int)(R1 - R0) * P; e += blockDim.x) {
                const vec v = src[e];
                __builtin_nontemporal_store(v, dst + e);
#pragma unroll
                for (int i = 0; i < W; ++i) acc[i] = fma(v[i], v[i], acc[i]);
            }
#pragma unroll
            for (int i = 0; i < W; ++i) {
#pragma unroll
                for (int off = P; off < kWave; off <<= 1) acc[i] += __shfl_xor(acc[i], off, kWave);
                if (lane < P) atomicAdd(lusq + lane * W + i, acc[i]);
            }
        }
        // finished stars: owned ones are stored (S is zero before the pass)
        const int ns = min(S1 - S0 + 1, p.nsb);
        const int e0 = shf ? kAstro * K : 0;
        const int e1 = (shl ? S1 - S0 : S1 - S0 + 1) * kAstro * K;
        double* xo = p.S + (d.col0 + (int64_t)kAstro * S0) * K;
        for (int e = threadIdx.x; e < ns * kAstro * K; e += blockDim.x) {
            const double v = sbuf[e];
            sbuf[e] = 0.0;
            if (e >= e0 && e < e1)
                __builtin_nontemporal_store(v, xo + e);
            else
                atomic_add_f64(xo + e, v);
        }
        __syncthreads();
        if (kDot && threadIdx.x < K) {
            p.partials[(int64_t)rd * K + threadIdx.x] = lusq[threadIdx.x];
            lusq[threadIdx.x] = 0.0;
        }
    }
    __syncthreads();
    if (cur >= 0) flush_sums();
}

// Attitude pass over the t-ordered copy (each system's rows keep their own range): the 12
// columns x K right-hand sides of a run of rows with one start t are a contraction over its
// rows, 12 x rows times rows x K, and go through the binary64 matrix instruction, four rows at
// a time: lane (i, k) = (lane % 16, lane / 16) holds coefficient i of row k and right-hand side
// i of row k (one 8-byte load each, no value twice), and the sums of column q of axis r end in
// register r of lane (j, q).  With the products in vector registers instead, every lane of a
// row needed all 12 coefficients and 8 rows were in flight per wave.
// Bound by memory: 1.31e7 rows with K = 8 0.70 -> 0.56 ms (3.9 TB/s); of these the coefficients
// cost 0.21 ms, the order of U's rows 0.09 (against U read in order) and the atomics of the
// finished runs 0.07.  1.76e6 rows with K = 2: 58 us before and after.
template <int MODE, int K>
static __global__ __launch_bounds__(256, 4) void k_baprod2_att(
    const SysDesc* __restrict__ sys, const Seg* __restrict__ chunks, int nchunks,
    const double* __restrict__ attT, const int32_t* __restrict__ rowT,
    const int32_t* __restrict__ tT, const double* __restrict__ Y, double* __restrict__ X,
    const LsqrState* __restrict__ st) {
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    constexpr int G = 8, B = 4 * G;  // groups of four rows, and rows, in flight
    constexpr int NA = 2;            // sums a run is split over: shorter chains of additions
    const int lane = threadIdx.x % kWave, i = lane % 16, kq = lane / 16;
    const int ic = min(i, kAttRow - 1), j = min(i, K - 1);
    const int wpb = blockDim.x / kWave;
    for (int ch = blockIdx.x * wpb + threadIdx.x / kWave; ch < nchunks; ch += gridDim.x * wpb) {
        const Seg c = chunks[ch];
        const SysDesc d = sys[c.sys];
        const bool live = i < K && (MODE != A2_LSQR || !st[(int64_t)c.sys * K + j].stop);
        if (!__any(live)) continue;
        const double* __restrict__ A = attT + (d.btile0 * kStepRows - d.row0) * kAttRow + ic;
        double* __restrict__ Xt = X + (d.col0 + d.att0) * K + j;
        f64x4 acc[NA] = {};
        int32_t ckey = -1;
        auto flush = [&]() {
            if (live && ckey >= 0)
#pragma unroll
                for (int ax = 0; ax < kAxes; ++ax)
                    atomic_add_f64(Xt + ((int64_t)ax * d.T + ckey + kq) * K,
                                   acc[0][ax] + acc[1][ax]);
#pragma unroll
            for (int h = 0; h < NA; ++h) acc[h] = {0.0, 0.0, 0.0, 0.0};
        };
        int64_t kn = min(c.e0 + lane % B, c.e1 - 1);
        int32_t nkey = tT[kn], nrow = rowT[kn];
        for (int64_t k0 = c.e0; k0 < c.e1; k0 += B) {
            const int32_t key = k0 + lane % B < c.e1 ? nkey : -1;
            const int32_t row = nrow;
            double a[G], y[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int r = 4 * g + kq;
                a[g] = __builtin_nontemporal_load(A + min(k0 + r, c.e1 - 1) * kAttRow);
                if (MODE != A2_SQ) y[g] = Y[(int64_t)__shfl(row, r, kWave) * K + j];
            }
            kn = min(k0 + B + lane % B, c.e1 - 1);
            nkey = tT[kn];
            nrow = rowT[kn];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (MODE == A2_SQ) {
                    a[g] *= a[g];
                    y[g] = 1.0;
                } else {
                    y[g] = live ? y[g] : 0.0;
                }
            }
            const int32_t kf = __builtin_amdgcn_readlane(key, 0);
            if (kf == __builtin_amdgcn_readlane(key, B - 1)) {  // one run, all rows present
                if (kf != ckey) {
                    flush();
                    ckey = kf;
                }
#pragma unroll
                for (int g = 0; g < G; ++g)
                    acc[g % NA] =
                        __builtin_amdgcn_mfma_f64_16x16x4f64(a[g], y[g], acc[g % NA], 0, 0, 0);
                continue;
            }
            for (int pos = 0; pos < B;) {  // each run of the block
                const int32_t k = __builtin_amdgcn_readlane(key, pos);
                if (k < 0) break;
                const uint32_t in = (uint32_t)__ballot(key == k);
                if (k != ckey) {
                    flush();
                    ckey = k;
                }
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if (((in >> (4 * g)) & 15) == 0) continue;
                    const bool m = (in >> (4 * g + kq)) & 1;
                    acc[g % NA] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                        m ? a[g] : 0.0, m ? y[g] : 0.0, acc[g % NA], 0, 0, 0);
                }
                pos = 32 - __clz(in);
            }
        }
        flush();
    }
}

// ---------------------------------------------------------------------------------------
// vectors (one block per segment; elements e = index * K + j)

// Per-segment, per-j block sums of NQ quantities -> part[(q * nseg + seg) * K + j]; a lane
// holds W neighbouring right-hand sides, lane % (K / W) the first of them.
template <int K, int W, int NQ>
__device__ __forceinline__ void seg_partials(double (&acc)[NQ][W], double* sh, double* part,
                                             int nseg, int seg) {
    constexpr int P = K / W;
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    constexpr int NW = 256 / kWave;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int i = 0; i < W; ++i) {
            double v = acc[q][i];
#pragma unroll
            for (int off = P; off < kWave; off <<= 1) v += __shfl_xor(v, off, kWave);
            if (lane < P) sh[(q * NW + w) * K + lane * W + i] = v;
        }
    __syncthreads();
    if (threadIdx.x < NQ * K) {
        const int q = threadIdx.x / K, j = threadIdx.x % K;
        double s = 0.0;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) s += sh[(q * NW + ww) * K + j];
        part[((int64_t)q * nseg + seg) * K + j] = s;
    }
    __syncthreads();
}

// u = b per pair (row segments); partial sum u^2
template <int K>
static __global__ __launch_bounds__(256) void k_bcopy_norm(const Seg* __restrict__ segs, int nseg,
                                                           const double* __restrict__ B,
                                                           double* __restrict__ U,
                                                           double* __restrict__ part) {
    __shared__ double sh[4 * K * 1];
    for (int sg = blockIdx.x; sg < nseg; sg += gridDim.x) {
        const Seg c = segs[sg];
        double acc[1][1] = {{0.0}};
        for (int64_t e = c.e0 * K + threadIdx.x; e < c.e1 * K; e += blockDim.x) {
            const double v = B[e];
            U[e] = v;
            acc[0][0] = fma(v, v, acc[0][0]);
        }
        seg_partials<K, 1, 1>(acc, sh, part, nseg, sg);
    }
}

// forward v-step over column tiles (see k_vec_v for the single system)
template <bool INIT, int K>
static __global__ __launch_bounds__(256) void k_bvec_v(const Seg* __restrict__ tiles, int ntile,
                                                       double* __restrict__ S,
                                                       const double* __restrict__ p,
                                                       double* __restrict__ V,
                                                       double* __restrict__ Wv,
                                                       double* __restrict__ Z,
                                                       double* __restrict__ XT,
                                                       const SysDesc* __restrict__ sys,
                                                       const LsqrState* __restrict__ st,
                                                       double* __restrict__ part) {
    constexpr int W = K >= 2 ? 2 : 1, P = K / W;
    __shared__ double sh[4 * 4 * K];
    const int j0 = threadIdx.x % P * W;
    for (int sg = blockIdx.x; sg < ntile; sg += gridDim.x) {
        const Seg c = tiles[sg];
        const SysDesc d = sys[c.sys];
        bool live[W], pending[W], any_live = INIT;
        double f1[W], f2[W], sv[W], c1[W], su[W];
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const LsqrState* ps = st + (int64_t)c.sys * K + j0 + i;
            live[i] = INIT || !ps->stop;
            any_live = any_live || live[i];
            pending[i] = !INIT && live[i] && ps->pending;
            f1[i] = ps->f1;
            f2[i] = ps->f2;
            sv[i] = ps->sv;
            c1[i] = INIT ? 0.0 : ps->beta * ps->sv;
            su[i] = ps->su;  // S holds A^T u~ unnormalized
        }
        double acc[4][W] = {};
        for (int64_t e = c.e0 * P + threadIdx.x; e < c.e1 * P; e += blockDim.x) {
            double s[W], v[W], w[W], z[W], x[W], zero[W] = {};
            if (any_live) {
                ld_r<W>(S + e * W, s);
                if (!INIT) {
                    ld_r<W>(V + e * W, v);
                    ld_r<W>(Wv + e * W, w);
                    ld_r<W>(Z + e * W, z);
                }
            }
            st_r<W>(S + e * W, zero);
            if (!any_live) continue;
            const int64_t col = e / P;
            const double pj = p[col];
#pragma unroll
            for (int i = 0; i < W; ++i) {
                double vn = pj * (su[i] * s[i]);
                if (INIT) {
                    z[i] = w[i] = 0.0;
                } else {
                    if (pending[i]) {
                        z[i] = fma(f1[i], w[i], z[i]);
                        w[i] = sv[i] * v[i] - f2[i] * w[i];
                        acc[1][i] = fma(z[i], z[i], acc[1][i]);
                        acc[2][i] = fma(z[i], w[i], acc[2][i]);
                        acc[3][i] = fma(w[i], w[i], acc[3][i]);
                    }
                    vn = live[i] ? vn - c1[i] * v[i] : v[i];  // a stopped pair keeps its vectors
                }
                v[i] = vn;
                x[i] = pj * vn;
                if (live[i]) acc[0][i] = fma(vn, vn, acc[0][i]);
            }
            st_r<W>(V + e * W, v);
            st_r<W>(Wv + e * W, w);
            st_r<W>(Z + e * W, z);
            st_r<W>(XT + (d.col0 + xt_col(d, col - d.col0)) * K + j0, x);
        }
        seg_partials<K, W, 4>(acc, sh, part, ntile, sg);
    }
}

// X = p o (z + pending updates) per pair
template <int K>
static __global__ __launch_bounds__(256) void k_bfinal(const Seg* __restrict__ tiles, int ntile,
                                                       const double* __restrict__ p,
                                                       double* __restrict__ Z,
                                                       double* __restrict__ Wv,
                                                       const double* __restrict__ V,
                                                       double* __restrict__ Xout,
                                                       const LsqrState* __restrict__ st) {
    const int j = threadIdx.x % K;
    for (int sg = blockIdx.x; sg < ntile; sg += gridDim.x) {
        const Seg c = tiles[sg];
        const LsqrState* ps = st + (int64_t)c.sys * K + j;
        const bool pending = ps->pending, pend_b = ps->pend_b;
        const double f1 = ps->f1, f2 = ps->f2, sv = ps->sv, fb = ps->fb;
        for (int64_t e = c.e0 * K + threadIdx.x; e < c.e1 * K; e += blockDim.x) {
            double zj = Z[e];
            if (pending) {
                const double wj = Wv[e];
                zj = fma(f1, wj, zj);
                const double wn = sv * V[e] - f2 * wj;
                if (pend_b) zj = fma(fb, wn, zj);
                Wv[e] = wn;
            }
            Z[e] = zj;
            Xout[e] = p[e / K] * zj;
        }
    }
}

// p = 1/sqrt(ss), ss reset (K = 1 vectors)
static __global__ void k_brecip_sqrt(int64_t n, double* __restrict__ ss, double* __restrict__ p,
                                     unsigned long long* __restrict__ n_empty) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    unsigned long long cnt = 0;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += stride) {
        const double s = ss[j];
        ss[j] = 0.0;
        p[j] = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
        cnt += (s > 0.0) ? 0 : 1;
    }
    if (cnt) atomicAdd(n_empty, cnt);
}

// ---------------------------------------------------------------------------------------
// scalars: one block per (system, rhs) pair

// Sums over a pair's `count` segments of NQ quantities; every thread gets them.  One wave per
// quantity when there are four, all waves on the one otherwise.
template <int K, int NQ>
__device__ __forceinline__ void pair_sums(const double* __restrict__ part, int nseg, int first,
                                          int count, int j, double (&out)[NQ]) {
    constexpr int NW = 256 / kWave;
    static_assert(NQ == 1 || NQ == NW, "quantities");
    __shared__ double sh[NW];
    const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int q = NQ == 1 ? 0 : w;
    const double* __restrict__ x = part + ((int64_t)q * nseg + first) * K + j;
    double a = 0.0;
#pragma unroll 4
    for (int s = NQ == 1 ? (int)threadIdx.x : lane; s < count; s += NQ == 1 ? 256 : kWave)
        a += x[(int64_t)s * K];
    a = wave_sum(a);
    if (lane == 0) sh[w] = a;
    __syncthreads();
    if (NQ == 1) {
        out[0] = 0.0;
        for (int k = 0; k < NW; ++k) out[0] += sh[k];
    } else {
#pragma unroll
        for (int k = 0; k < NQ; ++k) out[k] = sh[k];
    }
}

enum { BS_INIT1 = 0, BS_INIT2 = 1, BS_BETA = 2, BS_ALPHA = 3 };

template <int STEP, int K>
static __global__ __launch_bounds__(256) void k_bscal(LsqrState* __restrict__ st,
                                                      const SysDesc* __restrict__ sys, int n_sys,
                                                      const double* __restrict__ part, int nseg,
                                                      int32_t itnlim, int32_t fixed, double atol,
                                                      double btol, double conlim, int32_t k_used) {
    const int pair = blockIdx.x, sidx = pair / K, j = pair % K;
    const SysDesc d = sys[sidx];
    LsqrState* ps = st + pair;
    if (STEP == BS_INIT1) {
        double ss[1];
        pair_sums<K, 1>(part, nseg, d.chunk0, d.nchunk, j, ss);
        if (threadIdx.x == 0) {
            scal_init1(ps, ss[0], itnlim, fixed, atol, btol, conlim);
            if (j >= k_used) {  // padding right-hand side: never iterates
                ps->stop = 1;
                ps->istop = 4;
            }
        }
        return;
    }
    if (ps->stop) return;
    if (STEP == BS_INIT2) {
        double ss[1];
        pair_sums<K, 1>(part, nseg, d.tile0, d.ntile, j, ss);
        if (threadIdx.x == 0) scal_init2(ps, ss[0]);
    } else if (STEP == BS_BETA) {
        double ss[1];
        pair_sums<K, 1>(part, nseg, d.round0, d.nround, j, ss);
        if (threadIdx.x == 0) scal_beta(ps, ss[0]);
    } else {
        double ss[4];
        pair_sums<K, 4>(part, nseg, d.tile0, d.ntile, j, ss);
        if (threadIdx.x == 0) scal_alpha(ps, ss[0], ss[1], ss[2], ss[3]);
    }
}

// index checks per system (bits as k_validate)
static __global__ void k_bvalidate(const SysDesc* __restrict__ sys, const Seg* __restrict__ chunks,
                                   int nchunks, const int32_t* __restrict__ star,
                                   const int32_t* __restrict__ att,
                                   const int32_t* __restrict__ instr, int* __restrict__ flags) {
    int bad = 0;
    for (int ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
        const Seg c = chunks[ch];
        const SysDesc d = sys[c.sys];
        for (int64_t r = c.e0 + threadIdx.x; r < c.e1; r += blockDim.x) {
            const int32_t s = star[r];
            if (s < 0 || s >= d.n_stars) bad |= 1;
            if (r > d.row0 && star[r - 1] > s) bad |= 2;
            const int32_t t = att[r];
            if (t < 0 || t > d.T - kParAxis) bad |= 4;
            for (int q = 0; q < kInstr; ++q) {
                const int32_t ic = instr[r * kInstr + q];
                if (ic < 0 || ic >= d.I) bad |= 8;
            }
        }
    }
    if (bad) atomicOr(flags, bad);
}

// sort keys: (system << tbits) | t
static __global__ void k_bkeys(const SysDesc* __restrict__ sys, const Seg* __restrict__ chunks,
                               int nchunks, const int32_t* __restrict__ att, int tbits,
                               uint64_t* __restrict__ keys, int32_t* __restrict__ iota) {
    for (int ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
        const Seg c = chunks[ch];
        for (int64_t r = c.e0 + threadIdx.x; r < c.e1; r += blockDim.x) {
            keys[r] = ((uint64_t)c.sys << tbits) | (uint64_t)(uint32_t)att[r];
            iota[r] = (int32_t)r;
        }
    }
}

static __global__ void k_bkeys_to_t(int64_t m, const uint64_t* __restrict__ keys, int tbits,
                                    int32_t* __restrict__ tT) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const uint64_t mask = (tbits >= 64) ? ~0ull : ((1ull << tbits) - 1);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride)
        tT[i] = (int32_t)(keys[i] & mask);
}

}  // namespace gsr

using namespace gsr;

#define HIP_TRY(call)                                      \
    do {                                                   \
        hipError_t e_ = (call);                            \
        if (e_ != hipSuccess) return hip_fail(e_, #call);  \
    } while (0)
#define GSR_TRY(call)                \
    do {                             \
        gsr_status s_ = (call);      \
        if (s_ != GSR_OK) return s_; \
    } while (0)
#define HIP_TRY_VOID(call) (void)(call)

namespace {

constexpr int kChunkRows = 256;  // rows per wave chunk
constexpr int kStarBlock = 512;  // threads of the star-ordered aprod 2 blocks

struct Tuning {
    int threads = kBRowBlock;  // of a block of the row pass
    int steps = 8;             // most wave steps per wave and round
};

// Launch shape of the row pass.
struct BRowPlan {
    int threads = 0, rows = 0, nsb = 0, grid = 0;
    bool ldsi = true;
    size_t lds = 0;
};

std::mutex g_tune_mu;
std::map<std::tuple<int, int64_t, int>, Tuning> g_tune_cache;

template <typename T>
gsr_status balloc(T** p, size_t count, size_t contiguous_from = kContiguous) {
    if (count == 0) count = 1;
    hipError_t e = device_alloc((void**)p, count * sizeof(T), contiguous_from);
    if (e != hipSuccess) {
        *p = nullptr;
        return fail(GSR_E_NOMEM, "hipMalloc of %zu bytes failed", count * sizeof(T));
    }
    return GSR_OK;
}

void bfree(void* p) {
    if (p) (void)hipFree(p);
}

}  // namespace

struct gsr_batch {
    int device = 0, n_cu = 256;
    int n_sys = 0, k = 1;
    int64_t M = 0, N = 0;
    int max_instr = 0;
    std::vector<SysDesc> h_sys;
    std::vector<int64_t> col_off;
    const double* vals = nullptr;
    const int32_t *star = nullptr, *att = nullptr, *instr = nullptr;
    SysDesc* d_sys = nullptr;
    // segment lists (device) and their counts
    Seg *chunks = nullptr, *bchunks = nullptr, *tiles = nullptr, *rounds = nullptr,
        *achunks = nullptr;
    int nchunks = 0, nbchunks = 0, ntiles = 0, nrounds = 0, nachunks = 0;
    BRowPlan row;
    int64_t stars = 0;  // of all systems
    // row tiles of the row pass, as in the single-system form
    double* btiles = nullptr;
    int64_t nbtiles = 0;
    // t-ordered attitude copy
    int32_t *rowT = nullptr, *tT = nullptr;
    double* attT = nullptr;
    // preconditioner and LSQR state
    double* p = nullptr;
    LsqrState* st = nullptr;
    std::vector<LsqrState> st_host;
    double *U = nullptr, *V = nullptr, *W = nullptr, *Z = nullptr, *XT = nullptr, *S = nullptr;
    double* part = nullptr;
    size_t part_len = 0;
    int G1 = 1, G2s = 1, G2t = 1;
    hipStream_t cap = nullptr;
    hipGraphExec_t graph = nullptr;  // whole fixed-iteration solve
    int graph_itnlim = -1;
    const double *graph_B = nullptr;
    double* graph_X = nullptr;
    gsr_solve_opts graph_opts = {};
};

namespace {

// Shape of the row pass for the tuning `t`: rounds of at most t.steps wave steps per wave, as
// many as the LDS holds beside the sums (one block of 1,024 threads or two of 512 per compute
// unit share it).  Where the slots of one step do not fit beside the sums, as many as do (stars
// past the last slot take atomics); 0 rows when the sums alone do not fit.  The instrumental unknowns are staged
// where that leaves two steps or more (16 systems of 1.31e7 rows, 8 right-hand sides, 500 columns
// each: 1.61 ms staged, 1.95 ms read from the operand; 64 systems of 1.76e6 rows, 2 right-hand
// sides, 100 columns: 99 and 111 us) and read from the operand otherwise (above about 1,200
// columns with 8 right-hand sides).
BRowPlan plan_brow(const gsr_batch* b, const Tuning& t) {
    BRowPlan r;
    const int nw = t.threads / kWave;
    const int64_t lds = 160 * 1024 / (kBRowBlock / t.threads) / 8 - 16;  // doubles per block
    const double rows_per_star =
        std::max(1.0, (double)b->M / (double)std::max<int64_t>(1, b->stars));
    auto slots = [&](int64_t rows) {
        return std::min<int64_t>(rows, (int64_t)(1.25 * rows / rows_per_star) + 8);
    };
    auto need = [&](int64_t steps, bool ldsi) {
        const int64_t rows = steps * nw * kStepRows;
        return brow_fixed(b->k, b->max_instr, ldsi) + (b->k <= 2 ? rows * b->k : 0) + slots(rows) * kAstro * b->k;
    };
    int steps = t.steps;
    while (steps > 0 && need(steps, true) > lds) --steps;
    r.ldsi = steps >= std::min(2, t.steps);
    if (!r.ldsi) {
        steps = t.steps;
        while (steps > 0 && need(steps, false) > lds) --steps;
    }
    r.threads = t.threads;
    r.rows = std::max(1, steps) * nw * kStepRows;
    const int64_t base =
        brow_fixed(b->k, b->max_instr, r.ldsi) + (b->k <= 2 ? (int64_t)r.rows * b->k : 0);
    const int64_t fit = (lds - base) / (kAstro * b->k);
    if (fit < 1) return BRowPlan();
    r.nsb = (int)std::min(slots(r.rows), fit);
    r.lds = sizeof(double) * (size_t)(base + (int64_t)r.nsb * kAstro * b->k);
    return r;
}

// (Re)build the work lists for the row pass shape `r`; device copies replaced.
gsr_status build_lists(gsr_batch* b, const BRowPlan& r, hipStream_t s) {
    std::vector<Seg> ch, bch, tl, rd, ach;
    // attitude chunks: two per wave at eight blocks per compute unit, whole blocks of 32 rows
    // (longer ones are no faster: one chunk per wave 59 and 594 us for 1.76e6 and 1.31e7 rows,
    // two 57 and 565)
    const int64_t al =
        std::min<int64_t>(2048, std::max<int64_t>(128, b->M / (64 * b->n_cu) / 32 * 32));
    // column tiles: eight blocks per compute unit (64 systems of 3.3e5 columns in all: a vector
    // step of 2,048-column tiles, 164 blocks, takes 16 us)
    const int64_t cl = std::min<int64_t>(
        kBTileMax, std::max<int64_t>(kBTileMin, b->N / (8 * b->n_cu) / 64 * 64));
    for (int i = 0; i < b->n_sys; ++i) {
        SysDesc& d = b->h_sys[i];
        auto split = [&](std::vector<Seg>& v, int64_t at, int64_t n, int64_t len) {
            const size_t first = v.size();
            for (int64_t e = 0; e < n; e += len)
                v.push_back({at + e, at + std::min<int64_t>(n, e + len), i, 0});
            return std::make_pair((int)first, (int)(v.size() - first));
        };
        std::tie(d.chunk0, d.nchunk) = split(ch, d.row0, d.m, kChunkRows);
        split(bch, d.row0, d.m, (int64_t)kChunkRows * (kStarBlock / kWave));
        split(ach, d.row0, d.m, al);
        std::tie(d.tile0, d.ntile) = split(tl, d.col0, d.n, cl);
        // rounds of equal length, whole row tiles
        const int64_t nt = (d.m + kStepRows - 1) / kStepRows, cap = r.rows / kStepRows;
        const int64_t nr = std::max<int64_t>(1, (nt + cap - 1) / cap);
        std::tie(d.round0, d.nround) = split(rd, d.row0, d.m, (nt + nr - 1) / nr * kStepRows);
    }
    auto put = [&](Seg** p, int* n, const std::vector<Seg>& v) -> gsr_status {
        bfree(*p);
        *p = nullptr;
        *n = (int)v.size();
        GSR_TRY(balloc(p, v.size()));
        HIP_TRY(hipMemcpyAsync(*p, v.data(), v.size() * sizeof(Seg), hipMemcpyHostToDevice, s));
        return GSR_OK;
    };
    GSR_TRY(put(&b->chunks, &b->nchunks, ch));
    GSR_TRY(put(&b->bchunks, &b->nbchunks, bch));
    GSR_TRY(put(&b->tiles, &b->ntiles, tl));
    GSR_TRY(put(&b->rounds, &b->nrounds, rd));
    GSR_TRY(put(&b->achunks, &b->nachunks, ach));
    if (!b->d_sys) GSR_TRY(balloc(&b->d_sys, b->n_sys));
    HIP_TRY(hipMemcpyAsync(b->d_sys, b->h_sys.data(), b->n_sys * sizeof(SysDesc),
                           hipMemcpyHostToDevice, s));
    HIP_TRY(hipStreamSynchronize(s));
    // persistent grids
    auto cap_grid = [&](int64_t items, int per_cu) {
        return (int)std::max<int64_t>(1, std::min<int64_t>(items, (int64_t)b->n_cu * per_cu));
    };
    b->G1 = cap_grid((b->nchunks + 3) / 4, 8);
    b->G2t = cap_grid((b->nachunks + 3) / 4, 8);
    b->G2s = cap_grid(b->nbchunks, 2);
    b->row = r;
    b->row.grid = cap_grid(b->nrounds, kBRowBlock / r.threads);
    return GSR_OK;
}

template <typename F>
void with_k(int k, F&& f) {
    switch (k) {
        case 1: f(std::integral_constant<int, 1>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        default: f(std::integral_constant<int, 8>()); break;
    }
}

template <int MODE, int K>
void blaunch_aprod1(gsr_batch* b, const double* X, double* Y, const double* B, hipStream_t s) {
    hipLaunchKernelGGL((k_baprod1<double, MODE, K>), dim3(b->G1), dim3(256), 0, s, b->d_sys,
                       b->chunks, b->nchunks, b->vals, b->star, b->att, b->instr, X, Y, B, b->st,
                       b->part);
}

template <int MODE, int K>
void blaunch_att(gsr_batch* b, const double* Y, double* X, hipStream_t s) {
    hipLaunchKernelGGL((k_baprod2_att<MODE, K>), dim3(b->G2t), dim3(256), 0, s, b->d_sys,
                       b->achunks, b->nachunks, b->attT, b->rowT, b->tT, Y, X, b->st);
}

// The row pass and the attitude columns of S.
template <int MODE, int K>
void blaunch_row(gsr_batch* b, hipStream_t s) {
    const BRowPlan& r = b->row;
    const BRowArgs a = {b->d_sys, b->rounds, b->nrounds, b->btiles, b->star,      b->XT,  b->U,
                        b->S,     b->st,     b->part,    b->max_instr, r.rows, r.nsb};
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(r.grid), dim3(r.threads), r.lds, s, a);
    };
    if (r.ldsi)
        go(k_browpass<K, MODE, true>);
    else
        go(k_browpass<K, MODE, false>);
    blaunch_att<MODE == BR_SQ ? A2_SQ : A2_LSQR, K>(b, b->U, b->S, s);
}

template <int K>
void blaunch_aprod2(gsr_batch* b, const double* Y, double* X, hipStream_t s) {
    const size_t lds = sizeof(double) * (size_t)(b->max_instr + 1) * K;
    hipLaunchKernelGGL((k_baprod2_star<K>), dim3(b->G2s), dim3(kStarBlock), lds, s, b->d_sys,
                       b->bchunks, b->nbchunks, b->vals, b->star, b->instr, Y, X, b->max_instr);
    blaunch_att<A2_ADD, K>(b, Y, X, s);
}

template <int K>
void bscal(gsr_batch* b, int step, int nseg, const gsr_solve_opts& o, hipStream_t s) {
    const dim3 grid(b->n_sys * K), block(256);
    switch (step) {
        case BS_INIT1:
            hipLaunchKernelGGL((k_bscal<BS_INIT1, K>), grid, block, 0, s, b->st, b->d_sys,
                               b->n_sys, b->part, nseg, o.itnlim, o.fixed_iters, o.atol, o.btol,
                               o.conlim, b->k);
            break;
        case BS_INIT2:
            hipLaunchKernelGGL((k_bscal<BS_INIT2, K>), grid, block, 0, s, b->st, b->d_sys,
                               b->n_sys, b->part, nseg, 0, 0, 0.0, 0.0, 0.0, b->k);
            break;
        case BS_BETA:
            hipLaunchKernelGGL((k_bscal<BS_BETA, K>), grid, block, 0, s, b->st, b->d_sys,
                               b->n_sys, b->part, nseg, 0, 0, 0.0, 0.0, 0.0, b->k);
            break;
        default:
            hipLaunchKernelGGL((k_bscal<BS_ALPHA, K>), grid, block, 0, s, b->st, b->d_sys,
                               b->n_sys, b->part, nseg, 0, 0, 0.0, 0.0, 0.0, b->k);
    }
}

template <int K>
void b_iteration(gsr_batch* b, hipStream_t s) {
    const dim3 tgrid((unsigned)std::min(b->ntiles, b->n_cu * 8));
    // one read of every row: U = sv A XT - alpha su U and S = A^T U
    blaunch_row<BR_LSQR, K>(b, s);
    bscal<K>(b, BS_BETA, b->nrounds, gsr_solve_opts{}, s);
    hipLaunchKernelGGL((k_bvec_v<false, K>), tgrid, dim3(256), 0, s, b->tiles, b->ntiles, b->S,
                       b->p, b->V, b->W, b->Z, b->XT, b->d_sys, b->st, b->part);
    bscal<K>(b, BS_ALPHA, b->ntiles, gsr_solve_opts{}, s);
}

template <int K>
void b_solve_body(gsr_batch* b, const double* B, double* X, const gsr_solve_opts& o,
                  hipStream_t s, int iters) {
    const dim3 tgrid((unsigned)std::min(b->ntiles, b->n_cu * 8));
    const dim3 cgrid((unsigned)std::min(b->nchunks, b->n_cu * 8));
    hipLaunchKernelGGL((k_bcopy_norm<K>), cgrid, dim3(256), 0, s, b->chunks, b->nchunks, B, b->U,
                       b->part);
    bscal<K>(b, BS_INIT1, b->nchunks, o, s);
    hipLaunchKernelGGL(k_fill, dim3(grid_for(b->N * K, 256, 2048)), dim3(256), 0, s, b->S,
                       b->N * K, 0.0);
    blaunch_row<BR_T, K>(b, s);
    hipLaunchKernelGGL((k_bvec_v<true, K>), tgrid, dim3(256), 0, s, b->tiles, b->ntiles, b->S,
                       b->p, b->V, b->W, b->Z, b->XT, b->d_sys, b->st, b->part);
    bscal<K>(b, BS_INIT2, b->ntiles, o, s);
    for (int it = 0; it < iters; ++it) b_iteration<K>(b, s);
    if (X)
        hipLaunchKernelGGL((k_bfinal<K>), tgrid, dim3(256), 0, s, b->tiles, b->ntiles, b->p, b->Z,
                           b->W, b->V, X, b->st);
}

// Time the row pass for each candidate tuning; keep the fastest.  Synchronizes.
gsr_status autotune(gsr_batch* b, hipStream_t s) {
    const auto key = std::make_tuple(b->n_sys, b->M, b->k);
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tune_cache.find(key);
        if (it != g_tune_cache.end()) {
            const BRowPlan r = plan_brow(b, it->second);
            if (r.rows > 0) return build_lists(b, r, s);
        }
    }
    const Tuning cands[] = {{1024, 48}, {1024, 16}, {1024, 6}, {1024, 2}, {512, 16}, {512, 6}};
    Tuning best;
    float best_ms = 1e30f;
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    int last_rows = 0, last_threads = 0;
    for (const Tuning& t : cands) {
        const BRowPlan r = plan_brow(b, t);
        if (r.rows == 0 || (r.rows == last_rows && r.threads == last_threads)) continue;
        last_rows = r.rows;
        last_threads = r.threads;
        GSR_TRY(build_lists(b, r, s));
        float ms = 0.f;
        with_k(b->k, [&](auto kc) {
            constexpr int K = decltype(kc)::value;
            // on scratch contents (every pair's state is still zero here, so the values are
            // zeros); the partial sums need room for this candidate's rounds
            HIP_TRY_VOID(hipMemsetAsync(b->XT, 0, sizeof(double) * b->N * K, s));
            HIP_TRY_VOID(hipMemsetAsync(b->U, 0, sizeof(double) * b->M * K, s));
            for (int rep = 0; rep < 3; ++rep) {
                if (rep == 1) (void)hipEventRecord(e0, s);
                blaunch_row<BR_LSQR, K>(b, s);
            }
            (void)hipEventRecord(e1, s);
            (void)hipEventSynchronize(e1);
            (void)hipEventElapsedTime(&ms, e0, e1);
        });
        HIP_TRY(hipGetLastError());
        if (ms < best_ms) {
            best_ms = ms;
            best = t;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tune_cache[key] = best;
    }
    return build_lists(b, plan_brow(b, best), s);
}

gsr_status b_colnorm(gsr_batch* b, hipStream_t s, unsigned long long* n_empty) {
    // column sums of squares (stride-1 vectors)
    double* ss = b->S;  // N x k >= N doubles
    unsigned long long* d_cnt = nullptr;
    GSR_TRY(balloc(&d_cnt, 1));
    HIP_TRY(hipMemsetAsync(d_cnt, 0, sizeof(*d_cnt), s));
    HIP_TRY(hipMemsetAsync(ss, 0, sizeof(double) * b->N, s));
    blaunch_row<BR_SQ, 1>(b, s);
    hipLaunchKernelGGL(k_brecip_sqrt, dim3(grid_for(b->N, 256, 2048)), dim3(256), 0, s, b->N, ss,
                       b->p, d_cnt);
    HIP_TRY(hipMemsetAsync(ss, 0, sizeof(double) * b->N * b->k, s));
    hipError_t e = hipMemcpyAsync(n_empty, d_cnt, sizeof(*d_cnt), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    bfree(d_cnt);
    if (e != hipSuccess) return hip_fail(e, "batched column norms");
    return GSR_OK;
}

}  // namespace

extern "C" {

gsr_status gsr_batch_setup(int32_t n_sys, const gsr_dims* dims, const int64_t* row_offset,
                           const double* vals, const int32_t* star, const int32_t* att,
                           const int32_t* instr, int32_t k, const gsr_setup_opts* opts,
                           void* stream, gsr_batch** out) {
    g_last_error.clear();
    if (!out) return fail(GSR_E_INVAL, "out is NULL");
    *out = nullptr;
    if (n_sys < 1 || !dims || !row_offset) return fail(GSR_E_INVAL, "n_sys < 1 or null dims");
    if (k != 1 && k != 2 && k != 4 && k != 8)
        return fail(GSR_E_UNSUPPORTED, "k must be 1, 2, 4 or 8 (got %d)", k);
    if (row_offset[0] != 0) return fail(GSR_E_INVAL, "row_offset[0] must be 0");
    int max_instr = 0;
    for (int i = 0; i < n_sys; ++i) {
        GSR_TRY(check_dims(&dims[i]));
        if (row_offset[i + 1] - row_offset[i] != dims[i].n_rows)
            return fail(GSR_E_INVAL, "row_offset does not match dims[%d].n_rows", i);
        max_instr = std::max(max_instr, dims[i].n_instr);
    }
    const int64_t M = row_offset[n_sys];
    if (M > (int64_t)INT32_MAX) return fail(GSR_E_UNSUPPORTED, "more than 2^31-1 rows");
    if (M > 0 && (!vals || !star || !att || !instr)) return fail(GSR_E_INVAL, "null matrix array");
    if (((uintptr_t)vals & 15) || ((uintptr_t)instr & 7))
        return fail(GSR_E_INVAL, "vals must be 16-byte and instr 8-byte aligned");
    if ((size_t)((2 * max_instr + 1) * k + k) * sizeof(double) > 160 * 1024)
        return fail(GSR_E_UNSUPPORTED, "n_instr * k too large for the batched LDS accumulator");
    gsr_setup_opts so = {0, 1, 0, 0};
    if (opts) so = *opts;
    int dev = 0, n_cu = 0;
    GSR_TRY(check_device(&dev, &n_cu));
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);

    gsr_batch* b = new gsr_batch();
    auto bail = [&](gsr_status st) {
        gsr_batch_destroy(b);
        return st;
    };
    b->device = dev;
    b->n_cu = n_cu;
    b->n_sys = n_sys;
    b->k = k;
    b->M = M;
    b->max_instr = max_instr;
    b->vals = vals;
    b->star = star;
    b->att = att;
    b->instr = instr;
    b->h_sys.resize(n_sys);
    b->col_off.resize(n_sys + 1);
    int64_t col = 0, max_T = 4;
    for (int i = 0; i < n_sys; ++i) {
        const Geo g = make_geo(&dims[i]);
        SysDesc& d = b->h_sys[i];
        d.row0 = row_offset[i];
        d.m = dims[i].n_rows;
        d.col0 = col;
        d.n = g.n;
        d.att0 = g.att0;
        d.ins0 = g.ins0;
        d.glb0 = g.glb0;
        d.n_stars = dims[i].n_stars;
        d.T = g.T;
        d.I = g.I;
        b->stars += d.n_stars;
        d.btile0 = b->nbtiles;
        b->nbtiles += (d.m + kStepRows - 1) / kStepRows;
        b->col_off[i] = col;
        col += g.n;
        max_T = std::max<int64_t>(max_T, g.T);
    }
    b->col_off[n_sys] = col;
    b->N = col;
    gsr_status st;
    if ((st = build_lists(b, plan_brow(b, Tuning()), s)) != GSR_OK) return bail(st);
    const size_t NK = (size_t)b->N * k, MK = (size_t)M * k;
    if ((st = balloc(&b->p, b->N)) != GSR_OK) return bail(st);
    if ((st = balloc(&b->S, NK)) != GSR_OK) return bail(st);
    if ((st = balloc(&b->V, NK)) != GSR_OK) return bail(st);
    if ((st = balloc(&b->W, NK)) != GSR_OK) return bail(st);
    if ((st = balloc(&b->Z, NK)) != GSR_OK) return bail(st);
    if ((st = balloc(&b->XT, NK, kGathered)) != GSR_OK) return bail(st);
    if ((st = balloc(&b->U, MK, kGathered)) != GSR_OK) return bail(st);
    if ((st = balloc(&b->st, (size_t)n_sys * k)) != GSR_OK) return bail(st);
    if ((st = balloc(&b->btiles, (size_t)b->nbtiles * tile_elems<double>())) != GSR_OK)
        return bail(st);
    for (int i = 0; i < n_sys; ++i) {
        const SysDesc& d = b->h_sys[i];
        const int64_t nt = (d.m + kStepRows - 1) / kStepRows;
        if (nt == 0) continue;
        double* tiles = b->btiles + d.btile0 * tile_elems<double>();
        hipLaunchKernelGGL(k_make_tiles<double>, dim3(grid_for(nt * kTileVals, 256, 4096)),
                           dim3(256), 0, s, d.m, nt, vals + d.row0 * kPar, tiles);
        hipLaunchKernelGGL(k_make_itiles<double>, dim3(grid_for(nt * kTileIdx, 256, 4096)),
                           dim3(256), 0, s, d.m, nt, star + d.row0, att + d.row0,
                           instr + d.row0 * kInstr, tiles);
    }
    b->st_host.resize((size_t)n_sys * k);
    {
        hipError_t e = hipMemsetAsync(b->st, 0, sizeof(LsqrState) * n_sys * k, s);
        if (e == hipSuccess) e = hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking);
        if (e != hipSuccess) return bail(hip_fail(e, "batch setup"));
    }
    // validation
    if (so.validate && M > 0) {
        int* d_flags = nullptr;
        if ((st = balloc(&d_flags, 1)) != GSR_OK) return bail(st);
        int flags = 0;
        hipError_t e = hipMemsetAsync(d_flags, 0, sizeof(int), s);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_bvalidate, dim3(std::min(b->nchunks, 4096)), dim3(256), 0, s,
                               b->d_sys, b->chunks, b->nchunks, star, att, instr, d_flags);
            e = hipMemcpyAsync(&flags, d_flags, sizeof(int), hipMemcpyDeviceToHost, s);
        }
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        bfree(d_flags);
        if (e != hipSuccess) return bail(hip_fail(e, "batch validation"));
        if (flags)
            return bail(fail(GSR_E_LAYOUT, "index check failed:%s%s%s%s",
                             (flags & 1) ? " star out of range" : "",
                             (flags & 2) ? " stars not sorted" : "",
                             (flags & 4) ? " attitude start out of [0, n_dfa-4]" : "",
                             (flags & 8) ? " instrumental index out of range" : ""));
    }
    // attitude coefficients in (system, t) order
    if ((st = balloc(&b->rowT, M)) != GSR_OK) return bail(st);
    if ((st = balloc(&b->tT, M)) != GSR_OK) return bail(st);
    if ((st = balloc(&b->attT, (size_t)b->nbtiles * kStepRows * kAttRow)) != GSR_OK) return bail(st);
    if (M > 0) {
        int tbits = 1;
        while (tbits < 31 && (1LL << tbits) <= max_T) ++tbits;
        int sbits = 1;
        while ((1LL << sbits) < n_sys) ++sbits;
        uint64_t *keys = nullptr, *keys_out = nullptr;
        int32_t* iota = nullptr;
        void* temp = nullptr;
        size_t temp_bytes = 0;
        hipError_t e = hipMalloc(&keys, sizeof(uint64_t) * M);
        if (e == hipSuccess) e = hipMalloc(&keys_out, sizeof(uint64_t) * M);
        if (e == hipSuccess) e = hipMalloc(&iota, sizeof(int32_t) * M);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_bkeys, dim3(std::min(b->nchunks, 4096)), dim3(256), 0, s,
                               b->d_sys, b->chunks, b->nchunks, att, tbits, keys, iota);
            e = hipcub::DeviceRadixSort::SortPairs(nullptr, temp_bytes, keys, keys_out, iota,
                                                   b->rowT, (int)M, 0, tbits + sbits, s);
        }
        if (e == hipSuccess) e = hipMalloc(&temp, std::max<size_t>(temp_bytes, 1));
        if (e == hipSuccess)
            e = hipcub::DeviceRadixSort::SortPairs(temp, temp_bytes, keys, keys_out, iota, b->rowT,
                                                   (int)M, 0, tbits + sbits, s);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_bkeys_to_t, dim3(grid_for(M, 256, 4096)), dim3(256), 0, s, M,
                               keys_out, tbits, b->tT);
            for (int i = 0; i < n_sys; ++i) {
                const SysDesc& d = b->h_sys[i];
                if (d.m == 0) continue;
                hipLaunchKernelGGL(k_make_batt_rows, dim3(grid_for(d.m * kAttRow, 256, 4096)),
                                   dim3(256), 0, s, d.m, d.row0, vals, b->rowT,
                                   b->attT + d.btile0 * kStepRows * kAttRow);
            }
            e = hipStreamSynchronize(s);
        }
        bfree(keys);
        bfree(keys_out);
        bfree(iota);
        bfree(temp);
        if (e != hipSuccess) return bail(hip_fail(e, "batched attitude ordering"));
    }
    // partial sums: 4 quantities per (column tile, rhs), one per (row chunk or round, rhs); at
    // most one round per 8 row tiles of a system, and one more
    b->part_len = (size_t)k * std::max({(size_t)4 * b->ntiles, (size_t)b->nchunks,
                                        (size_t)(b->nbtiles / 8 + n_sys), (size_t)1});
    if ((st = balloc(&b->part, b->part_len)) != GSR_OK) return bail(st);
    unsigned long long n_empty = 0;
    if ((st = b_colnorm(b, s, &n_empty)) != GSR_OK) return bail(st);
    if (n_empty && !so.allow_empty_cols)
        return bail(fail(GSR_E_LAYOUT, "%llu all-zero column(s); set allow_empty_cols", n_empty));
    if ((st = autotune(b, s)) != GSR_OK) return bail(st);
    *out = b;
    return GSR_OK;
}

gsr_status gsr_batch_destroy(gsr_batch* b) {
    if (!b) return GSR_OK;
    (void)hipSetDevice(b->device);
    (void)hipDeviceSynchronize();
    if (b->graph) (void)hipGraphExecDestroy(b->graph);
    for (void* p : {(void*)b->d_sys, (void*)b->chunks, (void*)b->bchunks, (void*)b->tiles,
                    (void*)b->rowT, (void*)b->tT, (void*)b->attT, (void*)b->p, (void*)b->st,
                    (void*)b->U, (void*)b->V, (void*)b->W, (void*)b->Z, (void*)b->XT,
                    (void*)b->S, (void*)b->part, (void*)b->btiles, (void*)b->rounds,
                    (void*)b->achunks})
        bfree(p);
    if (b->cap) (void)hipStreamDestroy(b->cap);
    delete b;
    return GSR_OK;
}

gsr_status gsr_batch_col_offsets(const gsr_batch* b, int64_t* col_offset) {
    if (!b || !col_offset) return fail(GSR_E_INVAL, "null argument");
    std::memcpy(col_offset, b->col_off.data(), sizeof(int64_t) * (b->n_sys + 1));
    return GSR_OK;
}

gsr_status gsr_batch_aprod1(gsr_batch* b, const double* X, double* Y, void* stream) {
    if (!b || !X || !Y) return fail(GSR_E_INVAL, "null argument");
    if (((uintptr_t)X | (uintptr_t)Y) & 15) return fail(GSR_E_INVAL, "X and Y must be 16-byte aligned");
    HIP_TRY(hipSetDevice(b->device));
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    with_k(b->k, [&](auto kc) { blaunch_aprod1<A1_ADD, decltype(kc)::value>(b, X, Y, nullptr, s); });
    HIP_TRY(hipGetLastError());
    return GSR_OK;
}

gsr_status gsr_batch_aprod2(gsr_batch* b, const double* Y, double* X, void* stream) {
    if (!b || !X || !Y) return fail(GSR_E_INVAL, "null argument");
    if (((uintptr_t)X | (uintptr_t)Y) & 15) return fail(GSR_E_INVAL, "X and Y must be 16-byte aligned");
    HIP_TRY(hipSetDevice(b->device));
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    with_k(b->k, [&](auto kc) { blaunch_aprod2<decltype(kc)::value>(b, Y, X, s); });
    HIP_TRY(hipGetLastError());
    return GSR_OK;
}

gsr_status gsr_batch_solve(gsr_batch* b, const double* B, double* X, const gsr_solve_opts* opts,
                           gsr_solve_info* info, void* stream) {
    g_last_error.clear();
    if (!b || !X || (!B && b->M > 0)) return fail(GSR_E_INVAL, "null argument");
    gsr_solve_opts o;
    std::memset(&o, 0, sizeof o);
    o.itnlim = 100;
    o.fixed_iters = 1;
    o.atol = o.btol = 1e-14;
    if (opts) o = *opts;
    if (o.itnlim < 0) return fail(GSR_E_INVAL, "itnlim < 0");
    if (!(o.atol >= 0) || !(o.btol >= 0) || !(o.conlim >= 0))
        return fail(GSR_E_INVAL, "atol, btol and conlim must be >= 0");
    if (o.precision != GSR_F64) return fail(GSR_E_UNSUPPORTED, "batched solve is binary64 only");
    HIP_TRY(hipSetDevice(b->device));
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    gsr_status rc = GSR_OK;
    with_k(b->k, [&](auto kc) {
        constexpr int K = decltype(kc)::value;
        if (o.fixed_iters && !o.profile) {
            // the whole solve as one graph, reused while B, X and the options are unchanged
            const bool same = b->graph && b->graph_itnlim == o.itnlim && b->graph_B == B &&
                              b->graph_X == X &&
                              std::memcmp(&b->graph_opts, &o, sizeof o) == 0;
            if (!same) {
                if (b->graph) (void)hipGraphExecDestroy(b->graph);
                b->graph = nullptr;
                hipGraph_t g = nullptr;
                hipError_t e = hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal);
                if (e == hipSuccess) {
                    b_solve_body<K>(b, B, X, o, b->cap, o.itnlim);
                    e = hipStreamEndCapture(b->cap, &g);
                }
                if (e == hipSuccess) e = hipGraphInstantiate(&b->graph, g, nullptr, nullptr, 0);
                if (g) (void)hipGraphDestroy(g);
                if (e != hipSuccess) {
                    b->graph = nullptr;
                    rc = hip_fail(e, "batched solve graph");
                    return;
                }
                b->graph_itnlim = o.itnlim;
                b->graph_B = B;
                b->graph_X = X;
                b->graph_opts = o;
            }
            hipError_t e = hipGraphLaunch(b->graph, s);
            if (e != hipSuccess) rc = hip_fail(e, "hipGraphLaunch");
            return;
        }
        // convergence mode: iterate in launches of 16, checking every pair's stop flag
        b_solve_body<K>(b, B, nullptr, o, s, 0);
        const int every = o.check_every > 0 ? o.check_every : 16;
        for (int done = 0; done < o.itnlim; done += every) {
            for (int it = 0; it < every && done + it < o.itnlim; ++it) b_iteration<K>(b, s);
            hipError_t e = hipMemcpyAsync(b->st_host.data(), b->st,
                                          sizeof(LsqrState) * b->st_host.size(),
                                          hipMemcpyDeviceToHost, s);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            if (e != hipSuccess) {
                rc = hip_fail(e, "batched stop flags");
                return;
            }
            bool all = true;
            for (const LsqrState& t : b->st_host) all = all && t.stop;
            if (all) break;
        }
        const dim3 tgrid((unsigned)std::min(b->ntiles, b->n_cu * 8));
        hipLaunchKernelGGL((k_bfinal<K>), tgrid, dim3(256), 0, s, b->tiles, b->ntiles, b->p, b->Z,
                           b->W, b->V, X, b->st);
    });
    if (rc != GSR_OK) return rc;
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(b->st_host.data(), b->st, sizeof(LsqrState) * b->st_host.size(),
                           hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    bool nonfinite = false;
    for (size_t i = 0; i < b->st_host.size(); ++i) {
        const LsqrState& t = b->st_host[i];
        nonfinite = nonfinite || t.nonfinite;
        if (info) {
            gsr_solve_info& f = info[i];
            std::memset(&f, 0, sizeof f);
            f.itn = t.itn;
            f.istop = t.istop;
            f.n_refine = 1;
            f.nonfinite = t.nonfinite;  // which pair broke down, beside the status returned
            f.fused = 1;                // the batched row pass is always the fused one
            f.rnorm = t.rnorm;
            f.arnorm = t.arnorm;
            f.anorm = std::sqrt(t.anorm2);
            f.znorm = std::sqrt(t.znorm2);
            f.bnorm = t.bnorm;
            f.acond = std::sqrt(t.anorm2) * std::sqrt(t.ddnorm);
        }
    }
    if (nonfinite) return fail(GSR_E_BREAKDOWN, "non-finite value in a batched recurrence");
    return GSR_OK;
}

}  // extern "C"
