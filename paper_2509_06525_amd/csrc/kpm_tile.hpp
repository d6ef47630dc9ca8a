// Tiled form of the recurrence: several Chebyshev steps per launch.
//
// A sweep per step reads H and three vectors and writes one, 56 bytes per row
// and step for one complex-float vector, and runs at the HBM rate.  Here a
// workgroup takes a tile of consecutive rows, extends it by the rows within s
// bonds (its halo, s rings), holds T_n and T_{n-1} of the extended rows in LDS
// and their matrix entries in registers, and advances s steps before it
// writes the tile's T_{n+s} and T_{n+s-1}: step m covers the tile and its
// s - 1 - m inner rings, so every value is formed from the same operands in the
// same order as a sweep per step forms it (bit for bit the same vectors), and
// HBM sees one read of H and of each vector per s steps.
//
// The extended rows are listed by k_tile_plan once per run, ring by ring: the
// tile's own rows first (local index = row - first row), then the rows of ring 1,
// ring 2, ... in ascending order.  Matrix entries are stored again in local form:
// 16-bit LDS byte offsets of the columns beside the values, [entry][local row].
//
// One vector per workgroup: the vectors of a run live in planes [vector][row]
// while it lasts, so the tile is as large (and its halo as small) as LDS allows.
#pragma once

#include <type_traits>

#include "common.hpp"
#include "kpm.hpp"
#include "kpm_dev.hpp"

namespace tbk {

// Pointers and scalars of one launch of k_tile_steps.
template <class VT> struct TileArgs {
    const int32_t *row0;     // [n_tiles + 1] first row of each tile
    const int32_t *cnt;      // [n_tiles][S1] rows within k rings
    const int32_t *ext;      // [n_tiles][cap] halo rows (local index nr + e)
    const uint32_t *lcol2;   // [n_tiles][W / 2][cap] pairs of LDS byte offsets
    const uint16_t *lcol1;   // [n_tiles][cap] the odd column (W odd)
    const VT *val;           // [n_tiles][W][cap]
    const VT *hop;           // the value of every entry (val is not read then), or NULL
    const VT *ons;           // [n_tiles][cap] onsite energies, or NULL
    const int32_t *tile_seg; // structure of each tile, or NULL (one structure)
    const VT *seg_c1f, *seg_c1, *seg_shift;   // per structure (tile_seg != NULL)
    const VT *cur, *prev;    // T_n, T_{n-1} in planes [vector][rows]
    VT *out_cur, *out_prev;  // T_{n+s}, T_{n+s-1}; NULL: not kept
    const VT *r;             // start (or left) vectors in planes
    double *partial;         // [s][n_tiles][Rv] sums of the steps of this launch
    int64_t pstride;         // doubles per step of partial
    int64_t rows;            // plane pitch
    int32_t n_work;          // n_tiles * R
    int32_t R, Rv;
    int32_t S1, cap;         // rings listed + 1, slots of a tile
    int32_t s;               // steps of this launch
    int32_t first;           // 1: T_n is T_0 (step 0 is T_1 = Ht T_0)
    int32_t closed;          // 1: no tile has a halo, so s is not limited by rings
    VT c1f, c1, shift;       // 1/a, 2/a, b (one structure)
    // propagator form: acc += (cr + i ci)[m] T of step m; acc starts as (c0r + i c0i) T_0
    // (first) or from acc_in, and leaves multiplied by pr + i pi
    const VT *acc_in;
    VT *acc_out;
    double c0r, c0i, pr, pi;
    double cr[kTileMaxS], ci[kTileMaxS];
};

// What a launch gathers beside the vectors: the sums <r|T>, the two sums of the
// doubling identities, or the series of the propagator.
enum TileForm { kTileDirect = 0, kTileDoubling = 1, kTilePropagate = 2 };

// Sum over the wavefront; lane 63 holds it (fixed order).
__device__ __forceinline__ double wave_sum(double x) {
    auto add = [&](auto ctrl, auto mask) {
        const int2 v = *reinterpret_cast<int2 *>(&x);
        int2 o;
        o.x = __builtin_amdgcn_update_dpp(0, v.x, ctrl.value, mask.value, 0xf, false);
        o.y = __builtin_amdgcn_update_dpp(0, v.y, ctrl.value, mask.value, 0xf, false);
        x += *reinterpret_cast<double *>(&o);
    };
    using std::integral_constant;
    add(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});    // row_shr:1
    add(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});    // row_shr:2
    add(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});    // row_shr:4
    add(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});    // row_shr:8
    add(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});    // row_bcast:15
    add(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});    // row_bcast:31
    return x;
}

// x y rounded before anything is added to it (no contraction).
template <class VT> __device__ __forceinline__ VT rounded_product(VT x, VT y) {
#pragma clang fp contract(off)
    return x * y;
}

// Local rows a workgroup of NT threads with K rows each can hold: 128 fewer than
// its slots, whose LDS takes the moment sums (2 KB).
constexpr int tile_cap(int NT, int K) { return NT * K - 128; }
constexpr int kTileFlush = 8;      // steps between two writes of the moment sums

// UNI: every entry has one value (a.hop), so rows hold columns only, and padding
// points at a zero behind the rows.
template <class VT, int NT, int K, int W, bool DIAG, int FORM, bool UNI>
__global__ __launch_bounds__(NT, 4) void k_tile_steps(TileArgs<VT> a) {
    typedef std::conditional_t<sizeof(VT) == 4, f2v, d2v> C2;
    constexpr int CAP = tile_cap(NT, K);
    constexpr bool DBL = FORM == kTileDoubling, EVO = FORM == kTilePropagate;
    constexpr int NA = DBL ? 2 : 1;
    constexpr int NW = NT / 64;
    constexpr int NP = W / 2;
    constexpr int ALT = UNI ? CAP + 1 : CAP;        // first element of the second buffer
    __shared__ __align__(16) C2 buf[2 * ALT];
    __shared__ double red[2 * kTileFlush][NW][NA];
    const int tid = threadIdx.x;
    const int64_t l = logical_block(2);
    if (l >= a.n_work) return;
    const int t = (int)(l / a.R), v = (int)(l - (int64_t)t * a.R);
    const int row0 = a.row0[t], nr = a.row0[t + 1] - row0;
    const int32_t *cnt = a.cnt + (int64_t)t * a.S1;
    const int s = a.s;
    // lane k holds the rows within k rings: read from memory at each step their latency
    // stood between the barrier and the step (16 M row-vectors: 34.0 us a step, 30.4 so)
    const int rings = cnt[min(tid & 63, a.S1 - 1)];
    const int n_all = a.closed ? nr : __builtin_amdgcn_readlane(rings, s);         // rows whose T_n is read
    const int n_mat = a.closed ? nr : __builtin_amdgcn_readlane(rings, s - 1);     // rows the first step writes
    const int64_t plane = (int64_t)v * a.rows;
    const C2 *gcur = reinterpret_cast<const C2 *>(a.cur) + plane;
    const C2 *gprev = reinterpret_cast<const C2 *>(a.prev) + plane;
    const C2 *gr = reinterpret_cast<const C2 *>(a.r) + plane;
    const C2 *gacc = reinterpret_cast<const C2 *>(a.acc_in) + plane;
    const int32_t *ext = a.ext + (int64_t)t * a.cap - nr;
    VT c1f = a.c1f, c1 = a.c1, shift = a.shift;
    if (a.tile_seg) {
        const int sg = a.tile_seg[t];
        c1f = a.seg_c1f[sg];
        c1 = a.seg_c1[sg];
        shift = a.seg_shift[sg];
    }

    VT h[UNI ? 1 : K][W], dg[DIAG ? K : 1];
    const VT hop = UNI ? *a.hop : (VT)0;
    if (UNI && tid < 2) buf[CAP + tid * ALT].x = buf[CAP + tid * ALT].y = 0;
    uint32_t lc[K][NP + 1];
    C2 rr[DBL ? 1 : K];
    {
        // every load of the tile is issued before any is used (rows past the last are
        // clamped to it): the halo rows' numbers, the matrix, the vectors
        const int64_t mb = (int64_t)t * a.cap;
        int g[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = min(k * NT + tid, n_all - 1);
            g[k] = row0 + j;
            if (j >= nr) g[k] = ext[j];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = min(k * NT + tid, n_mat - 1);
            if constexpr (!UNI) {
#pragma unroll
                for (int w = 0; w < W; ++w) h[k][w] = a.val[mb * W + (int64_t)w * a.cap + j];
            }
#pragma unroll
            for (int p = 0; p < NP; ++p) lc[k][p] = a.lcol2[mb * NP + (int64_t)p * a.cap + j];
            if constexpr (W & 1) lc[k][NP] = a.lcol1[mb + j];
            if constexpr (DIAG) dg[k] = a.ons ? a.ons[mb + j] : (VT)0;
            if constexpr (FORM == kTileDirect) rr[k] = gr[row0 + min(j, nr - 1)];
            if constexpr (EVO) {
                if (!a.first) rr[k] = gacc[row0 + min(j, nr - 1)];
            }
        }
        C2 xc[K], xp[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            xc[k] = gcur[g[k]];
            xp[k] = gprev[g[k]];
        }
        if constexpr (DIAG) {
#pragma unroll
            for (int k = 0; k < K; ++k) dg[k] -= shift;
        }
        if constexpr (UNI) {        // a column of the row itself is padding: its value is 0 (k_tile_plan)
            constexpr uint32_t zero = CAP * sizeof(C2);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t own = (uint32_t)(min(k * NT + tid, n_mat - 1) * (int)sizeof(C2));
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const uint32_t lo = lc[k][p] & 0xffffu, hi = lc[k][p] >> 16;
                    lc[k][p] = (lo == own ? zero : lo) | (hi == own ? zero : hi) << 16;
                }
                if (W & 1) lc[k][NP] = lc[k][NP] == own ? zero : lc[k][NP];
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = k * NT + tid;
            if (a.first) {
                xp[k].x = xp[k].y = 0;
                if constexpr (EVO) {
                    rr[k].x = (VT)(a.c0r * (double)xc[k].x - a.c0i * (double)xc[k].y);
                    rr[k].y = (VT)(a.c0r * (double)xc[k].y + a.c0i * (double)xc[k].x);
                }
            }
            if (j < n_all) buf[j] = xc[k];
            if (j < n_mat) buf[ALT + j] = xp[k];
        }
    }
    __syncthreads();

    // one step: T of buffer SRC -> the other buffer (over T_{n-1}, in place)
    auto step = [&](auto par, int m) {
        constexpr int SRC = decltype(par)::value ? ALT : 0;
        constexpr int DST = decltype(par)::value ? 0 : ALT;
        const int lim = a.closed ? nr : __builtin_amdgcn_readlane(rings, s - 1 - m);
        const VT cc = (m == 0 && a.first) ? c1f : c1;
        const double cr = EVO ? a.cr[m] : 0.0, ci = EVO ? a.ci[m] : 0.0;
        const char *src = reinterpret_cast<const char *>(buf + SRC);
        double acc[NA];
#pragma unroll
        for (int q = 0; q < NA; ++q) acc[q] = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = k * NT + tid;
            if (j < lim) {
                C2 x[W];
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const uint32_t o = (w == W - 1 && (W & 1)) ? lc[k][NP]
                                                               : ((w & 1) ? lc[k][w / 2] >> 16 : lc[k][w / 2] & 0xffffu);
                    x[w] = *reinterpret_cast<const C2 *>(src + o);
                }
                const C2 p = buf[DST + j];
                C2 own;
                if constexpr (DIAG || DBL) own = buf[SRC + j];
                VT yr = 0, yi = 0;
                if constexpr (DIAG && EVO) {      // first, as in k_evolve_term
                    yr = rounded_product(dg[k], own.x);
                    yi = rounded_product(dg[k], own.y);
                }
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const VT hw = UNI ? hop : h[UNI ? 0 : k][w];
                    yr += hw * x[w].x;
                    yi += hw * x[w].y;
                }
                if constexpr (DIAG && !EVO) {
                    yr += dg[k] * own.x;
                    yi += dg[k] * own.y;
                }
                C2 o;
                o.x = cc * yr - p.x;
                o.y = cc * yi - p.y;
                buf[DST + j] = o;
                if (j < nr) {
                    if constexpr (EVO) {
                        rr[k].x += (VT)(cr * (double)o.x - ci * (double)o.y);
                        rr[k].y += (VT)(cr * (double)o.y + ci * (double)o.x);
                    } else if constexpr (DBL) {
                        acc[0] += (double)o.x * (double)o.x + (double)o.y * (double)o.y;
                        acc[1] += (double)own.x * (double)o.x + (double)own.y * (double)o.y;
                    } else {
                        // the widened r is formed anew each step: kept over the steps it
                        // would take twice r's registers
                        if constexpr (sizeof(VT) == 4) asm volatile("" : "+v"(rr[k]));
                        acc[0] += (double)rr[k].x * (double)o.x + (double)rr[k].y * (double)o.y;
                    }
                }
            }
        }
        if constexpr (EVO) {
            __syncthreads();
            return;
        }
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            const double w = wave_sum(acc[q]);
            if ((tid & 63) == 63) red[m & (2 * kTileFlush - 1)][tid >> 6][q] = w;
        }
        __syncthreads();
        // every kTileFlush steps the waves' sums are added (in wave order) and written;
        // the other half of `red` takes the next steps' meanwhile
        if (m == s - 1 || (m & (kTileFlush - 1)) == kTileFlush - 1) {
            const int base = m & ~(kTileFlush - 1);
            const int i = tid / NA, q = tid % NA;
            if (i <= m - base) {
                double sum = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) sum += red[(base + i) & (2 * kTileFlush - 1)][w][q];
                a.partial[(int64_t)(base + i) * a.pstride + (int64_t)t * a.Rv + v * NA + q] = sum;
            }
        }
    };
    int m = 0;
    for (; m + 1 < s; m += 2) {
        step(std::integral_constant<int, 0>{}, m);
        step(std::integral_constant<int, 1>{}, m + 1);
    }
    if (m < s) step(std::integral_constant<int, 0>{}, m);

    if constexpr (EVO) {
        C2 *oa = reinterpret_cast<C2 *>(a.acc_out) + plane + row0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = k * NT + tid;
            if (j < nr) {
                C2 y = rr[k];
                if (!a.out_cur) {      // the last group: the phase of the shift
                    y.x = (VT)(a.pr * (double)rr[k].x - a.pi * (double)rr[k].y);
                    y.y = (VT)(a.pr * (double)rr[k].y + a.pi * (double)rr[k].x);
                }
                oa[j] = y;
            }
        }
    }
    if (a.out_cur) {
        const int cur = (s & 1) ? ALT : 0, old = ALT - cur;
        C2 *oc = reinterpret_cast<C2 *>(a.out_cur) + plane + row0;
        C2 *op = reinterpret_cast<C2 *>(a.out_prev) + plane + row0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = k * NT + tid;
            if (j < nr) {
                oc[j] = buf[cur + j];
                op[j] = buf[old + j];
            }
        }
    }
}

// Launches one group of steps with the kernel of the plan's shape; instantiated
// per vector type and width in kpm_tile_inst_*.hip.
template <class VT, int W>
void launch_tile_steps(const TilePlan &tp, bool diag, int form, unsigned grid, hipStream_t s,
                       const TileArgs<VT> &a);

// Launch shapes (threads, rows per thread).  A row's entries stay in registers
// over the steps (W values, W / 2 + W % 2 column words, r: 7 words for W = 3 in
// complex float), so the rows per thread end where the 128 registers of four
// waves per SIMD do: one row more spills, which cost 1.45x (1 M atoms, 8 vectors
// with onsite energies: 26.9 us a step with ten rows, 18.5 with nine).
//   large, large_diag: two workgroups of 512 per CU share its LDS (with onsite
//     energies a row takes one word more);
//   small: half the rows, for complex-float systems of few tiles, where a CU has one
//     or two workgroups and the steps wait for LDS (30,212 rows, three vectors: 1.34 us a
//     step with 256 threads of eight rows, 1.18 so; 300,000 rows, two: 2.51 and 2.12);
//   whole: a workgroup of 1024 takes a CU, for a matrix that is one tile.
enum TileShape { kTileLarge = 0, kTileLargeDiag = 1, kTileSmall = 2, kTileWhole = 3 };
constexpr int tile_threads(int shape) { return shape == kTileWhole ? 1024 : 512; }
constexpr int tile_slots(int shape, int W, bool f64) {
    const int i = W == 3 ? 0 : (W == 4 ? 1 : 2);
    const int c32[4][3] = {{10, 8, 5}, {9, 7, 5}, {5, 4, 3}, {5, 5, 3}};
    const int c64[4][3] = {{5, 4, 3}, {5, 4, 3}, {0, 0, 0}, {4, 4, 3}};
    return f64 ? c64[shape][i] : c32[shape][i];
}

// Tile lists of h and the steps per launch (run.s = 0: no locality, use the sweep).
// n_first > 0: the caller has written that many tiles' first rows and structures.  defer: as build_tiles.
template <class VT>
tbk_status tile_build(const tbk_ham *h, const KpmPlan &pl, int n_first, char *work, hipStream_t s, TileRun &run,
                      bool defer);
template <class VT>
TileArgs<VT> tile_args(const tbk_ham *h, const KpmPlan &pl, const TileRun &run, char *work, int32_t R);
// planes: start and left are planes [vector][rows] (pair form).  *retry = true: run.unchecked
// tiles turned out not to hold the matrix, the sweep has to run.
template <class VT>
tbk_status run_tiled(const tbk_ham *h, const KpmPlan &pl, const TileRun &run, double a, double b, const VT *r,
                     int32_t R, int32_t M, char *work, double *mu, hipStream_t s, const VT *start, const VT *left,
                     bool planes = false, bool *retry = nullptr);
// phi_out = exp(-i b dt / hbar) sum_k c[k] T_k(Ht) phi for R vectors in planes
// (n_cheb >= 2 terms, coefficients cre + i cim, phase pr + i pi); phi_out is not phi.
template <class VT>
tbk_status propagate_tiled(const tbk_ham *h, const KpmPlan &pl, const TileRun &run, double a, double b, int32_t R,
                           int32_t n_cheb, const double *cre, const double *cim, double pr, double pi, char *work,
                           hipStream_t s, const VT *phi, VT *phi_out);
unsigned tile_grid(const TileRun &run, int32_t R);
// The first `need` planes of the workspace; fails where the layout reserves fewer.
template <class VT>
tbk_status tile_planes(const TilePlan &tp, char *work, int need, VT *(&plane)[kPlanesMax]) {
    TBK_CHECK(need <= tp.planes && need <= kPlanesMax, TBK_ERR_DEVICE, "%d planes needed, %d in the workspace", need,
              tp.planes);
    for (int k = 0; k < need; ++k) plane[k] = reinterpret_cast<VT *>(work + tp.off_planes + k * tp.plane_bytes);
    return TBK_OK;
}
// One launch of a group of steps.
template <class VT>
void launch_tile_group(const KpmPlan &pl, bool diag, int form, unsigned grid, hipStream_t s, const TileArgs<VT> &a);
// Start vectors (caller's order) to planes, and the sums of |r|^2 per tile.
template <class VT>
void tile_start_planes(const tbk_ham *h, const KpmPlan &pl, const TileRun &run, const VT *r, int32_t R, char *work,
                       VT *rp, double *part, hipStream_t s);

}  // namespace tbk
