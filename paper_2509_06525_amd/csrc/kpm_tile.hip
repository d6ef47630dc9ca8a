// Tiled recurrence (kpm_tile.hpp): tile lists, workspace layout and the driver
// of a run.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "kpm_run.hpp"
#include "kpm_tile.hpp"

namespace tbk {
namespace {

constexpr int kPlanThreads = 512;
constexpr int kHaloMax = 2048;         // halo rows a tile can list
constexpr int kLocalBond = 256;        // rows between the ends of a bond inside a strip, at most (about two lines of cells)
constexpr int kHashSize = 4096;        // open addressing, at most kHaloMax + kPlanThreads keys
constexpr int kTileMaxW = 6;           // entries per row
constexpr size_t kTilePartialBudget = 64ull << 20;       // a quarter of it for runs that the static workspace takes
constexpr size_t kPlaneBudget = 32ull << 30;

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct TileInfo {                       // what the host reads back
    int32_t rings;                      // rings complete in every tile
    int32_t n_tiles;                    // tiles after the split
    int32_t mixed, pad;                 // 1: some entry's value is not the first one's, or not 0 in the row's own column
    unsigned long long rows[kTileMaxS + 1];   // sum over tiles of the rows within k rings
};

// first[t] = first row of tile t of n_tiles tiles of equal size over n rows;
// clears the summary.
__global__ void k_tile_rows(int64_t n, int32_t n_tiles, int32_t S, int32_t *__restrict__ first,
                            TileInfo *__restrict__ info) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (first && t <= n_tiles) first[t] = (int32_t)((n * t) / n_tiles);
    if (t <= kTileMaxS) info->rows[t] = 0;
    if (t == 0) {
        info->rings = S;
        info->n_tiles = n_tiles;
        info->mixed = 0;
    }
}

// Cuts the tiles across a strip's end in two there (the builder orders rows in strips
// of cells; such a tile is two patches of the sheet, with two edges more than its
// neighbours, and would set the steps per launch for all of them: 96 snapshots of 1,000
// to 50,000 atoms, 8 vectors, 15.8 ms with tiles halved anywhere, 13.1 so), and halves
// those whose halo does not fit.  The rings k asked of every tile
// are those with the most steps per tile, k over the number of tiles that result:
// where only a few tiles reach S (long bonds), halving the rest costs more than
// the rings are worth (1 M rows of up to 5 entries, four vectors: 16.0 us a step at
// the S = 8 of half tiles, 11.2 at the 5 rings that fit).  One workgroup: every
// thread counts the pieces of a run of tiles, a scan places them.  At most `most`
// tiles result; entries past the last one hold n.
__global__ __launch_bounds__(1024) void k_tile_split(const int32_t *__restrict__ first, const int32_t *__restrict__ rings,
                                                     const int32_t *__restrict__ seg, int32_t n_tiles, int32_t most,
                                                     int32_t S, int32_t n, int32_t *__restrict__ row0,
                                                     int32_t *__restrict__ tseg, TileInfo *__restrict__ info) {
    __shared__ int32_t sum[1024];
    __shared__ int32_t reach[kTileMaxS + 1];      // tiles of just so many rings
    __shared__ int32_t cuts;
    const int tid = threadIdx.x;
    const int per = (n_tiles + 1023) / 1024;
    const int t0 = min(tid * per, n_tiles), t1 = min(t0 + per, n_tiles);
    if (tid <= kTileMaxS) reach[tid] = 0;
    __syncthreads();
    if (tid == 0) cuts = 0;
    __syncthreads();
    for (int t = t0; t < t1; ++t) {
        atomicAdd(&reach[rings[t] >> 8 ? S : min(rings[t] & 255, S)], 1);
        if (rings[t] >> 8) atomicAdd(&cuts, 1);
    }
    __syncthreads();
    const int base = n_tiles + cuts;
    int need = 1;
    int64_t need_tiles = base;
    for (int k = 1, less = 0; k <= S; ++k) {
        less += reach[k - 1];
        if (base + less <= most && k * need_tiles >= (int64_t)need * (base + less)) {
            need = k;
            need_tiles = base + less;
        }
    }
    // rows of tile t's first piece (all of them: one piece)
    auto piece = [&](int t) {
        const int len = first[t + 1] - first[t], cut = rings[t] >> 8;
        return cut ? cut : ((rings[t] & 255) < need && len >= 2 ? len / 2 : len);
    };
    auto pieces = [&](int t) { return piece(t) < first[t + 1] - first[t] ? 2 : 1; };
    int c = 0;
    for (int t = t0; t < t1; ++t) c += pieces(t);
    sum[tid] = c;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int x = tid >= d ? sum[tid - d] : 0;
        __syncthreads();
        sum[tid] += x;
        __syncthreads();
    }
    const int total = sum[1023];
    const bool split = total <= most;       // otherwise the tiles stay as they are
    int q = split ? sum[tid] - c : t0;
    for (int t = t0; t < t1; ++t) {
        const int lo = first[t], np = split ? pieces(t) : 1;
        for (int k = 0; k < np; ++k, ++q) {
            row0[q] = lo + (k ? piece(t) : 0);
            if (seg) tseg[q] = seg[t];
        }
    }
    const int count = split ? total : n_tiles;
    for (int k = count + tid; k <= most; k += 1024) row0[k] = n;
    if (tid == 0) info->n_tiles = count;
}

struct TilePlanArgs {
    const int64_t *ptr;
    const int32_t *col;
    const void *val, *onsite;
    const int32_t *row0;
    int32_t *cnt, *ext;
    uint32_t *lcol2;
    uint16_t *lcol1;
    void *tval, *tons;
    TileInfo *info;
    int32_t *rings;          // PROBE: complete rings and cut of each tile
    int32_t log2_slice, S, W, cap;
};

template <class VT> __device__ __forceinline__ bool same_bits(VT x, VT y) {
    if constexpr (sizeof(VT) == 4) return __float_as_int(x) == __float_as_int(y);
    else return __double_as_longlong(x) == __double_as_longlong(y);
}

// Lists of one tile: breadth-first over the bonds, ring by ring.  Rows outside
// the tile go through an LDS hash table (row -> local index) and take the next
// local index when first met, so a ring follows the order of the rows that reach
// it.  The order within a ring is not reproducible, the results are: every value
// depends on its own row's entries only, and only the tile's rows are summed.
// PROBE: counts the rings that fit, and looks for the end of a strip among the rows
// (no bond to a row within kLocalBond after crosses it): rings[t] = rings | cut << 8,
// cut = 0 or the row of the tile that starts the next strip.
template <class VT, bool PROBE>
__global__ __launch_bounds__(kPlanThreads) void k_tile_plan(TilePlanArgs a) {
    __shared__ int32_t keys[kHashSize];
    __shared__ uint16_t lidx[kHashSize];
    __shared__ int32_t list[kHaloMax];
    __shared__ int32_t s_count, s_over;
    const int t = blockIdx.x, tid = threadIdx.x;
    const int row0 = a.row0[t], nr = a.row0[t + 1] - row0;
    if (nr == 0) {
        if (PROBE && tid == 0) a.rings[t] = a.S;
        return;
    }
    const int cap_h = min(a.cap - nr, kHaloMax);
    const int64_t smask = ((int64_t)1 << a.log2_slice) - 1, stride = smask + 1;
    for (int i = tid; i < kHashSize; i += kPlanThreads) keys[i] = -1;
    if (tid == 0) { s_count = 0; s_over = 0; }
    __syncthreads();
    int32_t *cnt = a.cnt + (int64_t)t * (a.S + 1);
    if (!PROBE && tid == 0) cnt[0] = nr;
    auto hash = [](int32_t c) { return (uint32_t)c * 2654435761u >> 20; };      // 12 bits
    auto global_row = [&](int j) { return j < nr ? row0 + j : list[j - nr]; };
    auto entries = [&](int64_t g, int64_t &base, int &w) {
        const int64_t sl = g >> a.log2_slice;
        const int64_t p0 = a.ptr[sl], p1 = a.ptr[sl + 1];
        base = p0 + (g & smask);
        w = (int)((p1 - p0) >> a.log2_slice);
    };
    // the first a.W (<= kTileMaxW) columns of a row, all loaded before any is used; own row past w
    auto columns = [&](int64_t g, int64_t base, int w, int32_t (&c)[kTileMaxW]) {
#pragma unroll
        for (int q = 0; q < kTileMaxW; ++q) {
            c[q] = (int32_t)g;
            if (q < a.W && q < w) c[q] = a.col[base + q * stride];
        }
    };
    int lo = 0, hi = nr, done = 0, total = 0;     // rows of the previous ring; complete rings; halo rows
    bool closed = false;
    for (int k = 1; k <= a.S; ++k) {
        for (int j = lo + tid; j < hi; j += kPlanThreads) {
            int64_t base;
            int w;
            int32_t cc[kTileMaxW];
            const int64_t g = global_row(j);
            entries(g, base, w);
            if (w > a.W) s_over = 1;
            columns(g, base, w, cc);
#pragma unroll
            for (int q = 0; q < kTileMaxW; ++q) {
                const int32_t c = cc[q];
                if (c == g || (uint32_t)(c - row0) < (uint32_t)nr) continue;
                uint32_t p = hash(c);
                while (!*(volatile int32_t *)&s_over) {
                    const int32_t old = atomicCAS(&keys[p], -1, c);
                    if (old == c) break;
                    if (old == -1) {
                        const int pos = atomicAdd(&s_count, 1);
                        if (pos < cap_h) { list[pos] = c; lidx[p] = (uint16_t)(nr + pos); }
                        else s_over = 1;
                        break;
                    }
                    p = (p + 1) & (kHashSize - 1);
                }
            }
        }
        __syncthreads();
        if (s_over) break;
        const int now = s_count;
        __syncthreads();
        if (now == total) {             // nothing beyond: the list is closed under the bonds
            if (!PROBE)
                for (int q = k + tid; q <= a.S; q += kPlanThreads) cnt[q] = nr + total;
            done = a.S;
            closed = true;
            break;
        }
        lo = nr + total;
        hi = nr + now;
        total = now;
        done = k;
        if (!PROBE && tid == 0) cnt[k] = nr + now;
    }
    __syncthreads();
    if constexpr (PROBE) {
        if (nr > kHashSize) {
            if (tid == 0) a.rings[t] = done;
            return;
        }
        // place i of d: summed up to it, the rows with a bond, to a row at most kLocalBond after
        // them, across the gap between rows i and i + 1
        int32_t *d = keys, *part = list;
        if (tid == 0) { s_count = 0; s_over = INT32_MAX; }
        for (int i = tid; i < nr; i += kPlanThreads) d[i] = 0;
        __syncthreads();
        for (int j = tid; j < nr; j += kPlanThreads) {
            int64_t base;
            int w;
            int32_t cc[kTileMaxW];
            entries(row0 + j, base, w);
            columns(row0 + j, base, w, cc);
            int far = j;
#pragma unroll
            for (int q = 0; q < kTileMaxW; ++q) {
                const int c = cc[q] - row0;
                if (c <= j + kLocalBond && c < nr) far = max(far, c);
            }
            if (far > j) {
                atomicAdd(&d[j], 1);
                atomicAdd(&d[far], -1);
            }
        }
        __syncthreads();
        const int per = (nr + kPlanThreads - 1) / kPlanThreads;
        const int i0 = min(tid * per, nr), i1 = min(i0 + per, nr);
        int sum = 0;
        for (int i = i0; i < i1; ++i) sum += d[i];
        part[tid] = sum;
        __syncthreads();
        for (int o = 1; o < kPlanThreads; o <<= 1) {
            const int x = tid >= o ? part[tid - o] : 0;
            __syncthreads();
            part[tid] += x;
            __syncthreads();
        }
        int over = part[tid] - sum;
        for (int i = i0; i < i1; ++i) {
            over += d[i];
            if (over != 0 || i + 1 < nr / 16 || i + 1 > nr - nr / 16 || i + 1 == nr) continue;
            atomicAdd(&s_count, 1);
            atomicMin(&s_over, abs(i + 1 - nr / 2) << 16 | (i + 1));
        }
        __syncthreads();
        // many such gaps: rows of no order
        if (tid == 0) a.rings[t] = done | (s_count >= 1 && s_count <= 4 ? (s_over & 0xffff) << 8 : 0);
        return;
    }
    if (tid == 0) {
        atomicMin(&a.info->rings, done);
        for (int k = 0; k <= done; ++k) atomicAdd(&a.info->rows[k], (unsigned long long)cnt[k]);
    }
    const int64_t mb = (int64_t)t * a.cap;
    if (done == 0) {
        // a run that has not been told yet (TileRun::unchecked) may read these: offsets in range
        for (int i = tid; i < nr; i += kPlanThreads) {
            for (int q = 0; q < a.W / 2; ++q) a.lcol2[mb * (a.W / 2) + (int64_t)q * a.cap + i] = 0;
            if (a.W & 1) a.lcol1[mb + i] = 0;
        }
        return;
    }
    if (tid == 0) s_over = 0;
    __syncthreads();
    for (int i = tid; i < total; i += kPlanThreads) a.ext[mb + i] = list[i];
    // matrix rows of every ring but the last, in local form
    const int n_mat = closed ? nr + total : lo;
    const VT *val = static_cast<const VT *>(a.val);
    const VT *ons = static_cast<const VT *>(a.onsite);
    VT *tval = static_cast<VT *>(a.tval);
    VT *tons = static_cast<VT *>(a.tons);
    const int NP = a.W / 2;
    for (int j = tid; j < n_mat; j += kPlanThreads) {
        const int64_t g = global_row(j);
        int64_t base;
        int w;
        int32_t cc[kTileMaxW];
        VT v[kTileMaxW];
        entries(g, base, w);
        columns(g, base, w, cc);
#pragma unroll
        for (int q = 0; q < kTileMaxW; ++q) {
            v[q] = 0;
            if (q < a.W && q < w) v[q] = val[base + q * stride];
        }
        uint32_t lc[kTileMaxW];
#pragma unroll
        for (int q = 0; q < kTileMaxW; ++q) {
            const int32_t c = cc[q];
            lc[q] = (uint32_t)j;
            if (c != g) {
                if ((uint32_t)(c - row0) < (uint32_t)nr) {
                    lc[q] = (uint32_t)(c - row0);
                } else {
                    uint32_t p = hash(c);
                    while (keys[p] != c) p = (p + 1) & (kHashSize - 1);
                    lc[q] = lidx[p];
                }
            }
            lc[q] *= (uint32_t)(2 * sizeof(VT));
        }
#pragma unroll
        for (int q = 0; q < kTileMaxW; ++q) {
            if (q >= a.W) continue;
            tval[mb * a.W + (int64_t)q * a.cap + j] = v[q];
            if (q == a.W - 1 && (a.W & 1)) a.lcol1[mb + j] = (uint16_t)lc[q];
            else if (q & 1) a.lcol2[mb * NP + (int64_t)(q / 2) * a.cap + j] = lc[q - 1] | (lc[q] << 16);
        }
        if (ons) tons[mb + j] = ons[g];
#pragma unroll
        for (int q = 0; q < kTileMaxW; ++q)
            if (q < a.W && q < w && (cc[q] != g ? !same_bits(v[q], val[0]) : v[q] != 0)) s_over = 1;
    }
    __syncthreads();
    if (tid == 0 && s_over) a.info->mixed = 1;
}

// Elements a block turns from [row][vector] to [vector][row] or back at a time: they
// pass through LDS, since with 32 vectors a wavefront that writes planes straight from
// rows writes 16 bytes to each (4 M rows, 32 vectors, 200 moments: the call 49.3 ms with
// planes written straight, 47.4 so).
constexpr int kTurn = 2048;

// Start of a run.  MODE 0: start vectors r (caller's order, or seeded phases) to
// row order [rows][Rp] (r_int) and planes; sums of |r|^2 per tile.  MODE 1 (pair
// form): start and left, [rows][Rp] in row order, to planes; sums of
// Re <left|start>.  A block per tile; thread e takes elements e, e + NT, ... of
// the tile's [row][vector] range, all of one vector.  One tile: NT = 1024, as nothing
// else is there to hide its latencies.
template <class VT, int NT, int MODE, bool DBL>
__global__ __launch_bounds__(NT) void k_tile_prepare(const VT *__restrict__ r, const VT *__restrict__ left,
                                                           const int32_t *__restrict__ perm,
                                                           const int32_t *__restrict__ row0, int64_t rows, int32_t R,
                                                           int32_t Rp, int32_t seeded, uint64_t seed,
                                                           VT *__restrict__ r_int, VT *__restrict__ plane,
                                                           VT *__restrict__ lplane, double *__restrict__ partial) {
    typedef std::conditional_t<sizeof(VT) == 4, f2v, d2v> C2;
    constexpr int E = (NT == kThreads ? 1 : 2) * (MODE == 0 ? kTurn : kTurn / 2), NK = E / NT;
    __shared__ double red[NT];
    __shared__ C2 turn[MODE == 0 ? 1 : 2][E + kThreads];      // [vector][rows of the chunk + 1]
    const int t = blockIdx.x, tid = threadIdx.x;
    const int64_t i0 = row0[t];
    const int nr = row0[t + 1] - row0[t], ne = nr * Rp;
    const int v = tid % Rp, rb = E / Rp;
    const C2 *cr = reinterpret_cast<const C2 *>(r), *cl = reinterpret_cast<const C2 *>(left);
    const bool to_planes = MODE == 1 || plane != r_int;
    double acc = 0.0;
    for (int c0 = 0; c0 < ne; c0 += E) {
        const int j0 = c0 / Rp;              // first row of the chunk
        C2 x[NK], y[MODE == 0 ? 1 : NK];
        int64_t src[NK];
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            const int64_t i = i0 + min(c0 + k * NT + tid, ne - 1) / Rp;
            src[k] = MODE == 0 && perm ? (int64_t)perm[i] : i;
        }
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            x[k].x = x[k].y = 0;
            if (v >= R) continue;
            if constexpr (MODE == 0) {
                if (seeded) {
                    double c, sn;
                    seeded_phase(seed, (uint64_t)src[k] * (uint64_t)R + (uint64_t)v, c, sn);
                    x[k].x = (VT)c;
                    x[k].y = (VT)sn;
                } else {
                    x[k] = cr[src[k] * R + v];
                }
            } else {
                x[k] = cr[src[k] * Rp + v];
                y[k] = cl[src[k] * Rp + v];
            }
        }
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            const int e = c0 + k * NT + tid;
            if (e >= ne) continue;
            const int j = e / Rp;
            if constexpr (MODE == 0) {
                if (r_int) reinterpret_cast<C2 *>(r_int)[i0 * Rp + e] = x[k];
                acc += (double)x[k].x * (double)x[k].x + (double)x[k].y * (double)x[k].y;
            } else if (v < R) {
                turn[MODE == 0 ? 0 : 1][v * (rb + 1) + j - j0] = y[k];
                acc += (double)y[k].x * (double)x[k].x + (double)y[k].y * (double)x[k].y;
            }
            if (to_planes) turn[0][v * (rb + 1) + j - j0] = x[k];
        }
        if (!to_planes) continue;
        __syncthreads();
        for (int f = tid; f < E; f += NT) {
            const int pv = f / rb, j = f % rb;
            if (pv >= R || j0 + j >= nr) continue;
            const int64_t o = (int64_t)pv * rows + i0 + j0 + j;
            reinterpret_cast<C2 *>(plane)[o] = turn[0][pv * (rb + 1) + j];
            if constexpr (MODE == 1) reinterpret_cast<C2 *>(lplane)[o] = turn[1][pv * (rb + 1) + j];
        }
        __syncthreads();
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int g = NT / 2; g >= Rp; g >>= 1) {
        if ((int)threadIdx.x < g) red[threadIdx.x] += red[threadIdx.x + g];
        __syncthreads();
    }
    if ((int)threadIdx.x < Rp) {
        if constexpr (DBL) {
            partial[(int64_t)t * 2 * Rp + 2 * v] = red[v];
            partial[(int64_t)t * 2 * Rp + 2 * v + 1] = 0.0;
        } else {
            partial[(int64_t)t * Rp + v] = red[v];
        }
    }
}

// partial[t][v] = Re <left_v|start_v> over the rows of tile t (planes); grid (tiles, R).
template <class VT>
__global__ __launch_bounds__(kThreads) void k_tile_overlap(const VT *__restrict__ start, const VT *__restrict__ left,
                                                           const int32_t *__restrict__ row0, int64_t rows, int32_t Rp,
                                                           double *__restrict__ partial) {
    __shared__ double red[kThreads / 64];
    const int t = blockIdx.x, v = blockIdx.y;
    double acc = 0.0;
    for (int64_t i = row0[t] + threadIdx.x; i < row0[t + 1]; i += kThreads) {
        const int64_t o = 2 * ((int64_t)v * rows + i);
        acc += (double)left[o] * (double)start[o] + (double)left[o + 1] * (double)start[o + 1];
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) s += red[w];
        partial[(int64_t)t * Rp + v] = s;
    }
}

// Columns v0 .. v0 + Rp - 1 of [rows][pitch] <-> planes [vector][rows] of the first R of them,
// for up to three arrays (grid y; TO: into planes; columns past R are padding, of zeros).
template <class VT> struct PlaneSets {
    VT *x[3], *plane[3];
};
template <class VT, bool TO>
__global__ __launch_bounds__(kThreads) void k_planes(PlaneSets<VT> ps, int64_t rows, int32_t R, int32_t Rp,
                                                       int32_t pitch, int32_t v0) {
    typedef std::conditional_t<sizeof(VT) == 4, f2v, d2v> C2;
    __shared__ C2 turn[kTurn + kThreads];
    const int set = blockIdx.y, rb = kTurn / Rp;
    C2 *x = reinterpret_cast<C2 *>(set == 0 ? ps.x[0] : (set == 1 ? ps.x[1] : ps.x[2]));
    C2 *plane = reinterpret_cast<C2 *>(set == 0 ? ps.plane[0] : (set == 1 ? ps.plane[1] : ps.plane[2]));
    const int64_t i0 = (int64_t)blockIdx.x * rb;
    const int nr = (int)min((int64_t)rb, rows - i0);
    x += i0 * pitch + v0;
    // thread order of the row form (e = row * Rp + vector) and of the planes (f = vector * rb + row)
#pragma unroll
    for (int k = 0; k < kTurn / kThreads; ++k) {
        const int f = k * kThreads + threadIdx.x;
        const int j = TO ? f / Rp : f % rb, v = TO ? f % Rp : f / rb;
        if (j >= nr) continue;
        C2 y;
        y.x = y.y = 0;
        if (v < R) y = TO ? x[j * pitch + v] : plane[(int64_t)v * rows + i0 + j];
        turn[v * (rb + 1) + j] = y;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTurn / kThreads; ++k) {
        const int f = k * kThreads + threadIdx.x;
        const int j = TO ? f % rb : f / Rp, v = TO ? f / rb : f % Rp;
        if (j >= nr) continue;
        if (!TO) x[j * pitch + v] = turn[v * (rb + 1) + j];
        else if (v < R) plane[(int64_t)v * rows + i0 + j] = turn[v * (rb + 1) + j];
    }
}

template <class VT>
void launch_steps(const TilePlan &tp, bool diag, int form, unsigned grid, hipStream_t s, const TileArgs<VT> &a) {
    if (tp.W == 3) launch_tile_steps<VT, 3>(tp, diag, form, grid, s, a);
    else if (tp.W == 4) launch_tile_steps<VT, 4>(tp, diag, form, grid, s, a);
    else launch_tile_steps<VT, 6>(tp, diag, form, grid, s, a);
}

// Layout for rows of up to W entries from byte `base` on.
void layout_width(const tbk_ham *h, const KpmPlan &pl, size_t base, int32_t R, int32_t n_seg, int planes, bool sets,
                  int W, TilePlan &tp) {
    tp = TilePlan{};
    tp.W = W;
    tp.planes = planes;
    const int64_t n = h->n_rows, work = n * R;
    const bool f64 = pl.elem == sizeof(double);
    auto shape = [&](int sh) {
        tp.shape = sh;
        tp.NT = tile_threads(sh);
        tp.K = tile_slots(sh, W, f64);
        tp.cap = tile_cap(tp.NT, tp.K);
    };
    shape(kTileWhole);
    if (n_seg == 1 && n <= tp.cap) {
        tp.n_first = tp.n_tiles = 1;
        tp.tile_rows = n;
        tp.S = tp.L = 1;
    } else {
        // Rows per tile and rings.  Large systems: 0.7 of the capacity (0.6 in FP64 and for
        // rows of 5 and 6 entries) and up to eight (six) rings, of which k_tile_split takes
        // what pays; 16 M row-vectors, us per step: 31.4 with 0.75 of the capacity, 29.1 with
        // 0.7, 30.1 with 0.65, 31.0 with 0.55 and ten rings (the sweep: 148).  Systems with
        // fewer tiles than CUs: smaller tiles, whose larger halo costs less than idle CUs;
        // 30,212 rows, three vectors: 1.18 us per step with 354 rows (256 workgroups), the
        // sweep 4.8; 300,000 rows, two vectors: 0.4 of the capacity was 9% faster than 8/15.
        if (!f64 && work < 700000) {
            shape(kTileSmall);
            tp.tile_rows = std::min<int64_t>(tp.cap * (W <= 4 ? 6 : 8) / 15, std::max<int64_t>(256, work / 256));
        } else {
            shape(h->has_onsite ? kTileLargeDiag : kTileLarge);
            if (f64) tp.tile_rows = std::min<int64_t>(tp.cap * 3 / 5, std::max<int64_t>(256, work / 400));
            else tp.tile_rows = std::min<int64_t>(tp.cap * (W <= 4 ? 7 : 6) / 10, std::max<int64_t>(tp.cap * 7 / 25, work / 512));
        }
        tp.S = (f64 || tp.shape == kTileSmall) && tp.tile_rows > tp.cap * 2 / 5 ? 6 : 8;
        // Two rings more on small tiles: 5 us of lists, 0.06 us a step; no more than a run has
        // steps.  The cut asks for S whatever the number of moments: where tiles end decides the
        // grouping of the moments' sums, and the parts of a run split over calls add up as one run's.
        tp.L = std::min(tp.shape == kTileSmall && tp.S == 8 && pl.Mr > 200 ? 10 : tp.S, std::max(2, pl.Mr - 1));
        tp.n_first = ceil_div(n, tp.tile_rows) + (n_seg > 1 ? n_seg : 0);   // a partial tile per structure
        tp.n_tiles = tp.n_first + tp.n_first / 8 + 8 + (n_seg > 1 ? 2 * n_seg : 0);      // room for tiles cut in two
    }
    const size_t per_step = (size_t)tp.n_tiles * pl.Rv * sizeof(double);
    tp.reduce_every = (int)std::min<size_t>(kTilePartialBudget / (base > kStaticSweepBytes || n_seg > 1 ? 1 : 4) / per_step,
                                            (size_t)std::min(pl.Mr, 4096));
    tp.reduce_every = std::max(tp.reduce_every, kTileMaxS + 1);
    const size_t rows = (size_t)tp.n_tiles * tp.cap;
    const size_t chunks = (size_t)ceil_div(tp.n_tiles, kReduceChunk);
    size_t o = base;
    auto take = [&](size_t bytes) { const size_t at = o; o += align256(bytes); return at; };
    tp.off_first = take(sizeof(int32_t) * (tp.n_first + 1));
    tp.off_fseg = take(sizeof(int32_t) * tp.n_first);
    tp.off_rings = take(sizeof(int32_t) * tp.n_first);
    tp.off_row0 = take(sizeof(int32_t) * (tp.n_tiles + 1));
    tp.off_tseg = take(sizeof(int32_t) * tp.n_tiles);
    tp.off_info = take(sizeof(TileInfo));
    tp.off_cnt = take(sizeof(int32_t) * tp.n_tiles * (tp.L + 1));
    tp.off_ext = take(sizeof(int32_t) * rows);
    tp.off_lcol2 = take(sizeof(uint32_t) * rows * (W / 2));
    tp.off_lcol1 = take(sizeof(uint16_t) * rows * (W % 2));
    tp.off_val = take(pl.elem * rows * W);
    tp.off_ons = take(h->has_onsite ? pl.elem * rows : 0);
    tp.off_part = take((size_t)tp.reduce_every * per_step);
    tp.off_l1 = take((size_t)pl.Mr * pl.Rv * chunks * sizeof(double));
    // A plane holds all vectors, unless the planes took more than 32 GB: then as many as fit
    // (100 M rows: eight in complex float; 40 vectors: 161 + 32 GB, where planes of all took 194).
    tp.Rc = pl.Rp;
    while (sets && tp.Rc > 1 && (size_t)planes * n * tp.Rc * 2 * pl.elem > kPlaneBudget) tp.Rc /= 2;
    tp.plane_bytes = align256((size_t)n * std::min(R, tp.Rc) * 2 * pl.elem);
    tp.off_planes = take(planes * tp.plane_bytes);
    tp.total = o;
}

}  // namespace

// The probe, the lists and the wait between them against the sweep's steps, us per call on
// tiles and swept: 2,304 rows, 4 steps of doubling 81, 84; 30,212 rows, three vectors, 16 and
// 31 steps 161, 124 and 186, 205; a stack of 20,180 rows, eight vectors, 23 and 31 steps 230,
// 204 and 237, 236; 250,000 rows in FP64, four vectors, 8 and 12 steps 214, 181 and 223, 235; 16 M
// rows, 10 and 12 steps 1479, 1378 and 1519, 1628; a stack of 867,364 rows, eight vectors, 7
// and 11 steps 409, 429 and 502, 604.
bool tile_pays(const TilePlan &tp, int steps) {
    return steps >= (tp.shape == kTileWhole ? 4 : (tp.shape == kTileSmall ? 28 : 10));
}

void tile_layout(const tbk_ham *h, KpmPlan &pl, size_t base, int32_t R, int32_t n_seg, int planes, bool sets) {
    pl.tile = TilePlan{};
    pl.tile.total = base;
    if (pl.block || h->max_degree < 1 || h->max_degree > kTileMaxW || pl.cfg.persistent) return;
    TilePlan other;
    layout_width(h, pl, base, R, n_seg, planes, sets, h->max_degree <= 3 ? 3 : (h->max_degree <= 4 ? 4 : 6), pl.tile);
    if (pl.tile.W <= 4) {
        // one size for degrees up to 4, so that a workspace serves frames of either
        layout_width(h, pl, base, R, n_seg, planes, sets, pl.tile.W == 3 ? 4 : 3, other);
        pl.tile.total = std::max(pl.tile.total, other.total);
    }
    pl.tile.on = true;
}

// Tile lists of h (or of its structures, whose row0 table the caller has
// written) and the number of steps per launch.  run.s = 0: the halos do not fit
// (rows without locality), the sweep per step is to be used.
template <class VT>
tbk_status tile_build(const tbk_ham *h, const KpmPlan &pl, int n_first, char *work, hipStream_t s, TileRun &run,
                      bool defer) {
    const TilePlan &tp = pl.tile;
    run = TileRun{};
    int32_t *first = reinterpret_cast<int32_t *>(work + tp.off_first);
    int32_t *fseg = reinterpret_cast<int32_t *>(work + tp.off_fseg);
    int32_t *row0 = reinterpret_cast<int32_t *>(work + tp.off_row0);
    int32_t *tseg = reinterpret_cast<int32_t *>(work + tp.off_tseg);
    TileInfo *info = reinterpret_cast<TileInfo *>(work + tp.off_info);
    const bool whole = tp.shape == kTileWhole;             // the whole matrix in one tile
    const bool table = n_first > 0;               // the caller has written first and fseg
    const int nf = table ? n_first : (int)tp.n_first;
    k_tile_rows<<<(unsigned)ceil_div(nf + 1 + kTileMaxS, 256), 256, 0, s>>>(
        h->n_rows, nf, tp.L, whole ? row0 : (table ? nullptr : first), info);
    TilePlanArgs pa{};
    pa.ptr = h->ptr;
    pa.col = h->col;
    pa.val = h->val;
    pa.onsite = h->has_onsite ? h->onsite : nullptr;
    pa.cnt = reinterpret_cast<int32_t *>(work + tp.off_cnt);
    pa.ext = reinterpret_cast<int32_t *>(work + tp.off_ext);
    pa.lcol2 = reinterpret_cast<uint32_t *>(work + tp.off_lcol2);
    pa.lcol1 = reinterpret_cast<uint16_t *>(work + tp.off_lcol1);
    pa.tval = work + tp.off_val;
    pa.tons = work + tp.off_ons;
    pa.info = info;
    pa.rings = reinterpret_cast<int32_t *>(work + tp.off_rings);
    pa.log2_slice = pl.log2_slice;
    pa.W = tp.W;
    pa.cap = tp.cap;
    if (!whole) {
        pa.row0 = first;
        pa.S = tp.S;
        k_tile_plan<VT, true><<<(unsigned)nf, kPlanThreads, 0, s>>>(pa);
        k_tile_split<<<1, 1024, 0, s>>>(first, pa.rings, table ? fseg : nullptr, nf, (int)tp.n_tiles, tp.S,
                                        (int)h->n_rows, row0, tseg, info);
    }
    pa.row0 = row0;
    pa.S = tp.L;
    k_tile_plan<VT, false><<<(unsigned)(whole ? 1 : tp.n_tiles), kPlanThreads, 0, s>>>(pa);
    TBK_HIP(hipGetLastError());
    if (whole && defer) {       // closed, unless a row is wider than W: looked at after the run (no wait here)
        run.n_tiles = 1;
        run.closed = true;
        run.s = INT32_MAX;
        run.unchecked = &info->rings;
        return TBK_OK;
    }
    TileInfo hi;
    TBK_HIP(hipMemcpyAsync(&hi, info, sizeof hi, hipMemcpyDeviceToHost, s));
    TBK_HIP(hipStreamSynchronize(s));
    run.n_tiles = hi.n_tiles;
    run.uniform = !whole && hi.mixed == 0;
    if (hi.rings >= 1 && hi.rows[hi.rings] == hi.rows[0]) {
        run.closed = true;
        run.s = INT32_MAX;
        return TBK_OK;
    }
    if (hi.rings < 2) return TBK_OK;     // one ring saves nothing over the sweep
    run.s = hi.rings;
    return TBK_OK;
}

template <class VT>
TileArgs<VT> tile_args(const tbk_ham *h, const KpmPlan &pl, const TileRun &run, char *work, int32_t R) {
    const TilePlan &tp = pl.tile;
    TileArgs<VT> a{};
    a.row0 = reinterpret_cast<const int32_t *>(work + tp.off_row0);
    a.cnt = reinterpret_cast<const int32_t *>(work + tp.off_cnt);
    a.ext = reinterpret_cast<const int32_t *>(work + tp.off_ext);
    a.lcol2 = reinterpret_cast<const uint32_t *>(work + tp.off_lcol2);
    a.lcol1 = reinterpret_cast<const uint16_t *>(work + tp.off_lcol1);
    a.val = reinterpret_cast<const VT *>(work + tp.off_val);
    a.hop = run.uniform ? static_cast<const VT *>(h->val) : nullptr;
    a.ons = h->has_onsite ? reinterpret_cast<const VT *>(work + tp.off_ons) : nullptr;
    a.rows = h->n_rows;
    a.n_work = run.n_tiles * R;
    a.R = R;
    a.Rv = pl.cfg.doubling ? 2 * pl.Rp : pl.Rp;
    a.pstride = (int64_t)run.n_tiles * a.Rv;
    a.S1 = tp.L + 1;
    a.cap = tp.cap;
    a.closed = run.closed ? 1 : 0;
    return a;
}

unsigned tile_grid(const TileRun &run, int32_t R) {
    return (unsigned)(ceil_div((int64_t)run.n_tiles * R, xcd_grid_multiple(2)) * xcd_grid_multiple(2));
}

template <class VT>
tbk_status run_tiled(const tbk_ham *h, const KpmPlan &pl, const TileRun &run, double a, double b, const VT *r,
                     int32_t R, int32_t M, char *work, double *mu, hipStream_t s, const VT *start, const VT *left,
                     bool planes, bool *retry) {
    const TilePlan &tp = pl.tile;
    const bool pair = left != nullptr, dbl = pl.cfg.doubling != 0;
    const int n_start = pl.n_start;
    const int64_t n = h->n_rows;
    const int Rp = pl.Rp, Rc = tp.Rc;
    const bool direct = Rp == 1;                   // the row form is the plane
    const bool sets = Rc < Rp;                     // planes hold Rc vectors: set after set runs
    VT *r_int = reinterpret_cast<VT *>(work + pl.off_r);
    VT *T[2] = {reinterpret_cast<VT *>(work + pl.off_a), reinterpret_cast<VT *>(work + pl.off_b)};
    VT *plane[kPlanesMax] = {};
    const int need = pair ? (direct || planes ? 1 : kPlanesPair) : (direct ? kPlanesDirect : kPlanesRun);
    const tbk_status st = tile_planes<VT>(tp, work, need, plane);
    if (st != TBK_OK) return st;
    // pairs of vectors (even n, odd n); with one vector the first pair is the state's own, and
    // in the pair form, which keeps none, r, T_a and T_b serve as planes
    const bool own = direct || pair;
    VT *P[2][2] = {{own ? T[0] : plane[0], own ? T[1] : plane[1]},
                   {pair ? r_int : (direct ? plane[0] : plane[2]), pair ? plane[0] : (direct ? plane[1] : plane[3])}};
    VT *rp = direct ? r_int : plane[4], *sp = rp;
    double *part = reinterpret_cast<double *>(work + tp.off_part);
    double *l1 = reinterpret_cast<double *>(work + tp.off_l1);
    const int Rv = pl.Rv, Rout = dbl ? Rv : R;
    const int n_chunks = (int)ceil_div(run.n_tiles, kReduceChunk);
    const int32_t *row0 = reinterpret_cast<const int32_t *>(work + tp.off_row0);
    const unsigned gt = (unsigned)run.n_tiles;
    const bool one = run.n_tiles == 1;
    const unsigned ge = (unsigned)ceil_div(n * Rc, kTurn);

    if (pair) {
        if (direct || planes) {
            rp = const_cast<VT *>(left);
            sp = const_cast<VT *>(start);
            k_tile_overlap<VT><<<dim3(gt, R), kThreads, 0, s>>>(start, left, row0, n, Rp, part);
        } else {
            rp = plane[1];
            sp = plane[2];
            if (one) k_tile_prepare<VT, 1024, 1, false><<<gt, 1024, 0, s>>>(start, left, nullptr, row0, n, R, Rp, 0, 0,
                                                                           nullptr, sp, rp, part);
            else k_tile_prepare<VT, kThreads, 1, false><<<gt, kThreads, 0, s>>>(start, left, nullptr, row0, n, R, Rp, 0,
                                                                                0, nullptr, sp, rp, part);
        }
    } else if (n_start == 0) {
        const int seeded = pl.seeded ? 1 : 0;
        VT *to = sets ? r_int : rp;
        auto prepare = [&](auto d) {
            constexpr bool D = decltype(d)::value;
            if (one) k_tile_prepare<VT, 1024, 0, D><<<gt, 1024, 0, s>>>(r, nullptr, h->perm, row0, n, R, Rp, seeded,
                                                                       pl.seed, r_int, to, nullptr, part);
            else k_tile_prepare<VT, kThreads, 0, D><<<gt, kThreads, 0, s>>>(r, nullptr, h->perm, row0, n, R, Rp,
                                                                            seeded, pl.seed, r_int, to, nullptr, part);
        };
        if (dbl) prepare(std::true_type{});
        else prepare(std::false_type{});
    }
    TBK_HIP(hipGetLastError());

    TileArgs<VT> ta = tile_args<VT>(h, pl, run, work, R);
    ta.r = rp;
    ta.c1f = (VT)(1.0 / a);
    ta.c1 = (VT)(2.0 / a);
    ta.shift = (VT)b;
    const bool diag = h->has_onsite || b != 0.0;
    const int NA = dbl ? 2 : 1;
    // l1 rows of the moments n0 .. n0 + count - 1 from the partials of the vectors v0 .. v0 + w - 1 (Rv_c sums a tile)
    auto reduce = [&](int n0, int count, int v0, int w, int Rv_c) {
        dim3 g(n_chunks, count);
        k_reduce_l1<<<g, kThreads, 0, s>>>(part, run.n_tiles, Rv_c, w, Rout, n0, n_chunks,
                                           l1 + (int64_t)v0 * NA * n_chunks);
    };
    if (sets && n_start == 0) reduce(0, 1, 0, Rout, Rv);

    StepTimer &timer = step_timer();
    const bool timed = timer.on && !pair;
    bool open = false;
    if (timed) timer.used = 0;
    // the steps n0 + 1 .. Mr - 1, dealt evenly to `groups` launches
    const int n0 = n_start > 0 ? n_start - 1 : 0;       // T_{n0} is the newest vector at hand
    const int steps = pl.Mr - 1 - n0;
    const int most = std::min<int64_t>(run.s, run.closed ? tp.reduce_every - 1 : kTileMaxS);
    const int groups = (int)ceil_div(steps, most);
    run_form() = {run.n_tiles, (int32_t)ceil_div(steps, groups)};
    for (int v0 = 0; v0 < (sets ? Rp : 1); v0 += Rc) {
        const int Rs = std::max(0, std::min(R - v0, Rc));      // vectors of the set (0: only padding)
        const int w = sets ? Rs * NA : Rout, Rv_c = sets ? Rc * NA : Rv;
        if (Rs > 0) {
            if (n_start > 0 && !direct)
                k_planes<VT, true><<<dim3(ge, 3), kThreads, 0, s>>>(
                    {{r_int, T[0], T[1]}, {rp, P[0][0], P[0][1]}}, n, Rs, Rc, Rp, v0);
            else if (sets)
                k_planes<VT, true><<<dim3(ge, 1), kThreads, 0, s>>>({{r_int, nullptr, nullptr}, {rp, nullptr, nullptr}},
                                                                    n, Rs, Rc, Rp, v0);
            TBK_HIP(hipGetLastError());
        }
        ta.R = Rs;
        ta.n_work = run.n_tiles * Rs;
        ta.Rv = Rv_c;
        ta.pstride = (int64_t)run.n_tiles * Rv_c;
        const unsigned grid = tile_grid(run, Rs);
        // a fresh run ends in pair 0; a continued one starts there
        int dst = n_start > 0 ? 1 : (groups - 1) & 1;
        int batch0 = sets && n_start == 0 ? 1 : n_start;     // first row index of the pending batch of partials
        int at = n0;                                         // T_at is the newest vector
        const VT *cur = n_start > 0 ? P[0][at & 1] : sp;
        // T_0 of a run that ended at T_1 is r (the sweep leaves no copy of it)
        const VT *prev = n_start > 2 ? P[0][(at + 1) & 1] : (n_start == 2 ? rp : sp);
        for (int q = 0; q < groups && Rs > 0; ++q) {
            const int len = steps / groups + (q < steps % groups ? 1 : 0);
            if (at + 1 + len - batch0 > tp.reduce_every) {
                if (open) { TBK_HIP(timer.mark(s)); open = false; }
                reduce(batch0, at + 1 - batch0, v0, w, Rv_c);
                batch0 = at + 1;
            }
            if (timed && !open) { TBK_HIP(timer.mark(s)); open = true; }
            if (timed && v0 == 0) timer.launches += len;
            ta.first = at == 0;
            ta.s = len;
            ta.cur = cur;
            ta.prev = prev;
            const int end = at + len;
            const bool keep = q + 1 < groups || !(pair || dbl);    // the last group's vectors: only for a run to continue
            ta.out_cur = keep ? P[dst][end & 1] : nullptr;
            ta.out_prev = keep ? P[dst][(end + 1) & 1] : nullptr;
            ta.partial = part + (int64_t)(at + 1 - batch0) * ta.pstride;
            launch_steps<VT>(tp, diag, dbl ? kTileDoubling : kTileDirect, grid, s, ta);
            cur = ta.out_cur;
            prev = ta.out_prev;
            at = end;
            dst ^= 1;
        }
        if (open) { TBK_HIP(timer.mark(s)); open = false; }
        if (Rs > 0) reduce(batch0, pl.Mr - batch0, v0, w, Rv_c);
        TBK_HIP(hipGetLastError());
        if (pair || dbl) continue;
        // the state of the run, in row order
        const int last = pl.Mr - 1;
        VT *y[2] = {T[last & 1], T[(last + 1) & 1]};          // of T_last, T_{last-1}
        const VT *x[2] = {cur, prev};
        if (!direct)
            k_planes<VT, false><<<dim3(ge, 2), kThreads, 0, s>>>(
                {{y[0], y[1], nullptr}, {const_cast<VT *>(x[0]), const_cast<VT *>(x[1]), nullptr}}, n, Rs, Rc, Rp, v0);
        for (int q = 0; q < 2 && direct; ++q)
            if (x[q] != y[q])
                TBK_HIP(hipMemcpyAsync(y[q], x[q], sizeof(VT) * 2 * (size_t)n, hipMemcpyDeviceToDevice, s));
        TBK_HIP(hipGetLastError());
    }
    return finish_run<VT>(h, pl, a, b, R, M, work, mu, s, pair, dbl, 1, l1, n_chunks, timed, run.unchecked,
                          retry);
}

template <class VT>
void launch_tile_group(const KpmPlan &pl, bool diag, int form, unsigned grid, hipStream_t s, const TileArgs<VT> &a) {
    launch_steps<VT>(pl.tile, diag, form, grid, s, a);
}

template <class VT>
void tile_start_planes(const tbk_ham *h, const KpmPlan &pl, const TileRun &run, const VT *r, int32_t R, char *work,
                       VT *rp, double *part, hipStream_t s) {
    const int32_t *row0 = reinterpret_cast<const int32_t *>(work + pl.tile.off_row0);
    k_tile_prepare<VT, kThreads, 0, false><<<(unsigned)run.n_tiles, kThreads, 0, s>>>(
        r, nullptr, h->perm, row0, h->n_rows, R, pl.Rp, 0, 0, nullptr, rp, nullptr, part);
}

template <class VT>
tbk_status propagate_tiled(const tbk_ham *h, const KpmPlan &pl, const TileRun &run, double a, double b, int32_t R,
                           int32_t n_cheb, const double *cre, const double *cim, double pr, double pi, char *work,
                           hipStream_t s, const VT *phi, VT *phi_out) {
    const TilePlan &tp = pl.tile;
    VT *plane[kPlanesMax] = {};
    const tbk_status st = tile_planes<VT>(tp, work, kPlanesPropagate, plane);
    if (st != TBK_OK) return st;
    TileArgs<VT> ta = tile_args<VT>(h, pl, run, work, R);
    ta.c1f = (VT)(1.0 / a);
    ta.c1 = (VT)(2.0 / a);
    ta.shift = (VT)b;
    ta.c0r = cre[0];
    ta.c0i = cim[0];
    ta.pr = pr;
    ta.pi = pi;
    const bool diag = h->has_onsite || b != 0.0;
    const unsigned grid = tile_grid(run, R);
    const int steps = n_cheb - 1;
    const int groups = (int)ceil_div(steps, std::min<int64_t>(run.s, kTileMaxS));
    int at = 0, dst = 0;
    const VT *cur = phi, *prev = phi;
    for (int q = 0; q < groups; ++q) {
        const int len = steps / groups + (q < steps % groups ? 1 : 0);
        const bool last = q + 1 == groups;
        ta.first = at == 0;
        ta.s = len;
        ta.cur = cur;
        ta.prev = prev;
        ta.out_cur = last ? nullptr : plane[2 * dst];
        ta.out_prev = last ? nullptr : plane[2 * dst + 1];
        ta.acc_in = plane[4];
        ta.acc_out = last ? phi_out : plane[4];
        for (int m = 0; m < len; ++m) {
            ta.cr[m] = cre[at + 1 + m];
            ta.ci[m] = cim[at + 1 + m];
        }
        launch_steps<VT>(tp, diag, kTilePropagate, grid, s, ta);
        cur = ta.out_cur;
        prev = ta.out_prev;
        at += len;
        dst ^= 1;
    }
    TBK_HIP(hipGetLastError());
    return TBK_OK;
}

#define TBK_TILE_INST(VT)                                                                                              \
    template tbk_status tile_build<VT>(const tbk_ham *, const KpmPlan &, int, char *, hipStream_t, TileRun &, bool);  \
    template TileArgs<VT> tile_args<VT>(const tbk_ham *, const KpmPlan &, const TileRun &, char *, int32_t);           \
    template tbk_status run_tiled<VT>(const tbk_ham *, const KpmPlan &, const TileRun &, double, double, const VT *,   \
                                      int32_t, int32_t, char *, double *, hipStream_t, const VT *, const VT *, bool,   \
                                      bool *);                                                                        \
    template tbk_status propagate_tiled<VT>(const tbk_ham *, const KpmPlan &, const TileRun &, double, double,         \
                                            int32_t, int32_t, const double *, const double *, double, double, char *,  \
                                            hipStream_t, const VT *, VT *);                                            \
    template void launch_tile_group<VT>(const KpmPlan &, bool, int, unsigned, hipStream_t, const TileArgs<VT> &);           \
    template void tile_start_planes<VT>(const tbk_ham *, const KpmPlan &, const TileRun &, const VT *, int32_t,        \
                                        char *, VT *, double *, hipStream_t);
TBK_TILE_INST(float)
TBK_TILE_INST(double)
#undef TBK_TILE_INST

}  // namespace tbk
