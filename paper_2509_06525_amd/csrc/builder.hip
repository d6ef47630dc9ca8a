// Neighbour list and Hamiltonian assembly on the GPU (Eq. (1)).
//
// Build sequence for n_seg stacked structures (one structure = one segment):
//   1. k_segment_scan: per-segment coordinate range, NaN/Inf and species checks
//   2. cell list: cell id per atom (per-segment grids, global ids), counts,
//      exclusive scan, scatter, per-cell sort by atom index
//   3. k_degree: neighbours within r_cut per row, the first few of them kept for 5.
//   4. slice widths (max degree per slice) -> slice offsets (exclusive scan)
//   5. k_fill: columns and FP64 hoppings of each row, padding, in-row sort by
//      column, onsite, per-segment row Gershgorin bounds
// CSR is handled as SELL with slice height 1.  Rows of segment s occupy the
// segment's atom range, so stacked systems keep their own row blocks.
#include <hipcub/hipcub.hpp>

#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "builder.hpp"
#include "nlist.hpp"

namespace tbk {

namespace {

constexpr int kMaxDegree = 256;
constexpr int kMaxSpecies = 16;
constexpr int kCellStrip = 64;      // cells per strip of the row order

// seg_of[i] = s with seg_atoms[s] <= i < seg_atoms[s + 1] (offsets strictly
// increasing, so the binary search has one answer).
__global__ void k_seg_of(int64_t n, int32_t nseg, const int64_t *__restrict__ seg_atoms,
                         int32_t *__restrict__ seg_of) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t lo = 0, hi = nseg;
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (seg_atoms[mid] <= i) lo = mid;
        else hi = mid;
    }
    seg_of[i] = lo;
}

// Atoms per thread of k_segment_scan and rows per thread of k_fill, such that no more
// than `blocks` blocks end in atomics on the same few words: those come one every 60 ns
// or so (1 M atoms, k_segment_scan: 273 us with a block per 256 atoms, 50 with 512 blocks).
int rows_per_thread(int64_t n, int blocks) {
    return (int)std::max<int64_t>(1, ceil_div(n, (int64_t)kBlock * blocks));
}

// Per-segment coordinate ranges and input checks over the whole grid.
// keys[(k n_seg + s) 2 + {0, 1}] = order-preserving keys of min / max of
// coordinate k over the finite coordinates of segment s (k_init_bounds start);
// flags[2 s] = 1 if some coordinate of s is NaN/Inf, flags[2 s + 1] = 1 if a
// species index is outside [0, n_species) (flags start at 0).  A block covers
// chunk * kBlock consecutive atoms; a thread flushes its running range
// with atomics when its atoms cross into another segment, and the block folds
// the last ranges per segment before one atomic per segment and coordinate.
__global__ __launch_bounds__(kBlock) void k_segment_scan(const double *__restrict__ pos,
                                                         const int32_t *__restrict__ species, int64_t n,
                                                         const int32_t *__restrict__ seg_of, int32_t nseg,
                                                         int32_t n_species, int chunk, int64_t *__restrict__ keys,
                                                         int32_t *__restrict__ flags) {
    const int64_t base = (int64_t)blockIdx.x * kBlock * chunk;
    double mn[3], mx[3];
    int32_t cur = -1;
    auto reset = [&]() {
        for (int k = 0; k < 3; ++k) { mn[k] = INFINITY; mx[k] = -INFINITY; }
    };
    reset();
    for (int u = 0; u < chunk; ++u) {
        const int64_t i = base + (int64_t)u * kBlock + threadIdx.x;
        if (i >= n) break;
        const int32_t sg = seg_of[i];
        if (sg != cur) {
            if (cur >= 0) {
                for (int k = 0; k < 3; ++k)
                    if (mn[k] <= mx[k]) {
                        atomicMin((long long *)&keys[2 * ((int64_t)k * nseg + cur)], (long long)dkey(mn[k]));
                        atomicMax((long long *)&keys[2 * ((int64_t)k * nseg + cur) + 1], (long long)dkey(mx[k]));
                    }
            }
            cur = sg;
            reset();
        }
        for (int k = 0; k < 3; ++k) {
            const double x = pos[3 * i + k];
            if (!isfinite(x)) flags[2 * sg] = 1;
            else { mn[k] = fmin(mn[k], x); mx[k] = fmax(mx[k], x); }
        }
        if (species) {
            const int32_t t = species[i];
            if (t < 0 || t >= n_species) flags[2 * sg + 1] = 1;
        }
    }
    for (int k = 0; k < 3; ++k) block_segment_bounds(mn[k], mx[k], cur < 0 ? -1 : k * nseg + cur, keys);
}

__global__ void k_cell_of(const double *__restrict__ pos, int64_t n, const CellGrid *__restrict__ grids,
                          const int32_t *__restrict__ seg_of, int32_t *__restrict__ cell,
                          int32_t *__restrict__ slot, int32_t *__restrict__ count) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const CellGrid g = grids[seg_of[i]];
    int32_t cx = cell_coord(pos[3 * i], g, 0);
    int32_t cy = cell_coord(pos[3 * i + 1], g, 1);
    int32_t cz = cell_coord(pos[3 * i + 2], g, 2);
    int32_t c = (int32_t)(g.cell_off + cell_id(g, cx, cy, cz));
    cell[i] = c;
    slot[i] = atomicAdd(&count[c], 1);
}

__global__ void k_scatter(int64_t n, const int32_t *__restrict__ cell, const int32_t *__restrict__ slot,
                          const int32_t *__restrict__ start, int32_t *__restrict__ sorted) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    sorted[start[cell[i]] + slot[i]] = (int32_t)i;
}

// Ascending atom order inside each cell (the scatter order depends on atomics).
__global__ void k_sort_cells(int64_t ncell, const int32_t *__restrict__ start, int32_t *__restrict__ sorted) {
    int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c >= ncell) return;
    int32_t s0 = start[c], s1 = start[c + 1];
    for (int32_t a = s0 + 1; a < s1; ++a) {
        int32_t v = sorted[a];
        int32_t b = a - 1;
        while (b >= s0 && sorted[b] > v) { sorted[b + 1] = sorted[b]; --b; }
        sorted[b + 1] = v;
    }
}

__global__ void k_perm(int64_t n, int32_t reorder, const int32_t *__restrict__ sorted,
                       int32_t *__restrict__ perm, int32_t *__restrict__ iperm) {
    int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (r >= n) return;
    int32_t a = reorder ? sorted[r] : (int32_t)r;
    perm[r] = a;
    iperm[a] = (int32_t)r;
}

// Neighbours within r_cut per row, and (nbr != NULL) the first kShortRow of them for
// k_fill.
constexpr int kShortRow = 6;

__global__ void k_degree(CellList cl, const double *__restrict__ pos, int64_t n, double r_cut,
                         const int32_t *__restrict__ perm, int32_t *__restrict__ deg, int32_t *__restrict__ nbr) {
    int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (r >= n) return;
    int32_t cnt = 0;
    for_each_pair(cl, pos, perm[r], r_cut, [&](int32_t j, double, double, double, double) {
        if (nbr && cnt < kShortRow) nbr[cnt * n + r] = j;
        ++cnt;
    });
    deg[r] = cnt;
}

// Width of each slice (largest degree among its rows) and its stored entries.  A
// slice goes to min(slice, 64) lanes side by side: one thread per slice of 256 rows
// read each row from a line of its own (100 M rows: 1.3 ms, 0.15 ms so).
__global__ __launch_bounds__(kBlock) void k_slice_width(int64_t n, int32_t slice, int64_t n_slices,
                                                        const int32_t *__restrict__ deg,
                                                        int64_t *__restrict__ entries) {
    const int32_t lanes = slice < 64 ? slice : 64;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t s = t / lanes;
    const int32_t lane = (int32_t)(t - s * lanes);
    int32_t w = 0;
    const int64_t r1 = (s + 1) * slice < n ? (s + 1) * slice : n;
    for (int64_t r = s * slice + lane; r < r1; r += lanes) w = max(w, deg[r]);
    for (int d = lanes >> 1; d > 0; d >>= 1) w = max(w, __shfl_xor(w, d));
    if (lane == 0 && s <= n_slices) entries[s] = (int64_t)w * slice;      // 0 past the last
}

// n empty bounds, and `zeros` words of 0 after them.
__global__ void k_init_bounds(int32_t n, int64_t *__restrict__ keys, int32_t zeros) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < n) {
        keys[2 * s] = dkey(INFINITY);
        keys[2 * s + 1] = dkey(-INFINITY);
    }
    if (s < zeros) keys[2 * n + s] = 0;
}

// totals[0] = largest degree, totals[1] = sum of the degrees (both start at 0),
// totals[2] = stored entries.
__global__ __launch_bounds__(kBlock) void k_totals(const int32_t *__restrict__ deg, int64_t n,
                                                   const int64_t *__restrict__ ptr, int64_t n_slices,
                                                   int64_t *__restrict__ totals) {
    int32_t mx = 0;
    int64_t sum = 0;
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
        mx = max(mx, deg[i]);
        sum += deg[i];
    }
    for (int d = 32; d > 0; d >>= 1) {
        mx = max(mx, __shfl_xor(mx, d));
        sum += __shfl_xor(sum, d);
    }
    __shared__ int32_t wmx[kBlock / 64];
    __shared__ int64_t wsum[kBlock / 64];
    if ((threadIdx.x & 63) == 0) {
        wmx[threadIdx.x >> 6] = mx;
        wsum[threadIdx.x >> 6] = sum;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kBlock / 64; ++w) {
        mx = max(mx, wmx[w]);
        sum += wsum[w];
    }
    atomicMax((long long *)&totals[0], (long long)mx);
    atomicAdd((unsigned long long *)&totals[1], (unsigned long long)sum);
    if (blockIdx.x == 0) totals[2] = ptr[n_slices];
}

struct SpeciesTable {
    double onsite[kMaxSpecies];
    double t_pair[kMaxSpecies * kMaxSpecies];
};

// Columns, hoppings, onsite energies and Gershgorin bounds of the rows.  SHORT (no row
// of more than kShortRow entries): the neighbours are those k_degree found, in its
// order, and a row is sorted in registers and written once; otherwise the search runs
// again and rows are sorted in place.  The search beside exp and the rest takes 160
// registers, and waves per SIMD with them (100 M atoms: 19.5 ms with the search, 5.3
// without).  A block takes `rows` rows per thread (one where there are several segments).
template <class V, bool SHORT>
__global__ __launch_bounds__(kBlock) void k_fill(
    CellList cl, const double *__restrict__ pos, const int32_t *__restrict__ species, int64_t n, int32_t slice,
    double r_cut, double r0, double beta, int32_t n_species, const SpeciesTable *__restrict__ tab,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ iperm, const int64_t *__restrict__ ptr,
    int32_t *__restrict__ col, V *__restrict__ val, V *__restrict__ onsite, int64_t *__restrict__ bound_keys,
    int64_t *__restrict__ val_keys, int16_t *__restrict__ col16, const int32_t *__restrict__ deg,
    const int32_t *__restrict__ nbr, int rows) {
    double lo = INFINITY, hi = -INFINITY;
    double vlo = INFINITY, vhi = -INFINITY;   // range of the stored hoppings
    int32_t sg = -1;
    for (int it = 0; it < rows; ++it) {
        const int64_t r = ((int64_t)blockIdx.x * rows + it) * kBlock + threadIdx.x;
        if (r >= n) break;
        const int64_t s = r / slice, lane = r - s * slice;
        const int64_t base = ptr[s] + lane;
        const int32_t w = (int32_t)((ptr[s + 1] - ptr[s]) / slice);
        const int32_t i = perm[r];
        const int32_t si = species[i];
        sg = cl.seg_of[i];
        auto hopping = [&](int32_t j, double rij) {
            return tab->t_pair[si * n_species + species[j]] * exp(-beta * (rij / r0 - 1.0));
        };
        auto put = [&](int32_t q, int32_t c, V v) {
            col[base + (int64_t)q * slice] = c;
            val[base + (int64_t)q * slice] = v;
            if (col16) {    // 16-bit column offsets (escape -32768: read col)
                const int64_t d = (int64_t)c - r;
                col16[base + (int64_t)q * slice] = (d >= -32767 && d <= 32767) ? (int16_t)d : (int16_t)-32768;
            }
        };
        int32_t k = 0;
        double asum = 0.0;
        if constexpr (SHORT) {
            const CellGrid &g = cl.grids[sg];
            const double xi = pos[3 * (int64_t)i], yi = pos[3 * (int64_t)i + 1], zi = pos[3 * (int64_t)i + 2];
            k = deg[r];
            int32_t c[kShortRow];
            V v[kShortRow];
#pragma unroll
            for (int q = 0; q < kShortRow; ++q) {
                c[q] = INT32_MAX;
                v[q] = (V)0;
                if (q >= k) continue;
                const int32_t j = nbr[q * n + r];
                double dx, dy, dz;
                const double r2 = pair_r2(g, pos[3 * (int64_t)j] - xi, pos[3 * (int64_t)j + 1] - yi,
                                          pos[3 * (int64_t)j + 2] - zi, dx, dy, dz);
                const double t = hopping(j, sqrt(r2));
                c[q] = iperm[j];
                v[q] = (V)t;
                vlo = fmin(vlo, (double)(V)t);
                vhi = fmax(vhi, (double)(V)t);
                asum += fabs(t);
            }
            // ascending columns; the places without an entry stay last
#pragma unroll
            for (int e = 1; e < kShortRow; ++e)
#pragma unroll
                for (int q = e; q > 0; --q)
                    if (c[q - 1] > c[q]) {
                        const int32_t tc = c[q - 1];
                        const V tv = v[q - 1];
                        c[q - 1] = c[q];
                        v[q - 1] = v[q];
                        c[q] = tc;
                        v[q] = tv;
                    }
#pragma unroll
            for (int q = 0; q < kShortRow; ++q)
                if (q < w) put(q, q < k ? c[q] : (int32_t)r, v[q]);
            for (int32_t q = kShortRow; q < w; ++q) put(q, (int32_t)r, (V)0);
        } else {
            for_each_neighbor(cl, pos, i, r_cut, [&](int32_t j, double rij, double, double, double) {
                const double t = hopping(j, rij);
                if (k < w) {
                    col[base + (int64_t)k * slice] = iperm[j];
                    val[base + (int64_t)k * slice] = (V)t;
                }
                vlo = fmin(vlo, (double)(V)t);
                vhi = fmax(vhi, (double)(V)t);
                asum += fabs(t);
                ++k;
            });
            // Insertion sort of the row's real entries by column.
            const int32_t kk = k < w ? k : w;
            for (int32_t a = 1; a < kk; ++a) {
                const int32_t ca = col[base + (int64_t)a * slice];
                const V va = val[base + (int64_t)a * slice];
                int32_t b = a - 1;
                while (b >= 0 && col[base + (int64_t)b * slice] > ca) {
                    col[base + (int64_t)(b + 1) * slice] = col[base + (int64_t)b * slice];
                    val[base + (int64_t)(b + 1) * slice] = val[base + (int64_t)b * slice];
                    --b;
                }
                col[base + (int64_t)(b + 1) * slice] = ca;
                val[base + (int64_t)(b + 1) * slice] = va;
            }
            for (int32_t q = 0; q < w; ++q)
                put(q, q < kk ? col[base + (int64_t)q * slice] : (int32_t)r,
                    q < kk ? val[base + (int64_t)q * slice] : (V)0);
        }
        const double eps = tab->onsite[si];
        onsite[r] = (V)eps;
        lo = fmin(lo, eps - asum);
        hi = fmax(hi, eps + asum);
    }
    block_segment_bounds(lo, hi, sg, bound_keys);
    block_segment_bounds(vlo, vhi, vlo <= vhi ? 0 : -1, val_keys);
}

template <class T>
tbk_status exclusive_scan(const T *in, T *out, int64_t n, Arena &arena, hipStream_t s) {
    size_t tmp = 0;
    TBK_HIP(hipcub::DeviceScan::ExclusiveSum(nullptr, tmp, in, out, (int)n, s));
    DevBuf t;
    TBK_HIP(t.alloc(tmp, arena));
    TBK_HIP(hipcub::DeviceScan::ExclusiveSum(t.as<void>(), tmp, in, out, (int)n, s));
    return TBK_OK;
}

int32_t any_onsite(const tbk_tb_params *p) {
    for (int i = 0; i < p->n_species; ++i)
        if (p->onsite[i] != 0.0) return 1;
    return 0;
}

}  // namespace

tbk_status check_tb_params(const tbk_tb_params *p) {
    TBK_CHECK(p != nullptr, TBK_ERR_INVALID_ARG, "params is NULL");
    TBK_CHECK(std::isfinite(p->r_cut) && std::isfinite(p->r0) && std::isfinite(p->beta), TBK_ERR_NOT_FINITE,
              "r_cut, r0 or beta is not finite");
    TBK_CHECK(p->r_cut > 0 && p->r0 > 0 && p->beta >= 0, TBK_ERR_INVALID_ARG,
              "r_cut and r0 must be positive and beta non-negative");
    TBK_CHECK(p->n_species >= 1 && p->n_species <= kMaxSpecies, TBK_ERR_INVALID_ARG,
              "n_species must be in [1, %d]", kMaxSpecies);
    TBK_CHECK(p->onsite && p->t_pair, TBK_ERR_INVALID_ARG, "onsite/t_pair is NULL");
    for (int i = 0; i < p->n_species; ++i) {
        TBK_CHECK(std::isfinite(p->onsite[i]), TBK_ERR_NOT_FINITE, "onsite[%d] is not finite", i);
        for (int j = 0; j < p->n_species; ++j) {
            TBK_CHECK(std::isfinite(p->t_pair[i * p->n_species + j]), TBK_ERR_NOT_FINITE,
                      "t_pair[%d][%d] is not finite", i, j);
            TBK_CHECK(p->t_pair[i * p->n_species + j] == p->t_pair[j * p->n_species + i],
                      TBK_ERR_INVALID_ARG, "t_pair is not symmetric");
        }
    }
    return TBK_OK;
}

void decode_bounds(const std::vector<int64_t> &keys, int nseg, double *bounds) {
    for (int g = 0; g < nseg; ++g) {
        bounds[2 * g] = dunkey(keys[2 * g]);
        bounds[2 * g + 1] = dunkey(keys[2 * g + 1]);
    }
}

tbk_status init_bound_keys(DevBuf &keys, int n, Arena &arena, hipStream_t s) {
    TBK_HIP(keys.alloc(sizeof(int64_t) * 2 * n, arena));
    k_init_bounds<<<(n + 255) / 256, 256, 0, s>>>(n, keys.as<int64_t>(), 0);
    TBK_HIP(hipGetLastError());
    return TBK_OK;
}

tbk_status CellListOwner::build(const double *pos, const int32_t *species, int32_t n_species, int64_t n,
                                int32_t nseg, const int64_t *seg_atoms_h, const double *boxes,
                                const int32_t periodic[3], double r_cut, Arena &arena, hipStream_t s) {
    TBK_CHECK(pos && boxes && periodic && seg_atoms_h, TBK_ERR_INVALID_ARG, "NULL position/box/periodic/segments");
    TBK_CHECK(n >= 1 && n < (int64_t)INT32_MAX, TBK_ERR_INVALID_ARG, "n = %lld out of [1, 2^31-1)", (long long)n);
    TBK_CHECK(nseg >= 1 && nseg <= (1 << 20), TBK_ERR_INVALID_ARG, "n_seg = %d out of [1, 2^20]", nseg);
    TBK_CHECK(seg_atoms_h[0] == 0 && seg_atoms_h[nseg] == n, TBK_ERR_INVALID_ARG,
              "segment offsets must start at 0 and end at n");
    for (int g = 0; g < nseg; ++g)
        TBK_CHECK(seg_atoms_h[g + 1] > seg_atoms_h[g], TBK_ERR_INVALID_ARG, "segment %d is empty or unordered", g);
    for (int k = 0; k < 3; ++k)
        TBK_CHECK(periodic[k] == 0 || periodic[k] == 1, TBK_ERR_INVALID_ARG, "periodic[%d] must be 0 or 1", k);
    for (int g = 0; g < nseg; ++g)
        for (int k = 0; k < 3; ++k)
            if (periodic[k]) {
                const double L = boxes[3 * g + k];
                TBK_CHECK(std::isfinite(L), TBK_ERR_NOT_FINITE, "box[%d] of segment %d is not finite", k, g);
                TBK_CHECK(L >= 2.0 * r_cut, TBK_ERR_INVALID_ARG,
                          "periodic length %g (axis %d, segment %d) is below 2 r_cut = %g", L, k, g, 2.0 * r_cut);
            }
    n_seg = nseg;
    TBK_HIP(seg_atoms.alloc(sizeof(int64_t) * (nseg + 1), arena));
    TBK_HIP(seg_of.alloc(sizeof(int32_t) * n, arena));
    TBK_HIP(hipMemcpyAsync(seg_atoms.as<int64_t>(), seg_atoms_h, sizeof(int64_t) * (nseg + 1),
                           hipMemcpyHostToDevice, s));
    const int gseg = (int)ceil_div(n, kBlock);
    k_seg_of<<<gseg, kBlock, 0, s>>>(n, nseg, seg_atoms.as<int64_t>(), seg_of.as<int32_t>());
    TBK_HIP(hipGetLastError());

    // 1. ranges and validity per segment
    DevBuf rkeys;           // 6 nseg keys, then 2 nseg 32-bit flags
    TBK_HIP(rkeys.alloc(sizeof(int64_t) * 7 * nseg, arena));
    int32_t *rflags = reinterpret_cast<int32_t *>(rkeys.as<int64_t>() + 6 * (size_t)nseg);
    k_init_bounds<<<(3 * nseg + 255) / 256, 256, 0, s>>>(3 * nseg, rkeys.as<int64_t>(), nseg);
    TBK_HIP(hipGetLastError());
    const int chunk = nseg == 1 ? rows_per_thread(n, n < (1 << 22) ? 512 : 2048) : 1;
    k_segment_scan<<<(unsigned)ceil_div(n, (int64_t)kBlock * chunk), kBlock, 0, s>>>(
        pos, species, n, seg_of.as<int32_t>(), nseg, n_species, chunk, rkeys.as<int64_t>(), rflags);
    TBK_HIP(hipGetLastError());
    std::vector<int64_t> hk(7 * (size_t)nseg);
    TBK_HIP(hipMemcpyAsync(hk.data(), rkeys.as<int64_t>(), sizeof(int64_t) * 7 * nseg, hipMemcpyDeviceToHost, s));
    TBK_HIP(hipStreamSynchronize(s));
    std::vector<int32_t> hf(2 * (size_t)nseg);
    std::memcpy(hf.data(), hk.data() + 6 * (size_t)nseg, sizeof(int32_t) * 2 * nseg);
    // hp[8 g + k] = min, hp[8 g + 3 + k] = max of coordinate k in segment g
    std::vector<double> hp(8 * (size_t)nseg);
    for (int g = 0; g < nseg; ++g) {
        TBK_CHECK(hf[2 * g] == 0, TBK_ERR_NOT_FINITE, "a coordinate of segment %d is NaN or Inf", g);
        TBK_CHECK(hf[2 * g + 1] == 0, TBK_ERR_INVALID_ARG, "a species index of segment %d is outside [0, %d)",
                  g, n_species);
        for (int k = 0; k < 3; ++k) {
            hp[8 * g + k] = dunkey(hk[2 * ((size_t)k * nseg + g)]);
            hp[8 * g + 3 + k] = dunkey(hk[2 * ((size_t)k * nseg + g) + 1]);
        }
    }

    // 2. one cell grid per segment, global cell ids
    std::vector<CellGrid> hg(nseg);
    int64_t off = 0;
    for (int g = 0; g < nseg; ++g) {
        CellGrid &c = hg[g];
        const int64_t na = seg_atoms_h[g + 1] - seg_atoms_h[g];
        int64_t ncell = 1;
        for (int k = 0; k < 3; ++k) {
            c.periodic[k] = periodic[k];
            c.box[k] = periodic[k] ? boxes[3 * g + k] : 0.0;
            if (periodic[k]) { c.lo[k] = 0.0; c.len[k] = boxes[3 * g + k]; }
            else { c.lo[k] = hp[8 * g + k]; c.len[k] = std::max(hp[8 * g + 3 + k] - hp[8 * g + k], 0.0) + 1e-9; }
            double ncd = std::floor(c.len[k] / r_cut);
            ncd = std::max(1.0, std::min(ncd, 1.0e6));
            c.nc[k] = (int32_t)ncd;
            ncell *= c.nc[k];
        }
        // Cap the cell count near the atom count (cells stay >= r_cut wide).
        while (ncell > 4 * na + 64) {
            int k = (c.nc[0] >= c.nc[1] && c.nc[0] >= c.nc[2]) ? 0 : (c.nc[1] >= c.nc[2] ? 1 : 2);
            ncell /= c.nc[k];
            c.nc[k] = std::max(1, c.nc[k] / 2);
            ncell *= c.nc[k];
        }
        c.strip = std::min<int32_t>(c.nc[0], kCellStrip);
        c.nstrip = (c.nc[0] + c.strip - 1) / c.strip;
        c.ncell = (int64_t)c.nc[2] * c.nstrip * c.nc[1] * c.strip;
        c.cell_off = off;
        off += c.ncell;
        TBK_CHECK(off < (int64_t)INT32_MAX, TBK_ERR_UNSUPPORTED, "too many cells");
    }
    const int64_t ncell = off;
    TBK_HIP(grids.alloc(sizeof(CellGrid) * nseg, arena));
    TBK_HIP(hipMemcpyAsync(grids.as<CellGrid>(), hg.data(), sizeof(CellGrid) * nseg, hipMemcpyHostToDevice, s));

    DevBuf cell, slot, count;
    TBK_HIP(cell.alloc(sizeof(int32_t) * n, arena));
    TBK_HIP(slot.alloc(sizeof(int32_t) * n, arena));
    TBK_HIP(count.alloc(sizeof(int32_t) * (ncell + 1), arena));
    TBK_HIP(cell_start.alloc(sizeof(int32_t) * (ncell + 1), arena));
    TBK_HIP(sorted.alloc(sizeof(int32_t) * n, arena));
    TBK_HIP(hipMemsetAsync(count.as<int32_t>(), 0, sizeof(int32_t) * (ncell + 1), s));
    const int gn = (int)ceil_div(n, kBlock);
    k_cell_of<<<gn, kBlock, 0, s>>>(pos, n, grids.as<CellGrid>(), seg_of.as<int32_t>(), cell.as<int32_t>(),
                                    slot.as<int32_t>(), count.as<int32_t>());
    TBK_HIP(hipGetLastError());
    tbk_status st = exclusive_scan(count.as<int32_t>(), cell_start.as<int32_t>(), ncell + 1, arena, s);
    if (st != TBK_OK) return st;
    k_scatter<<<gn, kBlock, 0, s>>>(n, cell.as<int32_t>(), slot.as<int32_t>(), cell_start.as<int32_t>(),
                                    sorted.as<int32_t>());
    TBK_HIP(hipGetLastError());
    k_sort_cells<<<(int)ceil_div(ncell, kBlock), kBlock, 0, s>>>(ncell, cell_start.as<int32_t>(), sorted.as<int32_t>());
    TBK_HIP(hipGetLastError());
    view.grids = grids.as<CellGrid>();
    view.seg_of = seg_of.as<int32_t>();
    view.cell_start = cell_start.as<int32_t>();
    view.sorted = sorted.as<int32_t>();
    return TBK_OK;
}

tbk_status HamPlan::run(const double *pos, const int32_t *species, int64_t n, int32_t nseg, const int64_t *seg_atoms,
                        const double *boxes, const int32_t periodic[3], const tbk_tb_params *p, int32_t fmt,
                        int32_t slice_in, hipStream_t s, bool keep_nbr, size_t extra) {
    tbk_status st = check_tb_params(p);
    if (st != TBK_OK) return st;
    TBK_CHECK(species != nullptr, TBK_ERR_INVALID_ARG, "species is NULL");
    TBK_CHECK(fmt == TBK_CSR_F64 || fmt == TBK_SELL_F64 || fmt == TBK_SELL_F32, TBK_ERR_INVALID_ARG,
              "unknown format %d", fmt);
    TBK_CHECK(p->reorder == 0 || p->reorder == 1, TBK_ERR_INVALID_ARG, "reorder must be 0 or 1");
    if (fmt == TBK_CSR_F64) slice = 1;
    else {
        TBK_CHECK(slice_in >= 1 && slice_in <= 1024 && (slice_in & (slice_in - 1)) == 0, TBK_ERR_INVALID_ARG,
                  "slice = %d is not a power of two in [1, 1024]", slice_in);
        slice = slice_in;
    }
    const size_t per_atom = kCellBytes + sizeof(int32_t) * (3 + (keep_nbr ? kShortRow : 0)) + extra;
    arena.expect(per_atom * n + 2 * sizeof(int64_t) * (n / slice + 2) +
                     (sizeof(CellGrid) + 16 * sizeof(int64_t)) * nseg + 65536, s);
    st = cells.build(pos, species, p->n_species, n, nseg, seg_atoms, boxes, periodic, p->r_cut, arena, s);
    if (st != TBK_OK) return st;
    const int gn = (int)ceil_div(n, kBlock);
    TBK_HIP(perm.alloc(sizeof(int32_t) * n, arena));
    TBK_HIP(iperm.alloc(sizeof(int32_t) * n, arena));
    TBK_HIP(deg.alloc(sizeof(int32_t) * n, arena));
    k_perm<<<gn, kBlock, 0, s>>>(n, p->reorder, cells.view.sorted, perm.as<int32_t>(), iperm.as<int32_t>());
    TBK_HIP(hipGetLastError());
    if (keep_nbr) TBK_HIP(nbr.alloc(sizeof(int32_t) * kShortRow * n, arena));
    k_degree<<<gn, kBlock, 0, s>>>(cells.view, pos, n, p->r_cut, perm.as<int32_t>(), deg.as<int32_t>(),
                                   nbr.as<int32_t>());
    TBK_HIP(hipGetLastError());
    n_slices = ceil_div(n, slice);
    DevBuf entries;
    TBK_HIP(entries.alloc(sizeof(int64_t) * (n_slices + 1), arena));
    TBK_HIP(ptr.alloc(sizeof(int64_t) * (n_slices + 1), arena));
    k_slice_width<<<(unsigned)ceil_div((n_slices + 1) * std::min<int64_t>(slice, 64), kBlock), kBlock, 0, s>>>(
        n, slice, n_slices, deg.as<int32_t>(), entries.as<int64_t>());
    TBK_HIP(hipGetLastError());
    st = exclusive_scan(entries.as<int64_t>(), ptr.as<int64_t>(), n_slices + 1, arena, s);
    if (st != TBK_OK) return st;
    DevBuf totals;
    TBK_HIP(totals.alloc(sizeof(int64_t) * 3, arena));
    k_init_bounds<<<1, 64, 0, s>>>(0, totals.as<int64_t>(), 3);
    k_totals<<<(unsigned)std::min<int64_t>(256, ceil_div(n, 4 * kBlock)), kBlock, 0, s>>>(
        deg.as<int32_t>(), n, ptr.as<int64_t>(), n_slices, totals.as<int64_t>());
    TBK_HIP(hipGetLastError());
    int64_t host[3] = {0, 0, 0};
    TBK_HIP(hipMemcpyAsync(host, totals.as<int64_t>(), sizeof host, hipMemcpyDeviceToHost, s));
    TBK_HIP(hipStreamSynchronize(s));
    max_degree = (int32_t)host[0];
    n_bonds = host[1] / 2;
    n_entries = host[2];
    TBK_CHECK(max_degree <= kMaxDegree, TBK_ERR_UNSUPPORTED, "max degree %d exceeds %d", max_degree, kMaxDegree);
    TBK_CHECK(n_entries < (int64_t)1 << 40, TBK_ERR_UNSUPPORTED, "too many entries");
    return TBK_OK;
}

tbk_status HamPlan::check_buffers(int64_t n, const tbk_ham *h) const {
    TBK_CHECK(h->n_rows >= n && h->n_ptr >= n_slices + 1 && h->n_entries >= n_entries,
              TBK_ERR_BUFFER_TOO_SMALL, "Hamiltonian buffers sized for n_rows=%lld n_ptr=%lld n_entries=%lld; "
              "need %lld, %lld, %lld", (long long)h->n_rows, (long long)h->n_ptr, (long long)h->n_entries,
              (long long)n, (long long)(n_slices + 1), (long long)n_entries);
    TBK_CHECK(h->ptr && h->col && h->val && h->onsite && h->perm, TBK_ERR_INVALID_ARG,
              "a Hamiltonian array pointer is NULL");
    return TBK_OK;
}

void HamPlan::set_sizes(int64_t n, const tbk_tb_params *p, tbk_ham *h) const {
    h->n_rows = n;
    h->n_ptr = n_slices + 1;
    h->n_entries = n_entries;
    h->n_bonds = n_bonds;
    h->max_degree = max_degree;
    h->has_onsite = any_onsite(p);
    h->n_seg = cells.n_seg;
    h->n_orb = 1;
    if (h->fmt == TBK_CSR_F64) h->slice = 1;
}

tbk_status HamPlan::fill(const double *pos, const int32_t *species, int64_t n, const tbk_tb_params *p, tbk_ham *h,
                         double *bounds, hipStream_t s) {
    tbk_status st = check_buffers(n, h);
    if (st != TBK_OK) return st;
    const int nseg = cells.n_seg;
    SpeciesTable tab{};
    for (int i = 0; i < p->n_species; ++i) {
        tab.onsite[i] = p->onsite[i];
        for (int j = 0; j < p->n_species; ++j) tab.t_pair[i * p->n_species + j] = p->t_pair[i * p->n_species + j];
    }
    DevBuf dtab, keys;
    TBK_HIP(dtab.alloc(sizeof(SpeciesTable), arena));
    TBK_HIP(hipMemcpyAsync(dtab.as<void>(), &tab, sizeof(SpeciesTable), hipMemcpyHostToDevice, s));
    st = init_bound_keys(keys, nseg + 1, arena, s);       // the last: range of the stored hoppings
    if (st != TBK_OK) return st;
    const int rows = nseg == 1 ? rows_per_thread(n, 4096) : 1;
    const int gn = (int)ceil_div(n, (int64_t)kBlock * rows);
    TBK_HIP(hipMemcpyAsync(h->ptr, ptr.as<int64_t>(), sizeof(int64_t) * (n_slices + 1), hipMemcpyDeviceToDevice, s));
    TBK_HIP(hipMemcpyAsync(h->perm, perm.as<int32_t>(), sizeof(int32_t) * n, hipMemcpyDeviceToDevice, s));
    auto launch = [&](auto v, auto is_short) {
        typedef decltype(v) V;
        k_fill<V, decltype(is_short)::value><<<gn, kBlock, 0, s>>>(
            cells.view, pos, species, n, slice, p->r_cut, p->r0, p->beta, p->n_species, dtab.as<SpeciesTable>(),
            perm.as<int32_t>(), iperm.as<int32_t>(), h->ptr, h->col, static_cast<V *>(h->val),
            static_cast<V *>(h->onsite), keys.as<int64_t>(), keys.as<int64_t>() + 2 * nseg, h->col16, deg.as<int32_t>(),
            nbr.as<int32_t>(), rows);
    };
    const bool is_short = max_degree <= kShortRow;
    if (h->fmt == TBK_SELL_F32) is_short ? launch(0.0f, std::true_type{}) : launch(0.0f, std::false_type{});
    else is_short ? launch(0.0, std::true_type{}) : launch(0.0, std::false_type{});
    TBK_HIP(hipGetLastError());
    return finish(keys, true, n, p, h, bounds, s);
}

tbk_status HamPlan::finish(DevBuf &keys, bool with_values, int64_t n, const tbk_tb_params *p, tbk_ham *h,
                           double *bounds, hipStream_t s) {
    const int nseg = cells.n_seg;
    std::vector<int64_t> hk(2 * (size_t)(nseg + (with_values ? 1 : 0)));
    TBK_HIP(hipMemcpyAsync(hk.data(), keys.as<int64_t>(), sizeof(int64_t) * hk.size(), hipMemcpyDeviceToHost, s));
    if (h->seg_rows)
        TBK_HIP(hipMemcpyAsync(h->seg_rows, cells.seg_atoms.as<int64_t>(), sizeof(int64_t) * (nseg + 1),
                               hipMemcpyDeviceToDevice, s));
    TBK_HIP(hipStreamSynchronize(s));
    decode_bounds(hk, nseg, bounds);
    set_sizes(n, p, h);
    // uniform hoppings: every stored value (as stored) equal, at least one entry
    h->uniform_hop = 0;
    h->hop_value = 0.0;
    const int64_t *vk = hk.data() + 2 * (size_t)nseg;
    if (with_values && vk[0] == vk[1] && dunkey(vk[0]) <= dunkey(vk[1])) {
        h->uniform_hop = 1;
        h->hop_value = dunkey(vk[0]);
    }
    return TBK_OK;
}

}  // namespace tbk

using namespace tbk;

namespace {

tbk_status size_common(const double *pos, const int32_t *species, int64_t n, int32_t nseg, const int64_t *seg_atoms,
                       const double *boxes, const int32_t periodic[3], const tbk_tb_params *p, tbk_ham *h,
                       void *stream) {
    TBK_CHECK(h != nullptr, TBK_ERR_INVALID_ARG, "h is NULL");
    hipStream_t s = as_stream(stream);
    HamPlan plan;
    tbk_status st = plan.run(pos, species, n, nseg, seg_atoms, boxes, periodic, p, h->fmt, h->slice, s);
    if (st != TBK_OK) return st;
    plan.set_sizes(n, p, h);
    return TBK_OK;
}

tbk_status build_common(const double *pos, const int32_t *species, int64_t n, int32_t nseg, const int64_t *seg_atoms,
                        const double *boxes, const int32_t periodic[3], const tbk_tb_params *p, tbk_ham *h,
                        double *bounds, void *stream) {
    TBK_CHECK(h != nullptr && bounds != nullptr, TBK_ERR_INVALID_ARG, "h or bounds is NULL");
    hipStream_t s = as_stream(stream);
    HamPlan plan;
    tbk_status st = plan.run(pos, species, n, nseg, seg_atoms, boxes, periodic, p, h->fmt, h->slice, s, true);
    if (st != TBK_OK) return st;
    return plan.fill(pos, species, n, p, h, bounds, s);
}

}  // namespace

extern "C" tbk_status tbk_hamiltonian_size(const double *pos, const int32_t *species, int64_t n,
                                           const double box[3], const int32_t periodic[3],
                                           const tbk_tb_params *p, tbk_ham *h, void *stream) {
    clear_error();
    TBK_CHECK(box != nullptr, TBK_ERR_INVALID_ARG, "box is NULL");
    const int64_t seg[2] = {0, n};
    return size_common(pos, species, n, 1, seg, box, periodic, p, h, stream);
}

extern "C" tbk_status tb_build_hamiltonian(const double *pos, const int32_t *species, int64_t n,
                                           const double box[3], const int32_t periodic[3],
                                           const tbk_tb_params *p, tbk_ham *h, double spec_bounds[2],
                                           void *stream) {
    clear_error();
    TBK_CHECK(box != nullptr, TBK_ERR_INVALID_ARG, "box is NULL");
    const int64_t seg[2] = {0, n};
    if (h) h->seg_rows = nullptr;
    return build_common(pos, species, n, 1, seg, box, periodic, p, h, spec_bounds, stream);
}

extern "C" tbk_status tbk_hamiltonian_size_batched(const double *pos, const int32_t *species, int32_t n_seg,
                                                   const int64_t *seg_atoms, const double *boxes,
                                                   const int32_t periodic[3], const tbk_tb_params *p, tbk_ham *h,
                                                   void *stream) {
    clear_error();
    TBK_CHECK(seg_atoms != nullptr && n_seg >= 1, TBK_ERR_INVALID_ARG, "bad segment table");
    return size_common(pos, species, seg_atoms[n_seg], n_seg, seg_atoms, boxes, periodic, p, h, stream);
}

extern "C" tbk_status tb_build_hamiltonian_batched(const double *pos, const int32_t *species, int32_t n_seg,
                                                   const int64_t *seg_atoms, const double *boxes,
                                                   const int32_t periodic[3], const tbk_tb_params *p, tbk_ham *h,
                                                   double *spec_bounds, void *stream) {
    clear_error();
    TBK_CHECK(seg_atoms != nullptr && n_seg >= 1, TBK_ERR_INVALID_ARG, "bad segment table");
    TBK_CHECK(h != nullptr && h->seg_rows != nullptr, TBK_ERR_INVALID_ARG, "h->seg_rows must hold n_seg+1 entries");
    return build_common(pos, species, seg_atoms[n_seg], n_seg, seg_atoms, boxes, periodic, p, h, spec_bounds, stream);
}
