// Internal plan of the Hamiltonian builder (shared by the plain, batched and
// learned assembly entry points).
#pragma once

#include <cstring>
#include <vector>

#include "common.hpp"
#include "nlist.hpp"

namespace tbk {

constexpr int kBlock = 256;

// Order-preserving map of doubles to signed 64-bit integers (for atomic min/max).
__host__ __device__ __forceinline__ int64_t dkey(double x) {
    int64_t b;
    std::memcpy(&b, &x, sizeof b);
    return b >= 0 ? b : (b ^ INT64_MAX);
}
__host__ __device__ __forceinline__ double dunkey(int64_t k) {
    int64_t b = k >= 0 ? k : (k ^ INT64_MAX);
    double x;
    std::memcpy(&x, &b, sizeof x);
    return x;
}

// Per-segment block reduction of row bounds [lo, hi] (sg = segment of the
// thread's row, -1 for none), then one atomic min and max per segment the
// block touches (per wavefront where segments meet in the block).  Every thread of
// the block must call it.
static __device__ __forceinline__ void block_segment_bounds(double lo, double hi, int32_t sg,
                                                            int64_t *bound_keys) {
    constexpr int kWaves = kBlock / 64;
    __shared__ int32_t seg[kWaves];
    __shared__ double red[2][kWaves];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double a, b;
    auto fold = [&](int32_t q) {       // range of segment q's lanes, in every lane
        a = sg == q ? lo : INFINITY;
        b = sg == q ? hi : -INFINITY;
        for (int d = 32; d > 0; d >>= 1) {
            a = fmin(a, __shfl_xor(a, d));
            b = fmax(b, __shfl_xor(b, d));
        }
    };
    auto flush = [&](int32_t q, double mn, double mx) {
        if (mn <= mx) {
            atomicMin((long long *)&bound_keys[2 * (int64_t)q], (long long)dkey(mn));
            atomicMax((long long *)&bound_keys[2 * (int64_t)q + 1], (long long)dkey(mx));
        }
    };
    uint64_t left = __ballot(sg >= 0);
    const int32_t q0 = left ? __builtin_amdgcn_readlane(sg, __builtin_ctzll(left)) : -1;
    const bool mixed = __ballot(sg >= 0 && sg != q0) != 0;
    fold(q0);
    if (lane == 0) {
        seg[wave] = mixed ? -2 : q0;
        red[0][wave] = a;
        red[1][wave] = b;
    }
    __syncthreads();
    int32_t q = -1;
    bool one = true;
    for (int w = 0; w < kWaves; ++w) {
        if (seg[w] == -2 || (seg[w] >= 0 && q >= 0 && seg[w] != q)) one = false;
        else if (seg[w] >= 0) q = seg[w];
    }
    if (one) {
        if (threadIdx.x == 0 && q >= 0) {
            a = red[0][0];
            b = red[1][0];
            for (int w = 1; w < kWaves; ++w) {
                a = fmin(a, red[0][w]);
                b = fmax(b, red[1][w]);
            }
            flush(q, a, b);
        }
    } else {
        while (left) {
            const int32_t p = __builtin_amdgcn_readlane(sg, __builtin_ctzll(left));
            fold(p);
            if (lane == 0) flush(p, a, b);
            left &= ~__ballot(sg == p);
        }
    }
    __syncthreads();
}

tbk_status check_tb_params(const tbk_tb_params *p);
void decode_bounds(const std::vector<int64_t> &keys, int nseg, double *bounds);
// Keys of n empty bounds.
tbk_status init_bound_keys(DevBuf &keys, int n, Arena &arena, hipStream_t s);

struct HamPlan {
    Arena arena;     // of the plan's buffers and those of its caller
    CellListOwner cells;
    DevBuf perm, iperm, deg, ptr;
    DevBuf nbr;      // first neighbours of each row ([kShortRow][n] atoms), if kept
    int64_t n_slices = 0, n_entries = 0, n_bonds = 0;
    int32_t max_degree = 0;
    int32_t slice = 1;

    // Cell list, row order, degrees, slice offsets and totals.  keep_nbr: for fill();
    // extra: bytes per atom the caller will take from the arena.
    tbk_status run(const double *pos, const int32_t *species, int64_t n, int32_t nseg, const int64_t *seg_atoms,
                   const double *boxes, const int32_t periodic[3], const tbk_tb_params *p, int32_t fmt,
                   int32_t slice_in, hipStream_t s, bool keep_nbr = false, size_t extra = 0);
    // Columns, distance-formula values, onsite, per-segment Gershgorin bounds
    // (bounds: host [n_seg][2]); fills the size fields of h.
    tbk_status fill(const double *pos, const int32_t *species, int64_t n, const tbk_tb_params *p, tbk_ham *h,
                    double *bounds, hipStream_t s);
    tbk_status check_buffers(int64_t n, const tbk_ham *h) const;
    void set_sizes(int64_t n, const tbk_tb_params *p, tbk_ham *h) const;
    // Reads the bound keys back (one per segment and, with_values, the range of the stored
    // hoppings after them), copies the segment table, sets h's sizes.
    tbk_status finish(DevBuf &keys, bool with_values, int64_t n, const tbk_tb_params *p, tbk_ham *h, double *bounds,
                      hipStream_t s);
};

}  // namespace tbk
