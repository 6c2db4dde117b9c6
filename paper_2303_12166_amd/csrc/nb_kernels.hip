// nb_kernels.hip -- gfx950 kernels of libnbody.
//
// The O(N^2) all-pairs force evaluation (Methodology: every element moves only under the sum of
// all pairwise element-element interactions) is the hot path. It runs on the FP32 vector ALUs:
// the pair sum is not a dense contraction, so there is no MFMA here. The kernels that evaluate it:
//   - k_force_rows<T, LAW, R, BAND> (FP32 Kahan and FP64 modes): each unordered pair once, 4 R i elements
//     per lane in registers and the j sums rotating across the wave (see below);
//   - k_force_one_sided<T, LAW, STEP, LOOP> (the same modes, small systems): every ordered pair, in element
//     order, and in a step everything else of it; k_force_mixed runs both in one launch;
//   - k_force_f32 (FP32, plain mode): one-sided, one i element per lane, the block streams
//     256-element SoA j tiles through LDS (broadcast ds_read_b128), one FP32 running sum.
// The first and the last work on a Morton-sorted, star-by-star padded copy of the positions and
// skip the contact test on tiles whose bounding boxes are at least D apart. Per pair of the
// contact law:
//   d = r_j - r_i,  r2 = d.d + eps,  w = rsqrt(r2)  (v_rsq_f32),
//   s = min(w^3, c1 - c2 w),  acc += s d,
// where c1 = 11 / D^3 and c2 = 10 / D^2 for the pair's diameter D. Dividing the contact law
// f(r) = G m^2 / r^2 (r >= D), G m^2 r / D^3 - K (1 - r/D) (r < D, K = 10 G m^2 / D^2) by
// G m^2 r gives w^3 outside and c1 - c2 w inside; with x = r/D, 11 - 10/x - 1/x^3 is increasing
// and vanishes at x = 1, so the smaller of the two expressions is always the right branch.
// The self pair has d = 0 exactly and contributes 0; eps = 1e-24 keeps its w finite. The law of
// eqs. (4)-(6) is written out at pair_s.
//
// The remaining kernels are O(N): leap-frog kicks and drift, per-star centres of mass, the
// donor growth update (eq. 3), the L1-plane count and the FP64 diagnostics. Every reduction runs
// in a fixed order (butterfly within a wave, waves in index order, units in index order), so
// results do not depend on scheduling or on which other systems share a launch.
#include "nb_internal.h"

#include <math.h>

#include <algorithm>

namespace nbk {

// ------------------------------------------------------------------ helpers

// Pointers that a kernel reads from its segment table are global memory: without the address space
// every access would be a flat one, which also waits on the LDS counter. The table itself, and in
// the force kernels a system's state, unit list and boxes, do not change during a launch: read
// as constants they come through the scalar cache into scalar registers, where a plain uniform
// load in a loop with stores is a vector load into vector registers, read again in every round
// (ten steps of 3,001 elements under eqs. (4)-(6) 814 -> 758 us, two of 40,009 942 -> 897, ten of
// 2,048 under the contact law 138 -> 132; the eqs. (4)-(6) kernels spill less).
template <typename T>
using Glob = __attribute__((address_space(1))) T;
template <typename T>
__device__ __forceinline__ Glob<T> *glob(const void *p)
{
    return (Glob<T> *)const_cast<void *>(p);
}

template <typename T>
using Const = const __attribute__((address_space(4))) T;
template <typename T>
__device__ __forceinline__ Const<T> *cst(const T *p)
{
    return (Const<T> *)p;
}
using SysRef = Const<SysDesc> &;

__device__ __forceinline__ int find_sys(const Launch &L, int u, bool ounit)
{
    int lo = 0, hi = L.n_sys - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        int b = ounit ? cst(L.sys)[mid].ounit_begin : cst(L.sys)[mid].unit_begin;
        if (b <= u) {
            lo = mid;
        } else {
            hi = mid - 1;
        }
    }
    return lo;
}

// Fixed-order block sum of NV doubles per thread; the result is valid in thread 0.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double (*lds)[BT / 64])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double x = v[k];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
        v[k] = x;
    }
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) lds[k][wave] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double t = lds[k][0];
#pragma unroll
            for (int w = 1; w < BT / 64; ++w) t += lds[k][w];
            v[k] = t;
        }
    }
    __syncthreads();
}

__device__ __forceinline__ void kahan_add(float &sum, float &comp, float v)
{
    float y = v - comp;
    float t = sum + y;
    comp = (t - sum) - y;
    sum = t;
}

__device__ __forceinline__ int pair_class(int istar, int jstar) { return istar + jstar; }

constexpr double PI_D = 3.14159265358979323846;

// FP32 transcendentals, each issued at raised wave priority. A SIMD issues the ordinary FP32
// instructions of two waves side by side (measured 104-115 lanes per clock per CU for a stream of
// them, against 59 with a scalar-register source), but a transcendental, four times as long, leaves
// the other slot idle unless a second wave's transcendental fills it. With the priority raised
// around it, a wave that reaches one is picked at once and they pair up: the 15 instructions of a
// contact-law pair issue at 94 lanes per clock per CU at four waves per SIMD and 98 at eight (81
// and 83 without; 99 is what the parts allow: 14 at 115 and one at 32). The chip answers with a
// lower clock (2.09 against 2.22 GHz in the symmetric kernel), so at N = 262,144 the evaluation gains 3.6 %
// (10.95 -> 10.55 ms; eqs. (4)-(6) 14.67 -> 14.34), at 40,009 under eqs. (4)-(6) 5 %, and
// k_force_f32 at N = 131,072, at two waves per SIMD, 13 % (8.12 -> 7.07 ms before its staging). s_setprio after the
// transcendental is also the wait state that its first use needs.
__device__ __forceinline__ float rsq_p(float x)
{
    float w;
    asm("s_setprio 1\n\tv_rsq_f32 %0, %1\n\ts_setprio 0" : "=v"(w) : "v"(x));
    return w;
}

__device__ __forceinline__ float sqrt_p(float x)
{
    float w;
    asm("s_setprio 1\n\tv_sqrt_f32 %0, %1\n\ts_setprio 0" : "=v"(w) : "v"(x));
    return w;
}

__device__ __forceinline__ float rcp_p(float x)
{
    float w;
    asm("s_setprio 1\n\tv_rcp_f32 %0, %1\n\ts_setprio 0" : "=v"(w) : "v"(x));
    return w;
}

// ------------------------------------------------------------------ sorted layout

__device__ __forceinline__ int find_tile_sys(const Launch &L, int u)
{
    int lo = 0, hi = L.n_sys - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (cst(L.sys)[mid].tunit_begin <= u) {
            lo = mid;
        } else {
            hi = mid - 1;
        }
    }
    return lo;
}

__device__ __forceinline__ float wave_min(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fminf(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    return v;
}

// Sentinel positions in every slot of the sorted copy and -1 in the padding slots of the order.
template <typename T>
__global__ __launch_bounds__(BT) void k_reset_sorted(T *xs, T *ys, T *zs, int32_t *perm, int n, int n1,
                                                     int p1, int nalloc, T value)
{
    const int k = blockIdx.x * BT + threadIdx.x;
    if (k >= nalloc) return;
    xs[k] = value;
    ys[k] = value;
    zs[k] = value;
    if ((k >= n1 && k < p1) || k >= p1 + (n - n1)) perm[k] = -1;
}

template <typename T>
__global__ __launch_bounds__(BT) void k_zero_sorted(T *xs, T *ys, T *zs, int nalloc)
{
    const int k = blockIdx.x * BT + threadIdx.x;
    if (k < nalloc) xs[k] = ys[k] = zs[k] = 0;
}

// ------------------------------------------------------------------ sorted order
//
// The order of a system's slots: star by star, by the Morton code of the position (10 bits per axis
// inside the star's bounding box), ties by index. A least-digit radix sort of (star, code) from
// index order, four stable passes of eight bits over tiles of SORT_TILE elements: a histogram per
// tile, its prefix sums per digit, and the scatter. The arrays it works in are those of the sorted
// copy, which is rebuilt before anything reads it. Launches bound it (fifteen, a few microseconds
// each) up to some 100,000 elements; a read-back and a comparison sort on the host took 1.37 ms at
// 32,768 elements and 13.2 ms at 262,144 (nb_resort), this 0.08 and 0.09. Systems of one sort tile take
// one launch (k_sort_small).

// Each star's smallest and largest finite coordinates (per star: min x, y, z, then -max x, y, z) over
// the elements i0, i0 + stride, .. of every thread. Called by a whole workgroup; the
// result is in `box`, written by its first twelve threads.
template <typename T>
__device__ __forceinline__ void star_bounds(const T *x, const T *y, const T *z, int n, int n1, int i0,
                                            int stride, double (*lds)[BT / 64], double *box)
{
    double v[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = 1e300;
    for (int i = i0; i < n; i += stride) {
        const double p[3] = {(double)x[i], (double)y[i], (double)z[i]};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if (!isfinite(p[d])) continue;
#pragma unroll
            for (int star = 0; star < 2; ++star) {
                if ((i >= n1) != (star == 1)) continue;
                v[6 * star + d] = fmin(v[6 * star + d], p[d]);
                v[6 * star + 3 + d] = fmin(v[6 * star + 3 + d], -p[d]);
            }
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v[k] = fmin(v[k], __shfl_xor(v[k], off, 64));
        if (lane == 0) lds[k][wave] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < 12) {
        const int k = threadIdx.x;
        box[k] = fmin(fmin(lds[k][0], lds[k][1]), fmin(lds[k][2], lds[k][3]));
    }
}

template <typename T>
__global__ __launch_bounds__(BT) void k_sort_bounds(const T *x, const T *y, const T *z, int n, int n1,
                                                    double *out)
{
    __shared__ double lds[12][BT / 64];
    star_bounds(x, y, z, n, n1, blockIdx.x * BT + threadIdx.x, gridDim.x * BT, lds,
                out + 12 * blockIdx.x);
}

__device__ __forceinline__ uint32_t spread10(uint32_t v)
{
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

// Star and Morton code of a position inside its star's box.
__device__ __forceinline__ uint32_t sort_key(double x, double y, double z, int star, const double *box)
{
    const double p[3] = {x, y, z};
    uint32_t key = (uint32_t)star << 30;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double lo = box[6 * star + d], hi = -box[6 * star + 3 + d];
        const double span = hi > lo ? hi - lo : 1.0;
        double f = isfinite(p[d]) ? (p[d] - lo) / span : 0.0;
        f = f < 0.0 ? 0.0 : f;
        f = 1.0 < f ? 1.0 : f;
        f = f * 1024.0;
        key |= spread10((uint32_t)(f < 1023.0 ? f : 1023.0)) << d;
    }
    return key;
}

template <typename T>
__global__ __launch_bounds__(BT) void k_sort_keys(const T *x, const T *y, const T *z, int n, int n1,
                                                  const double *bounds, int n_bounds, uint32_t *keys)
{
    __shared__ double box[12];
    if (threadIdx.x < 64) {
        // one wave: lane 5 k .. 5 k + 4 take value k of every fifth workgroup's bounds
        const int k = threadIdx.x / 5, part = threadIdx.x % 5;
        double v = 1e300;
        if (k < 12) {
#pragma unroll 4
            for (int b = part; b < n_bounds; b += 5) v = fmin(v, bounds[12 * b + k]);
        }
        double m = v;
#pragma unroll
        for (int q = 1; q < 5; ++q) m = fmin(m, __shfl(v, min(63, 5 * k + (part + q) % 5), 64));
        if (k < 12 && part == 0) box[k] = m;
    }
    __syncthreads();
    const int i = blockIdx.x * BT + threadIdx.x;
    if (i < n) keys[i] = sort_key((double)x[i], (double)y[i], (double)z[i], i >= n1 ? 1 : 0, box);
}

// Digit counts of one tile, stored digit by digit (entry digit n_tiles + tile).
__global__ __launch_bounds__(BT) void k_sort_hist(const uint32_t *keys, int n, int shift, int n_tiles,
                                                  uint32_t *hist)
{
    __shared__ uint32_t cnt[256];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const int base = blockIdx.x * SORT_TILE;
#pragma unroll
    for (int r = 0; r < SORT_TILE / BT; ++r) {
        const int i = base + r * BT + threadIdx.x;
        if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(size_t)threadIdx.x * n_tiles + blockIdx.x] = cnt[threadIdx.x];
}

// Exclusive prefix sum of 256 values, one per thread; the last thread also returns the total.
__device__ __forceinline__ uint32_t scan256(uint32_t v, uint32_t *wsum, uint32_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
    return before + x - v;
}

// One digit per workgroup: its tiles' counts become the elements before each tile, and its total.
__global__ __launch_bounds__(BT) void k_sort_scan(uint32_t *hist, int n_tiles, uint32_t *totals)
{
    __shared__ uint32_t wsum[BT / 64];
    uint32_t *h = hist + (size_t)blockIdx.x * n_tiles;
    uint32_t carry = 0;
    for (int t0 = 0; t0 < n_tiles; t0 += BT) {
        const int t = t0 + threadIdx.x;
        const uint32_t v = t < n_tiles ? h[t] : 0u;
        uint32_t total;
        const uint32_t before = scan256(v, wsum, total);
        if (t < n_tiles) h[t] = carry + before;
        carry += total;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// The place of this lane's element (none: not `valid`) among the wave's elements of the same digit, of
// which `at` holds the next free place: the lanes before it that hold the same digit come first.
__device__ __forceinline__ uint32_t next_place(volatile uint32_t *at, uint32_t digit, bool valid,
                                               int lane)
{
    unsigned long long same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const unsigned long long one = __ballot((digit >> b) & 1u);
        same &= (digit >> b) & 1u ? one : ~one;
    }
    const int rank = __popcll(same & ((1ull << lane) - 1ull));
    uint32_t pos = 0;
    if (valid) pos = at[digit] + rank;
    __builtin_amdgcn_wave_barrier();
    if (valid && rank == 0) at[digit] = pos + __popcll(same);
    __builtin_amdgcn_wave_barrier();
    return pos;
}

// Moves one tile's elements to their places, in order within a digit: every wave takes a run of the
// tile, 64 elements at a time (next_place). vals_in null: the index itself (first pass). keys_out
// null: the last pass, where the values become the order of the slots.
__global__ __launch_bounds__(BT) void k_sort_scatter(const uint32_t *keys_in, const int32_t *vals_in,
                                                     uint32_t *keys_out, int32_t *vals_out, int n,
                                                     int shift, int n_tiles, const uint32_t *hist,
                                                     const uint32_t *totals, int n1, int p1)
{
    __shared__ uint32_t wsum[BT / 64];
    __shared__ volatile uint32_t at[BT / 64][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int ROWS = SORT_TILE / BT;
    const int base = blockIdx.x * SORT_TILE + wave * (SORT_TILE / 4);
    uint32_t key[ROWS];
#pragma unroll
    for (int w = 0; w < BT / 64; ++w) at[w][tid] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int i = base + 64 * r + lane;
        key[r] = i < n ? keys_in[i] : 0u;
        if (i < n) atomicAdd(const_cast<uint32_t *>(&at[wave][(key[r] >> shift) & 255u]), 1u);
    }
    uint32_t total;
    uint32_t place = scan256(totals[tid], wsum, total) + hist[(size_t)tid * n_tiles + blockIdx.x];
#pragma unroll
    for (int w = 0; w < BT / 64; ++w) {
        const uint32_t c = at[w][tid];
        at[w][tid] = place;
        place += c;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int i = base + 64 * r + lane;
        const bool valid = i < n;
        const uint32_t digit = (key[r] >> shift) & 255u;
        const uint32_t pos = next_place(at[wave], digit, valid, lane);
        if (valid) {
            const int32_t val = vals_in ? vals_in[i] : i;
            if (keys_out) {
                keys_out[pos] = key[r];
                vals_out[pos] = val;
            } else {
                vals_out[(int)pos < n1 ? pos : p1 + (pos - n1)] = val;
            }
        }
    }
}

// The whole order of a system of at most one sort tile, with what k_reset_sorted does, by one workgroup:
// the same passes in LDS. As fifteen launches nb_resort took 85 us at 64 to 2,048 elements, more
// than the host's sort below 1,500 (60 us at 64).
template <typename T>
__global__ __launch_bounds__(BT) void k_sort_small(const T *x, const T *y, const T *z, int n, int n1,
                                                   int p1, int nalloc, T *xs, T *ys, T *zs,
                                                   int32_t *perm, T value)
{
    constexpr int ROWS = SORT_TILE / BT;
    __shared__ double lds[12][BT / 64];
    __shared__ double box[12];
    __shared__ uint32_t wsum[BT / 64];
    __shared__ volatile uint32_t at[BT / 64][256];
    __shared__ uint32_t keys[SORT_TILE], vals[SORT_TILE];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int base = wave * (SORT_TILE / 4);
    star_bounds(x, y, z, n, n1, tid, BT, lds, box);
    __syncthreads();
    uint32_t key[ROWS], val[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int i = base + 64 * r + lane;
        key[r] = i < n ? sort_key((double)x[i], (double)y[i], (double)z[i], i >= n1 ? 1 : 0, box) : 0u;
        val[r] = i;
    }
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 8 * pass;
#pragma unroll
        for (int w = 0; w < BT / 64; ++w) at[w][tid] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if (base + 64 * r + lane < n)
                atomicAdd(const_cast<uint32_t *>(&at[wave][(key[r] >> shift) & 255u]), 1u);
        }
        __syncthreads();
        uint32_t count = 0, total;
#pragma unroll
        for (int w = 0; w < BT / 64; ++w) count += at[w][tid];
        uint32_t place = scan256(count, wsum, total);
#pragma unroll
        for (int w = 0; w < BT / 64; ++w) {
            const uint32_t c = at[w][tid];
            at[w][tid] = place;
            place += c;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const bool valid = base + 64 * r + lane < n;
            const uint32_t pos = next_place(at[wave], (key[r] >> shift) & 255u, valid, lane);
            if (!valid) continue;
            if (pass < 3) {
                keys[pos] = key[r];
                vals[pos] = val[r];
            } else {
                perm[(int)pos < n1 ? pos : p1 + (pos - n1)] = (int32_t)val[r];
            }
        }
        if (pass == 3) break;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int i = base + 64 * r + lane;
            if (i < n) {
                key[r] = keys[i];
                val[r] = vals[i];
            }
        }
    }
    for (int k = tid; k < nalloc; k += BT) {
        xs[k] = value;
        ys[k] = value;
        zs[k] = value;
        if ((k >= n1 && k < p1) || k >= p1 + (n - n1)) perm[k] = -1;
    }
}

// The nearest float not above x: an FP64 system's boxes hold its elements exactly.
__device__ __forceinline__ float float_below(float x) { return x; }
__device__ __forceinline__ float float_below(double x)
{
    const float f = (float)x;
    return (double)f > x ? nextafterf(f, -INFINITY) : f;
}

// Whether every squared distance to an element at this coordinate is finite in FP64.
__device__ __forceinline__ bool bounded(float x) { return isfinite(x); }
__device__ __forceinline__ bool bounded(double x) { return fabs(x) < 1.0e100; }

// One element of a tile into its sorted slot (none: `held` is false, the slot keeps its fill values and
// is left out of the box), and the tile's bounding box. Called by a whole workgroup.
template <typename T>
__device__ __forceinline__ void store_sorted(SysRef S, int tile, bool held, bool vel, T x, T y, T z, T vx,
                                             T vy, T vz, float (*lds)[BT / 64])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int slot = tile * TJ + threadIdx.x;
    float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (held) {
        glob<T>(S.xs)[slot] = x;
        glob<T>(S.ys)[slot] = y;
        glob<T>(S.zs)[slot] = z;
        if (vel) {
            glob<T>(S.vxs)[slot] = vx;
            glob<T>(S.vys)[slot] = vy;
            glob<T>(S.vzs)[slot] = vz;
        }
        v[0] = float_below(x);
        v[1] = float_below(y);
        v[2] = float_below(z);
        v[3] = -float_below(-x);
        v[4] = -float_below(-y);
        v[5] = -float_below(-z);
        // a tile with an element out of range is near everything: only the potential energy's
        // near form leaves such an element's pairs out
        if (!(bounded(x) && bounded(y) && bounded(z))) {
            v[0] = v[1] = v[2] = -INFINITY;
            v[3] = v[4] = v[5] = INFINITY;
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        v[k] = wave_min(v[k]);
        v[3 + k] = wave_max(v[3 + k]);
    }
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 6; ++k) lds[k][wave] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < 8) {
        const int k = threadIdx.x;
        float r = 0.0f;
        if (k < 3 || (k >= 4 && k < 7)) {
            const int q = k < 3 ? k : k - 1;
            r = lds[q][0];
            for (int w = 1; w < BT / 64; ++w) r = q < 3 ? fminf(r, lds[q][w]) : fmaxf(r, lds[q][w]);
        }
        glob<float>(S.tbox)[(size_t)tile * 8 + k] = r;
    }
    __syncthreads();
}

// Pulls the current positions (and, under eqs. (4)-(6), velocities) into sorted order and records
// each tile's bounding box. In the steps of the symmetric kernels k_advance does this.
template <typename T>
__global__ __launch_bounds__(BT) void k_gather(Launch L)
{
    __shared__ float lds[6][BT / 64];
    for (int u = blockIdx.x; u < L.total_tunits; u += gridDim.x) {
        SysRef S = cst(L.sys)[find_tile_sys(L, u)];
        const int tile = u - S.tunit_begin;
        const int idx = glob<const int32_t>(S.perm)[tile * TJ + threadIdx.x];
        T x = 0, y = 0, z = 0, vx = 0, vy = 0, vz = 0;
        if (idx >= 0) {
            x = glob<const T>(S.x)[idx];
            y = glob<const T>(S.y)[idx];
            z = glob<const T>(S.z)[idx];
            if (S.law != 0) {
                vx = glob<const T>(S.vx)[idx];
                vy = glob<const T>(S.vy)[idx];
                vz = glob<const T>(S.vz)[idx];
            }
        }
        store_sorted<T>(S, tile, idx >= 0, S.law != 0, x, y, z, vx, vy, vz, lds);
    }
}

// A value that is the same in every lane, moved to a scalar register.
__device__ __forceinline__ float wave_uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Whether a tile lies at least D from every i of the wave (its bounding box against the wave's),
// for the larger of the band's thresholds.
__device__ __forceinline__ bool far_tile(Const<float> *bx, const float (&lo)[3],
                                         const float (&hi)[3], float far2)
{
    const float gx = fmaxf(0.0f, fmaxf(bx[0] - hi[0], lo[0] - bx[4]));
    const float gy = fmaxf(0.0f, fmaxf(bx[1] - hi[1], lo[1] - bx[5]));
    const float gz = fmaxf(0.0f, fmaxf(bx[2] - hi[2], lo[2] - bx[6]));
    // a square above FP32's range is still below a limit of infinity
    const float gap2 = fminf(gx * gx + gy * gy + gz * gz, 3.0e38f);
    return __builtin_amdgcn_readfirstlane(gap2 >= far2 ? 1 : 0) != 0;
}

// ------------------------------------------------------------------ FP32 one-sided force kernel

__device__ __forceinline__ float4 lds4(const float *p) { return *reinterpret_cast<const float4 *>(p); }

// One tile's 256 j, eight at a time, each stage of the pair code for all eight before the next: one
// running sum per element leaves n / 64 waves, two per SIMD at 131,072 elements, and a wave on its
// own issues a dependent chain at half the rate of independent instructions (pair after pair
// 7.06 ms an evaluation at 131,072, staged 5.12; with at most one wave per SIMD the raised priority
// of the reciprocal square roots only costs issue slots: 2.25 -> 2.04 ms at 65,536 without it, 5.50
// with two waves without it). Near tiles: the contact law s = min(w^3, c1 - c2 w) for every
// pair; far tiles (every pair at r >= D, proven from bounding boxes): s = w^3, the value the contact
// law's minimum selects there.
template <bool FAR, bool PRIO>
__device__ __forceinline__ void plain_tile(const float *sx, const float *sy, const float *sz,
                                           float xi, float yi, float zi, float c1, float nc2,
                                           float eps, float &ax, float &ay, float &az)
{
    constexpr int G = 8;
    float4 X[2], Y[2], Z[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        X[h] = lds4(sx + 4 * h);
        Y[h] = lds4(sy + 4 * h);
        Z[h] = lds4(sz + 4 * h);
    }
#pragma unroll 1
    for (int jj = 0; jj < TJ; jj += G) {
        float dx[G], dy[G], dz[G], s[G];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float x[4] = {X[h].x, X[h].y, X[h].z, X[h].w};
            const float y[4] = {Y[h].x, Y[h].y, Y[h].z, Y[h].w};
            const float z[4] = {Z[h].x, Z[h].y, Z[h].z, Z[h].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                dx[4 * h + q] = x[q] - xi;
                dy[4 * h + q] = y[q] - yi;
                dz[4 * h + q] = z[q] - zi;
            }
        }
        const int nx = (jj + G) & (TJ - 1);  // the next eight (after the last the first: not used)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            X[h] = lds4(sx + nx + 4 * h);
            Y[h] = lds4(sy + nx + 4 * h);
            Z[h] = lds4(sz + nx + 4 * h);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < G; ++q) s[q] = fmaf(dz[q], dz[q], eps);
#pragma unroll
        for (int q = 0; q < G; ++q) s[q] = fmaf(dy[q], dy[q], s[q]);
#pragma unroll
        for (int q = 0; q < G; ++q) s[q] = fmaf(dx[q], dx[q], s[q]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < G; ++q) s[q] = PRIO ? rsq_p(s[q]) : __builtin_amdgcn_rsqf(s[q]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const float w = s[q];
            const float w3 = (w * w) * w;
            s[q] = FAR ? w3 : fminf(w3, fmaf(nc2, w, c1));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < G; ++q) {
            ax = fmaf(s[q], dx[q], ax);
            ay = fmaf(s[q], dy[q], ay);
            az = fmaf(s[q], dz[q], az);
        }
    }
}

// One force unit of the plain mode: the 256 elements from ib 256 in sorted order without padding, one
// per lane, against every tile, one running FP32 sum per element in tile order.
template <bool PRIO>
__device__ __forceinline__ void force_unit_f32(SysRef S, int ib, float (*sh)[3][TJ])
{
    const int tid = threadIdx.x;
    auto *__restrict__ XS = glob<const float>(S.xs);
    auto *__restrict__ YS = glob<const float>(S.ys);
    auto *__restrict__ ZS = glob<const float>(S.zs);
    auto *st = cst(S.st);

    const int g = ib * BT + tid;  // among the real elements: star 1's n1 slots, then from slot p1
    const bool real = g < S.n;
    const int gc = real ? g : S.n - 1;
    const int istar = gc >= S.n1 ? 1 : 0;
    const int slot = istar ? S.p1 + (gc - S.n1) : gc;
    const float xi = XS[slot], yi = YS[slot], zi = ZS[slot];
    float ax = 0.0f, ay = 0.0f, az = 0.0f;
    float lo[3] = {wave_min(xi), wave_min(yi), wave_min(zi)};
    float hi[3] = {wave_max(xi), wave_max(yi), wave_max(zi)};
    const float c1a = st->cur.c1f[istar], nc2a = -st->cur.c2f[istar];
    const float c1b = st->cur.c1f[istar + 1], nc2b = -st->cur.c2f[istar + 1];
    // the wave's (a wave may hold the end of one star and the start of the other)
    const float far2a = wave_uniform(wave_max(st->cur.far2f[istar]));
    const float far2b = wave_uniform(wave_max(st->cur.far2f[istar + 1]));
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = wave_uniform(lo[d]);
        hi[d] = wave_uniform(hi[d]);
    }
    float eps;  // in a vector register: a literal halves the issue rate
    asm("v_mov_b32 %0, 0x179abe15" : "=v"(eps));  // 1e-24

    const int ntiles = S.ntiles;
    float px = XS[tid], py = YS[tid], pz = ZS[tid];
    for (int t = 0; t < ntiles; ++t) {
        const int buf = t & 1;
        sh[buf][0][tid] = px;
        sh[buf][1][tid] = py;
        sh[buf][2][tid] = pz;
        __syncthreads();
        if (t + 1 < ntiles) {
            px = XS[(t + 1) * TJ + tid];
            py = YS[(t + 1) * TJ + tid];
            pz = ZS[(t + 1) * TJ + tid];
        }
        const bool jstar = t * TJ >= S.p1;
        const float *sx = sh[buf][0], *sy = sh[buf][1], *sz = sh[buf][2];
        if (far_tile(cst(S.tbox) + (size_t)t * 8, lo, hi, jstar ? far2b : far2a)) {
            plain_tile<true, PRIO>(sx, sy, sz, xi, yi, zi, 0.f, 0.f, eps, ax, ay, az);
        } else {
            plain_tile<false, PRIO>(sx, sy, sz, xi, yi, zi, jstar ? c1b : c1a, jstar ? nc2b : nc2a, eps,
                              ax, ay, az);
        }
    }
    __syncthreads();  // the next unit of this block reuses both LDS buffers

    if (!real) return;
    const int idx = glob<const int32_t>(S.perm)[slot];
    const float gm = st->gm_f;
    glob<float>(S.ax)[idx] = gm * ax;
    glob<float>(S.ay)[idx] = gm * ay;
    glob<float>(S.az)[idx] = gm * az;
}

template <bool PRIO>
__global__ __launch_bounds__(BT) __attribute__((amdgpu_waves_per_eu(PLAIN_WAVES)))
void k_force_f32(Launch L)
{
    __shared__ __attribute__((aligned(16))) float sh[2][3][TJ];
    for (int u = L.unit_base + blockIdx.x; u < L.total_units; u += gridDim.x) {
        SysRef S = cst(L.sys)[find_sys(L, u, false)];
        force_unit_f32<PRIO>(S, u - S.unit_begin, sh);
    }
}

// ------------------------------------------------------------------ symmetric force kernel
//
// Newton's third law halves the pair work: the pair (i, j) with i in tile I and j in a later
// tile J > I is evaluated once. The tile rows are taken in groups ("row bands") of KR consecutive
// rows (KR = 1, 2 or 4, chosen per system size; 1 in the FP64 mode): a work unit is group g, rows
// I = KR g .. KR g + KR - 1, against chunk c of its tiles, a run of `ch` tiles starting at KR g +
// c ch. The kernel holds R rows at a time (1 or 2; a band of four is taken two rows after the
// other). The tiles after a unit's rows are full pairs; of the tiles inside the band, tile KR g + k
// is one-sided for row k, full for the rows before it and skipped by the rows after it.
//
// The j are split over the block's four waves: every wave holds all 256 R elements i, 4 R per lane,
// and wave w takes the 64 j of quarter w of each tile. At step s (0..63) lane l meets element
// (l - s) mod 64 of them: its position is read from LDS once and paired with the lane's 4 R
// elements, and the j accumulator travels with it, one lane per step, through the LDS crossbar.
// After 64 steps lane l holds the whole reaction of the 256 R elements on its own j and stores it
// (with its sign turned: an added term takes the short form of the fused multiply-add). So a j read
// and a move of its sums serve 4 R pairs, and the waves share nothing inside the loop: each
// stages its own 64 j, with no barrier and no sum across waves per tile; their i sums, one FP32
// partial per tile under Kahan compensation, are added once per unit. A kernel with the i split
// over the waves instead (one element of each row per lane, KR pairs per read, the reactions of
// the four waves added through LDS) held four rows at most and needs twice the LDS traffic at
// the same registers. Measured against it, whole evaluations at the best split of either:
// contact law 97 -> 77 us at N = 16,384, 241 -> 217 at 32,768, 747 -> 724 at 65,536, 10.69 -> 10.15
// ms at 262,144; eqs. (4)-(6) 61 -> 50 us at 9,000, 458 -> 412 at 40,009, 13.97 -> 12.90 ms at
// 262,144; FP64 176 -> 156 us at 16,384, 1082 -> 965 at 50,021, eqs. (4)-(6) 216 -> 197 at 16,384.
// What bounds it: at 262,144 FP32 issue at the clock that the chip's power leaves (about 2.1 GHz
// of 2.4); below some 20,000 elements the few, long units.
//
// k_combine_sym adds, per element, its own row's chunk partials and then the reactions of every
// group with a row before the element's tile, in group order, with Kahan compensation. The order
// of every sum is fixed by the system's own size, so results do not depend on scheduling or on
// the other systems of a launch.

// Lane l receives lane l - 1's value (mod 64) through the LDS crossbar (ds_bpermute, no LDS
// storage): addr = 4 ((l - 1) mod 64) in lane l.
__device__ __forceinline__ float xbar_ror1(float v, int addr)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}

// Constants of one pair class for the FP32 kernels.
struct LawF {
    float c1, nc2;            // contact law: 11 / D^3 and -10 / D^2
    float D, twoD, eps, gc, gcb;  // eqs. (4)-(6): see DevState
};

__device__ __forceinline__ LawF law_uniform(LawF K)
{
    K.c1 = wave_uniform(K.c1);
    K.nc2 = wave_uniform(K.nc2);
    K.D = wave_uniform(K.D);
    K.twoD = wave_uniform(K.twoD);
    K.eps = wave_uniform(K.eps);
    K.gc = wave_uniform(K.gc);
    K.gcb = wave_uniform(K.gcb);
    return K;
}

__device__ __forceinline__ LawF law_f(Const<DevState> *st, Const<LawState> *ls, int cls)
{
    LawF K;
    K.c1 = ls->c1f[cls];
    K.nc2 = -ls->c2f[cls];
    K.D = ls->lD_f[cls];
    K.twoD = 2.0f * ls->lD_f[cls];
    K.eps = st->leps_f;
    K.gc = st->lgc_f;
    K.gcb = st->lgcb_f;
    return K;
}

// Pair scalar s = f / (G m^2 r) of one pair from r2 = |d|^2; the caller adds s d to the i sum.
//   contact law:  w = rsqrt(r2); min(w^3, c1 - c2 w) near, w^3 far.
//   eqs. (4)-(6): r = sqrt(r2), t = r + eps; s = 1 / (t^2 r) - g (D - r)_+^2 (1 + 2 D w) with
//                 w = 1 / r = t^2 s_att, g = gc for a converging pair ((v_j - v_i).(r_j - r_i)
//                 < 0) and gcb otherwise; the overlap term is left out on far tiles, where every
//                 pair has r >= D. (pi / 12) (D - r)^2 (r + 2D) is the overlap volume of eq. (5)
//                 in factored form, so it has no cancellation near D. The square root form takes
//                 one multiply fewer per far pair than r = r2 rsqrt(r2) (measured 2.5 % faster).
//                 A padding slot (r near 1.7e18) gives t^2 r = inf, s = 0 and w = 0. The near form
//                 works the overlap out only where a lane of the wave is in contact: it is half
//                 of the instructions, and in most steps of a near tile no pair touches (measured
//                 at 9,000 elements 53 -> 45 us, 16,384 111 -> 94, 262,144 12.99 -> 12.76 ms, and
//                 one-sided at 7,001 49 -> 36).
// On a far tile the near form gives the same bits (the contact law's minimum picks w^3 by a margin
// far above rounding once r^2 >= (1 + FAR_MARGIN) D^2; the overlap term is exactly 0 for r >= D),
// so the near/far choice changes speed only.
template <int LAW, bool NEAR>
__device__ __forceinline__ float pair_s(float r2, float dx, float dy, float dz, const float4 &vj,
                                        const float4 &vi, const LawF &K)
{
#pragma clang fp contract(off)
    if constexpr (LAW == 0) {
        const float w = rsq_p(r2);
        const float w3 = (w * w) * w;
        return NEAR ? fminf(w3, fmaf(K.nc2, w, K.c1)) : w3;
    } else {
        const float r = sqrt_p(r2);
        const float t = r + K.eps;
        const float t2 = t * t;
        float s = rcp_p(t2 * r);
        if constexpr (NEAR) {
            if (__any(r < K.D)) {
                const float w = t2 * s;
                const float dot = fmaf(vj.x - vi.x, dx, fmaf(vj.y - vi.y, dy, (vj.z - vi.z) * dz));
                const float g = dot < 0.0f ? K.gc : K.gcb;
                const float u = fmaxf(K.D - r, 0.0f);
                s = s - ((g * u) * u) * fmaf(K.twoD, w, 1.0f);
            }
        }
        return s;
    }
}

// Reactions are stored per group g (tile rows KR g .. KR g + KR - 1) for the tiles t after the
// group's first row, t = KR g + 1 .. T - 1: three components one after the other, each
// (T - KR g - 1) TJ values. Group g starts after
// sum_{g' < g} 3 TJ (T - KR g' - 1) = 3 TJ (g (T - 1) - KR g (g - 1) / 2) values.
__device__ __forceinline__ size_t react_group_offset(int g, int ntiles, int kr)
{
    return (size_t)3 * TJ *
           ((size_t)g * (ntiles - 1) - (size_t)kr * (size_t)g * (size_t)(g - 1) / 2);
}

// ------------------------------------------------------------------ second kick

constexpr int COMBINE_SEGS = 4;  // threads per element of the combine kernels

template <typename T, typename St>
__device__ __forceinline__ T h_of(St st)
{
    if constexpr (sizeof(T) == 4) {
        return st->h_f;
    } else {
        return st->h_d;
    }
}
template <typename T, typename St>
__device__ __forceinline__ T dt_of(St st)
{
    if constexpr (sizeof(T) == 4) {
        return st->dt_f;
    } else {
        return st->dt;
    }
}
template <typename T, typename St>
__device__ __forceinline__ T gm_of(St st)
{
    if constexpr (sizeof(T) == 4) {
        return st->gm_f;
    } else {
        return st->gm_d;
    }
}

// Per-unit record of a step: each star's position sums and the count of non-finite elements.
__device__ __forceinline__ void add_stats(double (&v)[7], double px, double py, double pz,
                                          double wx, double wy, double wz, bool star2)
{
    const int o = star2 ? 3 : 0;
    v[o + 0] = px;
    v[o + 1] = py;
    v[o + 2] = pz;
    const bool fin = isfinite(px) && isfinite(py) && isfinite(pz) && isfinite(wx) &&
                     isfinite(wy) && isfinite(wz);
    v[6] = fin ? 0.0 : 1.0;
}

// Row of the L1 log of a step: its number, then the counts.
__device__ __forceinline__ int32_t *log_row(SysRef S, int64_t step)
{
    return S.l1_log + 4 * (size_t)(step % L1_LOG_CAP);
}

// The counts of step number `step` start from nothing.
__device__ __forceinline__ void clear_counts(SysRef S, int64_t step)
{
    DevState *st = S.st;
    st->n_past = st->fwd = st->bwd = 0;
    int32_t *row = log_row(S, step);
    row[0] = (int32_t)step;
    row[1] = row[2] = row[3] = 0;
}

__device__ __forceinline__ float fma_t(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return fma(a, b, c); }

// The state of a slot's element as the force saw it.
template <typename T>
__device__ __forceinline__ void element_state(SysRef S, int slot, T (&x)[3], T (&v)[3])
{
    x[0] = glob<const T>(S.xs)[slot];
    x[1] = glob<const T>(S.ys)[slot];
    x[2] = glob<const T>(S.zs)[slot];
    v[0] = glob<const T>(S.vxs)[slot];
    v[1] = glob<const T>(S.vys)[slot];
    v[2] = glob<const T>(S.vzs)[slot];
}

// The second kick of this thread's element idx (none: -1) of tile J with its new acceleration, and the
// tile's record of the step. Between the steps of a call the elements stay in sorted order (S.xs, S.vxs
// and S.as): 4-byte writes all over the caller's arrays, six per element and step, cost as much
// as a pass of their own. The `last` step writes the caller's. Called by a whole workgroup of
// BT * COMBINE_SEGS threads, of which the first TJ hold the tile's elements; x and v are the
// element's, loaded before.
template <typename T>
__device__ __forceinline__ void kick_record(SysRef S, int J, int idx, const T (&x)[3], const T (&v)[3],
                                            const T (&a)[3], int last, double (*lds)[BT / 64])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x < TJ) {
        double r[7] = {0, 0, 0, 0, 0, 0, 0};
        if (idx >= 0) {
            const T h = h_of<T>(glob<const DevState>(S.st));
            const T wx = fma_t(h, a[0], v[0]), wy = fma_t(h, a[1], v[1]), wz = fma_t(h, a[2], v[2]);
            const int slot = J * TJ + threadIdx.x;
            if (last) {
                glob<T>(S.x)[idx] = x[0];
                glob<T>(S.y)[idx] = x[1];
                glob<T>(S.z)[idx] = x[2];
                glob<T>(S.vx)[idx] = wx;
                glob<T>(S.vy)[idx] = wy;
                glob<T>(S.vz)[idx] = wz;
            } else {
                glob<T>(S.vxs)[slot] = wx;
                glob<T>(S.vys)[slot] = wy;
                glob<T>(S.vzs)[slot] = wz;
                auto *A = glob<T>(S.as) + slot;
                A[0] = a[0];
                A[S.nalloc] = a[1];
                A[2 * (size_t)S.nalloc] = a[2];
            }
            add_stats(r, x[0], x[1], x[2], wx, wy, wz, idx >= S.n1);
        }
#pragma unroll
        for (int k = 0; k < 7; ++k) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) r[k] += __shfl_xor(r[k], off, 64);
            if (lane == 0) lds[k][wave] = r[k];
        }
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        const int k = threadIdx.x;
        double t = lds[k][0];
        for (int w = 1; w < TJ / 64; ++w) t += lds[k][w];
        glob<double>(S.rec)[(size_t)J * REC_STRIDE + k] = t;
    }
    if (threadIdx.x == 0 && J == 0) {
        // the step that this kick completes
        const int64_t step = S.st->step + 1;
        S.st->step = step;
        clear_counts(S, step);
    }
}

// a = G m (sum of the element's own chunk partials, then the reactions of every band with a
// row before the element's tile, in band order). KICK (in a step): the element's second kick and the
// tile's record follow (kick_record); otherwise a goes to the element's own index. KR is the
// system's band height. The element's terms (its cj chunk partials, then its ng band reactions)
// are cut into COMBINE_SEGS contiguous runs, one thread each; a run is a Kahan sum per component
// in term order, with the three components' loads issued together, eight terms at a time. The
// runs' results are then added in run order with Kahan compensation by the element's first
// thread. The order of every addition depends on the system's size alone.
template <int KR, bool KICK, bool MANY>
__device__ __forceinline__ void combine_tile(SysRef S, int J, int e, int k,
                                             int last, float (*part)[COMBINE_SEGS][TJ],
                                             double (*lds)[BT / 64])
{
    const int T = S.ntiles;
    const int slot = J * TJ + e;
    const int idx = glob<const int32_t>(S.perm)[slot];
    float x[3] = {0.f, 0.f, 0.f}, v0[3] = {0.f, 0.f, 0.f}, out[3] = {0.f, 0.f, 0.f};
    if (KICK && !MANY && k == 0 && idx >= 0) element_state(S, slot, x, v0);
    auto *P = glob<const float>(S.part);
    auto *R = glob<const float>(S.react);
    const size_t na = S.nalloc;
    const int own = J / KR;                           // the element's own band
    const int cj = (T - KR * own + S.ch - 1) / S.ch;  // its chunk count
    const int ng = (J + KR - 1) / KR;                 // bands with a row before J
    const int M = cj + ng;                            // terms
    const int t0 = (int)(((int64_t)M * k) / COMBINE_SEGS);
    const int t1 = (int)(((int64_t)M * (k + 1)) / COMBINE_SEGS);
    float sum[3] = {0.f, 0.f, 0.f}, comp[3] = {0.f, 0.f, 0.f};
    if (idx >= 0) {
        int t = t0;
        // chunk partials
        for (; t < min(t1, cj); ++t) {
            const size_t at = (size_t)t * 3 * na + slot;
            const float vx = P[at], vy = P[at + na], vz = P[at + 2 * na];
            kahan_add(sum[0], comp[0], vx);
            kahan_add(sum[1], comp[1], vy);
            kahan_add(sum[2], comp[2], vz);
        }
        // band reactions: band g's block starts at 3 TJ (g (T - 1) - KR g (g - 1) / 2) and holds
        // three components of (T - KR g - 1) TJ values; the element's value sits at slot -
        // TJ (KR g + 1) inside each
        int g = t - cj;
        const int g1 = t1 - cj;
        if (g < g1) {
            size_t off = react_group_offset(g, T, KR);
            size_t len = (size_t)(T - KR * g - 1) * TJ;
            for (; g + 8 <= g1; g += 8) {
                float v[8][3];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const size_t at = off + slot - (size_t)TJ * (KR * (g + q) + 1);
                    v[q][0] = R[at];
                    v[q][1] = R[at + len];
                    v[q][2] = R[at + 2 * len];
                    off += 3 * len;
                    len -= (size_t)KR * TJ;
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    kahan_add(sum[0], comp[0], v[q][0]);
                    kahan_add(sum[1], comp[1], v[q][1]);
                    kahan_add(sum[2], comp[2], v[q][2]);
                }
            }
            for (; g < g1; ++g) {
                const size_t at = off + slot - (size_t)TJ * (KR * g + 1);
                kahan_add(sum[0], comp[0], R[at]);
                kahan_add(sum[1], comp[1], R[at + len]);
                kahan_add(sum[2], comp[2], R[at + 2 * len]);
                off += 3 * len;
                len -= (size_t)KR * TJ;
            }
        }
    }
    if (KICK && MANY && k == 0 && idx >= 0) element_state(S, slot, x, v0);
#pragma unroll
    for (int d = 0; d < 3; ++d) part[d][k][e] = sum[d] - comp[d];
    __syncthreads();
    if (k == 0 && idx >= 0) {
        const float gm = glob<DevState>(S.st)->gm_f;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            float s = part[d][0][e], c = 0.f;
#pragma unroll
            for (int q = 1; q < COMBINE_SEGS; ++q) kahan_add(s, c, part[d][q][e]);
            out[d] = gm * (s - c);
        }
        if (!KICK || last) {
            glob<float>(S.ax)[idx] = out[0];
            glob<float>(S.ay)[idx] = out[1];
            glob<float>(S.az)[idx] = out[2];
        }
    }
    if constexpr (KICK) kick_record<float>(S, J, idx, x, v0, out, last, lds);
    __syncthreads();  // part and lds are rewritten by the block's next tile
}

// MANY (more tiles than CUs): 64 registers, so that two workgroups share a CU; with 76 the 258 tiles of
// 65,536 elements took two rounds (25 us a launch against 23, a batch of 24 systems of 4,096 to
// 32,768 1125 us a step against 1118). Up to one tile per CU the element's state is loaded
// ahead of the sums and the registers are free: 34.5 us a step at 7,500 elements against 37.0.
template <bool KICK, bool MANY>
__global__ __launch_bounds__(BT * COMBINE_SEGS) __attribute__((amdgpu_waves_per_eu(MANY ? 8 : 4)))
void k_combine_sym(Launch L, int last)
{
    __shared__ float part[3][COMBINE_SEGS][TJ];
    __shared__ double lds[7][BT / 64];
    const int e = threadIdx.x % TJ, k = threadIdx.x / TJ;
    for (int u = blockIdx.x; u < L.total_tunits; u += gridDim.x) {
        SysRef S = cst(L.sys)[find_tile_sys(L, u)];
        const int J = u - S.tunit_begin;
        switch (S.rows) {
        case 1: combine_tile<1, KICK, MANY>(S, J, e, k, last, part, lds); break;
        case 2: combine_tile<2, KICK, MANY>(S, J, e, k, last, part, lds); break;
        default: combine_tile<4, KICK, MANY>(S, J, e, k, last, part, lds); break;
        }
    }
}

// ------------------------------------------------------------------ FP64 force kernel

// FP64 reciprocal square root and reciprocal from the hardware estimates, each refined by one
// correction of higher order instead of two Newton steps. With e the estimate's residual,
// 1 / sqrt(x) = y (1 - e)^(-1/2) = y (1 + e/2 + 3 e^2/8 + ...) and 1 / b = y (1 - e)^(-1) =
// y (1 + e + e^2 + ...); the estimates' relative error measures below 2^-24 on this part, so
// the truncated terms are below 2^-70 and the results lie within an ulp of the exact values
// (measured over 1.7e7 arguments from 1e-200 to 1e300: at most 0.99 ulp for the square root,
// 0.50 for the reciprocal, tighter than two Newton steps' 1.75 and 0.50). Every argument the
// kernels pass is normal, with a normal result.
__device__ __forceinline__ double rsqrt_f64(double r2)
{
    const double y = __builtin_amdgcn_rsq(r2);
    const double e = fma(-r2 * y, y, 1.0);  // 1 - r2 y^2
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

__device__ __forceinline__ double rcp_f64(double b)
{
    const double y = __builtin_amdgcn_rcp(b);
    const double e = fma(-b, y, 1.0);  // 1 - b y
    return fma(y, fma(e, e, e), y);
}

// Per-tile constants of the FP64 pair code, read once per tile: the pair class's element diameter
// and contact-law coefficients, and the eqs. (4)-(6) softening and overlap scales.
struct LawD {
    double D, c1, c2, eps, gc, gcb;
};

__device__ __forceinline__ LawD law_d(Const<DevState> *st, Const<LawState> *ls, int cls)
{
    LawD K;
    K.D = cls == 0 ? st->D1 : (cls == 2 ? ls->D2 : 0.5 * (st->D1 + ls->D2));
    K.c1 = ls->c1d[cls];
    K.c2 = ls->c2d[cls];
    K.eps = st->leps_d;
    K.gc = st->lgc_d;
    K.gcb = st->lgcb_d;
    return K;
}

// Pair scalar s = f / (G m^2 r) in FP64 (see pair_s); w = 1 / r. Under eqs. (4)-(6) the
// attraction w / t^2 takes the refined reciprocal of t^2 (rcp_f64) instead of an IEEE division
// (measured 12 % faster; the division's scaling and fix-up steps cost more than the reciprocal
// itself). Coincident elements (d = 0, r^2 = 1e-200 after the floor added in pair_s64_at) get a
// large but finite s under both laws (w = 1e100, s at most about 1e300 with eps = 0), so their
// term s d is exactly 0, the oracle's r = 0 rule.
template <int LAW, bool NEAR = true>
__device__ __forceinline__ double pair_s64(double r2, double w, double dx, double dy, double dz,
                                           double dvx, double dvy, double dvz, const LawD &K)
{
    if constexpr (LAW == 0) {
        const double w3 = w * w * w;
        return NEAR ? fmin(w3, K.c1 - K.c2 * w) : w3;
    } else {
        const double r = r2 * w;
        const double t = r + K.eps;
        double s = w * rcp_f64(t * t);
        if (NEAR && r < K.D) {
            const double dot = dvx * dx + dvy * dy + dvz * dz;
            const double g = dot < 0.0 ? K.gc : K.gcb;
            const double u = K.D - r;
            s -= g * u * u * (1.0 + 2.0 * K.D * w);
        }
        return s;
    }
}

// ------------------------------------------------------------------ FP64 combine

// k_combine_sym's FP64 counterpart for bands of one row: the same runs, in plain FP64 (a run's
// terms in order, then the runs in order). One thread per element left two waves per SIMD at
// 50,021 elements, each waiting for one read after the other: 62 us, 1.9 TB/s; four take 29 us, 4.1 TB/s.
template <bool KICK>
__global__ __launch_bounds__(BT * COMBINE_SEGS) void k_combine_sym64(Launch L, int last)
{
    __shared__ double part[3][COMBINE_SEGS][TJ];
    __shared__ double lds[7][BT / 64];
    const int e = threadIdx.x % TJ, k = threadIdx.x / TJ;
    for (int u = blockIdx.x; u < L.total_tunits; u += gridDim.x) {
        SysRef S = cst(L.sys)[find_tile_sys(L, u)];
        const int J = u - S.tunit_begin;
        const int T = S.ntiles;
        const int slot = J * TJ + e;
        const int idx = glob<const int32_t>(S.perm)[slot];
        auto *P = glob<const double>(S.part);
        auto *R = glob<const double>(S.react);
        const size_t na = S.nalloc;
        const int cj = (T - J + S.ch - 1) / S.ch;  // the chunk count of the element's own row
        const int M = cj + J;
        double x[3] = {0, 0, 0}, v0[3] = {0, 0, 0}, out[3] = {0, 0, 0};
        if (KICK && k == 0 && idx >= 0) element_state(S, slot, x, v0);
        const int t0 = (int)(((int64_t)M * k) / COMBINE_SEGS);
        const int t1 = (int)(((int64_t)M * (k + 1)) / COMBINE_SEGS);
        double sum[3] = {0.0, 0.0, 0.0};
        if (idx >= 0) {
            int t = t0;
            for (; t < min(t1, cj); ++t) {
                const size_t at = (size_t)t * 3 * na + slot;
#pragma unroll
                for (int d = 0; d < 3; ++d) sum[d] += P[at + d * na];
            }
            int g = t - cj;
            const int g1 = t1 - cj;
            if (g < g1) {
                size_t off = react_group_offset(g, T, 1);
                size_t len = (size_t)(T - g - 1) * TJ;
                for (; g + 8 <= g1; g += 8) {
                    double v[8][3];
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const size_t at = off + slot - (size_t)TJ * (g + q + 1);
#pragma unroll
                        for (int d = 0; d < 3; ++d) v[q][d] = R[at + d * len];
                        off += 3 * len;
                        len -= TJ;
                    }
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
#pragma unroll
                        for (int d = 0; d < 3; ++d) sum[d] += v[q][d];
                    }
                }
                for (; g < g1; ++g) {
                    const size_t at = off + slot - (size_t)TJ * (g + 1);
#pragma unroll
                    for (int d = 0; d < 3; ++d) sum[d] += R[at + d * len];
                    off += 3 * len;
                    len -= TJ;
                }
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) part[d][k][e] = sum[d];
        __syncthreads();
        if (k == 0 && idx >= 0) {
            const double gm = glob<DevState>(S.st)->gm_d;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                double t = part[d][0][e];
#pragma unroll
                for (int q = 1; q < COMBINE_SEGS; ++q) t += part[d][q][e];
                out[d] = gm * t;
            }
            if (!KICK || last) {
                glob<double>(S.ax)[idx] = out[0];
                glob<double>(S.ay)[idx] = out[1];
                glob<double>(S.az)[idx] = out[2];
            }
        }
        if constexpr (KICK) kick_record<double>(S, J, idx, x, v0, out, last, lds);
        __syncthreads();  // part and lds are rewritten by the block's next tile
    }
}

// ------------------------------------------------------------------ leap-frog and L1 plane

// Optional second kick v += a dt/2, then per-unit FP64 sums of each star's positions and the
// count of non-finite elements. In the steps of a one-sided system the force kernel does this, in those
// of the symmetric kernels the combine.
template <typename T>
__global__ __launch_bounds__(BT) void k_kick_stats(Launch L, int do_kick)
{
    __shared__ double lds[7][BT / 64];
    for (int u = blockIdx.x; u < L.total_ounits; u += gridDim.x) {
        SysRef S = cst(L.sys)[find_sys(L, u, true)];
        if (do_kick && S.one_sided) continue;
        const int local = u - S.ounit_begin;
        const int i = local * BT + threadIdx.x;
        double v[7] = {0, 0, 0, 0, 0, 0, 0};
        if (i < S.n) {
            auto *vx = glob<T>(S.vx), *vy = glob<T>(S.vy),
              *vz = glob<T>(S.vz);
            T wx = vx[i], wy = vy[i], wz = vz[i];
            if (do_kick) {
                const T h = h_of<T>(glob<const DevState>(S.st));
                wx = wx + h * glob<const T>(S.ax)[i];
                wy = wy + h * glob<const T>(S.ay)[i];
                wz = wz + h * glob<const T>(S.az)[i];
                vx[i] = wx;
                vy[i] = wy;
                vz[i] = wz;
            }
            add_stats(v, glob<const T>(S.x)[i], glob<const T>(S.y)[i],
                      glob<const T>(S.z)[i], wx, wy, wz, i >= S.n1);
        }
        block_sum<7>(v, lds);
        if (threadIdx.x == 0) {
            auto *r = glob<double>(S.rec) + (size_t)local * REC_STRIDE;
            for (int k = 0; k < 7; ++k) r[k] = v[k];
            if (do_kick && local == 0) {
                // the step that this kick completes
                const int64_t step = S.st->step + 1;
                S.st->step = step;
                clear_counts(S, step);
            }
        }
    }
}

// ------------------------------------------------------------------ end of a step

// Star centres and L1 plane.
struct Plane {
    double com1[3], com2[3], e[3], xi_cut;
    int ok;
};

// The system's records summed by one workgroup, in the same order wherever it is done.
__device__ __forceinline__ void sum_records(SysRef S, int first, int n_rec, double (&v)[7],
                                            double (*lds)[BT / 64])
{
    for (int k = 0; k < 7; ++k) v[k] = 0.0;
    for (int u = threadIdx.x; u < n_rec; u += BT) {
        auto *r = glob<const double>(S.rec) + (size_t)(first + u) * REC_STRIDE;
        for (int k = 0; k < 7; ++k) v[k] += r[k];
    }
    block_sum<7>(v, lds);
}

__device__ __forceinline__ void plane_of(SysRef S, const double (&v)[7], Plane &p)
{
    const int n1 = S.n1, n2 = S.n - S.n1;
    for (int d = 0; d < 3; ++d) {
        p.com1[d] = n1 > 0 ? v[d] / (double)n1 : 0.0;
        p.com2[d] = n2 > 0 ? v[3 + d] / (double)n2 : 0.0;
        p.e[d] = p.com2[d] - p.com1[d];
    }
    const double dist = sqrt(p.e[0] * p.e[0] + p.e[1] * p.e[1] + p.e[2] * p.e[2]);
    p.ok = (n1 > 0 && n2 > 0 && dist > 0.0) ? 1 : 0;
    for (int d = 0; d < 3; ++d) p.e[d] = p.ok ? p.e[d] / dist : 0.0;
    p.xi_cut = glob<DevState>(S.st)->xi_l1 * dist;
}

// The donor growth update with the derived force constants: `to` is `from` after one more step.
__device__ __forceinline__ void grow(const DevState *st, const LawState *from, LawState *to)
{
    LawState w = *from;
    if (st->growth_on && !w.growth_stopped) {
        const double R2 = st->R2_0 * w.D2 / st->D2_0;
        if (R2 <= st->rL_a) {
            w.D2 = w.D2 * (1.0 + st->growth_rate);
            const double Ds[3] = {st->D1, 0.5 * (st->D1 + w.D2), w.D2};
            for (int k = 0; k < 3; ++k) {
                const double D = Ds[k];
                w.c1d[k] = 11.0 / (D * D * D);
                w.c2d[k] = 10.0 / (D * D);
                w.c1f[k] = (float)w.c1d[k];
                w.c2f[k] = (float)w.c2d[k];
                w.far2f[k] = far_limit(D);
                w.lD_f[k] = (float)D;
            }
        } else {
            w.growth_stopped = 1;
        }
    }
    *to = w;
}

// Records the plane and the non-finite count, and (optionally) grows the donor. Called by one thread
// of a system.
__device__ __forceinline__ void finish_step(SysRef S, const Plane &p, double nonfinite,
                                            int do_growth)
{
    DevState *st = S.st;
    for (int d = 0; d < 3; ++d) {
        st->com1[d] = p.com1[d];
        st->com2[d] = p.com2[d];
        st->e[d] = p.e[d];
    }
    st->xi_cut = p.xi_cut;
    st->plane_ok = p.ok;
    st->nonfinite = (int32_t)nonfinite;
    if (do_growth) grow(st, &st->cur, &st->cur);
}

struct FinishMem {
    double lds[7][BT / 64];
    Plane pl;
    int cnt[3][BT / 64];
};

// Donor elements' side of the plane and the crossings since the last step, for the element i of this
// lane at (px, py, pz); the plane is in m.pl. The counts are whole numbers, added atomically to
// `total` (null: not kept) and `row` (null: not kept), so their order does not matter.
template <typename T>
__device__ __forceinline__ void classify(SysRef S, int i, T px, T py, T pz, FinishMem &m, bool init,
                                         int32_t *total, int32_t *row)
{
    bool past = false, fwd = false, bwd = false;
    if (i < S.n && i >= S.n1) {
        const double xi = ((double)px - m.pl.com1[0]) * m.pl.e[0] +
                          ((double)py - m.pl.com1[1]) * m.pl.e[1] +
                          ((double)pz - m.pl.com1[2]) * m.pl.e[2];
        past = m.pl.ok && xi < m.pl.xi_cut;
        const int8_t now = past ? 1 : 0;
        int8_t old = 2;
        if (!init) {
            old = glob<int8_t>(S.side)[i];
            fwd = past && old == 0;
            bwd = !past && old != 0;
        }
        if (old != now) glob<int8_t>(S.side)[i] = now;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = __popcll(__ballot(past)), c1 = __popcll(__ballot(fwd)), c2 = __popcll(__ballot(bwd));
    if (lane == 0) {
        m.cnt[0][wave] = c0;
        m.cnt[1][wave] = c1;
        m.cnt[2][wave] = c2;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int k = threadIdx.x;
        const int c = m.cnt[k][0] + m.cnt[k][1] + m.cnt[k][2] + m.cnt[k][3];
        if (c != 0) {
            if (total) atomicAdd(total + k, c);
            if (row) atomicAdd(row + k, c);
        }
    }
}

// ------------------------------------------------------------------ one-sided force kernel
//
// Small systems (FP32 Kahan and FP64 modes; see the runtime's one_sided rule): every ordered pair, in
// element order, with nothing between the drift and the second kick but this kernel. A workgroup
// takes the system's ib elements i of one star (the runtime's one_sided_ib rule), all of them in
// every lane's registers, and its 256 lanes share out the j: lane t takes j = t, t + 256, ..., so a j
// is read once per workgroup, straight from memory, for ib pairs. Each lane's sums (at most n / 256
// terms per element) are added across the wave by a halving exchange and across the waves in
// order: the same order for every ib. In a step the elements then take their second kick and, at
// once, the next step's kick and drift into a set of their own (others still read this step's), the
// workgroup stores its record of the step, and further workgroups end the step before (its plane
// and counts). So a step is one launch: ten steps of 2,048 elements take 70 us; with the drift and
// the counts as a kernel of their own between the evaluations they took 132, and with every
// workgroup drifting all j itself, from three times the loads, 90 (but 326 against 312 at 7,001,
// where this one takes 221). The symmetric kernels need half the pairs, but also a sorted copy,
// reactions, a combine and the kick as kernels of their own, and one 256 x 256 tile pair takes a
// wave about 5000 instructions one after the other: 2,048 elements are 45 such units on 256 CUs.
// What bounds it: at 2,048 elements a launch and one workgroup's chain of loads, pairs and sums
// (7 us a step); at 7,001 FP32 issue, at 2,980 pairs a nanosecond. Taking all ib pairs through each
// operation together instead of one after the other changed nothing, eqs. (4)-(6) 5 to 25 % slower.
// The law is taken in its near form for every pair (the far form gives the same bits).

template <typename T>
struct OneSidedLaw;
template <>
struct OneSidedLaw<float> {
    LawF k;
    __device__ __forceinline__ void load(Const<DevState> *st, Const<LawState> *ls, int cls)
    {
        k = law_f(st, ls, cls);
        // in vector registers: a choice between two of them takes one instruction
        asm("" : "+v"(k.c1), "+v"(k.nc2));
    }
};
template <>
struct OneSidedLaw<double> {
    LawD k;
    __device__ __forceinline__ void load(Const<DevState> *st, Const<LawState> *ls, int cls)
    {
        k = law_d(st, ls, cls);
    }
};

template <int LAW>
__device__ __forceinline__ float one_sided_s(float dx, float dy, float dz, const float4 &vj,
                                             const float4 &vi, const LawF &K)
{
    float eps;  // in a vector register: a literal halves the issue rate
    asm("v_mov_b32 %0, 0x179abe15" : "=v"(eps));  // 1e-24
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps)));
    return pair_s<LAW, true>(r2, dx, dy, dz, vj, vi, K);
}

template <int LAW>
__device__ __forceinline__ double one_sided_s(double dx, double dy, double dz, const double4 &vj,
                                              const double4 &vi, const LawD &K)
{
    const double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, 1.0e-200)));
    return pair_s64<LAW>(r2, rsqrt_f64(r2), dx, dy, dz, vj.x - vi.x, vj.y - vi.y, vj.z - vi.z, K);
}

template <typename T>
struct Vec4;
template <>
struct Vec4<float> {
    using type = float4;
};
template <>
struct Vec4<double> {
    using type = double4;
};

template <int V>
struct Int {
    static constexpr int value = V;
};

// The power of two that holds IB.
constexpr int pow2_of(int ib) { return ib <= 1 ? 1 : (ib <= 2 ? 2 : (ib <= 4 ? 4 : 8)); }

// Sums IB elements' three values per lane over the wave: halves the elements that a lane holds at
// each of the first steps (elements beyond IB are zeros). With P = pow2_of(IB), on return lane l holds
// element l / (64 / P)'s three sums, summed over all lanes, in the same order for every IB.
template <typename T, int IB>
__device__ __forceinline__ void wave_reduce(const T (&in)[IB][3], T (&out)[3], int lane)
{
    constexpr int P = pow2_of(IB);
    T a[P][3];
#pragma unroll
    for (int k = 0; k < P; ++k) {
#pragma unroll
        for (int d = 0; d < 3; ++d) a[k][d] = k < IB ? in[k < IB ? k : 0][d] : (T)0;
    }
    int width = 32;
#pragma unroll
    for (int half = P / 2; half >= 1; half /= 2) {
        const bool upper = (lane & width) != 0;
#pragma unroll
        for (int k = 0; k < half; ++k) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const T keep = upper ? a[k + half][d] : a[k][d];
                const T give = upper ? a[k][d] : a[k + half][d];
                a[k][d] = keep + __shfl_xor(give, width, 64);
            }
        }
        width /= 2;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        T v = a[0][d];
        for (int w = width; w >= 1; w /= 2) v += __shfl_xor(v, w, 64);
        out[d] = v;
    }
}

// A step's beginning for one element: v' = v + a dt/2, x' = x + v' dt. The same operations wherever
// an element is worked out, so that every workgroup has the same x' of it.
template <typename T>
__device__ __forceinline__ void kick_drift(T h, T dt, T &x, T &v, T a)
{
    v = fma_t(h, a, v);
    x = fma_t(dt, v, x);
}

// One of the three sets (x, y, z, half-step vx, vy, vz) that hold the elements as step k's force sees
// them. Step k's workgroups read set k, leave set k + 1 and look back at set k - 1.
template <typename T>
__device__ __forceinline__ Glob<T> *step_set(SysRef S, int k)
{
    return glob<T>(S.alt) + (size_t)(k % 3) * 6 * S.nalloc;
}

// Workgroup `local` of a system: its IB elements i.
template <typename T>
__device__ __forceinline__ T at_byte(Glob<const T> *p, uint32_t offset)
{
    return *reinterpret_cast<Glob<const T> *>(reinterpret_cast<Glob<const char> *>(p) + offset);
}

// step 0: the forces at the current positions (nb_forces). step k >= 1: the k-th step of a call, from
// the drift to the next step's; the `last` one leaves the state in the caller's arrays.
template <typename T, int LAW, bool STEP, int IB>
__device__ __forceinline__ void one_sided_unit(SysRef S, int local, int step, int last, T (*part)[os_ib(sizeof(T) == 8, LAW)][3])
{
    using V4 = typename Vec4<T>::type;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool odd = (step & 1) != 0;
    const int n = S.n, n1 = S.n1;
    auto *st = cst(S.st);
    const size_t na = S.nalloc;
    auto *A = step_set<const T>(S, step);
    auto *X = STEP ? A : glob<const T>(S.x), *Y = STEP ? A + na : glob<const T>(S.y),
         *Z = STEP ? A + 2 * na : glob<const T>(S.z);
    auto *VX = STEP ? A + 3 * na : glob<const T>(S.vx), *VY = STEP ? A + 4 * na : glob<const T>(S.vy),
         *VZ = STEP ? A + 5 * na : glob<const T>(S.vz);
    // star 1's elements take the first ceil(n1 / IB) workgroups
    const int b1 = (n1 + IB - 1) / IB;
    const int istar = local >= b1 ? 1 : 0;
    const int i0 = istar ? n1 + (local - b1) * IB : local * IB;
    const int iend = istar ? n : n1;
    T xi[IB], yi[IB], zi[IB], acc[IB][3];
    V4 vi[LAW != 0 ? IB : 1];
#pragma unroll
    for (int k = 0; k < IB; ++k) {
        const int i = min(i0 + k, iend - 1);
        xi[k] = X[i];
        yi[k] = Y[i];
        zi[k] = Z[i];
        if constexpr (LAW != 0) vi[k] = V4{VX[i], VY[i], VZ[i], 0};
        acc[k][0] = acc[k][1] = acc[k][2] = 0;
    }
    // wave 0's lane k < IB finishes element i0 + k
    const int i = i0 + lane;
    const bool mine = wave == 0 && lane < IB && i < iend;
    T ox = 0, oy = 0, oz = 0, ovx = 0, ovy = 0, ovz = 0;
    if (STEP && mine) {
        ox = X[i];
        oy = Y[i];
        oz = Z[i];
        ovx = VX[i];
        ovy = VY[i];
        ovz = VZ[i];
    }
    auto *ls = !STEP || step == 1 ? &st->cur : &st->slot[odd ? 0 : 1];
    OneSidedLaw<T> Ka, Kb;
    Ka.load(st, ls, istar);
    Kb.load(st, ls, istar + 1);
    // UN j of the lane are fetched while the previous ones are worked on
    constexpr int UN = sizeof(T) == 4 ? (LAW == 0 ? 4 : (IB <= 6 ? 2 : 1)) : (LAW == 0 ? 2 : 1);
    T px[UN], py[UN], pz[UN];
    V4 pv[UN];
    auto fetch = [&](int j0) {
#pragma unroll
        for (int q = 0; q < UN; ++q) {
            // 32-bit offsets from uniform bases: one address for the lane's loads of a j
            const uint32_t at = (uint32_t)min(j0 + q * BT + tid, n - 1) * (uint32_t)sizeof(T);
            px[q] = at_byte(X, at);
            py[q] = at_byte(Y, at);
            pz[q] = at_byte(Z, at);
            pv[q] = V4{};
            if constexpr (LAW != 0) pv[q] = V4{at_byte(VX, at), at_byte(VY, at), at_byte(VZ, at), 0};
        }
    };
    fetch(0);
#pragma unroll 1
    for (int j0 = 0; j0 < n; j0 += UN * BT) {
        T xj[UN], yj[UN], zj[UN];
        V4 vj[UN];
#pragma unroll
        for (int q = 0; q < UN; ++q) {
            xj[q] = px[q];
            yj[q] = py[q];
            zj[q] = pz[q];
            vj[q] = pv[q];
        }
        if (j0 + UN * BT < n) fetch(j0 + UN * BT);
#pragma unroll
        for (int q = 0; q < UN; ++q) {
            const int j = j0 + q * BT + tid;
            if (j >= n) break;
            const auto K = j >= n1 ? Kb.k : Ka.k;
#pragma unroll
            for (int k = 0; k < IB; ++k) {
                const T dx = xj[q] - xi[k], dy = yj[q] - yi[k], dz = zj[q] - zi[k];
                T s = one_sided_s<LAW>(dx, dy, dz, vj[q], vi[LAW != 0 ? k : 0], K);
                // the self pair: d = 0 makes its term 0 under the contact law; the overlap term
                // of eqs. (4)-(6) is of order 1 / eps there
                if constexpr (LAW != 0) s = j - i0 == k ? (T)0 : s;
                acc[k][0] = fma_t(s, dx, acc[k][0]);
                acc[k][1] = fma_t(s, dy, acc[k][1]);
                acc[k][2] = fma_t(s, dz, acc[k][2]);
            }
        }
    }
    T sum[3];
    wave_reduce<T, IB>(acc, sum, lane);
    constexpr int LPE = 64 / pow2_of(IB);  // lanes that hold one element's sums
    if (lane % LPE == 0 && lane / LPE < IB) {
#pragma unroll
        for (int d = 0; d < 3; ++d) part[wave][lane / LPE][d] = sum[d];
    }
    __syncthreads();
    if (wave != 0) return;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    if (mine) {
        T a[3];
        const T gm = gm_of<T>(st);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            T t = part[0][lane][d];
#pragma unroll
            for (int w = 1; w < BT / 64; ++w) t += part[w][lane][d];
            a[d] = gm * t;
        }
        if (!STEP || last) {
            glob<T>(S.ax)[i] = a[0];
            glob<T>(S.ay)[i] = a[1];
            glob<T>(S.az)[i] = a[2];
        }
        if constexpr (STEP) {
            const T h = h_of<T>(st), dt = dt_of<T>(st);
            ovx = fma_t(h, a[0], ovx);
            ovy = fma_t(h, a[1], ovy);
            ovz = fma_t(h, a[2], ovz);
            add_stats(v, ox, oy, oz, ovx, ovy, ovz, istar != 0);
            if (last) {
                glob<T>(S.x)[i] = ox;
                glob<T>(S.y)[i] = oy;
                glob<T>(S.z)[i] = oz;
                glob<T>(S.vx)[i] = ovx;
                glob<T>(S.vy)[i] = ovy;
                glob<T>(S.vz)[i] = ovz;
            } else {
                kick_drift(h, dt, ox, ovx, a[0]);
                kick_drift(h, dt, oy, ovy, a[1]);
                kick_drift(h, dt, oz, ovz, a[2]);
                auto *N = step_set<T>(S, step + 1) + i;
                N[0] = ox;
                N[na] = oy;
                N[2 * na] = oz;
                N[3 * na] = ovx;
                N[4 * na] = ovy;
                N[5 * na] = ovz;
            }
        }
    }
    if constexpr (!STEP) return;
#pragma unroll
    for (int k = 0; k < 7; ++k) {
#pragma unroll
        for (int w = pow2_of(IB) / 2; w >= 1; w /= 2) v[k] += __shfl_xor(v[k], w, 64);
    }
    if (lane == 0) {
        auto *r = glob<double>(S.rec) + (size_t)((odd ? S.rec_len : 0) + local) * REC_STRIDE;
#pragma unroll
        for (int k = 0; k < 7; ++k) r[k] = v[k];
        if (local == 0) {
            DevState *w = S.st;
            const int64_t done = w->step + step;
            w->step_done = done;
            clear_counts(S, done);
            grow(w, step == 1 ? &w->cur : &w->slot[odd ? 0 : 1], &w->slot[odd ? 1 : 0]);
        }
    }
}

template <typename T, int LAW>
union OneSidedMem {
    T part[BT / 64][os_ib(sizeof(T) == 8, LAW)][3];
    FinishMem fin;
};

// Workgroup `block` of the one-sided systems, whose force units end before `end`.
template <typename T, int LAW, bool STEP>
__device__ __forceinline__ void one_sided_block(const Launch &L, int end, int block, int step, int last,
                                                OneSidedMem<T, LAW> &sh)
{
    constexpr int IB = os_ib(sizeof(T) == 8, LAW);
    const int tid = threadIdx.x;
    const bool odd = (step & 1) != 0;
    if (STEP && block >= end) {
        // the end of the step before: 256 elements' side of the L1 plane
        SysRef S = cst(L.sys)[find_sys(L, block - end, true)];
        if (!S.one_sided) return;  // an empty system
        const int local = block - end - S.ounit_begin;
        double v[7];
        sum_records(S, odd ? 0 : S.rec_len, S.n_rec, v, sh.fin.lds);
        if (tid == 0) plane_of(S, v, sh.fin.pl);
        __syncthreads();
        const int i = min(local * BT + tid, S.n - 1);
        const size_t na = S.nalloc;
        auto *A = step_set<const T>(S, step - 1);
        classify(S, local * BT + tid, (T)A[i], (T)A[na + i], (T)A[2 * na + i], sh.fin, false, nullptr,
                 log_row(S, cst(S.st)->step + step - 1) + 1);
        return;
    }
    SysRef S = cst(L.sys)[find_sys(L, block, false)];
    const int local = block - S.unit_begin;
    auto run = [&](auto ib) {
        one_sided_unit<T, LAW, STEP, decltype(ib)::value>(S, local, step, last, sh.part);
    };
    switch (S.ib) {
    case 2:
        if constexpr (sizeof(T) == 8) run(Int<2>{});
        break;
    case 3:
        if constexpr (sizeof(T) == 8) run(Int<3>{});
        break;
    case 4: run(Int<4>{}); break;
    case 5:
        if constexpr (IB >= 5) run(Int<5>{});
        break;
    case 6:
        if constexpr (IB >= 6) run(Int<6>{});
        break;
    case 7:
        if constexpr (IB >= 7) run(Int<7>{});
        break;
    case 8:
        if constexpr (IB >= 8) run(Int<8>{});
        break;
    }
}

// LOOP: a persistent launch, each workgroup takes units blockIdx, blockIdx + grid, .. of `total`. A kernel
// of its own: the loop costs 15 to 33 registers, a wave per SIMD.
template <typename T, int LAW, bool STEP, bool LOOP>
__global__ __launch_bounds__(BT) void k_force_one_sided(Launch L, int step, int last, int total)
{
    __shared__ OneSidedMem<T, LAW> sh;
    if constexpr (LOOP) {
        for (int b = blockIdx.x; b < total; b += gridDim.x) {
            one_sided_block<T, LAW, STEP>(L, L.total_units, b, step, last, sh);
            __syncthreads();  // sh is rewritten by the next
        }
    } else {
        one_sided_block<T, LAW, STEP>(L, L.total_units, blockIdx.x, step, last, sh);
    }
}

template <typename T, int LAW>
static hipError_t launch_one_sided(const Launch &L, int step, int last, int max_blocks, hipStream_t s)
{
    // from a call's second step on also one unit per 256 elements for the end of the step before
    const int total = L.total_units + (step > 1 ? L.ounit_base : 0);
    const bool loop = max_blocks > 0 && max_blocks < total;
    const auto k = step > 0 ? (loop ? k_force_one_sided<T, LAW, true, true> : k_force_one_sided<T, LAW, true, false>)
                            : (loop ? k_force_one_sided<T, LAW, false, true> : k_force_one_sided<T, LAW, false, false>);
    hipLaunchKernelGGL(k, dim3(loop ? max_blocks : total), dim3(BT), 0, s, L, step, last, total);
    return hipGetLastError();
}

// ------------------------------------------------------------------ symmetric force kernel: code

template <typename T>
struct RowsMem;  // one wave's staged j, each stored twice so that a rotating read never wraps
template <>
struct RowsMem<float> {
    float4 p[128];
    __device__ __forceinline__ void put(int lane, float x, float y, float z)
    {
        p[lane] = p[lane + 64] = make_float4(x, y, z, 0.0f);
    }
    __device__ __forceinline__ float4 get(int k) const { return p[k]; }
};
template <>
struct RowsMem<double> {
    double2 p[128];
    double q[128];
    __device__ __forceinline__ void put(int lane, double x, double y, double z)
    {
        p[lane] = p[lane + 64] = make_double2(x, y);
        q[lane] = q[lane + 64] = z;
    }
    __device__ __forceinline__ double4 get(int k) const
    {
        const double2 a = p[k];
        return make_double4(a.x, a.y, q[k], 0.0);
    }
};

__device__ __forceinline__ double xbar_ror1(double v, int addr)
{
    const int lo = __builtin_amdgcn_ds_bpermute(addr, __double2loint(v));
    const int hi = __builtin_amdgcn_ds_bpermute(addr, __double2hiint(v));
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ LawF law_of(Const<DevState> *st, int cls, float)
{
    return law_uniform(law_f(st, &st->cur, cls));
}
__device__ __forceinline__ LawD law_of(Const<DevState> *st, int cls, double)
{
    return law_d(st, &st->cur, cls);
}

template <int LAW, bool NEAR>
__device__ __forceinline__ float pair_at(float dx, float dy, float dz, const float4 &vj,
                                         const float4 &vi, const LawF &K)
{
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, 1.0e-24f)));
    return pair_s<LAW, NEAR>(r2, dx, dy, dz, vj, vi, K);
}
template <int LAW, bool NEAR>
__device__ __forceinline__ double pair_at(double dx, double dy, double dz, const double4 &vj,
                                          const double4 &vi, const LawD &K)
{
    const double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, 1.0e-200)));
    return pair_s64<LAW, NEAR>(r2, rsqrt_f64(r2), dx, dy, dz, vj.x - vi.x, vj.y - vi.y,
                               vj.z - vi.z, K);
}

// The band's elements of one lane.
template <typename T, int NI>
struct Rows {
    T x[NI], y[NI], z[NI], a[NI][3];
};

// The wave's 64 j against the elements [K0, K0 + NK) of every lane, with (REACT) their reaction added
// to aj, or one-sided (a row's own tile, where the self pair is at step 0 of element K0 + wave).
// vi: the elements' half-step velocities (eqs. 4-6, near form only).
// Two rows in FP32: a reaction is summed in four runs of 16 steps (128 terms), added in order through
// `runs`, because a running FP32 sum loses with its length what no later compensation brings back.
// With one run of 512 terms the forces at 32,768 elements were off by 7.3e-8 of the largest (root
// mean square; 6.6e-8 with the four waves' runs of 256 of the kernel before), so 4.3e-8, for half a
// percent (10.46 -> 10.51 ms a step at 262,144, 1419 -> 1426 us for two at 65,536). One row's single
// run of 256 terms stays below that kernel's error, and the same cut would cost it 2 % (700 -> 716 us,
// two steps of 40,009 elements under eqs. (4)-(6)).
template <typename T, int LAW, int NI, int K0, int NK, bool NEAR, bool REACT, typename Law, typename V4>
__device__ __forceinline__ void rows_tile(const RowsMem<T> &P, const RowsMem<T> &V, Rows<T, NI> &B,
                                          const Law *K, const V4 *vi, int lane, int wave,
                                          T (*runs)[64], T (&aj)[3])
{
    // (unrolled, the near form of eqs. (4)-(6) with its branches spills inside the loop)
    constexpr int U = LAW != 0 && NEAR ? 1 : (sizeof(T) == 4 ? 4 : 2);
    constexpr int RUN = sizeof(T) == 4 && NI > 4 ? 16 : 64;  // steps
    const int rot_addr = ((lane + 63) & 63) << 2;  // byte address of lane l - 1 (mod 64)
    T run[3] = {0, 0, 0};
    V4 p = P.get(lane + 64);
#pragma unroll 1
    for (int q0 = 0; q0 < 64; q0 += RUN) {
#pragma unroll 1
        for (int s0 = q0; s0 < q0 + RUN; s0 += U) {
            const int at = lane + 64 - s0 - U;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const V4 pn = P.get(at + U - u - 1);
                V4 vj{};
                if constexpr (LAW != 0 && NEAR) vj = V.get(at + U - u);
#pragma unroll
                for (int k = K0; k < K0 + NK; ++k) {
                    const T dx = p.x - B.x[k], dy = p.y - B.y[k], dz = p.z - B.z[k];
                    V4 v{};
                    if constexpr (LAW != 0 && NEAR) v = vi[k - K0];
                    T s = pair_at<LAW, NEAR>(dx, dy, dz, vj, v, K[k / 4]);
                    if constexpr (LAW != 0 && !REACT)
                        s = u == 0 && s0 == 0 && k - K0 == wave ? (T)0 : s;
                    B.a[k][0] = fma_t(s, dx, B.a[k][0]);
                    B.a[k][1] = fma_t(s, dy, B.a[k][1]);
                    B.a[k][2] = fma_t(s, dz, B.a[k][2]);
                    if constexpr (REACT) {
                        run[0] = fma_t(s, dx, run[0]);
                        run[1] = fma_t(s, dy, run[1]);
                        run[2] = fma_t(s, dz, run[2]);
                    }
                    if constexpr (LAW == 0 && sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (sizeof(T) == 4) asm volatile("" ::"v"(p.w));
                if constexpr (REACT) {
#pragma unroll
                    for (int d = 0; d < 3; ++d) run[d] = xbar_ror1(run[d], rot_addr);
                }
                p = pn;
            }
        }
        if constexpr (REACT) {
            // the lane holds the run of element l - q0 - RUN, in the end its own
            const int e = (lane - q0 - RUN) & 63;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const T t = q0 == 0 ? run[d] : runs[d][e] + run[d];
                if (q0 + RUN < 64) {
                    runs[d][e] = t;
                    run[d] = 0;
                } else {
                    aj[d] += t;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// The near form of the band's rows r0, r0 + 1, .. against tile k of the band's tiles (k >= R: a tile
// after the band): the rows before tile k with reactions, row k one-sided.
template <typename T, int LAW, int R, int r0, typename Law>
__device__ __forceinline__ void near_rows(SysRef S, const RowsMem<T> &P,
                                          const RowsMem<T> &V, Rows<T, 4 * R> &B, const Law *K,
                                          int I0, int k, int lane, int wave, T (*runs)[64],
                                          T (&aj)[3])
{
    using V4 = typename Vec4<T>::type;
    if (r0 <= k) {
        V4 vi[4];
        if constexpr (LAW != 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int slot = (I0 + r0) * TJ + 64 * q + lane;
                vi[q].x = glob<const T>(S.vxs)[slot];
                vi[q].y = glob<const T>(S.vys)[slot];
                vi[q].z = glob<const T>(S.vzs)[slot];
                vi[q].w = 0;
            }
        }
        if (r0 == k) {
            T none[3] = {0, 0, 0};
            rows_tile<T, LAW, 4 * R, 4 * r0, 4, true, false, Law, V4>(P, V, B, K, vi, lane, wave,
                                                                      runs, none);
        } else {
            rows_tile<T, LAW, 4 * R, 4 * r0, 4, true, true, Law, V4>(P, V, B, K, vi, lane, wave,
                                                                     runs, aj);
        }
    }
    if constexpr (r0 + 1 < R) near_rows<T, LAW, R, r0 + 1>(S, P, V, B, K, I0, k, lane, wave, runs, aj);
}

// R rows of a unit: rows I0 .. I0 + R - 1 of band grp (BAND rows high) against chunk c of the band's
// tiles. Where the band's rows before I0 have left reactions, these rows' are added to them.
template <typename T, int LAW, int R, int BAND>
__device__ __forceinline__ void rows_unit(SysRef S, int grp, int I0, int c, RowsMem<T> *mem,
                                          T (*runs)[3][64], T (*red)[3][TJ])
{
    constexpr int NI = 4 * R;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto *st = cst(S.st);
    auto *XS = glob<const T>(S.xs), *YS = glob<const T>(S.ys), *ZS = glob<const T>(S.zs);
    auto *VXS = glob<const T>(S.vxs), *VYS = glob<const T>(S.vys), *VZS = glob<const T>(S.vzs);
    const int ntiles = S.ntiles;
    const int G0 = BAND * grp;           // the band's first row
    const int nv = min(R, ntiles - I0);  // rows inside the system (the last band may be short)
    using V4 = typename Vec4<T>::type;
    Rows<T, NI> B;
    using Law = decltype(law_of(st, 0, (T)0));
    Law Ka[R], Kb[R];
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    float far2a = 0.0f, far2b = 0.0f;
    T sum[NI][3], comp[sizeof(T) == 4 ? NI : 1][3];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int row = r < nv ? I0 + r : I0;  // a missing row mirrors row 0 and stays unused
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 4 * r + q, slot = row * TJ + 64 * q + lane;
            B.x[k] = XS[slot];
            B.y[k] = YS[slot];
            B.z[k] = ZS[slot];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                B.a[k][d] = sum[k][d] = 0;
                if constexpr (sizeof(T) == 4) comp[k][d] = 0;
            }
        }
        auto *bx = cst(S.tbox) + (size_t)row * 8;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lo[d] = fminf(lo[d], bx[d]);
            hi[d] = fmaxf(hi[d], bx[4 + d]);
        }
        const int istar = row * TJ >= S.p1 ? 1 : 0;
        Ka[r] = law_of(st, istar, (T)0);
        Kb[r] = law_of(st, istar + 1, (T)0);
        far2a = fmaxf(far2a, st->cur.far2f[istar]);
        far2b = fmaxf(far2b, st->cur.far2f[istar + 1]);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = wave_uniform(lo[d]);
        hi[d] = wave_uniform(hi[d]);
    }
    far2a = wave_uniform(far2a);
    far2b = wave_uniform(far2b);
    RowsMem<T> &P = mem[wave], &V = mem[LAW != 0 ? 4 + wave : wave];
    auto *RE = glob<T>(S.react);
    const size_t roff = react_group_offset(grp, ntiles, BAND);
    const size_t rlen = (size_t)(ntiles - G0 - 1) * TJ;
    const int t1 = min(ntiles, G0 + (c + 1) * S.ch);
    const int t0 = max(I0, G0 + c * S.ch);  // the rows' own pairs begin at their own tile
    T px = 0, py = 0, pz = 0, qx = 0, qy = 0, qz = 0;
    auto fetch = [&](int t) {
        const int slot = t * TJ + 64 * wave + lane;
        px = XS[slot];
        py = YS[slot];
        pz = ZS[slot];
        if constexpr (LAW != 0) {
            qx = VXS[slot];
            qy = VYS[slot];
            qz = VZS[slot];
        }
    };
    if (t0 < t1) fetch(t0);
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
        P.put(lane, px, py, pz);
        if constexpr (LAW != 0) V.put(lane, qx, qy, qz);
        // one wave writes and reads its own part of LDS, in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (t + 1 < t1) fetch(t + 1);
        const bool jstar = t * TJ >= S.p1;
        Law K[R];
#pragma unroll
        for (int r = 0; r < R; ++r) K[r] = jstar ? Kb[r] : Ka[r];
        const int k = t - I0;  // tile t is one of these rows when k < R
        const size_t at = roff + (size_t)(t - G0 - 1) * TJ + 64 * wave + lane;
        T aj[3] = {0, 0, 0}, old[3] = {0, 0, 0};
        if (BAND > R && k > 0 && I0 > G0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) old[d] = RE[at + d * rlen];
        }
        if (k >= R && far_tile(cst(S.tbox) + (size_t)t * 8, lo, hi,
                               jstar ? far2b : far2a)) {
            rows_tile<T, LAW, NI, 0, NI, false, true, Law, V4>(P, V, B, K, nullptr, lane, wave,
                                                                 runs[wave], aj);
        } else if (LAW == 0 && k >= R) {
            rows_tile<T, LAW, NI, 0, NI, true, true, Law, V4>(P, V, B, K, nullptr, lane, wave,
                                                                 runs[wave], aj);
        } else {
            // one row at a time, so that only a row's velocities are held
            near_rows<T, LAW, R, 0>(S, P, V, B, K, I0, k, lane, wave, runs[wave], aj);
        }
        if (k > 0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) RE[at + d * rlen] = old[d] - aj[d];
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                if constexpr (sizeof(T) == 4) {
                    kahan_add(sum[i][d], comp[i][d], B.a[i][d]);
                } else {
                    sum[i][d] += B.a[i][d];
                }
                B.a[i][d] = 0;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    // the waves' sums of each element, in wave order
    auto *PA = glob<T>(S.part);
    const size_t na = S.nalloc;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        __syncthreads();  // red is the staging memory of the loop
        if (r < nv) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    T v = sum[4 * r + q][d];
                    if constexpr (sizeof(T) == 4) v -= comp[4 * r + q][d];
                    red[wave][d][64 * q + lane] = v;
                }
            }
        }
        __syncthreads();
        const int slot = (I0 + r) * TJ + tid;
        if (r < nv && glob<const int32_t>(S.perm)[slot] >= 0) {
            const size_t b = (size_t)c * 3 * na + slot;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                T v = red[0][d][tid];
                if constexpr (sizeof(T) == 4) {
                    T e = 0;
#pragma unroll
                    for (int w = 1; w < 4; ++w) kahan_add(v, e, red[w][d][tid]);
                    v -= e;
                } else {
                    v = ((v + red[1][d][tid]) + red[2][d][tid]) + red[3][d][tid];
                }
                PA[b + d * na] = v;
            }
        }
    }
    __syncthreads();  // the next unit's staging
}

template <typename T, int LAW, int R, int BAND = R>
__global__ __launch_bounds__(BT) __attribute__((amdgpu_waves_per_eu(rows_waves(sizeof(T) == 8, LAW, R))))
void k_force_rows(Launch L)
{
    union Shared {
        struct {
            RowsMem<T> mem[LAW == 0 ? 4 : 8];
            T runs[R > 1 ? 4 : 1][3][64];
        } w;
        T red[4][3][TJ];
    };
    __shared__ __attribute__((aligned(16))) char raw[sizeof(Shared)];
    Shared &sh = *reinterpret_cast<Shared *>(raw);
    for (int u = L.unit_base + blockIdx.x; u < L.total_units; u += gridDim.x) {
        SysRef S = cst(L.sys)[find_sys(L, u, false)];
        const auto *gc = cst(S.units) + 2 * (size_t)(u - S.unit_begin);
        const int grp = gc[0], c = gc[1];
        if constexpr (BAND == R) {
            rows_unit<T, LAW, R, BAND>(S, grp, R * grp, c, sh.w.mem, sh.w.runs, sh.red);
        } else {
#pragma unroll 1
            for (int I0 = BAND * grp; I0 < min(S.ntiles, BAND * (grp + 1)); I0 += R)
                rows_unit<T, LAW, R, BAND>(S, grp, I0, c, sh.w.mem, sh.w.runs, sh.red);
        }
    }
}

// One step's forces of one-sided systems and of those in bands of one row, in one launch: the first
// workgroups take a band unit each (`unit_base` to `total_units`), the others are the one-sided
// kernel's. As two launches either drains before the other begins: 24 systems of 4,096 to 32,768
// elements 1103 us a step as two, 1089 as one, four of 2,048 to 8,192 65 and 55, in FP64 118 and
// 103. Not for FP64 under eqs. (4)-(6), where a band unit's 236 registers would leave the one-sided
// workgroups two waves to a SIMD (32 systems of 2,048 to 8,192: 740 as two launches, 765 as one).
template <typename T, int LAW>
__global__ __launch_bounds__(BT) __attribute__((amdgpu_waves_per_eu(rows_waves(sizeof(T) == 8, LAW, 1))))
void k_force_mixed(Launch L, int step, int last)
{
    union Shared {
        RowsMem<T> mem[LAW == 0 ? 4 : 8];
        T red[4][3][TJ];
        OneSidedMem<T, LAW> one;
    };
    __shared__ __attribute__((aligned(16))) char raw[sizeof(Shared)];
    Shared &sh = *reinterpret_cast<Shared *>(raw);
    const int u = L.unit_base + blockIdx.x;
    if (u < L.total_units) {
        SysRef S = cst(L.sys)[find_sys(L, u, false)];
        const auto *gc = cst(S.units) + 2 * (size_t)(u - S.unit_begin);
        rows_unit<T, LAW, 1, 1>(S, gc[0], gc[0], gc[1], sh.mem, nullptr, sh.red);
    } else {
        one_sided_block<T, LAW, true>(L, L.unit_base, u - L.total_units, step, last, sh.one);
    }
}

// ------------------------------------------------------------------ between two evaluations

// Systems above COM_FUSE_UNITS units: one workgroup each sums the records and finishes the step
// (every workgroup of k_advance doing so would read n / 256 records n / 256 times).
__global__ __launch_bounds__(BT) void k_finalize_step(Launch L, int in_step)
{
    __shared__ double lds[7][BT / 64];
    for (int s = blockIdx.x; s < L.n_sys; s += gridDim.x) {
        SysRef S = cst(L.sys)[s];
        if (S.n_ounits <= COM_FUSE_UNITS) continue;
        double v[7];
        sum_records(S, 0, in_step ? S.n_rec : S.n_ounits, v, lds);
        if (threadIdx.x == 0) {
            Plane p;
            plane_of(S, v, p);
            finish_step(S, p, v[6], in_step);
        }
        __syncthreads();
    }
}

// One pass over the elements between two force evaluations. `finish`: ends the step whose second
// kick wrote the records (ADV_INIT: only records the sides at creation) -- star centres, L1
// plane, growth, and the donor elements' side of the plane with the crossings since the last
// step. `kick`: begins the next step, v += a dt/2, x += v dt. One kernel of a step in place of
// five: each had a few microseconds of launch and drain. A step of the symmetric kernels is this,
// the forces and the combine with the second kick; with the sort's gather and the second kick
// as kernels of their own it took 4.3 us more (38.8 -> 34.5 at 7,500 elements, 81 -> 77 at 16,384).
// Up to COM_FUSE_UNITS units every workgroup sums the system's records itself, in one order, and
// its first one records the result. One-sided systems come here at the beginning of a call (their
// kick and drift go to the first step's set) and at its end, after n_steps.
// Its first n_o units are 256 elements each in element order; the others (the symmetric kernels' systems)
// are tiles: the drifted elements also go to their sorted slots there, with the tile's bounding box.
template <typename T>
__global__ __launch_bounds__(BT) void k_advance(Launch L, int n_o, int n_t, int finish, int kick, int n_steps)
{
    __shared__ FinishMem m;
    __shared__ float box[6][BT / 64];
    for (int u = blockIdx.x; u < n_o + n_t; u += gridDim.x) {
        const bool tiles = u >= n_o;
        SysRef S = cst(L.sys)[tiles ? find_tile_sys(L, u - n_o) : find_sys(L, u, true)];
        if (S.one_sided && finish && kick) continue;
        const int local = tiles ? u - n_o - S.tunit_begin : u - S.ounit_begin;
        int i = local * BT + threadIdx.x, at = i;
        if (tiles) {
            const int idx = glob<const int32_t>(S.perm)[i];
            i = idx < 0 ? S.n : idx;
            if (!finish) at = i;  // the call's beginning: from the caller's arrays
        }
        const bool sorted = tiles && finish;
        auto *x = glob<T>(sorted ? S.xs : S.x), *y = glob<T>(sorted ? S.ys : S.y),
             *z = glob<T>(sorted ? S.zs : S.z);
        const bool call_end = S.one_sided && finish != ADV_INIT;
        const bool odd = call_end && (n_steps & 1) != 0;
        T px = 0, py = 0, pz = 0, vx = 0, vy = 0, vz = 0, a[3] = {0, 0, 0};
        if (i < S.n) {
            px = x[at];
            py = y[at];
            pz = z[at];
            if (kick) {
                const size_t na = S.nalloc;
                vx = glob<const T>(sorted ? S.vxs : S.vx)[at];
                vy = glob<const T>(sorted ? S.vys : S.vy)[at];
                vz = glob<const T>(sorted ? S.vzs : S.vz)[at];
                a[0] = (sorted ? glob<const T>(S.as) : glob<const T>(S.ax))[at];
                a[1] = (sorted ? glob<const T>(S.as) + na : glob<const T>(S.ay))[at];
                a[2] = (sorted ? glob<const T>(S.as) + 2 * na : glob<const T>(S.az))[at];
            }
        }
        if (finish) {
            DevState *st = S.st;
            if (S.n_ounits <= COM_FUSE_UNITS) {
                double v[7];
                sum_records(S, odd ? S.rec_len : 0, finish == ADV_INIT ? S.n_ounits : S.n_rec, v,
                            m.lds);
                if (threadIdx.x == 0) {
                    plane_of(S, v, m.pl);
                    if (local == 0) {
                        finish_step(S, m.pl, v[6], finish != ADV_INIT && !call_end);
                        if (call_end) {
                            st->cur = st->slot[odd ? 1 : 0];
                            st->step = st->step_done;
                        }
                    }
                }
            } else if (threadIdx.x == 0) {
                for (int d = 0; d < 3; ++d) {
                    m.pl.com1[d] = st->com1[d];
                    m.pl.e[d] = st->e[d];
                }
                m.pl.xi_cut = st->xi_cut;
                m.pl.ok = st->plane_ok;
            }
            __syncthreads();
            classify(S, i, px, py, pz, m, finish == ADV_INIT, &st->n_past,
                     finish == ADV_INIT ? nullptr
                                        : log_row(S, call_end ? st->step_done : st->step) + 1);
        }
        if (kick && i < S.n) {
            auto *st = glob<const DevState>(S.st);
            const T h = h_of<T>(st), dt = dt_of<T>(st);
            kick_drift(h, dt, px, vx, a[0]);
            kick_drift(h, dt, py, vy, a[1]);
            kick_drift(h, dt, pz, vz, a[2]);
            const size_t na = S.nalloc;
            auto *A = step_set<T>(S, 1);
            if (!tiles) {
                (S.one_sided ? A : x)[i] = px;
                (S.one_sided ? A + na : y)[i] = py;
                (S.one_sided ? A + 2 * na : z)[i] = pz;
                (S.one_sided ? A + 3 * na : glob<T>(S.vx))[i] = vx;
                (S.one_sided ? A + 4 * na : glob<T>(S.vy))[i] = vy;
                (S.one_sided ? A + 5 * na : glob<T>(S.vz))[i] = vz;
            }
        }
        if (kick && tiles) store_sorted<T>(S, local, i < S.n, true, px, py, pz, vx, vy, vz, box);
        __syncthreads();  // m is rewritten by the next unit
    }
}

__global__ void k_init_state(DevState *st, DevState init)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *st = init;
}

// ------------------------------------------------------------------ FP64 diagnostics

template <typename T>
__global__ __launch_bounds__(BT) void k_diag_partials(Launch L)
{
    __shared__ double lds[10][BT / 64];
    for (int u = blockIdx.x; u < L.total_ounits; u += gridDim.x) {
        SysRef S = cst(L.sys)[find_sys(L, u, true)];
        const int local = u - S.ounit_begin;
        const int i = local * BT + threadIdx.x;
        double v[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        if (i < S.n) {
            const double m = glob<DevState>(S.st)->m;
            const double x = glob<const T>(S.x)[i], y = glob<const T>(S.y)[i],
                         z = glob<const T>(S.z)[i];
            const double vx = glob<const T>(S.vx)[i],
                         vy = glob<const T>(S.vy)[i],
                         vz = glob<const T>(S.vz)[i];
            v[0] = m * x;
            v[1] = m * y;
            v[2] = m * z;
            v[3] = m * vx;
            v[4] = m * vy;
            v[5] = m * vz;
            v[6] = m * (y * vz - z * vy);
            v[7] = m * (z * vx - x * vz);
            v[8] = m * (x * vy - y * vx);
            v[9] = 0.5 * m * (vx * vx + vy * vy + vz * vz);
        }
        block_sum<10>(v, lds);
        if (threadIdx.x == 0) {
            auto *r = glob<double>(S.red) + (size_t)local * RED_STRIDE + RED_DIAG;
            for (int k = 0; k < 10; ++k) r[k] = v[k];
        }
    }
}

// Potential energy of tile row I against a chunk of `pe_ch` of the tiles I .. T - 1, from the sorted
// positions: every unordered pair once, in FP64.
// Contact law: U = -A / r for r >= D and A (11 r^2 - 20 D r + 7 D^2) / (2 D^3) inside, A = G m^2,
// the primitive of the law that is continuous at D.
// eqs. (4)-(6), converging branch: -A / (r + eps) plus the overlap energy
// gamma pi (D - r)^3 (r + 3D) / 48 inside D.
// FP64 issue bounds it (12 instructions of four cycles and one reciprocal square root of sixteen per
// far pair under the contact law). Wave w takes the 64 j of each tile's quarter w and every lane
// four i of the row, so a j read from LDS serves four pairs; tiles whose box is at least D away
// (most of them) skip the contact branch, which is a selection elsewhere. With gather and
// diagnostics sums 4.42 ms at N = 131,072 (its FP64 instructions need 3.95 at the 2.23 GHz held); a
// one-sided pass with an IEEE square root and division per pair took 36.7 ms.
template <bool NEAR, int LAW>
__device__ __forceinline__ double pair_u(double r2, double D, double A, double eps, double go,
                                         double ci2, double ci1, double ci0)
{
    const double w = rsqrt_f64(NEAR ? fmax(r2, 1.0e-200) : r2);
    if constexpr (LAW == 0) {
        if constexpr (!NEAR) return w;
        const double r = r2 * w;
        const double in = fma(r, fma(ci2, r, ci1), ci0);
        const double u = r >= D ? w : in;
        return r2 > 0.0 && r2 < INFINITY ? u : 0.0;
    } else {
        const double r = r2 * w;
        const double u = A * rcp_f64(r + eps);
        if constexpr (!NEAR) return u;
        const double o = fmax(D - r, 0.0);
        const double v = fma(-(go * o), (o * o) * fma(3.0, D, r), u);
        return r2 > 0.0 && r2 < INFINITY ? v : 0.0;
    }
}

// Real elements of a tile: they come first in it.
__device__ __forceinline__ int tile_count(SysRef S, int t)
{
    const int end = t * TJ >= S.p1 ? S.p1 + (S.n - S.n1) : S.n1;
    return min(TJ, max(0, end - t * TJ));
}

template <typename T, int LAW>
__global__ __launch_bounds__(BT) void k_pe(Launch L)
{
    __shared__ double sh[TJ][4];
    __shared__ double lds[1][BT / 64];
    SysRef S = cst(L.sys)[0];
    const int I = blockIdx.x % S.ntiles, c = blockIdx.x / S.ntiles;
    const int t0 = I + c * S.pe_ch, t1 = min(S.ntiles, t0 + S.pe_ch);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto *st = cst(S.st);
    auto *XS = glob<const T>(S.xs), *YS = glob<const T>(S.ys),
            *ZS = glob<const T>(S.zs);
    const double A = st->G * st->m * st->m, eps = st->leps_d;
    const double go = st->gamma * PI_D / 48.0;
    const int istar = I * TJ >= S.p1 ? 1 : 0, ni = tile_count(S, I);
    double x[4], y[4], z[4], acc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int slot = I * TJ + 64 * k + lane;
        x[k] = XS[slot];
        y[k] = YS[slot];
        z[k] = ZS[slot];
        acc[k] = 0.0;
    }
    auto *bi = cst(S.tbox) + (size_t)I * 8;
    const float lo[3] = {bi[0], bi[1], bi[2]}, hi[3] = {bi[4], bi[5], bi[6]};
    for (int t = t0; t < t1; ++t) {
        sh[tid][0] = XS[t * TJ + tid];
        sh[tid][1] = YS[t * TJ + tid];
        sh[tid][2] = ZS[t * TJ + tid];
        __syncthreads();
        const int cls = pair_class(istar, t * TJ >= S.p1 ? 1 : 0);
        const double D =
            cls == 0 ? st->D1 : (cls == 2 ? st->cur.D2 : 0.5 * (st->D1 + st->cur.D2));
        const int j1 = min(64, tile_count(S, t) - 64 * wave);
        const double(*sj)[4] = sh + 64 * wave;
        if (far_tile(cst(S.tbox) + (size_t)t * 8, lo, hi, st->cur.far2f[cls])) {
            for (int j = 0; j < j1; ++j) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double dx = sj[j][0] - x[k], dy = sj[j][1] - y[k], dz = sj[j][2] - z[k];
                    acc[k] += pair_u<false, LAW>(fma(dx, dx, fma(dy, dy, dz * dz)), D, A, eps, go,
                                                 0.0, 0.0, 0.0);
                }
            }
        } else {
            const double h = 0.5 / (D * D * D);
            const double ci2 = -11.0 * h, ci1 = 20.0 * D * h, ci0 = -7.0 * D * D * h;
            for (int j = 0; j < j1; ++j) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double dx = sj[j][0] - x[k], dy = sj[j][1] - y[k], dz = sj[j][2] - z[k];
                    const double u = pair_u<true, LAW>(fma(dx, dx, fma(dy, dy, dz * dz)), D, A, eps,
                                                       go, ci2, ci1, ci0);
                    // the row's own tile: each pair once
                    acc[k] += t > I || 64 * wave + j > 64 * k + lane ? u : 0.0;
                }
            }
        }
        __syncthreads();
    }
    double v[1] = {0.0};
#pragma unroll
    for (int k = 0; k < 4; ++k) v[0] += 64 * k + lane < ni ? acc[k] : 0.0;
    block_sum<1>(v, lds);
    if (tid == 0) glob<double>(S.pe_part)[blockIdx.x] = LAW == 0 ? -A * v[0] : -v[0];
}

__global__ __launch_bounds__(BT) void k_finalize_diag(Launch L, int with_pe)
{
    __shared__ double lds[11][BT / 64];
    for (int s = blockIdx.x; s < L.n_sys; s += gridDim.x) {
        SysRef S = cst(L.sys)[s];
        double v[11] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        for (int u = threadIdx.x; u < S.n_ounits; u += BT) {
            auto *r = glob<const double>(S.red) + (size_t)u * RED_STRIDE + RED_DIAG;
            for (int k = 0; k < 10; ++k) v[k] += r[k];
        }
        if (with_pe) {
            for (int u = threadIdx.x; u < S.n_peunits; u += BT) v[10] += glob<double>(S.pe_part)[u];
        }
        block_sum<11>(v, lds);
        if (threadIdx.x == 0) {
            const double M = glob<DevState>(S.st)->m * (double)S.n;
            DiagOut *o = S.diag;
            for (int d = 0; d < 3; ++d) o->v[d] = M > 0.0 ? v[d] / M : 0.0;
            for (int k = 3; k < 11; ++k) o->v[k] = v[k];
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ accretor-side retention

// Pass 1: per-unit sums of star 1's velocities.
template <typename T>
__global__ __launch_bounds__(BT) void k_ret_vsum(Launch L)
{
    __shared__ double lds[3][BT / 64];
    for (int u = blockIdx.x; u < L.total_ounits; u += gridDim.x) {
        SysRef S = cst(L.sys)[find_sys(L, u, true)];
        const int local = u - S.ounit_begin;
        const int i = local * BT + threadIdx.x;
        double v[3] = {0, 0, 0};
        if (i < S.n1) {
            v[0] = glob<const T>(S.vx)[i];
            v[1] = glob<const T>(S.vy)[i];
            v[2] = glob<const T>(S.vz)[i];
        }
        block_sum<3>(v, lds);
        if (threadIdx.x == 0) {
            auto *r = glob<double>(S.red) + (size_t)local * RED_STRIDE + RED_RET;
            for (int k = 0; k < 3; ++k) r[k] = v[k];
        }
    }
}

// One block per system: star 1's mean velocity.
__global__ __launch_bounds__(BT) void k_ret_mean(Launch L)
{
    __shared__ double lds[3][BT / 64];
    for (int s = blockIdx.x; s < L.n_sys; s += gridDim.x) {
        SysRef S = cst(L.sys)[s];
        double v[3] = {0, 0, 0};
        for (int u = threadIdx.x; u < S.n_ounits; u += BT) {
            auto *r = glob<const double>(S.red) + (size_t)u * RED_STRIDE + RED_RET;
            for (int k = 0; k < 3; ++k) v[k] += r[k];
        }
        block_sum<3>(v, lds);
        if (threadIdx.x == 0) {
            for (int k = 0; k < 3; ++k) glob<DevState>(S.st)->v1[k] = S.n1 > 0 ? v[k] / (double)S.n1 : 0.0;
        }
        __syncthreads();
    }
}

// Pass 2: donor elements past the L1 plane of the last step, and those of them bound to the
// accretor as a point mass n1 m at its centre, moving with its mean velocity:
// |v - V1|^2 / 2 - G n1 m / |r - C1| < 0, in FP64.
template <typename T>
__global__ __launch_bounds__(BT) void k_ret_count(Launch L)
{
    __shared__ double lds[2][BT / 64];
    for (int u = blockIdx.x; u < L.total_ounits; u += gridDim.x) {
        SysRef S = cst(L.sys)[find_sys(L, u, true)];
        const int local = u - S.ounit_begin;
        const int i = local * BT + threadIdx.x;
        const auto *st = glob<const DevState>(S.st);
        double v[2] = {0, 0};
        if (i < S.n && i >= S.n1 && S.n1 > 0 && st->plane_ok) {
            const double rx = (double)glob<const T>(S.x)[i] - st->com1[0];
            const double ry = (double)glob<const T>(S.y)[i] - st->com1[1];
            const double rz = (double)glob<const T>(S.z)[i] - st->com1[2];
            if (rx * st->e[0] + ry * st->e[1] + rz * st->e[2] < st->xi_cut) {
                v[0] = 1.0;
                const double ux = (double)glob<const T>(S.vx)[i] - st->v1[0];
                const double uy = (double)glob<const T>(S.vy)[i] - st->v1[1];
                const double uz = (double)glob<const T>(S.vz)[i] - st->v1[2];
                const double r = sqrt(rx * rx + ry * ry + rz * rz);
                const double gm1 = st->G * st->m * (double)S.n1;
                const double energy = 0.5 * (ux * ux + uy * uy + uz * uz) - gm1 / r;
                v[1] = energy < 0.0 ? 1.0 : 0.0;
            }
        }
        block_sum<2>(v, lds);
        if (threadIdx.x == 0) {
            auto *r = glob<double>(S.red) + (size_t)local * RED_STRIDE + RED_RET + 3;
            r[0] = v[0];
            r[1] = v[1];
        }
    }
}

__global__ __launch_bounds__(BT) void k_ret_total(Launch L)
{
    __shared__ double lds[2][BT / 64];
    for (int s = blockIdx.x; s < L.n_sys; s += gridDim.x) {
        SysRef S = cst(L.sys)[s];
        double v[2] = {0, 0};
        for (int u = threadIdx.x; u < S.n_ounits; u += BT) {
            auto *r = glob<const double>(S.red) + (size_t)u * RED_STRIDE + RED_RET + 3;
            v[0] += r[0];
            v[1] += r[1];
        }
        block_sum<2>(v, lds);
        if (threadIdx.x == 0) {
            glob<DevState>(S.st)->ret_past = (int32_t)v[0];
            glob<DevState>(S.st)->ret_bound = (int32_t)v[1];
        }
        __syncthreads();
    }
}

// Copies entry k of the chunk: the system's own SysDesc word by word, with the launch's prefix
// offsets in place of its zero ones. One block per entry.
__global__ __launch_bounds__(64) void k_copy_table(SysDesc *dst, TableChunk c)
{
    static_assert(sizeof(SysDesc) % 4 == 0, "SysDesc is copied in 32-bit words");
    constexpr int W = (int)(sizeof(SysDesc) / 4);
    constexpr int WU = (int)(offsetof(SysDesc, unit_begin) / 4);
    constexpr int WO = (int)(offsetof(SysDesc, ounit_begin) / 4);
    constexpr int WT = (int)(offsetof(SysDesc, tunit_begin) / 4);
    const int k = blockIdx.x;
    const uint32_t *src = reinterpret_cast<const uint32_t *>(c.src[k]);
    uint32_t *out = reinterpret_cast<uint32_t *>(dst + c.first + k);
    for (int w = threadIdx.x; w < W; w += blockDim.x) {
        uint32_t v = src[w];
        if (w == WU) v = (uint32_t)c.unit_begin[k];
        if (w == WO) v = (uint32_t)c.ounit_begin[k];
        if (w == WT) v = (uint32_t)c.tunit_begin[k];
        out[w] = v;
    }
}

// ------------------------------------------------------------------ launchers

static inline int grid_for(int units)
{
    return units < 1 ? 1 : units;
}

hipError_t launch_copy_table(SysDesc *dst, const TableChunk &c, hipStream_t s)
{
    if (c.count < 1 || c.count > TABLE_CHUNK) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy_table, dim3(c.count), dim3(64), 0, s, dst, c);
    return hipGetLastError();
}

hipError_t launch_init_state(DevState *st, const DevState &init, hipStream_t s)
{
    hipLaunchKernelGGL(k_init_state, dim3(1), dim3(64), 0, s, st, init);
    return hipGetLastError();
}

hipError_t launch_reset_sorted(const SysDesc &d, int mode, hipStream_t s)
{
    const dim3 g((d.nalloc + BT - 1) / BT), b(BT);
    if (mode == 2) {
        hipLaunchKernelGGL(k_reset_sorted<double>, g, b, 0, s, static_cast<double *>(d.xs),
                           static_cast<double *>(d.ys), static_cast<double *>(d.zs), d.perm, d.n,
                           d.n1, d.p1, d.nalloc, SENTINEL_F64);
    } else {
        hipLaunchKernelGGL(k_reset_sorted<float>, g, b, 0, s, static_cast<float *>(d.xs),
                           static_cast<float *>(d.ys), static_cast<float *>(d.zs), d.perm, d.n,
                           d.n1, d.p1, d.nalloc, SENTINEL_F32);
    }
    return hipGetLastError();
}

hipError_t launch_zero_velocities(const SysDesc &d, int mode, hipStream_t s)
{
    const dim3 g((d.nalloc + BT - 1) / BT), b(BT);
    if (mode == 2) {
        hipLaunchKernelGGL(k_zero_sorted<double>, g, b, 0, s, static_cast<double *>(d.vxs),
                           static_cast<double *>(d.vys), static_cast<double *>(d.vzs), d.nalloc);
    } else {
        hipLaunchKernelGGL(k_zero_sorted<float>, g, b, 0, s, static_cast<float *>(d.vxs),
                           static_cast<float *>(d.vys), static_cast<float *>(d.vzs), d.nalloc);
    }
    return hipGetLastError();
}

template <typename T>
static void sort_keys(const SysDesc &d, double *bounds, uint32_t *keys, hipStream_t s)
{
    const T *x = static_cast<const T *>(d.x), *y = static_cast<const T *>(d.y),
            *z = static_cast<const T *>(d.z);
    const int blocks = (d.n + BT - 1) / BT, nb = std::min(blocks, SORT_BOUNDS);
    hipLaunchKernelGGL(k_sort_bounds<T>, dim3(nb), dim3(BT), 0, s, x, y, z, d.n, d.n1, bounds);
    hipLaunchKernelGGL(k_sort_keys<T>, dim3(blocks), dim3(BT), 0, s, x, y, z, d.n, d.n1, bounds, nb,
                       keys);
}

template <typename T>
static void sort_small(const SysDesc &d, T value, hipStream_t s)
{
    hipLaunchKernelGGL(k_sort_small<T>, dim3(1), dim3(BT), 0, s, static_cast<const T *>(d.x),
                       static_cast<const T *>(d.y), static_cast<const T *>(d.z), d.n, d.n1, d.p1,
                       d.nalloc, static_cast<T *>(d.xs), static_cast<T *>(d.ys), static_cast<T *>(d.zs),
                       d.perm, value);
}

hipError_t launch_sort(const SysDesc &d, int mode, void *work, hipStream_t s)
{
    if (d.n > 0 && d.n <= SORT_TILE) {
        if (mode == 2) {
            sort_small<double>(d, SENTINEL_F64, s);
        } else {
            sort_small<float>(d, SENTINEL_F32, s);
        }
        return hipGetLastError();
    }
    if (d.n > 0) {
        double *bounds = static_cast<double *>(work);
        uint32_t *totals = reinterpret_cast<uint32_t *>(bounds + 12 * SORT_BOUNDS);
        uint32_t *hist = totals + 256;
        const int n_tiles = (d.n + SORT_TILE - 1) / SORT_TILE;
        uint32_t *keys[2] = {static_cast<uint32_t *>(d.xs), static_cast<uint32_t *>(d.ys)};
        int32_t *vals[2] = {d.perm, static_cast<int32_t *>(d.zs)};
        if (mode == 2) {
            sort_keys<double>(d, bounds, keys[0], s);
        } else {
            sort_keys<float>(d, bounds, keys[0], s);
        }
        for (int pass = 0; pass < 4; ++pass) {
            const int in = pass & 1, out = in ^ 1;
            hipLaunchKernelGGL(k_sort_hist, dim3(n_tiles), dim3(BT), 0, s, keys[in], d.n, 8 * pass,
                               n_tiles, hist);
            hipLaunchKernelGGL(k_sort_scan, dim3(256), dim3(BT), 0, s, hist, n_tiles, totals);
            hipLaunchKernelGGL(k_sort_scatter, dim3(n_tiles), dim3(BT), 0, s, keys[in],
                               pass == 0 ? nullptr : vals[in], pass == 3 ? nullptr : keys[out],
                               vals[out], d.n, 8 * pass, n_tiles, hist, totals, d.n1, d.p1);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_reset_sorted(d, mode, s);
}

hipError_t launch_gather(const Launch &L, int mode, hipStream_t s)
{
    if (L.total_tunits == 0) return hipSuccess;
    const dim3 g(grid_for(L.total_tunits)), b(BT);
    if (mode == 2) {
        hipLaunchKernelGGL(k_gather<double>, g, b, 0, s, L);
    } else {
        hipLaunchKernelGGL(k_gather<float>, g, b, 0, s, L);
    }
    return hipGetLastError();
}

hipError_t launch_forces(const Launch &L, int mode, int step, int last, int max_blocks,
                         hipStream_t s)
{
    if (L.total_units == 0) return hipSuccess;
    if (L.law != 0 && L.law != 1) return hipErrorInvalidValue;
    // max_blocks > 0: persistent launch, each block loops over units u, u + grid, ...
    auto grid = [&](int units) {
        return dim3(grid_for(max_blocks > 0 ? std::min(units, max_blocks) : units));
    };
    Launch R = L;
    int begin = 0;
    for (int b = 0; b < KERNEL_CLASSES; ++b) {
        const int end = L.band_end[b];
        if (end <= begin) continue;
        R.unit_base = begin;
        R.total_units = end;
        const dim3 g = grid(end - begin), blk(BT);
        const int end1 = L.band_end[1], all = end1 + (step > 1 ? L.ounit_base : 0);
        if (b == 0 && step > 0 && end1 > end && max_blocks <= 0 && !(mode == 2 && L.law != 0)) {
            R.unit_base = end;
            R.total_units = end1;
            const dim3 gs(all);
            if (mode == 2) {
                hipLaunchKernelGGL((k_force_mixed<double, 0>), gs, blk, 0, s, R, step, last);
            } else if (L.law == 0) {
                hipLaunchKernelGGL((k_force_mixed<float, 0>), gs, blk, 0, s, R, step, last);
            } else {
                hipLaunchKernelGGL((k_force_mixed<float, 1>), gs, blk, 0, s, R, step, last);
            }
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            begin = end1;
            continue;
        }
        if (b == 0) {
            if (mode == 0) return hipErrorInvalidValue;
            const hipError_t e =
                mode == 2 ? (L.law == 0 ? launch_one_sided<double, 0>(R, step, last, max_blocks, s)
                                        : launch_one_sided<double, 1>(R, step, last, max_blocks, s))
                          : (L.law == 0 ? launch_one_sided<float, 0>(R, step, last, max_blocks, s)
                                        : launch_one_sided<float, 1>(R, step, last, max_blocks, s));
            if (e != hipSuccess) return e;
        } else if (mode == 0) {
            if (L.law != 0 || b != 1) return hipErrorInvalidValue;  // no eqs. (4)-(6), no bands
            if (end - begin > CU_COUNT) {
                hipLaunchKernelGGL(k_force_f32<true>, g, blk, 0, s, R);
            } else {
                // at most one wave per SIMD
                hipLaunchKernelGGL(k_force_f32<false>, g, blk, 0, s, R);
            }
        } else if (mode == 2) {
            if (b != 1) return hipErrorInvalidValue;
            if (L.law == 0) {
                hipLaunchKernelGGL((k_force_rows<double, 0, 1>), g, blk, 0, s, R);
            } else {
                hipLaunchKernelGGL((k_force_rows<double, 1, 1>), g, blk, 0, s, R);
            }
        } else {
            // FP32 Kahan: one launch per band height present in the table
            switch (b * 2 + L.law) {
            case 2: hipLaunchKernelGGL((k_force_rows<float, 0, 1>), g, blk, 0, s, R); break;
            case 3: hipLaunchKernelGGL((k_force_rows<float, 1, 1>), g, blk, 0, s, R); break;
            case 4: hipLaunchKernelGGL((k_force_rows<float, 0, 2>), g, blk, 0, s, R); break;
            case 5: hipLaunchKernelGGL((k_force_rows<float, 1, 2>), g, blk, 0, s, R); break;
            case 6: hipLaunchKernelGGL((k_force_rows<float, 0, 2, 4>), g, blk, 0, s, R); break;
            default: hipLaunchKernelGGL((k_force_rows<float, 1, 2, 4>), g, blk, 0, s, R); break;
            }
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        begin = end;
    }
    return begin == L.total_units ? hipSuccess : hipErrorInvalidValue;
}

hipError_t launch_combine(const Launch &L, int mode, int kick, int last, hipStream_t s)
{
    if (L.total_tunits == 0) return hipSuccess;
    if (mode == 0) return hipErrorInvalidValue;  // no partial sums
    const dim3 g(grid_for(L.total_tunits));
    if (mode == 1) {
        const bool many = L.total_tunits > CU_COUNT;
        const auto k = kick ? (many ? k_combine_sym<true, true> : k_combine_sym<true, false>)
                            : (many ? k_combine_sym<false, true> : k_combine_sym<false, false>);
        hipLaunchKernelGGL(k, g, dim3(BT * COMBINE_SEGS), 0, s, L, last);
    } else {
        const auto k = kick ? k_combine_sym64<true> : k_combine_sym64<false>;
        hipLaunchKernelGGL(k, g, dim3(BT * COMBINE_SEGS), 0, s, L, last);
    }
    return hipGetLastError();
}

hipError_t launch_kick_stats(const Launch &L, int mode, int do_kick, hipStream_t s)
{
    // in a step the plain mode's systems and empty ones: the force kernel or the combine kicks the others
    if (do_kick && mode != 0 && !L.any_empty) return hipSuccess;
    Launch R = L;
    if (do_kick && mode != 0) R.total_ounits = L.ounit_base;
    if (R.total_ounits == 0) return hipSuccess;
    const dim3 g(grid_for(R.total_ounits)), b(BT);
    if (mode == 2) {
        hipLaunchKernelGGL(k_kick_stats<double>, g, b, 0, s, R, do_kick);
    } else {
        hipLaunchKernelGGL(k_kick_stats<float>, g, b, 0, s, R, do_kick);
    }
    return hipGetLastError();
}

hipError_t launch_finalize_step(const Launch &L, int in_step, hipStream_t s)
{
    if (!L.any_big) return hipSuccess;
    hipLaunchKernelGGL(k_finalize_step, dim3(grid_for(L.n_sys)), dim3(BT), 0, s, L, in_step);
    return hipGetLastError();
}

hipError_t launch_advance(const Launch &L, int mode, int finish, int kick, int n_steps, hipStream_t s)
{
    // the plain mode's systems pass in element order, as every one does at creation; of the others the
    // one-sided ones at a call's beginning and end, empty ones always, the rest tile by tile
    const bool sorted = mode != 0 && finish != ADV_INIT;
    const int n_o = !sorted ? L.total_ounits : (finish && kick && !L.any_empty ? 0 : L.ounit_base);
    const int n_t = sorted ? L.total_tunits : 0;
    if (n_o + n_t == 0) return hipSuccess;
    const dim3 g(grid_for(n_o + n_t)), b(BT);
    if (mode == 2) {
        hipLaunchKernelGGL(k_advance<double>, g, b, 0, s, L, n_o, n_t, finish, kick, n_steps);
    } else {
        hipLaunchKernelGGL(k_advance<float>, g, b, 0, s, L, n_o, n_t, finish, kick, n_steps);
    }
    return hipGetLastError();
}

// one system
hipError_t launch_diag(const Launch &L, int mode, int with_pe, int n_peunits, hipStream_t s)
{
    if (L.n_sys != 1) return hipErrorInvalidValue;
    if (L.total_ounits > 0) {
        const dim3 g(grid_for(L.total_ounits)), b(BT);
        if (mode == 2) {
            hipLaunchKernelGGL(k_diag_partials<double>, g, b, 0, s, L);
        } else {
            hipLaunchKernelGGL(k_diag_partials<float>, g, b, 0, s, L);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (with_pe && n_peunits > 0) {
            // the pair sum reads the sorted positions of the current state
            e = launch_gather(L, mode, s);
            if (e != hipSuccess) return e;
            const dim3 gp(n_peunits);
            switch ((mode == 2 ? 2 : 0) + L.law) {
            case 0: hipLaunchKernelGGL((k_pe<float, 0>), gp, b, 0, s, L); break;
            case 1: hipLaunchKernelGGL((k_pe<float, 1>), gp, b, 0, s, L); break;
            case 2: hipLaunchKernelGGL((k_pe<double, 0>), gp, b, 0, s, L); break;
            default: hipLaunchKernelGGL((k_pe<double, 1>), gp, b, 0, s, L); break;
            }
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    hipLaunchKernelGGL(k_finalize_diag, dim3(grid_for(L.n_sys)), dim3(BT), 0, s, L, with_pe);
    return hipGetLastError();
}

hipError_t launch_retention(const Launch &L, int mode, hipStream_t s)
{
    if (L.total_ounits > 0) {
        const dim3 g(grid_for(L.total_ounits)), b(BT);
        if (mode == 2) {
            hipLaunchKernelGGL(k_ret_vsum<double>, g, b, 0, s, L);
        } else {
            hipLaunchKernelGGL(k_ret_vsum<float>, g, b, 0, s, L);
        }
    }
    hipLaunchKernelGGL(k_ret_mean, dim3(grid_for(L.n_sys)), dim3(BT), 0, s, L);
    if (L.total_ounits > 0) {
        const dim3 g(grid_for(L.total_ounits)), b(BT);
        if (mode == 2) {
            hipLaunchKernelGGL(k_ret_count<double>, g, b, 0, s, L);
        } else {
            hipLaunchKernelGGL(k_ret_count<float>, g, b, 0, s, L);
        }
    }
    hipLaunchKernelGGL(k_ret_total, dim3(grid_for(L.n_sys)), dim3(BT), 0, s, L);
    return hipGetLastError();
}

}  // namespace nbk
