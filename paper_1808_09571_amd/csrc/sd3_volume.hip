// 3D volume of each row (Sec. 3.2.1): by the divergence theorem with the
// field F = p / 3 the volume is a sum over the faces (Eq. 1), and on a
// counter-clockwise triangle u v w the face term is u . n / 6 with
// n = (v - u) x (w - u) (Eq. 2).
//
// Each term is formed in double-double arithmetic (the differences v - u and
// w - u are exact two-term values, the products carry their rounding error
// through fused multiply-adds), and the terms are summed in double-double, so
// the result keeps about 100 bits of the terms' magnitude before the final
// rounding: far below 1e-12 relative unless the faces' terms cancel by more
// than 2^50 (a closed mesh about 10^5 of its own sizes away from the origin).
//
// Work items are (row, chunk of VOL_CHUNK consecutive triangles of that row,
// with its share of the row's vertices to check); a block reduces its chunk to
// one double-double partial; a second kernel adds each row's partials in chunk
// order and writes the volume, so the result does not depend on scheduling.
//
// Per triangle 12 bytes of indices, three 24-byte vertex gathers and about 240
// FP64 instructions.  The gathers are far from coalesced (a mesh's vertices
// may lie in any order), so what a row costs is how often its vertices come
// from HBM: blocks take the items in XCD-contiguous ranges, so that a row's
// vertices are fetched into one XCD's L2 and not into all eight, and a thread
// has VOL_BATCH triangles' gathers in flight.  1000 ore bodies (37.5M
// triangles): 1011 -> 785 us per call; bound by the address units (2.2 cache
// accesses a gathered vertex, busy 80% of the launch).
#include <algorithm>

#include "sd3_kernels.h"

#pragma clang fp contract(off)

namespace sd3 {

struct DD {
    double hi, lo;
};

__device__ __forceinline__ DD dd_two_sum(double a, double b) {
    const double s = a + b;
    const double bv = s - a;
    const double av = s - bv;
    return {s, (a - av) + (b - bv)};
}

__device__ __forceinline__ DD dd_fast(double hi, double lo) {
    const double s = hi + lo;
    return {s, lo - (s - hi)};
}

__device__ __forceinline__ DD dd_add(DD a, DD b) {
    DD s = dd_two_sum(a.hi, b.hi);
    DD t = dd_two_sum(a.lo, b.lo);
    s.lo += t.hi;
    s = dd_fast(s.hi, s.lo);
    s.lo += t.lo;
    return dd_fast(s.hi, s.lo);
}

__device__ __forceinline__ DD dd_neg(DD a) { return {-a.hi, -a.lo}; }

__device__ __forceinline__ DD dd_mul(DD a, DD b) {
    const double p = a.hi * b.hi;
    double e = fma(a.hi, b.hi, -p);
    e = fma(a.hi, b.lo, e);
    e = fma(a.lo, b.hi, e);
    return dd_fast(p, e);
}

__device__ __forceinline__ DD dd_mul_d(double a, DD b) {
    const double p = a * b.hi;
    double e = fma(a, b.hi, -p);
    e = fma(a, b.lo, e);
    return dd_fast(p, e);
}

// exact difference a - b as a double-double
__device__ __forceinline__ DD dd_diff(double a, double b) {
    const double s = a - b;
    const double bv = a - s;
    const double av = s + bv;
    return {s, (a - av) + (bv - b)};
}

__device__ __forceinline__ DD dd_shfl_xor(DD v, int o) { return {__shfl_xor(v.hi, o), __shfl_xor(v.lo, o)}; }

// u . ((v - u) x (w - u)) of the corners u, v, w.
__device__ __forceinline__ DD vol_term(const double (&p)[3][3]) {
    DD a[3], b[3];
    for (int c = 0; c < 3; c++) {
        a[c] = dd_diff(p[1][c], p[0][c]);
        b[c] = dd_diff(p[2][c], p[0][c]);
    }
    DD s = {0.0, 0.0};
    for (int c = 0; c < 3; c++) {
        const int j = (c + 1) % 3, l = (c + 2) % 3;
        const DD n = dd_add(dd_mul(a[j], b[l]), dd_neg(dd_mul(a[l], b[j])));
        s = dd_add(s, dd_mul_d(p[0][c], n));
    }
    return s;
}

constexpr int VOL_CHUNK = 4096;  // triangles per work item
constexpr int VOL_WG = 256;
constexpr int VOL_BATCH = 4;     // triangles a thread loads at once
constexpr int64_t VOL_SLICE = 1 << 23;  // items per launch

// Items per row: its triangle chunks, and one for a row of vertices alone.
__host__ __device__ __forceinline__ int64_t vol_row_items(int64_t nt, int64_t nv) {
    return nt > 0 ? (nt + VOL_CHUNK - 1) / VOL_CHUNK : (nv > 0 ? 1 : 0);
}

__device__ __forceinline__ uint32_t vol_coord(double v) {
    const double x = fabs(v);
    if (!(x <= 1.7976931348623157e308)) return V_NONFINITE;
    return x != 0.0 && (x < 0x1p-256 || x > 0x1p256) ? V_RANGE : 0u;
}

// One block per item from `first` on (witem[g]: row g's first item), a thread
// loading BATCH triangles at once.  ROWS: no row has more than VOL_CHUNK
// triangles, so an item is a row.  Such columns are bound by each block's chain
// of loads, not by the bytes: the first round of the row's search looks around
// the place it has where no row is empty, and rows of at most 256 or 512
// triangles load no more a thread than there are (200,000 rows of 20 triangles:
// 862 -> 342 us; the call on 50,000 rows of 320: 545 -> 400, 30,000 of 720: 407
// -> 362, 4000 of 3920: 250 -> 245).
template <int BATCH, bool ROWS>
__global__ __launch_bounds__(VOL_WG) void k_vol_partial(const double *xyz, const int32_t *tri,
                                                        const int64_t *v_off, const int64_t *t_off,
                                                        const int64_t *witem, int64_t first, int64_t G,
                                                        double rows_per_item, DD *part, uint32_t *flags) {
    __shared__ DD red[VOL_WG / 64];
    // consecutive items to one XCD (workgroups are dealt to the eight in turn)
    const unsigned x = blockIdx.x & 7u, nq = gridDim.x >> 3, nr = gridDim.x & 7u;
    const int64_t it = first + (int64_t)x * nq + min(x, nr) + (blockIdx.x >> 3);
    int64_t lo = 0, hi = G;  // the row, found by the wave: 64 probes a round
    if (ROWS) {
        const int64_t q = (int64_t)((double)it * rows_per_item) - 32;
        const int64_t at = q + lane_id();
        const int c = __popcll(__ballot(at <= 0 || (at < G && witem[at] <= it)));
        if (c > 0) lo = q + c - 1;
        if (c < 64) hi = q + c;
    }
    while (hi - lo > 1) {
        const int64_t step = (hi - lo + 63) >> 6;
        const int64_t q = lo + (int64_t)(lane_id() + 1) * step;
        const int c = __popcll(__ballot(q < hi && witem[q] <= it));
        hi = min(hi, lo + (int64_t)(c + 1) * step);
        lo += (int64_t)c * step;
    }
    const int64_t g = lo, j = ROWS ? 0 : it - witem[g], items = ROWS ? 1 : witem[g + 1] - witem[g];
    const int64_t t0 = t_off[g] + j * VOL_CHUNK, t1 = min(t_off[g + 1], t0 + (int64_t)VOL_CHUNK);
    const double *X = xyz + 3 * v_off[g];
    const int64_t nvr = v_off[g + 1] - v_off[g];
    uint32_t bad = 0;
    // this item's share of the row's vertices (the checks of the distance
    // operators), which the gathers then find in the L2
    const int64_t c0 = 3 * nvr * j / items, c1 = 3 * nvr * (j + 1) / items;
#pragma unroll 4
    for (int64_t i = c0 + threadIdx.x; i < c1; i += VOL_WG) bad |= vol_coord(X[i]);
    DD s = {0.0, 0.0};
    for (int64_t base = t0 + threadIdx.x; base < t1; base += BATCH * VOL_WG) {
        double p[BATCH][3][3];
        int64_t vi[BATCH][3];
        bool in[BATCH];
        // (vertex indices are clamped into the row)
#pragma unroll
        for (int r = 0; r < BATCH; r++) {
            const int64_t t = base + r * VOL_WG;
            in[r] = t < t1;
            for (int k = 0; k < 3; k++) vi[r][k] = tri[3 * (in[r] ? t : t1 - 1) + k];
        }
#pragma unroll
        for (int r = 0; r < BATCH; r++)
            for (int k = 0; k < 3; k++) {
                const bool ok = vi[r][k] >= 0 && vi[r][k] < nvr;
                bad |= ok ? 0u : V_INDEX;
                const double *v = X + 3 * (ok ? vi[r][k] : 0);
                for (int c = 0; c < 3; c++) p[r][k][c] = v[c];
            }
#pragma unroll
        for (int r = 0; r < BATCH; r++)
            if (in[r]) s = dd_add(s, vol_term(p[r]));
    }
    if (BATCH != 1 || t0 + (threadIdx.x & ~63u) < t1)  // (the other waves hold zeros)
        for (int o = 32; o > 0; o >>= 1) s = dd_add(s, dd_shfl_xor(s, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    if (bad) atomicOr(flags, bad);
    __syncthreads();
    if (threadIdx.x == 0) {
        DD r = red[0];
        for (int w = 1; w < VOL_WG / 64; w++) r = dd_add(r, red[w]);
        part[it] = r;
    }
}

// Row g: its partials (items witem[g] .. witem[g+1] - 1) in order, / 6.
__global__ void k_vol_rows(const DD *part, const int64_t *witem, int64_t G, double *vol,
                           const uint32_t *flags) {
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= G || *flags) return;
    DD s = {0.0, 0.0};
    const int64_t i1 = witem[g + 1];
    for (int64_t i = witem[g]; i < i1; i += 8) {
        DD p[8];  // (eight loads in flight)
#pragma unroll
        for (int k = 0; k < 8; k++) p[k] = part[min(i + k, i1 - 1)];
#pragma unroll
        for (int k = 0; k < 8; k++)
            if (i + k < i1) s = dd_add(s, p[k]);
    }
    // (hi + lo) / 6 rounded once more: hi / 6 plus the remainder's share
    const double q = s.hi / 6.0;
    const double r = fma(-q, 6.0, s.hi);  // exact remainder of hi - 6 q
    vol[g] = q + (r + s.lo) / 6.0;
}

__global__ void k_vol_clear(uint32_t *flags) {
    if (threadIdx.x == 0) *flags = 0;
}

void launch_volume(const double *xyz, const int32_t *tri, const int64_t *v_off, const int64_t *t_off,
                   int64_t nitems, const int64_t *witem, int64_t max_row, int64_t G, void *part, double *vol,
                   uint32_t *flags, hipStream_t s) {
    hipLaunchKernelGGL(k_vol_clear, dim3(1), dim3(64), 0, s, flags);
    // (a launch takes fewer than 2^32 threads)
    const auto partial = max_row <= VOL_WG       ? k_vol_partial<1, true>
                         : max_row <= 2 * VOL_WG ? k_vol_partial<2, true>
                         : max_row <= VOL_CHUNK  ? k_vol_partial<VOL_BATCH, true>
                                                 : k_vol_partial<VOL_BATCH, false>;
    for (int64_t i0 = 0; i0 < nitems; i0 += VOL_SLICE)
        hipLaunchKernelGGL(partial, dim3((unsigned)std::min(nitems - i0, VOL_SLICE)), dim3(VOL_WG), 0, s, xyz, tri, v_off,
                           t_off, witem, i0, G, (double)G / (double)nitems, (DD *)part, flags);
    if (G > 0)
        hipLaunchKernelGGL(k_vol_rows, dim3((unsigned)((G + 63) / 64)), dim3(64), 0, s, (const DD *)part, witem, G,
                           vol, flags);
}

int64_t volume_items(int64_t nt, int64_t nv) { return vol_row_items(nt, nv); }

}  // namespace sd3
