// Segments and points against one triangle mesh: the paper's measured
// workload (Sec. 4: drill-hole line segments against an ore-body mesh), with
// the three operators of Sec. 3.2.2 / 3.2.3 -- distance (items (i)-(iii):
// segment/segment, segment/surface, point/surface, then the minimum),
// intersects (Eq. 4 crossings with closed constraints) and the distance
// threshold filter (distance <= r, "filtering drill holes based on their
// distance").
//
// A segment P0 P1 is the degenerate triangle (P0, P1, P1) and a point the
// triangle (P, P, P): seg_pair64 gives the bits of the FP64 triangle-pair
// routine for it, and undecided contacts go to the exact intersection test of
// the mesh path (a zero-area triangle is the union of its edges), so the
// values are those sd3_distance returns for the same inputs.
//
// Layout: the mesh is prepared once per call, each run of RS_ITEMS triangles in
// the order of a Hilbert curve, into FP64 triangles (S_NTRI fields), FP32
// triangles (SEG_TRI4 words) and a tree of bounding cylinders over groups of
// 8, 64, 512, ... consecutive triangles in FP32 (SegNode, 32 bytes; level 0
// bounds the single triangles).  One wave owns 64 segments.  It tests the
// nodes of the top level (at most 16) against all of them, and keeps the
// (segment, node) pairs that survive on one LDS stack per level; from then on
// a lane works on any segment's pair: 64 pairs of one level are popped
// together, each lane tests its node's eight children, and the survivors are
// compacted with ballots onto the level below, the deepest level with 64 pairs
// first, so that the lanes stay full however the segments differ.  Distances
// take the FP32 bounds of the triangle pairs still live when popped, and what
// these leave is gathered for the FP64 test until the list is full or nothing
// else is to do: the bounds are at their lowest by then.
//
// Measured (before: every lane looped over the boxes of whole 64-triangle
// tiles, one scalar load chain per triangle, and crossing segments ran exact
// arithmetic): 5,000,000 segments against a 500-face body, distance, 14.1 ->
// 2.04 ms (75 triangle bounds and 2.6 FP64 tests a segment; 335 and 12.9
// before); 300,000 within 2 of a 20,480-face body 2.27 -> 0.17 ms.  Of that,
// on the first case's pass: FP64 tests right after the cylinders, in the
// input's order, 2.91 ms; FP32 bounds and the late FP64 tests 2.40; the first
// vertices' Morton order -> the centroids' Hilbert order 2.08.  Bound by FP32
// vector instructions.  The other operators' threshold never moves, so they keep
// no bounds in LDS (8.2 -> 5.1 KB a wave and 2.3 KB a level: two more waves a CU
// on the 20,480 faces, 189 -> 174 us).
#include <algorithm>

#include "sd3_kernels.h"
#include "sd3_sort.h"
#include "sd3_pair64.h"
#include "sd3_exact.h"

namespace sd3 {

constexpr int FAN = SEG_FAN;      // children per node
constexpr int STACK = 64 + 64 * FAN;  // a level below 64 pairs takes one expansion

// A bounding cylinder: every point of the node's triangles is c + a n + y
// with |a| <= w, y orthogonal to n and |y| <= rho.  Coordinates are relative
// to the mesh's frame (SegFrame): |c| <= sqrt(3).  c and n are FP32 values
// that rho and w are measured from, so they carry no error of their own.
struct SegNode {
    float c[3], rho, n[3], w;
};
static_assert(sizeof(SegNode) == SEG_NODE_BYTES, "two 16-byte loads");

// The mesh's frame: its box centre, and the power of two that takes the
// largest extent into [1, 2) (1 for a box of no extent), so that the FP32
// cull neither overflows near the mesh nor loses it to the origin.
struct SegFrame {
    double c[3], s;
};

__device__ __forceinline__ SegFrame seg_frame(const unsigned long long *box) {
    SegFrame f;
    double ext = 0.0;
    for (int k = 0; k < 3; k++) {
        const double lo = from_ordered_bits(box[k]), hi = from_ordered_bits(box[3 + k]);
        f.c[k] = 0.5 * lo + 0.5 * hi;
        ext = fmax(ext, hi - lo);
    }
    const bool ok = ext > 0.0 && ext < __builtin_inf();
    f.s = ok ? ldexp(1.0, -ilogb(ext)) : 1.0;
    return f;
}

// Place of a cell (6 bits an axis) along a Hilbert curve (Skilling, 2004:
// exchange and invert the low bits of the axes from the top bit down, then
// Gray decode).
__device__ __forceinline__ uint32_t hilbert18(uint32_t (&x)[3]) {
#pragma unroll
    for (uint32_t q = 32; q > 1; q >>= 1) {
        const uint32_t m = q - 1;
#pragma unroll
        for (int i = 0; i < 3; i++) {
            const uint32_t t = (x[0] ^ x[i]) & m;
            const bool b = (x[i] & q) != 0;
            x[0] ^= b ? m : t;
            x[i] ^= b ? 0u : t;
        }
    }
    x[1] ^= x[0];
    x[2] ^= x[1];
    uint32_t t = 0;
#pragma unroll
    for (uint32_t q = 32; q > 1; q >>= 1) t ^= (x[2] & q) ? q - 1 : 0u;
#pragma unroll
    for (int i = 0; i < 3; i++) x[i] ^= t;
    return spread10(x[2]) | (spread10(x[1]) << 1) | (spread10(x[0]) << 2);
}

// The order the tree takes the triangles in: each run of RS_ITEMS triangles by
// the place of their centroids' cells of the run's own box on the curve, so
// that a node's eight triangles are a patch and not a strip of the input's
// order (results never depend on it).  Against Morton order, whose jumps make
// long patches: 91 -> 75 triangle bounds a segment.  One block for run `run`;
// indices are clamped into the mesh.
__device__ __forceinline__ void order_run(int64_t run, const double *xyz, int64_t nv, const int32_t *tri, int64_t nt,
                                          int32_t *order, LocalSort &L, double (&red)[16][6]) {
    constexpr int PER = RS_ITEMS / 1024;
    const int tid = (int)threadIdx.x;
    const int64_t t0 = run * RS_ITEMS;
    const int n = (int)min((int64_t)RS_ITEMS, nt - t0);
    double p[PER][3], lo[3], hi[3];
    for (int c = 0; c < 3; c++) {
        lo[c] = __builtin_inf();
        hi[c] = -__builtin_inf();
    }
#pragma unroll
    for (int r = 0; r < PER; r++) {
        const int64_t t = t0 + min(r * 1024 + tid, n - 1);
        for (int c = 0; c < 3; c++) p[r][c] = 0.0;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const int32_t v = tri[3 * t + k];
            const int64_t vi = (v >= 0 && (int64_t)v < nv) ? v : 0;
#pragma unroll
            for (int c = 0; c < 3; c++) p[r][c] += xyz[3 * vi + c];
        }
#pragma unroll
        for (int c = 0; c < 3; c++) {
            lo[c] = fmin(lo[c], p[r][c]);
            hi[c] = fmax(hi[c], p[r][c]);
        }
    }
    for (int c = 0; c < 3; c++) {
        const double a = wave_min(lo[c]), b = wave_max(hi[c]);
        if (lane_id() == 0) {
            red[tid >> 6][c] = a;
            red[tid >> 6][3 + c] = b;
        }
    }
    __syncthreads();
    double ext = 0.0;
    for (int c = 0; c < 3; c++) {
        double a = red[0][c], b = red[0][3 + c];
        for (int w = 1; w < 16; w++) {
            a = fmin(a, red[w][c]);
            b = fmax(b, red[w][3 + c]);
        }
        lo[c] = a;
        ext = fmax(ext, b - a);
    }
    const double sc = ext > 0.0 && ext < __builtin_inf() ? 64.0 / ext : 0.0;
#pragma unroll
    for (int r = 0; r < PER; r++) {
        const int j = r * 1024 + tid;
        uint32_t x[3];
#pragma unroll
        for (int c = 0; c < 3; c++) x[c] = (uint32_t)fmin(fmax((p[r][c] - lo[c]) * sc, 0.0), 63.0);
        if (j < n) L.a[j] = (hilbert18(x) >> 2) << 16 | (uint32_t)j;
    }
    __syncthreads();
    local_pass(L, L.a, L.b, n, 16);
    local_pass(L, L.b, L.a, n, 24);
    for (int j = tid; j < n; j += 1024) order[t0 + j] = (int32_t)(t0 + (int64_t)(L.a[j] & 0xffffu));
}

__device__ __forceinline__ uint32_t coord_flags(double v) {
    const double x = fabs(v);
    const uint32_t range = x != 0.0 && (x < 0x1p-256 || x > 0x1p256) ? V_RANGE : 0u;
    return x <= 1.7976931348623157e308 ? range : (uint32_t)V_NONFINITE;
}

// Validation of the segment coordinates (flags[0]) and of the mesh
// (coordinates and indices, flags[1]), and the mesh's box (ordered bits) from
// its triangles' corners (a vertex that none uses must not widen the frame:
// what FP32 tells apart is a part of it); k_seg_clear set every word.  The first blocks, one per run, put
// the mesh's triangles in order meanwhile: the sort of a small mesh is a chain
// of waits in one block that no other work needs yet.
__global__ __launch_bounds__(1024) void k_seg_validate(const double *seg, int64_t n, const double *xyz,
                                                       int64_t nv, const int32_t *tri, int64_t nt, int32_t *order,
                                                       uint32_t *flags, unsigned long long *box) {
    __shared__ LocalSort L;
    __shared__ double red[16][6];
    const int64_t runs = (nt + RS_ITEMS - 1) / RS_ITEMS;
    if ((int64_t)blockIdx.x < runs) {
        order_run(blockIdx.x, xyz, nv, tri, nt, order, L, red);
        return;
    }
    const int64_t block = (int64_t)blockIdx.x - runs;
    uint32_t fs = 0, fm = 0;
    const int64_t stride = ((int64_t)gridDim.x - runs) * blockDim.x;
    const int64_t first = block * (int64_t)blockDim.x + threadIdx.x;
    int64_t i0 = first;
    for (; i0 + 7 * stride < 6 * n; i0 += 8 * stride) {  // (eight loads in flight)
        double x[8];
#pragma unroll
        for (int k = 0; k < 8; k++) x[k] = seg[i0 + k * stride];
#pragma unroll
        for (int k = 0; k < 8; k++) fs |= coord_flags(x[k]);
    }
    for (; i0 < 6 * n; i0 += stride) fs |= coord_flags(seg[i0]);
    for (int64_t i = first; i < 3 * nv; i += stride) fm |= coord_flags(xyz[i]);
    double lo[3] = {__builtin_inf(), __builtin_inf(), __builtin_inf()};
    double hi[3] = {-__builtin_inf(), -__builtin_inf(), -__builtin_inf()};
    for (int64_t i = first; i < 3 * nt; i += stride) {
        const int32_t v = tri[i];
        if (v < 0 || (int64_t)v >= nv) {
            fm |= V_INDEX;
            continue;
        }
        for (int c = 0; c < 3; c++) {
            const double x = xyz[3 * (int64_t)v + c];
            lo[c] = fmin(lo[c], x);
            hi[c] = fmax(hi[c], x);
        }
    }
    if (fs) atomicOr(&flags[0], fs);
    if (fm) atomicOr(&flags[1], fm);
    if (block * (int64_t)blockDim.x >= 3 * nt) return;  // (block-uniform)
    for (int c = 0; c < 3; c++) {
        const double a = wave_min(lo[c]), b = wave_max(hi[c]);
        if (lane_id() == 0) {
            red[threadIdx.x >> 6][c] = a;
            red[threadIdx.x >> 6][3 + c] = b;
        }
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int c = threadIdx.x;
        double v = red[0][c];
        for (int w = 1; w < 16; w++) v = c < 3 ? fmin(v, red[w][c]) : fmax(v, red[w][c]);
        if (c < 3) atomicMin(&box[c], ordered_bits(v));
        else atomicMax(&box[c], ordered_bits(v));
    }
}

// Minimum, maximum or sum over each aligned group of W lanes (8 or 64), in
// every lane of the group.
template <int W, typename F>
__device__ __forceinline__ double lanes_reduce(double v, F f) {
#pragma unroll
    for (int o = 1; o < W; o <<= 1) v = f(v, __shfl_xor(v, o));
    return v;
}

__device__ __forceinline__ float round_up(double x) { return (float)x * (1.0f + 0x1p-22f) + 0x1p-60f; }

__device__ __forceinline__ void write_node(float4 *nodes, int64_t i, const float (&c)[3], double rho,
                                           const float (&n)[3], double w) {
    nodes[2 * i] = make_float4(c[0], c[1], c[2], round_up(rho));
    nodes[2 * i + 1] = make_float4(n[0], n[1], n[2], round_up(w));
}

// A unit direction in FP32 (any one for a zero or unusable vector).
__device__ __forceinline__ void unit_dir(const double *v, float (&n)[3]) {
    const double l = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    const bool ok = l > 0x1p-400 && l < 0x1p400;
    for (int k = 0; k < 3; k++) n[k] = ok ? (float)(v[k] / l) : (k == 2 ? 1.0f : 0.0f);
}

// The cylinder of the triangles of each aligned group of W lanes (x: the
// lane's corners in the frame, a: its area normal; lanes without a triangle
// bring nothing).
template <int W>
__device__ __forceinline__ void group_node(const double (&x)[9], const double (&a)[3], bool in, float (&c)[3],
                                           float (&n)[3], double &rho, double &w) {
    double s[3];
    for (int k = 0; k < 3; k++) {
        const double l = in ? fmin(x[k], fmin(x[3 + k], x[6 + k])) : __builtin_inf();
        const double h = in ? fmax(x[k], fmax(x[3 + k], x[6 + k])) : -__builtin_inf();
        const double lo = lanes_reduce<W>(l, [](double p, double q) { return fmin(p, q); });
        const double hi = lanes_reduce<W>(h, [](double p, double q) { return fmax(p, q); });
        c[k] = (float)(0.5 * lo + 0.5 * hi);
        s[k] = lanes_reduce<W>(in ? a[k] : 0.0, [](double p, double q) { return p + q; });
    }
    unit_dir(s, n);
    double r2 = 0.0, h = 0.0;
    for (int k = 0; k < 3; k++) {
        const double d0 = x[3 * k] - c[0], d1 = x[3 * k + 1] - c[1], d2 = x[3 * k + 2] - c[2];
        const double t = n[0] * d0 + n[1] * d1 + n[2] * d2;
        // the part along n of a direction that is unit to 2^-22
        const double l0 = d0 - t * n[0], l1 = d1 - t * n[1], l2 = d2 - t * n[2];
        r2 = fmax(r2, l0 * l0 + l1 * l1 + l2 * l2);
        h = fmax(h, fabs(t));
    }
    rho = sqrt(lanes_reduce<W>(in ? r2 : 0.0, [](double p, double q) { return fmax(p, q); }));
    w = lanes_reduce<W>(in ? h : 0.0, [](double p, double q) { return fmax(p, q); });
    // (n is unit, and y orthogonal to it, to 2^-22 of w)
    rho += 0x1p-20 * w;
    w += 0x1p-20 * w;
}

// Prepared mesh: the S_NTRI fields of the t-th triangle in the tree's order and
// the cylinders of levels 0, 1 and 2 (one wave per 64 triangles; indices are
// clamped into the mesh so that invalid contents never address other memory).
__global__ __launch_bounds__(64) void k_seg_mesh(const double *xyz, int64_t nv, const int32_t *tri, int64_t nt,
                                                 const int32_t *order, const unsigned long long *box, double *P,
                                                 float4 *nodes, SegTree T) {
    const SegFrame F = seg_frame(box);
    const int64_t t = blockIdx.x * (int64_t)64 + threadIdx.x;
    const bool in = t < nt;
    double x[9], a[3];
    double f[F_NTRI];
    TriRef<double> R{f, 1};
    const int64_t ti = order[in ? t : nt - 1];
    for (int k = 0; k < 3; k++) {
        const int32_t v = tri[3 * ti + k];
        const int64_t vi = (v >= 0 && (int64_t)v < nv) ? v : 0;
        for (int c = 0; c < 3; c++) {
            f[F_V + 3 * k + c] = xyz[3 * vi + c];
            x[3 * k + c] = (f[F_V + 3 * k + c] - F.c[c]) * F.s;
        }
    }
    tri_prep64(R);
    if (in) {
        double *q = P + t * S_NTRI;
        for (int k = 0; k < 9; k++) q[S_V + k] = f[F_V + k];
        for (int k = 0; k < 3; k++) q[S_IE + k] = f[F_IE + k];
        for (int k = 0; k < 3; k++) q[S_G1 + k] = f[F_G1 + k];
        for (int k = 0; k < 3; k++) q[S_G2 + k] = f[F_G2 + k];
        // in the frame (a scale by a power of two)
        const double g = 1.0 / F.s;
        float4 *o = nodes + 2 * (int64_t)T.nodes + SEG_TRI4 * t;
        o[0] = make_float4((float)x[0], (float)x[1], (float)x[2], (float)x[3]);
        o[1] = make_float4((float)x[4], (float)x[5], (float)x[6], (float)x[7]);
        o[2] = make_float4((float)x[8], (float)(f[F_G1] * g), (float)(f[F_G1 + 1] * g), (float)(f[F_G1 + 2] * g));
        o[3] = make_float4((float)(f[F_G2] * g), (float)(f[F_G2 + 1] * g), (float)(f[F_G2 + 2] * g),
                           (float)(f[F_IE] * g * g));
        o[4] = make_float4((float)(f[F_IE + 1] * g * g), (float)(f[F_IE + 2] * g * g), 0.0f, 0.0f);
    }
    for (int k = 0; k < 3; k++) {
        const int i = (k + 1) % 3, j = (k + 2) % 3;
        a[k] = (x[3 + i] - x[i]) * (x[6 + j] - x[j]) - (x[3 + j] - x[j]) * (x[6 + i] - x[i]);
    }
    float c[3], n[3];
    double rho = 0.0, w = 0.0;
    // level 0: the centroid, a surface point (upper bounds are taken from it)
    unit_dir(a, n);
    for (int k = 0; k < 3; k++) c[k] = (float)((x[k] + x[3 + k] + x[6 + k]) * (1.0 / 3.0));
    for (int k = 0; k < 3; k++) {
        const double d0 = x[3 * k] - c[0], d1 = x[3 * k + 1] - c[1], d2 = x[3 * k + 2] - c[2];
        const double h = n[0] * d0 + n[1] * d1 + n[2] * d2;
        const double l0 = d0 - h * n[0], l1 = d1 - h * n[1], l2 = d2 - h * n[2];
        rho = fmax(rho, sqrt(l0 * l0 + l1 * l1 + l2 * l2));
        w = fmax(w, fabs(h));
    }
    if (in) write_node(nodes, T.off[0] + t, c, rho + 0x1p-20 * w, n, w + 0x1p-20 * w);
    group_node<8>(x, a, in, c, n, rho, w);
    if (in && (threadIdx.x & 7) == 0) write_node(nodes, T.off[1] + t / 8, c, rho, n, w);
    if (T.top >= 2) {
        group_node<64>(x, a, in, c, n, rho, w);
        if (in && threadIdx.x == 0) write_node(nodes, T.off[2] + t / 64, c, rho, n, w);
    }
}

// Levels 3 and up, each from the level below (one block; a mesh of 2^25
// triangles has 2^16 nodes in level 3).  A lane takes a child, eight lanes a
// node: a level is one round of loads and a few reductions (a thread a node,
// walking its children: 8.5 us for two levels, 4.7 now).
__global__ __launch_bounds__(1024) void k_seg_up(float4 *nodes, SegTree T) {
    auto dmin = [](double p, double q) { return fmin(p, q); };
    auto dmax = [](double p, double q) { return fmax(p, q); };
    auto dadd = [](double p, double q) { return p + q; };
    for (int l = 3; l <= T.top; l++) {
        const float4 *ch = nodes + 2 * (int64_t)T.off[l - 1];
        const int64_t n = T.cnt[l], nch = T.cnt[l - 1];
        // (a whole group of eight lanes goes round, or none of it)
        for (int64_t i = threadIdx.x / FAN; i < n; i += blockDim.x / FAN) {
            const int64_t j = i * FAN + threadIdx.x % FAN;
            const bool in = j < nch;
            const float4 a = ch[2 * (in ? j : nch - 1)], b = ch[2 * (in ? j : nch - 1) + 1];
            const double cc[3] = {a.x, a.y, a.z}, nn[3] = {b.x, b.y, b.z};
            const double rad = (double)a.w + (double)b.w;
            float c[3], m[3];
            double s[3];
            for (int k = 0; k < 3; k++) {
                const double lo = lanes_reduce<FAN>(in ? cc[k] - rad : __builtin_inf(), dmin);
                const double hi = lanes_reduce<FAN>(in ? cc[k] + rad : -__builtin_inf(), dmax);
                s[k] = lanes_reduce<FAN>(in ? nn[k] * (double)a.w * (double)a.w : 0.0, dadd);
                c[k] = (float)fmin(fmax(0.5 * lo + 0.5 * hi, -1.0), 1.0);
            }
            unit_dir(s, m);
            // the child's point c_j + a n_j + y: along m and across it
            const double d0 = cc[0] - c[0], d1 = cc[1] - c[1], d2 = cc[2] - c[2];
            const double h = m[0] * d0 + m[1] * d1 + m[2] * d2;
            const double l0 = d0 - h * m[0], l1 = d1 - h * m[1], l2 = d2 - h * m[2];
            const double co = fabs((double)m[0] * b.x + (double)m[1] * b.y + (double)m[2] * b.z);
            const double si = sqrt(fmax(1.0 - co * co, 0.0) + 0x1p-18);
            const double cw = fmin(co + 0x1p-18, 1.0 + 0x1p-18);
            const double r = sqrt(l0 * l0 + l1 * l1 + l2 * l2) + (double)a.w + (double)b.w * si;
            const double v = fabs(h) + (double)b.w * cw + (double)a.w * si;
            double rho = lanes_reduce<FAN>(in ? r : 0.0, dmax), w = lanes_reduce<FAN>(in ? v : 0.0, dmax);
            // (no two points of the frame are farther apart than 2 sqrt(3))
            rho = fmin((rho + 0x1p-18 * w) * (1.0 + 0x1p-18), 3.4642);
            w = fmin(w * (1.0 + 0x1p-18), 3.4642);
            if (threadIdx.x % FAN == 0) write_node(nodes, T.off[l] + i, c, rho, m, w);
        }
        __threadfence_block();
        __syncthreads();
    }
}

// The exact closed test for a pair the FP64 filter left undecided (rare; a
// call keeps its registers out of the common path).
__device__ __attribute__((noinline)) bool seg_pair_exact(const double *p, const double *q, const double *T) {
    double va[9], vb[9];
    for (int k = 0; k < 3; k++) {
        va[k] = p[k];
        va[3 + k] = va[6 + k] = q[k];
    }
    for (int k = 0; k < 9; k++) vb[k] = T[k];
    return ex::tri_tri_exact(va, vb);
}

// The pair test for intersects, where the signs alone leave a pair undecided:
// its separating direction settles most of these far faster than the exact
// test does (those of a long segment, whose signs the rounding of its extent
// hides: 10^6 extents long, 15.8 exact tests a segment, 1.4 with this).
__device__ __attribute__((noinline)) int seg_pair_settle(const double *p, const double *q, const double *T) {
    const double a[3] = {p[0], p[1], p[2]}, b[3] = {q[0], q[1], q[2]};
    return seg_pair64(a, b, T).status;
}

// A segment in the frame, in FP32.
struct SegF {
    float p[3], u[3], iu;  // p + t u, t in [0, 1]; iu = 1 / |u|^2 (0 for a point)
};

// Squared distance of the segment to c, and the offsets from c to its ends.
__device__ __forceinline__ float seg_point2(const SegF &s, const float4 &a, float (&r0)[3], float (&r1)[3]) {
    r0[0] = s.p[0] - a.x;
    r0[1] = s.p[1] - a.y;
    r0[2] = s.p[2] - a.z;
    float d = 0.0f, q = 0.0f;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        r1[k] = r0[k] + s.u[k];
        d = fmaf(r0[k], s.u[k], d);
    }
    const float t = fminf(fmaxf(-d * s.iu, 0.0f), 1.0f);
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const float w = fmaf(t, s.u[k], r0[k]);
        q = fmaf(w, w, q);
    }
    return q;
}

// Error of the FP32 cull.  With e = 2^-24 and S = q0 + q1 + 2 (q0, q1: the
// squared offsets of the segment's ends from c), rounding the segment into
// the frame moves it by at most e |p|, |p| <= |r| + sqrt(3), and every
// squared quantity below (q, h^2, l^2, d^2, the products with rho and w, both
// at most 2 sqrt(3)) is within 48 e S of its exact value; 64 e S is taken
// off, which leaves 2^-20 S >= 2^-20 of the squared extent of the segment and
// the mesh, far above the FP64 error of any pair distance and above the
// pruning margin of the mesh path (2^-36 of the extent).
constexpr float CULL_EPS = 0x1p-18f;

// A value at most the squared distance of the segment to the node, less the
// allowance.  For a point x = c + a n + y of the cylinder and p on the
// segment, |p - x|^2 >= |p - c|^2 - 2 |h| w - 2 l r + r^2 (h = n . (p - c), l
// the part of p - c across n, r = |y| <= rho): the segment's smallest |p - c|
// and its largest |h| and l (attained at an end) bound it.  Where both ends
// are on one side of the cylinder, (min |h| - w)^2 does too.  A segment beyond
// FP32's range of the mesh is NaN, so are its bounds, and these cull nothing.
// d2: the squared distance to c, up: that plus the allowance.
__device__ __forceinline__ float node_bound2(const SegF &s, const float4 &a, const float4 &b, float &up) {
    float r0[3], r1[3];
    const float d2 = seg_point2(s, a, r0, r1);
    const float n[3] = {b.x, b.y, b.z};
    float q0 = 0.0f, q1 = 0.0f, h0 = 0.0f, h1 = 0.0f;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        q0 = fmaf(r0[k], r0[k], q0);
        q1 = fmaf(r1[k], r1[k], q1);
        h0 = fmaf(n[k], r0[k], h0);
        h1 = fmaf(n[k], r1[k], h1);
    }
    const float S = q0 + q1 + 2.0f, slack = CULL_EPS * S;
    const float l2 = fmaxf(fmaxf(fmaf(-h0, h0, q0), fmaf(-h1, h1, q1)), 0.0f) + 0.5f * slack;
    const float l = __builtin_amdgcn_sqrtf(l2);
    const float g = l < a.w ? -l2 : a.w * fmaf(-2.0f, l, a.w);
    float B = fmaf(-2.0f * b.w, fmaxf(fabsf(h0), fabsf(h1)), d2 + g);
    const float hm = fminf(fabsf(h0), fabsf(h1)) - b.w;
    if (h0 * h1 > 0.0f && hm > 0.0f) B = fmaxf(B, hm * hm);
    up = d2 + slack;
    return B - slack;
}

// Bounds of the distance between a segment and a triangle of the frame in
// FP32, as pair32 takes them for two triangles: each candidate is the vector
// between a point of one and a point of the other up to rounding, the shortest
// bounds the distance from above, and the separation along it from below.
// With M the largest coordinate of the segment's ends and e = 2^-24, rounding
// into the frame moves the points by at most e sqrt(3) (3 M + 1), the vector
// and the separation (differences, three products, the quotient) add at most
// 40 e (3 M + 1) in all; 128 e (M + 1) is allowed.  A segment that is NaN
// (beyond FP32's range of the mesh) has no candidate: ub is +inf, lb (+inf
// times rsq(+inf) = 0) NaN, and neither decides anything.
struct SegBound {
    float ub, lb;
};
__device__ __forceinline__ SegBound seg_tri32(const SegF &s, const float4 *T) {
    const float4 a0 = T[0], a1 = T[1], a2 = T[2], a3 = T[3], a4 = T[4];
    const float v[9] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w, a2.x};
    const float g1[3] = {a2.y, a2.z, a2.w}, g2[3] = {a3.x, a3.y, a3.z}, ie[3] = {a3.w, a4.x, a4.y};
    float uu = 0.0f, M = 0.0f;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        uu = fmaf(s.u[k], s.u[k], uu);
        M = fmaxf(M, fmaxf(fabsf(s.p[k]), fabsf(s.p[k] + s.u[k])));
    }
    float best = __builtin_inff(), b[3] = {0.0f, 0.0f, 0.0f};
    float e0[3], e2[3];
#pragma unroll
    for (int l = 0; l < 3; l++) {
        float e[3], r[3], ee = 0.0f, bb = 0.0f, d = 0.0f, f = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            e[k] = v[3 * ((l + 1) % 3) + k] - v[3 * l + k];
            r[k] = s.p[k] - v[3 * l + k];
            if (l == 0) e0[k] = e[k];
            if (l == 2) e2[k] = e[k];
            ee = fmaf(e[k], e[k], ee);
            bb = fmaf(e[k], s.u[k], bb);
            d = fmaf(r[k], s.u[k], d);
            f = fmaf(r[k], e[k], f);
        }
        const float D = fmaf(uu, ee, -(bb * bb));
        float x = D > 0.0f ? fminf(fmaxf((bb * f - ee * d) * __builtin_amdgcn_rcpf(D), 0.0f), 1.0f) : 0.0f;
        const float y = fminf(fmaxf(fmaf(bb, x, f) * ie[l], 0.0f), 1.0f);
        x = fminf(fmaxf(fmaf(bb, y, -d) * s.iu, 0.0f), 1.0f);
        float w[3], q = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            w[k] = fmaf(x, s.u[k], fmaf(-y, e[k], r[k]));
            q = fmaf(w[k], w[k], q);
        }
        const bool better = q < best;
        best = better ? q : best;
#pragma unroll
        for (int k = 0; k < 3; k++) b[k] = better ? w[k] : b[k];
    }
#pragma unroll
    for (int i = 0; i < 2; i++) {
        float w[3], b1 = 0.0f, b2 = 0.0f, q = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            w[k] = (i ? s.p[k] + s.u[k] : s.p[k]) - v[k];
            b1 = fmaf(g1[k], w[k], b1);
            b2 = fmaf(g2[k], w[k], b2);
        }
#pragma unroll
        for (int k = 0; k < 3; k++) {
            w[k] = fmaf(b2, e2[k], fmaf(-b1, e0[k], w[k]));
            q = fmaf(w[k], w[k], q);
        }
        const bool better = b1 >= 0.0f && b2 >= 0.0f && b1 + b2 <= 1.0f && q < best;
        best = better ? q : best;
#pragma unroll
        for (int k = 0; k < 3; k++) b[k] = better ? w[k] : b[k];
    }
    float sep = __builtin_inff(), wu = 0.0f;
#pragma unroll
    for (int l = 0; l < 3; l++) {
        float h = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; k++) h = fmaf(b[k], s.p[k] - v[3 * l + k], h);
        sep = fminf(sep, h);
    }
#pragma unroll
    for (int k = 0; k < 3; k++) wu = fmaf(b[k], s.u[k], wu);
    sep += fminf(wu, 0.0f);
    const float err = 0x1p-17f * (M + 1.0f);
    return {sqrtf(best) * (1.0f + 0x1p-20f) + err,
            best > 0x1p-100f ? fmaf(sep, __builtin_amdgcn_rsqf(best), -err) : -__builtin_inff()};
}

// Squared FP32 threshold of an upper bound (frame units, rounded up).
__device__ __forceinline__ float cull2(float ub) {
    const float T = ub * (1.0f + 0x1p-20f);
    return T * T;
}

__device__ __forceinline__ void lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// MODE 0: distance (dist[i], hit[i] optional); 1: intersects (hit[i]);
// 2: within r (hit[i] = distance <= r).  cnt[0..2]: triangle bounds compared,
// full pair tests, exact tests (summed per wave, in replicas).
template <int MODE>
__global__ __launch_bounds__(64, 3) void k_segs(const double *seg, int64_t n, const double *P, int64_t nt,
                                             const float4 *nodes, SegTree T, const unsigned long long *box,
                                             double r, double *dist, uint8_t *hit, const uint32_t *flags,
                                             unsigned long long *cnt) {
    __shared__ float4 sf[2][64];             // in the frame: p and u.x, u.y u.z iu
    __shared__ unsigned long long best[MODE == 0 ? 64 : 1];  // squared distance bits
    __shared__ uint32_t ubf[MODE == 0 ? 64 : 1];  // upper bound in the frame, rounded up (bits)
    __shared__ uint32_t done[64];            // hit (MODE 0, 1) or within (MODE 2)
    __shared__ uint32_t tstk[STACK];         // live (triangle, segment) pairs and their bounds
    __shared__ float tlb[MODE == 0 ? STACK : 1];  // (the others' threshold stays, so these passed)
    constexpr int RDY = MODE == 0 ? 192 : 128;
    __shared__ uint32_t rdy[RDY];            // pairs to test, and MODE 0's bounds
    __shared__ float rlb[MODE == 0 ? RDY : 1];
    extern __shared__ uint32_t nstk[];       // (node, segment) pairs, STACK per level 1..top
    if (flags[0] | flags[1]) return;  // invalid contents: outputs stay untouched
    const int lane = lane_id();
    const unsigned long long below = lanes_below();
    const SegFrame F = seg_frame(box);
    const float rf = (float)(r * F.s) * (1.0f + 0x1p-22f);
    const float r2 = cull2(rf);                       // MODE 2: farther than r
    const float in2 = rf * rf * (1.0f - 0x1p-18f);    // a surface point this near: within r
    // lane l holds level l's first node and node count
    const int toff = lane < SEG_LEVELS ? (int)T.off[lane] : 0, tcnt = lane < SEG_LEVELS ? (int)T.cnt[lane] : 0;
    unsigned n_box = 0, n_full = 0, n_ex = 0;
    for (int64_t base = (int64_t)blockIdx.x * 64; base < n; base += (int64_t)gridDim.x * 64) {
        const int64_t i = base + lane;
        const bool mine = i < n;
        SegF me;
        {
            double p[3], u[3], pp = 0.0, uu = 0.0, pu = 0.0;
            for (int c = 0; c < 3; c++) {
                const double x = mine ? seg[6 * i + c] : 0.0, y = mine ? seg[6 * i + 3 + c] : 0.0;
                p[c] = (x - F.c[c]) * F.s;
                u[c] = (y - x) * F.s;
                pp += p[c] * p[c];
                uu += u[c] * u[c];
                pu += p[c] * u[c];
            }
            // a long segment is cut (FP32 offsets stay small; up to 2^26 frame
            // units, where FP64 places a cut, and a pair's distance, to 2^-21)
            const bool cut = uu < 0x1p52 && pp < 0x1p52;
            if (MODE == 0 && cut && uu > 64.0) {
                // to where the mesh's nearest point can be: the mesh lies
                // within sqrt(3) of the frame's origin, so within d + 1.75 of
                // the segment (d its distance to the origin), and a point of
                // it more than d + 3.5 from the origin is farther than that
                // from all of the mesh
                const double t = fmin(fmax(-pu / uu, 0.0), 1.0);
                double d2 = 0.0;
                for (int c = 0; c < 3; c++) d2 += (p[c] + t * u[c]) * (p[c] + t * u[c]);
                const double d = sqrt(d2) + 3.5;
                const double half = sqrt(fmax(d * d - d2, 0.0) / uu) * 1.0001 + 1e-9;
                const double t0 = fmax(t - half, 0.0), t1 = fmin(t + half, 1.0);
                for (int c = 0; c < 3; c++) {
                    p[c] += t0 * u[c];
                    u[c] *= t1 - t0;
                }
            }
            if (MODE != 0 && cut && uu > 0.25) {
                // to the mesh's box, wider by the threshold: the nodes' bounds
                // weaken with the segment's length (through 20,000 loose
                // triangles, one segment 30 long: the call 167 -> 64 us; 100,000:
                // 4.00 -> 0.66 ms)
                double t0 = 0.0, t1 = 1.0;
                const double e = (MODE == 2 ? r * F.s : 0.0) + 0x1p-16;
                for (int c = 0; c < 3; c++) {
                    const double lo = (from_ordered_bits(box[c]) - F.c[c]) * F.s - e;
                    const double hi = (from_ordered_bits(box[3 + c]) - F.c[c]) * F.s + e;
                    if (u[c] != 0.0) {
                        const double x0 = (lo - p[c]) / u[c], x1 = (hi - p[c]) / u[c];
                        t0 = fmax(t0, fmin(x0, x1));
                        t1 = fmin(t1, fmax(x0, x1));
                    } else if (p[c] < lo || p[c] > hi) {
                        t1 = -1.0;
                    }
                }
                // (nothing of it near: any point of it stands for it)
                if (!(t0 <= t1)) t0 = t1 = fmin(fmax(-pu / uu, 0.0), 1.0);
                for (int c = 0; c < 3; c++) {
                    p[c] += t0 * u[c];
                    u[c] *= t1 - t0;
                }
            }
            // a segment with an end beyond 2^56 frame units is NaN: its FP32
            // products could overflow one by one, which would leave bounds
            // that look like any other
            double far = 0.0;
            for (int c = 0; c < 3; c++) far = fmax(far, fmax(fabs(p[c]), fabs(p[c] + u[c])));
            float q = 0.0f;
            for (int c = 0; c < 3; c++) {
                me.p[c] = far < 0x1p56 ? (float)p[c] : __builtin_nanf("");
                me.u[c] = far < 0x1p56 ? (float)u[c] : __builtin_nanf("");
                q = fmaf(me.u[c], me.u[c], q);
            }
            me.iu = q > 0.0f ? 1.0f / q : 0.0f;
        }
        sf[0][lane] = make_float4(me.p[0], me.p[1], me.p[2], me.u[0]);
        sf[1][lane] = make_float4(me.u[1], me.u[2], me.iu, 0.0f);
        done[lane] = mine ? 0u : 1u;
        if (MODE == 0) {
            best[lane] = double_to_bits(__builtin_inf());
            ubf[lane] = __float_as_uint(__builtin_inff());
        }
        lds_sync();
        const float4 *tri32 = nodes + 2 * (int64_t)T.nodes;
        int cl = 0;  // lane l holds the pairs on level l's stack
        unsigned rc = 0;
        const int ntop = nt > 0 ? (int)T.cnt[T.top] : 0;
        int tt = 0;
        if (MODE == 0 && nt > 0) {
            // a first upper bound: that of the triangle that a way down the
            // tree by the nearest centre ends at (any one would do), so that
            // few nodes meet it
            uint32_t at = 0;
            float m = __builtin_inff();
            for (int t = 0; t < ntop; t++) {
                float r0[3], r1[3];
                const float d2 = seg_point2(me, nodes[2 * ((int64_t)T.off[T.top] + t)], r0, r1);
                at = d2 < m ? (uint32_t)t : at;
                m = fminf(m, d2);
            }
            for (int lv = T.top - 1; lv >= 0; lv--) {
                const float4 *cn = nodes + 2 * (int64_t)T.off[lv];
                const uint32_t ch = at * FAN, nch = T.cnt[lv];
                float4 na[FAN];
#pragma unroll
                for (int c = 0; c < FAN; c++) na[c] = cn[2 * (int64_t)min(ch + (uint32_t)c, nch - 1)];
                at = ch;
                m = __builtin_inff();
#pragma unroll
                for (int c = 0; c < FAN; c++) {
                    float r0[3], r1[3];
                    const float d2 = seg_point2(me, na[c], r0, r1);
                    at = d2 < m ? ch + (uint32_t)c : at;  // (past the end: the last child's equal)
                    m = fminf(m, d2);
                }
            }
            const SegBound sb = seg_tri32(me, tri32 + SEG_TRI4 * (int64_t)at);
            if (sb.ub >= 0.0f) ubf[lane] = __float_as_uint(sb.ub);
        }
        for (;;) {
            const unsigned long long full = __ballot(cl >= 64), any = __ballot(cl > 0);
            const bool last = !any && tt == ntop;
            if (rc > (unsigned)RDY - 64 || last) {
                lds_sync();
                if (MODE == 0) {
                    // (bounds have come down since)
                    unsigned m = 0;
                    for (unsigned c = 0; c < rc; c += 64) {
                        const unsigned j = min(c + (unsigned)lane, rc - 1);
                        const uint32_t e = rdy[j];
                        const float lb = rlb[j];
                        const bool keep =
                            c + (unsigned)lane < rc && !done[e & 63] && !(lb > __uint_as_float(ubf[e & 63]));
                        const unsigned long long mk = __ballot(keep);
                        lds_sync();
                        if (keep) {
                            rdy[m + __popcll(mk & below)] = e;
                            rlb[m + __popcll(mk & below)] = lb;
                        }
                        m += (unsigned)__popcll(mk);
                    }
                    rc = m;
                    lds_sync();
                }
                // test the last (at most 64) pairs of the ready list
                if (rc == 0 && last) break;
                if (rc < 64 && !last) continue;
                const unsigned k = min(rc, 64u);
                rc -= k;
                const uint32_t e = (unsigned)lane < k ? rdy[rc + lane] : 0u;
                const int slot = (int)(e & 63);
                if ((unsigned)lane < k && !done[slot]) {
                    const double *B = P + (int64_t)(e >> 6) * S_NTRI;
                    double p[3], q[3];
                    for (int c = 0; c < 3; c++) {
                        p[c] = seg[6 * (base + slot) + c];
                        q[c] = seg[6 * (base + slot) + 3 + c];
                    }
                    int st;
                    double d2 = 0.0;
                    if (MODE == 1) {
                        st = seg_tri_filtered64(p, q, B);
                        if (st == 2) st = seg_pair_settle(p, q, B);
                    } else {
                        const Pair64 pr = seg_pair64(p, q, B);
                        st = pr.status;
                        d2 = pr.d2;
                    }
                    n_full++;
                    if (st == 2) {
                        st = seg_pair_exact(p, q, B) ? 1 : 0;
                        n_ex++;
                    }
                    if (st == 1) {
                        atomicOr(&done[slot], 1u);
                    } else if (MODE == 0) {
                        atomicMin(&best[slot], double_to_bits(d2));
                        const float u = (float)(sqrt(d2) * F.s) * (1.0f + 0x1p-22f);
                        atomicMin(&ubf[slot], __float_as_uint(u));
                    } else if (MODE == 2 && sqrt(d2) <= r) {
                        atomicOr(&done[slot], 1u);
                    }
                }
                lds_sync();
                continue;
            }
            int lv;
            if (full) {
                lv = __ffsll(full) - 1;
            } else if (tt < ntop) {
                // the next top node against every segment of the wave
                const int64_t at = (int64_t)T.off[T.top] + tt;
                float up;
                const float B = node_bound2(me, nodes[2 * at], nodes[2 * at + 1], up);
                const float t2 = MODE == 0 ? cull2(__uint_as_float(ubf[lane])) : MODE == 2 ? r2 : 0.0f;
                const bool keep = !done[lane] && !(B > t2);
                const unsigned long long mk = __ballot(keep);
                const int c0 = __builtin_amdgcn_readlane(cl, T.top);
                if (keep) nstk[(T.top - 1) * STACK + c0 + __popcll(mk & below)] = (uint32_t)lane | ((uint32_t)tt << 6);
                if (lane == T.top) cl = c0 + __popcll(mk);
                tt++;
                continue;
            } else {
                lv = 63 - __clzll(any);
            }
            lds_sync();
            const int have = __builtin_amdgcn_readlane(cl, lv);
            const int k = min(have, 64), c0 = have - k;
            if (lane == lv) cl = c0;
            if (lv == 0) {
                const uint32_t e = lane < k ? tstk[c0 + lane] : 0u;
                const int slot = (int)(e & 63);
                bool keep = lane < k && !done[slot];
                if (MODE == 0) keep = keep && !(tlb[c0 + (lane < k ? lane : 0)] > cull2(__uint_as_float(ubf[slot])));
                float lb = 0.0f;
                if (MODE == 0 && keep) {
                    const float4 s0 = sf[0][slot], s1 = sf[1][slot];
                    const SegF sg{{s0.x, s0.y, s0.z}, {s0.w, s1.x, s1.y}, s1.z};
                    const SegBound sb = seg_tri32(sg, tri32 + SEG_TRI4 * (int64_t)(e >> 6));
                    lb = sb.lb;
                    if (sb.ub >= 0.0f) atomicMin(&ubf[slot], __float_as_uint(sb.ub));
                    keep = !(lb > fminf(sb.ub, __uint_as_float(ubf[slot])));
                }
                const unsigned long long mk = __ballot(keep);
                if (keep) {
                    rdy[rc + __popcll(mk & below)] = e;
                    if (MODE == 0) rlb[rc + __popcll(mk & below)] = lb;
                }
                rc += (unsigned)__popcll(mk);
                continue;
            }
            const uint32_t e = lane < k ? nstk[(lv - 1) * STACK + c0 + lane] : 0u;
            const int slot = (int)(e & 63);
            const bool on = lane < k && !done[slot];
            const float4 s0 = sf[0][slot], s1 = sf[1][slot];
            const SegF sg{{s0.x, s0.y, s0.z}, {s0.w, s1.x, s1.y}, s1.z};
            const uint32_t ch = (e >> 6) * FAN, nch = (uint32_t)__builtin_amdgcn_readlane(tcnt, lv - 1);
            const float4 *cn = nodes + 2 * (int64_t)(uint32_t)__builtin_amdgcn_readlane(toff, lv - 1);
            float4 na[FAN], nb[FAN];
#pragma unroll
            for (int c = 0; c < FAN; c++) {
                const uint32_t j = min(ch + (uint32_t)c, nch - 1);
                na[c] = cn[2 * (int64_t)j];
                nb[c] = cn[2 * (int64_t)j + 1];
            }
            float B[FAN], m = __builtin_inff();
#pragma unroll
            for (int c = 0; c < FAN; c++) {
                float up;
                B[c] = node_bound2(sg, na[c], nb[c], up);
                m = fminf(m, up);
            }
            float t2 = MODE == 2 ? r2 : 0.0f;
            if (MODE == 0) {
                t2 = cull2(__uint_as_float(ubf[slot]));
                if (lv == 1) {  // (the children's centres are surface points)
                    const float u = sqrtf(m) * (1.0f + 0x1p-22f);
                    if (on && u >= 0.0f) {
                        atomicMin(&ubf[slot], __float_as_uint(u));
                        t2 = fminf(t2, cull2(u));
                    }
                }
            }
            if (MODE == 2 && lv == 1 && on && m <= in2 && m < __builtin_inff()) {
                atomicOr(&done[slot], 1u);
                t2 = -1.0f;
            }
            int cc = __builtin_amdgcn_readlane(cl, lv - 1);
#pragma unroll
            for (int c = 0; c < FAN; c++) {
                const bool keep = on && ch + (uint32_t)c < nch && !(B[c] > t2);
                const unsigned long long mk = __ballot(keep);
                const int at = cc + __popcll(mk & below);
                const uint32_t en = (uint32_t)slot | ((ch + (uint32_t)c) << 6);
                if (lv == 1) {
                    if (keep) {
                        tstk[at] = en;
                        if (MODE == 0) tlb[at] = B[c];
                    }
                } else if (keep) {
                    nstk[(lv - 2) * STACK + at] = en;
                }
                cc += __popcll(mk);
            }
            if (lane == lv - 1) cl = cc;
            if (lv == 1) n_box += on ? (unsigned)min((uint32_t)FAN, nch - ch) : 0u;
        }
        if (mine) {
            if (MODE == 0) {
                const bool h = done[lane] != 0;
                dist[i] = h ? 0.0 : sqrt(bits_to_double(best[lane]));
                if (hit) hit[i] = h ? 1 : 0;
            } else {
                hit[i] = done[lane] ? 1 : 0;
            }
        }
        lds_sync();
    }
    const unsigned long long tb = wave_sum((unsigned long long)n_box), tf = wave_sum((unsigned long long)n_full),
                             te = wave_sum((unsigned long long)n_ex);
    if (lane == 0) {
        if (tb) atomicAdd(counter_of(cnt, 0), tb);
        if (tf) atomicAdd(counter_of(cnt, 1), tf);
        if (te) atomicAdd(counter_of(cnt, 2), te);
    }
}

// Flags and counters to 0, the mesh box to the empty one.
__global__ void k_seg_clear(uint32_t *flags, unsigned long long *cnt, unsigned long long *box) {
    if (threadIdx.x < 2) flags[threadIdx.x] = 0;
    if (threadIdx.x < C_REPLICAS * C_NCOUNTERS) cnt[threadIdx.x] = 0;
    if (threadIdx.x < 6) box[threadIdx.x] = threadIdx.x < 3 ? ~0ull : 0ull;
}

SegTree seg_tree(int64_t nt) {
    // the top level is the lowest with at most 16 nodes: a node tested there
    // costs every lane one test, one tested below it only the lanes that need
    // it (and the tree of 2^25 triangles has 7 levels)
    SegTree T{};
    int64_t at = 0, c = nt;
    for (int l = 0; l < SEG_LEVELS; l++) {
        T.off[l] = (uint32_t)at;
        T.cnt[l] = (uint32_t)c;
        T.top = l;
        at += c;
        T.nodes = at;
        if (l >= 1 && c <= 16) break;
        c = (c + FAN - 1) / FAN;
    }
    return T;
}

void launch_seg_validate(const double *seg, int64_t n, const double *xyz, int64_t nv, const int32_t *tri,
                         int64_t nt, int32_t *order, uint32_t *flags, unsigned long long *cnt,
                         unsigned long long *box, hipStream_t s) {
    hipLaunchKernelGGL(k_seg_clear, dim3(1), dim3(C_REPLICAS * C_NCOUNTERS), 0, s, flags, cnt, box);
    const int64_t work = std::max<int64_t>(6 * n, std::max<int64_t>(3 * nv, 3 * nt));
    const int64_t runs = (nt + RS_ITEMS - 1) / RS_ITEMS;
    const unsigned grid = (unsigned)(runs + std::min<int64_t>(std::max<int64_t>((work + 1023) / 1024, 1), 512));
    hipLaunchKernelGGL(k_seg_validate, dim3(grid), dim3(1024), 0, s, seg, n, xyz, nv, tri, nt, order, flags, box);
}

void launch_seg_mesh(const double *xyz, int64_t nv, const int32_t *tri, int64_t nt, const SegTree &T,
                     const unsigned long long *box, const int32_t *order, double *P, float *nodes, hipStream_t s) {
    if (nt <= 0) return;
    hipLaunchKernelGGL(k_seg_mesh, dim3((unsigned)((nt + 63) / 64)), dim3(64), 0, s, xyz, nv, tri, nt, order, box, P,
                       (float4 *)nodes, T);
    if (T.top >= 3) hipLaunchKernelGGL(k_seg_up, dim3(1), dim3(1024), 0, s, (float4 *)nodes, T);
}

static size_t seg_lds(const SegTree &T) { return sizeof(uint32_t) * STACK * (size_t)T.top; }

int seg_blocks_per_cu(int mode, const SegTree &T) {
    int b = 0;
    const size_t lds = seg_lds(T);
    hipError_t e = mode == 0   ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_segs<0>, 64, lds)
                   : mode == 1 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_segs<1>, 64, lds)
                               : hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_segs<2>, 64, lds);
    return e == hipSuccess && b > 0 ? b : 1;
}

void launch_segs(int mode, const double *seg, int64_t n, const double *P, int64_t nt, const SegTree &T,
                 const float *nodes, const unsigned long long *box, double r, double *dist, uint8_t *hit,
                 const uint32_t *flags, unsigned long long *cnt, int grid, hipStream_t s) {
    if (n <= 0) return;
    const unsigned g = (unsigned)std::min<int64_t>(grid, (n + 63) / 64);
    const size_t lds = seg_lds(T);
    const float4 *nd = (const float4 *)nodes;
    if (mode == 0)
        hipLaunchKernelGGL(k_segs<0>, dim3(g), dim3(64), lds, s, seg, n, P, nt, nd, T, box, r, dist, hit, flags, cnt);
    else if (mode == 1)
        hipLaunchKernelGGL(k_segs<1>, dim3(g), dim3(64), lds, s, seg, n, P, nt, nd, T, box, r, dist, hit, flags, cnt);
    else
        hipLaunchKernelGGL(k_segs<2>, dim3(g), dim3(64), lds, s, seg, n, P, nt, nd, T, box, r, dist, hit, flags, cnt);
}

}  // namespace sd3
