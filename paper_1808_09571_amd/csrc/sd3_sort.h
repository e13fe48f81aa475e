// Morton codes and the stable sort of one block's items in LDS, shared by the
// mesh path's keys and the segment path's mesh order.
#pragma once
#include "sd3_kernels.h"

namespace sd3 {

__device__ __forceinline__ uint32_t spread10(uint32_t x) {
    x &= 0x3ffu;
    x = (x | (x << 16)) & 0x030000ffu;
    x = (x | (x << 8)) & 0x0300f00fu;
    x = (x | (x << 4)) & 0x030c30c3u;
    x = (x | (x << 2)) & 0x09249249u;
    return x;
}

// Cells of a row: the origin (box minimum) and the scale mapping the largest
// extent onto 1024 cells, from the six ordered-bit box components.
__device__ __forceinline__ double row_cells(const unsigned long long *b, double lo[3]) {
    double ext = 0.0;
    for (int k = 0; k < 3; k++) {
        lo[k] = from_ordered_bits(b[k]);
        ext = fmax(ext, from_ordered_bits(b[3 + k]) - lo[k]);
    }
    return ext > 0.0 ? 1024.0 / ext : 0.0;
}

// 30-bit Morton code of point p on those cells.
__device__ __forceinline__ uint32_t morton_code(const double *p, const double *lo, double sc) {
    uint32_t q[3];
    for (int k = 0; k < 3; k++) {
        const double f = (p[k] - lo[k]) * sc;
        const int qi = (int)f;
        q[k] = (uint32_t)(qi < 0 ? 0 : (qi > 1023 ? 1023 : qi));
    }
    return spread10(q[0]) | (spread10(q[1]) << 1) | (spread10(q[2]) << 2);
}

// Inclusive prefix sum over the wave on DPP lane moves (every lane active):
// shifts by 1, 2, 4 and 8 lanes within each row of 16 (lanes with no source
// add 0), then the broadcasts of lane 15 to the next row and of lane 31 to
// the upper half.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

// One stable pass of 8 bits over a block's n items in LDS (the key in the
// upper 16 bits, the index below): wave w ranks items [w q, w q + q), q a
// multiple of 64, with ballots, and places them behind the lower digits' items
// and the earlier waves'.
struct LocalSort {
    uint32_t a[RS_ITEMS], b[RS_ITEMS];
    uint32_t wc[16][256];  // per-wave digit counts, then places
    uint32_t part[4];
};
__device__ __forceinline__ void local_pass(LocalSort &S, const uint32_t *src, uint32_t *dst, int n, int shift) {
    const int tid = (int)threadIdx.x, w = tid >> 6, lane = lane_id();
    for (int k = tid; k < 16 * 256; k += 1024) S.wc[k >> 8][k & 255] = 0;
    __syncthreads();
    constexpr int R = RS_ITEMS / 1024;  // rounds per wave
    uint32_t x[R], rk[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int j = (w * R + r) * 64 + lane;
        const bool in = j < n;
        x[r] = in ? src[j] : 0u;
        const uint32_t d = (x[r] >> shift) & 255u;
        unsigned long long peers = __ballot(in);
#pragma unroll
        for (int bit = 0; bit < 8; bit++) {
            const unsigned long long m = __ballot((d >> bit) & 1u);
            peers &= ((d >> bit) & 1u) ? m : ~m;
        }
        const uint32_t before = in ? S.wc[w][d] : 0u;
        __builtin_amdgcn_wave_barrier();
        const uint32_t rank = (uint32_t)__popcll(peers & lanes_below());
        rk[r] = before + rank;
        if (in && rank == 0) S.wc[w][d] = before + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    uint32_t c[16], tot = 0, inc = 0;
    if (tid < 256) {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            c[k] = S.wc[k][tid];
            tot += c[k];
        }
        inc = wave_incl_scan(tot);
        if (lane == 63) S.part[w] = inc;
    }
    __syncthreads();
    if (tid < 256) {
        uint32_t run = inc - tot;
        for (int k = 0; k < w; k++) run += S.part[k];
#pragma unroll
        for (int k = 0; k < 16; k++) {
            S.wc[k][tid] = run;
            run += c[k];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; r++)
        if ((w * R + r) * 64 + lane < n) dst[S.wc[w][(x[r] >> shift) & 255u] + rk[r]] = x[r];
    __syncthreads();
}

}  // namespace sd3
