// Extension operands of perturbed forwards: device code of the launches that write them (gemm_bf16.hip; skinny.hip, which writes the W side
// beside a narrow projection).
#pragma once
#include "agzo_internal.h"

namespace agzo {

// Extension operands of perturbed forwards, written once per layer instead of once per tile.
// Rows 0..M-1 are the X side ([Ph | Ph | Pl | 0], P = X B split hi + lo in bf16), rows M..M+N-1 the W side
// ([Gh | Gl | Gh | 0], G regenerated from the Philox seed, times coef: the signed eps); n_w = 2 adds rows M+N..M+2N-1, the
// W side once more with coef2 (the other sign's, or the shared-forward kernel's second pass, -2 eps).  Several layers per
// launch (fourteen launches of one operand set each took 62 us of a layer set's step).  M = 0 where the projection writes
// the X side itself; then the threads behind the W side split B into planes for that projection.
struct ExtDev {
    bf16_t* Xext; bf16_t* Wext;
    int64_t M, N; int ext_ld;
    const float* P; int r, rp;
    float coef, coef2; int n_w;
    uint32_t s_lo, s_hi;
    const float* B; bf16_t* planes; int64_t d;
};
// eight values as bf16 hi + lo
__device__ __forceinline__ void ext_split(const float (&v)[8], uint4& hi, uint4& lo) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        h[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
        l[i] = pack_bf16x2(v[2 * i] - __uint_as_float(h[i] << 16), v[2 * i + 1] - __uint_as_float(h[i] & 0xFFFF0000u));
    }
    hi = make_uint4(h[0], h[1], h[2], h[3]);
    lo = make_uint4(l[0], l[1], l[2], l[3]);
}
// columns k0 .. k0 + 7 of the segments [first | second | third | 0] of a row (the last one of rp columns, or not there)
__device__ __forceinline__ void ext_store(bf16_t* row, int ext_ld, int rp, int k0, uint4 first, uint4 second, uint4 third) {
    *reinterpret_cast<uint4*>(row + k0) = first;
    *reinterpret_cast<uint4*>(row + rp + k0) = second;
    *reinterpret_cast<uint4*>(row + 2 * rp + k0) = third;
    if (3 * rp < ext_ld) *reinterpret_cast<uint4*>(row + 3 * rp + k0) = make_uint4(0, 0, 0, 0);
}
// thread idx: eight columns of a row's segments, W side first; a row of the W side with both coefficients, so that its normals are made once
// (a thread for every sixteen bytes written made them three times for each; beside the sums of a projection, seven 4B-sized layers on
// 4096 tokens, r = 64, 30 us a launch and 20)
__device__ __forceinline__ void ext_prep_body(const ExtDev& a, int64_t idx) {
    const int ext_ld = a.ext_ld, r = a.r, rp = a.rp;
    const int64_t M = a.M, N = a.N;
    const int groups = rp / 8;
    if (idx >= (M + N) * groups) {
        // eight rows of one column of B
        const int64_t e = idx - (M + N) * groups;
        if (a.planes == nullptr || e >= a.d / 8 * rp) return;
        const int64_t i = e % (a.d / 8) * 8;
        const int k = (int)(e / (a.d / 8));
        uint32_t w[3][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bf16_t h[2], m[2], l[2];
#pragma unroll
            for (int v = 0; v < 2; ++v) split3_bf16(k < r ? a.B[(i + 2 * u + v) * r + k] : 0.f, h[v], m[v], l[v]);
            w[0][u] = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
            w[1][u] = (uint32_t)m[0] | ((uint32_t)m[1] << 16);
            w[2][u] = (uint32_t)l[0] | ((uint32_t)l[1] << 16);
        }
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint4*>(a.planes + ((int64_t)pl * rp + k) * a.d + i) = make_uint4(w[pl][0], w[pl][1], w[pl][2], w[pl][3]);
        return;
    }
    const int64_t row = idx / groups;
    const int k0 = (int)(idx - row * groups) * 8;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    uint4 hi, lo;
    if (row >= N) {
        const int64_t t = row - N;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (k0 + i < r) v[i] = a.P[t * r + k0 + i];
        ext_split(v, hi, lo);
        ext_store(a.Xext + t * ext_ld, ext_ld, rp, k0, hi, hi, lo);
        return;
    }
    if (k0 < r) {
        const float4 z = philox_normal4(a.s_lo, a.s_hi, AGZO_TAG_G, (uint32_t)row, (uint32_t)(k0 >> 2));
        v[0] = z.x; v[1] = z.y; v[2] = z.z; v[3] = z.w;
    }
    if (k0 + 4 < r) {
        const float4 z = philox_normal4(a.s_lo, a.s_hi, AGZO_TAG_G, (uint32_t)row, (uint32_t)((k0 >> 2) + 1));
        v[4] = z.x; v[5] = z.y; v[6] = z.z; v[7] = z.w;
    }
    for (int w = 0; w < a.n_w; ++w) {
        const float coef = w ? a.coef2 : a.coef;
        float c[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) c[i] = (k0 + i < r) ? coef * v[i] : 0.f;
        ext_split(c, hi, lo);
        ext_store(a.Wext + (row + w * N) * ext_ld, ext_ld, rp, k0, hi, lo, hi);
    }
}

// the W side of args (and the X side, from P, unless that is NULL) as the kernels take it, and the workgroups of `threads` for it
inline ExtDev ext_dev(const GemmExtArgs& a, uint64_t& workgroups, int threads = 256) {
    ExtDev d;
    d.M = a.M; d.N = a.N; d.ext_ld = gemm_bf16_ext_width(a.r);
    d.Xext = static_cast<bf16_t*>(a.ext_ws); d.Wext = d.Xext + d.M * d.ext_ld;
    if (!a.P) d.M = 0;
    d.B = a.B; d.planes = a.planes; d.d = a.d;
    d.P = a.P; d.r = a.r; d.rp = (a.r + 15) / 16 * 16;
    d.coef = a.coef; d.coef2 = a.coef2; d.n_w = a.two ? 2 : 1;
    d.s_lo = (uint32_t)a.seed; d.s_hi = (uint32_t)(a.seed >> 32);
    const int64_t items = (d.M + d.N) * (d.rp / 8) + (d.planes ? d.d / 8 * d.rp : 0);
    workgroups = (uint64_t)((items + threads - 1) / threads);
    return d;
}

}  // namespace agzo
