// Scalar tail of the step: final (fixed-order, fp64) loss sum and the two-point scalar of
// Eq. 10 / Alg. 2, g = (L+ - L-)/(2 eps) or, one-sided, (L+ - L0)/eps.  Everything stays on the
// device so a step never synchronises the host.
#include "agzo_internal.h"

namespace agzo {

// this thread's share of sum(p[0..n)) for a 256-thread workgroup: four independent strided sums keep four loads in
// flight (the finishing kernels are one workgroup each, bound by latency); the order is fixed
__device__ __forceinline__ double strided_sum4(const double* __restrict__ p, int n, int tid) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int i = tid;
    for (; i + 768 < n; i += 1024) {
        s0 += p[i]; s1 += p[i + 256]; s2 += p[i + 512]; s3 += p[i + 768];
    }
    for (; i < n; i += 256) s0 += p[i];
    return (s0 + s1) + (s2 + s3);
}

__global__ __launch_bounds__(256) void finish_loss_kernel(const double* __restrict__ partials, int n, double scale,
                                                          double* __restrict__ out) {
    __shared__ double red[256];
    const int tid = threadIdx.x;
    red[tid] = strided_sum4(partials + (int64_t)blockIdx.x * n, n, tid);
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (tid < k) red[tid] += red[tid + k];
        __syncthreads();
    }
    if (tid == 0) out[blockIdx.x] = red[0] * scale;
}

// out4 = {L0, L+, L-, g}
__global__ void two_point_kernel(double* __restrict__ out4, float eps, int one_sided) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const double e = (double)eps;
        if (one_sided) {
            out4[2] = 0.0;   // L- is not evaluated in the one-sided form
            out4[3] = (out4[1] - out4[0]) / e;
        } else {
            out4[3] = (out4[1] - out4[2]) / (2.0 * e);
        }
    }
}

// finish_loss for nphase (2 or 3) consecutive partial arrays and two_point: out4 = {L0, L+, L-, g}.  One workgroup per layer
// (seven launches of one workgroup each took 31 us of a layer set's step, one takes 5), the phases side by side; same
// summation order per loss as finish_loss_kernel.
struct FinishBatch { FinishTwoPointArgs a[kBatchMax]; };
__global__ __launch_bounds__(256) void finish_two_point_many_kernel(const FinishBatch tb, int nphase, float eps, int one_sided) {
    __shared__ double red[3][256];
    const FinishTwoPointArgs& a = tb.a[blockIdx.x];
    const int tid = threadIdx.x;
    double s[3];
#pragma unroll
    for (int ph = 0; ph < 3; ++ph) {
        s[ph] = ph < nphase ? strided_sum4(a.partials + (int64_t)ph * a.n, a.n, tid) : 0.0;
        red[ph][tid] = s[ph];
    }
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (tid < k) {
#pragma unroll
            for (int ph = 0; ph < 3; ++ph) red[ph][tid] += red[ph][tid + k];
        }
        __syncthreads();
    }
    if (tid == 0) {
        const double e = (double)eps, l0 = red[0][0] * a.scale, lp = red[1][0] * a.scale, lm = red[2][0] * a.scale;
        a.out4[0] = l0;
        a.out4[1] = lp;
        a.out4[2] = one_sided ? 0.0 : lm;      // L- is not evaluated in the one-sided form
        a.out4[3] = one_sided ? (lp - l0) / e : (lp - lm) / (2.0 * e);
    }
}

// ---- cross-entropy -----------------------------------------------------------------------------
// Merge the chunk statistics, loss_t = log(sum exp) - logit[target]; block sums of (loss, count) go to scratch[2*block], the
// last stage divides.  Bound by latency (16 MB for 8192 tokens of 250 chunks): 16 threads share a token and walk its chunks
// CE_FLIGHT loads at a time, sixteen tokens (128-byte runs) to a workgroup.  With a thread per token, 256 to a workgroup and two
// walks of one load at a time, it took 106 us for any number of tokens; this takes some 13 us for 385 or 3001.
constexpr int CE_TOK = kCeCombineTokens, CE_LANES = 256 / CE_TOK, CE_FLIGHT = 8;
__global__ __launch_bounds__(256) void ce_combine_kernel(const float2* __restrict__ ms, const float* __restrict__ tl,
                                                         const int32_t* __restrict__ target, int64_t M, int64_t N,
                                                         int nchunk, double* __restrict__ scratch) {
    __shared__ double rm[CE_LANES][CE_TOK], rs[CE_LANES][CE_TOK];
    const int tid = threadIdx.x, tok = tid % CE_TOK, part = tid / CE_TOK;
    const int ph = blockIdx.y;
    const int64_t t = (int64_t)blockIdx.x * CE_TOK + tok;
    // an id outside the layer's outputs has no logit: skipped
    const int tgt = t < M ? target[t] : -1;
    const bool counted = tgt >= 0 && tgt < N;
    double mx = -INFINITY, s = 0.0;
    if (counted) {
        const float2* m = ms + (int64_t)ph * nchunk * M + t;
        for (int c0 = part; c0 < nchunk; c0 += CE_LANES * CE_FLIGHT) {
            float2 v[CE_FLIGHT];
#pragma unroll
            for (int u = 0; u < CE_FLIGHT; ++u) {
                // (never conditional: around a condition the compiler waits for each load before the next)
                v[u] = m[(int64_t)min(c0 + u * CE_LANES, nchunk - 1) * M];
            }
#pragma unroll
            for (int u = 1; u < CE_FLIGHT; ++u)
                if (c0 + u * CE_LANES >= nchunk) v[u] = make_float2(-INFINITY, 0.f);
            float top = v[0].x;                                // (the first of the eight exists)
#pragma unroll
            for (int u = 1; u < CE_FLIGHT; ++u) top = fmaxf(top, v[u].x);
            const double mn = fmax(mx, (double)top);
            // nothing to move to a new maximum while there is no sum yet (and no -inf - -inf)
            s = s > 0.0 ? s * exp(mx - mn) : s;
#pragma unroll
            for (int u = 0; u < CE_FLIGHT; ++u)
                if (v[u].y != 0.f) s += (double)v[u].y * exp((double)v[u].x - mn);      // (0: a chunk past the last column, maximum -inf)
            mx = mn;
        }
    }
    rm[part][tok] = mx;
    rs[part][tok] = s;
    __syncthreads();
    if (part != 0) return;
    double loss = 0.0, cnt = 0.0;
    if (counted) {
        for (int l = 1; l < CE_LANES && l < nchunk; ++l) mx = fmax(mx, rm[l][tok]);
        s = 0.0;
        for (int l = 0; l < CE_LANES && l < nchunk; ++l) s += rs[l][tok] * exp(rm[l][tok] - mx);
        loss = log(s) + mx - (double)tl[(int64_t)ph * M + t];
        cnt = 1.0;
    }
    // (the first CE_TOK lanes of wave 0)
#pragma unroll
    for (int off = CE_TOK / 2; off > 0; off >>= 1) {
        loss += __shfl_xor(loss, off);
        cnt += __shfl_xor(cnt, off);
    }
    if (tid == 0) {
        scratch[((int64_t)ph * gridDim.x + blockIdx.x) * 2] = loss;
        scratch[((int64_t)ph * gridDim.x + blockIdx.x) * 2 + 1] = cnt;
    }
}

__global__ __launch_bounds__(256) void ce_finish_kernel(const double* __restrict__ scratch, int nblk, double* __restrict__ out) {
    __shared__ double rs[256], rc[256];
    const int tid = threadIdx.x, ph = blockIdx.x;
    double s = 0.0, c = 0.0;
    for (int i = tid; i < nblk; i += 256) {
        s += scratch[((int64_t)ph * nblk + i) * 2];
        c += scratch[((int64_t)ph * nblk + i) * 2 + 1];
    }
    rs[tid] = s; rc[tid] = c;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (tid < k) { rs[tid] += rs[tid + k]; rc[tid] += rc[tid + k]; }
        __syncthreads();
    }
    if (tid == 0) out[ph] = rc[0] > 0.0 ? rs[0] / rc[0] : 0.0;
}

hipError_t launch_ce_combine(const void* ms, const float* tl, const int32_t* target, int64_t M, int64_t N, int nchunk,
                             int nphase, double* scratch, double* out, hipStream_t st) {
    const int nblk = (int)((M + CE_TOK - 1) / CE_TOK);
    hipLaunchKernelGGL(ce_combine_kernel, dim3(nblk, nphase), dim3(256), 0, st, reinterpret_cast<const float2*>(ms), tl,
                       target, M, N, nchunk, scratch);
    hipLaunchKernelGGL(ce_finish_kernel, dim3(nphase), dim3(256), 0, st, scratch, nblk, out);
    return hipGetLastError();
}

// fp32-storage path: one workgroup per token row of stored logits, fp64 statistics
__global__ __launch_bounds__(256) void ce_rows_f32_kernel(const float* __restrict__ Y, int64_t ldy, int64_t M, int64_t N,
                                                          const int32_t* __restrict__ target, double* __restrict__ scratch) {
    __shared__ double red[256];
    const int tid = threadIdx.x;
    const int64_t t = blockIdx.x;
    const int tgt = target[t];
    if (tgt < 0 || tgt >= N) {   // ignored row; an id outside the layer's outputs has no logit and is skipped too
        if (tid == 0) { scratch[t * 2] = 0.0; scratch[t * 2 + 1] = 0.0; }
        return;
    }
    const float* y = Y + t * ldy;
    double mx = -INFINITY;
    for (int64_t j = tid; j < N; j += 256) mx = fmax(mx, (double)y[j]);
    red[tid] = mx;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (tid < k) red[tid] = fmax(red[tid], red[tid + k]);
        __syncthreads();
    }
    mx = red[0];
    __syncthreads();
    double s = 0.0;
    for (int64_t j = tid; j < N; j += 256) s += exp((double)y[j] - mx);
    red[tid] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (tid < k) red[tid] += red[tid + k];
        __syncthreads();
    }
    if (tid == 0) {
        scratch[t * 2] = log(red[0]) + mx - (double)y[tgt];
        scratch[t * 2 + 1] = 1.0;
    }
}

hipError_t launch_ce_rows_f32(const float* Y, int64_t ldy, int64_t M, int64_t N, const int32_t* target, double* scratch,
                              double* out, hipStream_t st) {
    hipLaunchKernelGGL(ce_rows_f32_kernel, dim3((unsigned)M), dim3(256), 0, st, Y, ldy, M, N, target, scratch);
    hipLaunchKernelGGL(ce_finish_kernel, dim3(1), dim3(256), 0, st, scratch, (int)M, out);
    return hipGetLastError();
}

hipError_t launch_finish_loss(const double* partials, int n, double scale, double* out, int nout, hipStream_t st) {
    hipLaunchKernelGGL(finish_loss_kernel, dim3(nout), dim3(256), 0, st, partials, n, scale, out);
    return hipGetLastError();
}

hipError_t launch_finish_two_point_many(const FinishTwoPointArgs* a, int n, int nphase, float eps, int one_sided, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    if (n == 0) return hipSuccess;
    FinishBatch tb;
    for (int i = 0; i < n; ++i) tb.a[i] = a[i];
    hipLaunchKernelGGL(finish_two_point_many_kernel, dim3((unsigned)n), dim3(256), 0, st, tb, nphase, eps, one_sided);
    return hipGetLastError();
}

hipError_t launch_two_point(double* out4, float eps, int one_sided, hipStream_t st) {
    hipLaunchKernelGGL(two_point_kernel, dim3(1), dim3(64), 0, st, out4, eps, one_sided);
    return hipGetLastError();
}

}  // namespace agzo
