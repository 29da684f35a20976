// What sits between the linear layers of the gated-MLP stack workload (Alg. 2 over a model): RMS normalisation, the
// SiLU gate and the residual sum.  They are not steps of the method, only the model around it, but a whole-model step
// runs them three times per block, so they are single-pass kernels here: bf16 in and out, fp32 arithmetic, one
// rounding to bf16, 16-byte accesses.  All three are bound by HBM.
#include "agzo_internal.h"

namespace agzo {

__device__ __forceinline__ void unpack8(const uint4& v, float (&f)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(w[i] << 16);
        f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
}
__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
    return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
}

// y[t][:] = gain * x[t][:] / sqrt(mean(x[t][:]^2) + eps); one workgroup per row, d a multiple of 8
__global__ __launch_bounds__(256) void glue_rmsnorm_kernel(const bf16_t* __restrict__ x, int64_t ldx, bf16_t* __restrict__ y,
                                                           int64_t ldy, const float* __restrict__ gain, int64_t d, float eps) {
    __shared__ float red[4];
    const int tid = threadIdx.x;
    const bf16_t* xr = x + (int64_t)blockIdx.x * ldx;
    bf16_t* yr = y + (int64_t)blockIdx.x * ldy;
    const int64_t nvec = d / 8;
    float ss = 0.f;
    for (int64_t v = tid; v < nvec; v += 256) {
        float f[8];
        unpack8(*reinterpret_cast<const uint4*>(xr + v * 8), f);
#pragma unroll
        for (int i = 0; i < 8; ++i) ss = fmaf(f[i], f[i], ss);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    const float scale = rsqrtf(((red[0] + red[1]) + (red[2] + red[3])) / (float)d + eps);
    for (int64_t v = tid; v < nvec; v += 256) {          // the row is re-read from cache
        float f[8];
        unpack8(*reinterpret_cast<const uint4*>(xr + v * 8), f);
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = f[i] * scale * (gain ? gain[v * 8 + i] : 1.f);
        *reinterpret_cast<uint4*>(yr + v * 8) = pack8(f);
    }
}

// m = silu(a) * u, rows of d (multiple of 8) with leading dimensions
__global__ __launch_bounds__(256) void glue_swiglu_kernel(const bf16_t* __restrict__ a, int64_t lda, const bf16_t* __restrict__ u,
                                                          int64_t ldu, bf16_t* __restrict__ m, int64_t ldm, int64_t n, int64_t d) {
    const int64_t nvec = d / 8;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n * nvec) return;
    const int64_t row = idx / nvec, v = idx - row * nvec;
    float fa[8], fu[8];
    unpack8(*reinterpret_cast<const uint4*>(a + row * lda + v * 8), fa);
    unpack8(*reinterpret_cast<const uint4*>(u + row * ldu + v * 8), fu);
#pragma unroll
    for (int i = 0; i < 8; ++i) fa[i] = fa[i] / (1.f + __expf(-fa[i])) * fu[i];
    *reinterpret_cast<uint4*>(m + row * ldm + v * 8) = pack8(fa);
}

// h += delta (in place)
__global__ __launch_bounds__(256) void glue_add_kernel(bf16_t* __restrict__ h, int64_t ldh, const bf16_t* __restrict__ dl,
                                                       int64_t ldd, int64_t n, int64_t d) {
    const int64_t nvec = d / 8;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n * nvec) return;
    const int64_t row = idx / nvec, v = idx - row * nvec;
    float fh[8], fd[8];
    uint4* ph = reinterpret_cast<uint4*>(h + row * ldh + v * 8);
    unpack8(*ph, fh);
    unpack8(*reinterpret_cast<const uint4*>(dl + row * ldd + v * 8), fd);
#pragma unroll
    for (int i = 0; i < 8; ++i) fh[i] += fd[i];
    *ph = pack8(fh);
}

// ---------------------------------------------------------------------------
// Attention core of a decoder layer (grouped-query, causal, 128-wide heads, per-head RMS normalisation of queries and
// keys, rotary embedding): the model between the q / k / v projections and the o projection.  Three kernels.
//
// prep: q, k <- rope(rmsnorm_per_head(.)), head-major [seq][head][t][128]; v transposed to [seq][kv head][128][t_pad]
//       (t_pad = seq_len rounded up to 64, the padding zero) so that the second product reads keys contiguously.
// attention: four waves of 32 queries of one head (two groups of 16) against tiles of 64 keys that they share in LDS.  Scores are
//       computed transposed, S^T = K Q^T (keys x queries), with
//       v_mfma_f32_16x16x32_bf16: a lane then holds, for ONE query (column lane % 16), the scores of keys 4 g + e of each
//       16-key block (g = lane / 16), so the softmax's running maximum and sum are per-lane scalars up to a reduction
//       over the four g, and the rescaling of the output accumulators (out^T = V^T P^T, same column = query) is a
//       per-lane scalar too.  The eight probabilities a lane holds per 32 keys (two 16-key blocks) go straight into
//       the second product as its operand: a sum over keys does not care about their order, so instead of re-laying P
//       out, V^T is stored in the order P is held (of every 32 keys, those at 4 g .. 4 g + 3 of both blocks side by side).
//       Per tile and group of queries a wave has 512 cycles of matrix work, about as much exponential and other vector work (the
//       mask only on tiles that reach past the group, the rescaling only where a maximum moved) and 8 KB of LDS reads; two
//       workgroups per compute unit overlap them.  With every wave fetching its own K and V^T fragments from memory 16 x 512
//       tokens of 16 heads took 160 us, now 51 (340 TFLOP/s of causal work); prep with a thread's own angles per head 34, now 21.
// ---------------------------------------------------------------------------
constexpr int HEAD_DIM = 128;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

// 16 lanes per item: PREP_HEADS heads of q or of k at one token, which share the angles; the rotary pair (i, i + 64) sits 8 lanes
// apart
constexpr int PREP_HEADS = 4;
__global__ __launch_bounds__(256) void glue_qk_prep_kernel(const bf16_t* __restrict__ q, int64_t ldq, const bf16_t* __restrict__ k,
                                                           int64_t ldk, bf16_t* __restrict__ Qr, bf16_t* __restrict__ Kr, int n_seq,
                                                           int seq_len, int n_heads, int n_kv, float log2_theta) {
    const int64_t item = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4;
    const int j = threadIdx.x & 15;
    const int gq = (n_heads + PREP_HEADS - 1) / PREP_HEADS, gk = (n_kv + PREP_HEADS - 1) / PREP_HEADS;
    if (item >= (int64_t)n_seq * seq_len * (gq + gk)) return;              // whole 16-lane groups leave together
    const int64_t tok = item / (gq + gk);
    const int grp = (int)(item - tok * (gq + gk));
    const bool is_q = grp < gq;
    const int heads = is_q ? n_heads : n_kv, h0 = (is_q ? grp : grp - gq) * PREP_HEADS;
    const int seq = (int)(tok / seq_len), t = (int)(tok - (int64_t)seq * seq_len);
    const bf16_t* src = (is_q ? q + tok * ldq : k + tok * ldk) + h0 * HEAD_DIM + 8 * j;
    uint4 raw[PREP_HEADS];
#pragma unroll
    for (int h = 0; h < PREP_HEADS; ++h) raw[h] = h0 + h < heads ? *reinterpret_cast<const uint4*>(src + h * HEAD_DIM) : make_uint4(0, 0, 0, 0);
    float sn[8], cs[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int idx = 8 * (j & 7) + i;                                   // pair index 0..63
        const float inv = exp2f(-(float)idx * (2.0f / HEAD_DIM) * log2_theta);
        sincosf((float)t * inv, &sn[i], &cs[i]);
    }
    bf16_t* dst = (is_q ? Qr : Kr) + (((int64_t)seq * heads + h0) * seq_len + t) * HEAD_DIM + 8 * j;
#pragma unroll
    for (int h = 0; h < PREP_HEADS; ++h) {
        float f[8];
        unpack8(raw[h], f);
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) ss = fmaf(f[i], f[i], ss);
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) ss += __shfl_xor(ss, off);  // the 16 lanes of this head
        const float scale = rsqrtf(ss / (float)HEAD_DIM + 1e-6f);
        float o[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float mine = f[i] * scale;
            const float other = __shfl_xor(mine, 8);
            o[i] = (j < 8) ? mine * cs[i] - other * sn[i] : mine * cs[i] + other * sn[i];  // first half: x1 c - x2 s; second: x2 c + x1 s
        }
        if (h0 + h < heads) *reinterpret_cast<uint4*>(dst + (int64_t)h * seq_len * HEAD_DIM) = pack8(o);
    }
}

// Vt[seq][kv head][d][t_pad]: a thread takes 8 values of one token (16-byte load) and stores them to 8 rows; the lanes of
// a wave are consecutive tokens, so every store instruction writes 128 contiguous bytes.  Tokens >= seq_len write zeros.
// Of every 32 tokens, token 16 b + 4 g + e is stored at 8 g + 4 b + e.
__global__ __launch_bounds__(256) void glue_v_transpose_kernel(const bf16_t* __restrict__ v, int64_t ldv, bf16_t* __restrict__ Vt,
                                                               int n_seq, int seq_len, int t_pad, int n_kv) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    const int c = blockIdx.y % (HEAD_DIM / 8), head = blockIdx.y / (HEAD_DIM / 8), seq = blockIdx.z;
    if (t >= t_pad) return;
    uint4 raw = make_uint4(0, 0, 0, 0);
    if (t < seq_len) raw = *reinterpret_cast<const uint4*>(v + ((int64_t)seq * seq_len + t) * ldv + head * HEAD_DIM + 8 * c);
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
    const int at = (t & ~31) | ((t >> 2) & 3) * 8 | ((t >> 4) & 1) * 4 | (t & 3);
    bf16_t* dst = Vt + (((int64_t)seq * n_kv + head) * HEAD_DIM + 8 * c) * t_pad + at;
#pragma unroll
    for (int i = 0; i < 8; ++i) dst[(int64_t)i * t_pad] = (bf16_t)((i & 1) ? (w[i >> 1] >> 16) : (w[i >> 1] & 0xFFFFu));
}

// QG 16-query groups per wave: every K and V^T fragment a wave reads serves QG matrix instructions
constexpr int ATT_QG = 2;
constexpr int ATT_WAVE_Q = 16 * ATT_QG;     // queries per wave
constexpr int ATT_WG_Q = 4 * ATT_WAVE_Q;    // queries per workgroup
constexpr int ATT_KEYS = 64;                // keys per tile
constexpr int ATT_TILE = ATT_KEYS * HEAD_DIM * 2;        // bytes of a K or V^T tile
constexpr int ATT_SMEM = 4 * ATT_TILE;      // two stages of both

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void glue_attention_kernel(
        const bf16_t* __restrict__ Qr, const bf16_t* __restrict__ Kr, const bf16_t* __restrict__ Vt, bf16_t* __restrict__ out, int64_t ldo,
        int seq_len, int t_pad, int n_heads, int n_kv) {
    extern __shared__ __align__(16) char att_smem[];
    typedef __attribute__((address_space(3))) void* lptr_t;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int head = blockIdx.y, seq = blockIdx.z, kvh = head / (n_heads / n_kv);
    // heavy tiles first: the last queries of a sequence see the most keys
    const int wg_q0 = (int)(gridDim.x - 1 - blockIdx.x) * ATT_WG_Q, q0 = wg_q0 + wave * ATT_WAVE_Q;
    const bf16_t* Qh = Qr + ((int64_t)seq * n_heads + head) * seq_len * HEAD_DIM;
    auto rsrc = [](const bf16_t* base) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, (int)0xFFFFFFFFu, 0x00020000); };
    const bf16_t* Kh = Kr + ((int64_t)seq * n_kv + kvh) * seq_len * HEAD_DIM;
    const bf16_t* Vh = Vt + ((int64_t)seq * n_kv + kvh) * HEAD_DIM * t_pad;
    union Frag { uint4 u; bf16x8_t v; };
    const int tiles = (min(wg_q0 + ATT_WG_Q, seq_len) + ATT_KEYS - 1) / ATT_KEYS;      // that any query of this workgroup may see
    // direct loads of tile j into stage j & 1: K rows of 256 bytes (16-byte chunk c of row r at c ^ (r mod 16)), V^T rows of 128
    // bytes (chunk c at c ^ (r / 2 mod 8)); four of each per wave.  Keys past the end repeat the last one, masked.  (Lanes' offsets
    // have 32 bits: the tile and, in V^T, whose rows are as long as the sequence, the row group are part of the base)
    auto request = [&](int j) __attribute__((always_inline)) {
        char* stage = att_smem + (j & 1) * (2 * ATT_TILE) + wave * 4096;
        const __amdgpu_buffer_rsrc_t rk = rsrc(Kh + (int64_t)j * (ATT_KEYS * HEAD_DIM));
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int row = 16 * wave + 4 * t + (lane >> 4);
            const int off = min(row, seq_len - 1 - j * ATT_KEYS) * (HEAD_DIM * 2) + (((lane & 15) ^ (row & 15)) << 4);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lptr_t)(stage + t * 1024), 16, off, 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int row = 32 * wave + 8 * t + (lane >> 3);
            const __amdgpu_buffer_rsrc_t rv = rsrc(Vh + (int64_t)(32 * wave + 8 * t) * t_pad + (int64_t)j * ATT_KEYS);
            const uint32_t off = (uint32_t)(lane >> 3) * (2u * (uint32_t)t_pad) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lptr_t)(stage + ATT_TILE + t * 1024), 16, (int)off, 0, 0, 0);
        }
    };
    request(0);
    int qi[ATT_QG];                                                    // rows past the end repeat the last query, unstored
    Frag qf[ATT_QG][4];
#pragma unroll
    for (int qg = 0; qg < ATT_QG; ++qg) {
        qi[qg] = min(q0 + 16 * qg + n, seq_len - 1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) qf[qg][ks].u = *reinterpret_cast<const uint4*>(Qh + (int64_t)qi[qg] * HEAD_DIM + 32 * ks + 8 * g);
    }
    floatx4_t acc[ATT_QG][8];
#pragma unroll
    for (int qg = 0; qg < ATT_QG; ++qg)
#pragma unroll
        for (int db = 0; db < 8; ++db) acc[qg][db] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    float m_run[ATT_QG], t_run[ATT_QG], l_run[ATT_QG];                 // maximum of the raw scores, the same scaled and rounded
#pragma unroll
    for (int qg = 0; qg < ATT_QG; ++qg) { m_run[qg] = t_run[qg] = -INFINITY; l_run[qg] = 0.f; }
    const float sc = 1.44269504088896341f * 0.08838834764831845f;      // log2(e) / sqrt(128)
    for (int j = 0; j < tiles; ++j) {
        // this wave's loads of tile j have landed, then everybody's; everybody is done with the other stage
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (j + 1 < tiles) request(j + 1);
        const int kb = j * ATT_KEYS;
        if (kb > q0 + ATT_WAVE_Q - 1) continue;                        // no query of this wave sees the tile (wave-uniform)
        // (fragments are read as bf16x8_t: behind a read of another type the compiler waits for every direct load in flight)
        const char* ks_ = att_smem + (j & 1) * (2 * ATT_TILE);
        const char* vs_ = ks_ + ATT_TILE;
        floatx4_t s[ATT_QG][4];
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
            Frag kf[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) kf[ks].v = *reinterpret_cast<const bf16x8_t*>(ks_ + (16 * blk + n) * 256 + (((4 * ks + g) ^ n) << 4));
#pragma unroll
            for (int qg = 0; qg < ATT_QG; ++qg) {
                s[qg][blk] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    s[qg][blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks].v, qf[qg][ks].v, s[qg][blk], 0, 0, 0);
            }
        }
        // The probabilities are rounded to bf16 around the maximum so far, the tile's two groups of 32 keys one after the other: the
        // largest of a group is then exact more often than around one maximum of 64 (0.5 % of the outputs' error, and no less than
        // with steps of 32 keys)
        Frag pf[ATT_QG][2];
        float back[ATT_QG];                                            // what the second group's maximum scales the first by
        bool moved[ATT_QG];
        const bool mask = kb + ATT_KEYS - 1 > q0;                      // wave-uniform: some query ends inside the tile
#pragma unroll
        for (int qg = 0; qg < ATT_QG; ++qg) {
            // lane: query qi[qg] (column n), keys kb + 16 blk + 4 g + e
            if (mask) {
                const int last = qi[qg] - kb - 4 * g;
#pragma unroll
                for (int blk = 0; blk < 4; ++blk)
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[qg][blk][e] = 16 * blk + e <= last ? s[qg][blk][e] : -INFINITY;
            }
            float mx[2] = {m_run[qg], -INFINITY};
#pragma unroll
            for (int blk = 0; blk < 4; ++blk)
#pragma unroll
                for (int e = 0; e < 4; ++e) mx[blk >> 1] = fmaxf(mx[blk >> 1], s[qg][blk][e]);
#pragma unroll
            for (int off = 16; off < 64; off *= 2) {
                const float o0 = __shfl_xor(mx[0], off), o1 = __shfl_xor(mx[1], off);
                mx[0] = fmaxf(mx[0], o0);
                mx[1] = fmaxf(mx[1], o1);
            }
            mx[1] = fmaxf(mx[1], mx[0]);
            // a group of queries that sees none of these keys (its rows all lie before kb) keeps its state: mx = m_run,
            // alpha = 1, every p = 0.  On a group's first tile m_run = -inf and mx is finite (key 0 is visible).
            float top[2] = {t_run[qg], t_run[qg]};
            if (__any(mx[0] != m_run[qg])) {
                top[0] = top[1] = mx[0] * sc;
                const float alpha = __builtin_amdgcn_exp2f(t_run[qg] - top[0]);
                l_run[qg] *= alpha;
#pragma unroll
                for (int db = 0; db < 8; ++db)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[qg][db][e] *= alpha;
            }
            moved[qg] = __any(mx[1] != mx[0]);
            if (moved[qg]) top[1] = mx[1] * sc;
            back[qg] = __builtin_amdgcn_exp2f(top[0] - top[1]);
            m_run[qg] = mx[1];
            t_run[qg] = top[1];
            float p[16], psum[2] = {0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                p[i] = __builtin_amdgcn_exp2f(fmaf(s[qg][i >> 2][i & 3], sc, -top[i >> 3]));
                psum[i >> 3] += p[i];
            }
            l_run[qg] = fmaf(l_run[qg] + psum[0], back[qg], psum[1]);
#pragma unroll
            for (int h = 0; h < 2; ++h)
                pf[qg][h].u = make_uint4(pack_bf16x2(p[8 * h], p[8 * h + 1]), pack_bf16x2(p[8 * h + 2], p[8 * h + 3]),
                                         pack_bf16x2(p[8 * h + 4], p[8 * h + 5]), pack_bf16x2(p[8 * h + 6], p[8 * h + 7]));
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // (the second 32 keys may lie behind every query of the wave (wave-uniform): their probabilities are 0, but a value
            // there that is not finite would still make NaNs of sums that it is no part of)
            if (kb + 32 * h > q0 + ATT_WAVE_Q - 1) break;
            if (h == 1) {
#pragma unroll
                for (int qg = 0; qg < ATT_QG; ++qg)
                    if (moved[qg]) {
#pragma unroll
                        for (int db = 0; db < 8; ++db)
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[qg][db][e] *= back[qg];
                    }
            }
#pragma unroll
            for (int db = 0; db < 8; ++db) {
                Frag vf;                                               // dim 16 db + n, the keys in the order the probabilities are held
                vf.v = *reinterpret_cast<const bf16x8_t*>(vs_ + (16 * db + n) * 128 + (((4 * h + g) ^ ((n >> 1) & 7)) << 4));
#pragma unroll
                for (int qg = 0; qg < ATT_QG; ++qg) acc[qg][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf.v, pf[qg][h].v, acc[qg][db], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int qg = 0; qg < ATT_QG; ++qg) {
        float l = l_run[qg];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (q0 + 16 * qg + n >= seq_len) continue;
        const float inv = 1.f / l;
        bf16_t* orow = out + ((int64_t)seq * seq_len + q0 + 16 * qg + n) * ldo + head * HEAD_DIM + 4 * g;    // dims 16 db + 4 g + e
#pragma unroll
        for (int db = 0; db < 8; ++db)
            *reinterpret_cast<uint2*>(orow + 16 * db) = make_uint2(pack_bf16x2(acc[qg][db][0] * inv, acc[qg][db][1] * inv),
                                                                   pack_bf16x2(acc[qg][db][2] * inv, acc[qg][db][3] * inv));
    }
}

size_t glue_attention_workspace_bytes(int n_seq, int seq_len, int n_heads, int n_kv) {
    const int64_t t_pad = (seq_len + ATT_KEYS - 1) / ATT_KEYS * ATT_KEYS;
    return (size_t)n_seq * ((int64_t)(n_heads + n_kv) * seq_len + (int64_t)n_kv * t_pad) * HEAD_DIM * sizeof(bf16_t) + 256;
}

hipError_t launch_glue_attention(const bf16_t* q, int64_t ldq, const bf16_t* k, int64_t ldk, const bf16_t* v, int64_t ldv,
                                 bf16_t* out, int64_t ldo, int n_seq, int seq_len, int n_heads, int n_kv, float rope_theta,
                                 void* workspace, hipStream_t st) {
    if (n_seq == 0 || seq_len == 0) return hipSuccess;
    const int t_pad = (seq_len + ATT_KEYS - 1) / ATT_KEYS * ATT_KEYS;
    bf16_t* Qr = static_cast<bf16_t*>(workspace);
    bf16_t* Kr = Qr + (int64_t)n_seq * n_heads * seq_len * HEAD_DIM;
    bf16_t* Vt = Kr + (int64_t)n_seq * n_kv * seq_len * HEAD_DIM;
    const int64_t items = (int64_t)n_seq * seq_len * ((n_heads + PREP_HEADS - 1) / PREP_HEADS + (n_kv + PREP_HEADS - 1) / PREP_HEADS) * 16;
    hipLaunchKernelGGL(glue_qk_prep_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, q, ldq, k, ldk, Qr, Kr, n_seq,
                       seq_len, n_heads, n_kv, log2f(rope_theta));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(glue_v_transpose_kernel, dim3((unsigned)((t_pad + 255) / 256), (unsigned)(n_kv * (HEAD_DIM / 8)), (unsigned)n_seq),
                       dim3(256), 0, st, v, ldv, Vt, n_seq, seq_len, t_pad, n_kv);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    static bool attr_set = false;
    if (!attr_set) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(glue_attention_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, ATT_SMEM);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(glue_attention_kernel, dim3((unsigned)((seq_len + ATT_WG_Q - 1) / ATT_WG_Q), (unsigned)n_heads, (unsigned)n_seq), dim3(256), ATT_SMEM, st,
                       Qr, Kr, Vt, out, ldo, seq_len, t_pad, n_heads, n_kv);
    return hipGetLastError();
}

hipError_t launch_glue_rmsnorm(const bf16_t* x, int64_t ldx, bf16_t* y, int64_t ldy, const float* gain, int64_t n, int64_t d,
                               float eps, hipStream_t st) {
    if (n == 0 || d == 0) return hipSuccess;
    hipLaunchKernelGGL(glue_rmsnorm_kernel, dim3((unsigned)n), dim3(256), 0, st, x, ldx, y, ldy, gain, d, eps);
    return hipGetLastError();
}

hipError_t launch_glue_swiglu(const bf16_t* a, int64_t lda, const bf16_t* u, int64_t ldu, bf16_t* m, int64_t ldm, int64_t n,
                              int64_t d, hipStream_t st) {
    if (n == 0 || d == 0) return hipSuccess;
    const int64_t items = n * (d / 8);
    hipLaunchKernelGGL(glue_swiglu_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, a, lda, u, ldu, m, ldm, n, d);
    return hipGetLastError();
}

hipError_t launch_glue_add(bf16_t* h, int64_t ldh, const bf16_t* dl, int64_t ldd, int64_t n, int64_t d, hipStream_t st) {
    if (n == 0 || d == 0) return hipSuccess;
    const int64_t items = n * (d / 8);
    hipLaunchKernelGGL(glue_add_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, h, ldh, dl, ldd, n, d);
    return hipGetLastError();
}

}  // namespace agzo
