// What sits between the linear layers of the gated-MLP stack workload (Alg. 2 over a model): RMS normalisation, the
// SiLU gate and the residual sum.  They are not steps of the method, only the model around it, but a whole-model step
// runs them three times per block, so they are single-pass kernels here: bf16 in and out, fp32 arithmetic, one
// rounding to bf16, 16-byte accesses.  All three are bound by HBM.
#include "agzo_internal.h"
#include "overlap.h"

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
// keys, rotary embedding): the model between the q / k / v projections and the o projection.  Two kernels.
//
// prep: k <- rope(rmsnorm_per_head(.)), head-major [seq][kv head][t][128], and the angles' cosines and sines
// attention: eight waves of 16 queries of one head, which a wave normalises and rotates as it loads them, against tiles of 64 keys that
//       they share in LDS.  Scores are computed transposed, S^T = K Q^T (keys x queries), with
//       v_mfma_f32_16x16x32_bf16: a lane then holds, for ONE query (column lane % 16), the scores of keys 4 g + e of each
//       16-key block (g = lane / 16), so the softmax's running maximum and sum are per-lane scalars up to a reduction
//       over the four g, and the rescaling of the output accumulators (out^T = V^T P^T, same column = query) is a
//       per-lane scalar too.  The eight probabilities a lane holds per 32 keys (two 16-key blocks) go straight into
//       the second product as its operand; V^T in the same order of keys comes from the row-major tile by reads that transpose.
//       Per tile a wave has 512 cycles of matrix work, some 1000 of exponential and other vector work (the
//       mask only on tiles that reach past the wave's queries, the rescaling only where a maximum moved) and 32 KB of LDS reads; four
//       waves to a SIMD overlap them, of which the vector units are busy half of the time.
//       16 x 512 tokens of 16 heads on 8: 84.5 us, with q through memory once more (prepared by a launch ahead) and V transposed
//       by another, and 67.5; 64 x 128 67.7 and 41; 5 x 77 14.5 and 12.3; 4 x 2048 169 and 161
// ---------------------------------------------------------------------------
constexpr int HEAD_DIM = 128;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

// 16 lanes per item: PREP_HEADS heads of k at one token, which share the angles; the rotary pair (i, i + 64) sits 8 lanes apart.  The
// first sequence's items also leave cosine and sine of every position and pair for the queries
constexpr int PREP_HEADS = 4;
__global__ __launch_bounds__(256) void glue_k_prep_kernel(const bf16_t* __restrict__ k, int64_t ldk, bf16_t* __restrict__ Kr, float2* __restrict__ angles,
                                                          int n_seq, int seq_len, int n_kv, float log2_theta) {
    const int64_t item = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4;
    const int j = threadIdx.x & 15;
    const int groups = (n_kv + PREP_HEADS - 1) / PREP_HEADS;
    if (item >= (int64_t)n_seq * seq_len * groups) return;                 // whole 16-lane groups leave together
    const int64_t tok = item / groups;
    const int h0 = (int)(item - tok * groups) * PREP_HEADS;
    const int seq = (int)(tok / seq_len), t = (int)(tok - (int64_t)seq * seq_len);
    const bf16_t* src = k + tok * ldk + h0 * HEAD_DIM + 8 * j;
    uint4 raw[PREP_HEADS];
#pragma unroll
    for (int h = 0; h < PREP_HEADS; ++h) raw[h] = h0 + h < n_kv ? *reinterpret_cast<const uint4*>(src + h * HEAD_DIM) : make_uint4(0, 0, 0, 0);
    // pairs 8 (j mod 8) .. + 8: both of a pair's lanes need them, and each makes four
    float sn[8], cs[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int idx = 8 * (j & 7) + (j >> 3) * 4 + i;                    // pair index 0..63
        const float inv = exp2f(-(float)idx * (2.0f / HEAD_DIM) * log2_theta);
        float sm, cm;
        sincosf((float)t * inv, &sm, &cm);
        const float so = __shfl_xor(sm, 8), co = __shfl_xor(cm, 8);
        sn[i] = j < 8 ? sm : so; cs[i] = j < 8 ? cm : co;
        sn[4 + i] = j < 8 ? so : sm; cs[4 + i] = j < 8 ? co : cm;
    }
    if (seq == 0 && h0 == 0 && j < 8) {
        float4* to = reinterpret_cast<float4*>(angles + (int64_t)t * (HEAD_DIM / 2) + 8 * j);
#pragma unroll
        for (int i = 0; i < 4; ++i) to[i] = make_float4(cs[2 * i], sn[2 * i], cs[2 * i + 1], sn[2 * i + 1]);
    }
    bf16_t* dst = Kr + (((int64_t)seq * n_kv + h0) * seq_len + t) * HEAD_DIM + 8 * j;
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
        if (h0 + h < n_kv) *reinterpret_cast<uint4*>(dst + (int64_t)h * seq_len * HEAD_DIM) = pack8(o);
    }
}

// QG 16-query groups per wave: every K and V^T fragment a wave reads serves QG matrix instructions.  (One group and four waves to a SIMD: with two
// and two, half the reads and as much of the rest, 16 x 512 tokens took 71.0 us, 67.5 so, 4 x 2048 169 and 161)
constexpr int ATT_QG = 1, ATT_WAVES = 8;
constexpr int ATT_WAVE_Q = 16 * ATT_QG;     // queries per wave
constexpr int ATT_WG_Q = ATT_WAVES * ATT_WAVE_Q;    // queries per workgroup
constexpr int ATT_KEYS = 64;                // keys per tile
constexpr int ATT_TILE = ATT_KEYS * HEAD_DIM * 2;        // bytes of a K or V^T tile
constexpr int ATT_SMEM = 4 * ATT_TILE;      // two stages of both

__global__ __launch_bounds__(64 * ATT_WAVES) __attribute__((amdgpu_waves_per_eu(4, 4))) void glue_attention_kernel(
        const bf16_t* __restrict__ q, int64_t ldq, const bf16_t* __restrict__ Kr, const bf16_t* __restrict__ v, int64_t ldv,
        const float2* __restrict__ angles, bf16_t* __restrict__ out, int64_t ldo, int seq_len, int n_heads, int n_kv) {
    extern __shared__ __align__(256) char att_smem[];
    typedef __attribute__((address_space(3))) void* lptr_t;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int head = blockIdx.y, seq = blockIdx.z, kvh = head / (n_heads / n_kv);
    // heavy tiles first: the last queries of a sequence see the most keys
    const int wg_q0 = (int)(gridDim.x - 1 - blockIdx.x) * ATT_WG_Q, q0 = wg_q0 + wave * ATT_WAVE_Q;
    typedef const __attribute__((address_space(1))) void* gptr_t;
    const bf16_t* Kh = Kr + ((int64_t)seq * n_kv + kvh) * seq_len * HEAD_DIM;
    const bf16_t* Vh = v + (int64_t)seq * seq_len * ldv + kvh * HEAD_DIM;
    union Frag { uint4 u; bf16x8_t v; };
    const int tiles = (min(wg_q0 + ATT_WG_Q, seq_len) + ATT_KEYS - 1) / ATT_KEYS;      // that any query of this workgroup may see
    // direct loads of tile j into stage j & 1: rows of 256 bytes of K (16-byte chunk c of row r at c ^ (r mod 16)) and of V (pairs of
    // chunks, pair c of row r at c ^ (r mod 8)), four rows a load.  Keys past the end repeat the last one, masked
    constexpr int LOADS = 16 / ATT_WAVES;
    auto rsrc = [](const bf16_t* base) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, (int)0xFFFFFFFFu, 0x00020000); };
    uint32_t koff[LOADS], voff[LOADS];
#pragma unroll
    for (int t = 0; t < LOADS; ++t) {
        const int row = 4 * (LOADS * wave + t) + (lane >> 4);
        koff[t] = (uint32_t)(row * (HEAD_DIM * 2) + (((lane & 15) ^ (row & 15)) << 4));
        voff[t] = (uint32_t)((lane >> 4) * (2 * ldv) + (((lane & 15) ^ (2 * (row & 7))) << 4));
    }
    const bool near = ldv < (1 << 28);                                     // offsets inside four rows of V have 32 bits
    auto request = [&](int j) __attribute__((always_inline)) {
        char* stage = att_smem + (j & 1) * (2 * ATT_TILE) + wave * (LOADS * 1024);
        if (near && (j + 1) * ATT_KEYS <= seq_len) {
            const __amdgpu_buffer_rsrc_t rk = rsrc(Kh + (int64_t)j * (ATT_KEYS * HEAD_DIM));
#pragma unroll
            for (int t = 0; t < LOADS; ++t) __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lptr_t)(stage + t * 1024), 16, (int)koff[t], 0, 0, 0);
#pragma unroll
            for (int t = 0; t < LOADS; ++t)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc(Vh + (int64_t)(j * ATT_KEYS + 4 * (LOADS * wave + t)) * ldv), (lptr_t)(stage + ATT_TILE + t * 1024), 16, (int)voff[t], 0, 0, 0);
            return;
        }
#pragma unroll
        for (int t = 0; t < LOADS; ++t) {
            const int row = 4 * (LOADS * wave + t) + (lane >> 4);
            const int64_t key = min(j * ATT_KEYS + row, seq_len - 1);
            __builtin_amdgcn_global_load_lds((gptr_t)(Kh + key * HEAD_DIM + (((lane & 15) ^ (row & 15)) << 3)), (lptr_t)(stage + t * 1024), 16, 0, 0);
            __builtin_amdgcn_global_load_lds((gptr_t)(Vh + key * ldv + (((lane & 15) ^ (2 * (row & 7))) << 3)), (lptr_t)(stage + ATT_TILE + t * 1024), 16, 0, 0);
        }
    };
    request(0);
    // queries: normalised and rotated on their way in; lane (n, g) has dims 32 ks + 8 g .. + 8 of query n, both values of its rotary pairs
    int qi[ATT_QG];                                                    // rows past the end repeat the last query, unstored
    Frag qf[ATT_QG][4];
#pragma unroll
    for (int qg = 0; qg < ATT_QG; ++qg) {
        qi[qg] = min(q0 + 16 * qg + n, seq_len - 1);
        const bf16_t* src = q + ((int64_t)seq * seq_len + qi[qg]) * ldq + head * HEAD_DIM + 8 * g;
        const float4* ang = reinterpret_cast<const float4*>(angles + (int64_t)qi[qg] * (HEAD_DIM / 2) + 8 * g);
        float f[4][8], o[4][8];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) unpack8(*reinterpret_cast<const uint4*>(src + 32 * ks), f[ks]);
        float ss = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int i = 0; i < 8; ++i) ss = fmaf(f[ks][i], f[ks][i], ss);
        ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
        const float scale = rsqrtf(ss / (float)HEAD_DIM + 1e-6f);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float4 two = ang[16 * ks + (i >> 1)];
                const float cs = (i & 1) ? two.z : two.x, sn = (i & 1) ? two.w : two.y;
                const float x1 = f[ks][i] * scale, x2 = f[ks + 2][i] * scale;
                o[ks][i] = x1 * cs - x2 * sn;
                o[ks + 2][i] = x2 * cs + x1 * sn;
            }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) qf[qg][ks].u = pack8(o[ks]);
    }
    // V^T fragments of dims 16 db .. + 16, 32 keys: two reads that transpose 4 keys x 16 dims in every 16 lanes, lane n asking for 8 bytes of key
    // 4 g + n / 4 and receiving the four keys' values of dim n.  (Written out with their wait: behind the builtin's the compiler waits for every
    // direct load in flight)
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const int vkey = 4 * g + (n >> 2);
    const uint32_t vat = (uint32_t)(uintptr_t)(lptr_t)att_smem + ATT_TILE + vkey * 256 + (n & 3) * 8 + ((vkey & 7) << 5);      // (dims 0 .. 16; others ^ db << 5)
    auto read_v = [](uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x2 (&lo)[4], u32x2 (&hi)[4]) __attribute__((always_inline)) {
        asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:4096\n\t"
                     "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:4096\n\t"
                     "ds_read_b64_tr_b16 %4, %10\n\tds_read_b64_tr_b16 %5, %10 offset:4096\n\t"
                     "ds_read_b64_tr_b16 %6, %11\n\tds_read_b64_tr_b16 %7, %11 offset:4096\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1]), "=&v"(lo[2]), "=&v"(hi[2]), "=&v"(lo[3]), "=&v"(hi[3])
                     : "v"(a0), "v"(a1), "v"(a2), "v"(a3) : "memory");
    };
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
        floatx4_t s[ATT_QG][4];
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
            Frag kf[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) kf[ks].v = *reinterpret_cast<const bf16x8_t*>(ks_ + 16 * blk * 256 + ((n * 256 + ((g ^ n) << 4)) ^ (ks << 6)));
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
            const uint32_t at = vat + (j & 1) * (2 * ATT_TILE) + h * 8192;
#pragma unroll
            for (int db = 0; db < 8; db += 4) {
                u32x2 lo[4], hi[4];
                read_v(at ^ (db << 5), at ^ ((db + 1) << 5), at ^ ((db + 2) << 5), at ^ ((db + 3) << 5), lo, hi);
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    Frag vf;                                           // the keys in the order the probabilities are held
                    vf.u = make_uint4(lo[d][0], lo[d][1], hi[d][0], hi[d][1]);
#pragma unroll
                    for (int qg = 0; qg < ATT_QG; ++qg) acc[qg][db + d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf.v, pf[qg][h].v, acc[qg][db + d], 0, 0, 0);
                }
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

// rows of d (a multiple of 8) side by side
__global__ __launch_bounds__(256) void glue_copy_rows_kernel(const bf16_t* __restrict__ x, int64_t ldx, bf16_t* __restrict__ y, int64_t n, int64_t d) {
    const int64_t nvec = d / 8, idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n * nvec) return;
    const int64_t row = idx / nvec, v = idx - row * nvec;
    *reinterpret_cast<uint4*>(y + row * d + v * 8) = *reinterpret_cast<const uint4*>(x + row * ldx + v * 8);
}
static hipError_t copy_rows(const bf16_t* x, int64_t ldx, bf16_t* y, int64_t n, int64_t d, hipStream_t st) {
    const int64_t blocks = (n * (d / 8) + 255) / 256;
    if (blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(glue_copy_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, st, x, ldx, y, n, d);
    return hipGetLastError();
}

// The kernel reads queries and values where the caller holds them, while other workgroups store: tensors that `out` lies in are copied ahead of it.
// (Not queries that it replaces row by row: a workgroup stores the rows and the head that it alone reads, behind its reads.  Keys are
// read by the launch ahead)
GlueCopies glue_attention_copies(const bf16_t* q, int64_t ldq, const bf16_t* v, int64_t ldv, const bf16_t* out, int64_t ldo, int n_seq, int seq_len, int n_heads, int n_kv) {
    const int64_t n = (int64_t)n_seq * seq_len, dq = (int64_t)n_heads * HEAD_DIM * 2, dv = (int64_t)n_kv * HEAD_DIM * 2;
    const Rows o{reinterpret_cast<uintptr_t>(out), 2 * ldo, n, dq};
    const bool in_place = q == out && ldq == ldo;
    return GlueCopies{!in_place && rows_overlap(Rows{reinterpret_cast<uintptr_t>(q), 2 * ldq, n, dq}, o), rows_overlap(Rows{reinterpret_cast<uintptr_t>(v), 2 * ldv, n, dv}, o)};
}

// prepared keys, angles, copies
size_t glue_attention_workspace_bytes(int n_seq, int seq_len, int n_heads, int n_kv, GlueCopies copies) {
    const size_t head = (size_t)n_seq * seq_len * HEAD_DIM * sizeof(bf16_t);
    return head * (n_kv + (copies.q ? n_heads : 0) + (copies.v ? n_kv : 0)) + (size_t)seq_len * (HEAD_DIM / 2) * sizeof(float2);
}

hipError_t launch_glue_attention(const bf16_t* q, int64_t ldq, const bf16_t* k, int64_t ldk, const bf16_t* v, int64_t ldv,
                                 bf16_t* out, int64_t ldo, int n_seq, int seq_len, int n_heads, int n_kv, float rope_theta,
                                 void* workspace, hipStream_t st) {
    if (n_seq == 0 || seq_len == 0) return hipSuccess;
    const int64_t n = (int64_t)n_seq * seq_len;
    bf16_t* Kr = static_cast<bf16_t*>(workspace);
    float2* angles = reinterpret_cast<float2*>(Kr + n * n_kv * HEAD_DIM);
    bf16_t* copy = reinterpret_cast<bf16_t*>(angles + (int64_t)seq_len * (HEAD_DIM / 2));
    const GlueCopies copies = glue_attention_copies(q, ldq, v, ldv, out, ldo, n_seq, seq_len, n_heads, n_kv);
    hipError_t e = hipSuccess;
    if (copies.q) {
        e = copy_rows(q, ldq, copy, n, (int64_t)n_heads * HEAD_DIM, st);
        if (e != hipSuccess) return e;
        q = copy;
        ldq = (int64_t)n_heads * HEAD_DIM;
        copy += n * ldq;
    }
    if (copies.v) {
        e = copy_rows(v, ldv, copy, n, (int64_t)n_kv * HEAD_DIM, st);
        if (e != hipSuccess) return e;
        v = copy;
        ldv = (int64_t)n_kv * HEAD_DIM;
    }
    const int64_t items = n * ((n_kv + PREP_HEADS - 1) / PREP_HEADS) * 16;
    hipLaunchKernelGGL(glue_k_prep_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, k, ldk, Kr, angles, n_seq, seq_len, n_kv, log2f(rope_theta));
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    static bool attr_set = false;
    if (!attr_set) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(glue_attention_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, ATT_SMEM);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(glue_attention_kernel, dim3((unsigned)((seq_len + ATT_WG_Q - 1) / ATT_WG_Q), (unsigned)n_heads, (unsigned)n_seq), dim3(64 * ATT_WAVES), ATT_SMEM, st,
                       q, ldq, Kr, v, ldv, angles, out, ldo, seq_len, n_heads, n_kv);
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
