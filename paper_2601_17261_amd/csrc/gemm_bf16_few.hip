// Forward GEMM of the bf16 path in 64 x 64 tiles whose four waves share d_in, for stored outputs of few tiles and no deep d_in:
//     Y = X W^T (+ eps (X B) G^T) as bf16, tokens and outputs of at least 128, the rank-r term as prepared operands
//
// A program calls the layers of a model one by one, and few tokens leave such a launch a few dozen 128 x 128 tiles, whose time is latency:
// a chain of slices with a barrier each, or shares of d_in that meet in memory and a second launch that adds them.  Here a wave has the
// whole tile and a quarter of d_in, in a ring of its own that only it fills and reads: nothing in the loop over slices waits for
// another wave.  A slice's fragments go to registers, then its slot is requested again, then they are multiplied.  The four sums meet
// in LDS at the end.  Bound by what a compute unit takes in, some 85 GB/s of direct loads (16 KiB a slice): eight waves of one slot
// each, loads spread between the matrix instructions and fragments read by hand take the same time.
// us, weights from memory, 128 x 128 tiles (with the launch that adds their shares) and this kernel: 385 tokens of 2048 -> 2048
// 18.2 and 9.2, -> 1024 14.0 and 8.8; 1000 of 2048 -> 1024 17.3 and 9.2, -> 2048 (two workgroups to a compute unit) 18.4 and 14.9; 432 of
// 1024 -> 1024 11.5 and 6.4; 128 of 256 -> 256 5.5 and 4.0.  A decoder's step on 385 tokens: 1606 and 1493
//
// Rows, columns and a last slice that do not fill a tile as in gemm_bf16_mid.hip: the last tile of a direction starts at the last 64
// rows, lanes past d_in load zeros.
#include "gemm_bf16_common.h"

namespace agzo {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int FT = 64;                              // tile edge
constexpr int FSLOT = 2 * FT * BK * 2;              // a slice of both operands: 16 KiB, X rows first
constexpr int WAVES = kFewShares;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t few_rsrc(const bf16_t* base, uint32_t bytes = 0xFFFFFFFFu) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, (int)bytes, 0x00020000);
}

// SK: also emits the range sketch of Alg. 1, S = X^T Omega, from the X slices in LDS: the tiles of a token block take the slices in turn, and a
// wave contracts those of its own that fall to its tile, ahead of the reads of the slice's fragments.  Omega^T of the 64 tokens stays in
// registers.  Y has the bits of the forward without it.  (128 x 128 tiles that add the same quarters, in four shares or in one, take longer.)  The whole
// call (Omega, forward, sum of the token tiles), us, 128 x 128 tiles in one share or as many as fill the chip, whose bits are others, in such
// quarters, and so: 1000 tokens of 256 -> 2048 13.1, 22.8 and 11.6, of 2048 -> 2048 27, 27 and 22.6, 432 of 1024 -> 1024 17.0, 17.8 and 13.2, 8192 of
// 256 -> 256 29, 40 and 19.4; 385 of 320 -> 2048 11.9, 21.3 and 13.0 is the worst against the first
template <int STAGES, bool SK>
__device__ __forceinline__ void few_body(const GemmItem& p) {
    extern __shared__ __align__(16) char smem[];
    typedef __attribute__((address_space(3))) void* lptr_t;
    const int tid = threadIdx.x, lane = tid & 63;
    if (p.clk && blockIdx.x == 0 && tid == 0) { p.clk[0] = __builtin_readcyclecounter(); p.clk[1] = wall_clock64(); }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = lane & 15, lg = lane >> 4;

    // workgroup -> tile, as in gemm_bf16_mid.hip: each XCD takes a contiguous run of tiles, in bands of eight token tiles
    const int tiles = p.tiles_m * p.tiles_n, per = tiles / 8;
    int lin = (int)blockIdx.x;
    if (lin < per * 8) lin = (lin % 8) * per + lin / 8;
    constexpr int BAND = 8;
    const int band = lin / (BAND * p.tiles_n), first = band * BAND;
    const int rows = min(BAND, p.tiles_m - first), in_band = lin - band * BAND * p.tiles_n;
    const int tm = __builtin_amdgcn_readfirstlane(first + in_band % rows), tn = __builtin_amdgcn_readfirstlane(in_band / rows);
    const int64_t m0 = min((int64_t)tm * FT, p.M - FT), n0 = min((int64_t)tn * FT, p.N - FT);

    // this wave's slices: its share of d_in's, the last wave's with the extension behind them
    const int nd_all = (int)((p.K + BK - 1) / BK), nfull = (int)(p.K / BK);
    const int kbeg = nd_all * wave / WAVES, nd = nd_all * (wave + 1) / WAVES - kbeg;
    const int n = nd + (p.Xext != nullptr && wave == WAVES - 1 ? p.ext_ld / BK : 0);
    char* const ring = smem + wave * STAGES * FSLOT;

    // fragment (plane, 32 tokens): row lc, 8 tokens from 8 lg on; tokens that the tile before this one has covered add nothing
    bf16x8 omega[SK ? 3 : 1][2];
    int sk_next = tn + max(0, kbeg - tn + p.tiles_n - 1) / p.tiles_n * p.tiles_n;
    if constexpr (SK) {
        const int skip = (int)((int64_t)tm * FT - m0);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
#pragma unroll
            for (int tc = 0; tc < 2; ++tc) {
                const int t = 32 * tc + 8 * lg;
                const uint4 raw = load16_any(p.sk_T + (int64_t)(pl * 16 + lc) * p.sk_mpad + m0 + t);
                uint32_t v[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] &= (t + 2 * u >= skip ? 0xFFFFu : 0u) | (t + 2 * u + 1 >= skip ? 0xFFFF0000u : 0u);
                omega[pl][tc] = __builtin_bit_cast(bf16x8, make_uint4(v[0], v[1], v[2], v[3]));
            }
    }
    // features 8 c + 2 w + (lc / 8), c = lc mod 8, of the slice at `at`, slice `it` of d_in
    auto sketch = [&](const char* at, int it) __attribute__((always_inline)) {
        int row = 8 * lg;
        asm volatile("" : "+v"(row));               // (addresses made here: kept over the loop they make one slot a wave spill)
        const int c = lc & 7;
        const uint32_t sel = (lc >> 3) ? 0x07060302u : 0x05040100u;
#pragma unroll 1
        for (int w = 0; w < 4; ++w) {
            floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int tc = 0; tc < 2; ++tc) {
                uint32_t v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const uint32_t*>(at + lds_off(32 * tc + row + i, c) + 4 * w);
                const uint4 b = make_uint4(__builtin_amdgcn_perm(v[1], v[0], sel), __builtin_amdgcn_perm(v[3], v[2], sel),
                                           __builtin_amdgcn_perm(v[5], v[4], sel), __builtin_amdgcn_perm(v[7], v[6], sel));
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(omega[pl][tc], __builtin_bit_cast(bf16x8, b), s, 0, 0, 0);
            }
            const int64_t f = (int64_t)it * BK + 8 * c + 2 * w + (lc >> 3);
            if (f < p.K) *reinterpret_cast<float4*>(p.sk_partial + ((int64_t)tm * p.K + f) * 16 + 4 * lg) = make_float4(s[0], s[1], s[2], s[3]);
        }
    };

    // direct load t of an operand: LDS rows 8 t + lane / 8 (of W the permuted ones: a lane then holds 16 consecutive outputs), the
    // chunks in the swizzled order, which turns by four between even and odd t
    const int row0 = lane >> 3, chunk0 = (lane & 7) ^ (row0 >> 1);
    auto w_row = [&](int t) __attribute__((always_inline)) { return (2 * (t & 1) + (row0 >> 2)) * 16 + (t >> 1) * 4 + (row0 & 3); };
    auto chunk = [&](int t) __attribute__((always_inline)) { return chunk0 ^ (4 * (t & 1)); };
    __amdgpu_buffer_rsrc_t rx = few_rsrc(p.X + m0 * p.ldx), rw = few_rsrc(p.W + n0 * p.ldw);
    int vx[8], vw[8], so = 0;
    auto offsets = [&](int64_t ldx, int64_t ldw) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            vx[t] = (int)(((int64_t)(8 * t + row0) * ldx + chunk(t) * 8) * 2);
            vw[t] = (int)(((int64_t)w_row(t) * ldw + chunk(t) * 8) * 2);
        }
    };
    offsets(p.ldx, p.ldw);
    // the source of the wave's slice i
    auto select = [&](int i) __attribute__((always_inline)) {
        if (__builtin_expect(i < nd && kbeg + i < nfull, 1)) { so = (kbeg + i) * (BK * 2); return; }
        if (i < nd) {                               // the slice that d_in does not fill: zeros past it
            rx = few_rsrc(p.X + m0 * p.ldx, (uint32_t)kPastEnd); rw = few_rsrc(p.W + n0 * p.ldw, (uint32_t)kPastEnd);
            so = nfull * (BK * 2);
            const int left = (int)(p.K % BK);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int past = chunk(t) * 8 >= left ? kPastEnd : 0;
                vx[t] += past; vw[t] += past;
            }
        } else {
            rx = few_rsrc(p.Xext + m0 * p.ext_ld); rw = few_rsrc(p.Wext + n0 * p.ext_ld);
            so = (i - nd) * (BK * 2);
            offsets(p.ext_ld, p.ext_ld);
        }
    };
    auto dma = [&](char* dst, int q) __attribute__((always_inline)) {
        if (q < 8) __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lptr_t)(dst + q * 1024), 16, vx[q], so, 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lptr_t)(dst + q * 1024), 16, vw[q - 8], so, 0, 0);
    };
    floatx4 acc[4][4];
    bf16x8 w[2][4], x[2][4];
#pragma unroll
    for (int I = 0; I < 4; ++I)
#pragma unroll
        for (int J = 0; J < 4; ++J) acc[I][J] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
        if (s < n) {
            select(s);
#pragma unroll
            for (int q = 0; q < 16; ++q) dma(ring + s * FSLOT, q);
        }
    const int off[2] = {lds_off(lc, lg), lds_off(lc, 4 + lg)};
    int slot = 0;
    for (int i = 0; i < n; ++i) {
        // the slice has landed; this wave's reads of it are all there before its slot is filled again
        if (STAGES == 2 && i + 1 < n) __builtin_amdgcn_s_waitcnt(0x4F70);      // vmcnt(16)
        else __builtin_amdgcn_s_waitcnt(0x0F70);
        __builtin_amdgcn_sched_barrier(0);
        char* const at = ring + slot * FSLOT;
        if constexpr (SK)
            if (kbeg + i == sk_next && i < nd) { sketch(at, sk_next); sk_next += p.tiles_n; }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int I = 0; I < 4; ++I) w[ks][I] = *reinterpret_cast<const bf16x8*>(at + 8192 + off[ks] + I * 2048);
#pragma unroll
            for (int J = 0; J < 4; ++J) x[ks][J] = *reinterpret_cast<const bf16x8*>(at + off[ks] + J * 2048);
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        if (i + STAGES < n) {
            select(i + STAGES);
#pragma unroll
            for (int q = 0; q < 16; ++q) dma(at, q);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int J = 0; J < 4; ++J)
#pragma unroll
                for (int I = 0; I < 4; ++I) acc[I][J] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][I], x[ks][J], acc[I][J], 0, 0, 0);
        slot = (slot + 1 == STAGES) ? 0 : slot + 1;
    }
    // the shares, added in pairs: wave w takes the tokens of block w
    floatx4* mine = reinterpret_cast<floatx4*>(ring) + lane;
#pragma unroll
    for (int J = 0; J < 4; ++J)
#pragma unroll
        for (int I = 0; I < 4; ++I) mine[(J * 4 + I) * 64] = acc[I][J];
    __syncthreads();
    auto share = [&](int s, int I) __attribute__((always_inline)) { return reinterpret_cast<const floatx4*>(smem + s * STAGES * FSLOT)[(wave * 4 + I) * 64 + lane]; };
    static_assert(WAVES == 4, "two pairs");
    floatx4 sum[4];
#pragma unroll
    for (int I = 0; I < 4; ++I) sum[I] = (share(0, I) + share(1, I)) + (share(2, I) + share(3, I));
    uint32_t o[8];
#pragma unroll
    for (int I = 0; I < 4; ++I) {
        o[2 * I] = pack_bf16x2(sum[I][0], sum[I][1]);
        o[2 * I + 1] = pack_bf16x2(sum[I][2], sum[I][3]);
    }
    bf16_t* dst = reinterpret_cast<bf16_t*>(p.Y) + (m0 + wave * 16 + lc) * p.ldy + n0 + lg * 16;
    store16_any(dst, make_uint4(o[0], o[1], o[2], o[3]));
    store16_any(dst + 8, make_uint4(o[4], o[5], o[6], o[7]));
    if (p.clk && blockIdx.x == 0 && tid == 0) { p.clk[2] = __builtin_readcyclecounter(); p.clk[3] = wall_clock64(); }
}

template <int STAGES, bool SK>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(STAGES == 1 ? 2 : 1))) void gemm_bf16_few_kernel(const GemmItem p) {
    few_body<STAGES, SK>(p);
}

template <int STAGES, bool SK>
static hipError_t launch_few(const GemmItem& g, unsigned tiles, hipStream_t st) {
    constexpr int smem = WAVES * STAGES * FSLOT;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_bf16_few_kernel<STAGES, SK>), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((gemm_bf16_few_kernel<STAGES, SK>), dim3(tiles), dim3(64 * WAVES), smem, st, g);
    return hipGetLastError();
}

// Up to two workgroups a compute unit, and a d_in that 128 x 128 tiles in shares do not walk as fast, for they take in half the bytes an output.  us,
// those and this kernel: 2048 -> 1024 outputs 23.5 and 19.5 at d_in = 2560, 28.6 and 26.2 at 4096, 385 -> 2048 18.7 and 12.5, 19.6 and 17.1, but 128 ->
// 4096 18.8 and 21.1 at 3064, 256 -> 2048 20.0 and 26.8 at 6144; of fewer than 64 tiles, which the shares spread over more compute units, 200 -> 256
// 11.0 and 11.7 at 2560, 9.6 and 6.7 at 1024.  More tiles: 1500 -> 2048, 768 of them, 16.4 and 23.2.
// Rows of X and W that do not start on 128 bytes cost two workgroups of one slot more: there 128 x 128 tiles are left what they walk in one share of 13 to 20
// slices (598 -> 3238, 1272: 12.9 and 15.5; 553 -> 3556, 952: 10.4 and 13.2; but 431 -> 3028, 824 8.9 and 9.3, 146 -> 10013, 1424 17.7 and 16.1) and, in two
// or three, of more than 32 (695 -> 1857, 2520: 22.8 and 27.2; 725 -> 2365, 2104 22.3 and 23.9; but 577 -> 2416, 1976 20.2 and 20.9, 603 -> 3178, 1032 20.5
// and 12.6)
bool gemm_bf16_few_shape(int64_t M, int64_t N, int64_t K) {
    const int64_t tiles = ((M + FT - 1) / FT) * ((N + FT - 1) / FT);
    if (tiles > 256 && K % BK != 0 && K >= 13 * BK) {
        const bool one_share = ((M + BT_SMALL - 1) / BT_SMALL) * ((N + BT_SMALL - 1) / BT_SMALL) > 128 || K < 16 * BK;
        if (one_share ? K < 21 * BK : K > 32 * BK) return false;
    }
    return M >= BT_SMALL && N >= BT_SMALL && tiles <= 512 && K >= WAVES * BK && K <= (tiles >= 64 ? 40 : 32) * BK;
}

hipError_t launch_gemm_bf16_few(const GemmItem& a, hipStream_t st) {
    if (!gemm_bf16_few_shape(a.M, a.N, a.K) || !a.Y) return hipErrorInvalidValue;
    if (a.sk_T && (!a.sk_partial || a.sk_tokens != FT || a.sk_mpad < (a.M + FT - 1) / FT * FT || a.Xext)) return hipErrorInvalidValue;
    GemmItem g = a;
    g.tiles_m = (int)((g.M + FT - 1) / FT);
    g.tiles_n = (int)((g.N + FT - 1) / FT);
    const int64_t tiles = (int64_t)g.tiles_m * g.tiles_n;
    // (two slots a wave and one workgroup to a compute unit, or one slot and two)
    if (g.sk_T) return tiles <= 256 ? launch_few<2, true>(g, (unsigned)tiles, st) : launch_few<1, true>(g, (unsigned)tiles, st);
    return tiles <= 256 ? launch_few<2, false>(g, (unsigned)tiles, st) : launch_few<1, false>(g, (unsigned)tiles, st);
}

}  // namespace agzo
