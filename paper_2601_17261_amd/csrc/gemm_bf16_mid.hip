// Forward GEMM of the bf16 path in 128 x 128 tiles, for layers that give too few 256 x 256 tiles to fill the chip:
//     OUT = 0:  f = sum over the tile of (X W^T (+ eps (X B) G^T) - Y*)^2     (f0, f+, f- of Sec. 4.1; Eq. 7 factored)
//     OUT = 1:  Y = X W^T (+ eps (X B) G^T) stored as bf16
//     OUT = 2:  the same sums over a share of the slices, stored as they are held; gemm_bf16_mid_finish_kernel adds the shares
//               in order and stores Y
// for d_in, tokens and outputs of at least 128, the rank-r extension as prepared operands.  Other shapes keep
// gemm_bf16_small.hip.
//
// One launch takes up to kBatchMax problems (the layers of a set, both signs of a perturbed evaluation): a 2048-token layer of
// 1024 outputs is 128 tiles, half a chip, and a launch of its own costs 5.6 us before its first and after its last slice.  The
// 21 forwards of a step over the seven 0.6B-sized layers at 2048 tokens: 540 us in 21 launches of gemm_bf16_small.hip, 340 in
// 21 of this kernel, 194 (1015 TFLOP/s) in two; over the 4B-sized layers at 512 tokens: 1130, 775 and 335 us.
//
// Four waves of 64 x 64 (4 x 4 blocks of v_mfma_f32_16x16x32_bf16), two workgroups per compute unit: while one starts or ends a
// tile or waits at its slice barrier the other multiplies.  80 KiB of LDS: three stages of W and two of X, 64-wide slices,
// filled by direct global -> LDS loads in the swizzled layout and with the row permutation of gemm_bf16_aligned.hip.  A slice is
// two blocks of 16 instructions: in the first the wave reads the fragments of the second half and requests the W of the slice
// after next, into the stage the previous slice left; then everything but those four loads has landed and the waves meet; in
// the second it reads the next slice's first fragments and requests the X of the slice after next.
//
// Rows and columns that do not fill a tile: the last tile of a direction starts at the last 128 rows instead of hanging over the
// edge, so that no load needs a bound; the squared error leaves out what the tile before it has counted, a stored output is
// stored twice with the same bits.  A last slice that d_in does not fill: its direct loads get a descriptor with a range and the
// lanes past d_in an offset beyond it, which loads zeros.  Rows of target or output need no alignment.
#include <algorithm>

#include "gemm_bf16_common.h"

namespace agzo {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int MT = BT_SMALL;                    // tile edge
constexpr int MTILE_BYTES = MT * BK * 2;        // one operand slice: 16 KiB
constexpr int MSK_RP = 16;                      // sketch columns (r <= 16)
constexpr int MSK_ROW = MT * 2 + 16;            // bytes per row of the Omega^T planes in LDS (padded against bank conflicts)
constexpr int MSK_SMEM = 3 * MSK_RP * MSK_ROW;

// LDS row m' of a 64-row group of the W tile holds W row mid_perm(m'): a lane's 4 x 4 values over four blocks of 16 outputs
// are then 16 consecutive outputs (as in gemm_bf16_aligned.hip)
__device__ __forceinline__ int mid_perm(int m) { return ((m >> 2) & 3) * 16 + (m >> 4) * 4 + (m & 3); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t mid_rsrc(const bf16_t* base, uint32_t bytes = 0xFFFFFFFFu) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, (int)bytes, 0x00020000);
}

// SK: also emits the range sketch of Alg. 1 from the X slices in LDS, as gemm_bf16_small.hip describes; the planes of Omega^T
// take another 12.75 KiB of LDS, so that the rings are shorter: two stages of both operands where two workgroups share a compute
// unit (the W of a slice is then requested with its X), four with DEEP.  A stored output in shares: each sketches its own slices.
// 3001 x 2048 -> 2048 stored and sketched 52 us in gemm_bf16_small.hip, 72 with the longer ring, one workgroup per compute unit and
// a full wait at every slice, 40 so; 130 x 9728 -> 2560 104, 122 and 29
// DEEP: five stages of both operands and one workgroup per compute unit, for launches that give a compute unit no second
// workgroup anyway: 16 us a launch against 17.1 on the 0.6B-sized layers, 35.8 against 39.3 at 512 tokens on the 4B-sized ones
// (with two workgroups for every compute unit it is the slower one, 42.6 against 34.7 us at 8192 x 2048 -> 1024).  Same bits
constexpr int mid_w_stages(bool sk, bool deep) { return deep ? (sk ? 4 : 5) : (sk ? 2 : 3); }
constexpr int mid_x_stages(bool sk, bool deep) { return deep ? (sk ? 4 : 5) : 2; }
template <int OUT, bool T_F32, bool SK, bool DEEP, int CAP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_bf16_mid_kernel(const KBatch<GemmItem, CAP> tb) {
    constexpr int WS = mid_w_stages(SK, DEEP), XS = mid_x_stages(SK, DEEP);
    constexpr int AHEAD = DEEP ? XS - 1 : 2;                  // slices between a request and its use
    constexpr bool LATE_W = WS == AHEAD;                      // no stage is free for the W of a slice before the barrier
    constexpr int X_BASE = WS * MTILE_BYTES;
    extern __shared__ __align__(16) char smem[];
    uint32_t bx_, by_;
    const GemmItem& p = tb.a[kbatch_find(tb, bx_, by_)];
    const int tid = threadIdx.x, lane = tid & 63;
    if (p.clk && bx_ == 0 && tid == 0) { p.clk[0] = __builtin_readcyclecounter(); p.clk[1] = wall_clock64(); }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wa = wave >> 1, wb = wave & 1;       // wa splits the outputs, wb the tokens
    const int lc = lane & 15, lg = lane >> 4;

    // workgroup -> tile: ids are dealt round-robin over the 8 XCDs; each XCD takes a contiguous run of the problem's tiles, in
    // bands of eight token tiles per output tile
    // (OUT = 2: the tiles once per share of the slices, share by share)
    const int tiles = p.tiles_m * p.tiles_n, count = OUT == 2 ? tiles * p.splits : tiles, per = count / 8;
    int lin = (int)bx_;
    if (lin < per * 8) lin = (lin % 8) * per + lin / 8;
    const int share = OUT == 2 ? __builtin_amdgcn_readfirstlane(lin / tiles) : 0;
    if (OUT == 2) lin -= share * tiles;
    constexpr int BAND = 8;
    const int band = lin / (BAND * p.tiles_n), first = band * BAND;
    const int rows = min(BAND, p.tiles_m - first), in_band = lin - band * BAND * p.tiles_n;
    const int tm = __builtin_amdgcn_readfirstlane(first + in_band % rows), tn = __builtin_amdgcn_readfirstlane(in_band / rows);
    const int64_t m0 = min((int64_t)tm * MT, p.M - MT), n0 = min((int64_t)tn * MT, p.N - MT);

    // this workgroup's slices: all, or a share of the d_in slices (the last share: with the extension behind them)
    const int nd_all = (int)((p.K + BK - 1) / BK);
    const int kbeg = OUT == 2 ? nd_all * share / p.splits : 0, kend = OUT == 2 ? nd_all * (share + 1) / p.splits : nd_all;
    const bool has_ext = p.Xext != nullptr && kend == nd_all;
    const bf16_t *xb = p.X + m0 * p.ldx + (int64_t)kbeg * BK, *wb_ = p.W + n0 * p.ldw + (int64_t)kbeg * BK;
    const bf16_t *xb2 = has_ext ? p.Xext + m0 * p.ext_ld : xb, *wb2 = has_ext ? p.Wext + n0 * p.ext_ld : wb_;
    const int row0 = 8 * wave + (lane >> 3);
    const int chunk0 = (lane & 7) ^ ((row0 >> 1) & 7);
    const int vx = (int)(((int64_t)row0 * p.ldx + chunk0 * 8) * 2), vw = (int)(((int64_t)mid_perm(row0) * p.ldw + chunk0 * 8) * 2);
    const int vx2 = (row0 * p.ext_ld + chunk0 * 8) * 2, vw2 = (mid_perm(row0) * p.ext_ld + chunk0 * 8) * 2;
    const int gsx = (int)(64 * p.ldx), gsw = (int)(64 * p.ldw), gs2 = 64 * p.ext_ld;   // bytes between row groups
    const int nfull = min((int)(p.K / BK), kend) - kbeg, nd = kend - kbeg;          // d_in slices: whole ones, all
    const int npipe = nd + (has_ext ? p.ext_ld / BK : 0);
    const int tail_off = (chunk0 * 8 >= (int)(p.K % BK)) ? kPastEnd : 0;             // (of the slice that is not whole)
    typedef __attribute__((address_space(3))) void* lptr_t;

    // ---- accumulators, and the target tile, which waits in registers for the last slice ----
    // (Accumulators that start at minus the target leave the loss 10 times further from its value in 64 bits, 5e-9 of it
    // against 4e-10: the rounding of the sums then follows the residual's sign.)
    floatx4 acc[4][4];
    uint4 traw[T_F32 ? 16 : 8];
    if constexpr (OUT == 0) {
#pragma unroll
        for (int J = 0; J < 4; ++J) {
            const int64_t row = m0 + wb * 64 + J * 16 + lc, col = n0 + wa * 64 + lg * 16;
            const uint4* src = T_F32 ? reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(p.target) + row * p.ldt + col)
                                     : reinterpret_cast<const uint4*>(reinterpret_cast<const bf16_t*>(p.target) + row * p.ldt + col);
#pragma unroll
            for (int q = 0; q < (T_F32 ? 4 : 2); ++q) traw[J * (T_F32 ? 4 : 2) + q] = load16_any(src + q);
        }
    }

    // ---- fused range sketch: this tile contracts its tokens for the d_in slices tn, tn + tiles_n, ... ----
    char* const Ts = smem + (WS + XS) * MTILE_BYTES;              // Omega^T planes [3][16][128 tokens]
    int sk_next = tn + max(0, kbeg - tn + p.tiles_n - 1) / p.tiles_n * p.tiles_n;      // (of this workgroup's slices)
    if constexpr (SK) {
        const int skip = (int)((int64_t)tm * MT - m0);            // tokens that the tile before this one has covered add nothing
#pragma unroll
        for (int i = 0; i < 3 * MSK_RP * (MT / 8) / 256; ++i) {
            const int v = tid + 256 * i, row = v / (MT / 8), t = v % (MT / 8) * 8;
            const uint4 raw = load16_any(p.sk_T + (int64_t)row * p.sk_mpad + m0 + t);
            uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] &= (t + 2 * u >= skip ? 0xFFFFu : 0u) | (t + 2 * u + 1 >= skip ? 0xFFFF0000u : 0u);
            *reinterpret_cast<uint4*>(Ts + row * MSK_ROW + 2 * t) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    auto sketch = [&](int buf, int it) __attribute__((always_inline)) {
        const int n = lane & 15, g = lane >> 4, c = n & 7;
        const uint32_t sel = (n >> 3) ? 0x07060302u : 0x05040100u;
        floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int tc = 0; tc < 4; ++tc) {
            uint32_t wv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                wv[i] = *reinterpret_cast<const uint32_t*>(smem + X_BASE + buf * MTILE_BYTES + lds_off(32 * tc + 8 * g + i, c) + 4 * wave);
            union { uint4 u; bf16x8 v; } b, a;
            b.u = make_uint4(__builtin_amdgcn_perm(wv[1], wv[0], sel), __builtin_amdgcn_perm(wv[3], wv[2], sel),
                             __builtin_amdgcn_perm(wv[5], wv[4], sel), __builtin_amdgcn_perm(wv[7], wv[6], sel));
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) {
                a.u = *reinterpret_cast<const uint4*>(Ts + (pl * MSK_RP + n) * MSK_ROW + (32 * tc + 8 * g) * 2);
                s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, s, 0, 0, 0);
            }
        }
        const int64_t f = (int64_t)it * BK + 8 * c + 2 * wave + (n >> 3);
        if (f < p.K) *reinterpret_cast<float4*>(p.sk_partial + ((int64_t)tm * p.K + f) * MSK_RP + 4 * g) = make_float4(s[0], s[1], s[2], s[3]);
    };

    // The matrix instructions below are written out and the compiler keeps no distance between them and what reads or writes
    // their accumulators: 24 wait states, which name the accumulators so that nothing that touches one comes on the wrong side
    auto settle = [&]() __attribute__((always_inline)) {
        asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7"
                     : "+v"(acc[0][0]), "+v"(acc[0][1]), "+v"(acc[0][2]), "+v"(acc[0][3]), "+v"(acc[1][0]), "+v"(acc[1][1]), "+v"(acc[1][2]), "+v"(acc[1][3]),
                       "+v"(acc[2][0]), "+v"(acc[2][1]), "+v"(acc[2][2]), "+v"(acc[2][3]), "+v"(acc[3][0]), "+v"(acc[3][1]), "+v"(acc[3][2]), "+v"(acc[3][3]));
    };
    // ---- source of a slice: d_in slices, then the extension operands ----
    __amdgpu_buffer_rsrc_t src_rsx = mid_rsrc(xb), src_rsw = mid_rsrc(wb_);
    int src_so = 0, src_vxt[4], src_vwt[4];
    auto set_offsets = [&](int v0x, int gx, int v0w, int gw) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t) { src_vxt[t] = v0x + t * gx; src_vwt[t] = v0w + (t >> 1) * (2 * gw) + (t & 1) * (gw >> 2); }
    };
    set_offsets(vx, gsx, vw, gsw);
    // past the last slice: that slice once more, into a stage nobody reads
    auto select_slice = [&](int kt) __attribute__((always_inline)) {
        const bf16_t *cxb = xb, *cwb = wb_, *cxb2 = xb2, *cwb2 = wb2;
        const int cvx = vx, cvw = vw, cvx2 = vx2, cvw2 = vw2, cgsx = gsx, cgsw = gsw, cgs2 = gs2;
        kt = min(kt, npipe - 1);
        const bool e = kt >= nd, last = kt == nfull && !e;          // last: the slice that d_in does not fill
        const bf16_t* xs = e ? cxb2 : cxb;
        const bf16_t* ws = e ? cwb2 : cwb;
        const int past = last ? tail_off : 0, svx = (e ? cvx2 : cvx) + past, svw = (e ? cvw2 : cvw) + past;
        const int sgx = e ? cgs2 : cgsx, sgw = e ? cgs2 : cgsw;
        const uint32_t bytes = last ? (uint32_t)kPastEnd : 0xFFFFFFFFu;
        src_rsx = mid_rsrc(xs, bytes);   src_rsw = mid_rsrc(ws, bytes);
        set_offsets(svx, sgx, svw, sgw);
        src_so = (e ? kt - nd : kt) * (BK * 2);
    };
    auto dma_x = [&](int buf, int t) __attribute__((always_inline)) {
        char* dst = smem + X_BASE + buf * MTILE_BYTES + wave * 1024 + t * 4096;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(src_rsx, (lptr_t)dst, 16, src_vxt[t], src_so, 0, 0);
    };
    auto dma_w = [&](int buf, int t) __attribute__((always_inline)) {
        char* dst = smem + buf * MTILE_BYTES + wave * 1024 + t * 4096;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(src_rsw, (lptr_t)dst, 16, src_vwt[t], src_so, 0, 0);
    };
#pragma unroll
    for (int sl = 0; sl < AHEAD; ++sl) {
        select_slice(sl);
#pragma unroll
        for (int t = 0; t < 4; ++t) dma_w(sl, t);
#pragma unroll
        for (int t = 0; t < 4; ++t) dma_x(sl, t);
    }

#pragma unroll
    for (int J = 0; J < 4; ++J) {
#pragma unroll
        for (int I = 0; I < 4; ++I) acc[I][J] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    // ---- multiply: fragment of block row I (W) or token block J (X), k step ks: lane (lc, lg) reads chunk 4 ks + lg of row 16 I + lc
    int aoff[2], boff[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        aoff[ks] = lds_off(wa * 64 + lc, ks * 4 + lg);
        boff[ks] = X_BASE + lds_off(wb * 64 + lc, ks * 4 + lg);
    }
    bf16x8 aw[2][4], bx[2][4];
    auto read_w = [&](int wbuf, int ks, int I) __attribute__((always_inline)) {
        aw[ks][I] = *reinterpret_cast<const bf16x8*>(smem + wbuf * MTILE_BYTES + aoff[ks] + I * 2048);
    };
    auto read_x = [&](int xbuf, int ks, int J) __attribute__((always_inline)) {
        bx[ks][J] = *reinterpret_cast<const bf16x8*>(smem + xbuf * MTILE_BYTES + boff[ks] + J * 2048);
    };
    // (written out with the accumulator tied to its registers, as in gemm_bf16_aligned.hip)
    auto mfma1 = [&](int ks, int I, int J) __attribute__((always_inline)) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[I][J]) : "v"(aw[ks][I]), "v"(bx[ks][J]));
    };
    // 16 instructions of k step KS; rides along: the eight fragments of k step 1 - KS (of W stage rw, X stage rx), one per other
    // instruction, and four direct loads (LOADS 1: W, 2: X) or eight (3: both)
    auto block = [&](auto KS, int rw, int rx, auto LOADS, int lbuf) __attribute__((always_inline)) {
        constexpr int ks = decltype(KS)::value, loads = decltype(LOADS)::value;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            mfma1(ks, q & 3, q >> 2);
            // the first token block and all block rows come first: the next block starts with them
            if (!(q & 1)) {
                const int f = q >> 1;
                if (f == 0) read_x(rx, ks ^ 1, 0);
                else if (f < 5) read_w(rw, ks ^ 1, f - 1);
                else read_x(rx, ks ^ 1, f - 4);
            }
            if ((q & 3) == 1) {
                if (loads == 1 || loads == 3) dma_w(lbuf, q >> 2);
                if (loads == 2) dma_x(lbuf, q >> 2);
            }
            if ((q & 3) == 3 && loads == 3) dma_x(lbuf, q >> 2);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    settle();
    // slice 0 has landed (SK: and this wave's part of the Omega^T planes is written, which a bare barrier does not wait for)
    constexpr int W0 = 8 * (AHEAD - 1), W1 = 8 * (AHEAD - 2) + (LATE_W ? 0 : 4);
    __builtin_amdgcn_s_waitcnt((SK ? 0x0070 : 0x0F70) | (W0 & 15) | ((W0 >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int I = 0; I < 4; ++I) { read_w(0, 0, I); read_x(0, 0, I); }
    int wcur = 0, xcur = 0, wput = (WS == AHEAD) ? 0 : AHEAD, xput = (XS == AHEAD) ? 0 : AHEAD;    // stages of this slice and of slice kt + AHEAD
    for (int kt = 0; kt < npipe; ++kt) {
        if (__builtin_expect(kt + AHEAD >= nfull, 0)) select_slice(kt + AHEAD);
        else src_so = (kt + AHEAD) * (BK * 2);
        block(IC<0>{}, wcur, xcur, IC<LATE_W ? 0 : 1>{}, wput);
        if constexpr (SK)
            if (kbeg + kt == sk_next && kt < nd) { sketch(xcur, kbeg + kt); sk_next += p.tiles_n; }
        // lgkmcnt(0) and all but the youngest loads: the whole next slice has landed (loads return in the order issued; a sketch's
        // stores, which count too, can only make this wait longer), this wave's reads of the current one are done
        __builtin_amdgcn_s_waitcnt(0x0070 | (W1 & 15) | ((W1 >> 4) << 14));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        wcur = (wcur == WS - 1) ? 0 : wcur + 1;
        xcur = (xcur == XS - 1) ? 0 : xcur + 1;
        block(IC<1>{}, wcur, xcur, IC<LATE_W ? 3 : 2>{}, xput);      // (LATE_W: wput = xput)
        wput = (wput == WS - 1) ? 0 : wput + 1;
        xput = (xput == XS - 1) ? 0 : xput + 1;
    }
    settle();
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // the slices fetched past the end
    const int64_t row_new = (int64_t)tm * MT, col_new = (int64_t)tn * MT;
    if constexpr (OUT == 2) {
        floatx4* dst = reinterpret_cast<floatx4*>(p.part) + ((int64_t)(share * tiles + tm * p.tiles_n + tn) * 4 + wave) * 16 * 64 + lane;
#pragma unroll
        for (int J = 0; J < 4; ++J)
#pragma unroll
            for (int I = 0; I < 4; ++I) dst[(J * 4 + I) * 64] = acc[I][J];
    } else if constexpr (OUT == 1) {
#pragma unroll
        for (int J = 0; J < 4; ++J) {
            const int64_t row = m0 + wb * 64 + J * 16 + lc, col = n0 + wa * 64 + lg * 16;
            uint32_t w[8];
#pragma unroll
            for (int I = 0; I < 4; ++I) {
                w[2 * I] = pack_bf16x2(acc[I][J][0], acc[I][J][1]);
                w[2 * I + 1] = pack_bf16x2(acc[I][J][2], acc[I][J][3]);
            }
            bf16_t* dst = reinterpret_cast<bf16_t*>(p.Y) + row * p.ldy + col;
            store16_any(dst, make_uint4(w[0], w[1], w[2], w[3]));
            store16_any(dst + 8, make_uint4(w[4], w[5], w[6], w[7]));
        }
    } else {
        // squares in fp32 four at a time, summed in fp64; lanes, then waves, in a fixed order.  A column tile that overlaps the one
        // before it by no multiple of 16, and all tiles of a layer whose target rows do not start on 16 bytes, are squared in fp64 as
        // well: what gemm_bf16_small.hip squares so keeps its precision here.  (Otherwise a lane's 16 columns count or do not count
        // together)
        double part = 0.0;
        // value of element e of block (I, J) among the raw vectors
        auto target_value = [&](int J, int I, int e) __attribute__((always_inline)) {
            if (T_F32) {
                const uint4 t = traw[J * 4 + I];
                return __uint_as_float(e == 0 ? t.x : e == 1 ? t.y : e == 2 ? t.z : t.w);
            }
            const uint4 t = traw[J * 2 + (I >> 1)];
            const int k = (I & 1) * 2 + (e >> 1);
            const uint32_t w = k == 0 ? t.x : k == 1 ? t.y : k == 2 ? t.z : t.w;
            return __uint_as_float((e & 1) ? w & 0xFFFF0000u : w << 16);
        };
        const int skip = (int)(col_new - (n0 + wa * 64 + lg * 16));      // so many of the lane's 16 columns are counted already
        auto sum = [&](auto WIDE) __attribute__((always_inline)) {
            constexpr bool wide = decltype(WIDE)::value != 0;
#pragma unroll
            for (int J = 0; J < 4; ++J) {
                const int from = m0 + wb * 64 + J * 16 + lc >= row_new ? skip : 16;
#pragma unroll
                for (int I = 0; I < 4; ++I) {
                    float s4 = 0.f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float x = acc[I][J][e] - target_value(J, I, e);
                        if (wide) {
                            const double xd = 4 * I + e >= from ? (double)x : 0.0;
                            part = fma(xd, xd, part);
                        } else {
                            s4 = fmaf(x, x, s4);
                        }
                    }
                    if (!wide) part += (double)(from <= 0 ? s4 : 0.f);
                }
            }
        };
        if (p.wide || ((int)(col_new - n0) & 15) != 0) sum(IC<1>{});
        else sum(IC<0>{});
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
        double* red = reinterpret_cast<double*>(smem);
        __syncthreads();                                     // every wave's fetches past the end have landed
        if (lane == 0) red[wave] = part;
        __syncthreads();
        if (tid == 0) p.partials[(int64_t)tm * p.tiles_n + tn] = (red[0] + red[1]) + (red[2] + red[3]);
    }
    if (p.clk && bx_ == 0 && tid == 0) { p.clk[2] = __builtin_readcyclecounter(); p.clk[3] = wall_clock64(); }
}

// Y from the shares' sums: one workgroup per tile and token block of every wave, four shares' loads of a thread in flight (a
// workgroup per tile took 7 us for 64 tiles of four shares: latency).  PAIRS: four shares, added as gemm_bf16_few.hip does (a launch that asks which
// of the two takes up to 1 us longer: 1009 tokens of 7568 -> 377 5.3 and 6.3 us)
template <bool PAIRS>
__global__ __launch_bounds__(256) void gemm_bf16_mid_finish_kernel(const GemmItem p) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wa = wave >> 1, wb = wave & 1, lc = lane & 15, lg = lane >> 4;
    const int tiles = p.tiles_m * p.tiles_n, tm = blockIdx.x / p.tiles_n, tn = blockIdx.x % p.tiles_n, J = blockIdx.y;
    const int64_t m0 = min((int64_t)tm * MT, p.M - MT), n0 = min((int64_t)tn * MT, p.N - MT);
    const floatx4* src = reinterpret_cast<const floatx4*>(p.part) + (((int64_t)blockIdx.x * 4 + wave) * 16 + J * 4) * 64 + lane;
    floatx4 sum[4] = {};
    if constexpr (PAIRS) {
        static_assert(kFewShares == 4, "two pairs");
        floatx4 v[4][4];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int I = 0; I < 4; ++I) v[s][I] = src[(int64_t)s * tiles * 4096 + I * 64];
#pragma unroll
        for (int I = 0; I < 4; ++I) sum[I] = (v[0][I] + v[1][I]) + (v[2][I] + v[3][I]);
    } else {
        for (int s0 = 0; s0 < p.splits; s0 += 4) {
            floatx4 v[4][4];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int I = 0; I < 4; ++I) v[s][I] = s0 + s < p.splits ? src[(int64_t)(s0 + s) * tiles * 4096 + I * 64] : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int I = 0; I < 4; ++I) sum[I] += v[s][I];
        }
    }
    uint32_t w[8];
#pragma unroll
    for (int I = 0; I < 4; ++I) {
        w[2 * I] = pack_bf16x2(sum[I][0], sum[I][1]);
        w[2 * I + 1] = pack_bf16x2(sum[I][2], sum[I][3]);
    }
    bf16_t* dst = reinterpret_cast<bf16_t*>(p.Y) + (m0 + wb * 64 + J * 16 + lc) * p.ldy + n0 + wa * 64 + lg * 16;
    store16_any(dst, make_uint4(w[0], w[1], w[2], w[3]));
    store16_any(dst + 8, make_uint4(w[4], w[5], w[6], w[7]));
}

// Shares of the d_in slices for a stored output.  A lone launch of few tiles leaves compute units idle while each tile walks all
// of d_in at 0.5 us a slice (one workgroup per compute unit: bound by LDS reads): as many shares as fill the chip, of eight
// slices at least, for the adding costs a launch of some 4 us.  The seven projections of a decoder layer on 385 tokens (32, 64 and 192
// tiles; d_in 2048 and 6144): 191 us in one share each, 139 so.  Not for losses, whose tiles several layers usually share a
// launch with
int gemm_bf16_mid_splits(int64_t M, int64_t N, int64_t K) {
    const int64_t tiles = ((M + MT - 1) / MT) * ((N + MT - 1) / MT), slices = K / BK;
    if (gemm_bf16_few_shape(M, N, K)) return kFewShares;      // (an output over an operand: the bits of gemm_bf16_few.hip)
    if (M < MT || N < MT || tiles > 128) return 1;
    return (int)std::max<int64_t>(1, std::min<int64_t>(256 / tiles, slices / 8));
}
size_t gemm_bf16_split_bytes(int64_t M, int64_t N, int64_t K, bool over) {
    if (!over && gemm_bf16_few_shape(M, N, K)) return 0;
    const int s = gemm_bf16_mid_splits(M, N, K);
    return s > 1 ? (size_t)s * ((M + MT - 1) / MT) * ((N + MT - 1) / MT) * MT * MT * sizeof(float) : 0;
}

// pad: LDS asked for beyond what the kernel uses, which keeps a second workgroup off the compute unit
constexpr int MID_HALF_CU = 8 * 1024;
template <int OUT, bool T_F32, bool SK, bool DEEP, int CAP>
static hipError_t launch_mid_ring(const KBatch<GemmItem, CAP>& tb, unsigned blocks, hipStream_t st, int pad = 0) {
    constexpr int smem = (mid_w_stages(SK, DEEP) + mid_x_stages(SK, DEEP)) * MTILE_BYTES + (SK ? MSK_SMEM : 0);
    static_assert(smem <= (DEEP ? 160 : 80) * 1024, "workgroups per compute unit");
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_bf16_mid_kernel<OUT, T_F32, SK, DEEP, CAP>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, smem + (DEEP ? 0 : MID_HALF_CU));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((gemm_bf16_mid_kernel<OUT, T_F32, SK, DEEP, CAP>), dim3(blocks), dim3(256), smem + pad, st, tb);
    return hipGetLastError();
}
template <int OUT, bool T_F32>
static hipError_t launch_mid_variant(const KBatch<GemmItem>& tb, unsigned blocks, bool sk, bool half_cu, hipStream_t st) {
    // (256: a workgroup per compute unit)
    if (sk) return blocks <= 256 ? launch_mid_ring<OUT, T_F32, true, true>(kbatch_one(tb), blocks, st) : launch_mid_ring<OUT, T_F32, true, false>(kbatch_one(tb), blocks, st);
    if constexpr (OUT == 0) {
        if (half_cu) return launch_mid_ring<OUT, T_F32, false, false>(tb, blocks, st, MID_HALF_CU);
        if (tb.n > 1) return blocks <= 256 ? launch_mid_ring<OUT, T_F32, false, true>(tb, blocks, st) : launch_mid_ring<OUT, T_F32, false, false>(tb, blocks, st);
    }
    return blocks <= 256 ? launch_mid_ring<OUT, T_F32, false, true>(kbatch_one(tb), blocks, st) : launch_mid_ring<OUT, T_F32, false, false>(kbatch_one(tb), blocks, st);
}

bool gemm_bf16_mid_ok(const GemmItem& g, int out) {
    return g.M >= MT && g.N >= MT && g.K >= 2 * BK && (out == 1 ? g.Y != nullptr : g.target != nullptr);
}

hipError_t launch_gemm_bf16_mid(const GemmItem* a, int n, int out, bool target_f32, bool half_cu, hipStream_t st) {
    if ((half_cu && out != 0) || n < 0 || n > (out == 1 ? 1 : kBatchMax)) return hipErrorInvalidValue;
    KBatch<GemmItem> tb;
    tb.n = 0;
    uint64_t blocks = 0;
    int order[kBatchMax];
    for (int i = 0; i < n; ++i) {
        if (!gemm_bf16_mid_ok(a[i], out)) return hipErrorInvalidValue;
        int at = i;             // deepest first, so that the launch does not end on a few long tiles
        for (; at > 0 && a[order[at - 1]].K < a[i].K; --at) order[at] = order[at - 1];
        order[at] = i;
    }
    const bool sk = n > 0 && a[0].sk_T != nullptr;
    if (sk && (n != 1 || !a[0].sk_partial || a[0].sk_tokens != MT || a[0].sk_mpad < (a[0].M + MT - 1) / MT * MT)) return hipErrorInvalidValue;
    if (out == 1 && n == 1 && a[0].part && a[0].splits > 1) {
        KBatch<GemmItem, 1> one{1, {0}, {0}, {a[0]}};
        GemmItem& g = one.a[0];
        g.tiles_m = (int)((g.M + MT - 1) / MT);
        g.tiles_n = (int)((g.N + MT - 1) / MT);
        if (g.splits > g.K / BK) return hipErrorInvalidValue;
        const unsigned tiles = (unsigned)(g.tiles_m * g.tiles_n);
        const bool pairs = gemm_bf16_few_shape(g.M, g.N, g.K);
        if (pairs && g.splits != kFewShares) return hipErrorInvalidValue;
        one.gx[0] = tiles * (unsigned)g.splits;
        hipError_t e = sk ? launch_mid_ring<2, false, true, true>(one, one.gx[0], st) : launch_mid_ring<2, false, false, true>(one, one.gx[0], st);
        if (e != hipSuccess) return e;
        if (pairs) hipLaunchKernelGGL(gemm_bf16_mid_finish_kernel<true>, dim3(tiles, 4), dim3(256), 0, st, g);
        else hipLaunchKernelGGL(gemm_bf16_mid_finish_kernel<false>, dim3(tiles, 4), dim3(256), 0, st, g);
        return hipGetLastError();
    }
    for (int i = 0; i < n; ++i) {
        GemmItem g = a[order[i]];
        g.tiles_m = (int)((g.M + MT - 1) / MT);
        g.tiles_n = (int)((g.N + MT - 1) / MT);
        tb.first[tb.n] = (uint32_t)blocks;
        tb.gx[tb.n] = (uint32_t)((int64_t)g.tiles_m * g.tiles_n);
        blocks += tb.gx[tb.n];
        tb.a[tb.n++] = g;
    }
    if (tb.n == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    if (out == 1) return launch_mid_variant<1, false>(tb, (unsigned)blocks, sk, false, st);
    return target_f32 ? launch_mid_variant<0, true>(tb, (unsigned)blocks, sk, half_cu, st) : launch_mid_variant<0, false>(tb, (unsigned)blocks, sk, half_cu, st);
}

}  // namespace agzo
