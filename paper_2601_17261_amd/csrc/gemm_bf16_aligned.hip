// Forward GEMM in 256 x 256 tiles, the kernel of the benchmark configurations:
//     OUT = 0:  f = sum over the tile of (X W^T (+ eps (X B) G^T) - Y*)^2     (f0, f+, f- of Sec. 4.1; Eq. 7 factored)
//     OUT = 1:  Y = X W^T (+ eps (X B) G^T) stored as bf16                     (a layer inside a model, Alg. 2)
//     OUT = 2:  the same logits never stored: per token and 128-column chunk their maximum and the sum of exponentials
//               around it, and the target's logit (token cross-entropy of a model's last layer; loss.hip combines them)
// Same tile, tile layout in LDS and direct global -> LDS operand loads as gemm_bf16.hip (256 x 256 tile, four waves of
// 128 x 128, 64-wide K slices), but a kernel of its own with one straight path and nothing else compiled in: M and N of
// at least 256, d_in of at least 128, the rank-r extension as prepared operands.
//
// RAGGED = false takes tile-aligned layers: M and N multiples of 256, d_in a multiple of 64, 16-byte aligned target / output
// rows.  RAGGED = true takes the others.  The last tile of a direction starts at the last 256 rows (or columns) instead of
// hanging over the edge, so no load needs a bound; softmax statistics leave out what the tile before it has counted, stored
// outputs are stored twice with the same bits.  For the squared error of bf16 targets the two halves of a tile do so each by itself (a tile's second
// 128 rows start at the last 128 of the matrix at the latest), so that a wave's 128 x 128 outputs are those of a tile of
// gemm_bf16_mid.hip, and leave out what the half before them has counted.  A last slice that d_in does not fill gets a descriptor with a
// range, and the lanes past d_in an offset beyond it: they load zeros.  gemm_bf16.hip, which bounded every access and drained
// its loads at every slice, ran 3001 x 2560 -> 9728 (both signs and none, with the smaller projections beside it) at 820
// TFLOP/s and the cross-entropy head 3001 x 2048 -> 32000 at 937; this kernel at 1130 and 1105.
//
// Matrix instruction.
// v_mfma_f32_16x16x32_bf16, 8 x 8 blocks per wave, two k steps of 32 per slice, where gemm_bf16.hip has 4 x 4 blocks of
// v_mfma_f32_32x32x16_bf16 and four k steps.  Both give the published rate at the top clock; under the device's power
// limit, on random operands, a register-only loop of the first holds 2.2 PFLOP/s at 2.1 GHz and one of the second
// 1.9 at 1.8, and this kernel spends 80 - 90 % of its time in these instructions.  A slice is four blocks of 32
// instructions (block rows 0..3 / 4..7 of k step 0, then of k step 1), each walked token block by token block with the
// four W fragments of its block rows and the eight X fragments of the k step in registers; the W fragments of the next
// block are read in the first half of a block, and in the second block of a k step each X fragment is replaced by the
// next k step's as soon as its last instruction has issued.
//
// LDS stages.
// A 64-wide slice is 32 KiB per operand and the compute unit has 160 KiB: three stages for W and two for X.  A stage
// can be filled again once every wave has read its last fragment, which the one barrier of a slice establishes (after
// the third of its four blocks of matrix instructions: fragments are read a block ahead).  With two stages per
// operand everything for the slice after next had to be requested behind that barrier and to land before the next
// one, the later half of it within two blocks: the barrier waited for the slowest line, 250 - 450 cycles per slice on
// the wide layers.  With the third W stage the W half of the slice after next is requested a block before the barrier,
// into the stage the previous slice left, and has six blocks to land; behind the barrier only the X half is
// requested, at once, and has three.  The wait in front of the barrier is for all but the eight youngest loads (loads
// return in the order issued).  Cycles per launch fell by 15 % on the wide layers; the clock, which the power limit
// sets, gave a third of that back.
//
// Squared error (OUT = 0).
// The accumulators do not start at zero but at minus the target tile: the target is requested before the first
// operand slice and converted while that slice is on its way, so after the last slice the registers hold the residual
// Y - Y* and the epilogue is a sum of squares of registers with no memory access.  (Reading the target in the epilogue
// left the matrix cores idle for 15 - 18 % of a tile: every workgroup asks for its 128 KiB at the same moment and
// waits out the latency, and the staging registers spilled.)  All evaluations of a step start from the same -Y*, so
// f+ and f- still share bit-identical accumulators up to the rank-r slices.  With RAGGED the target is subtracted behind the
// last slice instead: these layers' losses were that far from their 64-bit values (4e-10 of them; with the accumulators
// starting at minus the target 5e-9, as the sums' rounding then follows the sign of the residual), and they stay there.
//
// Persistent workgroups.
// One workgroup per compute unit walks through a list of tiles (its LDS and accumulators leave no room for a second one,
// so a workgroup per tile paid the launch of a workgroup, the latency of the first operand slices and of the target, and
// an unpipelined last slice once per tile, with the matrix cores idle; walking tile lists instead measured 1 - 3 % faster).  The slice
// loop runs across tile boundaries: every slice, the last one of a tile included, is a steady iteration whose loads
// fetch the slice after next - at the end of a tile the first two slices of the next tile - so when a tile's last
// matrix instruction has issued, the next tile's first slice is in LDS and its first fragments are in registers.
// Between two tiles only the accumulators change hands: the next target is requested, the finished tile is evaluated
// (or stored) while it travels, and the accumulators restart from minus the new target.  The tile list keeps the
// order that makes an XCD's 32 workgroups share operand slices in its L2: XCD x (workgroup id mod 8) owns a contiguous
// run of tiles, and its workgroups take them 32 at a time.
//
// CAP > 1: the lists go through the tiles of several problems (layers of a set, both signs); see TileLists and
// launch_gemm_bf16_aligned_lists().  The operands of the next tile are another problem's then, so the choice of a slice's source works
// out its offsets from that problem's row lengths.
//
// PHASES = 3 is the shared-forward schedule for a single layer: the d_in slices are multiplied once, f0 is the sum of
// squares of the accumulators as they stand, the extension slices with +eps make them the residual of f+, the same
// slices with -2 eps that of f-.  The extension operands of both passes are requested before the evaluation that
// precedes them, so their latency runs under it.  A workgroup takes one tile, and a launch the tiles of up to kBatchMax
// layers, the deepest first: a launch per layer ends on a round that is partly idle, seven times for a set (4096 tokens
// of the 4B-sized layers, 64 to 608 tiles each, r = 64: 1031 us in seven launches, 775 in one).
#include "gemm_bf16_common.h"
#include "slots.h"

namespace agzo {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// LDS row m' of a 64-row group of the W tile holds W row perm64(m'): block t = m' / 16 of the group, output register e
// of lane group g = (m' / 4) mod 4 of a 16 x 16 block is row 4 g + e of the block, which this makes output column
// 16 g + 4 t + e of the group: a lane's 4 x 4 values over four neighbouring blocks are 16 consecutive outputs.
__device__ __forceinline__ int w_perm64(int m) { return ((m >> 2) & 3) * 16 + (m >> 4) * 4 + (m & 3); }

// buffer descriptor over everything from `base` on (no range check: tiles lie inside their matrices), or over `bytes`
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const bf16_t* base, uint32_t bytes = 0xFFFFFFFFu) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, (int)bytes, 0x00020000);
}

// A value moved into an accumulation register by hand: the 256 start values of the accumulators are produced by
// vector instructions, and left to itself the compiler parks them in ordinary registers (and spills most of them)
// until the first multiply.
__device__ __forceinline__ float to_acc(float x) {
    float r;
    asm volatile("v_accvgpr_write_b32 %0, %1" : "=a"(r) : "v"(x));
    return r;
}

// ... and read back by hand, one value at a time in program order: left to itself the compiler copies all 256
// accumulators into ordinary registers at once before it sums their squares, and whatever else is live at that moment
// (the next tile's target) goes to scratch memory.  The compiler's hazard bookkeeping does not look inside the asm:
// the caller keeps the wait states that a matrix instruction needs before its result may be read (19 for the longest).
__device__ __forceinline__ float from_acc(float x) {
    float r;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r) : "a"(x));
    return r;
}

// what the kernel needs of one problem (GemmParams without the fields of the other kernels: sixteen fit a launch's arguments)
struct AlignedItem {
    const bf16_t *X, *W, *Xext, *Wext, *Wext2;
    int64_t ldx, ldw, M, N, K, ldt, ldy;
    const void* target;
    double* partials;
    void* Y;
    const int32_t* ce_target; float2* ce_ms; float* ce_tl;
    unsigned long long* clk;
    int ext_ld, tiles_m, tiles_n, group_m, vec_ok;
    int sub;                                       // partials are those of gemm_bf16_mid.hip: one per 128 x 128 outputs
};

// Tile lists over the tiles of several problems (one evaluation, squared error).  The tiles of a problem are dealt to the XCDs in runs
// of equal length, the runs that are one longer starting at XCD long_at[q].  An XCD's workgroups (its slots) take full[q] rounds of
// problem q together, problem after problem, and then what is left of the runs, slot s take[q][s] tiles of problem q.  (Operand slices
// are shared through an XCD's L2 by workgroups that walk them in step: lists dealt without the rounds, each problem's tiles to whoever
// is done first, took 2.4 % longer than launches of their own for the 8B-sized layers on 15028 tokens)
constexpr int kListSlots = 32;                    // workgroups per XCD
struct TileLists {
    int n, slots;
    uint8_t long_at[kBatchMax];
    int full[kBatchMax];
    uint32_t take[kBatchMax][kListSlots / 4];      // bytes
    AlignedItem a[kBatchMax];
};
static_assert(sizeof(TileLists) <= 4096, "kernel arguments");

template <int PHASES, int CAP>
using AlignedArgs = typename std::conditional<(PHASES == 1 && CAP > 1), TileLists, KBatch<AlignedItem, CAP>>::type;

template <int CAP>
__device__ __forceinline__ int own_problem(const KBatch<AlignedItem, CAP>& tb, uint32_t& wgid) {
    uint32_t unused;
    return kbatch_find(tb, wgid, unused);
}
__device__ __forceinline__ int own_problem(const TileLists&, uint32_t&) { return 0; }

template <int OUT, bool T_F32, int PHASES, bool RAGGED, int CAP>
__global__ __launch_bounds__(256) void gemm_bf16_aligned_kernel(const AlignedArgs<PHASES, CAP> tb) {
    static_assert(OUT == 0 || (PHASES == 1 && !T_F32), "the kernels without a squared-error target have one evaluation");
    constexpr bool LISTS = PHASES == 1 && CAP > 1;
    constexpr bool LATE_T = RAGGED && OUT == 0;    // the target is subtracted after the last slice
    // ... and the two 128-row halves of a tile end at the last row by themselves, as the tiles of gemm_bf16_mid.hip do.  (Only where lists
    // may join layers of that kernel, that is for one evaluation and bf16 targets: in the shared schedule, whose registers spill anyway,
    // halves took 9 % longer, with fp32 targets 128 registers spilled for 116, 1 % of a forward 8191 x 2048 -> 2048)
    constexpr bool HALVES = LATE_T && PHASES == 1 && !T_F32;
    constexpr int NT = 256, BA = 4, BB = 4;
    constexpr int W_BASE = 0, X_BASE = 3 * TILE_BYTES;       // LDS: three W stages, then two X stages (all 160 KiB)
    extern __shared__ __align__(16) char smem[];
    uint32_t wgid = blockIdx.x;                              // this problem's workgroups count from 0
    // the problems of the current and of the next tile, by their places in the arguments (as pointers the compiler copies all of them
    // to scratch memory; the only problem of a workgroup, whose place it would work out again, by reference)
    int cq = 0, nq = 0;
    const AlignedItem& only = tb.a[own_problem(tb, wgid)];
    auto item = [&](int q) __attribute__((always_inline)) -> const AlignedItem& {
        if constexpr (LISTS) return tb.a[q];
        else return only;
    };
    const int tid = threadIdx.x, lane = tid & 63;
    if (!LISTS && item(cq).clk && wgid == 0 && tid == 0) { item(cq).clk[0] = __builtin_readcyclecounter(); item(cq).clk[1] = wall_clock64(); }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wa = wave >> 1, wb = wave & 1;
    const int lc = lane & 15, lg = lane >> 4;      // matrix instruction 16x16x32: column (token) / row of a fragment, k group

    // ---- this workgroup's tiles ---------------------------------------------------------------------
    // XCD x = id mod 8 (ids are dealt round-robin over the XCDs) owns the run of tiles [x per, (x + 1) per), walked by
    // its S workgroups S at a time; the up to 7 tiles left over go to the last workgroup of the first XCDs.  Inside a
    // run, tiles are ordered in bands of group_m token tiles per output tile, so that the tiles an XCD works on at any
    // moment share a few W tiles and a band of X tiles.
    // LISTS: the same over the runs of several problems; the lists are the launch's, which knows what a tile of each takes.
    int64_t tm = 0, tn = 0;
    auto tile_of = [&](const AlignedItem& a, int lin, int64_t& tm_, int64_t& tn_) __attribute__((always_inline)) {
        const int group = lin / (a.group_m * a.tiles_n);
        const int first_m = group * a.group_m;
        const int gsz = min(a.group_m, a.tiles_m - first_m);
        const int in_group = lin - group * a.group_m * a.tiles_n;
        tm_ = __builtin_amdgcn_readfirstlane(first_m + in_group % gsz);
        tn_ = __builtin_amdgcn_readfirstlane(in_group / gsz);
    };
    // lists of one problem's tiles
    int G = 0;
    if constexpr (!LISTS) G = (int)tb.gx[CAP == 1 ? 0 : &only - tb.a];
    const int nwg = LISTS ? 0 : item(cq).tiles_m * item(cq).tiles_n;
    const bool by_xcd = (G % 8 == 0);
    const int S = by_xcd ? G / 8 : G;
    const int xcd = by_xcd ? (int)wgid % 8 : 0, slot = by_xcd ? (int)wgid / 8 : (int)wgid;
    const int per = by_xcd ? nwg / 8 : nwg;
    const int n_run = slot < per ? (per - slot + S - 1) / S : 0;
    const int n_tiles = __builtin_amdgcn_readfirstlane(n_run + ((by_xcd && slot == S - 1 && xcd < nwg - 8 * per) ? 1 : 0));
    auto tile_at = [&](int i, int64_t& tm_, int64_t& tn_) __attribute__((always_inline)) {
        tile_of(item(cq), (i < n_run) ? xcd * per + slot + i * S : 8 * per + xcd, tm_, tn_);
    };
    // lists over several problems: problem (l_rest: what is left of it) and round of this workgroup's next tile, the tiles of the run
    // taken in earlier rounds, and, lane by lane, how many tiles the slots of the XCD take of the problem
    int l_q = -1, l_rest = 0, l_base = 0, l_round = 0, l_run = 0, l_begin = 0, l_take = 0;
    int l_ext = 0, l_ldx = 0, l_ldw = 0, l_ldxn = 0, l_ldwn = 0;      // row lengths of the current and the next tile's problem
    bool l_more = true;
    // nq, tmn, tnn <- the next tile of the list; left alone behind its end
    int64_t tmn = 0, tnn = 0;
    auto advance = [&]() __attribute__((always_inline)) {
        if constexpr (LISTS) {
            const int lxcd = (int)(blockIdx.x % 8), lslot = (int)(blockIdx.x / 8);
            for (;;) {
                const uint32_t m = (uint32_t)__builtin_amdgcn_ballot_w64(l_take > l_round);
                if ((m >> lslot) & 1) {
                    const int at = l_base + __builtin_popcount(m & ((1u << lslot) - 1));
                    l_base += __builtin_popcount(m);
                    ++l_round;
                    if (at < l_run) {
                        nq = l_q;
                        tile_of(item(l_q), l_begin + at, tmn, tnn);
                        return;
                    }
                }
                ++l_q;
                if (l_q == tb.n) {
                    if (l_rest) { l_more = false; return; }
                    l_rest = 1;
                    l_q = 0;
                }
                const int q = l_q;
                const int tiles = item(q).tiles_m * item(q).tiles_n, share = tiles / 8, longer = tiles - 8 * share;
                const int at8 = (lxcd - (int)tb.long_at[q]) & 7;      // this XCD's place among the runs
                l_begin = at8 * share + min(at8, longer);
                l_run = share + (at8 < longer ? 1 : 0);
                l_round = 0;
                l_base = l_rest * tb.full[q] * tb.slots;
                uint32_t w = tb.take[q][0];
#pragma unroll
                for (int k = 1; k < kListSlots / 4; ++k) w = ((lane >> 2) & 7) == k ? tb.take[q][k] : w;
                l_take = (int)((w >> (8 * (lane & 3))) & 255u);
                l_take = l_rest ? l_take : (lane & 31) < tb.slots ? tb.full[q] : 0;
            }
        }
    };
    if constexpr (LISTS) {
        advance();
        if (!l_more) return;
        cq = nq; tm = tmn; tn = tnn;
        advance();
    } else {
        if (n_tiles == 0) return;
        tile_at(0, tm, tn);
    }
    // first row and column of a tile
    auto origin = [&](int64_t t, int64_t size) __attribute__((always_inline)) {
        return HALVES ? min(t * BT, size - BT / 2) : RAGGED ? min(t * BT, size - BT) : t * BT;
    };
    // HALVES: rows between the first row of the second half and where it would be in a tile that lies inside the matrix (<= 0)
    auto second_half = [&](int64_t t, int64_t size) __attribute__((always_inline)) {
        return HALVES ? (int)(min(t * BT + BT / 2, size - BT / 2) - (origin(t, size) + BT / 2)) : 0;
    };
    int64_t m0 = origin(tm, item(cq).M), n0 = origin(tn, item(cq).N);
    int hm = second_half(tm, item(cq).M), hn = second_half(tn, item(cq).N), hmn = 0, hnn = 0;

    // ---- operand sources: X / W slices, then the prepared extension operands ----------------------
    // operand bases of the current tile (d_in slices, extension slices) and of the next tile's d_in slices
    const bf16_t *xb, *wb_, *xb2, *wb2, *wb3, *xbn, *wbn;
    auto tile_sources = [&]() __attribute__((always_inline)) {
        const bool has_ext = item(cq).Xext != nullptr;
        xb = item(cq).X + m0 * item(cq).ldx;
        wb_ = item(cq).W + n0 * item(cq).ldw;
        xb2 = has_ext ? item(cq).Xext + m0 * item(cq).ext_ld : xb;
        wb2 = has_ext ? item(cq).Wext + n0 * item(cq).ext_ld : wb_;
        wb3 = (has_ext && PHASES == 3) ? item(cq).Wext2 + n0 * item(cq).ext_ld : wb_;
    };
    // the tile after the current one (i: its index; LISTS: the list's next); past the list: the current tile once more (its first
    // slices are fetched again into the stage nobody reads)
    auto next_sources = [&](int i) __attribute__((always_inline)) {
        if constexpr (LISTS) {
            if (!l_more) { nq = cq; tmn = tm; tnn = tn; }
        } else {
            nq = cq; tmn = tm; tnn = tn;
            if (i < n_tiles) tile_at(i, tmn, tnn);
        }
        xbn = item(nq).X + origin(tmn, item(nq).M) * item(nq).ldx;
        wbn = item(nq).W + origin(tnn, item(nq).N) * item(nq).ldw;
        hmn = second_half(tmn, item(nq).M);
        hnn = second_half(tnn, item(nq).N);
        if (LISTS) { l_ldxn = (int)item(nq).ldx; l_ldwn = (int)item(nq).ldw; }
    };
    // on to the next tile
    auto next_tile = [&](int it) __attribute__((always_inline)) {
        if constexpr (LISTS) {
            cq = nq; tm = tmn; tn = tnn;
            advance();
        } else {
            tile_at(it + 1, tm, tn);
        }
        m0 = origin(tm, item(cq).M);   n0 = origin(tn, item(cq).N);
        hm = second_half(tm, item(cq).M);   hn = second_half(tn, item(cq).N);
    };
    tile_sources();
    next_sources(1);
    // LDS row 32 t + row0 of a tile: X row 32 t + row0; W row 64 (t / 2) + 8 (t mod 2) + perm64(row0) (perm64 of a row 32
    // further on is 8 more)
    const int row0 = 8 * wave + (lane >> 3);
    const int chunk0 = (lane & 7) ^ ((row0 >> 1) & 7);       // the swizzle term does not depend on t
    const int wrow0 = w_perm64(row0);
    const int vx = (int)(((int64_t)row0 * item(cq).ldx + chunk0 * 8) * 2), vw = (int)(((int64_t)wrow0 * item(cq).ldw + chunk0 * 8) * 2);
    const int vx2 = (row0 * item(cq).ext_ld + chunk0 * 8) * 2, vw2 = (wrow0 * item(cq).ext_ld + chunk0 * 8) * 2;
    const int gsx = (int)(64 * item(cq).ldx), gsw = (int)(64 * item(cq).ldw), gs2 = 64 * item(cq).ext_ld;   // bytes between row groups
    const int tail_off = (RAGGED && !LISTS && chunk0 * 8 >= (int)(item(cq).K % BK)) ? kPastEnd : 0;     // (of the slice that d_in does not fill)
    int nfull = 0, nd = 0, next = 0, npipe = 0, ktail = 0;
    // d_in slices (whole ones, all) and extension slices of the current tile's problem; npipe: slices that ride the load
    // pipeline, the d_in slices and in the one-evaluation kernel the extension behind them (at least two: the first two slices of a
    // tile are always d_in slices)
    auto count_slices = [&]() __attribute__((always_inline)) {
        nfull = (int)(item(cq).K / BK);
        nd = RAGGED ? (int)((item(cq).K + BK - 1) / BK) : nfull;
        next = item(cq).Xext != nullptr ? item(cq).ext_ld / BK : 0;
        npipe = nd + (PHASES == 1 ? next : 0);
        if (RAGGED && LISTS) ktail = (int)(item(cq).K % BK);
        if (LISTS) { l_ext = item(cq).ext_ld; l_ldx = (int)item(cq).ldx; l_ldw = (int)item(cq).ldw; }
    };
    count_slices();
    typedef __attribute__((address_space(3))) void* lptr_t;

    // ---- accumulators <- minus the target tile ----------------------------------------------------
    // 8 x 8 blocks of 16 x 16 per wave.  Lane (lc, lg) holds token 16 J + lc of token block J and, over the four output
    // blocks 4 I4 .. 4 I4 + 3, the 16 consecutive outputs 64 I4 + 16 lg + [0, 16): value 4 t + e is register e of block
    // 4 I4 + t.  The raw 16-byte vectors of the target wait in 128 registers that nothing else needs before the first
    // multiply: a whole bf16 tile, or half an fp32 one (token blocks 0..3, then 4..7)
    floatx4 acc[8][8];
    uint4 traw[32];
    auto tload = [&](auto JJ) __attribute__((always_inline)) {
        constexpr int J = decltype(JJ)::value;
        const int64_t row = m0 + wb * (128 + hm) + J * 16 + lc;
        const int64_t colw = n0 + wa * (128 + hn) + lg * 16;
        if (T_F32) {
            const uint4* src = reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(item(cq).target) + row * item(cq).ldt + colw);
#pragma clang loop unroll(full)
            for (int i4 = 0; i4 < 2; ++i4)
#pragma clang loop unroll(full)
                for (int q = 0; q < 4; ++q) traw[(J & 3) * 8 + i4 * 4 + q] = RAGGED ? load16_any(src + i4 * 16 + q) : src[i4 * 16 + q];
        } else {
            const uint4* src = reinterpret_cast<const uint4*>(reinterpret_cast<const bf16_t*>(item(cq).target) + row * item(cq).ldt + colw);
#pragma clang loop unroll(full)
            for (int i4 = 0; i4 < 2; ++i4)
#pragma clang loop unroll(full)
                for (int q = 0; q < 2; ++q) traw[J * 4 + i4 * 2 + q] = RAGGED ? load16_any(src + i4 * 8 + q) : src[i4 * 8 + q];
        }
    };
    // value of element u of block (I, J) among the raw vectors
    auto target_value = [&](int J, int I, int u) __attribute__((always_inline)) {
        if (T_F32) {
            const uint4 t = traw[(J & 3) * 8 + I];
            return __uint_as_float(u == 0 ? t.x : u == 1 ? t.y : u == 2 ? t.z : t.w);
        }
        const uint4 t = traw[J * 4 + (I >> 2) * 2 + ((I & 3) >> 1)];
        const int k = (I & 1) * 2 + (u >> 1);
        const uint32_t w = k == 0 ? t.x : k == 1 ? t.y : k == 2 ? t.z : t.w;
        return __uint_as_float((u & 1) ? w & 0xFFFF0000u : w << 16);
    };
    auto tneg = [&](auto JJ) __attribute__((always_inline)) {
        constexpr int J = decltype(JJ)::value;
#pragma clang loop unroll(full)
        for (int i4 = 0; i4 < 2; ++i4) {
            float v[16];
            if (T_F32) {
#pragma clang loop unroll(full)
                for (int q = 0; q < 4; ++q) {
                    const uint4 t = traw[(J & 3) * 8 + i4 * 4 + q];
                    v[4 * q] = -__uint_as_float(t.x); v[4 * q + 1] = -__uint_as_float(t.y);
                    v[4 * q + 2] = -__uint_as_float(t.z); v[4 * q + 3] = -__uint_as_float(t.w);
                }
            } else {
#pragma clang loop unroll(full)
                for (int q = 0; q < 2; ++q) {
                    const uint4 t = traw[J * 4 + i4 * 2 + q];
                    const uint32_t w[4] = {t.x, t.y, t.z, t.w};
#pragma clang loop unroll(full)
                    for (int u = 0; u < 4; ++u) {     // widened to fp32 with the sign flipped on the raw bits (one
                        // instruction each: adding 2^31 to the shifted word flips its top bit)
                        v[8 * q + 2 * u] = __uint_as_float((w[u] << 16) + 0x80000000u);
                        v[8 * q + 2 * u + 1] = __uint_as_float((w[u] & 0xFFFF0000u) ^ 0x80000000u);
                    }
                }
            }
#pragma clang loop unroll(full)
            for (int t = 0; t < 4; ++t) {
                floatx4 o;
#pragma clang loop unroll(full)
                for (int e = 0; e < 4; ++e) o[e] = to_acc(v[4 * t + e]);
                acc[i4 * 4 + t][J] = o;
            }
        }
    };

    // ---- multiply ---------------------------------------------------------------------------------
    // v_mfma_f32_16x16x32_bf16: two k steps of 32 per slice.  Fragment of block row I (W) or token block J (X), k step s:
    // lane (lc, lg) reads 16-byte chunk 4 s + lg of tile row 16 I + lc.  (The same flop count from this instruction
    // draws less power than from the 32x32x16 one: under the device's power limit the register-only probe holds
    // 2.2 PFLOP/s with it against 1.9.)
    int aoff[2], boff[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        aoff[ks] = W_BASE + lds_off(wa * 128 + lc, ks * 4 + lg);
        boff[ks] = X_BASE + lds_off(wb * 128 + lc, ks * 4 + lg);
    }
    bf16x8 aw[2][4], bx[8];                      // W fragments of four block rows, two sets; X fragments of the eight token blocks
    auto read_w = [&](int wbuf, int ks, int set, int i) __attribute__((always_inline)) {      // block row 4 set + i
        aw[set][i] = *reinterpret_cast<const bf16x8*>(smem + wbuf * TILE_BYTES + aoff[ks] + (set * 4 + i) * 2048);
    };
    auto read_x = [&](int xbuf, int ks, int J) __attribute__((always_inline)) {
        bx[J] = *reinterpret_cast<const bf16x8*>(smem + xbuf * TILE_BYTES + boff[ks] + J * 2048);
    };
    auto mfma1 = [&](int set, int i, int J) __attribute__((always_inline)) {
        // (written out, with the accumulator tied to one register tuple: through the builtin the compiler rotated a dozen
        // tuples per slice through vector registers)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[set * 4 + i][J]) : "v"(aw[set][i]), "v"(bx[J]));
    };
    // source of a pipelined slice, chosen once per slice with scalar selects (no branches at the load sites)
    __amdgpu_buffer_rsrc_t src_rsx = rsrc(xb), src_rsw = rsrc(wb_);
    int src_so = 0;
    // vector offsets of a lane's eight row groups per operand, kept in registers: worked out in front of each load they
    // put an add and its latency between a matrix instruction and the load behind it
    int src_vxt[8], src_vwt[8];
    // (hx, hw: bytes that the second half's rows lie further on)
    auto set_offsets = [&](int v0x, int gx, int hx, int v0w, int gw, int hw) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            src_vxt[t] = v0x + t * gx + (HALVES && t >= 4 ? hx : 0);
            src_vwt[t] = v0w + (t >> 1) * (2 * gw) + (t & 1) * (gw >> 2) + (HALVES && t >= 4 ? hw : 0);
        }
    };
    // kt counts from the current tile's first slice; npipe and npipe + 1 are the first two slices of the next tile.
    // Two rounds of selects, each on one condition, between values (a select between captured references becomes a
    // computed address into the closure, which then stays in memory with everything it points to; and selects on
    // mixed conditions cost four scalar instructions each instead of one)
    auto select_slice = [&](int kt) __attribute__((always_inline)) {
        // (copies first: the selects then see values, not addresses of captured variables)
        const bf16_t *cxb = xb, *cwb = wb_, *cxb2 = xb2, *cwb2 = wb2, *cxbn = xbn, *cwbn = wbn;
        const bool e = kt >= nd;                             // extension operands (or, past npipe, the next tile)
        const bf16_t* xs = e ? cxb2 : cxb;
        const bf16_t* ws = e ? cwb2 : cwb;
        int so = e ? kt - nd : kt;
        const bool nxt = kt >= npipe;
        xs = nxt ? cxbn : xs;
        ws = nxt ? cwbn : ws;
        so = nxt ? kt - npipe : so;
        int svx, svw, sgx, sgw, hx = 0, hw = 0;
        if constexpr (LISTS) {
            // (the next tile may be another problem's: its offsets from its row lengths)
            const int cle = l_ext, clx = l_ldx, clw = l_ldw, cnx = l_ldxn, cnw = l_ldwn;
            int lx = e ? cle : clx, lw = e ? cle : clw;
            lx = nxt ? cnx : lx;   lw = nxt ? cnw : lw;
            svx = (row0 * lx + chunk0 * 8) * 2;   svw = (wrow0 * lw + chunk0 * 8) * 2;
            sgx = 64 * lx;   sgw = 64 * lw;
        } else {
            const int cvx = vx, cvw = vw, cvx2 = vx2, cvw2 = vw2, cgsx = gsx, cgsw = gsw, cgs2 = gs2;
            svx = e ? cvx2 : cvx;   svw = e ? cvw2 : cvw;   sgx = e ? cgs2 : cgsx;   sgw = e ? cgs2 : cgsw;
            svx = nxt ? cvx : svx;   svw = nxt ? cvw : svw;   sgx = nxt ? cgsx : sgx;   sgw = nxt ? cgsw : sgw;
        }
        if constexpr (HALVES) {
            const int chm = hm, chn = hn, chmn = hmn, chnn = hnn;
            hx = (nxt ? chmn : chm) * (sgx / 32);   hw = (nxt ? chnn : chn) * (sgw / 32);
        }
        uint32_t bytes = 0xFFFFFFFFu;
        if constexpr (RAGGED) {
            const bool last = kt == nfull && kt < nd;        // the slice that d_in does not fill
            const int past = !LISTS ? (last ? tail_off : 0) : (last && chunk0 * 8 >= ktail) ? kPastEnd : 0;
            svx += past;   svw += past;
            bytes = last ? (uint32_t)kPastEnd : bytes;
        }
        src_rsx = rsrc(xs, bytes);   src_rsw = rsrc(ws, bytes);
        set_offsets(svx, sgx, hx, svw, sgw, hw);
        src_so = so * (BK * 2);
    };
    // direct load of row group t (0..7) of the selected slice: X into X stage buf (0..1), W into W stage buf (0..2)
    auto dma_x = [&](int buf, int t) __attribute__((always_inline)) {
        char* dst = smem + X_BASE + buf * TILE_BYTES + wave * 1024 + t * 4096;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(src_rsx, (lptr_t)dst, 16, src_vxt[t], src_so, 0, 0);
    };
    auto dma_w = [&](int buf, int t) __attribute__((always_inline)) {
        char* dst = smem + W_BASE + buf * TILE_BYTES + wave * 1024 + t * 4096;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(src_rsw, (lptr_t)dst, 16, src_vwt[t], src_so, 0, 0);
    };
    // 32 MFMAs in fixed issue order: the block rows 4 SET .. 4 SET + 3 against the eight token blocks, token block by token
    // block, with the fragments in registers.  Rides along: the W fragments of the other set for the block after this one
    // (k step RKS of W stage rwbuf), one after the third instruction of every other token block; with REFILL, the X fragment
    // of token block J for the next k step (RKS of X stage rxbuf) as soon as the block's last instruction on it has issued;
    // the eight direct loads of one operand of the selected slice, one behind the first instruction of each token block
    // (LOADS: 0 none, 1 W, 2 X)
    auto block = [&](auto SET, auto RKS, auto REFILL, int rxbuf, int rwbuf, auto LOADS, int lbuf) __attribute__((always_inline)) {
        constexpr int set = decltype(SET)::value, rks = decltype(RKS)::value, loads = decltype(LOADS)::value;
        constexpr bool refill = decltype(REFILL)::value != 0;
#pragma unroll
        for (int J = 0; J < 8; ++J) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                mfma1(set, i, J);
                if (i == 0 && loads == 1) dma_w(lbuf, J);
                if (i == 0 && loads == 2) dma_x(lbuf, J);
                if (i == 2 && J < 4) read_w(rwbuf, rks, set ^ 1, J);
                if (i == 3 && refill) read_x(rxbuf, rks, J);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // The matrix instructions are written out, so the compiler does not know of them and keeps no distance between them and what
    // touches their results (8 wait states).  Behind a tile's slices: these 24, and then from_acc(), for such statements stay in
    // order where an ordinary read could come in front.  In the shared-forward schedule, which multiplies on between evaluations
    // and would copy what it read by hand, the wait is part of what multiplies: the last statement of a slice, below and in the
    // loop over the slices
    auto settle = [&]() __attribute__((always_inline)) { asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7"); };
    // a slice whose operands are complete in buffer `buf`, unpipelined; each k step is one statement, from the wait between a
    // value's last write and the first instruction to the one behind the last
#define MM(I, J) "v_mfma_f32_16x16x32_bf16 %[c" #I #J "], %[w" #I "], %[x" #J "], %[c" #I #J "]\n\t"
#define MM_TOKENS(A, B, C, D, J) MM(A, J) MM(B, J) MM(C, J) MM(D, J)
#define MM_SET(A, B, C, D)                                                                                                       \
    MM_TOKENS(A, B, C, D, 0) MM_TOKENS(A, B, C, D, 1) MM_TOKENS(A, B, C, D, 2) MM_TOKENS(A, B, C, D, 3)                          \
    MM_TOKENS(A, B, C, D, 4) MM_TOKENS(A, B, C, D, 5) MM_TOKENS(A, B, C, D, 6) MM_TOKENS(A, B, C, D, 7)
#define ACC(I, J) [c##I##J] "+a"(acc[I][J])
#define ACC_ROW(I) ACC(I, 0), ACC(I, 1), ACC(I, 2), ACC(I, 3), ACC(I, 4), ACC(I, 5), ACC(I, 6), ACC(I, 7)
    auto multiply_slice = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int J = 0; J < 8; ++J) read_x(buf, ks, J);
#pragma unroll
            for (int I = 0; I < 8; ++I) read_w(buf, ks, I >> 2, I & 3);
            asm volatile("s_nop 1\n\t" MM_SET(0, 1, 2, 3) MM_SET(4, 5, 6, 7) "s_nop 7"
                         : ACC_ROW(0), ACC_ROW(1), ACC_ROW(2), ACC_ROW(3), ACC_ROW(4), ACC_ROW(5), ACC_ROW(6), ACC_ROW(7)
                         : [w0] "v"(aw[0][0]), [w1] "v"(aw[0][1]), [w2] "v"(aw[0][2]), [w3] "v"(aw[0][3]),
                           [w4] "v"(aw[1][0]), [w5] "v"(aw[1][1]), [w6] "v"(aw[1][2]), [w7] "v"(aw[1][3]),
                           [x0] "v"(bx[0]), [x1] "v"(bx[1]), [x2] "v"(bx[2]), [x3] "v"(bx[3]),
                           [x4] "v"(bx[4]), [x5] "v"(bx[5]), [x6] "v"(bx[6]), [x7] "v"(bx[7]));
        }
    };
#undef MM
#undef MM_TOKENS
#undef MM_SET
#undef ACC
#undef ACC_ROW

    // ---- sum of squares of the accumulators: fp32 squares four at a time, summed in fp64; lanes, then waves, in a
    // fixed order ----
    // The four waves' sums meet in LDS, in `red`: the head of a W stage that nothing reads or fills at that moment
    // (the operand stages take all of the LDS)
    // HALVES: rows and columns of the wave's half that the half before it has counted are left out (a half beyond the last row or
    // column has nothing that counts).  A column tile that overlaps the one before it by no multiple of 16, and all tiles of
    // a layer whose target rows do not start on 16 bytes, are squared in fp64 as well: what gemm_bf16.hip squares so keeps its
    // precision here.  (Otherwise a lane's 16 columns of a group count or do not count together; the wide form takes some 2 us more
    // a tile)
    // HALVES: the sums of the wave's four 64 x 64 blocks (outputs, tokens) by themselves
    auto eval_sum = [&](double (&part)[2][2]) __attribute__((always_inline)) {
        part[0][0] = 0.0;
        if (HALVES) part[0][1] = part[1][0] = part[1][1] = 0.0;
        if constexpr (PHASES == 1) settle();
        const int rs = RAGGED ? (int)(tm * BT - m0) - (HALVES ? wb * hm : 0) : 0;
        const int cs0 = RAGGED ? (int)(tn * BT - n0) : 0, cs = cs0 - (HALVES ? wa * hn : 0);
        auto sum = [&](auto WIDE) __attribute__((always_inline)) {
            constexpr bool wide = decltype(WIDE)::value != 0;
#pragma clang loop unroll(full)
            for (int J = 0; J < 8; ++J) {
                if (LATE_T && PHASES == 1 && T_F32 && J == 4) { tload(IC<4>{}); tload(IC<5>{}); tload(IC<6>{}); tload(IC<7>{}); }
                // the first of the lane's 16 columns per group that counts
                int from[2] = {0, 0};
                if (RAGGED) {
                    const bool in = (HALVES ? 0 : wb * 128) + J * 16 + lc >= rs;
                    from[0] = in ? cs - ((HALVES ? 0 : wa * 128) + lg * 16) : 16;
                    from[1] = in ? cs - ((HALVES ? 0 : wa * 128) + 64 + lg * 16) : 16;
                    // (or the compiler works out all conditions ahead and keeps them)
                    asm volatile("" : "+v"(from[0]), "+v"(from[1]));
                }
#pragma clang loop unroll(full)
                for (int I = 0; I < 8; ++I) {
                    const floatx4 v = acc[I][J];
                    double& sum64 = part[HALVES ? I >> 2 : 0][HALVES ? J >> 2 : 0];
                    float s4 = 0.f;
#pragma clang loop unroll(full)
                    for (int u = 0; u < 4; ++u) {
                        // (the shared-forward schedule multiplies on after an evaluation and nothing else is live there)
                        float x = (PHASES == 1) ? from_acc(v[u]) : v[u];
                        if (LATE_T && PHASES == 1) x -= target_value(J, I, u);
                        if (wide) {
                            const double xd = (I & 3) * 4 + u >= from[I >> 2] ? (double)x : 0.0;
                            sum64 = fma(xd, xd, sum64);
                        } else {
                            s4 = fmaf(x, x, s4);
                        }
                    }
                    if (!wide) sum64 += (double)(!RAGGED || from[I >> 2] <= 0 ? s4 : 0.f);
                }
            }
        };
        if (RAGGED && (((LISTS && item(cq).sub ? cs : cs0 | (HALVES ? cs0 - hn : 0)) & 15) != 0 || !item(cq).vec_ok)) sum(IC<1>{});
        else sum(IC<0>{});
    };
    // of one problem's tile
    auto eval_finish = [&](const double (&part4)[2][2], const AlignedItem& a, int phase, int64_t tm_, int64_t tn_, double* red) __attribute__((always_inline)) {
        if (HALVES && a.sub) {
            // the wave's half of the tile is a tile of gemm_bf16_mid.hip: its lanes, then its four blocks, in the order of that kernel's
            // lanes and waves.  Each step of the sum over the lanes halves the blocks that a lane sums
            const bool out1 = (lane & 32) != 0, tok1 = (lane & 16) != 0;
            const double a0 = (out1 ? part4[1][0] : part4[0][0]) + __shfl_xor(out1 ? part4[0][0] : part4[1][0], 32);
            const double a1 = (out1 ? part4[1][1] : part4[0][1]) + __shfl_xor(out1 ? part4[0][1] : part4[1][1], 32);
            double b = (tok1 ? a1 : a0) + __shfl_xor(tok1 ? a0 : a1, 16);
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) b += __shfl_xor(b, off);
            b += __shfl_xor(b, 16);
            b += __shfl_xor(b, 32);
            const int64_t bm = 2 * tm_ + wb, bn = 2 * tn_ + wa, blocks_n = (a.N + BT / 2 - 1) / (BT / 2);
            if (lane == 0 && bm * (BT / 2) < a.M && bn < blocks_n) a.partials[bm * blocks_n + bn] = b;
            return;
        }
        double part = HALVES ? (part4[0][0] + part4[0][1]) + (part4[1][0] + part4[1][1]) : part4[0][0];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
        if (lane == 0) red[phase * 4 + wave] = part;
        __syncthreads();
        if (tid == 0)
            a.partials[(int64_t)phase * a.tiles_m * a.tiles_n + tm_ * a.tiles_n + tn_] =
                (red[phase * 4] + red[phase * 4 + 1]) + (red[phase * 4 + 2] + red[phase * 4 + 3]);
        // (one-evaluation kernel: the next slice's loads go into this stage, and no wave may issue them before the sums
        // have been read)
        if constexpr (PHASES == 1) __syncthreads();
    };
    auto evaluate = [&](int phase, double* red) __attribute__((always_inline)) {
        double part[2][2];
        eval_sum(part);
        eval_finish(part, item(cq), phase, tm, tn, red);
    };

    // accumulators <- minus the target tile (squared error) or zero (stored output)
    auto start_tile = [&]() __attribute__((always_inline)) {
        if constexpr (OUT == 0 && !LATE_T) {
            tneg(IC<0>{}); tneg(IC<1>{}); tneg(IC<2>{}); tneg(IC<3>{});
            if (T_F32) { tload(IC<4>{}); tload(IC<5>{}); tload(IC<6>{}); tload(IC<7>{}); }
            tneg(IC<4>{}); tneg(IC<5>{}); tneg(IC<6>{}); tneg(IC<7>{});
        } else {
#pragma unroll
            for (int I = 0; I < 8; ++I)
#pragma unroll
                for (int J = 0; J < 8; ++J)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[I][J][e] = 0.f;
        }
    };
    auto request_target = [&]() __attribute__((always_inline)) {
        if constexpr (OUT == 0) {
            tload(IC<0>{}); tload(IC<1>{}); tload(IC<2>{}); tload(IC<3>{});
            if (!T_F32) { tload(IC<4>{}); tload(IC<5>{}); tload(IC<6>{}); tload(IC<7>{}); }
        }
    };

    // ---- first tile: target and the first two slices ------------------------------------------------
    if constexpr (!LATE_T) request_target();
    select_slice(0);
#pragma unroll
    for (int t = 0; t < 8; ++t) { dma_x(0, t); dma_w(0, t); }
    select_slice(1);
#pragma unroll
    for (int t = 0; t < 8; ++t) { dma_x(1, t); dma_w(1, t); }

    int g = 0;                                   // slices multiplied so far: slice g sits in W stage g mod 3, X stage g & 1
    int wst = 0;                                  // g mod 3
    for (int it = 0;; ++it) {
        // the accumulators are written here and nowhere else, and are dead at the end of the loop body: carried around
        // the loop they would pass through a join, which the compiler answers by spilling them
        start_tile();
        if (it == 0) {
            __builtin_amdgcn_s_waitcnt(0x4F70);              // vmcnt(16): slice 0 has landed
            __syncthreads();
#pragma unroll
            for (int J = 0; J < 8; ++J) read_x(0, 0, J);
#pragma unroll
            for (int i = 0; i < 4; ++i) read_w(0, 0, 0, i);
        }
        // every slice of the tile, the last one included, with its W in stage wst and its X in stage cur: on entry the X
        // fragments and W fragment set 0 hold its first k step, the next slice's W has landed or is in flight and its X is
        // in flight; the same holds for the next slice on exit
        for (int kt = 0; kt < npipe; ++kt, ++g) {
            const int cur = g & 1;
            const int wst1 = (wst == 2) ? 0 : wst + 1, wst2 = (wst == 0) ? 2 : wst - 1;      // stages of slices g + 1, g + 2
            // while the slice after next is a d_in slice of this tile only the K offset moves; the general choice
            // (extension operands, next tile: some 60 scalar instructions in front of a matrix instruction) is left to
            // the last slices of a tile, behind a branch that is rarely taken
            const bool tail = kt + 2 >= nfull;
            if (__builtin_expect(tail, 0)) select_slice(kt + 2);
            else src_so = (kt + 2) * (BK * 2);
            // W of slice g + 2 goes into the stage that slice g - 1 left at the previous barrier, six blocks before its
            // first fragment is read (issued in the second block: the first still sees the X loads of the block before it)
            block(IC<0>{}, IC<0>{}, IC<0>{}, cur, wst, IC<0>{}, 0);
            block(IC<1>{}, IC<1>{}, IC<1>{}, cur, wst, IC<1>{}, wst2);
            block(IC<0>{}, IC<1>{}, IC<0>{}, cur, wst, IC<0>{}, 0);
            // vmcnt(8) lgkmcnt(0): all but the eight W loads of this slice have landed (loads return in the order
            // issued), which is the whole of the next slice
            __builtin_amdgcn_s_waitcnt(0x0078);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            // every wave has read this slice's X: X of slice g + 2 goes into its stage, three blocks ahead
            block(IC<1>{}, IC<0>{}, IC<1>{}, cur ^ 1, wst1, IC<2>{}, cur);
            // (half of the time that the last matrix instruction takes anyway)
            if constexpr (PHASES != 1) asm volatile("s_nop 7");
            wst = wst1;
        }
        // the tile's last matrix instruction has issued; the stages of slice g hold the next tile's first slice, fragment
        // set 0 its sub-step 0, and its second slice is in flight; W stage wst - 1 is idle until the next W loads
        const bool more = LISTS ? l_more : it + 1 < n_tiles;
        if constexpr (OUT == 1) {
            // A lane holds 16 consecutive outputs of one token per group of four blocks, so stored from the registers every
            // store touches 16 rows.  Instead each wave passes its 128 x 128 block through LDS, 32 tokens at a time, in its
            // quarter of the W stage that is idle between two tiles: written as held (16-byte chunk c of row t at
            // c ^ (t mod 16): the lanes of one write spread over all banks), read back 16 lanes to a 256-byte row, and
            // stored four whole rows to an instruction.
            settle();
            char* stg = smem + W_BASE + ((wst == 0) ? 2 : wst - 1) * TILE_BYTES + wave * 8192;
#pragma clang loop unroll(full)
            for (int r2 = 0; r2 < 4; ++r2) {
#pragma clang loop unroll(full)
                for (int jj = 0; jj < 2; ++jj) {
                    const int J = 2 * r2 + jj, trow = jj * 16 + lc;
#pragma clang loop unroll(full)
                    for (int i4 = 0; i4 < 2; ++i4) {
                        uint32_t w[8];
#pragma clang loop unroll(full)
                        for (int t = 0; t < 4; ++t) {
                            const floatx4 v = acc[i4 * 4 + t][J];
                            w[2 * t] = pack_bf16x2(from_acc(v[0]), from_acc(v[1]));
                            w[2 * t + 1] = pack_bf16x2(from_acc(v[2]), from_acc(v[3]));
                        }
                        const int c0 = i4 * 8 + lg * 2;
                        *reinterpret_cast<uint4*>(stg + trow * 256 + ((c0 ^ (trow & 15)) << 4)) = make_uint4(w[0], w[1], w[2], w[3]);
                        *reinterpret_cast<uint4*>(stg + trow * 256 + (((c0 + 1) ^ (trow & 15)) << 4)) = make_uint4(w[4], w[5], w[6], w[7]);
                    }
                }
                const int cc = lane & 15;
#pragma clang loop unroll(full)
                for (int n = 0; n < 8; ++n) {
                    const int t = 4 * n + (lane >> 4);
                    const uint4 v = *reinterpret_cast<const uint4*>(stg + t * 256 + ((cc ^ (t & 15)) << 4));
                    bf16_t* dst = reinterpret_cast<bf16_t*>(item(cq).Y) + (m0 + wb * 128 + r2 * 32 + t) * item(cq).ldy + n0 + wa * 128 + cc * 8;
                    if (RAGGED) store16_any(dst, v);
                    else *reinterpret_cast<uint4*>(dst) = v;
                }
            }
            __syncthreads();                                 // the next W loads go into that stage
            if (!more) break;
        } else if constexpr (OUT == 2) {
            // a lane holds 32 of the 128 logits of the wave's columns for each of eight tokens; the lanes lane ^ 16, ^ 32, ^ 48
            // hold the others.  Online softmax over the wave's 128 columns, per token
            settle();
            // columns that the tile before this one has counted stay out (rows that it has counted get the same values again);
            // cskip: how many of the lane's 16 columns per group those are
            const int cs = RAGGED ? (int)(tn * BT - n0) : 0;
            const int cskip[2] = {cs - (wa * 128 + lg * 16), cs - (wa * 128 + 64 + lg * 16)};
            // one token block; SKIP: some of the wave's columns may have been counted
            auto statistics = [&](int J, auto SKIP) __attribute__((always_inline)) {
                constexpr bool skip = decltype(SKIP)::value != 0;
                const int64_t row = m0 + wb * 128 + J * 16 + lc;
                const int tgt = item(cq).ce_target[row];
                // (the block's 32 values leave the accumulation registers once, for the maximum, the exponentials and the target)
                float y[8][4];
                float mx = -INFINITY;
#pragma clang loop unroll(full)
                for (int I = 0; I < 8; ++I)
#pragma clang loop unroll(full)
                    for (int e = 0; e < 4; ++e) {
                        y[I][e] = from_acc(acc[I][J][e]);
                        if (!skip || 4 * (I & 3) + e >= cskip[I >> 2]) mx = fmaxf(mx, y[I][e]);
                    }
                mx = fmaxf(mx, __shfl_xor(mx, 16));
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                // exp(y - mx) as 2^((y - mx) log2 e) on the hardware exponential: the difference is exact enough in fp32
                // (one rounding), the terms that matter have small exponents, and the far tail underflows to 0
                float sm = 0.f;
#pragma clang loop unroll(full)
                for (int I = 0; I < 8; ++I)
#pragma clang loop unroll(full)
                    for (int e = 0; e < 4; ++e) {
                        const float ex = __builtin_amdgcn_exp2f((y[I][e] - mx) * 1.44269504088896341f);
                        sm += (!skip || (I & 3) * 4 + e >= cskip[I >> 2]) ? ex : 0.f;
                    }
                sm += __shfl_xor(sm, 16);
                sm += __shfl_xor(sm, 32);
                const int64_t chunk = tn * 2 + wa;           // of tiles_n x 2 chunks per token
                if (lg == 0) item(cq).ce_ms[chunk * item(cq).M + row] = make_float2(mx, sm);
                // the target's logit: one token in d_out / 128 has its target among the wave's columns, so most waves have none in
                // the block's sixteen, and nothing to look for (looked for along with the maximum it was two instructions a logit)
                const int64_t trel = (int64_t)tgt - (n0 + wa * 128);
                const bool mine = tgt >= 0 && trel >= 0 && trel < 128 && (((int)trel >> 4) & 3) == lg;
                if (__builtin_amdgcn_ballot_w64(mine) != 0) {
                    float tl = 0.f;
                    const int at = (int)trel & 15, grp = (int)trel >> 6;
#pragma clang loop unroll(full)
                    for (int I = 0; I < 8; ++I)
#pragma clang loop unroll(full)
                        for (int e = 0; e < 4; ++e)
                            if (grp == (I >> 2) && at == 4 * (I & 3) + e) tl = y[I][e];
                    if (mine) item(cq).ce_tl[row] = tl;
                }
            };
            auto tile_statistics = [&](auto SKIP) __attribute__((always_inline)) {
                statistics(0, SKIP); statistics(1, SKIP); statistics(2, SKIP); statistics(3, SKIP);
                statistics(4, SKIP); statistics(5, SKIP); statistics(6, SKIP); statistics(7, SKIP);
            };
            // (only the last column tile overlaps the one before it)
            if (RAGGED && cs != 0) tile_statistics(IC<1>{});
            else tile_statistics(IC<0>{});
            if (!more) break;
        } else if constexpr (PHASES == 1) {
            const int64_t tm_done = tm, tn_done = tn;
            const int q_done = cq;
            double part[2][2];
            if constexpr (LATE_T) {
                request_target();
                eval_sum(part);
                if (more) next_tile(it);
            } else if (more) {
                next_tile(it);
                // The next tile's target is requested and the finished tile summed, in one order by two of the waves and in
                // the other by the other two: a request keeps its wave's issue port for as long as the address unit takes
                // over its 64 rows, and the address unit is the compute unit's one, so four waves requesting at once wait
                // for each other while nobody sums
                if (wave < 2) { request_target(); eval_sum(part); }
                else { eval_sum(part); request_target(); }
            } else {
                eval_sum(part);
            }
            eval_finish(part, item(q_done), 0, tm_done, tn_done, reinterpret_cast<double*>(smem + W_BASE + ((wst == 0) ? 2 : wst - 1) * TILE_BYTES));
            if (!more) break;
        } else {
            // shared forward: one tile per workgroup.  All LDS stages are free once the re-fetched slices have landed: the
            // first extension slice of each perturbed evaluation is requested before the evaluation that precedes it (X and
            // W stages 0 for +eps, 1 for -2 eps); further slices (r > 16) one at a time; the sums meet in W stage 2
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
            const __amdgpu_buffer_rsrc_t rx2 = rsrc(xb2), rw2 = rsrc(wb2), rw3 = rsrc(wb3);
            auto ext_dma = [&](const __amdgpu_buffer_rsrc_t& rws, int e, int buf) __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int t = q >> 1;
                    char* dst = smem + buf * TILE_BYTES + wave * 1024 + t * 4096 + ((q & 1) ? W_BASE : X_BASE);
                    if (q & 1) __builtin_amdgcn_raw_ptr_buffer_load_lds(rws, (lptr_t)dst, 16, vw2 + (t >> 1) * (2 * gs2) + (t & 1) * (gs2 >> 2), e * (BK * 2), 0, 0);
                    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rx2, (lptr_t)dst, 16, vx2 + t * gs2, e * (BK * 2), 0, 0);
                }
            };
            if (next > 0) ext_dma(rw2, 0, 0);
            double* red = reinterpret_cast<double*>(smem + W_BASE + 2 * TILE_BYTES);
            if constexpr (LATE_T) {                          // from here on the accumulators hold residuals
                request_target();
#pragma clang loop unroll(full)
                for (int J = 0; J < 8; ++J) {
                    if (T_F32 && J == 4) { tload(IC<4>{}); tload(IC<5>{}); tload(IC<6>{}); tload(IC<7>{}); }
#pragma clang loop unroll(full)
                    for (int I = 0; I < 8; ++I)
#pragma clang loop unroll(full)
                        for (int u = 0; u < 4; ++u) acc[I][J][u] -= target_value(J, I, u);
                }
            }
            // (rolled: the accumulators of three evaluations in a row end up in scratch memory)
#pragma clang loop unroll(disable)
            for (int ph = 0;; ++ph) {
                evaluate(ph, red);
                if (ph == 2) break;
                const __amdgpu_buffer_rsrc_t rwp = rsrc(ph == 0 ? wb2 : wb3);
                if (ph == 0) ext_dma(rw3, 0, 1);
#pragma clang loop unroll(disable)
                for (int e = 0; e < next; ++e) {
                    if (e > 0) {
                        __syncthreads();
                        ext_dma(rwp, e, ph);
                    }
                    __builtin_amdgcn_s_waitcnt(0x0F70);
                    __syncthreads();
                    multiply_slice(ph);
                }
            }
            break;
        }
        // ---- hand the accumulators to the next tile ----
        if constexpr (OUT != 0) next_tile(it);
        if constexpr (LISTS) count_slices();
        tile_sources();
        next_sources(it + 2);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // the slices fetched past the end of the list
    if (!LISTS && item(cq).clk && wgid == 0 && tid == 0) { item(cq).clk[2] = __builtin_readcyclecounter(); item(cq).clk[3] = wall_clock64(); }
}

template <int OUT, bool T_F32, int PHASES, bool RAGGED, int CAP>
static hipError_t launch_aligned_grid(const AlignedArgs<PHASES, CAP>& tb, unsigned blocks, hipStream_t st) {
    static bool attr_set = false;
    const int smem = 5 * TILE_BYTES;           // three W stages and two X stages: all 160 KiB of a compute unit's LDS
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_bf16_aligned_kernel<OUT, T_F32, PHASES, RAGGED, CAP>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((gemm_bf16_aligned_kernel<OUT, T_F32, PHASES, RAGGED, CAP>), dim3(blocks), dim3(256), smem, st, tb);
    return hipGetLastError();
}

static AlignedItem aligned_item(const GemmParams& p) {
    AlignedItem a;
    a.X = p.X; a.W = p.W; a.Xext = p.Xext; a.Wext = p.Wext; a.Wext2 = p.Wext2;
    a.ldx = p.ldx; a.ldw = p.ldw; a.M = p.M; a.N = p.N; a.K = p.K; a.ldt = p.ldt; a.ldy = p.ldy;
    a.target = p.target; a.partials = p.partials; a.Y = p.Y;
    a.ce_target = p.ce_target; a.ce_ms = p.ce_ms; a.ce_tl = p.ce_tl; a.clk = p.clk;
    a.ext_ld = p.ext_ld; a.tiles_m = (int)((p.M + BT - 1) / BT); a.tiles_n = (int)((p.N + BT - 1) / BT); a.group_m = p.group_m; a.vec_ok = p.vec_ok;
    a.sub = 0;
    return a;
}

// one workgroup per compute unit, each with a list of tiles (a multiple of 8 workgroups: one share per XCD)
template <int OUT, bool T_F32, bool RAGGED>
static hipError_t launch_aligned_lists(const GemmParams& p, hipStream_t st) {
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (cus < 1) return hipErrorInvalidDevice;
    // (rounded up: workgroups without a tile leave at once, while one short of a workgroup per tile 190 or 250 tiles took
    // the time of two)
    int64_t G = ((int64_t)p.tiles_m * p.tiles_n + 7) / 8 * 8;
    if (G > cus) G = cus >= 8 ? cus - cus % 8 : cus;
    if (p.slots > 0 && G > 8 * p.slots) G = 8 * p.slots;
    const KBatch<AlignedItem, 1> tb{1, {0}, {(uint32_t)G}, {aligned_item(p)}};
    return launch_aligned_grid<OUT, T_F32, 1, RAGGED, 1>(tb, (unsigned)G, st);
}

static hipError_t list_slots(int* slots) {
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    *slots = cus / 8 < kListSlots ? cus / 8 : kListSlots;
    return cus < 1 ? hipErrorInvalidDevice : hipSuccess;
}

// Microseconds that a slice and the change of tiles take, with all compute units at it
constexpr double kSliceUs = 1.3, kTileUs = 8.0;
// ... the softmax statistics of a tile, and a fork of a stream with its join
constexpr double kStatisticsUs = 6.0, kForkUs = 25.0;
static double tile_us(const AlignedItem& a) { return kSliceUs * (double)((a.K + BK - 1) / BK + (a.Xext ? a.ext_ld / BK : 0)) + kTileUs; }

// Deals the tiles of an XCD's runs to its workgroups; the deepest problems come first, and what is left behind the rounds goes
// tile by tile to the workgroup that is done first.  Returns when the last is done, in microseconds
static double deal_tiles(const AlignedItem* const* a, int n, int slots, TileLists& tb) {
    double busy[kListSlots] = {};
    int long_at = 0;
    tb.n = n;
    tb.slots = slots;
    for (int q = 0; q < n; ++q) {
        const int64_t tiles = (int64_t)a[q]->tiles_m * a[q]->tiles_n;
        const double cost = tile_us(*a[q]);
        tb.full[q] = (int)(tiles / 8 / slots);
        for (int s = 0; s < slots; ++s) busy[s] += (double)tb.full[q] * cost;
        tb.long_at[q] = (uint8_t)long_at;
        long_at = (int)((long_at + tiles % 8) % 8);
    }
    for (int q = 0; q < n; ++q) {
        const int64_t tiles = (int64_t)a[q]->tiles_m * a[q]->tiles_n;
        for (int w = 0; w < kListSlots / 4; ++w) tb.take[q][w] = 0;
        for (int64_t left = (tiles + 7) / 8 - (int64_t)tb.full[q] * slots; left > 0; --left) {      // (at most one a slot, or one more)
            int at = 0;
            for (int s = 1; s < slots; ++s) at = busy[s] < busy[at] ? s : at;
            tb.take[q][at / 4] += 1u << (8 * (at % 4));
            busy[at] += tile_us(*a[q]);
        }
    }
    double end = 0.0;
    for (int s = 0; s < slots; ++s) end = busy[s] > end ? busy[s] : end;
    return end;
}

// Forwards beside work on another stream, a chain of launches that is bound by its latencies and by the compute units it has: a
// workgroup of the lists holds its compute unit to the end, so a launch on all of them keeps the chain waiting, and one on too few
// outlasts it.  The number of workgroups per XCD for which both should be done first: the chain takes its latencies and its sweeps on
// the compute units left (29 GB/s each, of the 22 that each has of the rate of all together), and goes on with all of them behind the
// forwards.  Base forwards and extraction, us, in launches of their
// own (start) and in lists on 256, 224, 192 and 160 compute units: 4B-sized layers on 3001 tokens 824, 801, 760, 734 and 686, on 4096 924,
// 974, 933, 904 and 821 (but 68 more behind it), on 1500 556, 507, 472, 463 and 450, 8B-sized on 15028, r = 1, 5371, 5525, 5341 and
// 4879 (but 850 more behind it)
static int slots_beside(const GemmBeside& b, double total, double deepest, int slots) {
    int best = slots;
    double best_us = -1.0;
    for (int s = slots; s >= 1; s = s > 4 ? (s - 1) / 4 * 4 : s - 1) {      // (in fours: rounds of 25 share operand slices less well than of 24)
        const double forwards = total / (8.0 * s) > deepest ? total / (8.0 * s) : deepest;
        const double left = s < slots ? 22.0 / 29.0 * slots / (slots - s) : -1.0;
        const double all = b.latency_us + b.sweep_us, slow = left < 0.0 ? left : b.latency_us + b.sweep_us * (left > 1.0 ? left : 1.0);
        const double done = slow < 0.0 ? 0.0 : forwards / slow;
        const double us = done >= 1.0 ? forwards : forwards + (1.0 - done) * all;
        if (best_us < 0.0 || us < 1.05 * best_us) { best = s; best_us = best_us < 0.0 || us < best_us ? us : best_us; }      // (of about equal ones the fewest)
    }
    return best;
}

// The same for one problem in a launch of its own (slots.h).  Four compute units of each XCD at least are left (a chain on 16 in all took longer
// than its forward: 20000 outputs of 4096 on 1500 tokens, r =
// 16, 735 and 755).  A step of one layer, us, one stream and two (K = 3): cross-entropy, 2048 -> 32000 on 3001 tokens, r = 16, 1105 and 1003, on
// 8192 2522 and 2514, 1024 -> 9000 on 700 241 and 223, on 8192 629 and 531; squared error, 4096 -> 4096 on 3001 394 and 349, 1024 ->
// 8192 on 8192 489 and 422, 8192 -> 8192 on 8192 2507 and 2391, r = 1 2427 and 2374, r = 64 3072 and 2876.  Of 19 shapes and r = 1, 16 and 64 none
// was more than 0.5 % slower
int gemm_bf16_aligned_slots(const GemmParams& p, const GemmBeside& b) {
    int slots = 0;
    if (list_slots(&slots) != hipSuccess) return 0;
    const double tile = tile_us(aligned_item(p)) + (p.loss_kind == AGZO_LOSS_CE ? kStatisticsUs : 0.0);
    return lone_slots(((int64_t)p.tiles_m * p.tiles_n + 7) / 8, slots, tile, b.latency_us, b.sweep_us, kForkUs);
}

static bool aligned_fits(const GemmParams& p) { return p.M >= BT && p.N >= BT && p.K >= 2 * BK && (p.P == nullptr || p.Xext != nullptr); }
static bool aligned_ragged(const GemmParams& p) { return !(p.vec_ok && p.M % BT == 0 && p.N % BT == 0 && p.K % BK == 0); }

bool gemm_bf16_aligned_listed(const GemmParams& p) {
    return aligned_fits(p) && !p.shared && !p.Y && p.loss_kind == AGZO_LOSS_MSE && p.target_dtype == AGZO_BF16;
}

// Several layers' squared errors.  Layers of few tiles leave compute units idle in the last round of a launch of their own, most of all
// with few tokens; lists that go through the tiles of all of them do so once.  Where the rounds are full anyway (the 8B-sized layers on
// 16384 tokens) launches of their own are as fast, so the lists have to be ahead by 3 % in what the tiles should take.  Both signs of
// the seven 4B-sized layers, us, launches of their own and lists: on 3001 tokens 1055 (with those that 128 x 128 tiles took) and 868, on
// 4096 1423 and 1137, on 14080 4537 and 3960, 8B-sized on 15028 8226 and 7944
hipError_t launch_gemm_bf16_aligned_lists(const GemmParams* const* a, const bool* sub, int n, const GemmBeside* beside, double* us, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    int slots = 0;
    hipError_t e = list_slots(&slots);
    if (e != hipSuccess) return e;
    if (us) *us = 0.0;
    AlignedItem items[kBatchMax];
    double total = 0.0, deepest = 0.0;
    for (int i = 0; i < n; ++i) {
        if (!gemm_bf16_aligned_listed(*a[i])) return hipErrorInvalidValue;
        items[i] = aligned_item(*a[i]);
        items[i].sub = sub[i] ? 1 : 0;
        total += (double)items[i].tiles_m * items[i].tiles_n * tile_us(items[i]);
        deepest = tile_us(items[i]) > deepest ? tile_us(items[i]) : deepest;
    }
    if (beside && slots > 0) slots = slots_beside(*beside, total, deepest, slots);
    for (int ragged = 0; ragged < 2; ++ragged) {
        const AlignedItem* order[kBatchMax];
        const GemmParams* own[kBatchMax];
        int m = 0;
        bool joined = beside != nullptr;
        double alone = 0.0;
        for (int i = 0; i < n; ++i) {
            if ((sub[i] || aligned_ragged(*a[i])) != (ragged != 0)) continue;
            joined = joined || sub[i];
            if (slots > 0) alone += (double)(((int64_t)items[i].tiles_m * items[i].tiles_n + 8 * slots - 1) / (8 * slots)) * tile_us(items[i]);
            own[m] = a[i];
            int at = m++;
            for (; at > 0 && order[at - 1]->K < items[i].K; --at) order[at] = order[at - 1];
            order[at] = &items[i];
        }
        if (m == 0) continue;
        TileLists tb;
        const double span = slots > 0 ? deal_tiles(order, m, slots, tb) : -1.0;
        const bool lists = span >= 0.0 && (joined || span < 0.97 * alone);
        if (us) *us = *us < 0.0 || (joined && !lists) ? -1.0 : *us + (lists ? span : alone);
        if (us) continue;
        if (!lists) {
            if (joined) return hipErrorInvalidValue;
            for (int q = 0; q < m; ++q) {
                e = launch_gemm_bf16_aligned(*own[q], st);
                if (e != hipSuccess) return e;
            }
            continue;
        }
        for (int q = 0; q < m; ++q) tb.a[q] = *order[q];
        e = ragged ? launch_aligned_grid<0, false, 1, true, kBatchMax>(tb, 8u * slots, st) : launch_aligned_grid<0, false, 1, false, kBatchMax>(tb, 8u * slots, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool RAGGED>
static hipError_t launch_aligned(const GemmParams& p, hipStream_t st) {
    if (p.Y != nullptr) {       // stored output, no loss
        if (p.loss_kind != AGZO_LOSS_NONE || p.y_dtype != AGZO_BF16) return hipErrorInvalidValue;
        return launch_aligned_lists<1, false, RAGGED>(p, st);
    }
    if (p.loss_kind == AGZO_LOSS_CE) {
        if (!p.ce_target || !p.ce_ms || !p.ce_tl) return hipErrorInvalidValue;
        return launch_aligned_lists<2, false, RAGGED>(p, st);
    }
    if (p.loss_kind != AGZO_LOSS_MSE) return hipErrorInvalidValue;
    return p.target_dtype != AGZO_BF16 ? launch_aligned_lists<0, true, RAGGED>(p, st) : launch_aligned_lists<0, false, RAGGED>(p, st);
}

hipError_t launch_gemm_bf16_aligned(const GemmParams& p, hipStream_t st) {
    if (!aligned_fits(p) || p.shared) return hipErrorInvalidValue;
    return aligned_ragged(p) ? launch_aligned<true>(p, st) : launch_aligned<false>(p, st);
}

template <bool T_F32, bool RAGGED>
static hipError_t launch_shared(const KBatch<AlignedItem>& tb, unsigned blocks, hipStream_t st) {
    if (tb.n == 1) return launch_aligned_grid<0, T_F32, 3, RAGGED, 1>(kbatch_one(tb), blocks, st);
    return launch_aligned_grid<0, T_F32, 3, RAGGED, kBatchMax>(tb, blocks, st);
}

hipError_t launch_gemm_bf16_aligned_shared(const GemmParams* const* a, int n, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    int order[kBatchMax];
    for (int i = 0; i < n; ++i) {
        const GemmParams& p = *a[i];
        if (!aligned_fits(p) || !p.shared || p.Y || p.loss_kind != AGZO_LOSS_MSE || !p.Wext2) return hipErrorInvalidValue;
        int at = i;
        for (; at > 0 && a[order[at - 1]]->K < p.K; --at) order[at] = order[at - 1];
        order[at] = i;
    }
    for (int kind = 0; kind < 4; ++kind) {
        const bool f32 = kind & 1, ragged = kind & 2;
        KBatch<AlignedItem> tb;
        tb.n = 0;
        uint64_t blocks = 0;
        for (int i = 0; i < n; ++i) {
            const GemmParams& p = *a[order[i]];
            if ((p.target_dtype != AGZO_BF16) != f32 || aligned_ragged(p) != ragged) continue;
            // (a multiple of 8: workgroups of every problem start at the first XCD; those without a tile leave at once)
            tb.first[tb.n] = (uint32_t)blocks;
            tb.gx[tb.n] = (uint32_t)(((int64_t)p.tiles_m * p.tiles_n + 7) / 8 * 8);
            blocks += tb.gx[tb.n];
            tb.a[tb.n++] = aligned_item(p);
        }
        if (tb.n == 0) continue;
        if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
        const unsigned g = (unsigned)blocks;
        const hipError_t e = ragged ? (f32 ? launch_shared<true, true>(tb, g, st) : launch_shared<false, true>(tb, g, st))
                                    : (f32 ? launch_shared<true, false>(tb, g, st) : launch_shared<false, false>(tb, g, st));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace agzo
