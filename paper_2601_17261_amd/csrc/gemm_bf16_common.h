// Shared between the kernels of the bf16 forward GEMM: launch parameters and the LDS tile layout.  256 x 256 tiles for shapes that
// fill the chip with them (gemm_bf16_aligned.hip; gemm_bf16.hip for what that one has no output form for or does not fit into a layer),
// 128 x 128 tiles for the others (gemm_bf16_mid.hip; gemm_bf16_small.hip likewise), 64 x 64 ones for stored outputs of few of these (gemm_bf16_few.hip).
#pragma once
#include "agzo_internal.h"

namespace agzo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
template <int V> struct IC { static constexpr int value = V; };

constexpr int BT = 256;                        // tile edge (tokens and outputs)
constexpr int BK = 64;
constexpr int CHUNKS = BK / 8;                 // 16-byte chunks per tile row
constexpr int TILE_BYTES = BT * BK * 2;        // one operand tile: 32 KiB

// byte offset of 16-byte chunk `c` of row `row` inside a [256][64] bf16 tile; the XOR spreads the
// 16 rows touched by one pass of a ds_read_b128 over all LDS banks.
__device__ __forceinline__ int lds_off(int row, int c) { return row * (BK * 2) + ((c ^ ((row >> 1) & 7)) << 4); }

// LDS row m' of a 32-row block holds W row perm(m'): MFMA output register e of lane half h is
// row 8*(e/4) + 4*h + e%4 of the block, which this makes output column 16*h + e.
__device__ __forceinline__ int w_perm(int m) { return ((m >> 2) & 1) * 16 + ((m >> 3) & 3) * 4 + (m & 3); }

// 16 bytes at any 2-byte aligned address, one instruction each (global memory takes unaligned vectors; rows of an odd number
// of outputs make them so)
struct __attribute__((packed, aligned(2))) Any16 { uint32_t x, y, z, w; };
__device__ __forceinline__ uint4 load16_any(const void* src) {
    const Any16 v = *reinterpret_cast<const Any16*>(src);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store16_any(void* dst, uint4 v) {
    *reinterpret_cast<Any16*>(dst) = Any16{v.x, v.y, v.z, v.w};
}

// Direct loads of a last slice that d_in does not fill: lanes whose chunk lies past d_in add this to their offset, which the
// range of the slice's descriptor (below) turns into zeros.  Offsets inside a tile stay below it: 256 rows of 2^22 elements
constexpr int kPastEnd = (int)0x80000000u;

struct GemmParams {
    const bf16_t* X; int64_t ldx;
    const bf16_t* W; int64_t ldw;
    int64_t M, N, K;            // tokens, outputs, d_in
    void* Y; int y_dtype; int64_t ldy;
    const float* P; int r; int rp;
    // rank-r extension operands prepared ahead of the launch (NULL: the workgroups build them per tile):
    // Xext [M][ext_ld] = [Ph | Ph | Pl | 0], Wext [N][ext_ld] = [Gh | Gl | Gh | 0] with the signed eps folded into G
    // Wext2: the W side once more with -2 eps folded in (second pass of the shared-forward squared-error kernel)
    const bf16_t* Xext; const bf16_t* Wext; const bf16_t* Wext2; int ext_ld;
    float eps_signed; uint32_t s_lo, s_hi;
    int loss_kind; int target_dtype; const void* target; int64_t ldt; double* partials;
    int tiles_m, tiles_n;
    int group_m;                // token tiles walked per output tile inside an XCD's run
    int vec_ok;                 // 16-byte epilogue accesses are legal
    int shared;                 // one pass evaluates f0, f+ and f- (three loss partials per tile)
    // cross-entropy: per (128-column chunk, token) running max and sum of exponentials, and the target's logit
    const int32_t* ce_target; float2* ce_ms; float* ce_tl;
    // fused range sketch (128 x 128 tiling, or 64 x 64; NULL: none): Omega^T planes [3][16][sk_mpad] (sk_mpad a multiple of
    // 128 that covers every token tile, zero past the last token) and the partial sums of every sk_tokens tokens, a tile's edge, [tiles_m][K][16]
    const bf16_t* sk_T; int64_t sk_mpad; float* sk_partial; int sk_tokens;
    // optional telemetry: workgroup 0 leaves {shader clock, constant-rate clock} at entry and at exit
    unsigned long long* clk;
    int slots;                  // workgroups per XCD of the persistent kernel at most (0: one to a compute unit)
};


// small-tile variant (gemm_bf16_small.hip): plain or perturbed forward with optional Y store and squared-error loss;
// partials [tiles128_m * tiles128_n]
constexpr int BT_SMALL = 128;
hipError_t launch_gemm_bf16_small(const GemmParams& p, hipStream_t st);

// one forward of a launch that takes several (gemm_bf16_mid.hip)
struct GemmItem {
    const bf16_t* X; const bf16_t* W;
    int64_t ldx, ldw, M, N, K;
    const bf16_t* Xext; const bf16_t* Wext; int ext_ld;   // prepared rank-r extension operands (NULL: none)
    const void* target; int64_t ldt; double* partials;    // squared error: [ceil(M / 128) * ceil(N / 128)] partial sums
    int wide;                                              // (squares in fp64 everywhere)
    void* Y; int64_t ldy;                                  // stored bf16 output
    int tiles_m, tiles_n;                                  // (set by the launch)
    // fused range sketch (a launch of one problem; NULL: none): as in GemmParams
    const bf16_t* sk_T; int64_t sk_mpad; float* sk_partial; int sk_tokens;
    unsigned long long* clk;
    // out 1 in a launch of one problem: so many shares of the slices, their sums in part (gemm_bf16_split_bytes(); NULL: one share)
    int splits; float* part;
};
int gemm_bf16_mid_splits(int64_t M, int64_t N, int64_t K);
// out 0: squared error (target_f32: of fp32 targets), 1: stored bf16 output (one problem a launch)
bool gemm_bf16_mid_ok(const GemmItem& g, int out);
// half_cu (out 0): at most one workgroup to a compute unit, and 72 KiB of its LDS left
hipError_t launch_gemm_bf16_mid(const GemmItem* a, int n, int out, bool target_f32, bool half_cu, hipStream_t st);

// 64 x 64 tiles whose waves share d_in, for the stored outputs of few tiles (gemm_bf16_few.hip).  Sums over d_in in kFewShares shares,
// slices nd i / kFewShares to nd (i + 1) / kFewShares, which are added in pairs
constexpr int kFewShares = 4;
bool gemm_bf16_few_shape(int64_t M, int64_t N, int64_t K);
hipError_t launch_gemm_bf16_few(const GemmItem& a, hipStream_t st);

// persistent kernel in 256 x 256 tiles (gemm_bf16_aligned.hip): M, N >= 256, d_in >= 128, the rank-r term as prepared operands;
// either the squared-error loss without a stored Y, the cross-entropy statistics without a stored Y, or a bf16 Y without a loss
hipError_t launch_gemm_bf16_aligned(const GemmParams& p, hipStream_t st);
// p.slots for that launch beside other work, or 0 where it is done sooner one after the other
int gemm_bf16_aligned_slots(const GemmParams& p, const GemmBeside& beside);
// squared errors of several layers (gemm_bf16_aligned_listed()) over tile lists that go through all of them.  sub[i]: the loss
// partials of gemm_bf16_mid.hip, bit for bit (a layer that takes its 128 x 128 tiles when alone).  beside != NULL: in lists in any case, on
// as many compute units as the work beside them leaves.  us != NULL: nothing is launched, *us is about what it would take, below 0
// where the lists do not take the layers
bool gemm_bf16_aligned_listed(const GemmParams& p);
hipError_t launch_gemm_bf16_aligned_lists(const GemmParams* const* a, const bool* sub, int n, const GemmBeside* beside, double* us, hipStream_t st);
// squared error with p.shared (f0, f+, f- in one pass, needs Wext2, partials [3][tiles]): up to kBatchMax layers together
hipError_t launch_gemm_bf16_aligned_shared(const GemmParams* const* a, int n, hipStream_t st);

}  // namespace agzo
