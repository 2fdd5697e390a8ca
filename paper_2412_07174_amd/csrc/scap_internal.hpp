// Host-side internals of libscap: workspace layout, kernel argument blocks, launcher prototypes.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/scap.h"

namespace scap {

// dtype codes, numerically equal to scap_dtype
constexpr int kF16 = SCAP_F16;
constexpr int kBF16 = SCAP_BF16;
constexpr int kI8 = SCAP_I8_COLSCALE;

// GEMV input modes
constexpr int kModeSparse = 0;  // d = x - m, keep = |d| > tau        (Alg. 3)
constexpr int kModeDense = 1;   // d = x, every channel kept          (Eq. 1)
constexpr int kModeFold = 2;    // d = m for every channel            (Eq. 6, eta * column sums)

// ---------------------------------------------------------------------------------------------
// Workspace layout (byte offsets into the caller's buffer)
//   [0, +8)              calibration: the two statistics selected on the GPU
//   [65536, +32768)      int32 seg_cnt[17][256]  kept-channel counts per (token | union, K split)
//   [131072, +1 MiB)     int32 counter per column tile, one every 1 KiB so that the arrival tickets of
//                        different tiles go to different memory channels; zero at rest
//   [1179648, +2 MiB)    one-token kernel, fixed-point hand-over: uint64 acc[131072] (per output column: arrival
//                        count, escape count and the biased fixed-point sum of the arrivals' partial sums), then
//                        uint64 esc[131072] (which splits handed their partial over as fp32 instead); zero at rest
//   [3276800, +4*B*cap)  float partial[B][S][T][tile]   split-K partial sums; calibration: the count of every
//                        16-bit code in the first 512 KiB, uint64 -- or, for less than 2^32 values with m = 0 or
//                        the median, uint32 and behind them one bit per group of 64 codes that occur (32 words)
//   [.., +68*(K+16384))  batched path (B >= 2): union list of every list segment (64 bytes of A operands and
//                        the channel index per entry)
// ---------------------------------------------------------------------------------------------
constexpr size_t kOffSelected = 0;
constexpr size_t kOffSegCnt = 65536;
constexpr size_t kOffCounters = 131072;
constexpr int kCounterStride = 256;  // int32 words between the counters of neighbouring tiles
constexpr size_t kOffFx = kOffCounters + 1024 * (size_t)kCounterStride * 4;
constexpr int kFxCols = 131072;  // output columns the fixed-point hand-over covers (wider layers use partial sums)
constexpr size_t kOffPartial = kOffFx + (size_t)kFxCols * 16;
constexpr size_t kOffCodeHist = kOffPartial;
constexpr size_t kCalibBytes = kOffCodeHist + 65536 * 8;  // workspace bytes calibration needs
constexpr int kMaxTiles = 1024;
constexpr int kMaxSplits = 256;
constexpr int kHistBins = 2048;

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// columns rounded up to whole 1024-column blocks (covers the 512- and 1024-column tiles)
// entries of union-list storage for a K-channel layer: every split may round up to a multiple of 64
inline size_t union_list_entries(int64_t K) { return (size_t)K + 64 * 256; }

inline size_t padded_cols(int64_t N) { return align_up((size_t)N, 1024); }

// floats of split-K partial storage per token
inline size_t partial_capacity(int64_t N) {
    const size_t np = padded_cols(N);
    const size_t cap = np * 16;
    return cap > ((size_t)1 << 20) ? cap : ((size_t)1 << 20);
}

struct GemvArgs {
    const void* W;
    const uint16_t* col_scale;
    const uint16_t* x;
    const float* bias;
    float* y;
    int32_t* idx_out;
    int32_t* nnz_out;
    int32_t* union_nnz_out;
    int32_t* counters;
    int32_t* seg_cnt;
    unsigned long long* fx_acc;  // fixed-point hand-over words [kFxCols], then the escape masks [kFxCols]; or NULL
    float* partial;
    int32_t* u_idx;  // batched path: union list of each segment, [Sl][Kl] channel indices
    float* u_d;      // batched path: the union list's centred values as MFMA A operands: per 16 entries 64 lanes x
                     // (4 bf16 heads, 4 bf16 tails) = 1 KB, i.e. 64 bytes per entry
    int K, N, B, Kc, S, T, mode, xdt;
    int Kl, Sl;  // segmentation of the kept-channel lists: Sl segments of Kl channels (= S, Kc unless batched)
    float m, tau;
    // Fused SwiGLU block (Alg. 2).  The gate|up launch leaves the gated product z, centred and thresholded,
    // as one compacted list per 64 channels; the down launch takes those lists as its input.
    float m2, tau2;   // mode estimate and threshold of the gated product
    float* z_out;     // optional fp32 [B][F]: the gated product itself
    // More than one token: 64-channel segments -- except between the two launches of a two-token block over int8 weights in
    // 8-byte lanes: ceil(F/32) segments of 32 channels.  (One token: see Gemv1Args.)
    int32_t* zl_idx;  // [ceil(F/64)][64] channels of each segment kept by any token, ascending; [ceil(F/32)][32]
    float* zl_d;      // [ceil(F/64)][64][BT] their centred values per token (BT = 2 or 4 slots); [ceil(F/32)][32][2]
    int32_t* zl_cnt;  // [1 + BT][ceil(F/64)] entries per segment: union first, then per token; [ceil(F/32)]: the three
                      // counts in the low bytes of one word, union lowest
    int F;            // channels of the gated product (half the columns of the gate|up launch)
    // Batches of 5 and more, int8 blocks of 3-4 on the row steps (gate_to_planes): zl_d is the plane of operand heads, [BT][F rounded up to 64] 16-bit values, this
    // the plane of tails.
    uint16_t* zl_lo;
    // kernel over row steps (scap_gemm_rows.hip): the magnitude codes [keep_lo, keep_lo + keep_len) are kept; elements between the
    // tokens' rows of x
    uint32_t keep_lo, keep_len;
    int x_pitch;
};

// Enqueue one GEMV (sparse / dense / fold mode).  Returns a scap_status.
int launch_gemv(const GemvArgs& a, int wdt, const scap_launch_cfg* cfg, hipStream_t stream);

// One token (B == 1) through the one-token kernel.  Returns a scap_status, or kG1NotApplicable (positive) when a
// workgroup would own more channels than that kernel tests per wavefront: the caller takes launch_gemv's kernel.
constexpr int kG1NotApplicable = 1;
int launch_gemv1(const GemvArgs& a, int wdt, const scap_launch_cfg* cfg, hipStream_t stream);
// Two to four tokens through that kernel's two- to four-slot forms; kG1NotApplicable likewise (also for another token count,
// bias folding, and three or four tokens that it cannot hand over in fixed point).
int launch_gemv1b(const GemvArgs& a, int wdt, int flags, hipStream_t stream);
// Block of 2-4 tokens: whether launch `part` (0: gate|up with the gating epilogue, two tokens over int8 weights; 1: down reading
// the lists, two tokens, or up to four over 16-bit weights) can run on the two- or four-slot kernel, and that launch.  Both use
// the batched block kernels' list format, so the parts mix with theirs.
bool swiglu_block2_part_applies(const GemvArgs& up, const GemvArgs& down, int wdt, int part);
int launch_swiglu_block2_part(const GemvArgs& up, const GemvArgs& down, int wdt, int part, hipStream_t stream);
// Block of two tokens (int8 weights) with both launches on that kernel, in a list format of their own; kG1NotApplicable likewise,
// and where the format above is the faster one.
int launch_swiglu_block2_pair(const GemvArgs& up, const GemvArgs& down, int wdt, int flags, hipStream_t stream);
// The fused block of one token on the one-token kernel (two launches); kG1NotApplicable likewise.
int launch_swiglu_block1(const GemvArgs& up, const GemvArgs& down, int wdt, int up_flags, int down_flags,
                         hipStream_t stream);

// Fused SwiGLU block: two launches (gate|up with the gating epilogue, then down reading the lists).
// `up` and `down` carry the two layers' arguments; the list pointers and m2/tau2 are set in both.
constexpr int kBlockVectorTokens = 4;  // tokens per fused-block call on the vector kernel (any weight dtype)
constexpr int kBlockMaxTokens = 16;    // ... on the matrix cores (bf16 and int8 weights)
// token slots of the block's lists for B tokens
inline int block_token_slots(int64_t B) { return B <= 1 ? 1 : (B == 2 ? 2 : (B <= 4 ? 4 : 16)); }
int launch_swiglu_block(const GemvArgs& up, const GemvArgs& down, int wdt, hipStream_t stream, int flags1 = 0);

// Interleave two [rows, F] arrays of `elem_bytes`-byte elements in groups of 4 columns: out[rows, 2F].
int launch_pack_gate_up(const void* gate, const void* up, int64_t rows, int64_t F, int elem_bytes, void* out,
                        hipStream_t stream);

// Batched tokens over bf16 or int8 weights on the matrix cores: possible from kMfmaMinTokens tokens on (the
// workspace then carries the union lists of the two-launch form), chosen by default -- beside launch_gemv's rule for 3-4 tokens whose
// centred input is the operand itself -- from kMfmaAutoTokens
// (bf16) / kMfmaAutoTokensI8 (int8) tokens on, where launch_gemv's rules for 2-4 tokens have not chosen a kernel before.
// From 5 tokens on the vector kernel takes two launches' worth of FMAs (vector / matrix cores at 50 %, us: bf16 14336 x
// 4096, 5 tokens 44.3 / 28.0, 4096 x 14336, 8 tokens 46.3 / 29.2; fp16 4096 x 11008, 5 tokens 34.5 / 22.3); at 4 tokens
// over 16-bit weights it does not (14336 x 4096 29.8 / 27.4, 4096 x 14336 27.3 / 28.0, the four-slot kernel 25.8 and
// 25.7).  With int8 weights it is bound by its per-element converts from 3 tokens on (4096 x 28672 35.6 / 30.1; two 23.5 /
// 28.2).
constexpr int kMfmaMinTokens = 2;
constexpr int kMfmaAutoTokens = 5;
constexpr int kMfmaAutoTokensI8 = 3;
int launch_gemm_mfma(const GemvArgs& a, int wdt, const scap_launch_cfg* cfg, hipStream_t stream);
// The same in one launch: each workgroup compacts its own inputs into LDS (up to 160 KB on gfx950).
// SCAP_ERR_SHAPE when the input is too long to split into LDS-sized pieces.
int launch_gemm_inline(const GemvArgs& a, int wdt, const scap_launch_cfg* cfg, hipStream_t stream, bool slots16 = false);
// The same without lists or staged inputs, 16 token slots (scap_gemm_rows.hip).  src says what the inputs are; exact_operand: the centred input is
// the 16-bit operand itself (m = 0 or dense mode, activations of the operand's type).  kc: rows per workgroup, or 0.  SCAP_ERR_SHAPE where it cannot
// split the layer (kRowsCentre: where it has more column tiles than there are compute units).
constexpr int kRowsCodes = 0;   // x: 16-bit inputs that are the operand
constexpr int kRowsPlanes = 1;  // x, zl_lo: heads and tails
constexpr int kRowsCentre = 2;  // x: 16-bit inputs of any type, centred in fp32 and split
bool exact_operand(const GemvArgs& a, int wdt);
// Whether a plain call of three or more tokens, or the gate|up launch of a block of 2-4, is the faster one on that kernel.
bool rows_pay(const GemvArgs& a, int wdt);
bool rows_pay_gating(const GemvArgs& a, int wdt);
bool gemm_rows_plans(const GemvArgs& a, int wdt, int src, int fuse, int* splits = nullptr);
int launch_gemm_rows(const GemvArgs& a, int wdt, int src, int fuse, int kc, hipStream_t stream);
// The fused block's two launches on the matrix cores: row steps (more than 4 tokens, int8 from 3 where rows_pay_gating; a gate|up launch that
// they cannot split on the staged tile), else the value lists of 4 token slots.
int launch_swiglu_block_inline(const GemvArgs& up, const GemvArgs& down, int wdt, hipStream_t stream);

// Fill `n` int32 words with zero using a kernel (safe to record into a HIP graph).
int launch_zero_words(int32_t* p, size_t n, hipStream_t stream);

// Zero the fixed header of a workspace (arrival counters, calibration scratch, segment counts).
int launch_workspace_init(void* workspace, size_t bytes, hipStream_t stream);

int launch_read_probe(const void* src, size_t bytes, uint32_t* out, hipStream_t stream);

// Calibration (synchronous; returns a scap_status).
int run_calibrate(const uint16_t* X, int64_t M, int xdt, float s, int est, float* m_out, float* tau_out,
                  void* workspace, hipStream_t stream);

}  // namespace scap
