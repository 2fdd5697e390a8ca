// Launch of the one-token GEMV kernel (scap_gemv1.hpp): K split, argument block, dispatch by weight type.
#include "scap_gemv1b.hpp"

namespace scap {

extern template int launch_gemv1_wdt<kF16>(const Gemv1Args&, int, int, hipStream_t);
extern template int launch_gemv1_wdt<kBF16>(const Gemv1Args&, int, int, hipStream_t);
extern template int launch_gemv1_wdt<kI8>(const Gemv1Args&, int, int, hipStream_t);
extern template int launch_gemv1_wdt<kI8Half>(const Gemv1Args&, int, int, hipStream_t);
extern template int launch_gemv1b_wdt<kF16>(const Gemv1bArgs&, hipStream_t);
extern template int launch_gemv1b_wdt<kBF16>(const Gemv1bArgs&, hipStream_t);
extern template int launch_gemv1b_wdt<kI8>(const Gemv1bArgs&, hipStream_t);
extern template int launch_gemv1b_wdt<kI8Half>(const Gemv1bArgs&, hipStream_t);
extern template int launch_gemv1b_block_wdt<kF16>(const Gemv1bArgs&, int, hipStream_t);
extern template int launch_gemv1b_block_wdt<kBF16>(const Gemv1bArgs&, int, hipStream_t);
extern template int launch_gemv1b_block_wdt<kI8>(const Gemv1bArgs&, int, hipStream_t);
extern template int launch_gemv1b_block_wdt<kI8Half>(const Gemv1bArgs&, int, hipStream_t);
#define SCAP_G1_BLOCK_EXTERN(WD)                                                             \
    extern template int launch_gemv1_block<WD, kFuseSwiglu>(const Gemv1Args&, hipStream_t); \
    extern template int launch_gemv1_block<WD, kFuseList>(const Gemv1Args&, hipStream_t);
SCAP_G1_BLOCK_EXTERN(kF16)
SCAP_G1_BLOCK_EXTERN(kBF16)
SCAP_G1_BLOCK_EXTERN(kI8)
SCAP_G1_BLOCK_EXTERN(kI8Half)
#undef SCAP_G1_BLOCK_EXTERN

// One token through a K x N layer (sparse, dense or bias-folding mode).  Returns a scap_status, or
// kG1NotApplicable when the shape needs more than 2048 channels per workgroup (the caller then takes the
// general kernel).  cfg: rows_per_group and unroll are honoured, flags bit 0 forces device-scope loads.
namespace {

struct Plan1 {
    bool i8_half;
    int elems, tile, Kc, S, T;
};

// int8 weights: 8 bytes per lane (512-column tiles) up to kI8HalfCols columns -- twice the tiles, so half the K splits
// and half the sums per wavefront to add at the end --, 16 beyond, where there are tiles enough.  16-byte / 8-byte
// lanes at 50 %, us: 4096 x 11008 one token 9.9 / 8.9, two 14.0 / 11.9; 1024 x 8192 7.0 / 5.8 and 10.0 / 7.8;
// 4096 x 16384 11.5 / 10.4 and 16.5 / 14.4; 4096 x 28672 14.7 / 15.2 and 21.4 / 22.3.
constexpr int kI8HalfCols = 16384;
constexpr int kI8WideCols = 4096;
// Three and four slots over int8 weights spend one FMA per weight and token beside the widening; the staged tile on the matrix
// cores is the faster one for four tokens and for small layers, this kernel for three tokens over large ones (50 / 90 %, here /
// staged tile, us: 4 tokens 14336 x 4096 20.6 / 18.5 and 13.8 / 12.4, 4096 x 11008 18.7 / 16.2 and 12.8 / 10.9, 8192 x 8192
// 21.9 / 20.0 and 14.6 / 13.1, 4096 x 4096 13.7 / 9.6 and 11.2 / 7.7; 3 tokens 14336 x 4096 16.7 / 17.3 and 11.4 / 11.6,
// 4096 x 11008 15.0 / 15.7 and 10.6 / 10.4, 8192 x 8192 18.3 / 19.3 and 11.5 / 12.0, 4096 x 4096 11.4 / 9.3 and 9.1 / 7.5).  Up to
// this many weights, and up to kI8WideCols columns, calls run here all the same: x - m is an fp32 operand here and two bf16
// halves there (error with m != 0 about 1.8e-6 instead of 1.3e-7).
constexpr int64_t kI8FourSlotWeights = (int64_t)1 << 26;

// K split of one launch with the given lane width and split cost; SCAP_OK, kG1NotApplicable (also for more channels per
// workgroup than the kernel tests) or a scap_status.
int plan_gemv1_lanes(const GemvArgs& g, int wdt, int kc, bool kc_forced, int waves, int granule_min, int bt, bool i8_half,
                     bool split_cost, Plan1* out) {
    out->i8_half = i8_half;
    out->elems = wdt == kI8 && !out->i8_half ? 16 : 8;
    out->tile = kWave * out->elems;
    GemvArgs p = g;
    // LDS: header, the wavefronts' sums, then 8 bytes per listed channel (16 with 2 token slots)
    const int entry = bt == 1 ? 8 : g1b_entry_bytes(bt);
    const int64_t fixed_lds = bt == 1 ? (int64_t)waves * out->tile * 4 + 64 + kG1HdrBytes
                                      : (int64_t)bt * kG1HdrBytes + (int64_t)kG1bWaves * bt * out->tile * 4 + (int64_t)kG1bWaves * 4 * entry;
    const int64_t lds_max = bt == 1 ? 64 * 1024 : kG1bMaxLds;
    // (four slots of 1024-column tiles: the wavefronts' sums alone would fill LDS)
    if (fixed_lds + (int64_t)kWave * (4 + entry) > lds_max) return kG1NotApplicable;
    size_t lds_budget = (size_t)(lds_max - fixed_lds) + kHdrBytes;
    // Three slots have room for more channels than the kernel tests: shorter pieces in two rounds rather than another kernel (3
    // tokens at 60 %, us, staged tile or general kernel / here: 62240 x 4592 bf16 122.1 / 92.1, fp16 93.7 / 92.7, 40000 x 8192 bf16
    // 103 / 92.2), as four slots do.
    if (bt == 3) lds_budget = std::min(lds_budget, (size_t)kHdrBytes + (size_t)kG1MaxChunks * kG1Chunk * entry);
    // Rows per workgroup in multiples of 64, unless the input is so short that 64-row pieces would leave compute
    // units without a workgroup (finer pieces elsewhere gained and lost 2 % by turns)
    p.T = (p.N + out->tile - 1) / out->tile;
    int granule = ((int64_t)((p.K + kWave - 1) / kWave) * p.T < 256) ? 8 : kWave;
    if (granule < granule_min) granule = granule_min;
    // A split costs 2 rows' time and one more per 4096 columns: its atomics queue up on the columns' words.  Fitted to
    // sweeps of kc over 100 (shape, type, token count) points with kc from 16 to 1408; without it narrow layers
    // were cut into pieces of 8-32 rows (us, before / now: 1024 x 1024 bf16 8.8 / 4.6, 4096 x 1024 9.4 / 5.7, 2 tokens
    // 12.3 / 5.9 and 13.4 / 7.0).  Beyond 64 splits partial sums are handed over instead, about 4 us more.
    SplitCost sc;
    if (split_cost) {
        sc.rows = 2 + (p.N + 2048) / 4096;
        sc.soft_max = kFxMaxSplits;
        sc.beyond_rows = 512;
    }
    const int rc = plan_splits(p, out->tile, entry / 4 - 1, kc, kc_forced, lds_budget, granule, sc);
    if (rc != SCAP_OK) return rc == SCAP_ERR_SHAPE ? kG1NotApplicable : rc;
    if (p.Kc > kG1MaxChunks * kG1Chunk) return kG1NotApplicable;
    out->Kc = p.Kc;
    out->S = p.S;
    out->T = p.T;
    return SCAP_OK;
}

// K split and lane width of one launch.  SCAP_OK, kG1NotApplicable or a scap_status.
// bt = token slots: 1 (one-token kernel), 2, 3 or 4 (its multi-token forms, 8 wavefronts).
// wide_lanes: int8 weights in 16-byte lanes wherever there are more than 4 tiles of them
// must: no other kernel does what the call asks for (y += result)
// lanes8: int8 weights in 8-byte lanes whatever the columns, in the second plan too
int plan_gemv1(const GemvArgs& g, int wdt, int kc, bool kc_forced, int waves, int granule_min, int bt, Plan1* out,
               bool wide_lanes = false, bool must = false, bool lanes8 = false) {
    const bool half = lanes8 || (wdt == kI8 && g.N <= (wide_lanes ? kI8WideCols : kI8HalfCols));
    const int rc = plan_gemv1_lanes(g, wdt, kc, kc_forced, waves, granule_min, bt, half, true, out);
    if (rc != kG1NotApplicable) return rc;
    // Long inputs and very wide layers for which fewer, longer pieces than the kernel tests look best: the split that fills
    // the compute units alone, in wide lanes, if there is one.  It is worth taking with one workgroup per unit and the
    // fixed-point hand-over (us, general kernel / here, one and two tokens at 50 %: 62238 x 4592 int8 39.9 / 37.3 and 54.2 /
    // 51.6, 22968 x 11200 int8 33.8 / 32.4 and 45.9 / 44.2), not otherwise (132456 x 1040 int8, 83 splits, 29.2 / 30.9 and 39.2 /
    // 42.6; 98580 x 9328 int8, 500 workgroups, 94.2 / 96.1 and 135.5 / 138.9).
    const int rc2 = plan_gemv1_lanes(g, wdt, kc, kc_forced, waves, granule_min, bt, lanes8 || (wdt == kI8 && g.N <= kI8WideCols), false, out);
    if (rc2 != SCAP_OK || must) return rc2;
    return out->S <= kFxMaxSplits && (int64_t)out->S * out->T <= 256 ? SCAP_OK : kG1NotApplicable;
}

Gemv1Args args_of(const GemvArgs& g, const Plan1& pl, int wdt, int flags) {
    Gemv1Args a{};
    a.W = g.W;
    a.x = g.x;
    a.col_scale = g.col_scale;
    a.bias = g.bias;
    a.y = g.y;
    a.partial = g.partial;
    a.counters = g.counters;
    a.idx_out = g.idx_out;
    a.nnz_out = g.nnz_out;
    a.union_nnz_out = g.union_nnz_out;
    a.seg_cnt = g.seg_cnt;
    a.K = g.K;
    a.N = g.N;
    a.Kc = pl.Kc;
    a.S = pl.S;
    a.T = pl.T;
    a.mode = g.mode;
    a.xdt = g.xdt;
    // (turned_start) eight or more pieces that lie a power of two apart: from 4 MiB, long ones from 2 MiB.  Shorter pieces closer by lose as
    // much as they gain (dense, us, without / with: 8192 x 4096 bf16, 256 rows 2 MiB apart, 14.8 / 15.1, 8192 x 2048, 128 rows 0.5 MiB apart,
    // 9.7 / 10.5, but 16384 x 4096 int8, 512 rows 2 MiB apart, 16.1 / 15.0; 4096 x 8192 bf16, 256 rows 4 MiB apart, 15.8 / 14.5).
    const int64_t apart = (int64_t)pl.Kc * g.N * (wdt == kI8 ? 1 : 2), mib = (int64_t)1 << 20;
    const bool turn = pl.S >= 8 && (apart & (apart - 1)) == 0 && (apart >= 4 * mib || (apart >= 2 * mib && pl.Kc >= 512));
    a.flags = flags | (turn ? kG1FlagTurn : 0);
    a.m = g.m;
    a.tau = g.tau;
    // fixed-point hand-over unless the caller asks for partial sums (either flag), the layer is wider than the
    // words provided or a column has more arrivals than a word counts
    const bool fx = !(flags & (kG1FlagPartials | kG1FlagDeviceScope)) && g.N <= kFxCols && pl.S <= kFxMaxSplits;
    a.fx_acc = fx ? g.fx_acc : nullptr;
    return a;
}

}  // namespace

// One token (B == 1) through a K x N layer (sparse, dense or bias-folding mode).  Returns a scap_status, or
// kG1NotApplicable when the shape needs more than 2048 channels per workgroup (the caller then takes the
// general kernel).  cfg: wavefronts (4, 8), rows_per_group and unroll are honoured, flags bit 0 forces device-scope loads.
int launch_gemv1(const GemvArgs& g, int wdt, const scap_launch_cfg* cfg, hipStream_t stream) {
    if (g.B != 1) return kG1NotApplicable;
    int kc = 0, unroll = 0, flags = 0, waves = 8;
    if (cfg) {
        if (cfg->rows_per_group) kc = cfg->rows_per_group;
        if (cfg->unroll) unroll = cfg->unroll;
        if (cfg->waves_per_group) waves = cfg->waves_per_group;
        flags = cfg->flags;
        if (kc < 0 || (kc % 8) != 0) return SCAP_ERR_CONFIG;  // whole octets of channels per workgroup
        if (kc > kG1MaxChunks * kG1Chunk) return kG1NotApplicable;
    }
    Plan1 pl;
    const int rc = plan_gemv1(g, wdt, kc, cfg && cfg->rows_per_group, waves, 8, 1, &pl, false, (flags & kG1FlagAccumulate) != 0);
    if (rc != SCAP_OK) return rc;
    // rows in flight per wavefront: 4 x 1 KB (16-byte lanes), 8 x 512 bytes (8-byte lanes)
    if (unroll == 0) unroll = pl.i8_half ? 8 : 4;
    const Gemv1Args a = args_of(g, pl, wdt, flags);
    switch (wdt) {
        case kF16: return launch_gemv1_wdt<kF16>(a, waves, unroll, stream);
        case kBF16: return launch_gemv1_wdt<kBF16>(a, waves, unroll, stream);
        case kI8: return pl.i8_half ? launch_gemv1_wdt<kI8Half>(a, waves, unroll, stream) : launch_gemv1_wdt<kI8>(a, waves, unroll, stream);
    }
    return SCAP_ERR_DTYPE;
}

// Two to four tokens (three and four over int8 weights: in 8-byte lanes only), through the two-, three- or four-slot form of
// the one-token kernel (sparse or dense mode).  Returns a scap_status, or kG1NotApplicable: another token count, bias folding,
// more than 2048 channels per workgroup, or three or four tokens without the fixed-point hand-over.  flags as for launch_gemv1.
int launch_gemv1b(const GemvArgs& g, int wdt, int flags, hipStream_t stream) {
    if (g.B < 2 || g.B > 4 || g.mode == kModeFold) return kG1NotApplicable;

    if (wdt == kI8 && g.B > 2 && g.N > kI8WideCols && (int64_t)g.K * g.N > kI8FourSlotWeights) return kG1NotApplicable;

    Gemv1bArgs b;
    b.B = g.B;
    b.bt = (int)g.B;
    Plan1 pl;
    const int rc = plan_gemv1(g, wdt, 0, false, kG1bWaves, 8, b.bt, &pl);
    if (rc != SCAP_OK) return rc;
    if (wdt == kI8 && b.bt > 2 && !pl.i8_half) return kG1NotApplicable;  // 16-byte lanes: two slots only
    b.a = args_of(g, pl, wdt, flags);
    if ((size_t)g.B * (size_t)g.N > (size_t)kFxCols) b.a.fx_acc = nullptr;  // one fixed-point word per (token, column)
    // with more slots the partial-sum hand-over loses to the other kernels (its last arrivals fetch 4 S slices)
    if (b.bt > 2 && b.a.fx_acc == nullptr) return kG1NotApplicable;
    switch (wdt) {
        case kF16: return launch_gemv1b_wdt<kF16>(b, stream);
        case kBF16: return launch_gemv1b_wdt<kBF16>(b, stream);
        case kI8: return pl.i8_half ? launch_gemv1b_wdt<kI8Half>(b, stream) : launch_gemv1b_wdt<kI8>(b, stream);
    }
    return SCAP_ERR_DTYPE;
}

template <int FUSE>
static int launch_block_half(const Gemv1Args& a, int wdt, bool i8_half, hipStream_t stream) {
    switch (wdt) {
        case kF16: return launch_gemv1_block<kF16, FUSE>(a, stream);
        case kBF16: return launch_gemv1_block<kBF16, FUSE>(a, stream);
        case kI8: return i8_half ? launch_gemv1_block<kI8Half, FUSE>(a, stream) : launch_gemv1_block<kI8, FUSE>(a, stream);
    }
    return SCAP_ERR_DTYPE;
}

// Fused SwiGLU block of one token on the one-token kernel: the gate|up launch with the gating epilogue, then the
// down launch reading the lists.  `up` and `down` as for launch_swiglu_block; up_flags, down_flags: the launches'
// flags (kG1FlagPartials; up: kG1FlagParkSlices; down: kG1FlagAccumulate, y += block output).  kG1NotApplicable when either layer needs more than 2048 channels per
// workgroup.
int launch_swiglu_block1(const GemvArgs& up, const GemvArgs& dn, int wdt, int up_flags, int down_flags, hipStream_t stream) {
    if (up.B != 1) return kG1NotApplicable;
    Plan1 pu, pd;
    const bool must = (down_flags & kG1FlagAccumulate) != 0;
    int rc = plan_gemv1(up, wdt, 0, false, 8, kWave, 1, &pu, false, must);
    if (rc != SCAP_OK) return rc;
    rc = plan_gemv1(dn, wdt, 0, false, 8, kWave, 1, &pd, false, must);  // whole 64-channel pieces: whole list segments
    if (rc != SCAP_OK) return rc;
    const int segz = pu.tile / 8 / 2;  // gated channels a wavefront slice of the gate|up launch finishes: 32 or 64
    if (pd.Kc % segz != 0 || pd.Kc / segz > kWave) return kG1NotApplicable;
    Gemv1Args a = args_of(up, pu, wdt, up_flags);
    Gemv1Args b = args_of(dn, pd, wdt, down_flags);
    for (Gemv1Args* q : {&a, &b}) {
        q->m2 = up.m2;
        q->tau2 = up.tau2;
        q->zl_idx = up.zl_idx;
        q->zl_d = up.zl_d;
        q->zl_cnt = up.zl_cnt;
        q->F = up.F;
        q->segz = segz;
    }
    a.z_out = up.z_out;
    // the gating epilogue parks finished columns behind the partial-sum slots when a slice is finished piecemeal
    if ((size_t)(pu.S + 1) * pu.T * pu.tile > partial_capacity(up.N)) a.fx_acc = nullptr;
    a.idx_out = a.nnz_out = a.union_nnz_out = nullptr;
    b.x = nullptr;
    rc = launch_block_half<kFuseSwiglu>(a, wdt, pu.i8_half, stream);
    if (rc != SCAP_OK) return rc;
    return launch_block_half<kFuseList>(b, wdt, pd.i8_half, stream);
}

// Fused SwiGLU block of two tokens (down launch: up to four) on the multi-slot kernel.
//   part 0, the gate|up launch with the gating epilogue: int8 weights.  It leaves one list segment per wavefront slice:
//           64 channels in 16-byte lanes -- the format of the batched block kernels, so each launch can be paired with the
//           general kernel's other half --, 32 channels with packed counts in 8-byte lanes (lanes8), which only this
//           kernel's down launch reads (launch_swiglu_block2_pair);
//   part 1, the down launch reading the lists: any weights, unless 16-bit and too wide for the fixed-point hand-over
//           (with partial sums handed over the general kernel's down launch measured 0.5 us faster).
// Measured on 4096 -> 14336 -> 4096, two tokens, both launches general / these (us): int8 45.8 / 41.9 with nothing
// pruned, 38.0 / 34.5 at 50 %, 21.8 / 19.6 at 90 %; bf16 (down launch only) 65.3 / 64.3, 55.9 / 54.7, 25.9 / 24.8.
// Fills *g and returns SCAP_OK, or kG1NotApplicable.
// flags: kG1FlagParkSlices (8-byte lanes of part 0; 16-byte lanes hand partial sums over, where every slice is finished at once).
static int plan_block2_part(const GemvArgs& up, const GemvArgs& dn, int wdt, int part, bool lanes8, int flags, Gemv1bArgs* g,
                            bool* i8_half) {
    // 3-4 tokens: the down launch only, 16-bit weights, on the four-slot form (the lists then carry 4 token slots)
    const bool four = (up.B == 3 || up.B == 4) && part == 1 && wdt != kI8;
    if (up.B != 2 && !four) return kG1NotApplicable;
    const GemvArgs& src = part == 0 ? up : dn;
    if (part == 0 && wdt != kI8) return kG1NotApplicable;
    const bool fits_fx = (int64_t)up.B * (int64_t)src.N <= (int64_t)kFxCols;
    if (part == 1 && wdt != kI8 && !fits_fx) return kG1NotApplicable;
    Plan1 pl;
    // the down launch: whole 64-channel pieces, i.e. whole segments
    const int rc = plan_gemv1(src, wdt, 0, false, kG1bWaves, part == 0 && lanes8 ? 8 : kWave, four ? 4 : 2, &pl, part == 0, false, part == 0 && lanes8);
    if (rc != SCAP_OK) return kG1NotApplicable;
    if (part == 1 && four && pl.Kc > 2 * kG1Chunk) return kG1NotApplicable;  // (its prologue holds every entry slot in registers)
    if (part == 1 && (pl.Kc % kWave) != 0) return kG1NotApplicable;
    g->B = (int)up.B;
    g->bt = four ? 4 : 2;
    g->a = args_of(src, pl, wdt, flags);
    if (!fits_fx || (part == 0 && !pl.i8_half)) g->a.fx_acc = nullptr;
    // the gating epilogue parks finished columns behind the partial-sum slots when a slice is finished piecemeal
    if (part == 0 && (size_t)(pl.S + 1) * pl.T * pl.tile > partial_capacity(src.N)) g->a.fx_acc = nullptr;
    if (four && g->a.fx_acc == nullptr) return kG1NotApplicable;
    g->a.m2 = up.m2;
    g->a.tau2 = up.tau2;
    g->a.zl_idx = up.zl_idx;
    g->a.zl_d = up.zl_d;
    g->a.zl_cnt = up.zl_cnt;
    g->a.F = up.F;
    if (part == 0) {
        g->a.z_out = up.z_out;
        g->a.idx_out = g->a.nnz_out = g->a.union_nnz_out = nullptr;
    } else {
        g->a.x = nullptr;
        g->a.z_out = nullptr;
    }
    *i8_half = pl.i8_half;
    return SCAP_OK;
}

static int launch_block2(const Gemv1bArgs& g, int wdt, bool half, int fuse, hipStream_t stream) {
    switch (wdt) {
        case kF16: return launch_gemv1b_block_wdt<kF16>(g, fuse, stream);
        case kBF16: return launch_gemv1b_block_wdt<kBF16>(g, fuse, stream);
        case kI8: return half ? launch_gemv1b_block_wdt<kI8Half>(g, fuse, stream) : launch_gemv1b_block_wdt<kI8>(g, fuse, stream);
    }
    return SCAP_ERR_DTYPE;
}

// One of the launches in the batched block kernels' list format.
static int plan_block2_64(const GemvArgs& up, const GemvArgs& dn, int wdt, int part, Gemv1bArgs* g, bool* half) {
    const int rc = plan_block2_part(up, dn, wdt, part, false, 0, g, half);
    if (rc != SCAP_OK) return rc;
    return part == 0 && *half ? kG1NotApplicable : SCAP_OK;
}

bool swiglu_block2_part_applies(const GemvArgs& up, const GemvArgs& dn, int wdt, int part) {
    Gemv1bArgs g;
    bool half = false;
    return plan_block2_64(up, dn, wdt, part, &g, &half) == SCAP_OK;
}

int launch_swiglu_block2_part(const GemvArgs& up, const GemvArgs& dn, int wdt, int part, hipStream_t stream) {
    Gemv1bArgs g;
    bool half = false;
    const int rc = plan_block2_64(up, dn, wdt, part, &g, &half);
    if (rc != SCAP_OK) return rc;
    return launch_block2(g, wdt, half, part == 0 ? kFuseSwiglu : kFuseList, stream);
}

// Whether the gate|up launch of a two-token block over int8 weights is planned better in 8-byte lanes (`half`) than in 16-byte
// lanes (`wide`).  8-byte lanes save in the fixed part (half the sums of the wavefronts and half the splits, handed over in fixed
// point) and lose in the stream: they read rows in pieces of 512 instead of 1024 bytes.  From 110 blocks K -> F at 2-80 %
// sparsity (us per block, wide / half):
//  - up to 13312 gate|up columns, or pieces of at most 512 rows, half is faster however the tiles fall: 16384 -> 4096 37.3 / 34.6,
//    14976 -> 2688 33.7 / 30.0, 4096 -> 8192 25.6 / 24.0, 2048 -> 16384 26.6 / 24.8, 1064 -> 13848 22.3 / 21.8;
//  - pieces of up to 1024 rows: where the busiest unit reads no more bytes than in the wide plan (4096 -> 12800 34.9 / 33.9, 4096 ->
//    14336 37.1 / 37.0, 6144 -> 24576 76.8 / 76.0), not where a smaller share of the units is busy (4096 -> 11008 at 40 % 32.0 /
//    32.5, 4096 -> 18368 at 30 % 45.9 / 47.1);
//  - longer ones lose: 8192 -> 12288 54.7 / 56.6, 8192 -> 13568 62.1 / 65.1, 4096 -> 28672 60.9 / 61.7, 3584 -> 31680 60.5 / 61.2;
//  - pieces of 1024 rows or more that lie a multiple of 32 MiB apart meet on the same memory channels: half then 36.2 / 38.9 on
//    4096 -> 16384 and 38.6 / 42.3 on 2048 -> 32768.  Where the wide plan's do, half is the faster one (8192 -> 16384 78.4 / 75.0).
static bool half_lanes_are_faster(const Gemv1bArgs& half, const Gemv1bArgs& wide) {
    auto bytes = [](const Gemv1bArgs& g, int tile) { return ((int64_t)g.a.S * g.a.T + 255) / 256 * g.a.Kc * tile; };
    auto meet = [](const Gemv1bArgs& g) { return g.a.Kc >= 1024 && (int64_t)g.a.Kc * g.a.N % ((int64_t)1 << 25) == 0; };
    if (meet(half) || meet(wide)) return meet(wide);
    return half.a.N <= 13312 || half.a.Kc <= 512 ||
           (half.a.Kc <= 1024 && bytes(half, kWave * Vec<kI8Half>::kElems) <= bytes(wide, kWave * Vec<kI8>::kElems));
}

// Both launches, lists of 32-channel segments between them; kG1NotApplicable where either does not run here so, or the gate|up
// launch is faster in 16-byte lanes.  8-byte lanes have one column per lane and slice, so the gate|up launch hands over in
// fixed point, and small blocks have tiles enough (2F <= 4096 ran on the general kernel: 4096 -> 2048 -> 4096 23.7 / 18.2 us at
// 40 / 70 %).
int launch_swiglu_block2_pair(const GemvArgs& up, const GemvArgs& dn, int wdt, int flags, hipStream_t stream) {
    Gemv1bArgs gu, gd, wide;
    bool hu = false, hd = false, hw = false;
    if (plan_block2_part(up, dn, wdt, 0, true, flags & kG1FlagParkSlices, &gu, &hu) != SCAP_OK || !hu || gu.a.fx_acc == nullptr ||
        plan_block2_part(up, dn, wdt, 1, true, 0, &gd, &hd) != SCAP_OK)
        return kG1NotApplicable;
    if (plan_block2_64(up, dn, wdt, 0, &wide, &hw) == SCAP_OK && !half_lanes_are_faster(gu, wide)) return kG1NotApplicable;
    const int rc = launch_block2(gu, wdt, hu, kFuseSwiglu, stream);
    if (rc != SCAP_OK) return rc;
    return launch_block2(gd, wdt, hd, kFuseList32, stream);
}

}  // namespace scap
