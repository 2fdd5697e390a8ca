// Batched sparse FC on the matrix cores, row step by row step: most calls of 5-16 tokens and many of 3-4 (rows_pay), both launches of a
// batch's block and the gate|up launch of many blocks of 2-4 tokens.  No list and no staging: a wavefront takes steps of 32 rows.  Lane l takes
// 8 consecutive inputs of token l % 16 (16 bytes; the operand layout of the 32-deep matrix instruction), prunes them in registers -- that
// is the operand --, ORs the tokens' keep bits over its row of 16 lanes, and asks for its part of the 8 rows; a row that no token keeps is
// asked for at an offset behind the buffer and costs an issue slot, no memory traffic.  Nothing is exchanged between wavefronts before the
// sums are added, so the first weight rows are asked for one memory latency after the kernel starts, and a piece may be as long as the layer.
// The staged-tile kernel (scap_gemm_inline.hip) tests and lists a piece before its first row: 3.6 us of 18.7 on 14336 x 4096
// int8, 12 tokens, 4.3-6.7 of 46 on 4096 x 28672 bf16, 16 tokens, and its pieces have to fit LDS.  Here inputs are 1 KB more per
// 8 KB of rows (int8: per 4), out of L2.
//
// Where the operand comes from (SRC):
// kRowsCodes -- the centred input IS the 16-bit input: m = 0 (inputs that are already centred: everything behind a norm, a GLU block's inputs)
// or dense mode, activations of the operand's own type (bf16 over bf16 and int8 weights, fp16 over fp16 weights).  Then x - m needs no second half,
// and the pruner decides on the 16-bit codes, two elements a lane and instruction:
//
//   |x| > tau  <=>  (code & 0x7fff) > code(tau), and no NaN  <=>  (code & 0x7fff) - lo < len  as unsigned 16-bit numbers
//
// with code(tau) the largest 16-bit value that is not above tau (exact: a value above tau is above code(tau), too).
// kRowsPlanes -- the gated product of a block as the gate|up launch leaves it: planes of operand heads and tails, a pruned channel 0 in both.
// kRowsCentre -- any m and activation type: centred and tested in fp32, split into head and tail in registers.
//
// What bounds it: the row stream (6.3 TB/s in 256-byte pieces over a long launch, 7.1 over a short one), then the reduction of eight
// wavefronts (1 us) and the hand-over (2 us).  us per call, staged tile (3-4 tokens: four-slot kernel) / here: 4096 x 28672 bf16, 16 tokens at 70 %,
// 48.5 / 40.2, centred 51.0 / 44.5; 14336 x 4096, 16 tokens at 50 %, 27.3 / 24.9; 4096 x 11008 fp16, 8 tokens at 50 %, 22.4 / 20.1; 14336 x 4096 int8,
// 12 tokens at 70 %, 18.3 / 14.6; 4096 x 4096 bf16, 8 tokens at 50 %, 12.3 / 10.1, 4 tokens 13.9 / 9.6.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "scap_mfma_parts.hpp"

namespace scap {

constexpr int kStepRows = 32;  // rows of one matrix instruction
constexpr int kRowsFewCols = 32768;  // 2-4 tokens: most columns that run here
constexpr int kWideTokens = 4;  // up to so many tokens the K splits of a plain call meet as 64-bit values (finish_wide)
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));

// Elements of the two halves of a word that the pruner drops become 0; flags: 1 in each half that is kept.
__device__ __forceinline__ uint32_t keep_pair(uint32_t v, u16x2_t lo, u16x2_t len, u16x2_t one, uint32_t& flags) {
    union { uint32_t u; u16x2_t h; } a, x, f, r;
    a.u = v & 0x7fff7fffu;
    x.u = v;
    f.h = __builtin_elementwise_min(__builtin_elementwise_sub_sat(len, (u16x2_t)(a.h - lo)), one);
    r.h = x.h * f.h;
    flags = f.u;
    return r.u;
}

// OR over the sixteen lanes of a row
__device__ __forceinline__ uint32_t or_of_sixteen(uint32_t v) {
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);   // lanes 1,0,3,2 of a quad
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);   // lanes 2,3,0,1
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);  // mirrored in each half row
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);  // mirrored in each row
    return v;
}

template <int N> struct Words { uint32_t w[N]; };

// Two centred values as a word of heads and a word of tails (split_halves, two at a time).
template <int WDT>
__device__ __forceinline__ void split_pair(float d0, float d1, uint32_t& hi, uint32_t& lo) {
    if constexpr (WDT == kF16) {
        const uint32_t a = split_halves<WDT>(d0), b = split_halves<WDT>(d1);
        hi = (a & 0xffffu) | (b << 16);
        lo = (a >> 16) | (b & 0xffff0000u);
    } else {
        typedef float f32x2_t __attribute__((ext_vector_type(2)));
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
        union { bf16x2_t b; uint32_t u; } h, l;  // (round to nearest even, as split_halves does)
        h.b = __builtin_convertvector((f32x2_t{d0, d1}), bf16x2_t);
        const bool fin0 = (h.u & 0x7f80u) != 0x7f80u, fin1 = (h.u & 0x7f800000u) != 0x7f800000u;  // an infinite head has no tail
        l.b = __builtin_convertvector((f32x2_t{fin0 ? d0 - __uint_as_float(h.u << 16) : 0.f,
                                               fin1 ? d1 - __uint_as_float(h.u & 0xffff0000u) : 0.f}), bf16x2_t);
        hi = h.u;
        lo = l.u;
    }
}

// Per-token counts and lists and the size of the union, on request (the tile's own tokens; the union: tile 0).  kept_tok, kept_any:
// the calling lane's counts over its rows (lane = token l % 16, row group l / 16).  The lists are read off the inputs once more.
template <int WAVES, int SRC>
__device__ __forceinline__ void leave_lists(const GemvArgs& a, int tile, int split, int k0, int kend, int kept_tok, int kept_any,
                                            const Lds& L) {
    const uint32_t own = owned_tokens(a, tile);
    const bool own_union = tile == 0 && a.union_nnz_out != nullptr;
    if (own == 0 && !own_union) return;
    const int tid = threadIdx.x;
    const int w = uniform(tid >> 6);
    const int lane = tid & 63;
    const bool dense = a.mode == kModeDense;
    kept_tok += __shfl_xor(kept_tok, 16, kWave);
    kept_tok += __shfl_xor(kept_tok, 32, kWave);
    kept_any += __shfl_xor(kept_any, 16, kWave);
    kept_any += __shfl_xor(kept_any, 32, kWave);
    if (lane < kMfmaTokens) L.hdr[(1 + lane) * WAVES + w] = kept_tok;
    if (lane == 0) L.hdr[w] = kept_any;
    __syncthreads();
    if (tid < kMfmaTokens + 1) {
        int sum = 0;
        for (int i = 0; i < WAVES; ++i) sum += L.hdr[tid * WAVES + i];
        if (dense) sum = kend - k0;  // (rows past the last channel were counted)
        if (tid == 0 ? own_union : (own >> (tid - 1)) & 1u) store_dev(&a.seg_cnt[(tid == 0 ? a.B : tid - 1) * a.Sl + split], sum);
    }
    if (a.idx_out == nullptr || own == 0) return;
    // ascending lists: a wavefront takes a run of 64-channel chunks, its counts first, then the entries
    const int nchunk = (kend - k0 + kWave - 1) / kWave;
    const int cpw = (nchunk + WAVES - 1) / WAVES;
    const int c_begin = min(w * cpw, nchunk), c_end = min(c_begin + cpw, nchunk);
    auto kept_at = [&](int c, int b) {
        const int k = k0 + c * kWave + lane;
        if (k >= kend) return false;
        const int64_t at = (int64_t)b * a.x_pitch + k;
        if constexpr (SRC == kRowsPlanes)
            return (a.x[at] | a.zl_lo[at]) != 0;
        else if constexpr (SRC == kRowsCentre)
            return dense || fabsf(act_to_f32(a.x, at, a.xdt) - a.m) > a.tau;
        else
            return dense || ((((uint32_t)a.x[at] & 0x7fffu) - a.keep_lo) & 0xffffu) < a.keep_len;
    };
    for (int b = 0; b < a.B; ++b) {
        if (!((own >> b) & 1u)) continue;
        int n = 0;
        for (int c = c_begin; c < c_end; ++c) n += __popcll(__ballot(kept_at(c, b)));
        __syncthreads();  // the counts above, or the token before, have been read
        if (lane == 0) L.hdr[w] = n;
        __syncthreads();
        int at = 0;
        for (int i = 0; i < w; ++i) at += L.hdr[i];
        for (int c = c_begin; c < c_end; ++c) {
            const bool keep = kept_at(c, b);
            const uint64_t bal = __ballot(keep);
            if (keep) store_dev(&a.idx_out[(int64_t)b * a.K + k0 + at + lanes_below(bal)], k0 + c * kWave + lane);
            at += __popcll(bal);
        }
    }
}

// 32 rows against the operand `av`: acc[e] += A * B_e for the ELEMS column elements.  r[j] = this lane's part of row 8*(l/16) + j.
// HALVES = 2: av[4..7] are the operand's tails.
template <int WDT, int HALVES>
__device__ __forceinline__ void mfma_rows(f32x4_t* __restrict__ acc, const uint32_t (&av)[4 * HALVES], const uint4 (&r)[8]) {
    constexpr int ELEMS = Vec<WDT>::kElems;
    uint32_t q[8][4];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        q[j][0] = r[j].x;
        q[j][1] = r[j].y;
        q[j][2] = r[j].z;
        q[j][3] = r[j].w;
    }
    union Op { uint32_t u[4]; bf16x8_t b; f16x8_t f; } ao[HALVES];
#pragma unroll
    for (int i = 0; i < 4 * HALVES; ++i) ao[i / 4].u[i % 4] = av[i];
#pragma unroll
    for (int e = 0; e < ELEMS; ++e) {
        Op bo;  // rows (0,1), (2,3), ... of column element e
#pragma unroll
        for (int pr = 0; pr < 4; ++pr) {
            const uint32_t* x0 = q[2 * pr];
            const uint32_t* x1 = q[2 * pr + 1];
            if constexpr (is_int8(WDT)) {
                // byte e of each row, sign-extended, as a float: its low 16 bits are zero (|v| <= 128)
                const int c = e >> 2, sh = 24 - 8 * (e & 3);
                const uint32_t f0 = __float_as_uint((float)(((int)(x0[c] << sh)) >> 24));
                const uint32_t f1 = __float_as_uint((float)(((int)(x1[c] << sh)) >> 24));
                bo.u[pr] = __builtin_amdgcn_perm(f1, f0, 0x07060302u);
            } else {
                const int c = e >> 1;
                bo.u[pr] = __builtin_amdgcn_perm(x1[c], x0[c], (e & 1) ? 0x07060302u : 0x05040100u);
            }
        }
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
            if constexpr (WDT == kF16)
                acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ao[h].f, bo.f, acc[e], 0, 0, 0);
            else
                acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ao[h].b, bo.b, acc[e], 0, 0, 0);
        }
    }
}

// A wavefront's sums of the existing tokens go to its 8 KB of LDS, [16 tokens][32 groups of 4 columns], on top of what it has left there before.
__device__ __forceinline__ void park_sums(const GemvArgs& a, const f32x4_t (&acc)[8], float* s_red, bool more) {
    int tid = threadIdx.x;
    asm("" : "+v"(tid));  // (addresses are made here: kept, they would take registers of the loop)
    const int kg = (tid >> 4) & 3;
    f32x4_t* const at = reinterpret_cast<f32x4_t*>(s_red) + (tid >> 6) * (kMfmaTokens * 32) + 4 * kg * 32 + 2 * (tid & 15);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (4 * kg + i < a.B) {
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                f32x4_t t = f32x4_t{acc[4 * v][i], acc[4 * v + 1][i], acc[4 * v + 2][i], acc[4 * v + 3][i]};
                if (more) t += at[i * 32 + v];
                at[i * 32 + v] = t;
            }
        }
        __builtin_amdgcn_sched_barrier(0);  // (a few registers at a time)
    }
}

__device__ __forceinline__ float4 narrow(const double (&s)[4]) { return make_float4((float)s[0], (float)s[1], (float)s[2], (float)s[3]); }
__device__ __forceinline__ void add_to(double (&s)[4], const float4& v) {
    s[0] += (double)v.x;
    s[1] += (double)v.y;
    s[2] += (double)v.z;
    s[3] += (double)v.w;
}

// The eight wavefronts' sums of a thread's token and 4 columns, in wavefront order, added in 64 bits and rounded once, to a finished value
// or a split's sum (up to kWideTokens tokens, plain calls: not even that, finish_wide).  The matrix unit rounds twice a step (a sum of 16 products
// each); eight additions here and those over the splits, in 32 bits, came on top and took calls of 3-4 tokens to up to twice the error of the
// vector kernels, whose splits meet in fixed point.  Relative error against 64 bits, those / all in 32 bits / so: 4 tokens, 4096 x 4096 bf16 at 50 %
// 4.0e-8 / 7.8e-8 / 3.7e-8, 1024 x 4096 fp16 at 90 % 4.4e-8 / 7.1e-8 / 4.3e-8, 14336 x 4096 int8 dense 8.4e-8 / 8.8e-8 / 4.5e-8; 8 tokens, before the
// row steps / 32 bits / so: 8192 x 16384 fp16 at 50 % 1.25e-7 / 1.59e-7 / 0.94e-7.  Two columns a lane and eight loads in flight, the additions cost
// nothing that shows (1024 x 4096 bf16, 4 tokens, 5.8 us both ways, 2048 x 2048, 16 tokens, 6.8 / 6.6; four columns a lane 6.3).
template <int WDT, int FUSE>
__device__ __forceinline__ void add_waves_and_emit(const GemvArgs& a, __amdgpu_buffer_rsrc_t pbuf, int tile, int split, const float* s_red, float* s_fin) {
    const int b = threadIdx.x >> 5, g = threadIdx.x & 31;
    __syncthreads();
    if (b >= a.B) return;
    double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int w = 0; w < kInlineWaves; ++w) add_to(t, reinterpret_cast<const float4*>(s_red)[w * (kMfmaTokens * 32) + threadIdx.x]);
    emit_group<WDT, kMfmaTile, FUSE>(a, pbuf, tile, split, b, g, narrow(t), s_fin, a.S == 1 ? load_col_const<WDT, kMfmaTile>(a, tile, g) : ColConst{});
}

// Whether the calling wavefront is the last of the tile's workgroups at its ticket: its own stores are acknowledged first.
__device__ __forceinline__ bool last_arrival(const GemvArgs& a, int32_t* ticket) {
    wait_memory_ops();
    int old = 0;
    if ((threadIdx.x & 63) == 0) old = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return uniform(old) == a.S - 1;
}
// ... which makes the ticket ready for the next call, and (the first wavefront, whose threads have stored its split's) adds the counts up.
__device__ __forceinline__ void after_last(const GemvArgs& a, int32_t* ticket, uint32_t own, bool own_union) {
    const int lane = threadIdx.x & 63;
    if (lane == 0) store_dev(ticket, 0);
    if (uniform(threadIdx.x >> 6) != 0 || (own == 0 && !own_union)) return;
    for (int l = 0; l <= a.B; ++l) {
        const bool is_union = l == a.B;
        if (is_union ? !own_union : !((own >> l) & 1u)) continue;
        int run = 0;
        for (int sp = lane; sp < a.Sl; sp += kWave) run += load_dev(&a.seg_cnt[l * a.Sl + sp]);
        run = wave_sum(run);
        if (lane == 0) *(is_union ? a.union_nnz_out : a.nnz_out + l) = run;
    }
}

// Hand-over of a plain call: a wavefront finishes the two tokens whose sums it has emitted by itself -- stores
// acknowledged, one ticket per (tile, wavefront), 128 bytes apart, the last arrival adds the S partial sums in split order -- so that
// no wavefront waits for another behind the reduction and the last arrivals of a tile's tokens may be different workgroups
// (finish_tile: one ticket per workgroup, two barriers).  own, own_union: counts that are added up, too.  us per call, there / here: 1024 x 4096 bf16, 4
// tokens, 6.7 / 5.9, 2048 x 2048 fp16, 5 tokens, 6.9 / 6.1, 4096 x 4096 bf16, 8 tokens, 10.8 / 10.0, 14336 x 4096 int8, 12 tokens, 15.2 / 14.8.
template <int WDT, int TILE>
__device__ __forceinline__ void finish_slices(const GemvArgs& a, __amdgpu_buffer_rsrc_t pbuf, int tile, const ColConst& mine, uint32_t own,
                                              bool own_union) {
    const int w = uniform(threadIdx.x >> 6);
    const int b = threadIdx.x >> 5, g = threadIdx.x & 31;  // as add_waves_and_emit deals them out
    static_assert(TILE == 128, "32 groups of 4 columns, 16 tokens, 512 threads");
    if (2 * w >= a.B) return;  // wave-uniform: no token of this wavefront exists
    int32_t* ticket = a.counters + tile * kCounterStride + 32 * w;
    if (!last_arrival(a, ticket)) return;
    const uint32_t at = (uint32_t)(((b * a.S * a.T + tile) * TILE + 4 * g) * 4), stride = (uint32_t)a.T * TILE * 4u;
    double s[4] = {0.0, 0.0, 0.0, 0.0};  // (see add_waves_and_emit)
    for (int sp0 = 0; sp0 < a.S; sp0 += 8) {  // 8 loads in flight; slots past the last split ask behind the buffer and get zeros
        float4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = load_coherent16(pbuf, sp0 + j < a.S && b < a.B ? at + (uint32_t)(sp0 + j) * stride : kNoRow);
#pragma unroll
        for (int j = 0; j < 8; ++j) add_to(s, v[j]);
    }
    if (b < a.B) finish_columns<WDT, TILE>(a, tile, b, g, narrow(s), nullptr, mine);
    after_last(a, ticket, own, own_union);
}

// The same for up to kWideTokens tokens, from the wavefronts' sums on: wavefront b takes token b, two columns a lane, and hands them
// over as 64-bit values, [B][S][T][128] -- the splits' sums then meet without a rounding, as they do in fixed point on the vector kernels
// that ran these calls (add_waves_and_emit).
template <int WDT>
__device__ __forceinline__ void finish_wide(const GemvArgs& a, int tile, int split, const float* s_red, uint32_t own, bool own_union) {
    const int lane = threadIdx.x & 63, b = uniform(threadIdx.x >> 6);
    __syncthreads();
    if (b >= a.B) return;
    const int col = tile * kMfmaTile + 2 * lane;  // N is a multiple of 8: both columns exist or none
    float2 bias = make_float2(0.f, 0.f), scale = make_float2(1.f, 1.f);
    if (col < a.N) {
        if (a.bias) bias = *reinterpret_cast<const float2*>(a.bias + col);
        if (is_int8(WDT)) {
            const uint32_t h = *reinterpret_cast<const uint32_t*>(a.col_scale + col);
            scale = make_float2(f16_bits_to_f32(h & 0xFFFFu), f16_bits_to_f32(h >> 16));
        }
    }
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int w = 0; w < kInlineWaves; ++w) {
        const float2 v = reinterpret_cast<const float2*>(s_red)[(w * kMfmaTokens + b) * (kMfmaTile / 2) + lane];
        s0 += (double)v.x;
        s1 += (double)v.y;
    }
    if (a.S > 1) {
        const __amdgpu_buffer_rsrc_t wide = make_raw_buffer(a.partial, (uint32_t)a.B * a.S * a.T * kMfmaTile * 8u);
        const uint32_t at = (uint32_t)((b * a.S * a.T + tile) * kMfmaTile + 2 * lane) * 8u, stride = (uint32_t)a.T * kMfmaTile * 8u;
        store_coherent16(wide, at + (uint32_t)split * stride,
                         make_float4(__int_as_float(__double2loint(s0)), __int_as_float(__double2hiint(s0)), __int_as_float(__double2loint(s1)),
                                     __int_as_float(__double2hiint(s1))));
        int32_t* ticket = a.counters + tile * kCounterStride + 32 * b;
        if (!last_arrival(a, ticket)) return;
        s0 = s1 = 0.0;
        for (int sp0 = 0; sp0 < a.S; sp0 += 8) {
            float4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = load_coherent16(wide, sp0 + j < a.S ? at + (uint32_t)(sp0 + j) * stride : kNoRow);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                s0 += __hiloint2double(__float_as_int(v[j].y), __float_as_int(v[j].x));
                s1 += __hiloint2double(__float_as_int(v[j].w), __float_as_int(v[j].z));
            }
        }
        after_last(a, ticket, own, own_union);
    }
    if (col < a.N) {
        float2 y = make_float2((float)s0, (float)s1);
        if (is_int8(WDT)) y = make_float2(y.x * scale.x, y.y * scale.y);
        store_coherent8(make_raw_buffer(a.y, (uint32_t)((size_t)a.B * a.N * 4)), (uint32_t)(((int64_t)b * a.N + col) * 4), make_float2(y.x + bias.x, y.y + bias.y));
    }
}

// LDS floats of the wavefronts' sums: all eight side by side, or (16-byte int8 lanes) a tree
constexpr int sum_floats(int wdt) { return wdt == kI8 ? kTreeFloats : kInlineWaves * kMfmaTokens * kMfmaTile; }

// workgroups of a launch that a compute unit holds at once (registers)
constexpr int rows_resident(int wdt, int src, bool ragged) {
    return wdt == kI8Half || (src == kRowsCodes && !ragged && wdt != kI8) ? 2 : 1;
}

// SLOTS: token slots of what a gating launch leaves (2, 4: lists of centred values; 16: planes of operand halves), else 16.
template <int WDT, int FUSE, int SRC, bool RAGGED, int SLOTS>
__global__ __launch_bounds__(kInlineWaves* kWave, 2 * rows_resident(WDT, SRC, RAGGED)) void gemm_rows_kernel(const GemvArgs a) {
    constexpr int HALVES = SRC == kRowsCodes ? 1 : 2;
    constexpr int INPUTS = SRC == kRowsPlanes ? 8 : 4;  // words of a step's inputs
    constexpr int WAVES = kInlineWaves;
    constexpr int ELEMS = Vec<WDT>::kElems;
    constexpr int TILE = 16 * ELEMS;

    extern __shared__ uint4 smem_raw[];
    Lds L = carve_lds<WAVES, kMfmaTokens>(reinterpret_cast<char*>(smem_raw), 0);
    // A wavefront's accumulators are added to its place in LDS every so many steps: a long chain would lose what few-row sums keep (fp16, 8192 x
    // 16384, 8 tokens at 50 %, one chain of 32 steps 1.59e-7, of 8 1.15e-7, of 4 0.94e-7; over 63 layers at 0, 50 and 90 % no error above that before the row
    // steps but one, by 3 %, with 8 steps over 16-bit weights eight, by up to 9 %; int8 products fill fewer bits).  us, without / so: 14336 x 4096 bf16, 8 tokens,
    // 23.4 / 23.6, 4096 x 11008, 16 tokens, 21.9 / 21.9, blocks 4096 -> 14336, 16 tokens, 64.7 / 65.3, 14336 x 4096 int8, 8 tokens, 15.3 / 15.3 (every 4 steps 15.5).
    constexpr int kChainSteps = WDT == kI8Half ? 8 : 4;
    constexpr bool WHOLE = WDT != kI8;  // (16-byte int8 lanes have 256 columns: the sums meet in halves, through a tree)
    if constexpr (FUSE == kFuseSwiglu) L.fin = L.red + sum_floats(WDT);
    const int tid = threadIdx.x;
    const int w = uniform(tid >> 6);
    const int lane = tid & 63;
    const int tile = blockIdx.x % a.T;
    const int split = blockIdx.x / a.T;
    const int k0 = split * a.Kc;
    const int kend = min(k0 + a.Kc, a.K);

    const int cg = lane & 15;  // column group (B/C index n); also the token whose values this lane supplies (A index m)
    const int kg = lane >> 4;  // row group: rows 8*kg .. 8*kg+7 of a step
    const int col0 = tile * TILE + cg * ELEMS;
    const uint32_t lane_off = (col0 < a.N) ? (uint32_t)col0 * Vec<WDT>::kBytes : kNoRow;
    const uint32_t row_bytes = (uint32_t)a.N * Vec<WDT>::kBytes;
    const __amdgpu_buffer_rsrc_t wbuf = weight_rows(a, k0, row_bytes);
    const __amdgpu_buffer_rsrc_t xbuf = make_raw_buffer(const_cast<uint16_t*>(a.x), (uint32_t)a.B * (uint32_t)a.x_pitch * 2u);
    const __amdgpu_buffer_rsrc_t tbuf = make_raw_buffer(a.zl_lo, (uint32_t)a.B * (uint32_t)a.x_pitch * 2u);
    const u16x2_t lo = (u16x2_t)((unsigned short)a.keep_lo), len = (u16x2_t)((unsigned short)a.keep_len);
    // (a 1 that the compiler does not know: it would turn the packed steps into compares and selects, element by element)
    union { uint32_t u; u16x2_t h; } one = {0x00010001u};
    asm("" : "+v"(one.u));

    const bool dense = a.mode == kModeDense;
    const float m_eff = dense ? 0.f : a.m;  // (centred inputs) dense mode: x - 0 is x
    const uint32_t bf16_sel = a.xdt == kBF16 ? 0xffffffffu : 0u;

    f32x4_t acc[ELEMS];
#pragma unroll
    for (int e = 0; e < ELEMS; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // Steps in flight: four instead of two (207 registers, one workgroup per unit) were no faster on any of 19 layers.
    constexpr int DEPTH = 2;
    struct Stage {
        uint4 r[8];
        uint32_t op[4 * HALVES];
    };
    typedef Words<INPUTS> Inputs;  // 8 values of the lane's token (and their tails)
    const int n_all = (kend - k0 + kStepRows - 1) / kStepRows;
    const int n_steps = n_all > w ? (n_all - w + WAVES - 1) / WAVES : 0;  // steps w, w + WAVES, ... of 32 rows
    int kept_tok = 0, kept_any = 0;  // rows of this lane's group that its token keeps, that any token keeps
    // inputs of a step: 8 channels of the lane's token; 0 past the last channel and for slots past the batch
    auto load_x = [&](int st) {
        const int k = k0 + (w + st * WAVES) * kStepRows + 8 * kg;
        Inputs in;
        if constexpr (!RAGGED) {
            const uint32_t off = k < a.K && cg < a.B ? (uint32_t)(cg * a.x_pitch + k) * 2u : kNoRow;
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (int)off, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) in.w[q] = v[q];
            if constexpr (SRC == kRowsPlanes) {
                const auto t = __builtin_amdgcn_raw_buffer_load_b128(tbuf, (int)off, 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q) in.w[4 + q] = t[q];
            }
        } else {
            static_assert(!RAGGED || SRC != kRowsPlanes, "planes have whole octets");
            // rows that start at any 2-byte boundary; the last octet of a token runs into the next token's values, that of the last
            // token is read element by element
            const int total = a.B * a.K, p = min(cg, a.B - 1) * a.K + min(k, a.K - 1);
            uint4 v = total >= 8 ? load_octet(a.x + min(p, total - 8)) : make_uint4(0u, 0u, 0u, 0u);
            if (p > total - 8) v = load_octet_cut(a.x + p, total - p);
            const int n = cg < a.B ? a.K - k : 0;  // elements of the octet that exist
            const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) in.w[q] = n >= 2 * q + 2 ? wd[q] : (n == 2 * q + 1 ? wd[q] & 0xffffu : 0u);
        }
        return in;
    };
    // (Registers: 128 at two workgroups per compute unit, which shapes of more than 256 workgroups need -- 8192 x 28672, 6 tokens, 512-row
    // pieces 82.3 us against 88.4 with one.  An odd input length takes a few more and runs one.)
    // Prune the inputs of step st, replace them by those of step `ahead`, and fetch the rows that some token keeps; the others ask
    // for an offset behind the buffer: nothing is read.  (The inputs go first: loads come back in order, and the next step's test must
    // not wait for rows.)
    auto issue = [&](int st, Inputs& x, int ahead, Stage& sg) {
        uint32_t f[4], mine = 0;  // bit j: row 8*kg + j kept by this token
        // channels of the lane's octet that exist (centred values: a missing one would be -m)
        const int left = SRC == kRowsCentre && cg < a.B ? a.K - (k0 + (w + st * WAVES) * kStepRows + 8 * kg) : 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (SRC == kRowsCodes) {
                sg.op[q] = keep_pair(x.w[q], lo, len, one.h, f[q]);
            } else if constexpr (SRC == kRowsCentre) {
                float d[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t as_bf16 = h ? x.w[q] & 0xffff0000u : x.w[q] << 16;
                    const uint32_t as_f16 = __float_as_uint(f16_bits_to_f32(h ? x.w[q] >> 16 : x.w[q] & 0xffffu));
                    const float c = __uint_as_float((as_bf16 & bf16_sel) | (as_f16 & ~bf16_sel)) - m_eff;  // one fp32 subtraction
                    const bool keep = (RAGGED ? 2 * q + h < left : left > 0) & (dense | (fabsf(c) > a.tau));  // strict; NaN is pruned
                    d[h] = keep ? c : 0.f;
                    mine |= keep ? 1u << (2 * q + h) : 0u;
                }
                split_pair<WDT>(d[0], d[1], sg.op[q], sg.op[4 + q]);
            } else {
                sg.op[q] = x.w[q];
                sg.op[4 + q] = x.w[4 + q];
                union { uint32_t u; u16x2_t h; } any = {x.w[q] | x.w[4 + q]};
                any.h = __builtin_elementwise_min(any.h, one.h);  // a pruned channel is 0 in both planes
                f[q] = any.u;
            }
        }
        if constexpr (SRC != kRowsCentre) {
            const uint32_t t = f[0] | (f[1] << 2) | (f[2] << 4) | (f[3] << 6);
            mine = (t | (t >> 15)) & 0xffu;
        }
        const uint32_t any = or_of_sixteen(mine);
        if constexpr (FUSE == kFusePlain) {
            kept_tok += __popc(mine);
            kept_any += __popc(any);
        }
        x = load_x(ahead);
        const uint32_t drop = ~any;
        const uint32_t base = __umul24((uint32_t)((w + st * WAVES) * kStepRows + 8 * kg), row_bytes) + lane_off;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            sg.r[j] = load_row_part<WDT>(wbuf, (base + j * row_bytes) | ((drop << (31 - j)) & kNoRow));
    };
    bool any_parked = false;
    if (n_steps > 0) {
        // Steps st .. st + DEPTH-1 are in flight or in work, the inputs of the DEPTH after them too (loads come back in order: a
        // test that waited for younger inputs would wait for the rows before them).  One way out of the loop: where it also
        // ended between its turns, the compiler waited for all loads in each.
        Inputs X[DEPTH];
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) X[u] = load_x(u);
        Stage S[DEPTH];
#pragma unroll
        for (int u = 0; u < DEPTH - 1; ++u) issue(u, X[u], u + DEPTH, S[u]);
        int st = 0;
        const int last = n_steps - 2 * DEPTH + 1;  // turns begin at steps up to here
        while (st <= last) {
            const int stop = WHOLE ? min(st + kChainSteps - 1, last) : last;
            do {
#pragma unroll
                for (int u = 0; u < DEPTH; ++u) {
                    issue(st + u + DEPTH - 1, X[(u + DEPTH - 1) % DEPTH], st + u + 2 * DEPTH - 1, S[(u + DEPTH - 1) % DEPTH]);
                    __builtin_amdgcn_sched_barrier(0);
                    mfma_rows<WDT, HALVES>(acc, S[u].op, S[u].r);
                    __builtin_amdgcn_sched_barrier(0);
                }
                st += DEPTH;
            } while (st <= stop);
            if (st > last) break;
            if constexpr (WHOLE) {
                park_sums(a, acc, L.red, any_parked);
                any_parked = true;
#pragma unroll
                for (int e = 0; e < ELEMS; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int u = 0; u < 2 * DEPTH - 2; ++u) {  // the last ones
            if (st + u < n_steps) {
                if (u < DEPTH - 1 && st + u + DEPTH - 1 < n_steps)
                    issue(st + u + DEPTH - 1, X[(u + DEPTH - 1) % DEPTH], st + u + 2 * DEPTH - 1, S[(u + DEPTH - 1) % DEPTH]);
                __builtin_amdgcn_sched_barrier(0);
                mfma_rows<WDT, HALVES>(acc, S[u % DEPTH].op, S[u % DEPTH].r);
            }
        }
    }

    if constexpr (WHOLE) park_sums(a, acc, L.red, any_parked);
    if constexpr (FUSE == kFusePlain) leave_lists<WAVES, SRC>(a, tile, split, k0, kend, kept_tok, kept_any, L);  // (a block asks for none of its input)
    if constexpr (FUSE == kFusePlain && WHOLE) {
        const uint32_t own = owned_tokens(a, tile);
        const bool own_union = tile == 0 && a.union_nnz_out != nullptr, lists = a.idx_out != nullptr;
        if (a.B <= kWideTokens) {
            finish_wide<WDT>(a, tile, split, L.red, lists ? 0u : own, !lists && own_union);
        } else {
            const ColConst mine = load_col_const<WDT, TILE>(a, tile, tid % (TILE / 4));
            const __amdgpu_buffer_rsrc_t pbuf = partial_buffer<TILE>(a);
            add_waves_and_emit<WDT, FUSE>(a, pbuf, tile, split, L.red, nullptr);
            if (a.S > 1) finish_slices<WDT, TILE>(a, pbuf, tile, mine, lists ? 0u : own, !lists && own_union);
        }
        if ((own == 0 && !own_union) || (a.S > 1 && !lists)) return;
        // lists: a ticket of their own, taken by the workgroup (the sums above are the same without them)
        wait_memory_ops();
        __syncthreads();
        if (a.S > 1) {
            int32_t* ticket = a.counters + tile * kCounterStride + 16;
            if (tid == 0) L.flag[0] = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.S - 1;
            __syncthreads();
            if (L.flag[0] == 0) return;
            if (tid == 0) store_dev(ticket, 0);  // ready for the next call
        }
        close_lists<WAVES>(a, L, own, own_union);
    } else {
        // constants of the column group this thread finishes if its workgroup is the tile's last arrival
        const ColConst mine = load_col_const<WDT, TILE>(a, tile, tid % (TILE / 4));
        const __amdgpu_buffer_rsrc_t pbuf = partial_buffer<TILE>(a);
        if constexpr (WHOLE)
            add_waves_and_emit<WDT, FUSE>(a, pbuf, tile, split, L.red, L.fin);
        else
            reduce_waves_and_emit<WDT, WAVES, FUSE>(a, pbuf, tile, split, acc, L.red, L.fin);
        finish_tile<WDT, WAVES, TILE, SLOTS, FUSE>(a, pbuf, tile, L, mine);
    }
}

// ---------------------------------------------------------------------------------------------- launch
bool exact_operand(const GemvArgs& a, int wdt) {
    if (a.xdt != (wdt == kF16 ? kF16 : kBF16)) return false;
    return a.mode == kModeDense || (a.mode == kModeSparse && a.m == 0.f);
}

// A row that no token keeps costs its issue slot here, and over int8 weights its widening, where the list kernels never meet it: what the row steps
// gain at 50-70 % in a large layer turns over where few rows are kept, and the host does not know how many that will be.  From sweeps of 230 layers at 50,
// 70 and 90 % on either kernel: a kind of call runs here where its gains at the three add up.  us there / here at 50, 70 and 90 %, inside / beyond the line (odd: an input length that is
// not a multiple of 8):
// 3 tokens, whose lists are shorter, 2^25 weights (50 and 90 %): bf16 4096 x 4096 11.8 / 8.8, 9.1 / 6.4; beyond 8192 x 8192 24.7 / 23.1, 13.2 / 14.1.
// 4 tokens, 16-bit weights (50 and 90 %): 8192 x 16384 47.4 / 44.0, 24.1 / 24.5; odd 9001 x 9600 35.5 / 29.7, 19.9 / 20.7; beyond 16383 x 8192 48.0 / 46.5, 24.8 / 27.1.
// 4 tokens, int8: 5120 x 13824 21.5 / 17.5, 19.1 / 17.2, 15.0 / 14.4; 8192 x 14336 30.2 / 26.5, 25.2 / 24.3, 17.1 / 20.2; 28672 x 8192 50.0 / 43.7, 41.7 / 37.6, 28.7 / 32.3; wide 8192 x 26752 48.1 / 41.6, 41.2 /
// 40.6, 29.1 / 33.5; beyond 16384 x 20480 66.6 / 64.5, 56.1 / 53.1, 36.3 / 43.1; odd 16385 x 4608 23.1 / 19.4, 20.6 / 19.4, 16.5 / 16.6; beyond 8193 x 10112 23.9 / 22.5, 21.2 / 22.2, 16.5 / 19.2.
// 5-6 tokens, int8 (5 here): 8192 x 14336 31.1 / 27.3, 26.8 / 24.6, 18.4 / 20.6; 16384 x 12416 48.2 / 37.9, 40.9 / 35.2, 30.5 / 30.2; 16384 x 28672 94.4 / 89.3, 79.6 / 74.0, 51.2 / 57.4; odd 13889 x
// 12032 41.8 / 35.9, 37.0 / 34.8, 28.2 / 30.2; centred 5376 x 16384 26.2 / 20.9, 22.8 / 19.6, 16.2 / 17.6, 16384 x 7424 31.1 / 27.1, 28.1 / 26.7, 20.4 / 24.6, 4096 x 28672 30.1 / 27.9, 27.5 / 25.4, 19.9 / 22.6;
// centred and odd (50 and 90 %) 8193 x 8192 22.7 / 18.2, 16.5 / 16.6; beyond 9001 x 9600 26.4 / 23.9, 18.5 / 23.1.
// What that leaves at 90 %: up to 17 % more (16384 x 7424 centred, 8192 x 14336 int8, 4 tokens); at 95 % more.  From 12 tokens on the union is large enough everywhere
// (8192 x 16384, 12 tokens, 23.2 / 23.1).
bool rows_pay(const GemvArgs& a, int wdt) {
    const int64_t weights = (int64_t)a.K * a.N;
    const auto up_to = [&](int n) { return weights <= (int64_t)n << 23; };
    const bool exact = exact_operand(a, wdt), odd = a.K % 8 != 0;
    if (a.B <= 4) {
        if (!exact || a.B < 3 || a.N > kRowsFewCols) return false;
        if (a.B == 3) return up_to(4);
        if (wdt != kI8) return !odd || up_to(14);
        return up_to(odd ? 9 : 28);
    }
    return wdt != kI8 || a.B > 6 || !odd || exact || up_to(10);
}

// The gate|up launch of a block with centred inputs of the operand's type.  us per block, two- to four-slot or general kernels / here: 4 tokens 1408 -> 6656
// fp16 26.9 / 22.5, 4224 -> 14400 bf16 79.4 / 68.8, 4096 -> 11008 59.7 / 56.4 (90 and 95 % 44.7 / 42.6, 40.9 / 42.4); 3 tokens 3328 -> 2368 23.9 / 19.6, 5504 -> 12192 76.3 / 69.9
// (51.3 / 51.1, 46.0 / 48.0).  Not beyond one round of tiles (2280 -> 19032, 4 tokens, 59.6 / 62.0; 3840 -> 22864, 3 tokens at 94 %, 48.7 / 55.6).
// Two tokens: small layers (2176 -> 4880 bf16 21.8 / 21.1, 3264 -> 4448 24.7 / 22.4, at 90 % 19.5 / 19.5), and short inputs into many columns, whose tiles
// fill the chip in one split, nothing handed over, while the gains at 40, 70 and 90 % add up or nearly (as in rows_pay).  At 40, 70 and 90 %, to 512 outputs (tiles: gate|up
// columns / 128): bf16 1024 channels, 224 tiles 21.9 / 18.2, 18.4 / 15.4, 15.6 / 14.4; 2048, 132 tiles 23.0 / 22.4, 19.7 / 18.3, 16.4 / 17.2, 224 tiles 29.3 / 27.8, 24.0 / 21.3, 18.8 / 19.2; 3072, 200 tiles
// 35.2 / 33.3, 27.2 / 25.7, 19.8 / 22.1; beyond 3072, 172 tiles 32.6 / 31.5, 25.9 / 25.5, 19.8 / 21.7, 4096, 224 tiles 44.8 / 43.8, 33.0 / 31.5, 22.4 / 26.8; int8 256 channels, 104 tiles 14.1 / 11.2, 13.8 /
// 10.9, 13.2 / 10.6; 1024, 104 tiles 16.2 / 14.4, 15.1 / 14.1, 14.2 / 13.8; 1536, 132 tiles 17.4 / 16.1, 16.5 / 16.0, 14.8 / 15.5; 2048, 224 tiles 21.5 / 20.0, 18.9 / 18.8, 16.5 / 18.2; beyond 2048, 150 tiles 19.7 /
// 18.6, 17.7 / 18.0, 15.5 / 17.4; whole blocks 3072 -> 14336 29.1 / 27.2, 23.8 / 25.7, 19.9 / 23.6, 4096 -> 14336 33.1 / 31.9, 26.4 / 28.9, 21.4 / 26.8.
bool rows_pay_gating(const GemvArgs& a, int wdt) {
    int splits = 0;
    if (!exact_operand(a, wdt) || a.N > kRowsFewCols || !gemm_rows_plans(a, wdt, kRowsCodes, kFuseSwiglu, &splits)) return false;
    if (a.B > 2) return true;
    if (wdt == kI8) return splits == 1 && a.K <= 2048 && a.N >= (int64_t)10 * a.K;
    return (int64_t)a.K * a.N <= ((int64_t)1 << 25) || (splits == 1 && a.N >= (int64_t)8 * a.K);
}

// The interval of magnitude codes that the pruner keeps: [lo, lo + len) of the 16-bit patterns without their sign.
void keep_codes(const GemvArgs& a, uint32_t* lo, uint32_t* len) {
    if (a.mode == kModeDense) {
        *lo = 0;
        *len = 0x8000;
        return;
    }
    union { float f; uint32_t u; } t;
    t.f = a.tau;
    uint32_t code = (t.u & 0x7fffffffu) >> 16;  // the largest bf16 that is not above tau
    uint32_t inf = 0x7f80;
    if (a.xdt == kF16) {
        const float tau = t.f < 0.f ? 0.f : t.f;  // (-0)
        inf = 0x7c00;
        if (tau >= 65504.f) {
            code = 0x7bff;
        } else if (tau < 6.103515625e-05f) {
            code = (uint32_t)(tau * 16777216.f);  // multiples of 2^-24
        } else {
            const uint32_t u = t.u & 0x7fffffffu;
            code = ((u >> 23) - 112u) << 10 | ((u >> 13) & 0x3ffu);
        }
    }
    *lo = code + 1;
    *len = inf - code;
}

template <int WDT, int FUSE, int SRC, bool RAGGED, int SLOTS = kMfmaTokens>
static int launch_rows_kernel(const GemvArgs& a, hipStream_t stream) {
    constexpr size_t lds = kHdrBytes + (size_t)sum_floats(WDT) * 4 +
                           (FUSE == kFuseSwiglu ? (size_t)kMfmaTokens * 16 * Vec<WDT>::kElems * 4 : 0);
    static_assert(lds <= kInlineLdsBudget && 2 * lds <= 160 * 1024, "two workgroups per compute unit");
    if (lds > 64 * 1024) {
        // more dynamic LDS than the default limit: ask once per kernel and device
        constexpr int kMaxDevices = 64;
        static std::atomic<bool> asked[kMaxDevices];
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SCAP_ERR_HIP;
        if (!asked[dev].load(std::memory_order_acquire)) {
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_rows_kernel<WDT, FUSE, SRC, RAGGED, SLOTS>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kInlineLdsBudget) != hipSuccess)
                return SCAP_ERR_HIP;
            asked[dev].store(true, std::memory_order_release);
        }
    }
    hipLaunchKernelGGL((gemm_rows_kernel<WDT, FUSE, SRC, RAGGED, SLOTS>), dim3((unsigned)(a.S * a.T)), dim3(kInlineWaves * kWave), lds, stream, a);
    return hipGetLastError() == hipSuccess ? SCAP_OK : SCAP_ERR_HIP;
}

template <int WDT, int FUSE, int SLOTS>
static int launch_codes(const GemvArgs& a, hipStream_t stream) {
    return a.K % 8 == 0 ? launch_rows_kernel<WDT, FUSE, kRowsCodes, false, SLOTS>(a, stream)
                        : launch_rows_kernel<WDT, FUSE, kRowsCodes, true, SLOTS>(a, stream);
}

template <int FUSE, int SLOTS = kMfmaTokens>
static int launch_codes_any(const GemvArgs& a, int wdt, hipStream_t stream) {
    if (wdt == kBF16) return launch_codes<kBF16, FUSE, SLOTS>(a, stream);
    if (wdt == kF16) return launch_codes<kF16, FUSE, SLOTS>(a, stream);
    if constexpr (SLOTS != 4) {  // (int8 blocks of 3-4 tokens leave planes)
        if (wdt == kI8Half) return launch_codes<kI8Half, FUSE, SLOTS>(a, stream);
    }
    return SCAP_ERR_CONFIG;
}

template <int WDT, int FUSE>
static int launch_centre(const GemvArgs& a, hipStream_t stream) {
    return a.K % 8 == 0 ? launch_rows_kernel<WDT, FUSE, kRowsCentre, false>(a, stream) : launch_rows_kernel<WDT, FUSE, kRowsCentre, true>(a, stream);
}

template <int FUSE>
static int launch_centre_any(const GemvArgs& a, int wdt, hipStream_t stream) {
    if (wdt == kBF16) return launch_centre<kBF16, FUSE>(a, stream);
    if (wdt == kF16) return launch_centre<kF16, FUSE>(a, stream);
    return wdt == kI8Half ? launch_centre<kI8Half, FUSE>(a, stream) : SCAP_ERR_CONFIG;
}

static int launch_planes_any(const GemvArgs& a, int wdt, hipStream_t stream) {
    if (wdt == kBF16) return launch_rows_kernel<kBF16, kFusePlain, kRowsPlanes, false>(a, stream);
    if (wdt == kF16) return launch_rows_kernel<kF16, kFusePlain, kRowsPlanes, false>(a, stream);
    if (wdt == kI8Half) return launch_rows_kernel<kI8Half, kFusePlain, kRowsPlanes, false>(a, stream);
    return wdt == kI8 ? launch_rows_kernel<kI8, kFusePlain, kRowsPlanes, false>(a, stream) : SCAP_ERR_CONFIG;
}

// K split: fills a.T, a.Kc, a.S (and the list segmentation); kc: the caller's rows per workgroup, or 0.  SCAP_ERR_SHAPE where the
// layer has more tiles than there are arrival counters.
//
// The cost of a split in rows of one workgroup at the rate of a full chip.  Nothing but the weight buffer's offsets bounds a piece
// (no inputs in LDS), and a launch of fewer workgroups than compute units is not slower for it until a unit asks for more than it can
// take: 46 GB/s where its share of a full chip's stream is 25 (a sweep that reads 256-byte pieces with 32 / 64 / 128 / 192 / 224 / 256 workgroups:
// 1.5 / 2.8 / 5.1 / 6.0 / 6.3 / 6.1 TB/s): `part`, in a further round with less to win, since units that run two workgroups set its end.  One split hands
// nothing over (`hand`, `split`); a gating launch's hand-over is the dearer one: one ticket a workgroup, and the last arrival fetches all tokens' sums before
// it gates them.  `round`: a workgroup's prologue and reduction in each further round, less where two share a unit.  One set of constants, fitted to 2200
// sweeps of the splits over 196 layers, even and odd lengths, codes, centred inputs, planes and gating launches, both weight types, 4-13 tokens at 50-90 %.  The split
// chosen is above the best one by, on average, 16-bit / int8: plain codes 0.7 / 0.5 %, gating 0.4 / 0.3 %, centred 0.6 / 0.6 %, odd lengths 0.5 / 1.0 %, planes 0.5 / 0.2 %; the worst are
// 10-14 %, at 90 % (7168 x 6656 bf16, 5 tokens, 4 splits 13.8 / 9 12.3).  us at the split chosen / others, at 50 %: 4096 x 28672 bf16, 12 tokens, S = 1 43.6 / S = 2 48.2; 8192 x 28672 bf16,
// 12 tokens, 1 84.6 / 2 90.0, int8, 5 tokens, 1 48.8 / 2 51.0; 7808 x 13184 bf16, 12 tokens at 70 %, 2 32.5 / 4 37.2, as gate|up launch of a block 2 40.9 / 4 44.1, int8, 5 tokens, 2 29.6 / 4
// 30.7; 14336 x 4096 bf16, 12 tokens, 8 25.0 / 7 26.9 / 9 32.3; 4096 x 22016 bf16, 5 tokens, 4 35.0 / 1 36.2 / 2 39.6;
// 4096 x 11008 int8, 5 tokens, 5 12.8 / 2 14.4 / 3 15.4; 2048 x 20480 int8, 5 tokens, 3 12.6 / 1 14.3; 256 x 8192 bf16, 5 tokens, 1 4.5 / 4 5.0; beyond 256
// tiles 4096 x 49152 int8, 5 tokens, 2 42.0 / 1 46.9, 2048 x 45056 bf16 2 35.0 / 1 37.7, 4096 x 65536 bf16 1 83.8 / 2 85.4.
// int8 weights run in 8-byte lanes (128-column tiles; 5-16 tokens at 50-70 %, 16-byte / 8-byte lanes: 14336 x 4096 18.0 / 16.0, 4096 x
// 28672 27.3 / 25.9, 4096 x 4096 10.7 / 8.1); *wdt becomes kI8Half.  Planes also in 16-byte lanes, where there are more narrow tiles than
// arrival counters.
static int plan_rows(GemvArgs& a, int* wdt, int src, int fuse, int kc) {
    const bool i8 = *wdt == kI8;
    int tile = kMfmaTile;
    if (i8) {
        if ((a.N + tile - 1) / tile <= kMaxTiles)
            *wdt = kI8Half;
        else if (src == kRowsPlanes)
            tile = 2 * kMfmaTile;
    }
    a.T = (a.N + tile - 1) / tile;
    // Centred inputs of layers of more tiles than compute units stay on the staged-tile kernel.  Over 16-bit weights (144-157 registers, one
    // workgroup per unit) neither is the faster one throughout (us at 50 and 90 %, there / here: 4096 x 40000 bf16, 5 tokens, 61.9 / 61.4, 34.7 / 37.1, 2047 x
    // 40000 37.2 / 38.4, 25.9 / 29.4, 1024 x 65536 26.5 / 25.1, 14.3 / 15.8, but 4096 x 57344 87.2 / 81.9, 48.6 / 43.5, 512 x 40000 16.0 / 12.4, 12.8 / 9.0).  Over
    // int8 weights (110-125 registers, two per unit) the limit is the same one and not the best: 8 tokens 4096 x 40000 48.2 / 47.6, 35.8 / 34.9, 1024 x 36000
    // 20.3 / 17.8, 16.8 / 14.0, 1024 x 65536 18.0 / 16.1, 13.7 / 13.9.
    if (a.T > (src == kRowsCentre ? 256 : kMaxTiles)) return SCAP_ERR_SHAPE;
    const int64_t row_bytes = (int64_t)a.N * (i8 ? 1 : 2);
    const int64_t kc_max = (((int64_t)1 << 31) / row_bytes - 2 * kWave) / kWave * kWave;
    int64_t s_max = (int64_t)(partial_capacity(a.N) / ((size_t)a.T * tile));
    if (a.B <= kWideTokens) s_max /= 2;
    if (s_max > kMaxSplits) s_max = kMaxSplits;
    if (kc == 0) {
        const int split = 12, hand = fuse == kFuseSwiglu ? 280 : 130;
        const int round = rows_resident(*wdt, src, src != kRowsPlanes && a.K % 8 != 0) == 2 ? 125 : 300;
        double best = 0.0;
        for (int64_t sp = 1; sp <= s_max; ++sp) {
            const int64_t c = (int64_t)align_up((size_t)((a.K + sp - 1) / sp), kWave);
            if (c > kc_max) continue;
            const int64_t s = (a.K + c - 1) / c, n = s * a.T;
            auto part = [&](int64_t m) {
                const double x = (double)m / 256.0;
                return m == 0 ? 0.0 : std::max(0.55, n <= 256 ? 0.45 + 0.55 * x + 0.1 * x * (1.0 - x) : 0.4 + 0.6 * x);
            };
            const double cost = (double)c * ((double)(n / 256) + part(n % 256)) + (double)(round * ((n + 255) / 256 - 1) + split * s) + (s > 1 ? hand : 0);
            if (best == 0.0 || cost < best) {
                best = cost;
                kc = (int)c;
            }
            if (c == kWave) break;
        }
        if (kc == 0) return SCAP_ERR_SHAPE;
    }
    if (kc % kWave != 0) return SCAP_ERR_CONFIG;
    a.S = (a.K + kc - 1) / kc;
    if (kc > kc_max || a.S > s_max) return SCAP_ERR_SHAPE;
    a.Kc = kc;
    a.Kl = a.Kc;
    a.Sl = a.S;
    return SCAP_OK;
}

bool gemm_rows_plans(const GemvArgs& a_in, int wdt, int src, int fuse, int* splits) {
    GemvArgs a = a_in;
    if (plan_rows(a, &wdt, src, fuse, 0) != SCAP_OK) return false;
    if (splits) *splits = a.S;
    return true;
}

int launch_gemm_rows(const GemvArgs& a_in, int wdt, int src, int fuse, int kc, hipStream_t stream) {
    GemvArgs a = a_in;
    if (a.B < 1 || a.B > kMfmaTokens || (src == kRowsCodes && !exact_operand(a, wdt))) return SCAP_ERR_CONFIG;
    const int rc = plan_rows(a, &wdt, src, fuse, kc);
    if (rc != SCAP_OK) return rc;
    if (src == kRowsPlanes) {
        a.mode = kModeSparse;  // (the planes hold what is kept)
        a.x = reinterpret_cast<const uint16_t*>(a.zl_d);
        a.x_pitch = plane_pitch(a.K);
        return fuse == kFusePlain ? launch_planes_any(a, wdt, stream) : SCAP_ERR_CONFIG;
    }
    a.x_pitch = a.K;
    if (src == kRowsCentre) return fuse == kFuseSwiglu ? launch_centre_any<kFuseSwiglu>(a, wdt, stream) : launch_centre_any<kFusePlain>(a, wdt, stream);
    keep_codes(a, &a.keep_lo, &a.keep_len);
    if (fuse != kFuseSwiglu) return launch_codes_any<kFusePlain>(a, wdt, stream);
    // (a gating launch leaves planes where it is told where the tails go, else the lists of 2-4 tokens)
    if (a.zl_lo != nullptr) return launch_codes_any<kFuseSwiglu>(a, wdt, stream);
    if (a.B > 4) return SCAP_ERR_CONFIG;
    return a.B == 2 ? launch_codes_any<kFuseSwiglu, 2>(a, wdt, stream) : launch_codes_any<kFuseSwiglu, 4>(a, wdt, stream);
}

}  // namespace scap
