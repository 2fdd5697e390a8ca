// Batched sparse FC on the matrix cores in ONE launch (gfx950 MFMA) with lists in LDS: what the row-step kernel
// (scap_gemm_rows.hip) does not take -- centred inputs over more column tiles than compute units; over int8 weights 3-4 tokens that rows_pay
// refuses, 5-6 tokens over large layers of an odd input length, blocks of 3-4 tokens that rows_pay_gating refuses -- and calls of 2-4 tokens that name this kernel.
// Two kernels: gemm_inline_kernel (below) keeps per-token value lists in LDS (four token slots; 16 over int8 layers of an odd input length);
// gemm_inline_raw_kernel (further down, 16 token slots) stages the raw input tile instead and forms the centred values when the MFMA operand is assembled.
//
// Workgroup (K split, column tile of 16 lanes x 16 bytes) centres, thresholds and compacts its Kc input
// channels of every token into LDS exactly as the one-token kernel does (SCAP Alg. 3 steps 1-2; per-token
// masks, the union of the masks decides which rows are read, Appendix C), then walks the list in 16-row
// blocks: channel indices and centred values come out of LDS, the weight rows stream from HBM, and the
// products run on the matrix cores (operand layout: scap_mfma_parts.hpp).  gfx950 gives a workgroup up to
// 160 KB of LDS, which holds the list of ~2300 channels for 16 tokens (index + 16 centred values each), so
// the separate union launch of scap_gemm_mfma.hip, its kernel boundary and its lists in memory are not
// needed; that form remains for inputs too long to split into LDS-sized pieces.
//
// The column tile is narrow (128 columns for 16-bit weights, 128 or 256 for int8), so the prologue is repeated by more
// workgroups than in the vector kernel; it is loads from L2 and a few hundred ALU operations per thread
// and costs less than the kernel boundary it replaces.
#include <atomic>
#include <type_traits>

#include "scap_mfma_parts.hpp"

namespace scap {

// FUSE (kFusePlain / kFuseSwiglu / kFuseList) as in the vector kernel: where the inputs come from and what the
// tile's last arrival does with the finished columns (the two launches of the fused SwiGLU block, Alg. 2).
template <int WDT, int BT, int FUSE>
__global__ __launch_bounds__(kInlineWaves* kWave) void gemm_inline_kernel(const GemvArgs a) {
    constexpr int WAVES = kInlineWaves;
    constexpr int ELEMS = Vec<WDT>::kElems;
    constexpr int TILE = 16 * ELEMS;

    extern __shared__ uint4 smem_raw[];
    Lds L = carve_lds<WAVES, BT>(reinterpret_cast<char*>(smem_raw), a.Kc);
    if constexpr (FUSE == kFuseSwiglu) L.fin = L.red + kTreeFloats;  // behind both uses of the reduction buffer
    const int tid = threadIdx.x;
    const int w = uniform(tid >> 6);
    const int lane = tid & 63;
    const int tile = blockIdx.x % a.T;
    const int split = blockIdx.x / a.T;

    // ------------------------------------------------------------------ 1. centre, threshold, compact
    int cnt;
    if constexpr (FUSE == kFuseList)
        cnt = gather_lists<WAVES, BT>(a, split, L);
    else
        cnt = compact_inputs_wide<WAVES, BT, inline_max_chunks(BT)>(a, tile, split, L);
    const int n_blocks = (cnt + kMfmaBlock - 1) / kMfmaBlock;

    // ------------------------------------------------------------------ 2. stream the kept rows
    const int cg = lane & 15;  // column group (B/C index n); also the token whose values this lane supplies (A index m)
    const int kg = lane >> 4;  // row group: list rows 4*kg .. 4*kg+3 of a block
    const int col0 = tile * TILE + cg * ELEMS;
    const uint32_t lane_off = (col0 < a.N) ? (uint32_t)col0 * Vec<WDT>::kBytes : kNoRow;
    const uint32_t row_bytes = (uint32_t)a.N * Vec<WDT>::kBytes;
    const int k0 = split * a.Kc;
    const __amdgpu_buffer_rsrc_t wbuf = weight_rows(a, k0, row_bytes);
    const int tok = cg < BT ? cg : BT - 1;  // token slots past BT carry zeros (read slot BT-1, discard)
    const float* d_tok = L.d + tok * a.Kc;

    f32x4_t acc[ELEMS];
#pragma unroll
    for (int e = 0; e < ELEMS; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // Three stages per wavefront: list entries of block n+2 come out of LDS while the weight rows of block
    // n+1 are in flight and the MFMAs of block n run.  A slot past the end of the list reads LDS at a clamped position
    // and no weights.  16 slots: the loop stops issuing with the last block (see the staged-tile kernel: TAIL).  4 slots: it
    // issues one stage past it, for that loop's second copy of the multiply takes int8 weights from 127 to 183 registers, i.e.
    // to one workgroup per compute unit instead of two (us, that loop / this: 4097 x 17408 int8, 3 tokens, 22.6 / 21.3, 9001 x
    // 9600 24.2 / 22.8, blocks 4096 -> 11008 -> 4096 48.7 / 40.2 and 1024 -> 20480 -> 1024 40.5 / 32.1).
    struct Entries {
        int4 rows;
        float4 d;
        int left;  // valid entries from this lane's first one on (<= 0: none)
    };
    struct Stage {
        uint4 r[4];
        float4 d;
    };
    auto entries = [&](int blk, Entries& en) {  // blk is wave-uniform and may lie past the end
        const int e0 = blk * kMfmaBlock + 4 * kg;
        const int e0c = min(e0, a.Kc - 4);
        en.left = cnt - e0;
        en.rows = *reinterpret_cast<const int4*>(L.idx + e0c);
        en.d = *reinterpret_cast<const float4*>(d_tok + e0c);
    };
    auto issue = [&](const Entries& en, Stage& st) {
        const int rj[4] = {en.rows.x, en.rows.y, en.rows.z, en.rows.w};
        const float dj[4] = {en.d.x, en.d.y, en.d.z, en.d.w};
        float dm[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool ok = j < en.left;
            st.r[j] = load_row_part<WDT>(wbuf, ok ? __umul24((uint32_t)(rj[j] - k0), row_bytes) + lane_off : kNoRow);
            dm[j] = (ok && cg < BT) ? dj[j] : 0.f;
        }
        st.d = make_float4(dm[0], dm[1], dm[2], dm[3]);
    };
    auto compute = [&](const Stage& st) {
        s16x4_t a_hi, a_lo;
        split_operand<WDT>(st.d, a_hi, a_lo);
        mfma_block<WDT>(acc, a_hi, a_lo, st.r);
    };

    if constexpr (BT <= 4) {
        Entries E0, E1;
        Stage A, Bs;
        entries(w, E0);
        entries(w + WAVES, E1);
        issue(E0, A);
        for (int blk = w; blk < n_blocks;) {
            entries(blk + 2 * WAVES, E0);
            issue(E1, Bs);
            compute(A);
            blk += WAVES;
            if (blk >= n_blocks) break;
            entries(blk + 2 * WAVES, E1);
            issue(E0, A);
            compute(Bs);
            blk += WAVES;
        }
    } else if (w < n_blocks) {
        Entries E;
        Stage A, Bs;
        entries(w, E);
        issue(E, A);
        entries(w + WAVES, E);
        int blk = w;
        for (;;) {
            if (blk + WAVES >= n_blocks) break;
            issue(E, Bs);
            entries(blk + 2 * WAVES, E);
            compute(A);
            blk += WAVES;
            if (blk + WAVES >= n_blocks) {
                A = Bs;
                break;
            }
            issue(E, A);
            entries(blk + 2 * WAVES, E);
            compute(Bs);
            blk += WAVES;
        }
        compute(A);
    }

    // ------------------------------------------------------------------ 3. add the wavefronts' sums
    // constants of the column group this thread finishes if its workgroup is the tile's last arrival: fetched behind the
    // reduction (not at the start: no registers for them while the rows stream)
    const ColConst mine = load_col_const<WDT, TILE>(a, tile, tid % (TILE / 4));
    const __amdgpu_buffer_rsrc_t pbuf = partial_buffer<TILE>(a);
    reduce_waves_and_emit<WDT, WAVES, FUSE, WDT != kI8>(a, pbuf, tile, split, acc, L.red, L.fin);  // starts with a barrier: the list is done with

    // ------------------------------------------------------------------ 4. last arrival finishes the tile
    finish_tile<WDT, WAVES, TILE, BT, FUSE>(a, pbuf, tile, L, mine);
}

// ---------------------------------------------------------------------------------------------- staged-tile form
// 16 token slots.  The prologue above costs ~10 us at 16 tokens: 80 two-byte loads per lane,
// ~10 ALU operations per input element and 16 four-byte LDS writes per kept channel, repeated by every column
// tile.  Here the workgroup's input tile is staged as it is (16-byte loads, 16-byte LDS writes), only the union
// list of channels is compacted, and the centred, thresholded value of (token, channel) is formed from the
// staged tile when the matrix-core operand is assembled, in the shadow of the weight stream.  Same arithmetic
// per element (one fp32 subtraction, strict compare), so masks and values are those of the other forms.
// Chunks of 64 channels per wavefront (loads of all of them are in flight at once): 1, 2, 4 or 5 by the workgroup's
// channels; with 5 for all of them the others re-read what was there (4096 x 4096 bf16, 16 tokens: 15.8 -> 14.0 us with 1;
// 4096 x 11008 fp16, 8 tokens: 23.8 -> 22.9 with 2; 4096 x 28672 bf16, 16 tokens: 48.6 -> 46.8 with 4; odd input lengths,
// where an octet is two loads: 5461 x 2744 bf16, 16 tokens, 19.2 -> 13.5 with 1, 4097 x 11008 36.0 -> 26.8 with 2).  Instantiations,
// not a choice made inside: behind such a branch the first test waits for all loads.
constexpr int kRawChunks = 5;
constexpr int kRawPad = 16;    // bytes between token rows of the staged tile: rows start 4 LDS banks apart

__host__ __device__ constexpr size_t raw_tile_bytes(int Kc) { return (size_t)kMfmaTokens * ((size_t)Kc * 2 + kRawPad); }

// bit o of an 8-bit value to bit 8*o (two 4-bit halves: the partial products of a half never share a bit)
__device__ __forceinline__ uint64_t spread_bits_to_bytes(uint32_t v) {
    const uint32_t lo = ((v & 15u) * 0x00204081u) & 0x01010101u;
    const uint32_t hi = ((v >> 4) * 0x00204081u) & 0x01010101u;
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

// Input code (low 16 bits) to fp32 without a branch on the (uniform) activation type: both conversions, bit select.
__device__ __forceinline__ float act_code_to_f32(uint32_t code, uint32_t bf16_sel) {
    const uint32_t as_bf16 = code << 16;
    const uint32_t as_f16 = __float_as_uint(f16_bits_to_f32(code));
    return __uint_as_float((as_bf16 & bf16_sel) | (as_f16 & ~bf16_sel));
}

// One of the two 16-bit inputs of a word, activation type known at compile time.
template <bool BF16X>
__device__ __forceinline__ float word_half_to_f32(uint32_t wd, int half) {
    if constexpr (BF16X)
        return __uint_as_float(half ? (wd & 0xffff0000u) : (wd << 16));
    else
        return f16_bits_to_f32(half ? (wd >> 16) : (wd & 0xffffu));
}

// Stage the tile, build the ascending union list in L.idx.  Lane = (token group tg = lane % 8, octet o = lane / 8
// of 8 channels): it loads tokens tg and tg+8 of its octet and tests its 16 elements; the compare masks are
// scalar registers, so a channel's keep bits over all tokens are one byte of a mask and "kept by any token" is
// a nonzero-byte test.  Everything in the test is straight-line: the instruction count per element is what the
// prologue costs, repeated by every column tile.  Per-token lists and counts (on request, the tile's own tokens) are
// read back from the staged tile with one channel per lane.  Returns the list length; ends with a barrier.
// RAGGED (16-bit weights, int8 in 8-byte lanes): K is not a multiple of 8 -- token rows start at any 2-byte boundary and the last octet is cut.  A template
// argument: the tests for it cost a kernel that does not need them 1 us (14336 x 4096 int8, 12 tokens: 23.3 -> 24.2 us).
// It does not exist for 16-byte int8 lanes.
template <int WAVES, int MAXC, bool SUPERSET, bool RAGGED>
__device__ __forceinline__ int stage_inputs_and_list(const GemvArgs& a, int tile, int split, const Lds& L, char* xs,
                                                     uint32_t xrow) {
    constexpr int BT = kMfmaTokens;
    const int tid = threadIdx.x;
    const int w = uniform(tid >> 6);
    const int lane = tid & 63;
    const int k0 = split * a.Kc;
    const int kend = min(k0 + a.Kc, a.K);
    const uint32_t own = owned_tokens(a, tile);  // tokens whose lists and counts this tile's workgroups leave
    const bool want_idx = a.idx_out != nullptr;
    // dense mode as data, not as control flow: x - 0 is x, and every valid element is kept
    const bool dense = a.mode == kModeDense;
    const float m_eff = dense ? 0.f : a.m;
    const uint32_t bf16_sel = a.xdt == kBF16 ? 0xffffffffu : 0u;
    const uint32_t nan_pair = a.xdt == kBF16 ? 0x7fc07fc0u : 0x7e007e00u;  // two quiet NaNs: never above a threshold
    const int nchunk = (kend - k0 + kWave - 1) / kWave;
    const int cpw = (nchunk + WAVES - 1) / WAVES;
    const int c_begin = min(w * cpw, nchunk);
    const int c_end = min(c_begin + cpw, nchunk);
    const int tg = lane & 7, o = lane >> 3;

    // ---- all loads, branch-free (slots past the end re-read the last octet)
    uint4 xv[MAXC][2];
    if constexpr (!RAGGED) {
#pragma unroll
        for (int j = 0; j < MAXC; ++j) {
            const int kb = min(k0 + (c_begin + j) * kWave + 8 * o, a.K - 8);
#pragma unroll
            for (int r = 0; r < 2; ++r)
                xv[j][r] = *reinterpret_cast<const uint4*>(a.x + (int64_t)min(tg + 8 * r, a.B - 1) * a.K + kb);
        }
    } else {
        // Rows that start anywhere; a token's last octet runs into the next token's row (masked below).  Only the very
        // last octet of x can be cut: it is read from 8 elements before the end like any other load, then once more
        // element by element.
        const int last_octet = (a.K - 1) & ~7, total = a.B * a.K;
#pragma unroll
        for (int j = 0; j < MAXC; ++j) {
            const int kb = min(k0 + (c_begin + j) * kWave + 8 * o, last_octet);
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int p = min(tg + 8 * r, a.B - 1) * a.K + kb;
                xv[j][r] = total >= 8 ? load_octet(a.x + min(p, total - 8)) : make_uint4(0u, 0u, 0u, 0u);
            }
        }
#pragma unroll
        for (int j = 0; j < MAXC; ++j) {
            const int kb = min(k0 + (c_begin + j) * kWave + 8 * o, last_octet);
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int p = min(tg + 8 * r, a.B - 1) * a.K + kb;
                if (p > total - 8) xv[j][r] = load_octet_cut(a.x + p, total - p);
            }
        }
    }
    // ---- stage, test, union mask per chunk
    uint64_t um[MAXC];
    int ucount = 0;
    // The list only decides which rows are READ: what a token contributes is decided again, exactly, when the
    // operand is assembled.  So the list may be a superset of the union.  With many tokens the union is nearly
    // everything (Appendix C: 1 - s^B), and testing 16 tokens per channel to find that out is the larger part
    // of this prologue.  Each wavefront therefore tests its first chunk; if at most 2 of its 64 channels are
    // dropped by every token, it lists its other chunks whole (a few rows read for nothing against three
    // quarters of the tests).  Dense mode lists everything without a test (there that is the exact union).
    // The decision depends on the inputs only, so every column tile of a split takes the same one: the list,
    // and with it the order of every fp32 sum, never depends on which outputs the caller asked for.  When the
    // caller wants the size of the union, which has to be exact, column tile 0 also tests the chunks it lists
    // whole, for the count alone.
    const bool count_exactly = tile == 0 && a.union_nnz_out != nullptr;
    int ecount = 0;  // channels kept by at least one token among those tested (the exact union where all are)
    auto test_chunks = [&](auto bf16x) {
        constexpr bool BF16X = decltype(bf16x)::value;
        // stage chunk slot j and list all its channels (wave-uniform)
        auto list_whole = [&](int j) {
            const int c = c_begin + j;
            um[j] = 0;
            if (c < c_end) {
                const int nval = min((int)kWave, kend - (k0 + c * kWave));
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    if (r == 1 && a.B <= 8) break;
                    *reinterpret_cast<uint4*>(xs + (size_t)(tg + 8 * r) * xrow + (size_t)(c * kWave + 8 * o) * 2) = xv[j][r];
                }
                um[j] = nval >= kWave ? ~0ull : ((1ull << nval) - 1ull);
                ucount += nval;
            }
        };
        // stage chunk slot j and list the channels kept by at least one token
        auto test_slot = [&](int j) {
            const int c = c_begin + j;
            um[j] = 0;
            if (c < c_end) {  // wave-uniform
                const int nvo = kend - (k0 + c * kWave + 8 * o);  // elements of this lane's octet that exist
                const bool oct_ok = nvo > 0;
                const int nvc = kend - (k0 + c * kWave);  // the same for the chunk
                const bool cut_chunk = RAGGED && nvc < (int)kWave;  // wave-uniform
                uint64_t kp[8];  // lane masks (bit tg + 8*o): channel 8*o+e kept by token tg or tg+8
                uint64_t any_ok = 0;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    if (r == 1 && a.B <= 8) break;  // at most 8 tokens: the second token of every lane does not exist
                    const bool ok = oct_ok && (tg + 8 * r) < a.B;
                    any_ok |= __ballot(ok);
                    // an element that does not exist becomes a NaN: the strict compare drops it
                    uint4 v = xv[j][r];
                    v = make_uint4(ok ? v.x : nan_pair, ok ? v.y : nan_pair, ok ? v.z : nan_pair, ok ? v.w : nan_pair);
                    if (cut_chunk) {
                        uint32_t* vw = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            if (nvo <= 2 * q) vw[q] = nan_pair;
                            else if (nvo == 2 * q + 1) vw[q] = (vw[q] & 0xffffu) | (nan_pair & 0xffff0000u);
                        }
                    }
                    const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float dv = word_half_to_f32<BF16X>(wd[e >> 1], e & 1) - m_eff;  // one fp32 subtraction
                        const uint64_t kb = __ballot(fabsf(dv) > a.tau);                      // strict; NaN is pruned
                        kp[e] = r == 0 ? kb : (kp[e] | kb);
                    }
                    *reinterpret_cast<uint4*>(xs + (size_t)(tg + 8 * r) * xrow + (size_t)(c * kWave + 8 * o) * 2) = v;
                }
                const uint64_t dense_ok = dense ? any_ok : 0ull;  // dense mode keeps every element that exists
                uint64_t u = 0;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    // byte o of the mask holds the eight token groups: nonzero byte -> bit 8*o+7 -> bit 8*o+e
                    const uint64_t v = kp[e] | dense_ok;
                    const uint64_t nz = (((v & 0x7f7f7f7f7f7f7f7full) + 0x7f7f7f7f7f7f7f7full) | v) & 0x8080808080808080ull;
                    u |= nz >> (7 - e);
                }
                if (cut_chunk) u &= (1ull << nvc) - 1ull;  // (dense mode keeps whole octets above)
                um[j] = u;  // bit i: channel i of the chunk is kept by some token
                ucount += __popcll(u);
                ecount += __popcll(u);
            }
        };
        if constexpr (SUPERSET) {
            if (dense) {  // every element that exists is kept: the list is all valid channels, exactly
#pragma unroll
                for (int j = 0; j < MAXC; ++j) list_whole(j);
                ecount = ucount;
                return;
            }
            test_slot(0);
            const int nval0 = c_begin < c_end ? min((int)kWave, kend - (k0 + c_begin * kWave)) : 0;
            if (__popcll(um[0]) + 2 >= nval0) {  // wave-uniform
                if (count_exactly) {
                    const int listed = ucount;
#pragma unroll
                    for (int j = 1; j < MAXC; ++j) test_slot(j);  // adds to ecount; the list is rebuilt below
                    ucount = listed;
                }
#pragma unroll
                for (int j = 1; j < MAXC; ++j) list_whole(j);
            } else {
#pragma unroll
                for (int j = 1; j < MAXC; ++j) test_slot(j);
            }
        } else {
#pragma unroll
            for (int j = 0; j < MAXC; ++j) test_slot(j);
        }
    };
    if (a.xdt == kBF16)
        test_chunks(std::true_type{});
    else
        test_chunks(std::false_type{});
    if (lane == 0) {
        L.hdr[w] = ucount;
        L.hdr[(2 + BT) * WAVES + w] = ecount;  // behind the per-token rows and the flag row
    }
    __syncthreads();  // counts published, tile staged

    // ---- per-token counts (on request, the tile's own tokens): one channel per lane from the staged tile
    auto kept_by = [&](int j, int b) {
        const int c = min(c_begin + j, nchunk - 1);
        const int k = k0 + (c_begin + j) * kWave + lane;
        const bool valid = (c_begin + j) < c_end && k < kend && b < a.B;
        const uint32_t code = *reinterpret_cast<const uint16_t*>(xs + (size_t)min(b, a.B - 1) * xrow + (size_t)(c * kWave + lane) * 2);
        const float dv = act_code_to_f32(code, bf16_sel) - m_eff;
        return valid & (dense | (fabsf(dv) > a.tau));
    };
    if (own) {
        for (int b = 0; b < BT; ++b) {
            if (!((own >> b) & 1u)) continue;
            int tc = 0;
#pragma unroll
            for (int j = 0; j < MAXC; ++j) tc += __popcll(__ballot(kept_by(j, b)));
            if (lane == 0) L.hdr[(1 + b) * WAVES + w] = tc;
        }
        __syncthreads();
    }
    int ubase = 0, cnt = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
        const int v = L.hdr[i];
        if (i < w) ubase += v;
        cnt += v;
    }
    cnt = uniform(cnt);
    ubase = uniform(ubase);
    // ---- place the union list
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
        if ((um[j] >> lane) & 1ull) L.idx[ubase + lanes_below(um[j])] = k0 + (c_begin + j) * kWave + lane;
        ubase += __popcll(um[j]);
    }
    if (own) {
        for (int b = 0; b < BT; ++b) {
            if (!((own >> b) & 1u)) continue;
            int tbase = 0, ttotal = 0;
            for (int i = 0; i < WAVES; ++i) {
                const int v = L.hdr[(1 + b) * WAVES + i];
                if (i < w) tbase += v;
                ttotal += v;
            }
#pragma unroll
            for (int j = 0; j < MAXC; ++j) {
                const bool kb = kept_by(j, b);
                const uint64_t tb = __ballot(kb);
                if (want_idx && kb)
                    store_dev(&a.idx_out[(int64_t)b * a.K + k0 + tbase + lanes_below(tb)], k0 + (c_begin + j) * kWave + lane);
                tbase += __popcll(tb);
            }
            if (tid == 0) store_dev(&a.seg_cnt[b * a.Sl + split], ttotal);
        }
    }
    if (tile == 0 && tid == 0) {  // size of the union: the list's length, or the exact count where the list is a superset
        int exact = 0;
        for (int i = 0; i < WAVES; ++i) exact += L.hdr[(2 + BT) * WAVES + i];
        store_dev(&a.seg_cnt[a.B * a.Sl + split], count_exactly ? exact : cnt);
    }
    __syncthreads();
    return cnt;
}

// ALONE: one workgroup per compute unit (int8 weights in 16-byte lanes, 194 registers); the others leave room for two.
template <int WDT, int FUSE, bool ALONE, bool RAGGED, int MAXC>
__global__ __launch_bounds__(kInlineWaves* kWave, ALONE ? 2 : 4) void gemm_inline_raw_kernel(const GemvArgs a) {
    constexpr int WAVES = kInlineWaves;
    constexpr int BT = kMfmaTokens;
    constexpr int ELEMS = Vec<WDT>::kElems;
    constexpr int TILE = 16 * ELEMS;

    extern __shared__ uint4 smem_raw[];
    Lds L = carve_lds<WAVES, BT>(reinterpret_cast<char*>(smem_raw), a.Kc);
    if constexpr (FUSE == kFuseSwiglu) L.fin = L.red + kTreeFloats;
    char* xs = reinterpret_cast<char*>(L.idx + a.Kc);  // staged inputs [16][Kc * 2 + pad] in place of the value lists
    const uint32_t xrow = (uint32_t)a.Kc * 2 + kRawPad;
    const int tid = threadIdx.x;
    const int w = uniform(tid >> 6);
    const int lane = tid & 63;
    const int tile = blockIdx.x % a.T;
    const int split = blockIdx.x / a.T;
    const int k0 = split * a.Kc;
    const bool dense = a.mode == kModeDense;
    const float m_eff = dense ? 0.f : a.m;  // dense mode: x - 0 is x
    const uint32_t bf16_sel = a.xdt == kBF16 ? 0xffffffffu : 0u;

    // ------------------------------------------------------------------ 1. stage the inputs, list the union
    // int8 weights in 16-byte lanes: 256-column tiles, so half as many workgroups repeat a split's prologue and a wavefront
    // has two chunks; listing supersets measured no gain there (and 0.14 us lost to the extra code)
    const int cnt = stage_inputs_and_list<WAVES, MAXC, WDT != kI8, RAGGED>(a, tile, split, L, xs, xrow);
    const int n_blocks = (cnt + kMfmaBlock - 1) / kMfmaBlock;

    // ------------------------------------------------------------------ 2. stream the kept rows
    const int cg = lane & 15;  // column group (B/C index n); also the token whose values this lane supplies (A index m)
    const int kg = lane >> 4;  // row group: list rows 4*kg .. 4*kg+3 of a block
    const int col0 = tile * TILE + cg * ELEMS;
    const uint32_t lane_off = (col0 < a.N) ? (uint32_t)col0 * Vec<WDT>::kBytes : kNoRow;
    const uint32_t row_bytes = (uint32_t)a.N * Vec<WDT>::kBytes;
    const __amdgpu_buffer_rsrc_t wbuf = weight_rows(a, k0, row_bytes);
    const bool tok_ok = cg < a.B;  // token slots past B carry zeros
    const char* xs_tok = xs + (size_t)min(cg, a.B - 1) * xrow;

    f32x4_t acc[ELEMS];
#pragma unroll
    for (int e = 0; e < ELEMS; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // Four stages per wavefront: list rows of block n+3 and staged inputs of block n+2 come out of LDS while the weight
    // rows of block n+1 are in flight and the MFMAs of block n run.  A slot past the end of the list reads LDS at a
    // clamped position and no weights (zeros).  The loop runs as long as there is a next block to fetch and the last one
    // is multiplied behind it (TAIL): a stage of loads past the end, even of lanes that fetch nothing, costs a wavefront
    // as much time in the load pipe as a stage of rows (removing the one stage that the loop issued in vain: 1024 x 4096
    // bf16, 16 tokens, 9.7 -> 9.1 us, 4096 x 4096 13.8 -> 13.1; a second one added 1.2 us).  Over 16-bit
    // weights the copy of the stage behind the loop does not fit the 128 registers of two workgroups per unit.
    constexpr bool TAIL = is_int8(WDT);
    struct Rows {
        int4 rows;
        int left;  // valid entries from this lane's first one on (<= 0: none)
    };
    struct Entries {
        int4 rows;
        uint32_t code[4];
        int left;
    };
    struct Stage {
        uint4 r[4];
        float4 d;
    };
    auto rows_of = [&](int blk, Rows& rw) {  // blk is wave-uniform and may lie past the end
        const int e0 = blk * kMfmaBlock + 4 * kg;
        rw.left = cnt - e0;
        rw.rows = *reinterpret_cast<const int4*>(L.idx + min(e0, a.Kc - 4));
    };
    auto codes_of = [&](const Rows& rw, Entries& en) {
        const int rj[4] = {rw.rows.x, rw.rows.y, rw.rows.z, rw.rows.w};
        en.rows = rw.rows;
        en.left = rw.left;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int ch = j < rw.left ? rj[j] - k0 : 0;  // list entries lie in [k0, k0 + Kc)
            en.code[j] = *reinterpret_cast<const uint16_t*>(xs_tok + (size_t)ch * 2);
        }
    };
    auto issue = [&](const Entries& en, Stage& st) {
        const int rj[4] = {en.rows.x, en.rows.y, en.rows.z, en.rows.w};
        float dm[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool ok = j < en.left;
            st.r[j] = load_row_part<WDT>(wbuf, ok ? __umul24((uint32_t)(rj[j] - k0), row_bytes) + lane_off : kNoRow);
            const float dv = act_code_to_f32(en.code[j], bf16_sel) - m_eff;  // one fp32 subtraction
            const bool keep = ok & tok_ok & (dense | (fabsf(dv) > a.tau));    // strict; NaN is pruned
            dm[j] = keep ? dv : 0.f;
        }
        st.d = make_float4(dm[0], dm[1], dm[2], dm[3]);
    };
    auto compute = [&](const Stage& st) {
        s16x4_t a_hi, a_lo;
        split_operand<WDT>(st.d, a_hi, a_lo);
        mfma_block<WDT>(acc, a_hi, a_lo, st.r);
    };
    if (w < n_blocks) {
        Rows R;
        Entries E;
        Stage A, Bs;
        rows_of(w, R);
        codes_of(R, E);
        rows_of(w + WAVES, R);
        issue(E, A);
        codes_of(R, E);
        rows_of(w + 2 * WAVES, R);
        if constexpr (TAIL) {
            int blk = w;
            for (;;) {
                if (blk + WAVES >= n_blocks) break;
                issue(E, Bs);
                codes_of(R, E);
                rows_of(blk + 3 * WAVES, R);
                compute(A);
                blk += WAVES;
                if (blk + WAVES >= n_blocks) {
                    A = Bs;
                    break;
                }
                issue(E, A);
                codes_of(R, E);
                rows_of(blk + 3 * WAVES, R);
                compute(Bs);
                blk += WAVES;
            }
            compute(A);
        } else {
            for (int blk = w; blk < n_blocks;) {
                issue(E, Bs);
                codes_of(R, E);
                rows_of(blk + 3 * WAVES, R);
                compute(A);
                blk += WAVES;
                if (blk >= n_blocks) break;
                issue(E, A);
                codes_of(R, E);
                rows_of(blk + 3 * WAVES, R);
                compute(Bs);
                blk += WAVES;
            }
        }
    }

    // ------------------------------------------------------------------ 3. add the wavefronts' sums
    // constants of the column group this thread finishes if its workgroup is the tile's last arrival: fetched behind the
    // reduction (not at the start: no registers for them while the rows stream)
    const ColConst mine = load_col_const<WDT, TILE>(a, tile, tid % (TILE / 4));
    const __amdgpu_buffer_rsrc_t pbuf = partial_buffer<TILE>(a);
    reduce_waves_and_emit<WDT, WAVES, FUSE, WDT != kI8>(a, pbuf, tile, split, acc, L.red, L.fin);  // starts with a barrier: the tile is done with

    // ------------------------------------------------------------------ 4. last arrival finishes the tile
    finish_tile<WDT, WAVES, TILE, BT, FUSE>(a, pbuf, tile, L, mine);
}

template <int WDT, int BT, int FUSE>
static int launch_inline(const GemvArgs& a, size_t lds, hipStream_t stream) {
    if (lds > kInlineLdsBudget) return SCAP_ERR_SHAPE;
    if (lds > 64 * 1024) {
        // more dynamic LDS than the default limit: ask once per kernel and device
        constexpr int kMaxDevices = 64;
        static std::atomic<bool> asked[kMaxDevices];
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SCAP_ERR_HIP;
        if (!asked[dev].load(std::memory_order_acquire)) {
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_inline_kernel<WDT, BT, FUSE>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kInlineLdsBudget) != hipSuccess)
                return SCAP_ERR_HIP;
            asked[dev].store(true, std::memory_order_release);
        }
    }
    hipLaunchKernelGGL((gemm_inline_kernel<WDT, BT, FUSE>), dim3((unsigned)(a.S * a.T)), dim3(kInlineWaves * kWave), lds,
                       stream, a);
    return hipGetLastError() == hipSuccess ? SCAP_OK : SCAP_ERR_HIP;
}

template <int WDT, int FUSE, bool ALONE, bool RAGGED, int MAXC>
static int launch_inline_raw_chunks(const GemvArgs& a, size_t lds, hipStream_t stream) {
    if (lds > kInlineLdsBudget) return SCAP_ERR_SHAPE;
    if (lds > 64 * 1024) {
        constexpr int kMaxDevices = 64;
        static std::atomic<bool> asked[kMaxDevices];
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SCAP_ERR_HIP;
        if (!asked[dev].load(std::memory_order_acquire)) {
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_inline_raw_kernel<WDT, FUSE, ALONE, RAGGED, MAXC>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kInlineLdsBudget) != hipSuccess)
                return SCAP_ERR_HIP;
            asked[dev].store(true, std::memory_order_release);
        }
    }
    hipLaunchKernelGGL((gemm_inline_raw_kernel<WDT, FUSE, ALONE, RAGGED, MAXC>), dim3((unsigned)(a.S * a.T)),
                       dim3(kInlineWaves * kWave), lds, stream, a);
    return hipGetLastError() == hipSuccess ? SCAP_OK : SCAP_ERR_HIP;
}

template <int WDT, int FUSE, bool ALONE, bool RAGGED>
static int launch_inline_raw(const GemvArgs& a, size_t lds, hipStream_t stream) {
    if (a.Kc <= 1 * kInlineWaves * kWave) return launch_inline_raw_chunks<WDT, FUSE, ALONE, RAGGED, 1>(a, lds, stream);
    if (a.Kc <= 2 * kInlineWaves * kWave) return launch_inline_raw_chunks<WDT, FUSE, ALONE, RAGGED, 2>(a, lds, stream);
    if constexpr (!RAGGED || is_int8(WDT)) {
        if (a.Kc <= 4 * kInlineWaves * kWave) return launch_inline_raw_chunks<WDT, FUSE, ALONE, RAGGED, 4>(a, lds, stream);
    }
    // (the gating launch over narrow int8 tiles: pieces of at most four chunks, plan_inline)
    if constexpr (WDT == kI8Half && FUSE == kFuseSwiglu)
        return SCAP_ERR_SHAPE;
    else
        return launch_inline_raw_chunks<WDT, FUSE, ALONE, RAGGED, kRawChunks>(a, lds, stream);
}

// 16 token slots: the staged-tile kernel; 4 slots: the value-list kernel (not fp16 weights: 2-4 tokens stay on the vector kernels).
// An input length that is not a multiple of 8: the staged-tile kernel too (5461 x 2744 bf16, 8 tokens 19.7 -> 17.7 us
// per call, block 4095 -> 6144 -> 4096 56.0 -> 51.9), but not with int8 weights in 16-byte lanes, where a wavefront has
// only two chunks to test and the value lists stay 3 % faster (5461 x 2752, 16 tokens 23.3 against 24.0).
__host__ constexpr bool staged_tile(int wdt, int K) { return wdt != kI8 || K % 8 == 0; }

template <int WDT, int FUSE>
static int launch_inline_wdt(const GemvArgs& a, int bt, size_t lds, hipStream_t stream) {
    if constexpr (FUSE != kFuseList) {  // (lists of a gated product have four slots: batches leave planes, scap_gemm_rows.hip)
        if (bt == kMfmaTokens) {
            if constexpr (WDT == kI8) {
                if (!staged_tile(WDT, a.K)) return launch_inline<WDT, kMfmaTokens, FUSE>(a, lds, stream);
            } else {
                if (a.K % 8 != 0) return launch_inline_raw<WDT, FUSE, false, true>(a, lds, stream);
            }
            return launch_inline_raw<WDT, FUSE, WDT == kI8, false>(a, lds, stream);
        }
    }
    if constexpr (WDT == kI8 || (WDT == kBF16 && FUSE == kFusePlain))  // (16-bit blocks of 2-4 tokens: scap_swiglu.hip)
        return launch_inline<WDT, 4, FUSE>(a, lds, stream);
    else
        return SCAP_ERR_CONFIG;
}

template <int FUSE>
static int launch_inline_any(const GemvArgs& a, int wdt, int bt, size_t lds, hipStream_t stream) {
    if (wdt == kBF16) return launch_inline_wdt<kBF16, FUSE>(a, bt, lds, stream);
    if (wdt == kF16) return launch_inline_wdt<kF16, FUSE>(a, bt, lds, stream);
    if (wdt == kI8) return launch_inline_wdt<kI8, FUSE>(a, bt, lds, stream);
    if (wdt == kI8Half) return launch_inline_wdt<kI8Half, FUSE>(a, bt, lds, stream);
    return SCAP_ERR_CONFIG;
}

// Plan one launch: token slots, rows per workgroup (bounded by LDS and, for the input prologue, by the
// registers that hold a wavefront's chunks), LDS bytes.
static int plan_inline(GemvArgs& a, int wdt, int kc, bool kc_forced, int fuse, int* bt_out, size_t* lds_out,
                       bool slots16 = false) {
    if (wdt != kBF16 && !is_int8(wdt) && wdt != kF16) return SCAP_ERR_CONFIG;
    if (a.B < 1 || a.B > kMfmaTokens) return SCAP_ERR_CONFIG;
    const int bt = (a.B <= 4 && !slots16) ? 4 : 16;
    if (wdt == kF16 && bt != kMfmaTokens) return SCAP_ERR_CONFIG;  // fp16: the 16-slot kernels only
    const int tile_cols = wdt == kI8 ? 2 * kMfmaTile : kMfmaTile;
    size_t budget = kInlineLdsBudget;
    int kc_cap = kInlineWaves * kWave * inline_max_chunks(bt);
    if (fuse == kFuseList) kc_cap = 64 * kWave;  // gather_lists: at most 64 segments of 64 channels per workgroup
    // (a fifth chunk there takes the gating form past its scalar registers)
    if (wdt == kI8Half && fuse == kFuseSwiglu) kc_cap = kInlineWaves * kWave * 4;
    const size_t by_cap = kHdrBytes + (size_t)kc_cap * 4 * (1 + bt);
    if (by_cap < budget) budget = by_cap;
    // 16 slots: a split's partial sums cost the tile's last arrival as much time as kInlineSplitRows rows (sweeps of kc; 4096 x 1024,
    // 16 tokens, pieces of 128 / 256 rows: 13.2 / 11.6 us bf16, 8 tokens int8 13.1 / 12.8 against 15.9 with 64)
    SplitCost sc;
    sc.rows = bt == kMfmaTokens ? kInlineSplitRows : 0;
    const int rc = plan_splits(a, tile_cols, bt, kc, kc_forced, budget, kWave, sc);
    if (rc != SCAP_OK) return rc;
    if (a.Kc > kc_cap) return SCAP_ERR_SHAPE;
    size_t red = (size_t)kTreeFloats * 4;
    if (fuse == kFuseSwiglu) red += (size_t)bt * tile_cols * 4;
    *bt_out = bt;
    *lds_out = lds_bytes(a.Kc, bt, red);
    if (bt == kMfmaTokens && staged_tile(wdt, a.K)) {  // staged-tile form: the inputs as they are in place of the value lists
        const size_t body = (size_t)a.Kc * 4 + raw_tile_bytes(a.Kc);
        *lds_out = kHdrBytes + (body > red ? body : red);
    }
    return SCAP_OK;
}

// What a planned launch takes, in rows of one workgroup (as plan_splits weighs them), times the columns of its tile.
static int64_t inline_cost(const GemvArgs& a, int tile_cols) {
    return (((int64_t)a.S * a.T + 255) / 256 * (a.Kc + 128) + (int64_t)a.S * kInlineSplitRows) * tile_cols;
}

// The cost weighs a workgroup's fixed part like rows, but its prologue tests Kc channels whatever its tile: narrow tiles pay when
// they all run at once, otherwise only while the launch does not grow by more than the units can hide, and rows that start
// inside a cache line (N not a multiple of 128) are read in pieces that straddle two.  From 100 layers of more than 256 narrow
// workgroups (us, 16- / 8-byte lanes, with the workgroups of either): 24728 x 9856, 5 tokens, 51.3 / 48.7 (508 / 1001), 832 x 20096
// 11.5 / 10.4 (237 / 471), 520 x 17824 (pieces of 192 rows) 10.7 / 9.3, 4016 x 22128, 16 tokens, 37.3 / 34.7 (435 / 692), 2056 x
// 16624 (pieces of 704) 19.2 / 17.9, but with 5 tokens 16.4 / 17.0; 1024 x 43680, 4 tokens, 16.0 / 20.8 (171 / 684), 24288 x 5120, 5
// tokens, 30.1 / 32.1 (240 / 760), 2904 x 19312, 8 tokens, 22.6 / 25.7 (228 / 453, pieces of 1024), 62240 x 4592, 4 tokens, 76.0 /
// 95.7 (504 / 1008).
static bool narrow_tiles_fit(const GemvArgs& narrow, const GemvArgs& wide) {
    const int64_t n = (int64_t)narrow.S * narrow.T, w = (int64_t)wide.S * wide.T;
    if (n <= 256) return true;
    if (narrow.N % kMfmaTile == 0 || narrow.Kc <= (narrow.B > 8 ? 768 : 640)) return n < 3 * w;
    return narrow.Kc <= 1792 && 5 * n <= 8 * w;
}

// The same with the lane width of int8 weights chosen on the way (*wdt becomes kI8Half: 8-byte lanes, 128-column tiles).
// Narrow tiles halve the K splits, the wavefronts' sums and what a tile's last arrival collects, wide ones halve the
// prologues and read rows in pieces of 256 instead of 128 bytes.  Which is faster follows what the two plans cost (16
// tokens, wide / narrow, us: 1024 x 4096 12.0 / 8.5, 4096 x 4096 14.0 / 10.9, 14336 x 4096 21.5 / 19.6, 4096 x 24576 35.3 /
// 30.3, 16384 x 16384 69.7 / 66.4), where narrow tiles fit; where the two cost the same (4096 x 28672) so do the launches.  At
// 97-99 % of the cost few tokens gain less than many: 8192 x 16384, 5 tokens, 32.3 / 33.5, 16 tokens 36.3 / 35.9.
// An input length that is not a multiple of 8: the staged tile exists for narrow tiles only.  It beats the value lists up to 2^26
// weights (16 tokens, lists / tile: 513 x 1024 17.0 / 8.8, 5461 x 2752 23.3 / 12.5, 14337 x 4096 27.3 / 24.2; not with four times the
// workgroups: 1023 x 48016, 12 tokens, 25.1 / 26.4); beyond, with up to 8 tokens, where rows start on a cache line or the pieces are
// not long and many (6 tokens 5461 x 26128 70.0 / 53.4, 9001 x 9600, 5 tokens, 30.7 / 25.5, 2047 x 40000 43.0 / 32.0, but 16385 x
// 8784 48.3 / 58.3 and 62241 x 4592 95.7 / 111.6), and with more not (16 tokens 4097 x 28672 40.0 / 43.2, 10 tokens 36.4 / 37.4).
static int plan_inline_lanes(GemvArgs& a, int* wdt, int kc, bool kc_forced, int fuse, int* bt_out, size_t* lds_out,
                             bool slots16 = false) {
    const GemvArgs in = a;
    const int rc = plan_inline(a, *wdt, kc, kc_forced, fuse, bt_out, lds_out, slots16);
    if (rc != SCAP_OK || *wdt != kI8 || *bt_out != kMfmaTokens) return rc;
    GemvArgs h = in;
    int bt = 0;
    size_t lds = 0;
    if (plan_inline(h, kI8Half, kc, kc_forced, fuse, &bt, &lds, slots16) != SCAP_OK) return rc;
    if (in.K % 8 != 0) {
        const int64_t n = (int64_t)h.S * h.T, w = (int64_t)a.S * a.T;
        const bool little = (int64_t)in.K * in.N <= ((int64_t)1 << 26) && (n < 4 * w || h.Kc < 512);
        const bool few = in.N % kMfmaTile == 0 || h.Kc <= 640 || (h.Kc <= 1536 && n <= 2 * w);
        // (3-4 tokens: against the 4-slot lists, which launch_gemm_inline takes where this stays wide)
        if (!(in.B <= 4 ? little && narrow_tiles_fit(h, a) : little || (in.B <= 8 && few))) return rc;
    } else if (inline_cost(h, kMfmaTile) * 100 >= inline_cost(a, 2 * kMfmaTile) * 99 || !narrow_tiles_fit(h, a)) {
        return rc;
    }
    a = h;
    *lds_out = lds;
    *wdt = kI8Half;
    return rc;
}

// slots16: run 2-4 tokens in the 16-slot staged-tile kernel
int launch_gemm_inline(const GemvArgs& a_in, int wdt, const scap_launch_cfg* cfg, hipStream_t stream, bool slots16) {
    GemvArgs a = a_in;
    if (a.B < kMfmaMinTokens) return SCAP_ERR_CONFIG;
    int kc = 0;
    if (cfg) {
        if (cfg->rows_per_group) kc = cfg->rows_per_group;
        if (kc < 0 || (kc % kWave) != 0) return SCAP_ERR_CONFIG;
        if (cfg->waves_per_group && cfg->waves_per_group != kInlineWaves) return SCAP_ERR_CONFIG;
    }
    const int wdt_in = wdt;
    int bt = 0;
    size_t lds = 0;
    // 16 token slots: row step by row step where that is the faster kernel.  (Rows that the caller names have to fit here all the same.)
    const int src = exact_operand(a, wdt) ? kRowsCodes : kRowsCentre;
    const bool rows = a.B > 4 ? rows_pay(a, wdt) : slots16 && wdt != kI8;
    if (rows && kc == 0) {
        const int rc = launch_gemm_rows(a, wdt, src, kFusePlain, 0, stream);
        if (rc != SCAP_ERR_SHAPE) return rc;
    }
    const int rc = plan_inline_lanes(a, &wdt, kc, kc != 0, kFusePlain, &bt, &lds, slots16);
    if (rc != SCAP_OK) return rc;
    if (rows && kc != 0) {
        const int rc2 = launch_gemm_rows(a_in, wdt_in, src, kFusePlain, kc, stream);
        if (rc2 != SCAP_ERR_SHAPE) return rc2;
    }
    // Layers wider than 4 K and odd lengths: the 4-slot lists where they need fewer workgroups than the tile's LDS allows, or where
    // the tile would run in 16-byte lanes, one workgroup per compute unit, on more of them (or does not exist); two of the lists'
    // share a unit.  3 tokens at 70 %, tile / lists, us: 4096 x 57344 43.8 / 35.4, 6144 x 28672 38.1 / 32.3, 2664 x 56944 39.2 / 32.3,
    // 7912 x 33408 58.2 / 46.8, 5896 x 34816 47.0 / 40.8; elsewhere 4096 x 24576 21.7 / 23.2, 2048 x 20480 12.6 / 15.8, 512 x 24576 6.4 / 12.0.
    if (slots16 && wdt_in == kI8 && ((int64_t)a.N > 4 * (int64_t)a.K || a.K % 8 != 0)) {
        GemvArgs l = a_in;
        int bt_l = 0;
        size_t lds_l = 0;
        if (plan_inline(l, kI8, kc, kc != 0, kFusePlain, &bt_l, &lds_l) == SCAP_OK &&
            ((a.K % 8 == 0 && l.Kc > kTileRows) || (wdt == kI8 && (a.K % 8 != 0 || (int64_t)a.S * a.T > 256)))) {
            a = l;
            wdt = kI8;
            bt = bt_l;
            lds = lds_l;
        }
    }
    a.Kl = a.Kc;
    a.Sl = a.S;
    return launch_inline_any<kFusePlain>(a, wdt, bt, lds, stream);
}

// The two launches of the fused SwiGLU block on the matrix cores (see scap_swiglu.hip for the vector form).
int launch_swiglu_block_inline(const GemvArgs& up_in, const GemvArgs& dn_in, int wdt, hipStream_t stream) {
    GemvArgs up = up_in, dn = dn_in;
    int bt_up = 0, bt_dn = 0;
    size_t lds_up = 0, lds_dn = 0;
    int wup = wdt;
    const bool exact = exact_operand(up, wdt);
    if (up.B > 4 || ((int64_t)up.K * up.N <= ((int64_t)1 << 27) && rows_pay_gating(up, wdt) && gemm_rows_plans(dn, wdt, kRowsPlanes, kFusePlain))) {
        // 16 token slots: the gated product travels as planes of operand halves, and the down launch takes them row step by row step
        const int src = exact ? kRowsCodes : kRowsCentre;
        const bool codes = gemm_rows_plans(up, wdt, src, kFuseSwiglu);
        if (!codes) {
            const int rc = plan_inline_lanes(up, &wup, 0, false, kFuseSwiglu, &bt_up, &lds_up);
            if (rc != SCAP_OK) return rc;
            up.Kl = up.Kc;
            up.Sl = up.S;
        }
        if (!gemm_rows_plans(dn, wdt, kRowsPlanes, kFusePlain)) return SCAP_ERR_SHAPE;
        up.zl_lo = dn.zl_lo = reinterpret_cast<uint16_t*>(up.zl_d) + (size_t)block_token_slots(up.B) * plane_pitch(up.F);
        dn.seg_cnt = up.seg_cnt;
        const int rc = codes ? launch_gemm_rows(up, wdt, src, kFuseSwiglu, 0, stream)
                             : launch_inline_any<kFuseSwiglu>(up, wup, bt_up, lds_up, stream);
        if (rc != SCAP_OK) return rc;
        return launch_gemm_rows(dn, wdt, kRowsPlanes, kFusePlain, 0, stream);
    }
    // 4 token slots: lists of values
    int rc = plan_inline(up, wdt, 0, false, kFuseSwiglu, &bt_up, &lds_up);
    if (rc != SCAP_OK) return rc;
    up.Kl = up.Kc;
    up.Sl = up.S;
    rc = plan_inline(dn, wdt, 0, false, kFuseList, &bt_dn, &lds_dn);
    if (rc != SCAP_OK) return rc;
    dn.Kl = kWave;
    dn.Sl = (dn.K + kWave - 1) / kWave;
    const size_t tables = kHdrBytes + (size_t)dn.Sl * 4;  // offsets of every segment (a tile's last arrival, for its tokens' lists)
    if (lds_dn < tables) lds_dn = tables;
    rc = launch_inline_any<kFuseSwiglu>(up, wdt, bt_up, lds_up, stream);
    if (rc != SCAP_OK) return rc;
    return launch_inline_any<kFuseList>(dn, wdt, bt_dn, lds_dn, stream);
}

}  // namespace scap
