// Offline calibration (SCAP Eq. 2: tau = Quantile(|X_calib|, s); Section 3: mode estimate first, threshold
// on the centred sample).
//
// The calibration activations are 16-bit codes, so a pooled sample of any size has at most 65 536 distinct
// values.  ONE streaming pass over the sample counts how often each code occurs; every statistic the
// estimators need is then a function of those 65 536 counts, evaluated with the same IEEE operations the pruner
// uses (widening is exact, d = fp32(x) - m is one fp32 subtraction).  With the median or m = 0 that is two order
// statistics, which one workgroup selects from the counts on the GPU (select_kernel); the mean (an fp64 sum of count x
// value), the histogram mode (fp64 bin arithmetic) and samples of 2^32 values or more are evaluated on the host.
#include <math.h>
#include <cmath>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <utility>
#include <vector>

#include "scap_device.hpp"
#include "scap_internal.hpp"

namespace scap {

constexpr int kCodes = 65536;
constexpr int kHalf = 32768;        // codes counted by one workgroup: 128 KB of LDS counters (gfx950: 160 KB per workgroup)
constexpr int kHistThreads = 1024;
constexpr int kHistChunks = 128;    // workgroups per half of the code space

// Workgroup (chunk, half) reads its share of the sample 16 bytes per lane and counts the codes whose top bit
// equals `half` (the sign) in LDS, then adds its non-zero counters to the global histogram.  The kernel is bound
// by instruction issue (shift, compare, masked LDS add per code), so every code is looked at by as few
// workgroups as LDS allows: two.
// (16-bit counters, two to a word, hold the whole code space, so that every code is looked at once; with sweeps between
// rounds of 32768 codes against overflow that took 49 instead of 34 us on bf16 16384 x 4096 and 87 instead of 41 on fp16:
// neighbouring codes are the frequent ones, and their adds meet on one word.)
// COUNT: 32-bit counts and, behind them, one bit per group of 64 codes that has any (samples of less than 2^32 values whose
// statistics are selected on the GPU), or 64-bit counts.
template <typename COUNT>
__global__ __launch_bounds__(kHistThreads) void code_hist_kernel(const uint16_t* __restrict__ X, int64_t M,
                                                                COUNT* __restrict__ hist) {
    extern __shared__ uint32_t sh[];  // [kHalf]
    __shared__ uint32_t s_live[kHalf / kWave / 32];
    const int tid = threadIdx.x;
    // The two workgroups that read the same share sit on one XCD (blockIdx % 8) and start together, so the share
    // comes from HBM once and from that XCD's L2 the second time.
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const uint32_t half = (uint32_t)j & 1u;
    const int chunk = xcd + 8 * (j >> 1);
    const int nchunk = gridDim.x >> 1;
    for (int i = tid; i < kHalf; i += kHistThreads) sh[i] = 0;
    if (tid < kHalf / kWave / 32) s_live[tid] = 0;
    __syncthreads();
    auto count = [&](uint32_t code) {
        if ((code >> 15) == half) atomicAdd(&sh[code & (kHalf - 1)], 1u);
    };
    const int64_t nvec = M / 8;
    const uint4* __restrict__ X8 = reinterpret_cast<const uint4*>(X);
    auto count8 = [&](const uint4& v) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            count(w[q] & 0xFFFFu);
            count(w[q] >> 16);
        }
    };
    // four loads in flight per lane: with 16 wavefronts per compute unit (the counters fill LDS) one load per lane
    // leaves the memory latency exposed
    constexpr int FLY = 4;
    const int64_t stride = (int64_t)nchunk * kHistThreads;
    int64_t i = (int64_t)chunk * kHistThreads + tid;
    for (; i + (FLY - 1) * stride < nvec; i += FLY * stride) {
        uint4 v[FLY];
#pragma unroll
        for (int u = 0; u < FLY; ++u) v[u] = X8[i + u * stride];
#pragma unroll
        for (int u = 0; u < FLY; ++u) count8(v[u]);
    }
    for (; i < nvec; i += stride) count8(X8[i]);
    if (chunk == 0) {
        const int64_t j = nvec * 8 + tid;  // the last M % 8 codes
        if (j < M) count(X[j]);
    }
    __syncthreads();
    for (int i = tid; i < kHalf; i += kHistThreads) {
        const uint32_t v = sh[i];
        if (v) atomicAdd(&hist[half * kHalf + i], (COUNT)v);
        if constexpr (sizeof(COUNT) == 4) {
            const int g = i / kWave;  // wave-uniform
            if (__ballot(v != 0) != 0 && lane_id() == 0) atomicOr(&s_live[g >> 5], 1u << (g & 31));
        }
    }
    if constexpr (sizeof(COUNT) == 4) {
        __syncthreads();
        constexpr int WORDS = kHalf / kWave / 32;
        if (tid < WORDS && s_live[tid] != 0) atomicOr(&hist[kCodes + half * WORDS + tid], s_live[tid]);
    }
}

// ---------------------------------------------------------------------------------------------- order statistics
// m = median of the sample (or 0) and tau = k-th smallest |value - m| from the counts, by one workgroup (M < 2^32): each
// selection is a radix select over LDS bins.  The groups of 64 codes that have counts at all (most samples touch a tenth
// of the bf16 codes, and neighbouring ones) are known from the counting kernel's bits; their counts are fetched once, into
// LDS, and every pass reads them there.  A pass's work is shared out by runs of codes, one per thread, not by groups, one
// per wavefront: a few instructions per code and wavefront are what one compute unit spends its time on where many codes
// occur (fp16).  The groups past the LDS room are read from memory, a wavefront per group and eight in flight; taken as runs
// they were a second round of 32 loads in a row for few threads (a whole call over fp16, us, runs / this: 3 x 333 with 586
// groups, ZERO, 81.3 / 65.4; 64 x 1024 with almost all, ZERO 99.8 / 87.2, MEDIAN 117.8 / 99.6).  The loops are rolled: with the
// counts in registers and every loop unrolled the kernel waited for its own 100 KB of instructions.  16384 x 4096 sample,
// before (every pass read 64-bit counts from L2, behind one that looked for the groups) / now: bf16 35.6 / 21.7 us, fp16
// 98 / 61; the whole call with the median 94 / 81 and 157 / 119.
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kGroups = kCodes / kWave;
constexpr int kSelBins = 2048;
constexpr int kSelFly = 8;  // groups in flight per wavefront
constexpr int kSelGroups = 512;  // groups whose counts are kept in LDS: as many as make one run of 32 codes per thread
constexpr uint32_t kNoRank = 0xFFFFFFFFu;

struct SelLds {
    uint32_t bins[kSelBins];
    uint32_t wave[kSelWaves];
    uint16_t live[kGroups];  // groups with counts, in no particular order
    uint32_t held;           // entries of the bin where the last rank fell
    int nlive;
    uint32_t bin, rank;  // where a rank fell: its bin and the rank inside it
    uint32_t counts[kSelGroups * kWave];  // counts of the first kSelGroups listed groups
};

// sum over each row of 16 lanes, in every lane
__device__ __forceinline__ uint32_t row_total(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);   // lanes 1,0,3,2 of a quad
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);   // lanes 2,3,0,1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);  // mirrored in each half row
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);  // mirrored in each row
    return v;
}

__device__ __forceinline__ void sel_clear(SelLds& s) {
    for (int i = threadIdx.x; i < kSelBins; i += kSelThreads) s.bins[i] = 0;
    __syncthreads();
}

// The bin that holds rank r (1-based; s.bin = kNoRank past the total) and the rank inside it.  Ends with a barrier.
__device__ __forceinline__ void sel_find(SelLds& s, uint32_t r) {
    const int tid = threadIdx.x, w = tid >> 6;
    __syncthreads();
    if (tid == 0) s.bin = kNoRank;
    const uint32_t a = s.bins[2 * tid], b = s.bins[2 * tid + 1];
    const uint32_t inc = (uint32_t)wave_inclusive_scan((int)(a + b));
    if (lane_id() == kWave - 1) s.wave[w] = inc;
    __syncthreads();
    uint32_t before = inc - (a + b);
    for (int i = 0; i < w; ++i) before += s.wave[i];
    if (r > before && r - before <= a) {
        s.bin = 2 * tid;
        s.rank = r - before;
        s.held = a;
    } else if (r > before + a && r - before - a <= b) {
        s.bin = 2 * tid + 1;
        s.rank = r - before - a;
        s.held = b;
    }
    __syncthreads();
}
static_assert(kSelBins == 2 * kSelThreads, "two bins per thread");

// position of a code in ascending value order (sign-magnitude; -0 before +0) and back
__device__ __forceinline__ uint32_t code_rank(uint32_t c) { return (c & 0x8000u) ? 0xFFFFu - c : 0x8000u + c; }
__device__ __forceinline__ uint32_t rank_code(uint32_t p) { return p < 0x8000u ? 0xFFFFu - p : p - 0x8000u; }

__global__ __launch_bounds__(kSelThreads) void select_kernel(const uint32_t* __restrict__ hist, uint32_t M, int xdt,
                                                            int median, uint32_t k, float* __restrict__ out) {
    extern __shared__ uint32_t sel_raw[];
    SelLds& s = *reinterpret_cast<SelLds*>(sel_raw);
    const int tid = threadIdx.x, lane = lane_id();
    const int w = uniform(tid >> 6);
    const float nan = __uint_as_float(0x7FFFFFFFu);
    auto value = [&](uint32_t c) { return xdt == kBF16 ? bf16_bits_to_f32(c) : f16_bits_to_f32(c); };
    if (tid == 0) s.nlive = 0;
    __syncthreads();
    {  // one bit per thread: the groups that have counts
        const bool live = (hist[kCodes + tid / 32] >> (tid & 31)) & 1u;
        const uint64_t bal = __ballot(live);
        int base = 0;
        if (lane == 0 && bal != 0) base = atomicAdd(&s.nlive, __popcll(bal));
        base = uniform(base);
        if (live) s.live[base + lanes_below(bal)] = (uint16_t)tid;
    }
    static_assert(kGroups == kSelThreads, "one group per thread");
    __syncthreads();
    const int n = s.nlive;
    // NaN codes rank behind every number and are not counted
    auto counted = [&](uint32_t code) {
        const uint32_t c = hist[code];
        const float v = value(code);
        return v == v ? c : 0u;
    };
    for (int g0 = w * kSelFly; g0 < min(n, kSelGroups); g0 += kSelWaves * kSelFly) {
        uint32_t c[kSelFly];
#pragma unroll
        for (int u = 0; u < kSelFly; ++u) c[u] = counted((uint32_t)s.live[min(g0 + u, n - 1)] * kWave + lane);
#pragma unroll
        for (int u = 0; u < kSelFly; ++u)
            if (g0 + u < min(n, kSelGroups)) s.counts[(g0 + u) * kWave + lane] = c[u];
    }
    // Adds the counts of the listed groups to the bins: bin(code) of a code, kNoRank where it is not counted.  Every thread
    // takes runs of 16 or 32 neighbouring codes, whose bins are mostly the same, and adds a run of equal bins at once.
    // (Every pass begins with sel_clear, whose barrier also stands between the counts' fetch and their first reader.)
    const int run = n <= kSelThreads / 4 ? 16 : 32;
    auto add_to_bins = [&](auto bin) {
        const int per_group = kWave / run;
        for (int r = tid; r < min(n, kSelGroups) * per_group; r += kSelThreads) {
            const int g = r / per_group, e0 = (r % per_group) * run;
            const uint32_t c0 = (uint32_t)s.live[g] * kWave;
            uint32_t cur = kNoRank, sum = 0;
#pragma unroll 4
            for (int j = 0; j < run; ++j) {
                const int e = e0 + ((j + lane) & (run - 1));  // lanes start at different places: fewer meet on one LDS bank
                const uint32_t c = s.counts[g * kWave + e];
                const uint32_t b = c != 0 ? bin(c0 + e) : kNoRank;
                if (b != cur) {
                    if (sum != 0) atomicAdd(&s.bins[cur], sum);
                    cur = b;
                    sum = 0;
                }
                sum += b != kNoRank ? c : 0u;
            }
            if (sum != 0) atomicAdd(&s.bins[cur], sum);
        }
        // the others: one code per lane
        for (int g0 = kSelGroups + w * kSelFly; g0 < n; g0 += kSelWaves * kSelFly) {
            uint32_t code[kSelFly], c[kSelFly];
#pragma unroll
            for (int u = 0; u < kSelFly; ++u) {
                code[u] = (uint32_t)s.live[min(g0 + u, n - 1)] * kWave + lane;
                c[u] = counted(code[u]);
            }
#pragma unroll
            for (int u = 0; u < kSelFly; ++u) {
                const uint32_t b = bin(code[u]);
                const uint32_t k = g0 + u < n && b != kNoRank ? c[u] : 0u;
                if (__ballot(b != (uint32_t)__shfl((int)b, lane & ~15, kWave)) == 0) {  // one bin per row of 16 lanes: one add
                    const uint32_t sum = row_total(k);
                    if ((lane & 15) == 0 && sum != 0) atomicAdd(&s.bins[b], sum);
                } else if (k != 0) {
                    atomicAdd(&s.bins[b], k);
                }
            }
        }
    };
    float m = 0.f;
    if (median) {  // the middle value, or the mean of the two middle ones; 2048 bins of 32 codes, then the 32 codes
        float mid[2];
        sel_clear(s);
        add_to_bins([&](uint32_t code) { return code_rank(code) >> 5; });
        uint32_t bin[2], rank[2];
        for (int j = 0; j < 2; ++j) {
            if (j == 1 && (M % 2 == 1 || (bin[0] != kNoRank && rank[0] < s.held))) {  // the same value, or the next in the same bin
                bin[1] = bin[0];
                rank[1] = rank[0] + (M % 2 == 1 ? 0u : 1u);
                break;
            }
            sel_find(s, (M % 2 == 1) ? M / 2 + 1 : M / 2 + (uint32_t)j);
            bin[j] = s.bin;
            rank[j] = s.rank;
        }
        // the 32 codes of a bin: lanes 0-31 the first rank's, 32-63 the second's, in every wavefront alike
        const uint32_t b = lane < 32 ? bin[0] : bin[1];
        const uint32_t code = b == kNoRank ? 0u : rank_code((b << 5) | (lane & 31u));
        uint32_t c = b == kNoRank ? 0u : hist[code];
        if (value(code) != value(code)) c = 0u;
        uint32_t inc = c;
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            const uint32_t t = (uint32_t)__shfl_up((int)inc, off, 32);
            if ((lane & 31) >= off) inc += t;
        }
        const uint64_t at = __ballot(inc >= (lane < 32 ? rank[0] : rank[1]) && b != kNoRank);
        for (int j = 0; j < 2; ++j) {
            const uint32_t half = (uint32_t)(at >> (32 * j));
            mid[j] = half == 0u ? nan : value(rank_code((bin[j] << 5) | (uint32_t)__builtin_ctz(half)));
        }
        m = (M % 2 == 1) ? mid[0] : (float)(((double)mid[0] + (double)mid[1]) / 2.0);
    }
    float tau = 0.f;
    if (k > 0) {
        tau = nan;
        if (m == m) {
            // |value - m| as a 31-bit key: bits 30-20, 19-10, 9-0 (infinite values of the sign of an infinite m: NaN, last)
            uint32_t prefix = 0, rank = k;
            bool found = true;
            for (int pass = 0; pass < 3 && found; ++pass) {
                const int shift = pass == 0 ? 20 : (pass == 1 ? 10 : 0);
                sel_clear(s);
                add_to_bins([&](uint32_t code) {
                    const float d = fabsf(value(code) - m);
                    const uint32_t key = __float_as_uint(d);
                    if (!(d == d && (pass == 0 || (key >> (shift + 10)) == prefix))) return kNoRank;
                    return pass == 0 ? key >> 20 : (key >> shift) & 1023u;
                });
                sel_find(s, rank);
                found = s.bin != kNoRank;
                prefix = pass == 0 ? s.bin : (prefix << 10) | s.bin;
                rank = s.rank;
            }
            if (found) tau = __uint_as_float(prefix);
        }
    }
    if (tid == 0) {
        out[0] = m;
        out[1] = tau;
    }
}

namespace {

bool ok(hipError_t e) { return e == hipSuccess; }

// exact widening of a 16-bit code on the host
float code_to_float(uint32_t c, int xdt) {
    uint32_t u;
    if (xdt == kBF16) {
        u = c << 16;
    } else {
        const uint32_t sign = (c & 0x8000u) << 16, e = (c >> 10) & 0x1Fu, f = c & 0x3FFu;
        if (e == 0x1Fu) {
            u = sign | 0x7F800000u | (f << 13);
        } else if (e != 0) {
            u = sign | ((e + 112u) << 23) | (f << 13);
        } else if (f == 0) {
            u = sign;
        } else {  // subnormal half: normalise
            int sh = 0;
            uint32_t m = f;
            while (!(m & 0x400u)) {
                m <<= 1;
                ++sh;
            }
            u = sign | ((113u - sh) << 23) | ((m & 0x3FFu) << 13);
        }
    }
    float v;
    memcpy(&v, &u, 4);
    return v;
}

// The sample as (value, count) pairs in ascending value order; NaNs counted apart (they rank last).
struct Table {
    std::vector<float> val;
    std::vector<unsigned long long> cnt;
    unsigned long long nans = 0;
};

Table make_table(const std::vector<unsigned long long>& hist, int xdt) {
    Table t;
    auto push = [&](uint32_t c) {
        if (!hist[c]) return;
        const float v = code_to_float(c, xdt);
        if (v != v) {
            t.nans += hist[c];
        } else {
            t.val.push_back(v);
            t.cnt.push_back(hist[c]);
        }
    };
    // both formats order like sign-magnitude integers: negatives from the largest magnitude down, then
    // positives up (-0 sorts before +0; they are equal as numbers, which no statistic below can tell apart)
    for (int c = 0xFFFF; c >= 0x8000; --c) push((uint32_t)c);
    for (int c = 0x0000; c <= 0x7FFF; ++c) push((uint32_t)c);
    return t;
}

float quiet_nan() {
    const uint32_t u = 0x7FFFFFFFu;
    float v;
    memcpy(&v, &u, 4);
    return v;
}

// k-th smallest of the raw values, 1 <= k <= M
float select_raw(const Table& t, unsigned long long k) {
    unsigned long long run = 0;
    for (size_t i = 0; i < t.val.size(); ++i) {
        run += t.cnt[i];
        if (k <= run) return t.val[i];
    }
    return quiet_nan();
}

// k-th smallest of |value - m| (one fp32 subtraction, as the pruner forms it).  Below m the importance
// falls as the value rises, above m it rises (fp32 rounding is monotone), so the sorted order is a merge
// of the two runs that start at the value nearest m.
float select_centred(const Table& t, float m, unsigned long long k) {
    if (m != m) return quiet_nan();
    const size_t n = t.val.size();
    std::vector<float> imp(n);
    size_t p = n;  // first entry with value - m >= 0
    bool any_nan = false;
    for (size_t i = 0; i < n; ++i) {
        volatile float d = t.val[i] - m;
        imp[i] = fabsf(d);
        any_nan |= imp[i] != imp[i];
        if (p == n && !(d < 0.f)) p = i;
    }
    if (any_nan) {
        // infinite m meeting an infinite sample: no monotone runs; sort outright, NaN importances last
        std::vector<std::pair<float, unsigned long long>> e;
        unsigned long long run = 0;
        for (size_t i = 0; i < n; ++i)
            if (imp[i] == imp[i]) e.emplace_back(imp[i], t.cnt[i]);
        std::sort(e.begin(), e.end());
        for (const auto& x : e) {
            run += x.second;
            if (k <= run) return x.first;
        }
        return quiet_nan();
    }
    size_t up = p;          // next candidate of the rising run
    size_t down = p;        // one past the next candidate of the falling run
    unsigned long long run = 0;
    while (up < n || down > 0) {
        size_t pick;
        if (up >= n)
            pick = --down;
        else if (down == 0)
            pick = up++;
        else if (imp[down - 1] <= imp[up])
            pick = --down;
        else
            pick = up++;
        run += t.cnt[pick];
        if (k <= run) return imp[pick];
    }
    return quiet_nan();
}

// 1-based rank of the q-quantile among M pooled values: the smallest integer >= q*M (product formed in fp64),
// kept inside [0, M]
int64_t quantile_rank(double q, int64_t M) {
    return std::min<int64_t>(M, std::max<int64_t>(0, (int64_t)std::ceil(q * (double)M)));
}

// Histogram estimate of the mode from the (value, count) table: kHistBins equal bins between the 0.001 and
// 0.999 order statistics (a value equal to the upper one belongs to the last bin), each bin scored by the
// number of samples in the five bins centred on it (fewer at the edges), the centre of the first bin with the
// top score.  The bins are filled as a running total, so a score is the difference of two totals.
float histogram_mode(const Table& t, int64_t M) {
#pragma clang fp contract(off)  // (b + 1/2) * w and lo + ... each round once, in fp64
    const float lo = select_raw(t, (unsigned long long)std::max<int64_t>(1, quantile_rank(0.001, M)));
    const float hi = select_raw(t, (unsigned long long)std::max<int64_t>(1, quantile_rank(0.999, M)));
    if (!(hi > lo)) return lo;
    const double width = ((double)hi - (double)lo) / (double)kHistBins;
    // upto[b] = samples in bins 0 .. b-1; the table is ascending, so bins are met in order
    std::vector<unsigned long long> upto(kHistBins + 1, 0);
    for (size_t i = 0; i < t.val.size(); ++i) {
        const float v = t.val[i];
        if (v < lo || v > hi) continue;
        const double pos = std::floor(((double)v - (double)lo) / width);
        // an infinite order statistic makes the width infinite and positions 0 or NaN: those values count in bin 0
        const int bin = !(pos > 0.0) ? 0 : (pos >= (double)kHistBins ? kHistBins - 1 : (int)pos);
        upto[bin + 1] += t.cnt[i];
    }
    for (int b = 0; b < kHistBins; ++b) upto[b + 1] += upto[b];
    int top_bin = 0;
    unsigned long long top = 0;
    for (int b = 0; b < kHistBins; ++b) {
        const unsigned long long score = upto[std::min(b + 3, kHistBins)] - upto[std::max(b - 2, 0)];
        if (b == 0 || score > top) {
            top = score;
            top_bin = b;
        }
    }
    const double offset = ((double)top_bin + 0.5) * width;
    const double centre = (double)lo + offset;
    return (float)centre;
}

// More dynamic LDS than the default limit for `kernel`: asked for once per device.
constexpr int kMaxDevices = 64;
int allow_lds(std::atomic<bool> (&asked)[kMaxDevices], const void* kernel, int bytes) {
    int dev = 0;
    if (!ok(hipGetDevice(&dev)) || dev < 0 || dev >= kMaxDevices) return SCAP_ERR_HIP;
    if (!asked[dev].load(std::memory_order_acquire)) {
        if (!ok(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes))) return SCAP_ERR_HIP;
        asked[dev].store(true, std::memory_order_release);
    }
    return SCAP_OK;
}

// Counts of every code of the sample into `hist`, `words` 32-bit words of which are cleared first.
template <typename COUNT>
int count_codes(const uint16_t* X, int64_t M, COUNT* hist, size_t words, hipStream_t stream) {
    int rc = launch_zero_words(reinterpret_cast<int32_t*>(hist), words, stream);
    if (rc != SCAP_OK) return rc;
    static std::atomic<bool> asked[kMaxDevices];
    rc = allow_lds(asked, reinterpret_cast<const void*>(&code_hist_kernel<COUNT>), kHalf * 4);
    if (rc != SCAP_OK) return rc;
    hipLaunchKernelGGL(code_hist_kernel<COUNT>, dim3(2 * kHistChunks), dim3(kHistThreads), kHalf * 4, stream, X, M, hist);
    return ok(hipGetLastError()) ? SCAP_OK : SCAP_ERR_HIP;
}

}  // namespace

int run_calibrate(const uint16_t* X, int64_t M, int xdt, float s, int est, float* m_out, float* tau_out, void* workspace,
                  hipStream_t stream) {
    if (est < SCAP_MODE_ZERO || est > SCAP_MODE_HIST) return SCAP_ERR_DTYPE;
    const int64_t k = quantile_rank((double)s, M);
    void* counts = static_cast<char*>(workspace) + kOffCodeHist;
    if ((est == SCAP_MODE_ZERO || est == SCAP_MODE_MEDIAN) && M < ((int64_t)1 << 32)) {
        uint32_t* d_hist = static_cast<uint32_t*>(counts);
        int rc = count_codes<uint32_t>(X, M, d_hist, kCodes + kGroups / 32, stream);
        if (rc != SCAP_OK) return rc;
        static std::atomic<bool> asked[kMaxDevices];
        rc = allow_lds(asked, reinterpret_cast<const void*>(&select_kernel), (int)sizeof(SelLds));
        if (rc != SCAP_OK) return rc;
        float* d_out = reinterpret_cast<float*>(static_cast<char*>(workspace) + kOffSelected);
        hipLaunchKernelGGL(select_kernel, dim3(1), dim3(kSelThreads), sizeof(SelLds), stream, d_hist, (uint32_t)M, xdt,
                           est == SCAP_MODE_MEDIAN ? 1 : 0, (uint32_t)k, d_out);
        float got[2];
        if (!ok(hipGetLastError()) || !ok(hipMemcpyAsync(got, d_out, sizeof(got), hipMemcpyDeviceToHost, stream)) ||
            !ok(hipStreamSynchronize(stream)))
            return SCAP_ERR_HIP;
        *m_out = got[0];
        *tau_out = got[1];
        return SCAP_OK;
    }
    unsigned long long* d_hist = static_cast<unsigned long long*>(counts);
    const int rc = count_codes<unsigned long long>(X, M, d_hist, 2 * (size_t)kCodes, stream);
    if (rc != SCAP_OK) return rc;
    std::vector<unsigned long long> hist(kCodes);
    if (!ok(hipMemcpyAsync(hist.data(), d_hist, sizeof(unsigned long long) * kCodes, hipMemcpyDeviceToHost, stream)))
        return SCAP_ERR_HIP;
    if (!ok(hipStreamSynchronize(stream))) return SCAP_ERR_HIP;
    const Table t = make_table(hist, xdt);

    float m = 0.f;
    if (est == SCAP_MODE_MEAN) {
        double sum = t.nans ? (double)quiet_nan() : 0.0;
        for (size_t i = 0; i < t.val.size(); ++i) sum += (double)t.cnt[i] * (double)t.val[i];
        m = (float)(sum / (double)M);
    } else if (est == SCAP_MODE_MEDIAN) {  // 2^32 values or more
        if (M % 2 == 1) {
            m = select_raw(t, (unsigned long long)(M / 2 + 1));
        } else {
            const float a = select_raw(t, (unsigned long long)(M / 2));
            const float b = select_raw(t, (unsigned long long)(M / 2 + 1));
            m = (float)(((double)a + (double)b) / 2.0);
        }
    } else if (est == SCAP_MODE_HIST) {
        m = histogram_mode(t, M);
    }

    float tau = 0.f;
    if (k > 0) tau = select_centred(t, m, (unsigned long long)k);
    *m_out = m;
    *tau_out = tau;
    return SCAP_OK;
}

}  // namespace scap
