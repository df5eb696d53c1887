// Bandwidth of the SVGD kernel by the median heuristic (Appendix D-B): the
// lower median m2 of the P = N(N-1)/2 squared distances D_ij (i < j, FP32 by
// direct differences in coordinate order), h = max(m2 / ln N, 1e-12).
//
// Exact path (interval select).  Non-negative floats order like their bit
// patterns, so the median is the rank-k bit pattern, k = ceil(P/2).
//   1. A fixed sample of kMedSample pairs is measured (the same squared
//      distances, summed in a fixed order of their own, so within rounding of
//      the passes' values) and its order statistics at ranks
//      S(1/2 -+ 2/sqrt S) give a bracket [lo, hi] that holds rank k unless the
//      sample is off by four standard deviations (about once in 16 000
//      selects; a rank outside it sends the passes back over every pair, step
//      3, so the result stays exact).  A wider bracket makes every pass 0
//      stage and every candidate pass read more candidates.  When all pairs fit in the
//      sample, it is the population and its median is final.  The sample sits
//      in LDS for the select.
//   2. Pass 0 over every pair counts the pairs below lo and copies the
//      in-bracket bit patterns into a candidate buffer.
//   3. Pass 1 histograms the bracket into 2048 linear bins, pass 2 the bin that
//      holds rank k: below a bracket of 2^22 bit patterns (nearly always) its
//      bins are single values and pass 3 only looks up rank k; else pass 3 is
//      the third histogram (widths are below 2^32).  The passes read the
//      candidates when they cover the interval, else every pair again (rank k
//      outside the bracket, or the buffer overflowed).
// Every count is an integer and every comparison exact, so the result is the
// exact order statistic, independent of scheduling.
//
// Problems with at most 2^20 pairs finish after pass 0 in one workgroup of
// 1024 that reads the candidates once into registers and histograms them there
// (or, rarely, runs the passes over every pair), so their select takes four
// kernels.
//
// An all-pairs work item is (ROWS-row block, 64-column chunk) in a workgroup of
// 256: each thread keeps its row's coordinates in registers and reads the
// staged columns as LDS broadcasts, four columns at a time.  A lane keeps its
// in-bracket values in a list of its own in LDS, and a wave appends its lists
// to one of kCandSegs buffer segments with one atomic per flush, which carries
// its count of pairs below the bracket too.
//
// Sampled path: the bandwidth from the sample's own lower median.
#include <math.h>

#include <type_traits>

#include "bf16_operands.h"
#include "common.h"
#include "internal.h"
#include "operands32.h"

namespace stamp {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f4v;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8v;

namespace {

constexpr uint32_t kModeDone = 0, kModePass0 = 1;
constexpr float kBracketSigmas = 4.0f;
constexpr uint32_t kSentinel = 0xffffffffu;  // above every candidate interval
constexpr int kSelThreads = 1024;         // threads of the sample select

__device__ __forceinline__ uint32_t mix32(uint32_t x) {  // MurmurHash3 finaliser
    x ^= x >> 16;
    x *= 0x85ebca6bu;
    x ^= x >> 13;
    x *= 0xc2b2ae35u;
    x ^= x >> 16;
    return x;
}

__host__ __device__ __forceinline__ uint64_t pair_count(int N) { return (uint64_t)N * (uint64_t)(N - 1) / 2; }

// Bin shift so that an interval of `width` bit patterns fits 2048 bins.
// The smallest s with ceil(width / 2^s) <= 2048, i.e. bitlen(width - 1) - 11.
__device__ __forceinline__ uint32_t shift_for(uint64_t width) {
    const uint64_t m = width - 1;
    const int bl = m ? 64 - __clzll((long long)m) : 0;
    return bl > 11 ? (uint32_t)(bl - 11) : 0u;
}

// One problem's select workspace.
struct MedView {
    int N, d;
    float fixed_h;
    int rows, rb, cc;    // all-pairs items: rows each, row blocks, column chunks
    uint32_t seg_cap;    // candidate slots of a segment, whole 16-byte words
    float* smp;
    SelState* sel;
    uint32_t* hist;      // [3][kMedBins], one histogram per pass
    uint32_t* cand;
    const float* xr;     // Gram form: centred rows in MFMA operand order (4 ks floats each)
    const float* nrm;    // and their squared norms (FP32 matrix-core operands)
    const __bf16* xs3;   // split form (d <= 31): the same rows as three BF16 parts, [npad][3][32]
};

__device__ __forceinline__ MedView med_view(int N, int d, float fixed_h, const SvgdLayout& L, char* b) {
    MedView v;
    v.N = N;
    v.d = d;
    v.fixed_h = fixed_h;
    v.rows = L.med_rows;
    v.rb = L.med_rb;
    v.cc = L.med_cc;
    v.seg_cap = L.cand_cap / kCandSegs & ~3u;
    v.smp = reinterpret_cast<float*>(b + L.smp_off);
    v.sel = sel_state(b, L.sel_off);
    v.hist = reinterpret_cast<uint32_t*>(b + L.hist_off);
    v.cand = reinterpret_cast<uint32_t*>(b + L.cand_off);
    v.xr = reinterpret_cast<const float*>(b + L.x32_off);
    v.nrm = reinterpret_cast<const float*>(b + L.n32_off);
    v.xs3 = reinterpret_cast<const __bf16*>(b + L.xs3_off);
    return v;
}

// Sample slot t: pair t of the row-major enumeration of i < j when all pairs
// fit (N <= 128), else a hashed pair i != j (oriented i < j, as in the
// all-pairs passes); false beyond the sample.
__device__ bool sample_pair(int N, int t, int& i, int& j) {
    const uint64_t P = pair_count(N);
    const bool all = P <= (uint64_t)kMedSample;
    if (N < 2 || (all && (uint64_t)t >= P)) return false;
    if (all) {
        int r = t;
        i = 0;
        while (r >= N - 1 - i) {
            r -= N - 1 - i;
            ++i;
        }
        j = i + 1 + r;
    } else {
        i = (int)(mix32(2u * (uint32_t)t + 1u) % (uint32_t)N);
        j = (int)(mix32((2u * (uint32_t)t + 2u) ^ 0x9e3779b9u) % (uint32_t)(N - 1));
        if (j >= i) ++j;
        if (j < i) {
            const int x = i;
            i = j;
            j = x;
        }
    }
    return true;
}

// Slot t's squared distance (+inf beyond the sample), by the four lanes q of
// a DPP quad: lane q adds coordinates q, q + 4, q + 8, ... in order (eight
// gathers of each particle in flight, indices clamped so no load is
// predicated) and the quad adds its four sums as (s0 + s1) + (s2 + s3).  The
// random gathers are what a sample slot costs; four lanes per slot put four
// times the waves on them.  Every lane of the quad must call this.
__device__ float sample_dist4(int N, int d, int t, int q, const float* __restrict__ theta) {
    int i = 0, j = 0;
    const bool ok = sample_pair(N, t, i, j);
    float acc = 0.0f;
    if (ok) {
        const float* ti = theta + i;
        const float* tj = theta + j;
        for (int l0 = 0; l0 < d; l0 += 32) {
            float a[8], b[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t o = (int64_t)min(l0 + q + 4 * u, d - 1) * N;
                a[u] = ti[o];
                b[u] = tj[o];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (l0 + q + 4 * u < d) {
                    const float df = a[u] - b[u];
                    acc = fmaf(df, df, acc);
                }
        }
    }
    const float s = quad_sum(acc);
    return ok ? s : __int_as_float(0x7f800000);
}

// Leaves sel->mode alone: the passes' workgroups branch on it at their start,
// and in the last pass one of them may end here before another one starts.
// Only the sample select writes it.
__device__ __forceinline__ void set_bandwidth(SelState* sel, int N, uint32_t m2_bits, float* h_out) {
    const float m2 = __uint_as_float(m2_bits);
    const float h = fmaxf(m2 / logf((float)N), 1e-12f);
    sel->m2 = m2;
    sel->h = h;
    if (h_out) *h_out = h;
}

// The bandwidth when no median is wanted: the caller's, or 1 for a lone particle.
__device__ __forceinline__ void given_bandwidth(const MedView& v, float* h_out) {
    const float h = v.N < 2 ? 1.0f : v.fixed_h;
    v.sel->h = h;
    v.sel->m2 = -1.0f;
    v.sel->mode = kModeDone;
    if (h_out) *h_out = h;
}

// ---- select inside one workgroup of NT threads -----------------------------------
// Inclusive prefix sum over the workgroup in thread order.
template <int NT>
__device__ __forceinline__ uint32_t wg_scan(uint32_t x, uint32_t* wt) {
    static_assert(NT % 256 == 0, "wave totals are read four at a time");
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) wt[w] = x;
    __syncthreads();
    uint32_t base = 0;
#pragma unroll
    for (int q = 0; q < NT / 64; q += 4) {  // every wave total at once, 16-byte reads
        const uint4 t = *reinterpret_cast<const uint4*>(&wt[q]);
        base += (q + 0 < w ? t.x : 0u) + (q + 1 < w ? t.y : 0u) + (q + 2 < w ? t.z : 0u) + (q + 3 < w ? t.w : 0u);
    }
    __syncthreads();
    return x + base;
}

// Histogram into lh (2048 bins, bin = (x - lo) >> s) of the values x of a[0, n)
// with lo <= x <= hi, read by the T threads numbered sub = 0..T-1; 8 loads in
// flight per thread.
template <int T>
__device__ __forceinline__ void strided_hist(const uint32_t* __restrict__ a, uint32_t n, int sub, uint32_t lo,
                                             uint32_t hi, uint32_t s, uint32_t* lh) {
    const uint32_t w = hi - lo;  // x in [lo, hi] iff x - lo <= w (unsigned)
    uint32_t e = (uint32_t)sub;
    for (; e + 7 * T < n; e += 8 * T) {
        uint32_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = a[e + T * u] - lo;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (x[u] <= w) atomicAdd(&lh[x[u] >> s], 1u);
    }
    for (; e < n; e += T) {
        const uint32_t x = a[e] - lo;
        if (x <= w) atomicAdd(&lh[x >> s], 1u);
    }
}

// The same by a workgroup of 256 over a 16-byte aligned array, sixteen values a
// thread in flight.
__device__ __forceinline__ void wide_hist(const uint32_t* __restrict__ a, uint32_t n, uint32_t lo, uint32_t hi,
                                          uint32_t s, uint32_t* lh) {
    const uint32_t w = hi - lo, whole = n & ~4095u;
    for (uint32_t e = 4 * threadIdx.x; e < whole; e += 4096) {
        uint4 q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = *reinterpret_cast<const uint4*>(a + e + 1024 * u);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t x[4] = {q[u].x - lo, q[u].y - lo, q[u].z - lo, q[u].w - lo};
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (x[t] <= w) atomicAdd(&lh[x[t] >> s], 1u);
        }
    }
    strided_hist<256>(a + whole, n - whole, threadIdx.x, lo, hi, s, lh);
}

template <int NT>
__device__ __forceinline__ void wg_hist(const uint32_t* __restrict__ a, uint32_t n, uint32_t lo, uint32_t hi,
                                        uint32_t s, uint32_t* lh) {
    strided_hist<NT>(a, n, threadIdx.x, lo, hi, s, lh);
}

// After a histogram of [lo, hi] with shift s: narrow [lo, hi] to the bin that
// holds rank r (1-based among the counted values) and make r relative to it.
// Clears lh when `clear`.  Every thread returns with the same lo, hi, r, and
// the return value is the number of values in the chosen bin.
template <int NT>
__device__ uint32_t wg_narrow(uint32_t* lh, uint32_t* wt, uint32_t* part, uint32_t s, uint32_t& lo, uint32_t& hi,
                              uint32_t& r, bool clear = true) {
    constexpr int PER = kMedBins / NT;
    const int tid = threadIdx.x;
    __syncthreads();
    uint32_t loc[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        loc[q] = lh[tid * PER + q];
        if (clear) lh[tid * PER + q] = 0;
        sum += loc[q];
    }
    const uint32_t incl = wg_scan<NT>(sum, wt), excl = incl - sum;
    if (excl < r && r <= incl) {
        uint32_t c = excl;
        for (int q = 0; q < PER; ++q) {
            if (c < r && r <= c + loc[q]) {
                part[0] = (uint32_t)(tid * PER + q);
                part[1] = r - c;
                part[2] = loc[q];
                break;
            }
            c += loc[q];
        }
    }
    __syncthreads();
    const uint64_t nlo = (uint64_t)lo + ((uint64_t)part[0] << s);
    const uint64_t top = nlo + ((uint64_t)1 << s) - 1;
    hi = (uint32_t)(top < (uint64_t)hi ? top : (uint64_t)hi);
    lo = (uint32_t)nlo;
    r = part[1];
    const uint32_t nbin = part[2];
    __syncthreads();
    return nbin;
}

// Exact rank-r value (1-based) among the values in [lo, hi] of a[0, n).
// Expects lh clear; leaves it clear.
template <int NT>
__device__ uint32_t wg_select_array(const uint32_t* __restrict__ a, uint32_t n, uint32_t lo, uint32_t hi, uint32_t r,
                                    uint32_t* lh, uint32_t* wt, uint32_t* part) {
    while (lo < hi) {
        const uint32_t s = shift_for((uint64_t)hi - lo + 1);
        wg_hist<NT>(a, n, lo, hi, s, lh);
        wg_narrow<NT>(lh, wt, part, s, lo, hi, r);
    }
    return lo;
}

// The sample's order statistics (one workgroup of kSelThreads = 1024, exact selects over
// the 8192 sample values; +inf padding ranks last).  exact = 0: the sample
// median is the result; exact = 1: the bracket of the full select (or the
// result, when the sample holds every pair).
__device__ void sample_select_body(const MedView& v, int exact, float* h_out) {
    constexpr int NT = kSelThreads;
    __shared__ uint32_t xs[kMedSample];
    __shared__ uint32_t lh[kMedBins];
    __shared__ __align__(16) uint32_t wt[NT / 64];
    __shared__ uint32_t part[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    SelState* sel = v.sel;
    const int N = v.N;
    if (N < 2 || v.fixed_h > 0.0f) {
        if (tid == 0) given_bandwidth(v, h_out);
        return;
    }
    const uint64_t P = pair_count(N);
    const bool all = P <= (uint64_t)kMedSample;
    const uint32_t S = all ? (uint32_t)P : (uint32_t)kMedSample;
    uint32_t rank[3];
    rank[1] = (S + 1) / 2;
    const float half = kBracketSigmas * 0.5f / sqrtf((float)S);  // four sigmas of the sample median's rank
    rank[0] = (uint32_t)fmaxf(1.0f, floorf((float)S * (0.5f - half)));
    rank[2] = (uint32_t)fminf((float)S, ceilf((float)S * (0.5f + half)));
    uint32_t mn = 0xffffffffu, mx = 0u;  // range of the sample's values
    {  // the sample into LDS, all loads in flight; a NaN ranks as +inf, so that every
       // rank is found
        const uint32_t* g = reinterpret_cast<const uint32_t*>(v.smp);
        uint32_t x[kMedSample / NT];
#pragma unroll
        for (int u = 0; u < kMedSample / NT; ++u) x[u] = g[tid + NT * u];
#pragma unroll
        for (int u = 0; u < kMedSample / NT; ++u) {
            x[u] = min(x[u], 0x7f800000u);
            xs[tid + NT * u] = x[u];
            if ((uint32_t)(tid + NT * u) < S) {
                mn = min(mn, x[u]);
                mx = max(mx, x[u]);
            }
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        mn = min(mn, (uint32_t)__shfl_xor(mn, off));
        mx = max(mx, (uint32_t)__shfl_xor(mx, off));
    }
    if (lane == 0) {
        lh[wave] = mn;
        lh[NT / 64 + wave] = mx;
    }
    __syncthreads();
    for (int w = 0; w < NT / 64; ++w) {
        mn = min(mn, lh[w]);
        mx = max(mx, lh[NT / 64 + w]);
    }
    __syncthreads();
    for (int b = tid; b < kMedBins; b += NT) lh[b] = 0;
    __syncthreads();
    uint32_t lo0 = 0u, hi2 = 0u, m = 0u;
    if (!exact || all) {
        m = wg_select_array<NT>(xs, kMedSample, mn, mx, rank[1], lh, wt, part);
    } else {
        // bracket ends: the bins of one histogram of the sample's range that
        // hold ranks r0 and r2 (at least as wide as the sample's exact
        // quantiles, by at most a bin, 1/2048 of the range, on each side).  Where
        // such a bin holds more than kBinMost of the sample (tight clusters: most
        // distances within a fraction of the range) a second histogram narrows it,
        // or the bracket would hold more pairs than the candidate buffer and the
        // passes would go over every pair (two clusters, N = 8192, d = 30: 644 us,
        // now 92).  To 1024 patterns, and kBinPad more for the rounding the sample's
        // distances do not share: equal distances overflow all the same, but pass 1
        // resolves a bracket of 2048 (three points, N = 4096, d = 30: 134 us, now 87).
        // Smooth sets, some 20 values a bin, never come here.
        constexpr uint32_t kBinMost = kMedSample / 64, kBinPad = 512;
        auto narrow_end = [&](uint32_t n, uint32_t& a, uint32_t& z, uint32_t& r) {
            if (n <= kBinMost || a >= z || z - a < 1024) return;
            const uint32_t s = shift_for((uint64_t)z - a + 1);
            wg_hist<NT>(xs, kMedSample, a, z, s, lh);
            wg_narrow<NT>(lh, wt, part, s, a, z, r);
            a -= min(a, kBinPad);
            z = min(z + kBinPad, 0x7f800000u);
        };
        uint32_t a0 = mn, z0 = mx, r0 = rank[0];
        uint32_t a2 = a0, z2 = z0, r2 = rank[2];
        const uint32_t s1 = shift_for((uint64_t)z0 - a0 + 1);
        wg_hist<NT>(xs, kMedSample, a0, z0, s1, lh);
        const uint32_t n0 = wg_narrow<NT>(lh, wt, part, s1, a0, z0, r0, false);
        const uint32_t n2 = wg_narrow<NT>(lh, wt, part, s1, a2, z2, r2, true);
        narrow_end(n0, a0, z0, r0);
        narrow_end(n2, a2, z2, r2);
        lo0 = a0;
        hi2 = z2;
    }
    if (exact && !all) {  // the passes add into a clear histogram and fresh segment counters
        for (int b = tid; b < 3 * kMedBins; b += NT) v.hist[b] = 0;
        for (int g = tid; g < kCandSegs; g += NT) sel->seg[g][0] = 0;
    }
    if (tid != 0) return;
    if (!exact || all) {
        set_bandwidth(sel, N, m, h_out);
        sel->mode = kModeDone;
        return;
    }
    sel->lo = lo0;
    sel->hi = hi2;
    sel->rank = (uint32_t)((P + 1) / 2);
    sel->arrived = 0;
    sel->mode = kModePass0;
}

// ---- candidate lists -----------------------------------------------------------
// Pass 0 appends about one pair in twenty.  Each lane keeps its own list, a
// column of the wave's LDS region [kDepth + 1][64]: every value is stored at
// the lane's next place and the place advances when the value is inside the
// bracket, so an append is one count, one address and one LDS store with no
// ballot and nothing shared between lanes (a wave-wide compaction per value
// took 34 VALU and scalar instructions and made every value wait for the one
// before it).  The flush compacts: place by place, the lanes that hold a value
// write it to consecutive slots.
constexpr int kListStep = 4;  // values a lane may take between two depth checks
template <int DEPTH>
struct LaneList {
    uint32_t* col;  // this lane's column
    uint32_t cnt = 0, nb = 0;  // values held; pairs below the bracket since the last flush
    uint32_t nb_wave = 0;      // more of them, counted for the whole wave
    uint32_t flushes = 0;
    static constexpr int kWords = (DEPTH + 1) * 64;
    __device__ __forceinline__ void put(uint32_t x, bool in) {
        col[cnt * 64] = x;
        cnt += in ? 1u : 0u;
    }
    // The next flush's segment (hashed, so that the segments fill evenly).
    __device__ __forceinline__ int segment() {
        const uint32_t w = (blockIdx.x << 4) + (threadIdx.x >> 6);
        return (int)(mix32(w + mix32(flushes++)) % kCandSegs);
    }
    // Room for another kListStep values in every lane (wave-uniform).
    __device__ __forceinline__ bool full() const { return __any(cnt > (uint32_t)(DEPTH - kListStep)); }
};

// Sum over the wave (wave-uniform), by DPP moves: no LDS round trips.
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true);  // row_half_mirror
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, true);  // row_mirror: every lane its row's sum
    uint32_t t = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) t += (uint32_t)__builtin_amdgcn_readlane((int)x, 16 * r);
    return t;
}

// The wave's lists to its candidate segment in one reservation, which also
// counts its pairs below the bracket.  conv(x): the distance's bit pattern.
template <int DEPTH, class F>
__device__ __forceinline__ void flush_lists(const MedView& v, LaneList<DEPTH>& l, F&& conv) {
    const int lane = threadIdx.x & 63, seg = l.segment();
    const uint32_t tot = wave_sum(l.cnt), below = wave_sum(l.nb) + l.nb_wave;
    const uint32_t seg_cap = v.seg_cap;
    uint32_t base = 0;
    if (lane == 0 && (tot | below))
        base = (uint32_t)atomicAdd(&v.sel->seg[seg][0], ((unsigned long long)below << 32) | tot);
    base = __builtin_amdgcn_readfirstlane(base);
    uint32_t* segbuf = v.cand + (size_t)seg * seg_cap;
    static_assert(DEPTH % 4 == 0, "the values leave four places at a time");
    for (uint32_t s = 0; __any(l.cnt > s); s += 4) {
        uint32_t x[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) x[u] = l.col[(s + u) * 64];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) {
            const bool has = l.cnt > s + u;
            const uint64_t m = __ballot(has);
            const uint32_t pos =
                base + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (has && pos < seg_cap) segbuf[pos] = conv(x[u]);
            base += (uint32_t)__popcll(m);
        }
    }
    l.cnt = l.nb = l.nb_wave = 0;
}

// What a pass over every pair does with a pair: pass 0, or the histogram of
// [lo, hi] into lh.
constexpr int kPass0 = 0, kPassHist = 1;

// ---- all-pairs work item (row block rb, column chunk cc) ---------------------------
// 256 threads: ROWS rows and 256 / ROWS column groups (a 64-row item gives each
// wave a quarter of the columns, so small problems still fill the chip).  A
// thread measures four columns at a time (four independent FMA chains, 16-byte
// LDS broadcasts); each distance is summed over the coordinates in order, the
// coordinates past d, which are zero, skipped four at a time.
template <int ROWS>
constexpr int kItemDepth = ROWS == 64 ? 16 : 32;  // 16 columns a wave, or 64

template <int DP, int ROWS, int MODE>
__device__ void med_item(const MedView& v, const float* __restrict__ theta, int rb, int cc, uint32_t lo, uint32_t hi,
                         uint32_t s, uint32_t* lh) {
    constexpr int NT = 256;
    constexpr int CG = NT / ROWS;       // column groups
    constexpr int CPG = kMedCols / CG;  // columns per group
    constexpr int LD = DP + 4;          // staged row stride: 16-byte aligned rows
    constexpr int DEPTH = kItemDepth<ROWS>;
    using List = LaneList<DEPTH>;
    static_assert(NT % ROWS == 0 && CPG % kListStep == 0 && ROWS % 64 == 0, "item shape");
    static_assert(kMedCols * DP % NT == 0, "staging covers the columns exactly");
    __shared__ __align__(16) float tj[kMedCols][LD];
    __shared__ uint32_t lists[MODE == kPass0 ? NT / 64 : 1][MODE == kPass0 ? List::kWords : 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int rloc = tid % ROWS, cg = tid / ROWS;
    const int N = v.N, d = v.d;
    const int row0 = rb * ROWS, col0 = cc * kMedCols;
    if (col0 + kMedCols <= row0 + 1) return;  // no pair i < j in this item
    if (MODE != kPass0) __syncthreads();      // a pass takes several items: the columns before are read
    {  // stage the columns: consecutive threads read consecutive columns
        constexpr int SPT = kMedCols * DP / NT;
        float x[SPT];
#pragma unroll
        for (int u = 0; u < SPT; ++u) {
            const int e = tid + NT * u, c = e % kMedCols, l = e / kMedCols;
            const int j = col0 + c;
            x[u] = (j < N && l < d) ? theta[(int64_t)l * N + j] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < SPT; ++u) {
            const int e = tid + NT * u;
            tj[e % kMedCols][e / kMedCols] = x[u];
        }
    }
    const int i = row0 + rloc;
    float ti[DP];
#pragma unroll
    for (int l = 0; l < DP; ++l) ti[l] = (i < N && l < d) ? theta[(int64_t)l * N + i] : 0.0f;
    __syncthreads();
    List list;
    list.col = lists[MODE == kPass0 ? tid >> 6 : 0] + (MODE == kPass0 ? lane : 0);
    auto same = [](uint32_t x) { return x; };
    const uint32_t wlo = hi - lo;  // x in [lo, hi] iff x - lo <= hi - lo (unsigned)
    // the wave's columns, from the first one past its first row (j > i)
    const int wrow0 = row0 + (rloc & ~63);
    const int cbeg = cg * CPG, cend = cbeg + CPG;
    const int jskip = wrow0 + 1 - col0 - cbeg;
    const int cstart = cbeg + (jskip > 0 ? (jskip & ~3) : 0);
    for (int c = cstart; c < cend; c += 4) {
        if (MODE == kPass0 && CPG > DEPTH && list.full())
            flush_lists(v, list, same);
        float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int l = 0; l < DP; l += 4) {
            if (l < d) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 t = *reinterpret_cast<const float4*>(&tj[c + q][l]);
                    float df = ti[l] - t.x;
                    acc[q] = fmaf(df, df, acc[q]);
                    df = ti[l + 1] - t.y;
                    acc[q] = fmaf(df, df, acc[q]);
                    df = ti[l + 2] - t.z;
                    acc[q] = fmaf(df, df, acc[q]);
                    df = ti[l + 3] - t.w;
                    acc[q] = fmaf(df, df, acc[q]);
                }
            }
        }
        const int jb = col0 + c;
        auto classify = [&](auto whole_tag) __attribute__((always_inline)) {
            constexpr bool WHOLE = decltype(whole_tag)::value;  // every pair of the four columns is one
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t x = __float_as_uint(acc[q]);
                bool valid = true;
                if constexpr (!WHOLE) {
                    const int j = jb + q;
                    valid = i < N && j < N && j > i;
                }
                if (MODE == kPass0) {
                    if constexpr (!WHOLE) x = valid ? x : 0xffffffffu;  // above every bracket (hi is no NaN)
                    list.nb += x < lo ? 1u : 0u;
                    list.put(x, x - lo <= wlo);
                } else {
                    const bool in = valid && x - lo <= wlo;
                    if (in) atomicAdd(&lh[(x - lo) >> s], 1u);
                }
            }
        };
        if (MODE == kPass0 && jb > wrow0 + 63 && jb + 4 <= N) classify(std::true_type{});  // wave-uniform
        else classify(std::false_type{});
    }
    if (MODE == kPass0) flush_lists(v, list, same);
}

// The same with the distances in Gram form on the matrix cores, from the
// centred rows the FP32 contraction uses (built before the median):
// S = x_i . x_j + (e_i + e_j) with e = -|x|^2 / 2, D_ij = max(-2 S, 0).  Each
// wave takes 64 rows as four 16-row tiles, of its own in a 256-row block, shared
// by the four waves, which take a 16-column quarter each, in a 64-row block.  Per 16 columns
// and row tile the MFMAs give S[i][j] with lane l holding rows 4 (l / 16) + t
// of column l % 16.  KS > 0: KS FP32 products (16x16x4) and the two e added
// after.  KS = 0 is the split form (d <= 31): the rows as three BF16 parts and
// x_i . x_j as the six part products of order >= 2^-16 on the BF16 matrix cores
// (16x16x32, the same output layout), FP32-accurate as the FP32 direction's
// split form (the contraction's e_j in slot 31 meets a zero of the row operand).
// Every pass computes a pair's S with the same instructions, so the counts stay
// exact.
//
// Pass 0 classifies S itself: D in [lo, hi] iff S in [-hi/2, -lo/2] (exact
// halves of normal values), whose bit patterns are consecutive.  Bounds this
// does not hold for (a subnormal or zero lo, an infinite hi) take the general
// classification on D.
// Bound: VALU issue, eight instructions a value beside six MFMAs per four
// values a lane (45 us of issue at N = 16384).  d = 30, a grid of equal items
// and a compaction per value -> one resident round of equal runs and lane lists:
// N = 16384 129 -> 74 us (a quarter of it the appends), 8192 46 -> 27 us.
// The split form's part products (row part, column part), smallest first.
__device__ constexpr int kGramPairs3[6][2] = {{1, 1}, {2, 0}, {0, 2}, {1, 0}, {0, 1}, {0, 0}};

// A workgroup's share of the sweep: the steps (16 columns for each wave of a
// 256-row block; 64 columns, 16 a wave, of a 64-row block) of row block after
// row block from its diagonal to the last column, counted through, in equal
// runs of consecutive steps.  A run that ends in one row block goes on in the
// next.
struct GramSteps {
    int cols, per, rb;  // steps of the first row block, steps fewer per block, row blocks
    __host__ __device__ int64_t before(int64_t r) const { return r * cols - per * (r * (r - 1) / 2); }
    __host__ __device__ int64_t count() const { return before(rb); }
    __device__ int block_of(int64_t t) const {  // the row block of step t
        int a = 0, b = rb;                      // before(a) <= t < before(b)
        while (b - a > 1) {
            const int m = (a + b) >> 1;
            if (before(m) <= t) a = m;
            else b = m;
        }
        return a;
    }
};

__host__ __device__ __forceinline__ GramSteps gram_steps(int N, int rows, int rb) {
    return rows == 256 ? GramSteps{(N + 15) / 16, 16, rb} : GramSteps{(N + 63) / 64, 1, rb};
}

template <int KS, int ROWS, int MODE>
__device__ void med_gram(const MedView& v, int blk, int nblk, uint32_t lo, uint32_t hi, uint32_t s, uint32_t* lh) {
    constexpr int NT = 256;
    constexpr int DEPTH = 32;
    using List = LaneList<DEPTH>;
    static_assert(ROWS == 64 || ROWS == 256, "item shape");
    __shared__ uint32_t lists[MODE == kPass0 ? NT / 64 : 1][MODE == kPass0 ? List::kWords : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kq = lane >> 4;
    const int N = v.N;
    const GramSteps steps = gram_steps(N, ROWS, v.rb);
    const uint32_t n_steps = (uint32_t)steps.count(), per = n_steps / nblk, more = n_steps % nblk;
    const int64_t t0 = (int64_t)per * blk + min((uint32_t)blk, more), t1 = t0 + per + ((uint32_t)blk < more ? 1 : 0);
    if (t0 == t1) return;
    constexpr int cstep = ROWS == 256 ? 16 : 64;
    constexpr bool SPLIT = KS == 0;
    constexpr int KA = SPLIT ? 1 : KS;   // FP32 operand steps
    constexpr int NP = SPLIT ? 3 : 1;    // split-form parts
    List list;
    list.col = lists[MODE == kPass0 ? wave : 0] + (MODE == kPass0 ? lane : 0);
    auto load = [&](int c, float (&x)[KA], bf16x8v (&x3)[NP], float& e) __attribute__((always_inline)) {
        if constexpr (SPLIT) {
            const __bf16* p = v.xs3 + (int64_t)(c + col) * 96 + 8 * kq;
#pragma unroll
            for (int q = 0; q < NP; ++q) x3[q] = *reinterpret_cast<const bf16x8v*>(p + 32 * q);
        } else {
            const float* p = v.xr + (int64_t)(c + col) * (4 * KS) + kq * KS;
#pragma unroll
            for (int k = 0; k < KS; ++k) x[k] = p[k];
        }
        e = v.nrm[c + col] * -0.5f;
    };
    const uint32_t wlo = hi - lo;
    // the bracket in S: bits of -lo/2 and -hi/2
    const float slo = __uint_as_float(lo) * -0.5f;
    const uint32_t blo = __float_as_uint(slo), bw = __float_as_uint(__uint_as_float(hi) * -0.5f) - blo;
    auto dist_bits = [](float S) { return __float_as_uint(fmaxf(-2.0f * S, 0.0f)); };
    using std::false_type;
    using std::true_type;
    auto sweep = [&](auto fast_tag) __attribute__((always_inline)) {
        constexpr bool FAST = decltype(fast_tag)::value;
        auto conv = [&](uint32_t x) { return FAST ? dist_bits(__uint_as_float(x)) : x; };
        int rb = steps.block_of(t0);
        int64_t before = steps.before(rb);
        for (int64_t t = t0; t < t1; ++rb) {
            // columns [c0, cend) of this row block, for this wave
            const int64_t after = before + steps.cols - (int64_t)steps.per * rb, end = t1 < after ? t1 : after;
            const int wrow = rb * ROWS + (ROWS == 256 ? 64 * wave : 0);
            const int off = rb * ROWS + (ROWS == 256 ? 0 : 16 * wave);
            int c0 = off + (int)(t - before) * cstep;
            const int cend = off + (int)(end - before) * cstep;
            t = end;
            before = after;
            while (c0 < cend && c0 + 15 <= wrow) c0 += cstep;  // no pair j > i for the wave's rows
            if (c0 >= cend) continue;
            float xa[4][KA];
            bf16x8v xa3[NP][4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (SPLIT) {
                    const __bf16* p = v.xs3 + (int64_t)(wrow + 16 * r + col) * 96 + 8 * kq;
#pragma unroll
                    for (int q = 0; q < NP; ++q) {
                        xa3[q][r] = *reinterpret_cast<const bf16x8v*>(p + 32 * q);
                        if (kq == 3) xa3[q][r][7] = (__bf16)0.0f;
                    }
                } else {
                    const float* p = v.xr + (int64_t)(wrow + 16 * r + col) * (4 * KS) + kq * KS;
#pragma unroll
                    for (int k = 0; k < KS; ++k) xa[r][k] = p[k];
                }
            }
            f4v ei[4];  // e_i for i = wrow + 16 r + 4 kq + t
#pragma unroll
            for (int r = 0; r < 4; ++r) ei[r] = *reinterpret_cast<const f4v*>(v.nrm + wrow + 16 * r + 4 * kq) * -0.5f;
            float xb[KA];
            bf16x8v xb3[NP];
            float ej = 0.0f;
            auto step = [&](int c, const float (&xb)[KA], const bf16x8v (&xb3)[NP], float ej) __attribute__((always_inline)) {
                const int jb = c, j = jb + col;
                // two row tiles at a time: their products in turn, two chains in
                // flight beside the other waves', then their sixteen pairs
                auto tiles = [&](int r0, float (&S)[8]) __attribute__((always_inline)) {
                    f4v a[2] = {};
                    if constexpr (SPLIT) {
#pragma unroll
                        for (int e = 0; e < 6; ++e)
#pragma unroll
                            for (int r = 0; r < 2; ++r)
                                a[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    xa3[kGramPairs3[e][0]][r0 + r], xb3[kGramPairs3[e][1]], a[r], 0, 0, 0);
                    } else {
#pragma unroll
                        for (int k = 0; k < KS; ++k)
#pragma unroll
                            for (int r = 0; r < 2; ++r)
                                a[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[r0 + r][k], xb[k], a[r], 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int t = 0; t < 4; ++t) S[4 * r + t] = a[r][t] + (ei[r0 + r][t] + ej);
                };
                auto classify = [&](auto whole_tag, int r0, const float (&S)[8]) __attribute__((always_inline)) {
                    constexpr bool WHOLE = decltype(whole_tag)::value;  // every pair of the step is one
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        if (MODE == kPass0 && e % kListStep == 0 && list.full()) flush_lists(v, list, conv);
                        bool valid = true;
                        if constexpr (!WHOLE) {
                            const int i = wrow + 16 * (r0 + (e >> 2)) + 4 * kq + (e & 3);
                            valid = i < N && j < N && j > i;
                        }
                        if (FAST) {
                            float x = S[e];
                            if constexpr (!WHOLE) x = valid ? x : -INFINITY;  // above the bracket
                            // a NaN counts as D = 0, as max(-2 S, 0) does; counted by the scalar unit
                            list.nb_wave += (uint32_t)__popcll(__ballot(!(x <= slo)));
                            const uint32_t b = __float_as_uint(x);
                            list.put(b, b - blo <= bw);
                        } else {
                            const uint32_t x = dist_bits(S[e]);
                            const bool in = valid && x - lo <= wlo;
                            if (MODE == kPass0) {
                                list.nb += valid && x < lo ? 1u : 0u;
                                list.put(x, in);
                            } else if (in) {
                                atomicAdd(&lh[(x - lo) >> s], 1u);
                            }
                        }
                    }
                };
                const bool whole = FAST && jb > wrow + 63 && jb + 16 <= N;  // wave-uniform
#pragma unroll
                for (int r0 = 0; r0 < 4; r0 += 2) {
                    float S[8];
                    tiles(r0, S);
                    if (whole) classify(true_type{}, r0, S);
                    else classify(false_type{}, r0, S);
                }
            };
            // no prefetch: four waves on a SIMD hide the loads, and a second
            // operand buffer would not fit their registers
            for (int c = c0; c < cend; c += cstep) {
                load(c, xb, xb3, ej);
                step(c, xb, xb3, ej);
            }
        }
        if (MODE == kPass0) flush_lists(v, list, conv);
    };
    if constexpr (MODE == kPass0) {
        if (lo >= 0x01000000u && hi < 0x7f800000u) sweep(true_type{});
        else sweep(false_type{});
    } else {
        sweep(false_type{});
    }
}

// ---- the passes after pass 0 -------------------------------------------------------
// blk of nblk workgroups of 256; items(lo, hi, s, lh) histograms this
// workgroup's share of all pairs.
//   1: where rank k lies (the bracket's candidates, or, when it lies outside
//      or a segment overflowed, every pair), and the histogram of that interval;
//   2: the bin with rank k, and its histogram;
//   3: the bin with rank k of that; if it is wider than one value (a bracket
//      of more than 2^22 patterns) the next histogram, which the workgroup that
//      ends last narrows to the one value left.
// Every workgroup derives the interval itself from the counts before it, so no
// launch of a single workgroup sits between the passes.
struct Interval {
    uint32_t lo, hi, rank;
};

template <class Items>
__device__ __forceinline__ void pass_values(const MedView& v, int blk, int nblk, bool all, const Interval& I, uint32_t s,
                                            uint32_t* lh, Items&& items) {
    if (all) {
        items(I.lo, I.hi, s, lh);
        return;
    }
    const int parts = nblk / kCandSegs, g = blk / parts, part = blk % parts;
    const uint32_t got = (uint32_t)v.sel->seg[g][0];
    const uint32_t n = got < v.seg_cap ? got : v.seg_cap;
    const uint32_t per = ((n + parts - 1) / parts + 3) & ~3u, b0 = (uint32_t)part * per;
    if (b0 >= n) return;
    wide_hist(v.cand + (size_t)g * v.seg_cap + b0, b0 + per < n ? per : n - b0, I.lo, I.hi, s, lh);
}

// The interval's bin with rank I.rank in the histogram h (shift s), by the
// workgroup; the number of values in it.
__device__ __forceinline__ uint32_t narrow_from(const uint32_t* __restrict__ h, uint32_t s, Interval& I, uint32_t* lh,
                                                uint32_t* wt, uint32_t* part) {
    for (int b = threadIdx.x; b < kMedBins; b += 256) lh[b] = h[b];
    return wg_narrow<256>(lh, wt, part, s, I.lo, I.hi, I.rank);
}

template <class Items>
__device__ __forceinline__ void med_pass(const MedView& v, int pass, int blk, int nblk, float* h_out, Items&& items) {
    __shared__ uint32_t lh[kMedBins];
    __shared__ __align__(16) uint32_t wt[4];
    __shared__ uint32_t part[4];
    SelState* sel = v.sel;
    if (sel->mode != kModePass0) return;
    const int tid = threadIdx.x;
    auto flush = [&](uint32_t* h) {
        __syncthreads();
        for (int b = tid; b < kMedBins; b += 256)
            if (lh[b]) atomicAdd(&h[b], lh[b]);
    };
    if (pass == 1) {
        const uint32_t seg_cap = v.seg_cap;
        const unsigned long long q = sel->seg[tid & 63][0];
        static_assert(kCandSegs == 64, "a lane per segment");
        const uint32_t inside = wave_sum((uint32_t)q), below = wave_sum((uint32_t)(q >> 32));
        bool all = __any((uint32_t)q > seg_cap);
        Interval I{sel->lo, sel->hi, sel->rank};
        if (I.rank <= below) {
            all = true;
            I.hi = I.lo - 1;
            I.lo = 0;
        } else if (I.rank > below + inside) {
            all = true;
            I.rank -= below + inside;
            I.lo = I.hi + 1;
            I.hi = 0xffffffffu;
        } else {
            I.rank -= below;
        }
        if (blk == 0 && tid == 0) {
            sel->lo1 = I.lo;
            sel->hi1 = I.hi;
            sel->rank1 = I.rank;
            sel->all = all;
        }
        if (I.lo == I.hi) return;
        for (int b = tid; b < kMedBins; b += 256) lh[b] = 0;
        __syncthreads();
        pass_values(v, blk, nblk, all, I, shift_for((uint64_t)I.hi - I.lo + 1), lh, items);
        flush(v.hist);
        return;
    }
    const bool all = sel->all != 0;
    Interval I{sel->lo1, sel->hi1, sel->rank1};
    if (pass == 2) {
        if (I.lo == I.hi) return;
        narrow_from(v.hist, shift_for((uint64_t)I.hi - I.lo + 1), I, lh, wt, part);  // clears lh
        if (blk == 0 && tid == 0) {
            sel->lo2 = I.lo;
            sel->hi2 = I.hi;
            sel->rank2 = I.rank;
        }
        if (I.lo == I.hi) return;
        pass_values(v, blk, nblk, all, I, shift_for((uint64_t)I.hi - I.lo + 1), lh, items);
        flush(v.hist + kMedBins);
        return;
    }
    if (I.lo != I.hi) I = Interval{sel->lo2, sel->hi2, sel->rank2};
    if (I.lo != I.hi) narrow_from(v.hist + kMedBins, shift_for((uint64_t)I.hi - I.lo + 1), I, lh, wt, part);
    if (I.lo == I.hi) {
        if (blk == 0 && tid == 0) set_bandwidth(sel, v.N, I.lo, h_out);
        return;
    }
    const uint32_t s = shift_for((uint64_t)I.hi - I.lo + 1);
    pass_values(v, blk, nblk, all, I, s, lh, items);
    flush(v.hist + 2 * kMedBins);
    __threadfence();  // this workgroup's counts before its arrival
    __syncthreads();
    if (tid == 0) part[3] = atomicAdd(&sel->arrived, 1u);
    __syncthreads();
    if (part[3] != (uint32_t)nblk - 1) return;
    __threadfence();
    for (int b = tid; b < kMedBins; b += 256) lh[b] = __hip_atomic_load(&v.hist[2 * kMedBins + b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wg_narrow<256>(lh, wt, part, s, I.lo, I.hi, I.rank);
    if (tid == 0) set_bandwidth(sel, v.N, I.lo, h_out);
}

// Small problems (P <= kFinishPairs): everything after pass 0 in one
// workgroup of kFinishThreads.  The counts decide where rank k lies.  Inside
// the bracket (and without overflow) the candidates are read into registers
// once and histogram passes over them narrow the interval (two, for the usual
// bracket width).  Else (rare) histogram passes run over every pair,
// recomputed here.
constexpr uint64_t kFinishPairs = 1ull << 20;

// Problems above kFinishPairs pairs take the Gram-form distances in their
// all-pairs passes (when the caller provides the operands); smaller ones keep
// direct differences, in the single-problem and the batched paths alike, so
// both reach the same bandwidth bit for bit.
__host__ __device__ __forceinline__ bool med_takes_gram(int N) { return pair_count(N) > kFinishPairs; }
constexpr int kFinishThreads = 1024;
constexpr int kFinishRegs = 40;         // candidate slots per thread held in registers
constexpr int kSegThreads = kFinishThreads / kCandSegs;
static_assert(kFinishThreads % kCandSegs == 0, "whole thread groups per candidate segment");

__device__ void med_finish_body(const MedView& v, const float* __restrict__ theta, float* h_out) {
    constexpr int NT = kFinishThreads;
    __shared__ uint32_t lh[kMedBins];
    __shared__ __align__(16) uint32_t wt[NT / 64];
    __shared__ uint32_t part[4];
    const int tid = threadIdx.x;
    SelState* sel = v.sel;
    if (sel->mode != kModePass0) return;
    const int N = v.N, d = v.d;
    uint32_t lo = sel->lo, hi = sel->hi;
    uint32_t r = sel->rank;
    const uint32_t seg_cap = v.seg_cap;
    const unsigned long long q64 = sel->seg[tid & 63][0];
    const uint32_t inside = wave_sum((uint32_t)q64), below = wave_sum((uint32_t)(q64 >> 32));
    const bool overflow = __any((uint32_t)q64 > seg_cap);
    for (int q = tid; q < kMedBins; q += NT) lh[q] = 0;
    __syncthreads();
    if (r > below && r <= below + inside && !overflow) {
        // select among the candidates in [lo, hi] (sentinels lie above hi)
        r -= below;
        const int g = tid / kSegThreads, sub = tid % kSegThreads;
        const uint32_t n = (uint32_t)sel->seg[g][0];
        const uint32_t* sb = v.cand + (size_t)g * seg_cap;
        // the first kFinishRegs * kSegThreads slots of each segment stay in
        // registers (one load round trip); longer segments stream the rest
        constexpr uint32_t nreg = kFinishRegs * kSegThreads;
        // slots past n lie inside the segment (at least kCandSegMin slots) and
        // read as sentinels
        static_assert(kFinishRegs * kSegThreads <= (int)kCandSegMin, "register slots inside every segment");
        uint32_t xr[kFinishRegs];
#pragma unroll
        for (int u = 0; u < kFinishRegs; ++u) xr[u] = sb[sub + kSegThreads * u];
#pragma unroll
        for (int u = 0; u < kFinishRegs; ++u)
            if ((uint32_t)(sub + kSegThreads * u) >= n) xr[u] = kSentinel;
        auto hist_pass = [&](uint32_t s) {
            const uint32_t w = hi - lo;
#pragma unroll
            for (int u = 0; u < kFinishRegs; ++u) {
                const uint32_t dx = xr[u] - lo;  // in [lo, hi] iff dx <= hi - lo (unsigned)
                if (dx <= w) atomicAdd(&lh[dx >> s], 1u);
            }
            if (n > nreg) strided_hist<kSegThreads>(sb + nreg, n - nreg, sub, lo, hi, s, lh);
        };
        while (lo < hi) {  // each pass narrows the width 2048-fold: two passes, usually
            const uint32_t s = shift_for((uint64_t)hi - lo + 1);
            hist_pass(s);
            wg_narrow<NT>(lh, wt, part, s, lo, hi, r);
        }
        if (tid == 0) set_bandwidth(sel, N, lo, h_out);
        return;
    }
    if (r <= below) {
        hi = lo - 1;
        lo = 0;
    } else if (r > below + inside) {
        r -= below + inside;
        lo = hi + 1;
        hi = 0xffffffffu;
    } else {
        r -= below;  // inside, but the candidates overflowed
    }
    while (lo < hi) {  // histogram passes over every pair (rare)
        const uint32_t s = shift_for((uint64_t)hi - lo + 1);
        for (int i = tid; i < N; i += NT)
            for (int j = i + 1; j < N; j += 4) {  // four at once share the row's loads
                float acc[4] = {};
                for (int l = 0; l < d; ++l) {
                    const float* t = theta + (int64_t)l * N;
                    const float ti = t[i];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float df = ti - t[min(j + q, N - 1)];
                        acc[q] = fmaf(df, df, acc[q]);
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t x = __float_as_uint(acc[q]);
                    if (j + q < N && x >= lo && x <= hi) atomicAdd(&lh[(x - lo) >> s], 1u);
                }
            }
        wg_narrow<NT>(lh, wt, part, s, lo, hi, r);
    }
    if (tid == 0) set_bandwidth(sel, N, lo, h_out);
}

// The items with a pair i < j, counted column group by column group (`width`
// columns a group, a multiple of `rows` or a divisor): below(g) = items of the
// groups before g, whose items are their first row blocks.  The grid holds
// only these: workgroups go to the shader engines in turn, whether or not an
// engine is free, and a (row block, column group) grid, half of it below the
// diagonal, gives one engine up to three times the items of another (the Gram
// form of N = 16384 on such a grid took 102 us, on a list like this 82).
struct ItemList {
    int rows, width, rb, groups;
    __host__ __device__ int64_t below(int64_t g) const {
        if (width >= rows) return (width / rows) * (g * (g + 1) / 2);
        const int64_t m = rows / width, q = g / m;
        return m * (q * (q + 1) / 2) + (g % m) * (q + 1);
    }
    __host__ __device__ int64_t count() const {
        const int64_t last = below(groups) - below(groups - 1);
        return below(groups - 1) + (last < rb ? last : rb);
    }
    // item t's row block and column group
    __device__ void at(int64_t t, int& r, int& g) const {
        g = (int)sqrtf(2.0f * (float)rows / (float)width * (float)t);
        while (g > 0 && below(g) > t) --g;
        while (below(g + 1) <= t) ++g;
        r = (int)(t - below(g));
    }
};

__host__ __device__ __forceinline__ ItemList item_list(int rows, int rb, int cc) {
    return ItemList{rows, kMedCols, rb, cc};
}

// ---- single-problem kernels -----------------------------------------------------
struct OneMed {
    int N, d;
    float fixed_h;
    SvgdLayout L;
    char* ws;
};

// The step's first two launches, each of two stages that do not depend on each
// other: the sample distances (four lanes a slot, 64 slots a workgroup) beside
// the coordinates' means, then the select (the first workgroup, of 1024)
// beside the packing of the centred rows (256 a workgroup).  All four are
// latency: with a launch for each the step took 45.6 us at N = 1024, d = 18 and
// 33.9 at N = 32, in pairs 40.2 and 23.4.  n_dist = 0 or no centre workgroups
// leave a stage out.
template <int NT>
__global__ __launch_bounds__(256) void k_med_gather(OneMed a, const float* theta, int n_dist) {
    const int b = blockIdx.x;
    if (b >= n_dist) {
        particle_mean_body<NT, 256>(a.N, b - n_dist, theta, reinterpret_cast<float*>(a.ws + a.L.ctr_off));
        return;
    }
    const int t = b * 64 + (threadIdx.x >> 2), q = threadIdx.x & 3;
    const float v = sample_dist4(a.N, a.d, t, q, theta);
    if (q == 0) med_view(a.N, a.d, a.fixed_h, a.L, a.ws).smp[t] = v;
}

__global__ __launch_bounds__(kSelThreads) void k_sample_select(OneMed a, int exact, float* h_out) {
    sample_select_body(med_view(a.N, a.d, a.fixed_h, a.L, a.ws), exact, h_out);
}

constexpr int kPackRows = 256;  // rows of a packing workgroup of kSelThreads
__global__ __launch_bounds__(kSelThreads) void k_select_pack(OneMed a, const float* theta, int exact, float* h_out) {
    if (blockIdx.x == 0) sample_select_body(med_view(a.N, a.d, a.fixed_h, a.L, a.ws), exact, h_out);
    else
        pack32_x_rows<kSelThreads / 256>(a.N, a.d, a.L.ks32, (blockIdx.x - 1) * kPackRows, theta, view32(a.L, a.ws),
                                         a.L.split3);
}

// The FP32 operands at a given bandwidth, in two launches: the means, then the
// packing, whose first thread records h.  With nothing beside them to hide in, the
// two stages take their own shapes, 1024 threads a mean and 64 rows a workgroup
// (by the launches above: a step of 8192 particles, d = 30, 72.6 us, now 67.8; 3001, d = 48
// 71.3, now 61.4).
__global__ __launch_bounds__(kMeanThreads) void k_mean(OneMed a, const float* theta) {
    particle_mean_body(a.N, blockIdx.x, theta, reinterpret_cast<float*>(a.ws + a.L.ctr_off));
}

__global__ __launch_bounds__(256) void k_pack_given(OneMed a, const float* theta, float* h_out) {
    if (blockIdx.x == 0 && threadIdx.x == 0) given_bandwidth(med_view(a.N, a.d, a.fixed_h, a.L, a.ws), h_out);
    pack32_x_rows(a.N, a.d, a.L.ks32, blockIdx.x * 64, theta, view32(a.L, a.ws), a.L.split3);
}

template <int DP, int ROWS>
__global__ __launch_bounds__(256) void k_med_items(OneMed a, const float* theta) {
    const MedView v = med_view(a.N, a.d, a.fixed_h, a.L, a.ws);
    if (v.sel->mode != kModePass0) return;
    int rb, g;
    item_list(ROWS, v.rb, v.cc).at(blockIdx.x, rb, g);
    med_item<DP, ROWS, kPass0>(v, theta, rb, g, v.sel->lo, v.sel->hi, 0, nullptr);
}

template <int KS, int ROWS>
__device__ __forceinline__ void gram_pass0(const MedView& v, int blk, int nblk) {
    if (v.sel->mode != kModePass0) return;
    med_gram<KS, ROWS, kPass0>(v, blk, nblk, v.sel->lo, v.sel->hi, 0, nullptr);
}

template <int KS, int ROWS>
__global__ __launch_bounds__(256, 4) void k_med_items_gram(OneMed a) {
    const MedView v = med_view(a.N, a.d, a.fixed_h, a.L, a.ws);
    gram_pass0<KS, ROWS>(v, blockIdx.x, gridDim.x);
}

// passes 1..3 (grid: a multiple of kCandSegs workgroups)
template <int DP, int ROWS>
__global__ __launch_bounds__(256) void k_med_pass(OneMed a, const float* theta, int pass, float* h_out) {
    const MedView v = med_view(a.N, a.d, a.fixed_h, a.L, a.ws);
    med_pass(v, pass, blockIdx.x, gridDim.x, h_out,
             [&](uint32_t lo, uint32_t hi, uint32_t s, uint32_t* lh) {
                 const ItemList l = item_list(ROWS, v.rb, v.cc);
                 const int64_t n = l.count();
                 for (int64_t it = blockIdx.x; it < n; it += gridDim.x) {
                     int rb, g;
                     l.at(it, rb, g);
                     med_item<DP, ROWS, kPassHist>(v, theta, rb, g, lo, hi, s, lh);
                 }
             });
}

template <int KS, int ROWS>
__device__ __forceinline__ void gram_pass(const MedView& v, int pass, int blk, int nblk, float* h_out) {
    med_pass(v, pass, blk, nblk, h_out, [&](uint32_t lo, uint32_t hi, uint32_t s, uint32_t* lh) {
        med_gram<KS, ROWS, kPassHist>(v, blk, nblk, lo, hi, s, lh);
    });
}

template <int KS, int ROWS>
__global__ __launch_bounds__(256) void k_med_pass_gram(OneMed a, int pass, float* h_out) {
    gram_pass<KS, ROWS>(med_view(a.N, a.d, a.fixed_h, a.L, a.ws), pass, blockIdx.x, gridDim.x, h_out);
}

__global__ __launch_bounds__(kFinishThreads) void k_med_finish(OneMed a, const float* theta, float* h_out) {
    med_finish_body(med_view(a.N, a.d, a.fixed_h, a.L, a.ws), theta, h_out);
}

// ---- batched kernels ---------------------------------------------------------------
__device__ __forceinline__ MedView med_of(const ProblemDesc& D, char* ws) {
    return med_view(D.N, D.d, D.fixed_h, D.sv, ws + D.svgd_off);
}

__global__ __launch_bounds__(kSelThreads) void k_sample_select_batched(const ProblemDesc* __restrict__ descs, char* ws,
                                                                int exact) {
    sample_select_body(med_of(descs[blockIdx.x], ws), exact, nullptr);
}

// np problems' selects, then the packing: entry = (problem, first row of a
// 256-row chunk, -, -)
__global__ __launch_bounds__(kSelThreads) void k_select_pack_batched(const ProblemDesc* __restrict__ descs, int np,
                                                                     const int4* __restrict__ work, const float* theta,
                                                                     char* ws) {
    if ((int)blockIdx.x < np) {
        sample_select_body(med_of(descs[blockIdx.x], ws), 1, nullptr);
        return;
    }
    const int4 e = work[blockIdx.x - np];
    const ProblemDesc& D = descs[e.x];
    if (D.N < 2) return;
    pack32_x_rows<kSelThreads / 256>(D.N, D.d, D.sv.ks32, e.y, theta + D.theta_off, view32(D.sv, ws + D.svgd_off),
                                     D.sv.split3);
}

// A batch's first launch, and with the select the BF16 form's whole bandwidth
// stage: blocks below nd = (kMedSample / 64) x problems gather the sample distances (four lanes a
// slot), the rest take one entry (problem, coordinate) of the centre list
// each (NT partial sums).  A non-null step counter is advanced once (a solve's
// iteration counter, read by the update at the iteration's end).
template <int NT>
__global__ __launch_bounds__(256) void k_gather_batched(const ProblemDesc* __restrict__ descs,
                                                             const int4* __restrict__ ctr_work, int nd,
                                                             const float* theta, char* ws, int* step) {
    constexpr int per = kMedSample / 64;
    if (step && blockIdx.x == 0 && threadIdx.x == 0) *step += 1;
    if ((int)blockIdx.x < nd) {
        const ProblemDesc& D = descs[blockIdx.x / per];
        if (D.N < 2 || D.fixed_h > 0.0f) return;
        const int t = (blockIdx.x % per) * 64 + (threadIdx.x >> 2), q = threadIdx.x & 3;
        const float v = sample_dist4(D.N, D.d, t, q, theta + D.theta_off);
        if (q == 0) med_of(D, ws).smp[t] = v;
        return;
    }
    const int4 e = ctr_work[blockIdx.x - nd];
    const ProblemDesc& D = descs[e.x];
    particle_mean_body<NT, 256>(D.N, e.y, theta + D.theta_off,
                                reinterpret_cast<float*>(ws + D.svgd_off + D.sv.ctr_off));
}

// entry = (problem, row block, column chunk, -) of this item shape's work list
template <int DP, int ROWS>
__global__ __launch_bounds__(256) void k_med_items_batched(const ProblemDesc* __restrict__ descs,
                                                            const int4* __restrict__ work, const float* theta,
                                                            char* ws) {
    const int4 w = work[blockIdx.x];
    const ProblemDesc& D = descs[w.x];
    const MedView v = med_of(D, ws);
    if (v.sel->mode != kModePass0) return;
    med_item<DP, ROWS, kPass0>(v, theta + D.theta_off, w.y, w.z, v.sel->lo, v.sel->hi, 0, nullptr);
}

// entry = (problem, workgroup, workgroups, -) of the problem's equal runs of steps
template <int KS, int ROWS>
__global__ __launch_bounds__(256, 4) void k_med_items_gram_batched(const ProblemDesc* __restrict__ descs,
                                                                 const int4* __restrict__ work, char* ws) {
    const int4 w = work[blockIdx.x];
    gram_pass0<KS, ROWS>(med_of(descs[w.x], ws), w.y, w.z);
}

// entry = (problem, workgroup, workgroups, -)
template <int KS, int ROWS>
__global__ __launch_bounds__(256) void k_med_pass_gram_batched(const ProblemDesc* __restrict__ descs,
                                                                const int4* __restrict__ work, char* ws, int pass) {
    const int4 w = work[blockIdx.x];
    gram_pass<KS, ROWS>(med_of(descs[w.x], ws), pass, w.y, w.z, nullptr);
}

// entry = (problem, -, -, -) of a problem of 2^20 pairs at most: the select
// ends in one workgroup after pass 0, as in the single-problem path
__global__ __launch_bounds__(kFinishThreads) void k_med_finish_batched(const ProblemDesc* __restrict__ descs,
                                                                       const int4* __restrict__ work,
                                                                       const float* theta, char* ws) {
    const ProblemDesc& D = descs[work[blockIdx.x].x];
    med_finish_body(med_of(D, ws), theta + D.theta_off, nullptr);
}

// f(padded dimension, rows) as constants
template <class F>
void by_item_shape(int d, int rows, F&& f) {
    auto dp = [&](auto r) {
        switch (med_dp(d)) {
            case 16: f(std::integral_constant<int, 16>{}, r); break;
            case 32: f(std::integral_constant<int, 32>{}, r); break;
            default: f(std::integral_constant<int, 64>{}, r); break;
        }
    };
    if (rows == 64) dp(std::integral_constant<int, 64>{});
    else dp(std::integral_constant<int, 256>{});
}

// f(Gram k-steps (0: split form), rows) as constants, by med_gram_ks
template <class F>
void by_gram_shape(int ks, int rows, F&& f) {
    auto k = [&](auto r) {
        switch (ks) {
            case 0: f(std::integral_constant<int, 0>{}, r); break;
            case 8: f(std::integral_constant<int, 8>{}, r); break;
            case 10: f(std::integral_constant<int, 10>{}, r); break;
            case 12: f(std::integral_constant<int, 12>{}, r); break;
            case 14: f(std::integral_constant<int, 14>{}, r); break;
            default: f(std::integral_constant<int, 16>{}, r); break;
        }
    };
    if (rows == 64) k(std::integral_constant<int, 64>{});
    else k(std::integral_constant<int, 256>{});
}

// pass 0 over the items of every shape present, each from its own work list
void launch_items_batched(const BatchPlan& P, const ProblemDesc* descs, const float* theta, char* ws,
                          hipStream_t st) {
    for (int rows : {64, 256}) {
        for (int d : {16, 32, 64})
            by_item_shape(d, rows, [&](auto dp, auto r) {
                const int c = med_class(dp.value, r.value);
                if (P.dist_n[c])
                    hipLaunchKernelGGL((k_med_items_batched<dp.value, r.value>), dim3(P.dist_n[c]), dim3(256), 0, st,
                                       descs, P.dist_work + P.dist_start[c], theta, ws);
            });
        for (int ks : {0, 8, 10, 12, 14, 16})
            by_gram_shape(ks, rows, [&](auto k, auto r) {
                const int c = med_gram_list(k.value, r.value);
                if (P.dist_n[c])
                    hipLaunchKernelGGL((k_med_items_gram_batched<k.value, r.value>), dim3(P.dist_n[c]), dim3(256), 0,
                                       st, descs, P.dist_work + P.dist_start[c], ws);
            });
    }
}

void launch_pass_batched(const BatchPlan& P, const ProblemDesc* descs, char* ws, int pass, hipStream_t st) {
    for (int rows : {64, 256})
        for (int ks : {0, 8, 10, 12, 14, 16})
            by_gram_shape(ks, rows, [&](auto k, auto r) {
                const int c = med_gram_list(k.value, r.value) - kMedDirect;
                if (P.pass_n[c])
                    hipLaunchKernelGGL((k_med_pass_gram_batched<k.value, r.value>), dim3(P.pass_n[c]), dim3(256), 0, st,
                                       descs, P.pass_work + P.pass_start[c], ws, pass);
            });
}

}  // namespace

hipError_t launch_median(int N, int d, const float* theta, float bandwidth, int exact, void* ws, const SvgdLayout& L,
                         float* h_out, hipStream_t st, int operands) {
    OneMed a{N, d, bandwidth > 0.0f ? bandwidth : 0.0f, L, static_cast<char*>(ws)};
    if (operands == kOperands32 && N >= 2 && bandwidth > 0.0f) {
        hipLaunchKernelGGL(k_mean, dim3(d), dim3(kMeanThreads), 0, st, a, theta);
        hipLaunchKernelGGL(k_pack_given, dim3(L.npad / 64), dim3(256), 0, st, a, theta, h_out);
        return hipGetLastError();
    }
    // the sample distances only when a median is wanted: with a given
    // bandwidth (or one particle) the select just records h
    const int n_dist = N >= 2 && !(bandwidth > 0.0f) ? kMedSample / 64 : 0, n_ctr = operands && N >= 2 ? d : 0;
    if (n_dist + n_ctr) {
        const dim3 grid(n_dist + n_ctr);
        if (operands == kOperands16)
            hipLaunchKernelGGL(k_med_gather<kCentreThreads>, grid, dim3(256), 0, st, a, theta, n_dist);
        else
            hipLaunchKernelGGL(k_med_gather<kMeanThreads>, grid, dim3(256), 0, st, a, theta, n_dist);
    }
    if (n_ctr && operands == kOperands32)
        hipLaunchKernelGGL(k_select_pack, dim3(1 + L.npad / kPackRows), dim3(kSelThreads), 0, st, a, theta,
                           exact, h_out);
    else
        hipLaunchKernelGGL(k_sample_select, dim3(1), dim3(kSelThreads), 0, st, a, exact, h_out);
    if (exact && N >= 2 && !(bandwidth > 0.0f) && pair_count(N) > (uint64_t)kMedSample) {
        // pass 0; small problems keep direct differences, whose every-pair
        // fallback lives in the finishing workgroup
        const bool small = !med_takes_gram(N);
        if (operands == kOperands32 && !small)
            by_gram_shape(med_gram_ks(L), L.med_rows, [&](auto k, auto r) {
                hipLaunchKernelGGL((k_med_items_gram<k.value, r.value>), dim3(med_gram_groups(N)), dim3(256), 0, st, a);
                for (int pass = 1; pass <= 3; ++pass)
                    hipLaunchKernelGGL((k_med_pass_gram<k.value, r.value>), dim3(med_pass_groups(N)), dim3(256), 0, st,
                                       a, pass, h_out);
            });
        else
            by_item_shape(d, L.med_rows, [&](auto dp, auto r) {
                const int64_t items = item_list(r.value, L.med_rb, L.med_cc).count();
                hipLaunchKernelGGL((k_med_items<dp.value, r.value>), dim3((uint32_t)items), dim3(256), 0, st, a, theta);
                if (small) {  // one workgroup finishes
                    hipLaunchKernelGGL(k_med_finish, dim3(1), dim3(kFinishThreads), 0, st, a, theta, h_out);
                    return;
                }
                for (int pass = 1; pass <= 3; ++pass)
                    hipLaunchKernelGGL((k_med_pass<dp.value, r.value>), dim3(med_pass_groups(N)), dim3(256), 0, st, a,
                                       theta, pass, h_out);
            });
    }
    return hipGetLastError();
}

hipError_t launch_bandwidth16_batched(const BatchPlan& P, const ProblemDesc* descs, const float* theta, char* ws,
                                      hipStream_t st, int* step) {
    const int np = P.n_problems, nd = (kMedSample / 64) * np;
    hipLaunchKernelGGL(k_gather_batched<kCentreThreads>, dim3(nd + P.n_ctr), dim3(256), 0, st, descs, P.ctr_work, nd,
                       theta, ws, step);
    hipLaunchKernelGGL(k_sample_select_batched, dim3(np), dim3(kSelThreads), 0, st, descs, ws, 0);
    return hipGetLastError();
}

hipError_t launch_median_batched(const BatchPlan& P, const ProblemDesc* descs, const float* theta, char* ws,
                                 hipStream_t st, int* step) {
    const int np = P.n_problems, nd = (kMedSample / 64) * np;
    hipLaunchKernelGGL(k_gather_batched<kMeanThreads>, dim3(nd + P.n_ctr), dim3(256), 0, st, descs, P.ctr_work, nd,
                       theta, ws, P.n_ctr ? step : nullptr);
    hipLaunchKernelGGL(k_select_pack_batched, dim3(np + P.n_row16), dim3(kSelThreads), 0, st, descs, np, P.row16_work,
                       theta, ws);
    if (P.n_dist) {
        launch_items_batched(P, descs, theta, ws, st);
        // problems of 2^20 pairs at most end in one workgroup each, the larger
        // ones in the passes
        if (P.n_fin)
            hipLaunchKernelGGL(k_med_finish_batched, dim3(P.n_fin), dim3(kFinishThreads), 0, st, descs, P.fin_work,
                               theta, ws);
        for (int pass = 1; pass <= 3; ++pass) launch_pass_batched(P, descs, ws, pass, st);
    }
    return hipGetLastError();
}

}  // namespace stamp
