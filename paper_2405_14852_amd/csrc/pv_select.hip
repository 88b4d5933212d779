// Group scores and top-k selection (Alg. 2 line 5, per matrix as in Sec. 3.4).
//
// score_n = sum_i (T[n,i] - W[n,i])^2 as an fp32 fused-multiply-add chain in
// index order, so that every implementation of this rule gives the same bits.
// Scores are non-negative floats, so their bit patterns order like unsigned
// integers.  The k-th largest key is found by a 3-digit radix select (12 + 11 +
// 8 bits below the sign, most significant first); groups above the threshold are taken, groups
// equal to it are taken lowest id first, and the ids are written in ascending
// order.  Nothing returns to the host.
//
// Launches: [scores + digit-0 histogram] [collect] [last digit] [ordered write]; up to
// kSmallGroups groups the last three are one block's work, and for k = N the sweep writes the
// ids itself.  Among many single weights the sweep collects and writes no scores (k_targets_lists).
// - The sweep counts digit 0 (exponent and four mantissa bits) in an LDS histogram; its blocks
//   are persistent so that clearing and flushing it is paid once per block.
// - k_collect is the only pass over all scores after the sweep.  It resolves digit 0, counts
//   digit 1 of the keys that share it, and copies every key at or above that digit's range, with
//   its id, into a short list per wave - a little more than the k that will be chosen.
// - k_last_digit and k_write_ids read those lists only.
// A list that does not fit (nearly all keys share digit 0, as after an optimiser's sign-like
// first step, or k is a large part of N) is dropped, and the two kernels read that wave's scores
// instead: slower, the same result.
//
// Histograms in device memory are kept in kCopies copies, block b adding to copy b % kCopies:
// workgroups are dealt to the eight dies round robin, so the blocks that share a copy share an
// L2 and their atomics stay in it.  One copy for all moves each line from die to die: 1 M
// atomics on 2048 counters took 11 us against 1.3 us (512 blocks; 110 and 150 per ns).  That is
// what makes a 12-bit digit 0 affordable, and a fine digit 0 keeps the lists and the later
// histograms short.  Every histogram also has a coarse level (sums of 64 counters), so that a
// reader adds up two rounds of 64 counters and not the whole table.
#include "pv_internal.h"

#ifndef PV_VOTE_ROUNDS
#define PV_VOTE_ROUNDS 1   // wave-wide merges before per-lane LDS atomics (guards degenerate inputs)
#endif

namespace {

constexpr int kBlock = 256;
constexpr int kRestBits = 19;                   // bits of a key below digit 0
constexpr int kLastBits = 8;                    // bits of digit 2
constexpr int kFirstBins = 1 << (31 - kRestBits);        // digit 0 (keys are clamped below 2^31)
constexpr int kMidBins = 1 << (kRestBits - kLastBits);   // digit 1
constexpr int kLastBins = 1 << kLastBits;                // digit 2
#ifndef PV_SEL_BLOCKS
#define PV_SEL_BLOCKS 512
#endif
constexpr int kMaxBlocks = PV_SEL_BLOCKS;      // persistent grid of the streaming kernels: two blocks per compute unit (1024 cost 1 us on 2 M groups and 4 to 6 us on 3.7 to 5.6 M, 256 lose a sixth of the bandwidth)

// Histograms in device memory: [copy][bin] and [copy][bin / 64], one after the other.
constexpr int kCopies = 8;
constexpr int kFine = 64;                      // counters per coarse counter, one per lane of a wave
constexpr int hist_words(int bins) { return kCopies * (bins + bins / kFine); }
constexpr int kHist0 = 0, kHist1 = kHist0 + hist_words(kFirstBins), kHist2 = kHist1 + hist_words(kMidBins);
constexpr int kHistTotal = kHist2 + hist_words(kLastBins);

// The passes after the sweep: region r of kSelWaves * blocks is the contiguous range of groups
// that wave r works on in every one of them.
constexpr int kSelBlock = 1024;
constexpr int kSelWaves = kSelBlock / 64;
constexpr int kSelBlocks = 256;                // at most: one block per compute unit (collect on 5.6 M scores: 12.9 us; 128 blocks 15.1, 512 blocks 16.2)
constexpr int kAhead = 4;                      // 16-byte loads in flight per lane
constexpr int kSuffix = kLastBins + 8;         // row of a block's suffix counts (kLastBins + 1 used)
// A single block selects among at most so many: a call with 24 576 groups 21.3 us against 22.9 by three
// kernels, with 32 768 24.0 against 22.8 (every key is in a register: the code grows with the limit too).
constexpr int kSmallGroups = 24576;

// The key of a score: its bits, which order like the values because scores are sums of squares
// (never negative); a pattern with the sign bit set can only be a NaN and is clamped to the
// largest key, so that digit 0 needs no bit for the sign.
__device__ __forceinline__ unsigned score_key(float s) { return min(__float_as_uint(s), 0x7FFFFFFFu); }

__device__ __forceinline__ int digit0_of(unsigned key) { return (int)(key >> kRestBits); }

// Add one count per valid lane to an LDS histogram.  Lanes of a wave that hit
// the same bin as the first pending lane are merged first (catches the
// dominant bins of a narrow score distribution); the rest use one atomic each.
template <int ROUNDS>
__device__ __forceinline__ void hist_add(unsigned *hist, int bin, bool valid)
{
    const int lane = threadIdx.x & 63;
    if (ROUNDS > 0) {
        unsigned long long todo = __ballot(valid);
#pragma unroll 1
        for (int round = 0; round < ROUNDS && todo; ++round) {
            int leader = __ffsll((long long)todo) - 1;
            int lb = __shfl(bin, leader);
            unsigned long long same = __ballot(valid && bin == lb);
            if (lane == leader) atomicAdd(&hist[lb], (unsigned)__popcll(same));
            if (valid && bin == lb) valid = false;
            todo &= ~same;
        }
    }
    if (valid) atomicAdd(&hist[bin], 1u);
}

// The later digits: few keys count as a rule, but all of them in a few bins where scores are alike (a
// sign-like optimiser step, equal scores), and the atomics of one instruction on one address queue
// up in the LDS.  Such a histogram is kept in 2^log copies, lane l adding to copy l % 2^log: eight
// lanes at most on an address.  (One block, 32 768 equal scores, a whole call: 76 -> 29 us; merging the lanes
// of a bin by ballots instead took 38, and 2.7 us more on scores that are not alike.)
constexpr int kSpreadLog = 3;
__device__ __forceinline__ void spread_add(unsigned *hist, unsigned bin, int log)
{
    atomicAdd(&hist[(bin << log) + (threadIdx.x & ((1u << log) - 1u))], 1u);
}
__device__ __forceinline__ unsigned spread_at(const unsigned *hist, int bin, int log)
{
    if (log == 0) return hist[bin];
    unsigned t = 0;
#pragma unroll
    for (int c = 0; c < 1 << kSpreadLog; ++c) t += hist[(bin << kSpreadLog) + c];
    return t;
}
// copies of digit 1's histogram: more than one where the keys that share digit 0 are many
__device__ __forceinline__ int mid_log(unsigned share, int64_t N) { return (int64_t)share * 8 > N ? kSpreadLog : 0; }

// inclusive prefix sum over the lanes of a wave
__device__ __forceinline__ unsigned wave_incl_scan(unsigned v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned u = __shfl_up(v, off);
        if (lane >= off) v += u;
    }
    return v;
}

__device__ __forceinline__ unsigned wave_sum(unsigned v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// One counter per lane, lane 0 holding the LARGEST digit: the lane in which the rank kk (1-based,
// counted from the top) falls; kk becomes the rank within that lane's counter.
__device__ __forceinline__ int pick_lane(unsigned count, unsigned &kk)
{
    const unsigned inc = wave_incl_scan(count);
    const unsigned long long at = __ballot(inc >= kk);
    const int src = at ? __ffsll((long long)at) - 1 : 63;
    kk -= __shfl(inc - count, src);
    return src;
}

// The digit d of the histogram `h` (in device memory, `bins` counters) with
// count(> d) < kk <= count(>= d); kk becomes kk - count(> d).  Called by all threads of a block:
// its waves fetch the 64 counters of a copy each, every wave adds up all copies (the result needs
// no broadcast).  `tmp`: 2 * kCopies * 64 unsigneds of LDS.
// `share`: the count of the digit.
template <int WAVES>
__device__ __forceinline__ int pick_digit(const unsigned *__restrict__ h, int bins, unsigned &kk, unsigned *tmp,
                                          unsigned *share = nullptr)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ncoarse = bins / kFine;
    for (int i = wave; i < kCopies; i += WAVES)
        tmp[i * 64 + lane] = lane < ncoarse ? h[kCopies * bins + i * ncoarse + (ncoarse - 1 - lane)] : 0u;
    __syncthreads();
    unsigned c = 0;
#pragma unroll
    for (int i = 0; i < kCopies; ++i) c += tmp[i * 64 + lane];
    const int top = ncoarse - 1 - pick_lane(c, kk);
    unsigned *fine = tmp + kCopies * 64;
    for (int i = wave; i < kCopies; i += WAVES) fine[i * 64 + lane] = h[i * bins + top * kFine + (kFine - 1 - lane)];
    __syncthreads();
    c = 0;
#pragma unroll
    for (int i = 0; i < kCopies; ++i) c += fine[i * 64 + lane];
    const int at = pick_lane(c, kk);
    if (share) *share = __shfl(c, at);
    return top * kFine + (kFine - 1 - at);
}

// Add a block's LDS histogram to the block's copy in device memory.  An atomic instruction of a
// wave costs by the cache lines it touches, one after the other per line: the coarse counters
// go out in one instruction (one per wave that counted something took 5 us, all on one line).
// `s_coarse`: 64 unsigneds of LDS; log: see spread_add.
__device__ __forceinline__ void flush_hist(const unsigned *lh, unsigned *__restrict__ h, int bins,
                                           unsigned *s_coarse, int log = 0)
{
    const int copy = blockIdx.x % kCopies, lane = threadIdx.x & 63;
    unsigned *fine = h + copy * bins, *coarse = h + kCopies * bins + copy * (bins / kFine);
    for (int b = threadIdx.x; b < bins; b += blockDim.x) {   // a wave takes the kFine bins of one coarse counter
        const unsigned v = spread_at(lh, b, log);
        unsigned t = 0;
        if (__any(v != 0u)) {
            if (v) atomicAdd(&fine[b], v);
            t = wave_sum(v);
        }
        if (lane == 0) s_coarse[b / kFine] = t;
    }
    __syncthreads();
    if ((int)threadIdx.x < bins / kFine) {
        const unsigned t = s_coarse[threadIdx.x];
        if (t) atomicAdd(&coarse[threadIdx.x], t);
    }
}

__device__ __forceinline__ float score_group(const float *__restrict__ t,
                                             const float *__restrict__ w, int g)
{
    float s = 0.0f;
    if ((g & 3) == 0) {
        const pv_f4 *t4 = reinterpret_cast<const pv_f4 *>(t);
        const pv_f4 *w4 = reinterpret_cast<const pv_f4 *>(w);
        for (int i = 0; i < g / 4; ++i) {
            pv_f4 a = __builtin_nontemporal_load(&t4[i]);
            pv_f4 b = __builtin_nontemporal_load(&w4[i]);
            float d;
            d = a.x - b.x; s = fmaf(d, d, s);
            d = a.y - b.y; s = fmaf(d, d, s);
            d = a.z - b.z; s = fmaf(d, d, s);
            d = a.w - b.w; s = fmaf(d, d, s);
        }
    } else {
        for (int i = 0; i < g; ++i) {
            float d = t[i] - w[i];
            s = fmaf(d, d, s);
        }
    }
    return s;
}

// Pass 0, any group size: one thread per group.
__global__ __launch_bounds__(kBlock) void k_scores_hist0(const float *__restrict__ T,
                                                         const float *__restrict__ W,
                                                         float *__restrict__ scores,
                                                         unsigned *__restrict__ hist0, int N, int g,
                                                         int want_hist, int32_t *__restrict__ all_ids)
{
    __shared__ unsigned lh[kFirstBins];
    __shared__ unsigned s_coarse[64];
    if (want_hist)
        for (int b = threadIdx.x; b < kFirstBins; b += kBlock) lh[b] = 0;
    __syncthreads();
    for (int64_t base = (int64_t)blockIdx.x * kBlock; base < N; base += (int64_t)gridDim.x * kBlock) {
        const int64_t n = base + threadIdx.x;
        const bool valid = n < N;
        unsigned key = 0;
        if (valid) {
            float s = score_group(T + n * g, W + n * g, g);
            scores[n] = s;
            if (all_ids) all_ids[n] = (int32_t)n;
            key = score_key(s);
        }
        if (want_hist) hist_add<PV_VOTE_ROUNDS>(lh, digit0_of(key), valid);
    }
    __syncthreads();
    if (want_hist) flush_hist(lh, hist0, kFirstBins, s_coarse);
}

// Pass 0 for g = 4 * PARTS (PARTS a power of two): every lane loads one 16-byte
// vector of T and of W, so a wave reads two contiguous 1 KiB runs per step.
// The fused-multiply-add chain of a group runs over PARTS neighbouring lanes in
// index order: each lane folds its four differences onto the partial sum of
// the lane before it; the last lane of the group holds the score.
constexpr int kVecUnroll = 4;

// NORM: the sweep also adds up (scales[row] * codeword element)^2 over the dequantised weights
// of the codes (one codebook; lane `part` of a group takes the same 16-byte piece of its
// codeword as of its target), in double, every thread in the order of its loop, the block
// in the fixed order of the reduction below: partial[block].
struct norm_args {
    const uint16_t *codes;
    const pv_f4 *cb4;
    const float *scales;
    double *partial;
    unsigned mask;
    double inv_gpr;
};

template <int PARTS, bool NORM>
__global__ __launch_bounds__(kBlock) void k_scores_hist0_vec(const float *__restrict__ T,
                                                             const float *__restrict__ W,
                                                             float *__restrict__ scores,
                                                             unsigned *__restrict__ hist0,
                                                             int64_t nvec, int want_hist,
                                                             int32_t *__restrict__ all_ids, norm_args na)
{
    __shared__ unsigned lh[kFirstBins];
    __shared__ unsigned s_coarse[64];
    double nacc = 0.0;
    if (want_hist)
        for (int b = threadIdx.x; b < kFirstBins; b += kBlock) lh[b] = 0;
    __syncthreads();
    const pv_f4 *T4 = reinterpret_cast<const pv_f4 *>(T);
    const pv_f4 *W4 = reinterpret_cast<const pv_f4 *>(W);
    const int part = threadIdx.x & (PARTS - 1);   // kBlock and every stride are multiples of PARTS
    for (int64_t cbase = (int64_t)blockIdx.x * (kBlock * kVecUnroll); cbase < nvec;
         cbase += (int64_t)gridDim.x * (kBlock * kVecUnroll)) {
        const int64_t base = cbase + threadIdx.x;
        pv_f4 a[kVecUnroll], b[kVecUnroll];
#pragma unroll
        for (int u = 0; u < kVecUnroll; ++u) {
            const int64_t i = base + (int64_t)u * kBlock;
            if (i < nvec) {
                a[u] = __builtin_nontemporal_load(&T4[i]);
                b[u] = __builtin_nontemporal_load(&W4[i]);
            } else {
                a[u] = pv_f4{0.f, 0.f, 0.f, 0.f};
                b[u] = a[u];
            }
        }
        // (requesting the codes a chunk ahead, so that the pieces go out with the chunk's targets
        // and weights, measured 3 us slower on 2 M groups)
        pv_f4 cw[kVecUnroll];
        float sc[kVecUnroll];
        if constexpr (NORM) {
            unsigned code[kVecUnroll];
#pragma unroll
            for (int u = 0; u < kVecUnroll; ++u) {      // codes and scales first, all in flight ...
                const int64_t i = base + (int64_t)u * kBlock;
                const unsigned n = (unsigned)((i < nvec ? i : 0) / PARTS);
                code[u] = na.codes[n] & na.mask;
                sc[u] = i < nvec ? na.scales[pv_row_of(n, na.inv_gpr)] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < kVecUnroll; ++u)        // ... then the codeword pieces
                cw[u] = na.cb4[(int64_t)code[u] * PARTS + part];
        }
#pragma unroll
        for (int u = 0; u < kVecUnroll; ++u) {
            const int64_t i = base + (int64_t)u * kBlock;
            if constexpr (NORM) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double w = (double)(sc[u] * cw[u][e]);
                    nacc = nacc + w * w;
                }
            }
            const float d0 = a[u].x - b[u].x, d1 = a[u].y - b[u].y;
            const float d2 = a[u].z - b[u].z, d3 = a[u].w - b[u].w;
            float s = 0.0f;
#pragma unroll
            for (int r = 0; r < PARTS; ++r) {
                // after round r the lanes with part <= r hold their final prefix
                float in = r == 0 ? 0.0f : __shfl_up(s, 1);
                if (part >= r) {
                    float c = part == 0 ? 0.0f : in;
                    c = fmaf(d0, d0, c);
                    c = fmaf(d1, d1, c);
                    c = fmaf(d2, d2, c);
                    c = fmaf(d3, d3, c);
                    if (part == r) s = c;
                }
            }
            const bool valid = i < nvec && part == PARTS - 1;
            if (valid) {
                scores[i / PARTS] = s;
                if (all_ids) all_ids[i / PARTS] = (int32_t)(i / PARTS);
            }
            if (want_hist) hist_add<PV_VOTE_ROUNDS>(lh, digit0_of(score_key(s)), valid);
        }
    }
    __syncthreads();
    if (want_hist) flush_hist(lh, hist0, kFirstBins, s_coarse);
    if constexpr (NORM) {
        __shared__ double ntmp[kBlock / 64];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) nacc = nacc + __shfl_down(nacc, off);
        if ((threadIdx.x & 63) == 0) ntmp[threadIdx.x >> 6] = nacc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int w = 0; w < kBlock / 64; ++w) t = t + ntmp[w];
            na.partial[blockIdx.x] = t;
        }
    }
}

// Targets and pass 0 in one sweep (g = 4 * PARTS): T = W - alpha * G is formed and stored, and
// the scores and the digit-0 histogram are taken from the same registers, so T and W are
// not read back from memory.  The arithmetic is the one of the separate kernels: one fused
// multiply-add per element of T, then the subtraction T - W and the chain above.
template <int PARTS, bool ADAM>
__global__ __launch_bounds__(kBlock) void k_targets_scores_hist0_vec(const float *W, const float *G,
                                                                     float alpha, float *T,
                                                                     float *__restrict__ scores,
                                                                     unsigned *__restrict__ hist0,
                                                                     int64_t nvec, int want_hist,
                                                                     int32_t *__restrict__ all_ids,
                                                                     pv_adam_t adam, float *m, float *v)
{
    __shared__ unsigned lh[kFirstBins];
    __shared__ unsigned s_coarse[64];
    const pv_f4 *W4 = reinterpret_cast<const pv_f4 *>(W);
    const pv_f4 *G4 = reinterpret_cast<const pv_f4 *>(G);
    pv_f4 *T4 = reinterpret_cast<pv_f4 *>(T);
    const int part = threadIdx.x & (PARTS - 1);
    const int64_t step = (int64_t)gridDim.x * (kBlock * kVecUnroll);
    pv_f4 *M4 = reinterpret_cast<pv_f4 *>(m);
    pv_f4 *V4 = reinterpret_cast<pv_f4 *>(v);
    pv_f4 w[kVecUnroll], gr[kVecUnroll], wn[kVecUnroll], gn[kVecUnroll];
    auto load = [&](int64_t cbase, pv_f4 *pw, pv_f4 *pg) {
#pragma unroll
        for (int u = 0; u < kVecUnroll; ++u) {
            const int64_t i = cbase + threadIdx.x + (int64_t)u * kBlock;
            if (i < nvec) {
                pw[u] = __builtin_nontemporal_load(&W4[i]);
                pg[u] = __builtin_nontemporal_load(&G4[i]);
            } else {
                pw[u] = pv_f4{0.f, 0.f, 0.f, 0.f};
                pg[u] = pw[u];
            }
        }
    };
    int64_t cbase = (int64_t)blockIdx.x * (kBlock * kVecUnroll);
    if (cbase < nvec) load(cbase, w, gr);
    if (want_hist)
        for (int b = threadIdx.x; b < kFirstBins; b += kBlock) lh[b] = 0;
    __syncthreads();
    for (; cbase < nvec; cbase += step) {
        // the loads of the next chunk are in flight while this one is scored
        if (cbase + step < nvec) load(cbase + step, wn, gn);
        const int64_t base = cbase + threadIdx.x;
#pragma unroll
        for (int u = 0; u < kVecUnroll; ++u) {
            const int64_t i = base + (int64_t)u * kBlock;
            pv_f4 t;
            if constexpr (ADAM) {
                pv_f4 mm = pv_f4{0.f, 0.f, 0.f, 0.f}, vv = mm;
                if (i < nvec) {
                    mm = __builtin_nontemporal_load(&M4[i]);
                    vv = __builtin_nontemporal_load(&V4[i]);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float mi = mm[e], vi = vv[e];
                    t[e] = pv_adam_one(w[u][e], gr[u][e], mi, vi, adam);
                    mm[e] = mi;
                    vv[e] = vi;
                }
                // Past the caches: the moments are read next a whole step later.  Several matrices in turn,
                // 8 of 4096 x 4096: 905 us a step with plain stores, 887 this way; 4 of 8192 x 4096 828, 792.  (One
                // matrix of 12 to 34 M weights stepped over and over finds part of them in the caches: 105, 110.)
                if (i < nvec) {
                    __builtin_nontemporal_store(mm, &M4[i]);
                    __builtin_nontemporal_store(vv, &V4[i]);
                }
            } else {
                t.x = fmaf(-alpha, gr[u].x, w[u].x);
                t.y = fmaf(-alpha, gr[u].y, w[u].y);
                t.z = fmaf(-alpha, gr[u].z, w[u].z);
                t.w = fmaf(-alpha, gr[u].w, w[u].w);
            }
            if (i < nvec) __builtin_nontemporal_store(t, &T4[i]);
            const float d0 = t.x - w[u].x, d1 = t.y - w[u].y;
            const float d2 = t.z - w[u].z, d3 = t.w - w[u].w;
            float s = 0.0f;
#pragma unroll
            for (int r = 0; r < PARTS; ++r) {
                float in = r == 0 ? 0.0f : __shfl_up(s, 1);
                if (part >= r) {
                    float c = part == 0 ? 0.0f : in;
                    c = fmaf(d0, d0, c);
                    c = fmaf(d1, d1, c);
                    c = fmaf(d2, d2, c);
                    c = fmaf(d3, d3, c);
                    if (part == r) s = c;
                }
            }
            const bool valid = i < nvec && part == PARTS - 1;
            if (valid) {
                scores[i / PARTS] = s;
                if (all_ids) all_ids[i / PARTS] = (int32_t)(i / PARTS);
            }
            if (want_hist) hist_add<PV_VOTE_ROUNDS>(lh, digit0_of(score_key(s)), valid);
        }
#pragma unroll
        for (int u = 0; u < kVecUnroll; ++u) {
            w[u] = wn[u];
            gr[u] = gn[u];
        }
    }
    __syncthreads();
    if (want_hist) flush_hist(lh, hist0, kFirstBins, s_coarse);
}

// The same sweep for group sizes 1 and 2: a 16-byte vector holds 4 / GS whole groups and every
// lane scores its own (no exchange between lanes).  The last nelem % 4 elements, which fill
// no vector, are left to thread 0 of block 0.
template <int GS>
__global__ __launch_bounds__(kBlock) void k_targets_scores_hist0_sub(const float *W, const float *G,
                                                                     float alpha, float *T,
                                                                     float *__restrict__ scores,
                                                                     unsigned *__restrict__ hist0,
                                                                     int64_t nelem, int want_hist,
                                                                     int32_t *__restrict__ all_ids)
{
    constexpr int kPerVec = 4 / GS;               // groups per vector
    __shared__ unsigned lh[kFirstBins];
    __shared__ unsigned s_coarse[64];
    if (want_hist)
        for (int b = threadIdx.x; b < kFirstBins; b += kBlock) lh[b] = 0;
    __syncthreads();
    const pv_f4 *W4 = reinterpret_cast<const pv_f4 *>(W);
    const pv_f4 *G4 = reinterpret_cast<const pv_f4 *>(G);
    pv_f4 *T4 = reinterpret_cast<pv_f4 *>(T);
    const int64_t nvec = nelem >> 2;
    // whole blocks stay in the loop together (the histogram update uses wave-wide votes)
    for (int64_t cbase = (int64_t)blockIdx.x * (kBlock * kVecUnroll); cbase < nvec;
         cbase += (int64_t)gridDim.x * (kBlock * kVecUnroll)) {
        pv_f4 w[kVecUnroll], gr[kVecUnroll];
#pragma unroll
        for (int u = 0; u < kVecUnroll; ++u) {
            const int64_t i = cbase + threadIdx.x + (int64_t)u * kBlock;
            if (i < nvec) {
                w[u] = __builtin_nontemporal_load(&W4[i]);
                gr[u] = __builtin_nontemporal_load(&G4[i]);
            } else {
                w[u] = pv_f4{0.f, 0.f, 0.f, 0.f};
                gr[u] = w[u];
            }
        }
#pragma unroll
        for (int u = 0; u < kVecUnroll; ++u) {
            const int64_t i = cbase + threadIdx.x + (int64_t)u * kBlock;
            const bool valid = i < nvec;
            pv_f4 t;
            float sc[kPerVec];
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = fmaf(-alpha, gr[u][e], w[u][e]);
#pragma unroll
            for (int q = 0; q < kPerVec; ++q) {
                float s = 0.0f;
#pragma unroll
                for (int e = 0; e < GS; ++e) {
                    const float d = t[q * GS + e] - w[u][q * GS + e];
                    s = fmaf(d, d, s);
                }
                sc[q] = s;
            }
            if (valid) {
                __builtin_nontemporal_store(t, &T4[i]);
#pragma unroll
                for (int q = 0; q < kPerVec; ++q) scores[i * kPerVec + q] = sc[q];
                if (all_ids)
#pragma unroll
                    for (int q = 0; q < kPerVec; ++q) all_ids[i * kPerVec + q] = (int32_t)(i * kPerVec + q);
            }
            if (want_hist) {
#pragma unroll
                for (int q = 0; q < kPerVec; ++q)
                    hist_add<PV_VOTE_ROUNDS>(lh, digit0_of(score_key(sc[q])), valid);
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // the elements after the last whole vector: whole groups, since nelem is a multiple of GS
        for (int64_t i = nvec << 2; i < nelem; i += GS) {
            float s = 0.0f;
            for (int e = 0; e < GS; ++e) {
                const float tv = fmaf(-alpha, G[i + e], W[i + e]);
                T[i + e] = tv;
                const float d = tv - W[i + e];
                s = fmaf(d, d, s);
            }
            scores[i / GS] = s;
            if (all_ids) all_ids[i / GS] = (int32_t)(i / GS);
            if (want_hist) atomicAdd(&lh[digit0_of(score_key(s))], 1u);
        }
    }
    __syncthreads();
    if (want_hist) flush_hist(lh, hist0, kFirstBins, s_coarse);
}

// What a region holds at or above the range of digit 0: `count` entries of `list`, or, if the
// count exceeds the list's room, the region's scores themselves.
// Where no scores were written (one weight a group, see k_targets_lists), `scores` is T, W lies beside it, and the keys kept
// are in cells of kCell consecutive weights: up to kCellList of them as a list, else all the cell's scores.
constexpr int kCell = 256 * kAhead;
constexpr int kCellList = kCell / 2;
struct cell_args {
    uint2 *lists;                    // [cells][kCellList] {key, id}, or kCell scores in the same place
    unsigned *counts;                // [cells] keys kept
    unsigned *waves;                 // [waves of the sweep] the sum of their cells
    unsigned *sample;                // digit 0 of the sample, zero between calls
};
struct region_t {
    const uint2 *list;      // {key, id}
    const float *scores, *W;
    int64_t base;
    int n;
    bool raw;
};
__device__ __forceinline__ region_t region_of(int r, const uint2 *list, const unsigned *counts,
                                              const float *scores, const float *W, int64_t N, int span, int cap,
                                              bool all_raw)
{
    region_t g;
    const unsigned c = counts[r];
    g.raw = all_raw || c > (unsigned)cap;
    g.W = W;
    g.base = (int64_t)r * span;
    const int64_t left = N - g.base;
    g.list = list + (int64_t)r * cap;
    g.scores = scores;
    g.n = g.raw ? (int)(left < span ? (left < 0 ? 0 : left) : span) : (int)c;
    return g;
}
// entry i of a list of n; key 0 past its end
__device__ __forceinline__ uint2 list_at(const uint2 *list, int n, int i)
{
    return i < n ? list[i] : make_uint2(0u, 0u);
}
// kAhead steps of a wave through scores: four consecutive ones a lane, 256 a step; 0 past the n-th.
// SKIP: no instructions for steps past the n-th score.
template <bool SKIP>
__device__ __forceinline__ void load_scores(const float *s, int at, int n, pv_f4 (&v)[kAhead])
{
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
        const int i = at + u * 256 + (int)(threadIdx.x & 63) * 4;
        v[u] = pv_f4{0.f, 0.f, 0.f, 0.f};
        if (SKIP && at + u * 256 >= n) continue;          // uniform over the wave
        if (i + 4 <= n) {
            v[u] = *reinterpret_cast<const pv_f4 *>(s + i);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e < n) v[u][e] = s[i + e];
        }
    }
}
// f(scores, place of the first one) for every step of a wave through the n scores of a region whose list
// does not fit.  Sixteen bytes a lane (with four: 45 M single weights 541 us a call against 430).  Short code
// rather than the next steps' loads ahead: it lies between the instructions of the kernels' usual way,
// and their registers decide what fits beside them (a 224-matrix sweep on four streams: 1 %).
// TW: the scores from T and W.
template <bool TW, class F>
__device__ __forceinline__ void for_scores(const region_t &g, F f)
{
    const float *s = g.scores + g.base;
    const int n = g.n;
#pragma unroll 1
    for (int at = 0; at < n; at += 256 * kAhead) {
        pv_f4 v[kAhead];
        load_scores<true>(s, at, n, v);
        if constexpr (TW) {
            pv_f4 w[kAhead];
            load_scores<true>(g.W + g.base, at, n, w);
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float d = v[u][e] - w[u][e];
                    v[u][e] = d * d;               // (the chain of one element: fma(d, d, 0))
                }
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (at + u * 256 < n) f(v[u], at + u * 256);      // uniform over the wave
    }
}
// A region's keys one way or another: on_list(list, entries) or on_scores(region of scores in memory or of T and W, see
// for_scores), in id order.  WAY 0: scores in memory, where the list does not fit; 1: from T and W, every region; 2: from
// the cells, where it does not fit (a region is a whole number of them).
template <int WAY, class L, class S>
__device__ __forceinline__ void for_region(const cell_args &c, const region_t &g, L on_list, S on_scores)
{
    if (WAY == 2) {
        const int cells = g.raw ? (g.n + kCell - 1) / kCell : 1;
#pragma unroll 1
        for (int i = 0; i < cells; ++i) {
            const int64_t cell = g.base / kCell + i;
            const unsigned cnt = g.raw ? c.counts[cell] : 0u;
            const uint2 *list = g.raw ? c.lists + cell * kCellList : g.list;
            if (cnt > (unsigned)kCellList) {
                region_t d;
                d.base = g.base + (int64_t)i * kCell;
                d.n = g.n - i * kCell < kCell ? g.n - i * kCell : kCell;
                d.scores = reinterpret_cast<const float *>(list) - d.base;
                on_scores(d);
            } else {
                on_list(list, g.raw ? (int)cnt : g.n);
            }
        }
    } else if (WAY == 1 || g.raw) {
        on_scores(g);
    } else {
        on_list(g.list, g.n);
    }
}

// Pass over all scores: digit 0 is resolved, digit 1 of the keys that share it is counted, the
// keys at or above its range go to the region's list in id order (a wave's 256 keys of a step
// find their places from four ballots, so nothing is exchanged between waves).
// Block 0 publishes digit 0 and the rank left after it: state[4], state[6].
// Bound by the read of the scores: 4 bytes a group.
__global__ __launch_bounds__(kSelBlock) void k_collect(const float *__restrict__ scores,
                                                       unsigned *__restrict__ hist_all,
                                                       unsigned *__restrict__ state, int64_t N,
                                                       unsigned k, int span, int cap,
                                                       uint2 *__restrict__ list,
                                                       unsigned *__restrict__ counts)
{
    __shared__ unsigned tmp[2 * kCopies * 64];
    __shared__ unsigned lh[kMidBins << kSpreadLog];
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * kSelWaves + (threadIdx.x >> 6);
    const int64_t base = (int64_t)r * span;
    const float *mine_scores = scores + base;
    const int n = base >= N ? 0 : (int)(N - base < span ? N - base : span);
    uint2 *mine = list + (int64_t)r * cap;
    pv_f4 cur[kAhead], nxt[kAhead];
    load_scores<false>(mine_scores, 0, n, cur);     // in flight while digit 0 is resolved
    for (int b = threadIdx.x; b < kMidBins; b += kSelBlock) lh[b] = 0;
    // the last digit's histogram starts at zero (its reader of the call before has run)
    for (int z = kHist2 + blockIdx.x * kSelBlock + threadIdx.x; z < kHistTotal; z += gridDim.x * kSelBlock)
        hist_all[z] = 0u;
    unsigned kk = k;
    unsigned share;
    const int d0 = pick_digit<kSelWaves>(hist_all + kHist0, kFirstBins, kk, tmp, &share);   // its barriers also order the clearing above
    const int log = mid_log(share, N);                       // the same in every thread
    if (log) {
        for (int b = kMidBins + threadIdx.x; b < kMidBins << kSpreadLog; b += kSelBlock) lh[b] = 0;
        __syncthreads();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        state[4] = (unsigned)d0;
        state[6] = kk;
    }
    const unsigned lo = (unsigned)d0 << kRestBits, hi = ((unsigned)d0 + 1u) << kRestBits;
    unsigned cnt = 0;
    auto take = [&](const pv_f4 &v, int at, bool whole) {
        const int i = at + lane * 4;
        unsigned long long hits[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)          // (a NaN with its sign bit set is above every range as it is)
            hits[e] = __ballot(__float_as_uint(v[e]) >= lo && (whole || i + e < n));
        if (!(hits[0] | hits[1] | hits[2] | hits[3])) return;   // uniform over the wave
        unsigned pos = cnt;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pos = __builtin_amdgcn_mbcnt_hi((unsigned)(hits[e] >> 32),
                                            __builtin_amdgcn_mbcnt_lo((unsigned)hits[e], pos));
            cnt += (unsigned)__popcll(hits[e]);
        }
        const bool room = cnt <= (unsigned)cap;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if ((hits[e] >> lane) & 1ull) {
                const unsigned key = score_key(v[e]);
                if (room) mine[pos] = make_uint2(key, (unsigned)(base + i + e));
                ++pos;
                if (key < hi) spread_add(lh, (key >> kLastBits) & (kMidBins - 1), log);
            }
    };
    for (int at = 0; at < n; at += 256 * kAhead) {
        if (at + 256 * kAhead < n) load_scores<false>(mine_scores, at + 256 * kAhead, n, nxt);
        const bool whole = at + 256 * kAhead <= n;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) take(cur[u], at + u * 256, whole);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) cur[u] = nxt[u];
    }
    if (lane == 0) counts[r] = cnt;
    __syncthreads();
    flush_hist(lh, hist_all + kHist1, kMidBins, tmp, log);
}

// Digit 1 is resolved; among the keys collected, those above digits 0 and 1 are counted per
// block, those equal are counted by digit 2: per block as suffix sums (how many have digit 2 >= d,
// so that the next kernel reads two numbers a block) and over all blocks in the histogram.
// Publishes digit 1 and the rank left: state[5], state[7].
struct sel_args {
    const float *scores;     // (or T, and)
    const float *W;
    unsigned *hist_all, *state;
    int64_t N;
    int span, cap;
    const uint2 *list;
    const unsigned *counts;
    unsigned *above, *suffix;
    cell_args cells;
};
// WAY: see for_region
template <int WAY>
__device__ __forceinline__ void last_digit(const sel_args &a, unsigned *tmp, unsigned *lh)
{
    __shared__ unsigned s_above;
    unsigned *hist_all = a.hist_all, *state = a.state;
    const int lane = threadIdx.x & 63;
    for (int b = threadIdx.x; b < kLastBins << kSpreadLog; b += kSelBlock) lh[b] = 0;
    if (threadIdx.x == 0) s_above = 0;
    // digit 0's histogram is done with: zero for the next call
    for (int z = kHist0 + blockIdx.x * kSelBlock + threadIdx.x; z < kHist1; z += gridDim.x * kSelBlock)
        hist_all[z] = 0u;
    const region_t g = region_of(blockIdx.x * kSelWaves + (threadIdx.x >> 6), a.list, a.counts, a.scores, a.W, a.N, a.span, a.cap, WAY == 1);
    unsigned kk = state[6];
    const unsigned d0 = state[4];
    const unsigned d1 = (unsigned)pick_digit<kSelWaves>(hist_all + kHist1, kMidBins, kk, tmp);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        state[5] = d1;
        state[7] = kk;
    }
    const unsigned want = (d0 << (kRestBits - kLastBits)) | d1;
    unsigned gt = 0;
    auto count = [&](unsigned key, bool in) {
        const unsigned p = key >> kLastBits;
        gt += p > want;
        if (p == want && in) spread_add(lh, key & (kLastBins - 1), kSpreadLog);
    };
    for_region<WAY>(
        a.cells, g,
        [&](const uint2 *list, int n) {
            for (int i0 = 0; i0 < n; i0 += 64 * kAhead) {
                unsigned key[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) key[u] = list_at(list, n, i0 + u * 64 + lane).x;
#pragma unroll
                for (int u = 0; u < kAhead; ++u) count(key[u], i0 + u * 64 + lane < n);
            }
        },
        [&](const region_t &d) {
            for_scores<WAY == 1>(d, [&](const pv_f4 &v, int at) {
#pragma unroll
                for (int e = 0; e < 4; ++e) count(score_key(v[e]), at + lane * 4 + e < d.n);
            });
        });
    gt = wave_sum(gt);
    if (lane == 0 && gt) atomicAdd(&s_above, gt);
    __syncthreads();
    flush_hist(lh, hist_all + kHist2, kLastBins, tmp, kSpreadLog);
    if (threadIdx.x == 0) a.above[blockIdx.x] = s_above;
    if (threadIdx.x < 64) {
        // four digits a lane, lane 0 the largest
        unsigned c[kLastBins / 64], sum = 0;
#pragma unroll
        for (int q = 0; q < kLastBins / 64; ++q) {
            c[q] = spread_at(lh, kLastBins - 1 - (lane * (kLastBins / 64) + q), kSpreadLog);
            sum += c[q];
        }
        unsigned run = wave_incl_scan(sum) - sum;
        unsigned *row = a.suffix + (int64_t)blockIdx.x * kSuffix;
#pragma unroll
        for (int q = 0; q < kLastBins / 64; ++q) {
            run += c[q];
            row[kLastBins - 1 - (lane * (kLastBins / 64) + q)] = run;
        }
        if (lane == 0) row[kLastBins] = 0u;
    }
}

__global__ __launch_bounds__(kSelBlock) void k_last_digit(sel_args a)
{
    __shared__ unsigned tmp[2 * kCopies * 64];
    __shared__ unsigned lh[kLastBins << kSpreadLog];
    last_digit<0>(a, tmp, lh);
}

// Digit 2 and with it the threshold and the number of ties to take; then the ids, in order:
// position of a chosen group = (#greater with a lower id) + min(#equal with a lower id, ties to
// take).  What the blocks before this one hold comes from their counts.
template <int WAY>
__device__ __forceinline__ void write_ids(const sel_args &a, unsigned *tmp, int32_t *__restrict__ out_idx)
{
    unsigned *hist_all = a.hist_all;
    const unsigned *state = a.state;
    __shared__ unsigned s_gt[kSelWaves], s_eq[kSelWaves], s_bg[kSelWaves], s_be[kSelWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // digit 1's histogram is done with: zero for the next call
    for (int z = kHist1 + blockIdx.x * kSelBlock + threadIdx.x; z < kHist2; z += gridDim.x * kSelBlock)
        hist_all[z] = 0u;
    const region_t g = region_of(blockIdx.x * kSelWaves + wave, a.list, a.counts, a.scores, a.W, a.N, a.span, a.cap, WAY == 1);
    const unsigned d0 = state[4], d1 = state[5];
    unsigned need = state[7];
    const unsigned d2 = (unsigned)pick_digit<kSelWaves>(hist_all + kHist2, kLastBins, need, tmp);
    const unsigned thr = (((d0 << (kRestBits - kLastBits)) | d1) << kLastBits) | d2;
    // the blocks before this one (at most kSelBlocks <= kSelBlock of them, one a thread)
    unsigned bg = 0, be = 0;
    if (threadIdx.x < blockIdx.x) {
        const unsigned *row = a.suffix + (int64_t)threadIdx.x * kSuffix;
        const unsigned more = row[d2 + 1];
        bg = a.above[threadIdx.x] + more;
        be = row[d2] - more;
    }
    bg = wave_sum(bg);
    be = wave_sum(be);
    unsigned gt = 0, eq = 0;
    auto count = [&](unsigned key, bool in) {
        gt += key > thr;
        eq += key == thr && in;
    };
    for_region<WAY>(
        a.cells, g,
        [&](const uint2 *list, int n) {
            for (int i0 = 0; i0 < n; i0 += 64 * kAhead) {
                unsigned key[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) key[u] = list_at(list, n, i0 + u * 64 + lane).x;
#pragma unroll
                for (int u = 0; u < kAhead; ++u) count(key[u], i0 + u * 64 + lane < n);
            }
        },
        [&](const region_t &d) {
            for_scores<WAY == 1>(d, [&](const pv_f4 &v, int at) {
#pragma unroll
                for (int e = 0; e < 4; ++e) count(score_key(v[e]), at + lane * 4 + e < d.n);
            });
        });
    gt = wave_sum(gt);
    eq = wave_sum(eq);
    if (lane == 0) {
        s_gt[wave] = gt;
        s_eq[wave] = eq;
        s_bg[wave] = bg;
        s_be[wave] = be;
    }
    __syncthreads();
    unsigned rg = 0, re = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
        rg += s_bg[w] + (w < wave ? s_gt[w] : 0u);
        re += s_be[w] + (w < wave ? s_eq[w] : 0u);
    }
    for_region<WAY>(
        a.cells, g,
        [&](const uint2 *list, int n) {
            for (int i0 = 0; i0 < n; i0 += 64 * kAhead) {
                uint2 en[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) en[u] = list_at(list, n, i0 + u * 64 + lane);
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const bool in = i0 + u * 64 + lane < n;
                    const bool isg = en[u].x > thr, ise = in && en[u].x == thr;
                    const unsigned long long bgt = __ballot(isg), beq = __ballot(ise);
                    const unsigned long long below = (1ull << lane) - 1ull;
                    const unsigned pg = rg + __popcll(bgt & below), pe = re + __popcll(beq & below);
                    if (isg || (ise && pe < need)) out_idx[pg + (pe < need ? pe : need)] = (int32_t)en[u].y;
                    rg += __popcll(bgt);
                    re += __popcll(beq);
                }
            }
        },
        [&](const region_t &d) {
            for_scores<WAY == 1>(d, [&](const pv_f4 &v, int at) {
                unsigned long long bgt[4], beq[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned key = score_key(v[e]);
                    bgt[e] = __ballot(key > thr);
                    beq[e] = __ballot(key == thr && at + lane * 4 + e < d.n);
                }
                if (!(bgt[0] | bgt[1] | bgt[2] | bgt[3] | beq[0] | beq[1] | beq[2] | beq[3])) return;   // uniform over the wave
                unsigned pg = rg, pe = re;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    pg = __builtin_amdgcn_mbcnt_hi((unsigned)(bgt[e] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bgt[e], pg));
                    pe = __builtin_amdgcn_mbcnt_hi((unsigned)(beq[e] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)beq[e], pe));
                    rg += (unsigned)__popcll(bgt[e]);
                    re += (unsigned)__popcll(beq[e]);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool isg = (bgt[e] >> lane) & 1ull, ise = (beq[e] >> lane) & 1ull;
                    if (isg || (ise && pe < need)) out_idx[pg + (pe < need ? pe : need)] = (int32_t)(d.base + at + lane * 4 + e);
                    pg += isg;
                    pe += ise;
                }
            });
        });
}

__global__ __launch_bounds__(kSelBlock) void k_write_ids(sel_args a, int32_t *__restrict__ out_idx)
{
    __shared__ unsigned tmp[2 * kCopies * 64];
    write_ids<0>(a, tmp, out_idx);
}

// ---- one weight a group, many of them: the sweep itself collects
// Scores of single weights are as many bytes as the weights: written and read again they cost a third of
// the sweep.  A sample of the scores says beforehand which digit 0 the k-th largest will hardly fall below;
// the sweep keeps the keys from there on, with their ids, in short lists, and writes no scores.  Where a
// list does not fit, and everywhere if the sample said too much (fewer than k keys were
// kept: the three kernels then do the steps from the first digit on, and a fourth, which returns at once
// otherwise, the last), the scores are taken from T and W again.
constexpr int kSampleBlock = 512;
constexpr int kSampleBlocks = 32;
constexpr int kSampleWords = hist_words(kFirstBins);
constexpr int kSampleVecs = kSampleBlock * kSampleBlocks;    // four weights each, one in every 1 / kSampleVecs of the matrix
__global__ __launch_bounds__(kSampleBlock) void k_sample(const float *__restrict__ W, const float *__restrict__ G,
                                                         float alpha, int64_t nvec, unsigned *__restrict__ hist)
{
    __shared__ unsigned lh[kFirstBins];
    __shared__ unsigned s_coarse[64];
    for (int b = threadIdx.x; b < kFirstBins; b += kSampleBlock) lh[b] = 0;
    const int i = blockIdx.x * kSampleBlock + threadIdx.x;
    // a place in the i-th part: anywhere, so that no pattern of rows or columns is missed
    unsigned h = (unsigned)i * 0x9E3779B9u;
    h = (h ^ (h >> 15)) * 0x2C1B3C6Du;
    h ^= h >> 13;
    const int64_t width = nvec / kSampleVecs;
    const int64_t at = (int64_t)i * nvec / kSampleVecs + (int64_t)(((unsigned long long)h * (unsigned long long)width) >> 32);
    const pv_f4 w = reinterpret_cast<const pv_f4 *>(W)[at], g = reinterpret_cast<const pv_f4 *>(G)[at];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float d = fmaf(-alpha, g[e], w[e]) - w[e];
        hist_add<PV_VOTE_ROUNDS>(lh, digit0_of(score_key(d * d)), true);
    }
    __syncthreads();
    flush_hist(lh, hist, kFirstBins, s_coarse);
}

// how many of the sample's keys lie at or above the digit that the sweep collects from: k's share, and ten times
// its root more (the weights of a vector may go together, and so may vectors)
static unsigned sample_rank(int64_t N, int64_t k)
{
    double m = 4.0 * kSampleVecs * (double)k / (double)N, r = 1.0;
    for (int i = 0; i < 40; ++i) r = 0.5 * (r + m / r);
    return (unsigned)(m + 10.0 * r + 32.0);
}

// T = W - alpha * G, and the keys kept: cell by cell, kCell consecutive weights a wave at a time, all waves side by
// side (a contiguous range a wave is 120 us for 45 M weights, a range a block 112, this 96: it is
// bound by the 12 bytes a weight).  Scores that are alike cost no more than writing them
// would.
constexpr int kListBlock = 256;
constexpr int kListBlocks = 1024;
__global__ __launch_bounds__(kListBlock, 4) void k_targets_lists(const float *W, const float *G, float alpha, float *T,
                                                              unsigned *__restrict__ hist_all,
                                                              unsigned *__restrict__ state, int64_t N,
                                                              unsigned sample_kk, cell_args c)
{
    __shared__ unsigned tmp[2 * kCopies * 64];
    __shared__ unsigned lh[kFirstBins];
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * (kListBlock / 64) + (threadIdx.x >> 6), waves = gridDim.x * (kListBlock / 64);
    const int ncells = (int)((N + kCell - 1) / kCell);
    pv_f4 w[kAhead], g[kAhead], wn[kAhead], gn[kAhead];
    auto load = [&](const float *p, int cell, pv_f4 (&v)[kAhead]) {
        const int64_t base = (int64_t)cell * kCell;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t i = base + u * 256 + lane * 4;
            v[u] = pv_f4{0.f, 0.f, 0.f, 0.f};
            if (i + 4 <= N) {
                v[u] = __builtin_nontemporal_load(reinterpret_cast<const pv_f4 *>(p + i));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < N) v[u][e] = p[i + e];
            }
        }
    };
    load(W, wave, w);                               // in flight while the digit is looked up
    load(G, wave, g);
    for (int b = threadIdx.x; b < kFirstBins; b += kListBlock) lh[b] = 0;
    unsigned kk = sample_kk;
    const unsigned lo = (unsigned)pick_digit<kListBlock / 64>(c.sample, kFirstBins, kk, tmp) << kRestBits;   // its barriers also order the clearing above
    if (blockIdx.x == 0 && threadIdx.x == 0) state[2] = lo;
    unsigned total = 0;
    for (int cell = wave; cell < ncells; cell += waves) {
        if (cell + waves < ncells) {
            load(W, cell + waves, wn);
            load(G, cell + waves, gn);
        }
        const int64_t base = (int64_t)cell * kCell;
        uint2 *mine = c.lists + (int64_t)cell * kCellList;
        unsigned cnt = 0;
        unsigned long long hits[kAhead][4];
        auto score = [&](int u, int e) {
            const float d = fmaf(-alpha, g[u][e], w[u][e]) - w[u][e];
            return d * d;
        };
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t i = base + u * 256 + lane * 4;
            pv_f4 t;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                t[e] = fmaf(-alpha, g[u][e], w[u][e]);
                hits[u][e] = __ballot(score_key(score(u, e)) >= lo && i + e < N);
                cnt += (unsigned)__popcll(hits[u][e]);
            }
            if (i + 4 <= N) {
                __builtin_nontemporal_store(t, reinterpret_cast<pv_f4 *>(T + i));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < N) T[i + e] = t[e];
            }
        }
        if (lane == 0) c.counts[cell] = cnt;
        total += cnt;
        if (cnt > (unsigned)kCellList) {            // uniform over the wave
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                pv_f4 sc;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sc[e] = score(u, e);
                    hist_add<PV_VOTE_ROUNDS>(lh, digit0_of(score_key(sc[e])), (hits[u][e] >> lane) & 1ull);
                }
                reinterpret_cast<pv_f4 *>(mine)[u * 64 + lane] = sc;   // (past the matrix' end: nobody reads them)
            }
        } else {
            unsigned at = 0;
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (!(hits[u][0] | hits[u][1] | hits[u][2] | hits[u][3])) continue;   // uniform over the wave
                unsigned pos = at;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    pos = __builtin_amdgcn_mbcnt_hi((unsigned)(hits[u][e] >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((unsigned)hits[u][e], pos));
                    at += (unsigned)__popcll(hits[u][e]);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (!hits[u][e]) continue;       // uniform over the wave
                    const bool hit = (hits[u][e] >> lane) & 1ull;
                    const unsigned key = score_key(score(u, e));
                    if (hit) mine[pos++] = make_uint2(key, (unsigned)(base + u * 256 + lane * 4 + e));
                    hist_add<PV_VOTE_ROUNDS>(lh, digit0_of(key), hit);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            w[u] = wn[u];
            g[u] = gn[u];
        }
    }
    if (lane == 0) c.waves[wave] = total;
    __syncthreads();
    flush_hist(lh, hist_all + kHist0, kFirstBins, tmp);
}

// Digit 0 is resolved and published with the rank left (state[4], state[6]); returns it.  lh: zeroed here.
__device__ __forceinline__ unsigned first_digit(const sel_args &a, unsigned k, unsigned *tmp, unsigned *lh, int *log,
                                                unsigned &share)
{
    for (int b = threadIdx.x; b < kMidBins << kSpreadLog; b += kSelBlock) lh[b] = 0;
    unsigned kk = k;
    const unsigned d0 = (unsigned)pick_digit<kSelWaves>(a.hist_all + kHist0, kFirstBins, kk, tmp, &share);   // its barriers also order the clearing above
    *log = mid_log(share, a.N);                              // the same in every thread
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.state[4] = d0;
        a.state[6] = kk;
    }
    return d0;
}

// Digit 1 of the keys that share digit 0, from T and W.
__device__ __forceinline__ void mid_digit_raw(const sel_args &a, unsigned k, unsigned *tmp, unsigned *lh)
{
    int log;
    unsigned share;
    const unsigned d0 = first_digit(a, k, tmp, lh, &log, share);
    const region_t g = region_of(blockIdx.x * kSelWaves + (threadIdx.x >> 6), a.list, a.counts, a.scores, a.W, a.N, a.span, a.cap, true);
    for_scores<true>(g, [&](const pv_f4 &v, int at) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned key = score_key(v[e]);
            if (at + (int)(threadIdx.x & 63) * 4 + e < g.n && (key >> kRestBits) == d0)
                spread_add(lh, (key >> kLastBits) & (kMidBins - 1), log);
        }
    });
    __syncthreads();
    flush_hist(lh, a.hist_all + kHist1, kMidBins, tmp, log);
}

// The same from the cells; the keys at or above digit 0's range go to the region's list, as in k_collect.
__device__ __forceinline__ void mid_digit_cells(const sel_args &a, unsigned k, uint2 *list, unsigned *counts, unsigned *tmp,
                                                unsigned *lh)
{
    constexpr int kCells = 6;                     // cells whose entries are in flight together
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * kSelWaves + (threadIdx.x >> 6);
    const int ncells = (int)((a.N + kCell - 1) / kCell), per = a.span / kCell;
    const int first = r * per, end = first + per < ncells ? first + per : ncells;
    int log;
    unsigned share;
    const unsigned d0 = first_digit(a, k, tmp, lh, &log, share);
    const unsigned lo = d0 << kRestBits, hi = (d0 + 1u) << kRestBits;
    uint2 *mine = list + (int64_t)r * a.cap;
    // Where most of all weights share digit 0, a region's list (a quarter of its weights) will hardly hold its share: it
    // is not begun, 8 bytes a key that would be written in vain (45 M scores alike: 71.7 us, 41.6 this way).
    const unsigned cap = (int64_t)share * 2 > a.N ? 0u : (unsigned)a.cap;
    unsigned cnt = 0;
    auto take = [&](unsigned key, unsigned id, bool in) {
        const bool hit = in && key >= lo;
        const unsigned long long hits = __ballot(hit);
        if (!hits) return;                        // uniform over the wave
        const unsigned pos = __builtin_amdgcn_mbcnt_hi((unsigned)(hits >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)hits, cnt));
        cnt += (unsigned)__popcll(hits);
        if (hit) {
            if (pos < cap) mine[pos] = make_uint2(key, id);
            if (key < hi) spread_add(lh, (key >> kLastBits) & (kMidBins - 1), log);
        }
    };
    unsigned counts64 = 0;                        // of 64 cells, one a lane
    for (int c0 = first; c0 < end; c0 += kCells) {
        const int in64 = (c0 - first) % (64 / kCells * kCells);
        if (in64 == 0) counts64 = c0 + lane < end ? a.cells.counts[c0 + lane] : 0u;
        unsigned have[kCells];
        uint2 e[kCells];
#pragma unroll
        for (int u = 0; u < kCells; ++u) have[u] = (unsigned)__builtin_amdgcn_readlane((int)counts64, in64 + u);
#pragma unroll
        for (int u = 0; u < kCells; ++u)
            e[u] = lane < (int)have[u] ? a.cells.lists[(int64_t)(c0 + u) * kCellList + lane] : make_uint2(0u, 0u);
#pragma unroll
        for (int u = 0; u < kCells; ++u) {
            const int n = (int)have[u];
            const uint2 *cell = a.cells.lists + (int64_t)(c0 + u) * kCellList;
            if (n <= kCellList) {
                take(e[u].x, e[u].y, lane < n);
#pragma unroll 1
                for (int q = 64; q < n; q += 64) {
                    const uint2 x = list_at(cell, n, q + lane);
                    take(x.x, x.y, q + lane < n);
                }
            } else {
                const int64_t base = (int64_t)(c0 + u) * kCell + lane * 4;
                pv_f4 v[kAhead];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) v[q] = reinterpret_cast<const pv_f4 *>(cell)[q * 64 + lane];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    unsigned long long hits[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) hits[x] = __ballot(score_key(v[q][x]) >= lo && base + q * 256 + x < a.N);
                    if (!(hits[0] | hits[1] | hits[2] | hits[3])) continue;   // uniform over the wave
                    unsigned pos = cnt;
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        pos = __builtin_amdgcn_mbcnt_hi((unsigned)(hits[x] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)hits[x], pos));
                        cnt += (unsigned)__popcll(hits[x]);
                    }
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        if ((hits[x] >> lane) & 1ull) {
                            const unsigned key = score_key(v[q][x]);
                            if (pos < cap) mine[pos] = make_uint2(key, (unsigned)(base + q * 256 + x));
                            ++pos;
                            if (key < hi) spread_add(lh, (key >> kLastBits) & (kMidBins - 1), log);
                        }
                }
            }
        }
    }
    if (lane == 0) counts[r] = cap ? cnt : max(cnt, (unsigned)a.cap + 1u);
    __syncthreads();
    flush_hist(lh, a.hist_all + kHist1, kMidBins, tmp, log);
}

// The sweep kept at least k keys: digit 1 of those.  It kept fewer (state[3]): digit 0 of the others is counted
// first, and everything after it comes a launch later.
__global__ __launch_bounds__(kSelBlock) void k_mid_or_first(sel_args a, int waves, unsigned k, uint2 *list,
                                                            unsigned *counts)
{
    __shared__ unsigned tmp[2 * kCopies * 64];
    __shared__ unsigned lh[kMidBins << kSpreadLog];
    __shared__ unsigned s_sum[kSelWaves];
    static_assert(kFirstBins <= kMidBins << kSpreadLog, "either histogram fits");
    const int lane = threadIdx.x & 63;
    // the last digit's histogram starts at zero, and the sample's is done with
    for (int z = kHist2 + blockIdx.x * kSelBlock + threadIdx.x; z < kHistTotal; z += gridDim.x * kSelBlock)
        a.hist_all[z] = 0u;
    for (int z = blockIdx.x * kSelBlock + threadIdx.x; z < kSampleWords; z += gridDim.x * kSelBlock) a.cells.sample[z] = 0u;
    // from the waves' counts and not from digit 0's histogram, to which blocks of this launch may add
    unsigned kept = 0;
    for (int i = threadIdx.x; i < waves; i += kSelBlock) kept += a.cells.waves[i];
    kept = wave_sum(kept);
    if (lane == 0) s_sum[threadIdx.x >> 6] = kept;
    __syncthreads();
    kept = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) kept += s_sum[w];
    const bool few = kept < k;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.state[3] = few;
    if (!few) {
        mid_digit_cells(a, k, list, counts, tmp, lh);
        return;
    }
    for (int b = threadIdx.x; b < kFirstBins; b += kSelBlock) lh[b] = 0;
    __syncthreads();
    const unsigned lo = a.state[2];
    const region_t g = region_of(blockIdx.x * kSelWaves + (threadIdx.x >> 6), a.list, a.counts, a.scores, a.W, a.N, a.span, a.cap, true);
    for_scores<true>(g, [&](const pv_f4 &v, int at) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned key = score_key(v[e]);
            hist_add<PV_VOTE_ROUNDS>(lh, digit0_of(key), key < lo && at + lane * 4 + e < g.n);
        }
    });
    __syncthreads();
    flush_hist(lh, a.hist_all + kHist0, kFirstBins, tmp);
}

__global__ __launch_bounds__(kSelBlock) void k_last_or_mid(sel_args a, unsigned k)
{
    __shared__ unsigned tmp[2 * kCopies * 64];
    __shared__ unsigned lh[kMidBins << kSpreadLog];
    if (a.state[3]) mid_digit_raw(a, k, tmp, lh);
    else last_digit<2>(a, tmp, lh);
}

__global__ __launch_bounds__(kSelBlock) void k_write_or_last(sel_args a, int32_t *__restrict__ out_idx)
{
    __shared__ unsigned tmp[2 * kCopies * 64];
    __shared__ unsigned lh[kLastBins << kSpreadLog];
    if (a.state[3]) last_digit<1>(a, tmp, lh);
    else write_ids<2>(a, tmp, out_idx);
}

__global__ __launch_bounds__(kSelBlock) void k_write_if_few(sel_args a, int32_t *__restrict__ out_idx)
{
    __shared__ unsigned tmp[2 * kCopies * 64];
    if (a.state[3]) write_ids<1>(a, tmp, out_idx);
}

// Few groups: one block does what the three kernels above do, every key in a register (thread t
// holds kSmallPer consecutive groups), digits 1 and 2 counted in LDS.
constexpr int kSmallPer = kSmallGroups / kSelBlock;
__global__ __launch_bounds__(kSelBlock) void k_select_small(const float *__restrict__ scores,
                                                            unsigned *__restrict__ hist_all, int N,
                                                            unsigned k, int32_t *__restrict__ out_idx)
{
    __shared__ unsigned tmp[2 * kCopies * 64];
    __shared__ unsigned lh[kMidBins << kSpreadLog];
    __shared__ unsigned ll[kLastBins << kSpreadLog];
    __shared__ unsigned s_w[kSelWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = ((N + kSelBlock - 1) / kSelBlock + 3) & ~3;   // whole 16-byte vectors
    const int first = threadIdx.x * per;
    unsigned key[kSmallPer];
#pragma unroll
    for (int q = 0; q < kSmallPer; q += 4) {
        pv_f4 v = {0.f, 0.f, 0.f, 0.f};
        const int i = first + q;
        if (q < per && i + 4 <= N) {
            v = *reinterpret_cast<const pv_f4 *>(scores + i);
        } else if (q < per) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e < N) v[e] = scores[i + e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) key[q + e] = score_key(v[e]);
    }
    const int have = N - first < per ? (N - first < 0 ? 0 : N - first) : per;   // groups of this thread
    for (int b = threadIdx.x; b < kMidBins; b += kSelBlock) lh[b] = 0;
    if (threadIdx.x < kLastBins) ll[threadIdx.x] = 0;
    unsigned kk = k, share;
    const unsigned d0 = (unsigned)pick_digit<kSelWaves>(hist_all + kHist0, kFirstBins, kk, tmp, &share);
    const int log = mid_log(share, N);                       // the same in every thread
    if (log) {
        for (int b = kMidBins + threadIdx.x; b < kMidBins << kSpreadLog; b += kSelBlock) lh[b] = 0;
        for (int b = kLastBins + threadIdx.x; b < kLastBins << kSpreadLog; b += kSelBlock) ll[b] = 0;
        __syncthreads();
    }
    // a digit of an LDS histogram: 64 coarse sums by the waves, then the chosen 64 (every wave alike)
    auto pick_lds = [&](const unsigned *h, int bins) {
        const int nc = bins / kFine;
        __syncthreads();
        for (int c = wave; c < nc; c += kSelWaves) {
            const unsigned t = wave_sum(spread_at(h, c * kFine + lane, log));
            if (lane == 0) tmp[c] = t;
        }
        __syncthreads();
        const int top = nc - 1 - pick_lane(lane < nc ? tmp[nc - 1 - lane] : 0u, kk);
        const int d = top * kFine + (kFine - 1 - pick_lane(spread_at(h, top * kFine + (kFine - 1 - lane), log), kk));
        return (unsigned)d;
    };
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q)
        if (q < have && (key[q] >> kRestBits) == d0) spread_add(lh, (key[q] >> kLastBits) & (kMidBins - 1), log);
    const unsigned want = (d0 << (kRestBits - kLastBits)) | pick_lds(lh, kMidBins);
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q)
        if (q < have && (key[q] >> kLastBits) == want) spread_add(ll, key[q] & (kLastBins - 1), log);
    const unsigned thr = (want << kLastBits) | pick_lds(ll, kLastBins);
    const unsigned need = kk;

    unsigned gt = 0, eq = 0;
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q)
        if (q < have) {
            gt += key[q] > thr;
            eq += key[q] == thr;
        }
    const unsigned both = gt | (eq << 16);   // N < 2^16: neither sum reaches it
    const unsigned inc = wave_incl_scan(both);
    if (lane == 63) s_w[wave] = inc;
    __syncthreads();
    unsigned before = inc - both;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) before += w < wave ? s_w[w] : 0u;
    unsigned rg = before & 0xFFFFu, re = before >> 16;
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q)
        if (q < have) {
            if (key[q] > thr) {
                out_idx[rg + (re < need ? re : need)] = first + q;
                ++rg;
            } else if (key[q] == thr) {
                if (re < need) out_idx[rg + re] = first + q;
                ++re;
            }
        }
    // digit 0's histogram, the only one this path uses, is left zero (its readers are past their barriers)
    for (int z = kHist0 + threadIdx.x; z < kHist1; z += kSelBlock) hist_all[z] = 0u;
}

}  // namespace

// How the groups are dealt to the waves of the passes after the sweep.  A wave needs at least one
// step of 256 keys; a list has room for a quarter of the wave's keys, twice the largest share
// of them that a list is asked to hold on average.  With more than an eighth of all groups chosen
// there are no lists (cap = 0), nor where there is no memory for them.
struct sel_plan {
    int blocks, span, cap;
};
static sel_plan make_sel_plan(int64_t N, int64_t k, bool lists)
{
    sel_plan p;
    const int64_t blocks = (N + kSelWaves * 256 - 1) / (kSelWaves * 256);
    p.blocks = (int)(blocks < kSelBlocks ? (blocks < 1 ? 1 : blocks) : kSelBlocks);
    const int64_t regions = (int64_t)p.blocks * kSelWaves;
    p.span = (int)(((N + regions - 1) / regions + 255) & ~INT64_C(255));
    p.cap = lists && k <= N / 8 ? p.span / 4 : 0;
    return p;
}
static size_t sel_list_bytes(int64_t N)      // whatever k: a later call with another k finds the same block
{
    if (N <= kSmallGroups) return 0;
    const sel_plan p = make_sel_plan(N, 0, true);
    return (size_t)p.blocks * kSelWaves * p.cap * sizeof(uint2);
}
// counts per region, keys above digits 0 and 1 per block, suffix counts per block
constexpr size_t kSelCountWords = (size_t)kSelBlocks * (kSelWaves + 1 + kSuffix);

// The scratch memory of one selection: every group's score (unless the caller keeps them),
// the radix-select histograms (all zero when a call starts, but for the last digit's, which the
// call clears itself), the lists and counts of the passes after the sweep, the digits found so far.
struct sel_bufs {
    float *scores = nullptr;
    unsigned *hist = nullptr, *counts = nullptr, *state = nullptr;
    uint2 *list = nullptr;
    sel_plan plan{};
    pv_norm_req *norm = nullptr;
    cell_args cells{};       // lists: nullptr unless the sweep collects
};

__global__ void k_sel_clear(unsigned *p, int n)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

static pv_status select_run(pv_ctx *ctx, const pv_layout *l, const float *T, const float *W,
                            int64_t k, int32_t *out_idx, const sel_bufs &bufs, const float *G,
                            float alpha, const pv_adam_t *adam, float *m, float *v);

// A context's scratch, one block: histograms, counts and state | lists | scores.  Lists are
// left out where the device has no room for them (then, and for that size from then on: a call of
// a size that was seen before does not allocate).
constexpr int64_t kCollectMin = 3 << 22;
static int64_t cells_of(int64_t N) { return (N + kCell - 1) / kCell; }
static pv_status sel_scratch(pv_ctx *ctx, int64_t N, bool own_scores, sel_bufs *b, bool *lists)
{
    constexpr size_t head = ((kHistTotal + kSelCountWords + 8) * sizeof(unsigned) + 255) & ~(size_t)255;
    const size_t list = sel_list_bytes(N);
    // whatever the group size: the scores, or the cells in their place
    const size_t rest = own_scores ? (size_t)cells_of(N) * (kCellList * sizeof(uint2) + sizeof(unsigned)) : 0;
    *lists = list == 0 || ctx->select.bytes >= head + list + rest;
    if (!*lists && head + list + rest < ctx->select_refused) {
        *lists = pv_ensure(ctx, ctx->select, head + list + rest, kHistTotal * sizeof(unsigned)) == PV_OK;
        if (!*lists) ctx->select_refused = head + list + rest;
    }
    const size_t scores_at = head + (*lists ? list : 0);
    const pv_status st = pv_ensure(ctx, ctx->select, scores_at + rest, kHistTotal * sizeof(unsigned));
    if (st != PV_OK) return st;
    char *base = static_cast<char *>(ctx->select.ptr);
    b->hist = reinterpret_cast<unsigned *>(base);
    b->counts = b->hist + kHistTotal;
    b->state = b->counts + kSelCountWords;
    b->list = *lists ? reinterpret_cast<uint2 *>(base + head) : nullptr;
    b->scores = own_scores ? reinterpret_cast<float *>(base + scores_at) : nullptr;
    return PV_OK;
}

pv_status pv_select_scores(pv_ctx *ctx, int64_t N, float **scores)
{
    sel_bufs b;
    bool lists;
    const pv_status st = sel_scratch(ctx, N, /*own_scores=*/true, &b, &lists);
    *scores = b.scores;
    return st;
}

// One weight a group, and so many that the scores' way through memory costs more than the sample (6 us) and a launch that
// returns at once (4.6).  The call, scores written / collected: k = N / 100, 4 M weights 40.0 / 39.6 us, 8 M 53.6 /
// 50.3, 12.6 M 65.4 / 59.8, 16.8 M 79.6 / 69.0, 25 M 105 / 85.6, 45 M 164 / 130; rows of their own size 78.2 / 76.1,
// 96.9 / 92.6, 129 / 112, 202 / 169 from 12.6 M on.  The keys kept are 8 bytes each, so fewer of fewer weights pay:
// k = N / 16, 12.6 M 69.4 / 67.4 (rows 85.1 / 85.0); N / 10, 12.6 M 70.9 / 71.6, 16.8 M 85.7 / 82.6 (102.2 / 103.8); N / 8,
// 16.8 M 88.1 / 86.2 (103.6 / 106.9), 25 M 119 / 111 (146 / 141).  Scores all alike are written and read all the same:
// 12.6 M 98.4 / 105.2, 16.8 M 125.3 / 128.5, 25 M 172.4 / 171.6, 45 M 295 / 277.
static bool sweep_collects(const pv_layout *l, int64_t k)
{
    const int64_t N = pv_num_groups(l);
    const int64_t most = N / (N >= 3 << 23 ? 8 : N >= 1 << 24 ? 10 : 16);
    return l->group_size == 1 && N >= kCollectMin && k > 0 && k <= most;
}

// G != nullptr: T is an OUTPUT, formed here as W - alpha * G in the same pass that scores it.
pv_status pv_launch_select(pv_ctx *ctx, const pv_layout *l, const float *T, const float *W,
                           int64_t k, int32_t *out_idx, float *scores, const float *G, float alpha,
                           const pv_adam_t *adam, float *m, float *v, pv_norm_req *norm)
{
    const int N = (int)pv_num_groups(l);
    pv_status st;
    if (norm && (G || !pv_select_norm_supported(l)))
        return pv_fail(ctx, PV_ERR_UNSUPPORTED, "norm request: scores-only sweep, one codebook, g = 8 or 16");
    sel_bufs bufs;
    bool lists;
    st = sel_scratch(ctx, N, /*own_scores=*/!scores, &bufs, &lists);
    if (st != PV_OK) return st;
    bufs.plan = make_sel_plan(N, k, lists);
    // whatever k and the direction: a later call of the shape does not allocate.  A block of its own: in the one
    // above it took smaller matrices past sizes from which an allocation costs more (2 MiB for 1003 x 2072 in groups of 8)
    bool sample = !scores && l->group_size == 1 && N >= kCollectMin && !ctx->sample_refused;
    // a first call of such a shape into a graph, its other scratch large enough from a call of another shape: scores are written
    if (sample && !ctx->sample.ptr && pv_capturing(ctx)) sample = false;
    if (sample) {
        sample = pv_ensure(ctx, ctx->sample, kSampleWords * sizeof(unsigned), kSampleWords * sizeof(unsigned)) == PV_OK;
        ctx->sample_refused = !sample;
    }
    if (G && !adam && sample && lists && sweep_collects(l, k)) {
        bufs.cells.sample = static_cast<unsigned *>(ctx->sample.ptr);
        // the cells take the place of the scores
        bufs.cells.lists = reinterpret_cast<uint2 *>(bufs.scores);
        bufs.cells.counts = reinterpret_cast<unsigned *>(bufs.cells.lists + cells_of(N) * kCellList);
        bufs.cells.waves = bufs.counts + (size_t)kSelBlocks * (kSelWaves + 1);   // where the suffix counts come later
        static_assert(kListBlocks * (kListBlock / 64) <= kSelBlocks * kSuffix, "a count a wave");
        bufs.plan.span = (bufs.plan.span + kCell - 1) / kCell * kCell;           // (cap stays: a quarter of the span that the lists were sized for)
    }
    if (scores) bufs.scores = scores;
    bufs.norm = norm;
    return select_run(ctx, l, T, W, k, out_idx, bufs, G, alpha, adam, m, v);
}

bool pv_select_norm_supported(const pv_layout *l)
{
    return l->num_codebooks == 1 && (l->group_size == 8 || l->group_size == 16);
}

int pv_select_norm_parts() { return kMaxBlocks; }

// ---------------------------------------------------------------- selection without allocation
// For callers that cannot allocate device memory (code under HIP graph capture, tight serving
// loops, harnesses that forbid it): the same selection with its scratch in one static device
// array.  Each GPU holds its own copy of the array for the life of the process; every call on
// a GPU shares it, so calls that overlap on one GPU (two streams, two contexts) race.
constexpr int64_t kStaticMaxGroups = INT64_C(1) << 22;            // 4 194 304 groups
constexpr size_t kStaticScoresOff = 0;
constexpr size_t kStaticHistOff = kStaticScoresOff + (size_t)kStaticMaxGroups * sizeof(float) + 256;
constexpr size_t kStaticCcOff = kStaticHistOff + (size_t)kHistTotal * sizeof(unsigned);
constexpr size_t kStaticStateOff = kStaticCcOff + kSelCountWords * sizeof(unsigned);
constexpr size_t kStaticBytes = kStaticStateOff + 256;            // about 16.5 MiB
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

// In host code `scratch` is only a stand-in for the symbol: the memory is reached through the
// address the runtime reports for it on each device.
constexpr int kMaxDevices = 64;
static unsigned char *g_static_ptr[kMaxDevices] = {nullptr};

// The device must be current.  Called by pv_create (once per context) and again by the entry
// point itself; the first call on a device asks the runtime, later ones return the kept address.
pv_status pv_static_scratch_init(pv_ctx *ctx, int device)
{
    if (device < 0 || device >= kMaxDevices)
        return pv_fail(ctx, PV_ERR_INVALID_ARG, "device %d outside 0..%d", device, kMaxDevices - 1);
    unsigned char *p = __atomic_load_n(&g_static_ptr[device], __ATOMIC_ACQUIRE);
    if (p) return PV_OK;
    void *sym = nullptr;
    hipError_t e = hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !sym) {
        (void)hipGetLastError();
        return pv_fail(ctx, PV_ERR_DEVICE, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    }
    __atomic_store_n(&g_static_ptr[device], static_cast<unsigned char *>(sym), __ATOMIC_RELEASE);
    return PV_OK;
}

int64_t pv_static_max_groups() { return kStaticMaxGroups; }

pv_status pv_launch_select_static(pv_ctx *ctx, const pv_layout *l, const float *T, const float *W,
                                  int64_t k, int32_t *out_idx, float *scores)
{
    pv_status st = pv_static_scratch_init(ctx, ctx->device);
    if (st != PV_OK) return st;
    unsigned char *base = __atomic_load_n(&g_static_ptr[ctx->device], __ATOMIC_ACQUIRE);
    sel_bufs bufs;
    bufs.scores = scores ? scores : reinterpret_cast<float *>(base + kStaticScoresOff);
    bufs.hist = reinterpret_cast<unsigned *>(base + kStaticHistOff);
    bufs.counts = reinterpret_cast<unsigned *>(base + kStaticCcOff);
    bufs.list = nullptr;   // no room for lists: the passes after the sweep read the scores
    bufs.plan = make_sel_plan(pv_num_groups(l), k, /*lists=*/false);
    bufs.state = reinterpret_cast<unsigned *>(base + kStaticStateOff);
    // the array keeps what the last call (of any context) left: the histograms must start at
    // zero whatever that was (a fill kernel, which a capturing caller may record)
    hipLaunchKernelGGL(k_sel_clear, dim3(16), dim3(kBlock), 0, ctx->stream, bufs.hist, kHistTotal);
    const bool timing = ctx->timing;   // timing brackets create events: not in this call
    ctx->timing = false;
    st = select_run(ctx, l, T, W, k, out_idx, bufs, nullptr, 0.0f, nullptr, nullptr, nullptr);
    ctx->timing = timing;
    return st;
}

static pv_status select_run(pv_ctx *ctx, const pv_layout *l, const float *T, const float *W,
                            int64_t k, int32_t *out_idx, const sel_bufs &bufs, const float *G,
                            float alpha, const pv_adam_t *adam, float *m, float *v)
{
    const int N = (int)pv_num_groups(l);
    const int g = l->group_size;
    pv_status st;
    float *scores = bufs.scores;
    unsigned *hist = bufs.hist;
    unsigned *state = bufs.state;
    int32_t *all_ids = k == N ? out_idx : nullptr;   // every group is chosen: the sweep writes the ids as it goes
    const int want_hist = k > 0 && k < N ? 1 : 0;
    const bool vec_g = g == 4 || g == 8 || g == 16 || g == 32 || g == 64;
    if (bufs.cells.lists) {   // (see sweep_collects)
        const sel_plan p = bufs.plan;
        unsigned *counts = bufs.counts, *above = counts + (size_t)kSelBlocks * kSelWaves;
        const sel_args a{T, W, hist, state, (int64_t)N, p.span, p.cap, bufs.list, counts, above, above + kSelBlocks, bufs.cells};
        int64_t blocks = ((int64_t)N + kCell * (kListBlock / 64) - 1) / (kCell * (kListBlock / 64));
        if (blocks > kListBlocks) blocks = kListBlocks;
        {
            pv_timed t(ctx, PV_K_ENCODE_TARGETS);
            hipLaunchKernelGGL(k_sample, dim3(kSampleBlocks), dim3(kSampleBlock), 0, ctx->stream, W, G, alpha,
                               (int64_t)N / 4, bufs.cells.sample);
            hipLaunchKernelGGL(k_targets_lists, dim3((unsigned)blocks), dim3(kListBlock), 0, ctx->stream, W, G, alpha,
                               const_cast<float *>(T), hist, state, (int64_t)N, sample_rank(N, k), bufs.cells);
        }
        pv_timed t(ctx, PV_K_SELECT);
        hipLaunchKernelGGL(k_mid_or_first, dim3(p.blocks), dim3(kSelBlock), 0, ctx->stream, a,
                           (int)blocks * (kListBlock / 64), (unsigned)k, bufs.list, counts);
        hipLaunchKernelGGL(k_last_or_mid, dim3(p.blocks), dim3(kSelBlock), 0, ctx->stream, a, (unsigned)k);
        hipLaunchKernelGGL(k_write_or_last, dim3(p.blocks), dim3(kSelBlock), 0, ctx->stream, a, out_idx);
        hipLaunchKernelGGL(k_write_if_few, dim3(p.blocks), dim3(kSelBlock), 0, ctx->stream, a, out_idx);
        PV_HIP(ctx, hipGetLastError());
        return PV_OK;
    }
    if (G && !adam && (g == 1 || g == 2)) {
        pv_timed t(ctx, PV_K_ENCODE_TARGETS);
        const int64_t nelem = (int64_t)N * g;
        int64_t vb = ((nelem >> 2) + kBlock * kVecUnroll - 1) / (kBlock * kVecUnroll);
        const unsigned vblocks = (unsigned)(vb < 1 ? 1 : (vb < kMaxBlocks ? vb : kMaxBlocks));
        float *Tw = const_cast<float *>(T);
        if (g == 1)
            hipLaunchKernelGGL(k_targets_scores_hist0_sub<1>, dim3(vblocks), dim3(kBlock), 0, ctx->stream,
                               W, G, alpha, Tw, scores, hist, nelem, want_hist, all_ids);
        else
            hipLaunchKernelGGL(k_targets_scores_hist0_sub<2>, dim3(vblocks), dim3(kBlock), 0, ctx->stream,
                               W, G, alpha, Tw, scores, hist, nelem, want_hist, all_ids);
    } else {
    if (G && !vec_g) {   // no fused kernel for this group size: form T first
        // (the Adam variant reaches this launcher only for the group sizes that have one)
        st = pv_launch_encode_targets(ctx, W, G, alpha, const_cast<float *>(T),
                                      l->out_features * l->in_features);
        if (st != PV_OK) return st;
        G = nullptr;
    }
    if (G) {
        pv_timed t(ctx, PV_K_ENCODE_TARGETS);
        const int64_t nvec = (int64_t)N * (g / 4);
        int64_t vb = (nvec + kBlock * kVecUnroll - 1) / (kBlock * kVecUnroll);
        const unsigned vblocks = (unsigned)(vb < kMaxBlocks ? vb : kMaxBlocks);
        float *Tw = const_cast<float *>(T);
        const pv_adam_t a = adam ? *adam : pv_adam_t{};
#define PV_FUSED(PARTS_)                                                                            \
    do {                                                                                            \
        if (adam)                                                                                   \
            hipLaunchKernelGGL((k_targets_scores_hist0_vec<PARTS_, true>), dim3(vblocks), dim3(kBlock), \
                               0, ctx->stream, W, G, alpha, Tw, scores, hist, nvec, want_hist, all_ids, a, m, v); \
        else                                                                                        \
            hipLaunchKernelGGL((k_targets_scores_hist0_vec<PARTS_, false>), dim3(vblocks),          \
                               dim3(kBlock), 0, ctx->stream, W, G, alpha, Tw, scores, hist, nvec,   \
                               want_hist, all_ids, a, m, v);                                                 \
    } while (0)
        if (g == 4) PV_FUSED(1);
        else if (g == 8) PV_FUSED(2);
        else if (g == 16) PV_FUSED(4);
        else if (g == 32) PV_FUSED(8);
        else PV_FUSED(16);
#undef PV_FUSED
    } else {
        pv_timed t(ctx, PV_K_GROUP_SCORES);
        const int64_t nvec = (int64_t)N * (g / 4);
        int64_t vb = (nvec + kBlock * kVecUnroll - 1) / (kBlock * kVecUnroll);
        const unsigned vblocks = (unsigned)(vb < kMaxBlocks ? vb : kMaxBlocks);
        int64_t sb = ((int64_t)N + kBlock - 1) / kBlock;
        const unsigned sblocks = (unsigned)(sb < kMaxBlocks ? sb : kMaxBlocks);
        norm_args na{};
        if (bufs.norm) {
            na.codes = bufs.norm->codes;
            na.cb4 = reinterpret_cast<const pv_f4 *>(bufs.norm->codebooks);
            na.scales = bufs.norm->scales;
            na.partial = bufs.norm->partial;
            na.mask = (1u << l->nbits) - 1u;
            na.inv_gpr = 1.0 / (double)(l->in_features / g);
            bufs.norm->parts = (int)vblocks;
        }
#define PV_SCORES(PARTS_)                                                                          \
    do {                                                                                           \
        if (bufs.norm)                                                                             \
            hipLaunchKernelGGL((k_scores_hist0_vec<PARTS_, true>), dim3(vblocks), dim3(kBlock), 0, \
                               ctx->stream, T, W, scores, hist, nvec, want_hist, all_ids, na);              \
        else                                                                                       \
            hipLaunchKernelGGL((k_scores_hist0_vec<PARTS_, false>), dim3(vblocks), dim3(kBlock), 0, \
                               ctx->stream, T, W, scores, hist, nvec, want_hist, all_ids, na);              \
    } while (0)
        if (g == 4) PV_SCORES(1);
        else if (g == 8) PV_SCORES(2);
        else if (g == 16) PV_SCORES(4);
        else if (g == 32) PV_SCORES(8);
        else if (g == 64) PV_SCORES(16);
        else
            hipLaunchKernelGGL(k_scores_hist0, dim3(sblocks), dim3(kBlock), 0, ctx->stream, T, W,
                               scores, hist, N, g, want_hist, all_ids);
#undef PV_SCORES
    }
    }   // group sizes other than 1 and 2
    if (want_hist && N <= kSmallGroups) {
        // one block's three phases cost less than three launches up to here
        pv_timed t(ctx, PV_K_SELECT);
        hipLaunchKernelGGL(k_select_small, dim3(1), dim3(kSelBlock), 0, ctx->stream, scores, hist, N,
                           (unsigned)k, out_idx);
    } else if (want_hist) {
        pv_timed t(ctx, PV_K_SELECT);
        const sel_plan p = bufs.plan;
        unsigned *counts = bufs.counts, *above = counts + (size_t)kSelBlocks * kSelWaves;
        unsigned *suffix = above + kSelBlocks;
        hipLaunchKernelGGL(k_collect, dim3(p.blocks), dim3(kSelBlock), 0, ctx->stream, scores, hist, state,
                           (int64_t)N, (unsigned)k, p.span, p.cap, bufs.list, counts);
        const sel_args a{scores, nullptr, hist, state, (int64_t)N, p.span, p.cap, bufs.list, counts, above, suffix, {}};
        hipLaunchKernelGGL(k_last_digit, dim3(p.blocks), dim3(kSelBlock), 0, ctx->stream, a);
        hipLaunchKernelGGL(k_write_ids, dim3(p.blocks), dim3(kSelBlock), 0, ctx->stream, a, out_idx);
    }
    PV_HIP(ctx, hipGetLastError());
    return PV_OK;
}
