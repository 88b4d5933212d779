// Nearest-codeword search for one codebook (M = 1) on the matrix cores.
//
// The decision "which codeword minimises || s * C[c] - t ||^2" (Eq. 7 argmin,
// App. K "try every code") is taken in double precision, exactly as the plain
// definition does.  The matrix cores only FILTER: by App. D's identity
//     || c - x ||^2 = ||c||^2 - 2 <c, x> + ||x||^2 ,   x = t / s ,
// the distance of every codeword to every selected group is one dense
// contraction.  It is evaluated on fp16 MFMA (fp32 accumulate) for fp16-rounded
// copies c_hi, x_hi of the operands, scaled by a power of two P so that the
// largest codebook entry lies in [16, 32), in the form of a "closeness"
//     kv(c) = SHIFT + 2 <c_hi, x_hi> - ||c_hi||^2  =  SHIFT + ||x_hi||^2 - || c_hi - x_hi ||^2
// which is LARGE for near codewords.  SHIFT = (||x_hi|| + min_c ||c|| + margin)^2 is a constant
// of the group that makes kv non-negative for at least the smallest codeword, so a negative kv
// marks a codeword farther away than that one.
//   g = 8:  the spare K slots of the 32x32x16 instruction carry -||c_hi||^2 (three fp16
//           pieces against -1) and SHIFT (three pieces against 1): the accumulator IS kv.
//   g = 16: all 16 K slots carry data, so the accumulator is 2 <c_hi, x_hi> alone.  The
//           codebook is laid out in ascending order of ||c_hi||^2, so that the norms of the
//           32 U codewords behind one key differ by next to nothing: after the maximum of the
//           products was taken (never below zero, which can only raise it), the smallest of
//           those norms is subtracted (again raising the key at most) and SHIFT added.
//
// Running maximum (per lane, in registers): the 16 accumulators of a lane belong to one group
// (column) and to 16 consecutive codeword positions (a "half tile"); they are reduced with
// v_max3_i32 on the float bits (correct whenever the maximum is non-negative; if every value
// is negative the result is some negative value, which is all that is needed), the chain runs
// on over the U tiles of a "super-unit", the low 11 bits of the result are replaced by the
// super-unit number, and the lane keeps the largest and second largest such key per partition.
// A partition is (codeword range of the work item) x (half wave) x (super-unit residue class).
//
// Exact re-rank + certificate (k_rerank): the 16 U codewords behind the best key and the
// previous code are evaluated in double -> E*.  With the triangle inequality
//     | ||P C[c] - P x|| - ||c_hi - x_hi|| | <= dC + dx
// (dC = max_c ||P C[c] - c_hi||, dx = ||P x - x_hi|| + division rounding) a codeword can reach
// E* only if  kv(c) >= SHIFT + ||x_hi||^2 - (P sqrt(E*)/|s| + dC + dx)^2, and the key behind
// which it sits is at least kv(c) - E1 (fp32 accumulation, dropped pieces, truncation).  Every
// best key at or above that cut is evaluated as well; a partition whose runner-up key reaches
// the cut may hide further codewords and is scanned completely, in the same kernel.  Hence the
// chosen code is the double-precision argmin with the tie rule of the definition, whatever the
// fp16 rounding did.
#include "pv_internal.h"
#include "pv_counts.h"
#include "pv_dpp.h"

// Launch shape of the contraction kernel (tunable at build time).
#ifndef PV_STAGE
#define PV_STAGE 32   // KiB of operand A per LDS stage (= codeword tiles per stage)
#endif
#ifndef PV_NBX
#define PV_NBX 2      // group tiles (32 groups) per wave
#endif
#ifndef PV_WAVES
#define PV_WAVES 8    // waves per block
#endif
#ifndef PV_OCC
#define PV_OCC 2      // blocks per compute unit the register / LDS budget allows
#endif
#ifndef PV_SUPER
#define PV_SUPER 2    // codeword tiles behind one key (a super-unit)
#endif
#ifndef PV_TEAM
#define PV_TEAM 8     // lanes of the re-rank kernel that share one group at g = 8 (twice as many at g = 16: measured)
#endif
constexpr int rerank_team(int g) { return g == 16 && PV_TEAM < 16 ? 2 * PV_TEAM : PV_TEAM; }
#ifndef PV_DEPTH
#define PV_DEPTH 2    // units (matrix instructions) in flight before a unit's accumulators are reduced
#endif

namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));

constexpr int kBlock = 256;
constexpr int kU = PV_SUPER;
constexpr int kResidues = 4;         // super-unit residue classes tracked separately per lane
constexpr unsigned kKeyMask = 0x7FFu;
constexpr int kNoKey = (int)0x80000000;             // "no key": below every key a lane can form
constexpr float kHalfMinNormal = 6.103515625e-05f;  // 2^-14
constexpr float kGamma = 7.62939453125e-06f;        // 2^-17: fp32 accumulation bound per unit of sum|terms|
constexpr float kNormMargin = 0.04f;                // >= max_c | ||c_hi|| - ||P c|| | (half an fp16 ulp below 32, 16 dims)
constexpr int kNormFine = 5 * 2048;                 // buckets of the norm ordering (g = 16): five octaves finely,
constexpr int kNormCoarse = 1024;                   // the octaves below and those above coarsely
constexpr int kNormBins = kNormFine + 2 * kNormCoarse;
constexpr int kCbCopies = 8;                        // copies of the bucket counters, one per die

// cb_meta layout (unsigned[8]): [0] bits of max|C|, [1] ~bits of min_c ||c||^2 (unscaled),
// [2] bits of max ||P c - c_hi||^2 (written by the scoring kernel), [3] bad-codebook flag,
// [5] bits of max_c ||c||^2 (unscaled)
// x_meta layout (float[4] per selected group): SHIFT as the kernel adds it, ||x_hi||^2, E1,
// dx (negative: the filter is skipped for this group)

__device__ __forceinline__ float scale_from_maxabs(unsigned maxbits, bool *ok)
{
    float m = __uint_as_float(maxbits);
    *ok = (m > 0.0f) && (m < 3.0e38f) && (m >= 1.0e-30f);
    if (!*ok) return 1.0f;
    int ex;
    (void)frexpf(m, &ex);          // m = f * 2^ex, f in [0.5, 1)
    return ldexpf(1.0f, 5 - ex);   // m * P in [16, 32)
}

__device__ __forceinline__ _Float16 to_half_flush(float v)
{
    return fabsf(v) < kHalfMinNormal ? (_Float16)0.0f : (_Float16)v;
}

// value -> three fp16 pieces p1 + p2 + p3 ~= v (pieces below the normal range dropped)
__device__ __forceinline__ void split3(float v, _Float16 *p)
{
    p[0] = to_half_flush(v);
    float r = v - (float)p[0];
    p[1] = to_half_flush(r);
    r = r - (float)p[1];
    p[2] = to_half_flush(r);
}

// Residue cycles of the table owned by codeword split `split` of `nsplit`: cycles are dealt to
// the splits round robin by rank (for g = 16 the rank is the norm order, so every split sees
// every norm band: codewords near a target have similar norms, and they should fall into
// different partitions), and a split's cycles lie next to each other in memory.
__device__ __host__ __forceinline__ int split_count(int split, int ncyc, int nsplit)
{
    return (ncyc - split + nsplit - 1) / nsplit;
}
__device__ __host__ __forceinline__ int split_begin(int split, int ncyc, int nsplit)
{
    // sum of split_count over the splits before: the first ncyc % nsplit splits hold one more
    const int q = ncyc / nsplit, r = ncyc % nsplit;
    return split * q + (split < r ? split : r);
}

// fp16 copy of one scaled codeword: c_hi (as floats), its squared norm, the squared rounding error
template <int G>
__device__ __forceinline__ void round_codeword(const float *__restrict__ cw, float P, bool ok,
                                               float (&hf)[G], float &n2, float &d2)
{
    n2 = 0.0f;
    d2 = 0.0f;
    const pv_f4 *src = reinterpret_cast<const pv_f4 *>(cw);
#pragma unroll
    for (int v4 = 0; v4 < G / 4; ++v4) {
        pv_f4 raw = src[v4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = v4 * 4 + e;
            float v = ok ? P * raw[e] : 0.0f;
            hf[i] = (float)to_half_flush(v);
            n2 = fmaf(hf[i], hf[i], n2);
            float d = v - hf[i];
            d2 = fmaf(d, d, d2);
        }
    }
}

// ---------------------------------------------------------------- the codebook's statistics
//
// Codebooks beyond kOneBlock codewords: k_cb_stats, one block per kCbChunk codewords, leaves its
// part as a plain store, and whoever needs the whole adds up at most 64 parts (atomics of all
// blocks end up on one cache line, one after the other: 3 us).  Up to kOneBlock codewords there is
// no such launch: every block of k_prep takes the statistics of the whole codebook itself.
constexpr int kCbPer = 4;                     // codewords a thread of the codebook part
constexpr int kCbChunk = kBlock * kCbPer;     // codewords a block
constexpr int kCbParts = 65536 / kCbChunk;    // blocks of the largest codebook
constexpr int kOneBlock = kCbChunk;
static_assert(kCbParts <= 64, "one wave reduces the parts");

// Device scratch of the preparation.
struct cb_mem {
    pv_f4 *part;          // [kCbParts] {max |c|, min norm^2, max norm^2, bad}
    float *dpart;         // [kCbParts] largest rounding error ||P c - c_hi||^2 of a block's codewords
    float *anchor;        // [1] g = 16: norm that the buckets are counted from
    unsigned *count;      // [copies][kNormBins / 2] g = 16: codewords per bucket (two in a word: a copy
                          // has at most 65536 / kCbCopies), zero between calls
    unsigned *cursor;     // [copies][kNormBins / 2] g = 16: codewords of a bucket placed so far
};
constexpr size_t kCbWords = kCbParts * 4 + kCbParts + 16 + (size_t)kCbCopies * (kNormBins / 2);     // without `count`

__device__ __forceinline__ float wave_min_f(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fminf(v, __shfl_xor(v, off));
    return v;
}
__device__ __forceinline__ float wave_max_f(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    return v;
}

struct cb_stat {
    float m = 0.0f, nmin = __builtin_huge_valf(), nmax = 0.0f;
    bool bad = false;
};

// statistics of one codeword
template <int G>
__device__ __forceinline__ void stat_add(cb_stat &s, const pv_f4 (&cw)[G / 4])
{
    float n2 = 0.0f;
#pragma unroll
    for (int v4 = 0; v4 < G / 4; ++v4)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = fabsf(cw[v4][e]);
            s.bad |= !(a <= 3.0e38f);
            s.m = fmaxf(s.m, a);
            n2 = fmaf(cw[v4][e], cw[v4][e], n2);
        }
    s.nmin = fminf(s.nmin, n2);
    s.nmax = fmaxf(s.nmax, n2);
}

// a block's statistics, in thread 0; `tmp`: one pv_f4 a wave of LDS
__device__ __forceinline__ pv_f4 stat_block(const cb_stat &s, pv_f4 *tmp)
{
    pv_f4 p = {wave_max_f(s.m), wave_min_f(s.nmin), wave_max_f(s.nmax), __any(s.bad) ? 1.0f : 0.0f};
    if ((threadIdx.x & 63) == 0) tmp[threadIdx.x >> 6] = p;
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int w = 1; w < kBlock / 64; ++w) {
            p.x = fmaxf(p.x, tmp[w].x);
            p.y = fminf(p.y, tmp[w].y);
            p.z = fmaxf(p.z, tmp[w].z);
            p.w = fmaxf(p.w, tmp[w].w);
        }
    return p;
}

// statistics -> the words that the other kernels read (see cb_meta)
__device__ __forceinline__ void meta_words(const pv_f4 &p, unsigned *out)
{
    out[0] = __float_as_uint(p.x);
    out[1] = p.y >= 0.0f && p.y < 3.0e38f ? ~__float_as_uint(p.y) : 0u;
    out[2] = 0u;
    out[3] = p.w != 0.0f || !(p.z < 3.0e38f) ? 1u : 0u;
    out[4] = 0u;
    out[5] = __float_as_uint(p.z);
    out[6] = out[7] = 0u;
}

// ... of all blocks' parts, to `out` (8 unsigneds of LDS); called by all threads of a block
__device__ __forceinline__ void meta_of_parts(const pv_f4 *part, int nparts, unsigned *out)
{
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        pv_f4 p = {0.0f, __builtin_huge_valf(), 0.0f, 0.0f};
        if (lane < nparts) p = part[lane];
        p.x = wave_max_f(p.x);
        p.y = wave_min_f(p.y);
        p.z = wave_max_f(p.z);
        p.w = wave_max_f(p.w);
        if (lane == 0) meta_words(p, out);
    }
    __syncthreads();
}

// A slot of the changed codes' count has a line of its own: the atomics of different slots would
// queue on a shared one (406 blocks, seven slots in one line: 1.5 us of the re-rank's 13).
constexpr int kSlotStride = 16;

// What a call counts in starts at zero: done by the call's first kernel.
struct clear_args {
    unsigned long long *stats, *num_changed, *change_slots;
    unsigned *fb_count;
    int nslots;
};
__device__ __forceinline__ void clear_counters(const clear_args &a, int block, int nblocks)
{
    for (int i = block * kBlock + threadIdx.x; i < a.nslots; i += nblocks * kBlock) a.change_slots[i * kSlotStride] = 0ull;
    if (block == 0) {
        if (threadIdx.x < 8) a.stats[threadIdx.x] = 0ull;
        if (threadIdx.x < 4) a.fb_count[threadIdx.x] = 0u;
        if (threadIdx.x == 0 && a.num_changed) *a.num_changed = 0ull;
    }
}

// Norm ordering (g = 16): buckets of ||c_hi||^2.  A key's bound lies off by up to the width of its
// bucket, and that decides how many groups the re-rank has to search again: 2048 buckets an octave
// where most norms lie (four octaves below `anchor`, the largest norm of a sample, and one above), 32
// an octave beyond.  P is a power of two, so ||c_hi|| / P is known before P is: the entries rounded to
// fp16's 11 bits (those that P c leaves below fp16's normal range count as zero in c_hi, see
// norm_bucket_floor).
constexpr int kNormShift = 12;
template <int G>
__device__ __forceinline__ float norm_rounded(const pv_f4 (&cw)[G / 4])
{
    float n2 = 0.0f;
#pragma unroll
    for (int i = 0; i < G; ++i) {
        unsigned u = __float_as_uint(cw[i >> 2][i & 3]);
        u = (u + 0xFFFu + ((u >> 13) & 1u)) & ~0x1FFFu;
        const float v = __uint_as_float(u);
        n2 = fmaf(v, v, n2);
    }
    return n2;
}
__device__ __forceinline__ int norm_fine(float v) { return (int)((__float_as_uint(v) & 0x7FFFFFFFu) >> kNormShift); }
__device__ __forceinline__ int norm_bucket(float n2, float anchor)
{
    const int d = norm_fine(n2) - norm_fine(anchor) + 4 * 2048;
    const int key = kNormCoarse + (d < 0 ? d >> 6 : d < kNormFine ? d : kNormFine + ((d - kNormFine) >> 6));
    return key < 0 ? 0 : (key > kNormBins - 1 ? kNormBins - 1 : key);
}
// A bound from below for the computed ||c_hi||^2 of the bucket's codewords: its edge, less the
// rounding of two fp32 sums of 16 terms (2 * 16 * 2^-24 of the sum) and 16 flushed entries (2^-28 each).
__device__ __forceinline__ float norm_bucket_floor(int bucket, float anchor, float P)
{
    const int key = bucket - kNormCoarse;
    const int d = key < 0 ? key * 64 : key < kNormFine ? key : kNormFine + (key - kNormFine) * 64;
    const int e = d + norm_fine(anchor) - 4 * 2048;
    const float edge = __uint_as_float(bucket == 0 || e <= 0 ? 0u : (unsigned)e << kNormShift);
    // (below 1e-30 the squares of the entries have lost bits to the bottom of fp32's range)
    return edge < 1.0e-30f ? 0.0f : fmaxf(edge * P * P * 0.999997f - 6.0e-8f, 0.0f);
}
// two 16-bit counters a word
__device__ __forceinline__ unsigned half_of(unsigned w, int e) { return e & 1 ? w >> 16 : w & 0xFFFFu; }
__device__ __forceinline__ unsigned half_one(int e) { return 1u << (16 * (e & 1)); }

// Codebook statistics, one block per kCbChunk codewords; g = 16 also counts the norm buckets (the
// anchor from a sample that every block takes alike; block b counts into copy b % kCbCopies:
// workgroups are dealt to the dies round robin, so a copy's atomics stay in one L2).  Latency: 65536
// codewords, g = 16, 7.2 us; statistics, buckets and their scan as three kernels took 23 us.
template <int G>
__global__ __launch_bounds__(kBlock) void k_cb_stats(const float *__restrict__ cb, int csize, cb_mem mem,
                                                     uint16_t *__restrict__ bucket, clear_args ca)
{
    __shared__ pv_f4 s_tmp[kBlock / 64];
    __shared__ float s_n[kBlock / 64];
    __shared__ unsigned s_hist[G == 16 ? kNormBins / 2 : 1];     // as in mem.count
    const int tid = threadIdx.x;
    const pv_f4 *cb4 = reinterpret_cast<const pv_f4 *>(cb);
    pv_f4 own[kCbPer][G / 4], smp[G / 4];
    if (G == 16)
#pragma unroll
        for (int v = 0; v < G / 4; ++v) smp[v] = cb4[(int64_t)tid * (csize / kBlock) * (G / 4) + v];
#pragma unroll
    for (int r = 0; r < kCbPer; ++r)      // csize is a multiple of kCbChunk here
#pragma unroll
        for (int v = 0; v < G / 4; ++v) own[r][v] = cb4[(int64_t)(blockIdx.x * kCbChunk + r * kBlock + tid) * (G / 4) + v];
    clear_counters(ca, blockIdx.x, gridDim.x);
    float anchor = 0.0f;
    if (G == 16) {
        for (int i = blockIdx.x * kBlock + tid; i < kCbCopies * (kNormBins / 2); i += gridDim.x * kBlock) mem.cursor[i] = 0u;
        for (int b = tid; b < kNormBins / 2; b += kBlock) s_hist[b] = 0u;
        const float n = wave_max_f(norm_rounded<G>(smp));
        if ((tid & 63) == 0) s_n[tid >> 6] = n;
        __syncthreads();
        anchor = fmaxf(fmaxf(s_n[0], s_n[1]), fmaxf(s_n[2], s_n[3]));
        if (blockIdx.x == 0 && tid == 0) *mem.anchor = anchor;
    }
    cb_stat s;
#pragma unroll
    for (int r = 0; r < kCbPer; ++r) {
        stat_add<G>(s, own[r]);
        if constexpr (G == 16) {
            const int b = norm_bucket(norm_rounded<G>(own[r]), anchor);
            bucket[blockIdx.x * kCbChunk + r * kBlock + tid] = (uint16_t)b;
            atomicAdd(&s_hist[b >> 1], half_one(b));
        }
    }
    const pv_f4 p = stat_block(s, s_tmp);       // its barrier also ends the counting
    if (tid == 0) mem.part[blockIdx.x] = p;
    if (G == 16) {
        unsigned *count = mem.count + (blockIdx.x % kCbCopies) * (kNormBins / 2);
        for (int b = tid; b < kNormBins / 2; b += kBlock) {
            const unsigned v = s_hist[b];
            if (v) atomicAdd(&count[b], v);
        }
    }
}

// Table position -> tile and row of the operand (see k_prep).
struct operand_row {
    int tile, row;
};
__device__ __forceinline__ operand_row operand_row_of(int pos)
{
    const int q = pos & 15, uu = (pos >> 4) % kU, hw = (pos / (16 * kU)) & 1;
    return {(pos / (32 * kU)) * kU + uu, 8 * (q >> 2) + 4 * hw + (q & 3)};
}

// Place of the smallest norm behind the key of a position: the keys of a residue cycle lie next to
// each other for each half wave, so that one 16-byte read brings a lane all it closes in a cycle.
__device__ __forceinline__ int key_norm_at(int pos)
{
    const int key = pos / (16 * kU), su = key >> 1, hw = key & 1;
    return (su / kResidues * 2 + hw) * kResidues + su % kResidues;
}

// What the preparation of the selected groups reads and writes.
struct group_args {
    const float *T, *scales, *codebook;
    const int32_t *group_idx;
    const uint16_t *codes;
    int k, k_pad, gpr, N, csize_mask;
    h8 *X;
    float *x_meta, *x_stage;
    float *reach;          // cells only: squared radius beyond which a cell is left out
};

// One selected group (position j in the list): x = t / s, its fp16 copy, per-group bounds.
// CELLS: SHIFT is what makes kv non-negative for every codeword at most as far as the current one
// (and hardly any other), and reach[j] is that distance's square for the test of whole cells.
template <int G, bool CELLS>
__device__ __forceinline__ void prep_group(const group_args &ga, int j, float P, bool ok, const unsigned *meta)
{
    // ||c_hi|| <= P max_c ||c|| + rounding
    const float cmax = P * sqrtf(__uint_as_float(meta[5])) * 1.0001f + kNormMargin;
    float shift = 0.0f, xx = 0.0f, e1 = 0.0f, dx = -1.0f, reach = -1.0f;
    h8 chunk[2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) chunk[u][e] = (_Float16)0.0f;
    int n = j < ga.k ? ga.group_idx[j] : -1;
    if (n >= ga.N) n = -1;
    // everything is read before anything is written: the loads of one step are in flight together
    float s = 0.0f;
    int code = 0;
    pv_f4 tgt[G / 4], cur[G / 4];
#pragma unroll
    for (int v4 = 0; v4 < G / 4; ++v4) tgt[v4] = cur[v4] = pv_f4{0.0f, 0.0f, 0.0f, 0.0f};
    if (n >= 0) {
        code = (int)ga.codes[n] & ga.csize_mask;
        s = ga.scales[n / ga.gpr];
        const pv_f4 *src = reinterpret_cast<const pv_f4 *>(ga.T + (int64_t)n * G);
#pragma unroll
        for (int v4 = 0; v4 < G / 4; ++v4) tgt[v4] = src[v4];
        if constexpr (CELLS) {
            const pv_f4 *cw = reinterpret_cast<const pv_f4 *>(ga.codebook + (int64_t)code * G);
#pragma unroll
            for (int v4 = 0; v4 < G / 4; ++v4) cur[v4] = cw[v4];
        }
    }
    {
        pv_f4 *stage = reinterpret_cast<pv_f4 *>(ga.x_stage + (int64_t)j * (G + 4));
        pv_f4 tail = {s, __int_as_float(code), __int_as_float(n), 0.0f};
        stage[G / 4] = tail;
        if (n >= 0)
#pragma unroll
            for (int v4 = 0; v4 < G / 4; ++v4) stage[v4] = tgt[v4];
    }
    if (n >= 0 && ok) {
        bool fits = (s != 0.0f) && (fabsf(s) < 3.0e38f);
        const float div = fits ? s : 1.0f;
        float d2 = 0.0f, u2 = 0.0f, p2 = 0.0f;      // p2: squared distance of the current code's codeword, scaled
#pragma unroll
        for (int v4 = 0; v4 < G / 4; ++v4) {
            const pv_f4 raw = tgt[v4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = v4 * 4 + e;
                float u = P * (raw[e] / div);
                if (!(fabsf(u) < 240.0f)) fits = false;   // also catches NaN / inf
                _Float16 hv = to_half_flush(fits ? u : 0.0f);
                float hf = (float)hv;
                xx = fmaf(hf, hf, xx);
                float d = u - hf;
                d2 = fmaf(d, d, d2);
                u2 = fmaf(u, u, u2);
                if constexpr (CELLS) {
                    const float dp = P * cur[v4][e] - u;
                    p2 = fmaf(dp, dp, p2);
                }
                chunk[i >> 3][i & 7] = hv;
            }
        }
        const float xn = sqrtf(xx) * 1.0001f;
        // the smallest codeword, scaled: kv of that codeword is then non-negative
        const float cn0 = P * sqrtf(__uint_as_float(~meta[1])) * 1.0001f + kNormMargin;
        float want = (xn + cn0) * (xn + cn0) * 1.0001f + 1.0e-3f;
        if (fits && xx < 57000.0f && want < 60000.0f) {
            // bound of the fp32 accumulation error of one accumulator (g = 8: products, norm
            // pieces and SHIFT add up to at most 2 (cmax + xn)^2 in magnitude; g = 16: the
            // products alone, then two fp32 additions on the vector ALU), plus dropped fp16 pieces
            const float e1p = (G == 8 ? 2.0f : 1.0f) * kGamma * (cmax + xn) * (cmax + xn) * 1.01f +
                              (G == 8 ? 5.0e-4f : 4.0e-7f * (cmax + xn) * (cmax + xn));
            e1 = 1.01f * e1p;
            // rounding of x to fp16, plus the fp32 division and scaling roundings (2^-22 ||u||)
            dx = sqrtf(d2) * 1.0001f + 2.4e-7f * sqrtf(u2) + 1.0e-30f;
            if constexpr (CELLS) {
                // a codeword that beats the current one has ||P c - u|| <= dp, hence ||c_hi - x_hi|| <=
                // dp + dx + kNormMargin (rounding of a codeword): kv is non-negative for those.
                // dp: fp32 differences of elements up to (32 + |u|), each rounded once
                const float dp = sqrtf(p2) * 1.00001f + 3.0e-7f * (cmax + xn);
                reach = (dp + dx) * (dp + dx) * 1.0001f;
                want = (dp + dx + kNormMargin) * (dp + dx + kNormMargin) * 1.0001f + e1 - xx * 0.9999f + 1.0e-3f;
                if (!(fabsf(want) < 60000.0f)) {     // also NaN: every codeword is looked at instead
                    dx = reach = -1.0f;
                    want = 0.0f;
                }
            }
            if (G == 8) {
                _Float16 pieces[3];
                split3(want, pieces);
                shift = ((float)pieces[0] + (float)pieces[1]) + (float)pieces[2];
                chunk[1][0] = (_Float16)-1.0f;
                chunk[1][1] = (_Float16)-1.0f;
                chunk[1][2] = (_Float16)-1.0f;
                chunk[1][3] = pieces[0];
                chunk[1][4] = pieces[1];
                chunk[1][5] = pieces[2];
            } else {
                shift = want;
            }
        } else {
            xx = 0.0f;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) chunk[u][e] = (_Float16)0.0f;
        }
    }
    const int gt = j >> 5, col = j & 31;
#pragma unroll
    for (int u = 0; u < 2; ++u) ga.X[((int64_t)gt * 2 + u) * 32 + col] = chunk[u];
    pv_f4 m;
    m.x = shift;
    m.y = xx;
    m.z = e1;
    m.w = dx;
    reinterpret_cast<pv_f4 *>(ga.x_meta)[j] = m;
    if constexpr (CELLS) ga.reach[j] = reach;
}

// Operand preparation, one launch for both sides.
//
// Blocks [0, cb_blocks): kCbPer codeword positions of the padded table a thread.  A codeword is
// placed at position pos (g = 8: its own index; g = 16: the next free rank of its norm bucket -
// what the buckets before hold, what the copies of the counters before this block's hold, what
// blocks of the same copy placed already - and the residue cycles of the ranking
// dealt round robin to the codeword splits), perm[pos] names it.  The 32 U
// positions of super-unit su are split in two runs of 16 U, one per half wave hw, each run in
// U pieces of 16, one per tile: position pos = ((su * 2 + hw) * U + uu) * 16 + q sits in tile
// su * U + uu at row 8*(q/4) + 4*hw + q%4, so that accumulator q of half wave hw is that
// position, and the 16 U positions behind one key of a lane are consecutive (for g = 16: in
// norm order, none of their norms is below nmin[key_norm_at(pos)]).  Operand A of tile t, k-half h, row r
// is the 16-byte chunk A[(t * 2 + h) * 32 + r]:
//   g = 8:  k-half 0 = 2 c_hi, k-half 1 = { three pieces of ||c_hi||^2, 1, 1, 1, 0, 0 }
//   g = 16: k-half 0 = 2 c_hi[0..8), k-half 1 = 2 c_hi[8..16)
// Positions past the codebook's end (padding up to whole super-units) are zero rows.
//
// Remaining blocks: one thread per selected group (position j in the list): x = t / s, its
// fp16 copy, per-group bounds.  Operand B of group tile gt, k-half h, column col is the chunk
// X[(gt * 2 + h) * 32 + col]:
//   g = 8:  k-half 0 = x_hi, k-half 1 = { -1, -1, -1, three pieces of SHIFT, 0, 0 }
//   g = 16: the two halves of x_hi (SHIFT travels in x_meta)
// and x_stage[j] = { the g target values, the row scale, the current code, the group id } is
// what the re-rank kernel needs of the group, in one place (its loads then depend on nothing
// but the list position).
//
// The codebook's blocks are a chain of latencies (parts, counters, codewords, stores) that runs
// beside the groups' blocks, so what can go out early does: the claim of a place in a bucket needs
// only the bucket.  Code runs once per block, cold: the loop over the counters stays rolled, and
// the key bounds come from the codeword that got a key's first rank (written out per bucket they
// cost 5 us of instruction fetch).  65536 codewords, g = 16: codebook alone 16 us, 183k groups alone
// 16 us, both 21 us.
template <int G, bool ONE>
__global__ __launch_bounds__(kBlock) void k_prep(const float *__restrict__ cb, int csize, int cpad,
                                                 int cb_blocks, unsigned *__restrict__ meta, cb_mem mem,
                                                 h8 *__restrict__ A, uint16_t *__restrict__ perm,
                                                 const uint16_t *__restrict__ bucket,
                                                 float *__restrict__ nmin, float *__restrict__ cnorm,
                                                 group_args ga, int ncyc, int nsplit, clear_args ca)
{
    __shared__ unsigned s_meta[8];
    __shared__ pv_f4 s_tmp[kBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const pv_f4 *cb4 = reinterpret_cast<const pv_f4 *>(cb);
    if (ONE) {           // no k_cb_stats before: this block looks at the whole codebook
        cb_stat s;
        pv_f4 cw[kCbPer][G / 4];
#pragma unroll
        for (int r = 0; r < kCbPer; ++r)
#pragma unroll
            for (int v = 0; v < G / 4; ++v) {
                const int c = r * kBlock + tid;
                cw[r][v] = cb4[(int64_t)(c < csize ? c : csize - 1) * (G / 4) + v];
            }
#pragma unroll
        for (int r = 0; r < kCbPer; ++r) stat_add<G>(s, cw[r]);
        const pv_f4 p = stat_block(s, s_tmp);
        if (tid == 0) meta_words(p, s_meta);
        __syncthreads();
        clear_counters(ca, blockIdx.x, gridDim.x);
    } else {
        meta_of_parts(mem.part, csize / kCbChunk, s_meta);
    }
    bool ok;
    const float P = scale_from_maxabs(s_meta[0], &ok);
    if (blockIdx.x == 0 && tid < 8) meta[tid] = s_meta[tid];
    if ((int)blockIdx.x >= cb_blocks) {
        const int j = ((int)blockIdx.x - cb_blocks) * kBlock + tid;
        if (j < ga.k_pad) prep_group<G, false>(ga, j, P, ok && s_meta[3] == 0u && s_meta[1] != 0u, s_meta);
        return;
    }

    // ranks of the codewords in norm order (g = 16)
    constexpr int kRun = 16, kRuns = kNormBins / (kBlock * kRun);      // buckets a thread looks at together
    __shared__ unsigned s_base[G == 16 ? kNormBins / 2 : 1], s_w[2][kBlock / 64];
    int bkt[kCbPer];
    unsigned placed[kCbPer];
    float anchor = 0.0f;
    const int copy = blockIdx.x % kCbCopies;
    auto place_of = [&](int rank) {       // cycle rc of the ranking is cycle rc / nsplit of split rc % nsplit
        constexpr int per_cycle = 32 * kU * kResidues;
        const int rc = rank / per_cycle;
        return (split_begin(rc % nsplit, ncyc, nsplit) + rc / nsplit) * per_cycle + rank % per_cycle;
    };
    if constexpr (G == 16) {
        anchor = ONE ? __uint_as_float(s_meta[5]) : *mem.anchor;
        if constexpr (ONE) {
            for (int b = tid; b < kNormBins / 2; b += kBlock) s_base[b] = 0u;
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kCbPer; ++r) {
                const int c = r * kBlock + tid;
                if (c < csize) {
                    pv_f4 cw[G / 4];
#pragma unroll
                    for (int v = 0; v < G / 4; ++v) cw[v] = cb4[(int64_t)c * (G / 4) + v];
                    bkt[r] = norm_bucket(norm_rounded<G>(cw), anchor);
                    atomicAdd(&s_base[bkt[r] >> 1], half_one(bkt[r]));
                }
            }
            __syncthreads();
        } else {
#pragma unroll
            for (int r = 0; r < kCbPer; ++r) bkt[r] = bucket[blockIdx.x * kCbChunk + r * kBlock + tid];
#pragma unroll
            for (int r = 0; r < kCbPer; ++r)
                placed[r] = atomicAdd(&mem.cursor[copy * (kNormBins / 2) + (bkt[r] >> 1)], half_one(bkt[r]));
        }
        unsigned first = 0;
#pragma unroll 1
        for (int run = 0; run < kRuns; ++run) {
            // the buckets' codewords in copies 0 - 3, in the others, in those before this block's
            const int w0 = (run * kBlock + tid) * (kRun / 2);
            unsigned lo[kRun / 2], hi[kRun / 2], before[kRun / 2], sum = 0;
#pragma unroll
            for (int e = 0; e < kRun / 2; ++e) {
                lo[e] = ONE ? s_base[w0 + e] : 0u;
                hi[e] = before[e] = 0u;
            }
            if (!ONE) {
#pragma unroll
                for (int q = 0; q < kCbCopies; ++q) {
                    const uint4 *src = reinterpret_cast<const uint4 *>(mem.count + q * (kNormBins / 2) + w0);
#pragma unroll
                    for (int v = 0; v < kRun / 8; ++v) {
                        const uint4 x = src[v];
                        const unsigned n4[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            (q < kCbCopies / 2 ? lo : hi)[v * 4 + e] += n4[e];
                            before[v * 4 + e] += q < copy ? n4[e] : 0u;
                        }
                    }
                }
            }
            auto all = [&](int e) { return half_of(lo[e >> 1], e) + half_of(hi[e >> 1], e); };
#pragma unroll
            for (int e = 0; e < kRun; ++e) sum += all(e);
            unsigned inc = sum;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const unsigned u = __shfl_up(inc, off);
                if (lane >= off) inc += u;
            }
            if (lane == 63) s_w[run & 1][wave] = inc;
            __syncthreads();
            unsigned rank = first + inc - sum;
#pragma unroll
            for (int w = 0; w < kBlock / 64; ++w) {
                const unsigned n = s_w[run & 1][w];
                rank += w < wave ? n : 0u;
                first += n;
            }
#pragma unroll
            for (int e = 0; e < kRun; ++e) {
                const unsigned at = rank + half_of(before[e >> 1], e);
                // (a bucket behind the last codeword may be at 65536, which no one asks for)
                if (e & 1) s_base[w0 + (e >> 1)] |= at << 16;
                else s_base[w0 + (e >> 1)] = at & 0xFFFFu;
                rank += all(e);
            }
        }
        // keys with nothing but padding behind them
        if (blockIdx.x == 0)
            for (int h = (csize + 16 * kU - 1) / (16 * kU) + tid; h < cpad / (16 * kU); h += kBlock) nmin[key_norm_at(place_of(h * (16 * kU)))] = 3.0e38f;
        __syncthreads();
    }

    float d2 = 0.0f;
#pragma unroll
    for (int r = 0; r < kCbPer; ++r) {
        const int c = blockIdx.x * kCbChunk + r * kBlock + tid;
        if (ONE && c >= cpad) continue;
        h8 chunk[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) chunk[u][e] = (_Float16)0.0f;
        int pos = c;                          // (padding exists only where the ranks are places already)
        if (!ONE || c < csize) {        // (larger codebooks are whole chunks)
            float hf[G], n2, d2c;
            round_codeword<G>(cb + (int64_t)c * G, P, ok, hf, n2, d2c);
            d2 = fmaxf(d2, d2c);
#pragma unroll
            for (int i = 0; i < G; ++i) chunk[i >> 3][i & 7] = (_Float16)(2.0f * hf[i]);
            if constexpr (G == 8) {
                _Float16 pieces[3];
                split3(n2, pieces);
                chunk[1][0] = pieces[0];
                chunk[1][1] = pieces[1];
                chunk[1][2] = pieces[2];
                chunk[1][3] = (_Float16)1.0f;
                chunk[1][4] = (_Float16)1.0f;
                chunk[1][5] = (_Float16)1.0f;
            } else {
                const int b = bkt[r];
                unsigned rank;
                if (ONE) {
                    rank = half_of(atomicAdd(&s_base[b >> 1], half_one(b)), b);
                } else {
                    rank = half_of(s_base[b >> 1], b) + half_of(placed[r], b);
                }
                pos = place_of((int)rank);
                cnorm[pos] = n2;           // for the re-rank kernel's cheap distances
                // the ranks of a key's positions lie in the bucket of the first of them, or above it
                if (rank % (16 * kU) == 0) nmin[key_norm_at(pos)] = norm_bucket_floor(b, anchor, P);
            }
            perm[pos] = (uint16_t)c;
        } else if (G == 16) {
            cnorm[pos] = 0.0f;
        }
        const operand_row o = operand_row_of(pos);
#pragma unroll
        for (int u = 0; u < 2; ++u) A[((int64_t)o.tile * 2 + u) * 32 + o.row] = chunk[u];
    }
    d2 = wave_max_f(d2);
    __syncthreads();
    if (lane == 0) s_tmp[wave].x = d2;
    __syncthreads();
    if (tid == 0) mem.dpart[blockIdx.x] = fmaxf(fmaxf(s_tmp[0].x, s_tmp[1].x), fmaxf(s_tmp[2].x, s_tmp[3].x));
}

// Plain C so that the compiler sees the reads of MFMA results and inserts the
// wait states the hardware requires between a matrix instruction and a vector
// read of its destination (it does not look inside inline assembly).  It folds
// the pair of maxima into one v_max3_i32.
__device__ __forceinline__ int imax3(int a, int b, int c)
{
    return max(max(a, b), c);
}

// (m & mask) | unit in one instruction; operands are ordinary vector results.
__device__ __forceinline__ int and_or(int m, unsigned vmask, unsigned unit)
{
    int r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(m), "v"(vmask), "s"(unit));
    return r;
}

__device__ __forceinline__ int imed3(int a, int b, int c)
{
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Largest of a running value and the 16 accumulators (float bits compared as signed integers:
// the order of non-negative floats; a negative float lies below every non-negative one).
// A single chain: a tree of independent v_max3 measured no faster here (the waves of a SIMD
// interleave).
template <bool FIRST>
__device__ __forceinline__ int acc_max(const f16v &acc, int run)
{
    int m;
    if (FIRST && run == kNoKey) {
        m = imax3(__float_as_int(acc[0]), __float_as_int(acc[1]), __float_as_int(acc[2]));
        m = imax3(m, __float_as_int(acc[3]), __float_as_int(acc[4]));
        m = imax3(m, __float_as_int(acc[5]), __float_as_int(acc[6]));
        m = imax3(m, __float_as_int(acc[7]), __float_as_int(acc[8]));
        m = imax3(m, __float_as_int(acc[9]), __float_as_int(acc[10]));
        m = imax3(m, __float_as_int(acc[11]), __float_as_int(acc[12]));
        m = imax3(m, __float_as_int(acc[13]), __float_as_int(acc[14]));
        return max(m, __float_as_int(acc[15]));
    }
    m = imax3(run, __float_as_int(acc[0]), __float_as_int(acc[1]));
    m = imax3(m, __float_as_int(acc[2]), __float_as_int(acc[3]));
    m = imax3(m, __float_as_int(acc[4]), __float_as_int(acc[5]));
    m = imax3(m, __float_as_int(acc[6]), __float_as_int(acc[7]));
    m = imax3(m, __float_as_int(acc[8]), __float_as_int(acc[9]));
    m = imax3(m, __float_as_int(acc[10]), __float_as_int(acc[11]));
    m = imax3(m, __float_as_int(acc[12]), __float_as_int(acc[13]));
    return imax3(m, __float_as_int(acc[14]), __float_as_int(acc[15]));
}

// place of the record of (partition p, list position j)
__device__ __forceinline__ int64_t rec_at(int p, int64_t j, int P, int k_pad)
{
    (void)P;
    return (int64_t)p * k_pad + j;
}

// The distance contraction.  Block = PV_WAVES waves; wave w owns NB group tiles (32 groups
// each) whose B operands stay in registers; the block streams the codeword tiles of its split
// through a double-buffered LDS stage shared by its waves.  A stage is filled with direct
// global->LDS loads (no staging registers) one stage ahead of its use.  Inside a stage the
// loop is software pipelined: the MFMA of unit (tile, group tile) is issued, then the
// accumulators of the unit before it are reduced on the vector ALU while the matrix core
// works.  Output: for every group and partition the largest and second largest key.
template <int G, int NB>
__global__ __launch_bounds__(PV_WAVES * 64, (PV_OCC * PV_WAVES) / 4) void k_score_mfma(
    const h8 *__restrict__ A, const h8 *__restrict__ X, const float *__restrict__ x_meta,
    const float *__restrict__ nmin, int2 *__restrict__ partials, int ncyc, int nsplit, int per_half,
    int gblocks, int k_pad, unsigned *__restrict__ next_item, const float *__restrict__ wanted,
    const float *__restrict__ dpart, int cb_parts, unsigned *__restrict__ counts, int ncounts,
    unsigned *__restrict__ meta)
{
    if (wanted && *wanted == 0.0f) return;   // the cells do the work (pv_cells.h)
    // the largest rounding error of the codebook, for the re-rank; the counts are done with
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        const float d = wave_max_f((int)threadIdx.x < cb_parts ? dpart[threadIdx.x] : 0.0f);
        if (threadIdx.x == 0) meta[2] = __float_as_uint(d);
    }
    for (int i = blockIdx.x * (PV_WAVES * 64) + threadIdx.x; i < ncounts; i += gridDim.x * (PV_WAVES * 64)) counts[i] = 0u;
    constexpr int S = PV_STAGE;                                    // tiles per stage
    constexpr int kStageChunks = S * 64;                           // 16-byte chunks per stage
    constexpr int kW = PV_WAVES;                                   // waves per block
    constexpr int kRounds = (kStageChunks / 64 + kW - 1) / kW;     // 64-chunk rows per wave
    constexpr int kSuStage = S / kU;                               // super-units per stage
    constexpr int kCycle = kResidues * kU;                         // tiles per residue cycle
    static_assert(S % kCycle == 0, "stage must hold whole residue cycles");
    static_assert(2 * kSuStage <= 64, "one lane per staged norm");
    // two stages in SEPARATE arrays (+ one tile of padding each): the compiler then knows that
    // the asynchronous fill of one does not alias the reads of the other and does not wait
    // for the fill before every read
    __shared__ h8 lds0[kStageChunks + 64];
    __shared__ h8 lds1[kStageChunks + 64];
    __shared__ __align__(16) float ldn0[64], ldn1[64];     // smallest norm behind each key of the stage (g = 16)
    __shared__ unsigned s_item;
    // the wave's number in a scalar register: what follows from it is uniform (g = 16: 18 spilled registers without
    // it, some reloaded inside the loop over the tiles, 7 with it)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    unsigned vmask = ~kKeyMask;
    asm volatile("" : "+v"(vmask));   // keep the mask in a vector register
    // Work items = (group block, codeword split).  A block starts with item blockIdx.x; when
    // there are more items than blocks the rest is handed out through a counter, so the
    // blocks in flight stay busy until the items run out (every block leaves when its next
    // item number passes the item count).
    const unsigned items = (unsigned)gblocks * (unsigned)nsplit;
    for (unsigned item = blockIdx.x; item < items;) {
    const int gb = (int)(item % (unsigned)gblocks), split = (int)(item / (unsigned)gblocks);
    const int gtile0 = (gb * kW + wave) * NB;
    // a split is a whole number of residue cycles (the table is padded to one)
    const int t_begin = split_begin(split, ncyc, nsplit) * kCycle;
    const int t_end = t_begin + split_count(split, ncyc, nsplit) * kCycle;

    h8 b[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) b[nb] = X[(int64_t)(gtile0 + nb) * 64 + lane];
    // g = 16: SHIFT of the lane's group (added to the key on the vector ALU)
    float shift[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
        shift[nb] = G == 16 ? x_meta[((int64_t)(gtile0 + nb) * 32 + (lane & 31)) * 4] : 0.0f;

    int best[NB][kResidues], second[NB][kResidues], run[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        run[nb] = kNoKey;
#pragma unroll
        for (int r = 0; r < kResidues; ++r) best[nb][r] = second[nb][r] = kNoKey;
    }

    // rows of 64 chunks (1 KiB) are copied by one wave each: lane i -> chunk row + i
    auto fetch = [&](int t0, h8 *dst, float *dstn) {
        const int valid = (t_end - t0 < S ? t_end - t0 : S) * 64;
        const h8 *src = A + (int64_t)t0 * 64;
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const int row = (u * kW + wave) * 64;   // uniform over the wave
            if (row < valid && row < kStageChunks)
                __builtin_amdgcn_global_load_lds(
                    (const void *)(src + row + lane),
                    (__attribute__((address_space(3))) void *)(&dst[row]), 16, 0, 0);
        }
        if (G == 16 && wave == kW - 1)   // the norm table is padded: reads past the split's end are harmless
            __builtin_amdgcn_global_load_lds((const void *)(nmin + (t0 / kU) * 2 + lane),
                                             (__attribute__((address_space(3))) void *)(&dstn[0]), 4,
                                             0, 0);
    };

    // Units (tile, nb) are issued in order; while the matrix core works on the last kD of them
    // the vector ALU reduces the unit kD back.  Four accumulator sets, used round robin, so a
    // set is rewritten three units after it was last read.
    constexpr int kD = PV_DEPTH;
    constexpr int kSets = 4;
    constexpr int kUnitsCycle = NB * kCycle;            // units per residue cycle (unrolled)
    static_assert(kUnitsCycle % kSets == 0 && kD >= 1 && kD < kSets, "accumulator sets must line up");
    f16v acc[kSets];
    h8 a_cur, a_nxt;
    pv_f4 norm = {0.0f, 0.0f, 0.0f, 0.0f};              // g = 16: of the keys of a residue cycle
    static_assert(kResidues == 4, "a cycle's norms are one vector");
    // they are read with the kNormTile-th tile: after the last key of the cycle before is closed (kD units into this one),
    // and not after the first of this one
    constexpr int kNormTile = (kD + NB - 1) / NB;
    static_assert(G != 16 || (kNormTile * NB <= kD + (kU - 1) * NB && kNormTile < kCycle), "norms come before they are used");
    auto issue = [&](int nb, int set) {
        const f16v z = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        acc[set] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a_cur, b[nb], z, 0, 0, 0);
    };
    // rel: the tile's place in its residue cycle (a constant after unrolling: it picks the
    // registers); su_stage: its super-unit within the stage.  The key is closed at the last
    // tile of a super-unit.
    auto reduce = [&](int t0, int su_stage, int rel, int nb, int set) {
        const int uu = rel % kU;
        // g = 16: the chain starts at zero (the products can be negative, and a negative
        // maximum would not come out of the integer comparison: zero bounds it from above)
        if (uu == 0) run[nb] = G == 16 ? acc_max<false>(acc[set], 0) : acc_max<true>(acc[set], kNoKey);
        else run[nb] = acc_max<false>(acc[set], run[nb]);
        if (uu == kU - 1) {
            const int r = rel / kU;
            int kv = run[nb];
            if (G == 16) kv = __float_as_int((__int_as_float(kv) - norm[r]) + shift[nb]);
            const int key = and_or(kv, vmask, (unsigned)(t0 / kU + su_stage));
            second[nb][r] = imed3(best[nb][r], second[nb][r], key);
            best[nb][r] = max(best[nb][r], key);
        }
    };
    // One stage of `cnt` tiles (a whole number of residue cycles).
    auto run_stage = [&](const h8 *buf, const float *bufn, int t0, int cnt) {
        a_cur = buf[lane];
#pragma unroll 1
        for (int q4 = 0; q4 < cnt; q4 += kCycle) {
#pragma unroll
            for (int vr = 0; vr < kUnitsCycle; ++vr) {
                const int u = vr / NB, nb = vr % NB, ts = q4 + u;
                if (G == 8 && nb == 0) a_nxt = buf[(ts + 1) * 64 + lane];   // one spare tile pads the LDS array
                // g = 16: the wave asks for priority while it hands its matrix instruction over
                // (measured: 384.0 -> 382.0 us on 183 500 groups; at g = 8 it costs 2 %)
                if (G == 16) __builtin_amdgcn_s_setprio(3);
                issue(nb, vr % kSets);
                if (G == 16) {
                    __builtin_amdgcn_s_setprio(0);
                    // Reads of LDS behind the matrix instruction that waits for the ones before: the wait counts
                    // all reads, and one issued just before it would be waited for in full.  The cycle's norms
                    // once the last key of the cycle before is closed, a tile ahead of the first use (183 500
                    // groups x 65536 codewords: 413 -> 390 us in the mean, 397 -> 376 at best, with this and scalar
                    // wave numbers; the two norms of a key read where it is closed held the wave up for a round trip
                    // twice a super-unit).  Seven vector registers are still spilled (18 before).
                    // Matrix instruction and maxima alone, nothing read, take 27 ns a unit on random operands
                    // (18 on zeros: the clock gives way to the power); this loop takes 33.
                    if (nb == 0) {
                        __builtin_amdgcn_sched_barrier(0);
                        a_nxt = buf[(ts + 1) * 64 + lane];
                        if (u == kNormTile)
                            norm = *reinterpret_cast<const pv_f4 *>(bufn + q4 / kCycle * 2 * kResidues + (lane >> 5) * kResidues);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                // the unit kD back: tile q4 + dq (dq may point into the cycle before), group tile wnb
                const int dq = (vr - kD >= 0) ? (vr - kD) / NB : -((kD - vr + NB - 1) / NB);
                const int wnb = ((vr - kD) % NB + NB) % NB;
                if (q4 > 0 || vr >= kD)
                    reduce(t0, (q4 + dq) / kU, (dq + kCycle) % kCycle, wnb,
                           ((vr - kD) % kSets + kSets) % kSets);
                // keep this order: left to itself the scheduler moves a unit's reduction up
                // behind its own matrix instruction, and the wave then waits out that
                // instruction's whole latency instead of working on older units
                __builtin_amdgcn_sched_barrier(0);
                if (nb == NB - 1) a_cur = a_nxt;
            }
        }
        // the last kD units of the stage (its last residue cycle)
#pragma unroll
        for (int w = kUnitsCycle - kD; w < kUnitsCycle; ++w)
            reduce(t0, (cnt - kCycle + w / NB) / kU, w / NB, w % NB, w % kSets);
    };

    if (t_begin < t_end) fetch(t_begin, lds0, ldn0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    // stages alternate between the two arrays; each half of the loop body names its arrays
    // statically
    for (int t0 = t_begin; t0 < t_end; t0 += 2 * S) {
        {
            if (t0 + S < t_end) fetch(t0 + S, lds1, ldn1);
            run_stage(lds0, ldn0, t0, t_end - t0 < S ? t_end - t0 : S);      // uniform
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
        const int t1 = t0 + S;
        if (t1 < t_end) {
            if (t1 + S < t_end) fetch(t1 + S, lds0, ldn0);
            run_stage(lds1, ldn1, t1, t_end - t1 < S ? t_end - t1 : S);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
    }

    // records: partials[p * k_pad + j], so that the 32 lanes of a half wave write 256
    // consecutive bytes
    const int col = lane & 31, hw = lane >> 5;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int64_t jpos = (int64_t)(gtile0 + nb) * 32 + col;
        // the two largest of two (largest, second largest) pairs
        auto join = [](int &b1, int &b2, int c1, int c2) {
            const int hi = max(b1, c1), lo = min(b1, c1);
            b2 = max(max(b2, c2), lo);
            b1 = hi;
        };
        if (per_half == 1) {          // all residue classes in one record
            int b1 = best[nb][0], b2 = second[nb][0];
#pragma unroll
            for (int r = 1; r < kResidues; ++r) join(b1, b2, best[nb][r], second[nb][r]);
            partials[rec_at(split * 2 + hw, jpos, nsplit * 2, k_pad)] = make_int2(b1, b2);
        } else if (per_half == 2) {   // classes r and r + 2 share a record
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                int b1 = best[nb][r], b2 = second[nb][r];
                join(b1, b2, best[nb][r + 2], second[nb][r + 2]);
                partials[rec_at((split * 2 + hw) * 2 + r, jpos, nsplit * 4, k_pad)] = make_int2(b1, b2);
            }
        } else {
#pragma unroll
            for (int r = 0; r < kResidues; ++r)
                partials[rec_at((split * 2 + hw) * kResidues + r, jpos, nsplit * 2 * kResidues, k_pad)] =
                    make_int2(best[nb][r], second[nb][r]);
        }
    }
    if (items <= gridDim.x) break;          // one item per block: nothing to fetch
    __syncthreads();                        // every wave is done with the LDS stages
    if (threadIdx.x == 0) s_item = gridDim.x + atomicAdd(next_item, 1u);
    __syncthreads();
    item = s_item;                          // uniform over the block
    }
}

}  // namespace
#include "pv_cells.h"
namespace {

// ---------------------------------------------------------------- exact re-rank

struct cand_t {
    double obj;
    int idx;
};

__device__ __forceinline__ bool cand_better(double o1, int i1, double o2, int i2)
{
    return o1 < o2 || (o1 == o2 && i1 < i2);
}

template <int G>
__device__ __forceinline__ double exact_obj(const float *__restrict__ cw, float s, const float *t)
{
    const pv_f4 *c4 = reinterpret_cast<const pv_f4 *>(cw);
    double obj = 0.0;
#pragma unroll
    for (int v4 = 0; v4 < G / 4; ++v4) {
        pv_f4 c = c4[v4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double acc = (double)c[e];
            // s * c is exact in double (two 24-bit factors): the fused form rounds exactly
            // like the product followed by the subtraction
            double r = fma((double)s, acc, -(double)t[v4 * 4 + e]);
            obj = obj + r * r;
        }
    }
    return obj;
}

// The same for 16 dimensions, one a lane of a row of 16 that works on one codeword together: the lane's square, then
// the sum in the order of the dimensions, every lane adding the same numbers.  A lane that takes all dimensions
// alone keeps its team waiting for 80 instructions a codeword, this is 35 and a load of 64 bytes; and the best needs no search
// over the team.  Many groups of 16 are bound by instructions issued (60 % of the re-rank's cycles, at the clock that the
// matrix product before it leaves): 35.0 -> 29.3 M wave instructions, 119 -> 110 us on 183 500 groups, 65 536 codewords.
__device__ __forceinline__ double exact_obj_row(const float *__restrict__ cw, float s, float t, int q)
{
    const double r = fma((double)s, (double)cw[q], -(double)t);
    return pv_row_sum_in_order(r * r, std::make_integer_sequence<int, 16>{});
}

// largest value a key can stand for: the super-unit bits replaced by ones; a negative key
// (every value behind it negative) is bounded by zero
__device__ __forceinline__ float key_upper(int key)
{
    return key < 0 ? 0.0f : __int_as_float(key | (int)kKeyMask);
}

// || c_hi - x_hi ||^2 of one table position as || x_hi ||^2 + || c_hi ||^2 - <2 c_hi, x_hi>: the
// product straight from the fp16 operands the matrix cores saw, two terms per instruction
// (v_dot2c_f32_f16, fp32 accumulate), the codeword's norm from the operand row (g = 8: its
// three pieces) or from the table k_prep keeps in position order (g = 16).  The three terms
// cancel, so the error is absolute: (G + 4) 2^-24 (|| c_hi || + || x_hi ||)^2 bounds the
// roundings of the two norms, of the G / 2 accumulation steps and of the final sum; kDdAbs
// times that square covers it eight times over.  The value is only ever compared from below
// (value - bound <= reach), so a generous bound costs a few needless exact evaluations.
constexpr float kDdAbs = 1.0e-5f;
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
// what it reads of a codeword: g = 8: operand row and the row with the norm; g = 16: the two operand rows, the norm aside
struct row_t {
    h8 a, b;
    float cc;
};
template <int G>
__device__ __forceinline__ row_t row_of(const h8 *__restrict__ A, const float *__restrict__ cnorm, int tile, int row, int pos)
{
    const h8 *at = A + (int64_t)tile * 64 + row;
    return row_t{at[0], at[32], G == 8 ? 0.0f : cnorm[pos]};
}
template <int G, bool CELLS = false>
__device__ __forceinline__ float dd_of(const row_t &r, const h8 (&xq)[G / 8], float xx)
{
    float dot = 0.0f;
#pragma unroll
    for (int h = 0; h < G / 8; ++h) {
        const h8 a = h ? r.b : r.a;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const h2 av = {a[2 * e], a[2 * e + 1]};
            const h2 xv = {xq[h][2 * e], xq[h][2 * e + 1]};
            dot = __builtin_amdgcn_fdot2(av, xv, dot, false);
        }
    }
    float cc = r.cc;
    if (G == 8) {
        cc = ((float)r.b[0] + (float)r.b[1]) + (float)r.b[2];
        if (CELLS && cc > 0.8f * kPadNorm) return __builtin_huge_valf();   // a padding row
    }
    return fmaxf((xx + cc) - dot, 0.0f);
}
template <int G, bool CELLS = false>
__device__ __forceinline__ float approx_dd(const h8 *__restrict__ A, const float *__restrict__ cnorm,
                                           int tile, int row, int pos, const h8 (&xq)[G / 8], float xx)
{
    return dd_of<G, CELLS>(row_of<G>(A, cnorm, tile, row, pos), xq, xx);
}

// A group the team could not decide alone: the partitions whose codewords must all be
// evaluated (bit p = partition p), and the best candidate found so far.
struct open_rec_t {
    double obj;
    float reach2;              // a codeword can reach obj only if ||c_hi - x_hi||^2 <= reach2
    unsigned long long mask;
    int idx;
    int n;
    int j;                     // position in the list (names the group's fp16 operand)
};

// A team of kTeam lanes per selected group; a lane scores 16 / kTeam positions of each half tile
// behind a key.  Groups
// with a partition left open are finished by the whole block afterwards, one at a time: for
// every position of the open partitions || c_hi - x_hi ||^2 is formed from the fp16 operands
// the matrix cores saw and the codewords that can still reach the best objective found are
// evaluated.  Every block leaves its counters in block_counts (summed by
// whoever asks for the call's statistics) and passes its changed codes on through atomics; no
// block waits for another and none publishes plain stores to another (a device-wide release
// costs a write-back of the whole L2 of the block's die).
#ifndef PV_RR_OCC
#define PV_RR_OCC 4   // waves per SIMD that the register budget of the re-rank kernel must allow (g = 16: 149 -> 128 registers, four waves instead of three; five would spill, but where a lane holds one dimension)
#endif
// v_sqrt_f32 and v_rcp_f32 as they are (1 ulp each; the library's sqrtf and the division add a
// dozen instructions apiece to round correctly and to scale denormal arguments).  Every use
// multiplies the result by a margin far above the few ulps that leaves open; a vanishing or
// denormal scale gives an infinite reciprocal, with which nothing is excluded.
__device__ __forceinline__ float fast_sqrt(float v) { return __builtin_amdgcn_sqrtf(v); }
__device__ __forceinline__ float fast_rcp(float v) { return __builtin_amdgcn_rcpf(v); }
// an upper bound of a non-negative double as a float: rounding to nearest is off by at most
// 2^-24 of the value, the factor makes up for that; below the smallest normal float the floor
// applied before the root takes over
__device__ __forceinline__ float float_above(double v) { return (float)v * 1.0000002f; }

// The certificate, the same in every kernel that decides from keys.  A codeword reaches the objective e only if
// || c_hi - x_hi ||^2 <= (P sqrt(e) / |s| + dC + dx)^2, of which this is an upper bound in fp32, every rounding covered.
__device__ __forceinline__ float reach2_of(double e, float p_over_s, float dC, float dx)
{
    const float ef = float_above(e);
    // (a NaN passes the floor and the root, and is caught below)
    const float rr = fast_sqrt(ef < 1.2e-38f ? 1.2e-38f : ef) * p_over_s * 1.000002f + dC + dx;
    const float r2 = rr * rr * 1.000002f;
    return r2 == r2 ? r2 : __builtin_huge_valf();   // NaN: nothing can be excluded
}
// Such a codeword, if it was not evaluated, sits behind a key whose upper bound is at least `at`: a lower bound of
// SHIFT + ||x_hi||^2 - reach2 - E1 (meta: x_meta's, fp32, every rounding covered).
struct key_cut {
    float at;
    bool none;                                      // also for NaN: nothing can be excluded
    __device__ __forceinline__ key_cut(const pv_f4 &meta, float reach2)
    {
        const float base = meta.x + meta.y;
        at = (base * 0.999999f - reach2 * 1.000001f) - meta.z - 1.0e-6f * (base + reach2);
        none = !(at > -3.0e38f);
    }
    __device__ __forceinline__ bool open(int key) const { return none || key_upper(key) >= at; }
};
// best of a team; all its lanes get it
template <int TEAM>
__device__ __forceinline__ cand_t cand_team_min(cand_t c)
{
    pv_team_stages<TEAM>([&](auto ctrl) {
        constexpr int C = decltype(ctrl)::value;
        const double o = pv_dpp_f64<C>(c.obj);
        const int i = pv_dpp<C>(c.idx);
        if (cand_better(o, i, c.obj, c.idx)) {
            c.obj = o;
            c.idx = i;
        }
    });
    return c;
}

// WIDE from two rounds of blocks on, where the instructions issued count; below, the chain of one block does, which the
// sums over a row make longer.  Kernels of a search, a lane a codeword / WIDE, 14 bits: 7 864 groups 48.3 / 48.8 us, 16 252
// 57.2 / 56.1, 32 505 76.0 / 76.0, 65 536 111.4 / 109.1; 16 bits: 32 505 115.7 / 115.5, 183 500 524 / 512; 12 bits: 183 500
// 153 / 143.
constexpr int64_t kWideFrom = 32768;
// A row of lanes a codeword pays only where few codewords need their exact objective: with more than kRowMost lanes of a
// team in need, each takes its own.  Whole searches with a lane a codeword throughout / the row throughout / as it is.  12 bits,
// 52 428 groups: 30 % of the codewords zero 405 / 1737 / 405 us, one codeword 100 times the others 167 / 252 / 167, targets
// far from every codeword 136 / 187 / 131, ordinary ones 76.9 / 73.3 / 72.7; 16 bits, 183 500 ordinary ones 519 / 507 / 507.
// (Two lanes one after the other: 177 with the one large codeword.)
constexpr int kRowMost = 1;
template <int G, bool CELLS, bool WIDE = false>
__global__ __launch_bounds__(kBlock, WIDE ? 5 : PV_RR_OCC) void k_rerank(
    const float *__restrict__ x_stage, const float *__restrict__ codebook, int k, int k_pad,
    const int2 *__restrict__ partials, int P, int per_half, int ncyc, int nsplit,
    const int *__restrict__ su_bounds, const float *__restrict__ dense, int dense_P, int dense_per_half,
    const float *__restrict__ x_meta, const unsigned *__restrict__ cb_meta, const h8 *__restrict__ A,
    const float *__restrict__ cnorm, const h8 *__restrict__ X, const uint16_t *__restrict__ perm,
    uint16_t *__restrict__ codes,
    unsigned *__restrict__ block_counts, unsigned long long *__restrict__ change_slots,
    unsigned long long *__restrict__ num_changed, int nbits)
{
    constexpr int kTeam = rerank_team(G);          // lanes per group
    constexpr int kTeams = kBlock / kTeam;         // groups per block
    constexpr int kPer = 16 / kTeam;               // positions of a half tile per lane
    constexpr bool kWide = WIDE && G == 16 && kTeam == 16; // a lane a dimension, the team takes one objective together
    static_assert(kTeam == 8 || kTeam == 16, "a team is 8 or 16 consecutive lanes");
    __shared__ unsigned s_cnt[4];   // groups decided by the teams, codes changed, candidates evaluated, groups scanned
    __shared__ open_rec_t s_open[kTeams];
    __shared__ float s_tgt[kWide ? kTeams : 1][G];  // the block's targets, for a lane that takes a codeword alone
    __shared__ unsigned s_nopen;
    if (threadIdx.x < 4) s_cnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) s_nopen = 0;
    __syncthreads();
    if (CELLS && *dense != 0.0f) {           // the dense contraction filled the records, in its own partitions
        P = dense_P;
        per_half = dense_per_half;
    }
    const int csize = 1 << nbits;
    const int gid = blockIdx.x * kBlock + threadIdx.x;
    const int j = gid / kTeam, q = gid % kTeam;
    // everything the team needs of its group sits at the list position: one round of loads
    const bool inlist = j < k;
    const pv_f4 *stage = reinterpret_cast<const pv_f4 *>(x_stage + (int64_t)(inlist ? j : 0) * (G + 4));
    const pv_f4 tail = stage[G / 4];
    pv_f4 meta = reinterpret_cast<const pv_f4 *>(x_meta)[inlist ? j : 0];
    const int n = inlist ? __float_as_int(tail.z) : -1;
    bool live = n >= 0;                      // whole teams agree on every branch below
    if (!live) meta.w = -1.0f;
    if constexpr (kWide) s_tgt[threadIdx.x / kTeam][q] = reinterpret_cast<const float *>(stage)[q];
    if (live && meta.w < 0.0f) {             // the filter was skipped for this group: every partition
        if (q == 0) {
            open_rec_t r;
            r.obj = __builtin_huge_val();
            r.reach2 = __builtin_huge_valf();      // no operand to test against: every codeword
            r.mask = P >= 64 ? ~0ull : ((1ull << P) - 1ull);
            r.idx = 0x7fffffff;
            r.n = n;
            r.j = j;
            s_open[atomicAdd(&s_nopen, 1u)] = r;
        }
        live = false;
    }
    if (live) {
        const float s = tail.x;
        float t[kWide ? 1 : G];
        if constexpr (kWide) {
            t[0] = reinterpret_cast<const float *>(stage)[q];
        } else {
#pragma unroll
            for (int v4 = 0; v4 < G / 4; ++v4) {
                pv_f4 v = stage[v4];
                t[v4 * 4 + 0] = v.x;
                t[v4 * 4 + 1] = v.y;
                t[v4 * 4 + 2] = v.z;
                t[v4 * 4 + 3] = v.w;
            }
        }
        // of one codeword for the whole team (kWide), else of each lane's own
        auto objective = [&](int cw) {
            if constexpr (kWide) return exact_obj_row(codebook + (int64_t)cw * G, s, t[0], q);
            else return exact_obj<G>(codebook + (int64_t)cw * G, s, t);
        };
        const int prev = __float_as_int(tail.y);
        constexpr int kMaxRec = 64 / kTeam;  // P <= 64
        int2 rec[kMaxRec];
#pragma unroll
        for (int u = 0; u < kMaxRec; ++u) {
            int p = q + kTeam * u;
            rec[u] = p < P ? partials[rec_at(p, j, P, k_pad)] : make_int2(kNoKey, kNoKey);
        }
        const double o_prev = objective(prev);
        // best key over all partitions, with its partition
        long long bk = (long long)0x8000000000000000ull;
#pragma unroll
        for (int u = 0; u < kMaxRec; ++u) {
            int p = q + kTeam * u;
            long long v = ((long long)rec[u].x << 32) | (long long)(unsigned)(63 - p);
            bk = v > bk ? v : bk;
        }
        bk = pv_team_max_i64<kTeam>(bk);
        const int best_key = (int)(bk >> 32);
        const int best_p = 63 - (int)(bk & 0xFFFFFFFFll);

        // the group's fp16 operand as the matrix cores saw it
        h8 xq[G / 8];
        {
            const int gt = j >> 5, col = j & 31;
#pragma unroll
            for (int h = 0; h < G / 8; ++h) xq[h] = X[((int64_t)gt * 2 + h) * 32 + col];
        }
        bool okP;
        const float Pscale = scale_from_maxabs(cb_meta[0], &okP);
        // what the cheap distance may be off by, at most (see approx_dd)
        const float nsum = Pscale * fast_sqrt(__uint_as_float(cb_meta[5])) * 1.0001f + kNormMargin +
                           fast_sqrt(meta.y) * 1.0001f;
        const float dabs = kDdAbs * nsum * nsum;
        const float dC = fast_sqrt(__uint_as_float(cb_meta[2])) * 1.0001f + 1e-30f;
        const float p_over_s = Pscale * fast_rcp(fabsf(s));   // inf for a vanishing scale: nothing is excluded then
        // The 16 U positions behind a key (lane q takes positions q, q + kTeam, ... of each of the
        // U half tiles) are looked at in two levels: || c_hi - x_hi ||^2 from the fp16 operand rows (cheap,
        // consecutive rows), and the exact objective only for positions that can still reach
        // the best objective known: || c_hi - x_hi || <= P sqrt(E) / |s| + dC + dx.
        constexpr int kMine = kU * kPer;               // positions of a key per lane
        auto level1 = [&](int key, int p, float (&dd)[kMine], int (&pos)[kMine], int (&cwd)[kMine]) {
            const int su = key & (int)kKeyMask;
            const int hw = (p / per_half) & 1;
#pragma unroll
            for (int uu = 0; uu < kU; ++uu)
#pragma unroll
                for (int e = 0; e < kPer; ++e) {
                    const int qq = q + kTeam * e;
                    const int row = 8 * (qq >> 2) + 4 * hw + (qq & 3);
                    pos[uu * kPer + e] = ((su * 2 + hw) * kU + uu) * 16 + qq;
                    // unconditional (the padded table has the row), so that the loads of all the
                    // lane's positions are in flight together
                    dd[uu * kPer + e] = approx_dd<G, CELLS>(A, cnorm, su * kU + uu, row, pos[uu * kPer + e], xq, meta.y);
                    // the codeword behind the position comes along (g = 8: positions are
                    // codewords), so that an exact evaluation is one more round trip, not two
                    cwd[uu * kPer + e] = G == 8 && !CELLS ? pos[uu * kPer + e] : (int)perm[pos[uu * kPer + e]];
                }
#pragma unroll
            for (int i = 0; i < kMine; ++i)
                if (!CELLS && pos[i] >= csize) dd[i] = __builtin_huge_valf();
        };
        auto exact_at = [&](int cw, cand_t &c) {
            const double o = objective(cw);
            if (cand_better(o, cw, c.obj, c.idx)) {
                c.obj = o;
                c.idx = cw;
            }
        };
        // Exact objectives of every lane's positions in `todo`.  kWide: those of up to kRowMost lanes one after the other for
        // the team, those of more by each lane alone, which then has a best of its own.
        unsigned exact_evals = 1;                      // the previous code
        bool alike = kWide;                            // the lanes of the team hold the same best
        const int team_shift = (threadIdx.x & 63) & ~(kTeam - 1);
        auto exact_of = [&](unsigned todo, const int (&cwd)[kMine], cand_t &c) {
            if constexpr (kWide) {
                unsigned team = (unsigned)((__ballot(todo != 0) >> team_shift) & ((1ull << kTeam) - 1ull));
                if (__builtin_expect(__popc(team) > kRowMost, 0)) {
                    exact_evals += pv_team_sum_u32<kTeam>((unsigned)__popc(todo));
#pragma unroll
                    for (int uu = 0; uu < kMine; ++uu)
                        if ((todo >> uu) & 1u) {
                            const double o = exact_obj<G>(codebook + (int64_t)cwd[uu] * G, s, s_tgt[threadIdx.x / kTeam]);
                            if (cand_better(o, cwd[uu], c.obj, c.idx)) {
                                c.obj = o;
                                c.idx = cwd[uu];
                            }
                        }
                    alike = false;
                    return;
                }
                while (team) {
                    int cw = cwd[kMine - 1];
#pragma unroll
                    for (int uu = kMine - 1; uu-- > 0;) cw = (todo >> uu) & 1u ? cwd[uu] : cw;
                    const int src = __ffs((int)team) - 1;
                    exact_at(__shfl(cw, src, kTeam), c);
                    if (q == src) todo &= todo - 1u;
                    ++exact_evals;
                    team = (unsigned)((__ballot(todo != 0) >> team_shift) & ((1ull << kTeam) - 1ull));
                }
            } else {
#pragma unroll
                for (int uu = 0; uu < kMine; ++uu)
                    if ((todo >> uu) & 1u) {
                        exact_at(cwd[uu], c);
                        ++exact_evals;
                    }
            }
        };
        auto reach2 = [&](double e) { return reach2_of(e, p_over_s, dC, meta.w); };

        cand_t mine;
        mine.obj = __builtin_huge_val();
        mine.idx = 0x7fffffff;
        double e_star = o_prev;
        if (best_key != kNoKey) {
            float dd[kMine];
            int pos[kMine], cwd[kMine];
            level1(best_key, best_p, dd, pos, cwd);
            // the position that looks nearest is evaluated first: it fixes the reach for the rest
            int wu = 0;
            float dmin = dd[0];
#pragma unroll
            for (int uu = 1; uu < kMine; ++uu)
                if (dd[uu] < dmin) {
                    dmin = dd[uu];
                    wu = uu;
                }
            int pw = cwd[0];                       // cwd[wu] without dynamic register indexing
#pragma unroll
            for (int uu = 1; uu < kMine; ++uu)
                if (uu == wu) pw = cwd[uu];
            unsigned long long pick = ((unsigned long long)__float_as_uint(dmin) << 32) | (kWide ? ((unsigned)pw << 4) | q : (unsigned)q);
            pick = pv_team_min_u64<kTeam>(pick);
            const bool chosen = (int)(pick & 15u) == q && dmin < 3.0e38f;
            double o0;
            if constexpr (kWide) {
                const bool any = __uint_as_float((unsigned)(pick >> 32)) < 3.0e38f;      // the same in the whole team
                if (any) {
                    exact_at((int)((unsigned)pick >> 4), mine);
                    ++exact_evals;
                }
                o0 = mine.obj;
            } else {
                if (chosen) {
                    exact_at(pw, mine);
                    ++exact_evals;
                }
                o0 = __shfl(mine.obj, (int)(pick & 15u), kTeam);
            }
            if (o0 < e_star) e_star = o0;
            const float r2f = reach2(e_star);
            unsigned todo = 0;
#pragma unroll
            for (int uu = 0; uu < kMine; ++uu)
                if (!(chosen && uu == wu) && dd[uu] - dabs <= r2f && dd[uu] < 3.0e38f) todo |= 1u << uu;
            exact_of(todo, cwd, mine);
        }
        cand_t first = alike ? mine : cand_team_min<kTeam>(mine);
        if (first.obj < e_star) e_star = first.obj;

        // what was not evaluated and could still reach E*
        const float reach2f = reach2(e_star);
        const key_cut cut(meta, reach2f);
        unsigned pending = 0;                         // bit u: rec[u].x needs evaluation
        unsigned long long open = 0;                  // partitions with a second key at or above the cut
#pragma unroll
        for (int u = 0; u < kMaxRec; ++u) {
            int p = q + kTeam * u;
            if (p < P) {
                if (rec[u].y != kNoKey && cut.open(rec[u].y)) open |= 1ull << p;
                if (p != best_p && rec[u].x != kNoKey && cut.open(rec[u].x)) pending |= 1u << u;
            }
        }
        open = pv_team_or_u64<kTeam>(open);
        // the best key of every other partition at or above the cut: its positions are evaluated here
        for (;;) {
            const unsigned long long pb = __ballot(pending != 0);
            const unsigned team = (unsigned)((pb >> team_shift) & ((1ull << kTeam) - 1ull));
            if (!team) break;
            const int src = __ffs(team) - 1;      // lane of the team with work
            const unsigned their = __shfl(pending, src, kTeam);
            const int u = __ffs(their) - 1;
            int key = 0;
#pragma unroll
            for (int uu = 0; uu < kMaxRec; ++uu)
                if (uu == u) key = rec[uu].x;
            key = __shfl(key, src, kTeam);
            {
                float dd[kMine];
                int pos[kMine], cwd[kMine];
                level1(key, src + kTeam * u, dd, pos, cwd);
                unsigned todo = 0;
#pragma unroll
                for (int uu = 0; uu < kMine; ++uu)
                    if (dd[uu] - dabs <= reach2f && dd[uu] < 3.0e38f) todo |= 1u << uu;
                exact_of(todo, cwd, mine);
            }
            if (q == src) pending &= ~(1u << u);
        }
        if (!kWide) exact_evals = pv_team_sum_u32<kTeam>(exact_evals);
        const cand_t win = alike ? mine : cand_team_min<kTeam>(mine);
        if (q == 0) {
            if (open) {
                // a partition may hide further codewords at or above the cut: all of its
                // positions are evaluated by the block, which also takes the decision
                open_rec_t r;
                r.obj = win.obj;
                r.reach2 = cut.none ? __builtin_huge_valf() : reach2(o_prev < win.obj ? o_prev : win.obj);
                r.mask = open;
                r.idx = win.idx;
                r.n = n;
                r.j = j;
                s_open[atomicAdd(&s_nopen, 1u)] = r;
            } else {
                int pick = win.idx;
                if (o_prev <= win.obj || pick == 0x7fffffff) pick = prev;
                if (pick != prev) {
                    codes[n] = (uint16_t)pick;
                    atomicAdd(&s_cnt[1], 1u);
                }
                atomicAdd(&s_cnt[0], 1u);
            }
            atomicAdd(&s_cnt[2], exact_evals - (kWide ? 0u : (unsigned)(kTeam - 1)));   // the previous code was counted by every lane
        }
    }
    __syncthreads();

    // ---- groups left open: every position of their open partitions, by the whole block, one
    // group at a time.
    // Partition p = (codeword split, half wave, residue class) as the scoring kernel numbers them.
    const unsigned nopen = s_nopen;
    __shared__ double s_obj[kBlock / 64];
    __shared__ int s_idx[kBlock / 64];
    for (unsigned item = 0; item < nopen; ++item) {
        const open_rec_t &rec = s_open[item];
        const pv_f4 *stage2 = reinterpret_cast<const pv_f4 *>(x_stage + (int64_t)rec.j * (G + 4));
        const pv_f4 tail2 = stage2[G / 4];
        const float s = tail2.x;
        const int prev = __float_as_int(tail2.y);
        const int lane = threadIdx.x & 63;
        const int qq = threadIdx.x & 15, slot = threadIdx.x >> 4;
        // kWide: the targets are read from LDS for each exact objective, they are registers that spill
        float own[kWide ? 1 : G];
        if constexpr (!kWide) {
#pragma unroll
            for (int v4 = 0; v4 < G / 4; ++v4) {
                pv_f4 v = stage2[v4];
                own[v4 * 4 + 0] = v.x;
                own[v4 * 4 + 1] = v.y;
                own[v4 * 4 + 2] = v.z;
                own[v4 * 4 + 3] = v.w;
            }
        }
        const int team_of = kWide ? rec.j - (int)blockIdx.x * kTeams : 0;
        auto exact = [&](int cw) {
            if constexpr (kWide) {
                int at = team_of;
                asm volatile("" : "+v"(at));             // (else the targets are kept over the loop)
                return exact_obj<G>(codebook + (int64_t)cw * G, s, s_tgt[at]);
            } else {
                return exact_obj<G>(codebook + (int64_t)cw * G, s, own);
            }
        };
        constexpr int kSlots = kBlock / 16;
        // the group's fp16 operand as the matrix cores saw it
        h8 xq[G / 8];
        {
            const int gt = rec.j >> 5, col = rec.j & 31;
#pragma unroll
            for (int h = 0; h < G / 8; ++h) xq[h] = X[((int64_t)gt * 2 + h) * 32 + col];
        }
        const float xx = x_meta[(int64_t)rec.j * 4 + 1];
        bool okP2;
        const float nsum = scale_from_maxabs(cb_meta[0], &okP2) * fast_sqrt(__uint_as_float(cb_meta[5])) * 1.0001f +
                           kNormMargin + fast_sqrt(xx) * 1.0001f;
        const float dabs = kDdAbs * nsum * nsum;
        const bool test = rec.reach2 < 3.0e38f;
        const float r2f = rec.reach2;
        cand_t mine;
        mine.obj = __builtin_huge_val();
        mine.idx = 0x7fffffff;
        for (unsigned long long left = rec.mask; left; left &= left - 1) {   // uniform over the block
            const int p = __ffsll((long long)left) - 1;
            const int hw = (p / per_half) & 1;
            const int split = p / (2 * per_half);
            const int su_begin = CELLS ? su_bounds[split] : split_begin(split, ncyc, nsplit) * kResidues;
            const int su_end = CELLS ? su_bounds[split + 1] : su_begin + split_count(split, ncyc, nsplit) * kResidues;
            const int row = 8 * (qq >> 2) + 4 * hw + (qq & 3);
            // the classes of the record: p % per_half, + per_half, ... (relative to the split's
            // start); kBatch super-units per lane at a time, so that their operand rows are in
            // flight together
            constexpr int kBatch = 2;
            for (int rel0 = (p % per_half) + slot * per_half; su_begin + rel0 < su_end;
                 rel0 += kSlots * per_half * kBatch) {
                float dd[kBatch][kU];
#pragma unroll
                for (int bb = 0; bb < kBatch; ++bb) {
                    // unconditional loads (a row of the split's last super-unit stands in past its
                    // end), so that the whole batch is in flight together
                    const int su = su_begin + rel0 + bb * kSlots * per_half;
                    const int su_c = su < su_end ? su : su_end - 1;
#pragma unroll
                    for (int uu = 0; uu < kU; ++uu)
                        dd[bb][uu] = approx_dd<G, CELLS>(A, cnorm, su_c * kU + uu, row,
                                                  ((su_c * 2 + hw) * kU + uu) * 16 + qq, xq, xx);
                }
#pragma unroll
                for (int bb = 0; bb < kBatch; ++bb) {
                    const int su = su_begin + rel0 + bb * kSlots * per_half;
#pragma unroll
                    for (int uu = 0; uu < kU; ++uu) {
                        const int pos = ((su * 2 + hw) * kU + uu) * 16 + qq;
                        if (su < su_end && (CELLS ? dd[bb][uu] < 3.0e38f : pos < csize) &&
                            (!test || dd[bb][uu] - dabs <= r2f)) {
                            const int cw = G == 8 && !CELLS ? pos : (int)perm[pos];
                            const double obj = exact(cw);
                            if (cand_better(obj, cw, mine.obj, mine.idx)) {
                                mine.obj = obj;
                                mine.idx = cw;
                            }
                        }
                    }
                }
            }
        }
        // block-wide lexicographic minimum
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            double o = __shfl_xor(mine.obj, off);
            int i = __shfl_xor(mine.idx, off);
            if (cand_better(o, i, mine.obj, mine.idx)) {
                mine.obj = o;
                mine.idx = i;
            }
        }
        __syncthreads();
        if (lane == 0) {
            s_obj[threadIdx.x >> 6] = mine.obj;
            s_idx[threadIdx.x >> 6] = mine.idx;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            cand_t win;
            win.obj = rec.obj;
            win.idx = rec.idx;
            for (int w = 0; w < kBlock / 64; ++w)
                if (cand_better(s_obj[w], s_idx[w], win.obj, win.idx)) {
                    win.obj = s_obj[w];
                    win.idx = s_idx[w];
                }
            const double o_prev = exact(prev);
            int pick = win.idx;
            if (o_prev <= win.obj || pick == 0x7fffffff) pick = prev;
            if (pick != prev) {
                codes[rec.n] = (uint16_t)pick;
                atomicAdd(&s_cnt[1], 1u);
            }
            atomicAdd(&s_cnt[3], 1u);
        }
    }
    __syncthreads();
    // per-block totals: groups decided by the teams, codes changed, candidates evaluated, groups scanned
    if (threadIdx.x < 4) block_counts[4 * blockIdx.x + threadIdx.x] = s_cnt[threadIdx.x];
    // *num_changed: thousands of atomics on one address would queue for longer than the kernel
    // runs, so 64 blocks share a slot that carries (arrivals << 40 | sum); the block that finds
    // all others arrived passes the sum on
    if (threadIdx.x == 0 && num_changed) {
        const unsigned first = (blockIdx.x >> 6) << 6;
        const unsigned members = gridDim.x - first < 64u ? gridDim.x - first : 64u;
        const unsigned long long old =
            atomicAdd(&change_slots[(blockIdx.x >> 6) * kSlotStride], (1ull << 40) | (unsigned long long)s_cnt[1]);
        if ((unsigned)(old >> 40) == members - 1u) {
            const unsigned long long total = (old & ((1ull << 40) - 1ull)) + s_cnt[1];
            if (total) atomicAdd(num_changed, total);
        }
    }
}

}  // namespace
#include "pv_smallcb.h"
namespace {

// ------------------------------------------------ stochastic rounding over the two nearest
//
// The same filter serves App. F's rounding over the TWO nearest codewords: the certificate is
// the one of k_rerank with the best objective replaced by the second best found so far, E2.
// A codeword that was not evaluated can belong to the two nearest only if its objective
// reaches E2, hence only if its key is at least the cut taken from E2; every best key at or
// above that cut has its 16 U positions looked at (cheap distance first, exact objective for
// those within reach of E2), and a partition whose runner-up key reaches the cut is scanned
// completely by a wave.  The two nearest (objective, then index) go to pv_round_pick.
struct two_t {
    double o1, o2;
    int i1, i2;
};

__device__ __forceinline__ void two_clear(two_t &b)
{
    b.o1 = b.o2 = __builtin_huge_val();
    b.i1 = b.i2 = kPvNoCode;
}

__device__ __forceinline__ void two_insert(two_t &b, double o, int c)
{
    if (cand_better(o, c, b.o1, b.i1)) {
        b.o2 = b.o1; b.i2 = b.i1;
        b.o1 = o; b.i1 = c;
    } else if (cand_better(o, c, b.o2, b.i2)) {
        b.o2 = o; b.i2 = c;
    }
}

// the two smallest of the union of two such pairs (a codeword sits in at most one of them)
__device__ __forceinline__ two_t two_merge(two_t a, const two_t &b)
{
    if (b.i1 != kPvNoCode) two_insert(a, b.o1, b.i1);
    if (b.i2 != kPvNoCode) two_insert(a, b.o2, b.i2);
    return a;
}

// The same over a team; all its lanes get the result.
template <int TEAM>
__device__ __forceinline__ two_t two_team(two_t b)
{
    pv_team_stages<TEAM>([&](auto ctrl) {
        constexpr int C = decltype(ctrl)::value;
        two_t o;
        o.o1 = pv_dpp_f64<C>(b.o1);
        o.o2 = pv_dpp_f64<C>(b.o2);
        o.i1 = pv_dpp<C>(b.i1);
        o.i2 = pv_dpp<C>(b.i2);
        b = two_merge(b, o);
    });
    return b;
}

template <int G>
struct open2_t {
    two_t best;
    unsigned long long mask;
    float reach2, s, xx, dabs;
    int n, prev;
    float t[G];
    h8 xq[G / 8];
};

template <int G>
__global__ __launch_bounds__(kBlock, PV_RR_OCC) void k_round_top2(
    const float *__restrict__ x_stage, const float *__restrict__ codebook, int k, int k_pad,
    const int2 *__restrict__ partials, int P, int per_half, int ncyc, int nsplit,
    const float *__restrict__ x_meta, const unsigned *__restrict__ cb_meta, const h8 *__restrict__ A,
    const float *__restrict__ cnorm, const h8 *__restrict__ X, const uint16_t *__restrict__ perm,
    uint16_t *__restrict__ codes, unsigned *__restrict__ block_counts,
    unsigned long long *__restrict__ change_slots, unsigned long long *__restrict__ num_changed,
    int nbits, int power, unsigned long long seed)
{
    constexpr int kTeam = rerank_team(G);
    constexpr int kTeams = kBlock / kTeam;
    constexpr int kPer = 16 / kTeam;
    __shared__ unsigned s_cnt[4];   // groups decided by the teams, codes changed, candidates evaluated, groups scanned
    __shared__ open2_t<G> s_open[kTeams];
    __shared__ unsigned s_nopen;
    if (threadIdx.x < 4) s_cnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) s_nopen = 0;
    __syncthreads();
    const int csize = 1 << nbits;
    const int gid = blockIdx.x * kBlock + threadIdx.x;
    const int j = gid / kTeam, q = gid % kTeam;
    const bool inlist = j < k;
    const pv_f4 *stage = reinterpret_cast<const pv_f4 *>(x_stage + (int64_t)(inlist ? j : 0) * (G + 4));
    const pv_f4 tail = stage[G / 4];
    pv_f4 meta = reinterpret_cast<const pv_f4 *>(x_meta)[inlist ? j : 0];
    const int n = inlist ? __float_as_int(tail.z) : -1;
    bool live = n >= 0;                      // whole teams agree on every branch below
    if (!live) meta.w = -1.0f;
    bool okP;
    const float Pscale = scale_from_maxabs(cb_meta[0], &okP);
    const float cmaxn = Pscale * fast_sqrt(__uint_as_float(cb_meta[5])) * 1.0001f + kNormMargin;
    auto decide = [&](const two_t &b, int group, int prev) {
        int pick = prev;                     // nothing could be evaluated (non-finite input): keep
        if (b.i1 != kPvNoCode) pick = pv_round_pick(b.o1, b.i1, b.o2, b.i2, power, seed, (unsigned long long)group);
        if (pick != prev) {
            codes[group] = (uint16_t)pick;
            atomicAdd(&s_cnt[1], 1u);
        }
    };
    const float s = tail.x;
    const int prev = __float_as_int(tail.y);
    float t[G];
#pragma unroll
    for (int v4 = 0; v4 < G / 4; ++v4) {
        const pv_f4 v = stage[v4];
        t[v4 * 4 + 0] = v.x;
        t[v4 * 4 + 1] = v.y;
        t[v4 * 4 + 2] = v.z;
        t[v4 * 4 + 3] = v.w;
    }
    h8 xq[G / 8];
    {
        const int gt = (inlist ? j : 0) >> 5, col = (inlist ? j : 0) & 31;
#pragma unroll
        for (int h = 0; h < G / 8; ++h) xq[h] = X[((int64_t)gt * 2 + h) * 32 + col];
    }
    const float nsum = cmaxn + fast_sqrt(meta.y) * 1.0001f;
    const float dabs = kDdAbs * nsum * nsum;
    // one lane hands the group over for a look at all the positions of the partitions in `mask`
    auto leave_open = [&](const two_t &best, float reach2, unsigned long long mask) {
        open2_t<G> &r = s_open[atomicAdd(&s_nopen, 1u)];
        r.best = best;
        r.mask = mask;
        r.reach2 = reach2;
        r.s = s;
        r.xx = meta.y;
        r.dabs = dabs;
        r.n = n;
        r.prev = prev;
#pragma unroll
        for (int e = 0; e < G; ++e) r.t[e] = t[e];
#pragma unroll
        for (int h = 0; h < G / 8; ++h) r.xq[h] = xq[h];
    };
    if (live && meta.w < 0.0f) {             // the filter was skipped for this group: every partition
        if (q == 0) {
            two_t none;
            two_clear(none);
            leave_open(none, __builtin_huge_valf(), P >= 64 ? ~0ull : ((1ull << P) - 1ull));
        }
        live = false;
    }
    if (live) {
        constexpr int kMaxRec = 64 / kTeam;  // P <= 64
        int2 rec[kMaxRec];
#pragma unroll
        for (int u = 0; u < kMaxRec; ++u) {
            int p = q + kTeam * u;
            rec[u] = p < P ? partials[rec_at(p, j, P, k_pad)] : make_int2(kNoKey, kNoKey);
        }
        // the two largest keys over all partitions, runner-up keys included: entry = key, partition,
        // whether it is the partition's best (low bit) - the largest key is always a best one
        auto entry = [](int key, int p, int is_best) {
            return ((long long)key << 32) | (long long)(unsigned)(((63 - p) << 1) | is_best);
        };
        long long bk = (long long)0x8000000000000000ull;
#pragma unroll
        for (int u = 0; u < kMaxRec; ++u) {
            const long long v = entry(rec[u].x, q + kTeam * u, 1);
            bk = v > bk ? v : bk;
        }
        bk = pv_team_max_i64<kTeam>(bk);
        long long bk2 = (long long)0x8000000000000000ull;
#pragma unroll
        for (int u = 0; u < kMaxRec; ++u) {
            const long long vx = entry(rec[u].x, q + kTeam * u, 1), vy = entry(rec[u].y, q + kTeam * u, 0);
            if (vx != bk && vx > bk2) bk2 = vx;
            if (vy > bk2) bk2 = vy;
        }
        bk2 = pv_team_max_i64<kTeam>(bk2);
        const int best_key = (int)(bk >> 32);
        const int best_p = 63 - (int)((bk & 0xFFFFFFFFll) >> 1);
        const int next_key = (int)(bk2 >> 32);
        const int next_p = 63 - (int)((bk2 & 0xFFFFFFFFll) >> 1);
        const bool next_is_best = (bk2 & 1ll) != 0;      // the best key of its partition (else its runner-up)
        const float p_over_s = Pscale * fast_rcp(fabsf(s));
        const float dC = fast_sqrt(__uint_as_float(cb_meta[2])) * 1.0001f + 1e-30f;
        auto reach2_at = [&](double e) { return reach2_of(e, p_over_s, dC, meta.w); };
        two_t mine;
        two_clear(mine);
        unsigned exact_evals = 0;
        // A lane has kMine positions of a key: half tile e / kPer, row q + kTeam (e % kPer) there.
        constexpr int kMine = kU * kPer;
        auto first_pos = [&](int key, int p) {
            return (((key & (int)kKeyMask) * 2 + ((p / per_half) & 1)) * kU) * 16 + q;
        };
        auto pos_of = [&](int first, int i) { return first + (i / kPer) * 16 + (i % kPer) * kTeam; };
        // their cheap distances, all loads under way together; the result has a bit for each that is a codeword
        auto level1 = [&](int first, auto &dd) {
            const int su = first / (32 * kU), hw = (first / (16 * kU)) & 1;
            unsigned ok = 0;
#pragma unroll
            for (int i = 0; i < kMine; ++i) {
                const int qq = q + kTeam * (i % kPer);
                const int pos = pos_of(first, i);
                dd[i] = approx_dd<G>(A, cnorm, su * kU + i / kPer, 8 * (qq >> 2) + 4 * hw + (qq & 3), pos, xq, meta.y);
                if (pos < csize) ok |= 1u << i;
            }
            return ok;
        };
        // exact objectives of the positions in `todo`: bits [0, kMine) from position `a` on, the next kMine from `b` on
        auto evaluate = [&](unsigned todo, int a, int b) {
            while (todo) {
                const int i = __ffs((int)todo) - 1;
                todo &= todo - 1u;
                const int pos = i < kMine ? pos_of(a, i) : pos_of(b, i - kMine);
                const int cw = G == 8 ? pos : (int)perm[pos];
                two_insert(mine, exact_obj<G>(codebook + (int64_t)cw * G, s, t), cw);
                ++exact_evals;
            }
        };
        // The second nearest usually sits behind the second largest key, not among the neighbours of the nearest: both
        // keys' positions are looked at together.  The two that look nearest are evaluated first, and fix the reach for
        // the others: 2.0 exact objectives a group instead of 34 (every position behind the largest key, then those of
        // the second within reach), the kernel 33.0 -> 29.3 us on 20 971 groups of 8, 65 536 codewords.
        two_t first;
        {
            const bool has_a = best_key != kNoKey, has_b = next_key != kNoKey && next_p < P;
            const int a = has_a ? first_pos(best_key, best_p) : q, b = has_b ? first_pos(next_key, next_p) : q;
            float da[kMine], db[kMine];
            unsigned oka = level1(a, da), okb = level1(b, db);
            if (!has_a) oka = 0;
            if (!has_b) okb = 0;
            const unsigned ok = oka | (okb << kMine);
            float d1 = __builtin_huge_valf(), d2 = d1;
#pragma unroll
            for (int i = 0; i < 2 * kMine; ++i) {
                const float d = (ok >> i) & 1u ? (i < kMine ? da[i % kMine] : db[i % kMine]) : __builtin_huge_valf();
                d2 = fminf(d2, fmaxf(d1, d));
                d1 = fminf(d1, d);
            }
            pv_team_stages<kTeam>([&](auto ctrl) {
                constexpr int C = decltype(ctrl)::value;
                const float o1 = __int_as_float(pv_dpp<C>(__float_as_int(d1)));
                const float o2 = __int_as_float(pv_dpp<C>(__float_as_int(d2)));
                d2 = fminf(fmaxf(d1, o1), fminf(d2, o2));
                d1 = fminf(d1, o1);
            });
            unsigned todo = 0;
#pragma unroll
            for (int i = 0; i < 2 * kMine; ++i)
                if ((i < kMine ? da[i % kMine] : db[i % kMine]) <= d2) todo |= 1u << i;
            todo &= ok;
            evaluate(todo, a, b);
            first = two_team<kTeam>(mine);
            const float reach2 = first.i2 == kPvNoCode ? __builtin_huge_valf() : reach2_at(first.o2);
            unsigned more = 0;
#pragma unroll
            for (int i = 0; i < 2 * kMine; ++i)
                if ((i < kMine ? da[i % kMine] : db[i % kMine]) - dabs <= reach2) more |= 1u << i;
            more &= ok & ~todo;
            if (__ballot(more != 0)) {
                evaluate(more, a, b);
                first = two_team<kTeam>(mine);
            }
        }
        // what was not evaluated and could still reach E2
        const float reach2f = first.i2 == kPvNoCode ? __builtin_huge_valf() : reach2_at(first.o2);
        const key_cut cut(meta, reach2f);
        unsigned pending = 0;
        unsigned long long open = 0;
#pragma unroll
        for (int u = 0; u < kMaxRec; ++u) {
            int p = q + kTeam * u;
            if (p < P) {
                if (rec[u].y != kNoKey && cut.open(rec[u].y)) open |= 1ull << p;
                if (p != best_p && !(next_is_best && p == next_p) && rec[u].x != kNoKey && cut.open(rec[u].x))
                    pending |= 1u << u;
            }
        }
        open = pv_team_or_u64<kTeam>(open);
        const int team_shift = (threadIdx.x & 63) & ~(kTeam - 1);
        for (;;) {
            const unsigned long long pb = __ballot(pending != 0);
            const unsigned team = (unsigned)((pb >> team_shift) & ((1ull << kTeam) - 1ull));
            if (!team) break;
            const int src = __ffs(team) - 1;
            const unsigned their = __shfl(pending, src, kTeam);
            const int u = __ffs(their) - 1;
            int key = 0;
#pragma unroll
            for (int uu = 0; uu < kMaxRec; ++uu)
                if (uu == u) key = rec[uu].x;
            key = __shfl(key, src, kTeam);
            {
                float dd[kMine];
                const int a = first_pos(key, src + kTeam * u);
                const unsigned ok = level1(a, dd);
                unsigned todo = 0;
#pragma unroll
                for (int i = 0; i < kMine; ++i)
                    if (dd[i] - dabs <= reach2f) todo |= 1u << i;
                evaluate(todo & ok, a, a);
            }
            if (q == src) pending &= ~(1u << u);
        }
        exact_evals = pv_team_sum_u32<kTeam>(exact_evals);
        const two_t win = two_team<kTeam>(mine);
        if (q == 0) {
            if (open) {
                leave_open(win, (cut.none || win.i2 == kPvNoCode) ? __builtin_huge_valf() : reach2_at(win.o2), open);
            } else {
                decide(win, n, prev);
                atomicAdd(&s_cnt[0], 1u);
            }
            atomicAdd(&s_cnt[2], exact_evals);
        }
    }
    __syncthreads();

    // ---- groups left open: every position of their open partitions, a wave a group, one or two groups all the waves.
    // One group in 45 is left open, in half of the blocks none, in the fullest five: one after the other by the whole
    // block, which read the group again for each, the kernel took 29.3 us; so, with the group handed over in LDS,
    // 23.3.  (One wave for the only group too: a short list of groups of 16, 65 536 codewords, 5 us slower.)
    const unsigned nopen = s_nopen;
    __shared__ two_t s_two[kBlock / 64];
    const unsigned wave = threadIdx.x >> 6;
    const unsigned share = nopen == 1u ? kBlock / 64 : nopen == 2u ? kBlock / 128 : 1u;      // waves a group
    auto finish = [&](const open2_t<G> &rec, two_t win, const two_t *o, unsigned parts) {
        // a codeword of an open partition may already sit in the team's pair (it was behind an
        // evaluated key): the same index is not taken twice
        const int t1 = win.i1, t2 = win.i2;
        for (unsigned w = 0; w < parts; ++w) {
            if (o[w].i1 != kPvNoCode && o[w].i1 != t1 && o[w].i1 != t2) two_insert(win, o[w].o1, o[w].i1);
            if (o[w].i2 != kPvNoCode && o[w].i2 != t1 && o[w].i2 != t2) two_insert(win, o[w].o2, o[w].i2);
        }
        decide(win, rec.n, rec.prev);
        atomicAdd(&s_cnt[3], 1u);
    };
    for (unsigned item = wave / share; item < nopen; item += (kBlock / 64) / share) {
        const open2_t<G> &rec = s_open[item];
        const float xx = rec.xx, cut = rec.dabs, r2f = rec.reach2;
        h8 xo[G / 8];
#pragma unroll
        for (int h = 0; h < G / 8; ++h) xo[h] = rec.xq[h];
        const int lane = threadIdx.x & 63;
        const int qq = lane & 15, slot = (int)(wave % share) * 4 + (lane >> 4);
        const bool test = r2f < 3.0e38f;
        two_t mine;
        two_clear(mine);
        for (unsigned long long left = rec.mask; left; left &= left - 1) {   // uniform over the wave
            const int p = __ffsll((long long)left) - 1;
            const int hw = (p / per_half) & 1;
            const int split = p / (2 * per_half);
            const int su_begin = split_begin(split, ncyc, nsplit) * kResidues;
            const int su_end = su_begin + split_count(split, ncyc, nsplit) * kResidues;
            const int row = 8 * (qq >> 2) + 4 * hw + (qq & 3);
            constexpr int kBatch = G == 8 ? 4 : 2;
            // A lane's super-units: su0, su0 + step, ..; up to kPass of them are looked at before the exact objectives.  (Those are
            // all: make_plan leaves a partition 64 super-units at most.)
            constexpr int kPass = 32 / kU;
            const int step = 4 * (int)share * per_half;
            for (int su0 = su_begin + (p % per_half) + slot * per_half; su0 < su_end; su0 += kPass * step) {
                unsigned todo = 0;
                for (int c = 0; c < kPass && su0 + c * step < su_end; c += kBatch) {
                    // unconditional loads (a row of the split's last super-unit stands in past its end), all of a
                    // lane's batch on their way before the first is looked at
                    row_t rows[kBatch][kU];
#pragma unroll
                    for (int bb = 0; bb < kBatch; ++bb) {
                        const int su = su0 + (c + bb) * step;
                        const int su_c = su < su_end ? su : su_end - 1;
#pragma unroll
                        for (int uu = 0; uu < kU; ++uu)
                            rows[bb][uu] = row_of<G>(A, cnorm, su_c * kU + uu, row, ((su_c * 2 + hw) * kU + uu) * 16 + qq);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    unsigned bits = 0;
#pragma unroll
                    for (int bb = 0; bb < kBatch; ++bb) {
                        const int su = su0 + (c + bb) * step;
#pragma unroll
                        for (int uu = 0; uu < kU; ++uu) {
                            const float dd = dd_of<G>(rows[bb][uu], xo, xx);
                            const bool in = (su < su_end) & (((su * 2 + hw) * kU + uu) * 16 + qq < csize) &
                                            (!test | (dd - cut <= r2f));
                            bits |= (unsigned)in << (bb * kU + uu);
                        }
                    }
                    todo |= bits << (c * kU);
                }
                while (todo) {
                    const int i = __ffs((int)todo) - 1;
                    todo &= todo - 1u;
                    const int pos = (((su0 + (i / kU) * step) * 2 + hw) * kU + i % kU) * 16 + qq;
                    const int cw = G == 8 ? pos : (int)perm[pos];
                    two_insert(mine, exact_obj<G>(codebook + (int64_t)cw * G, rec.s, rec.t), cw);
                }
            }
        }
        two_t o = two_team<16>(mine);
#pragma unroll
        for (int m = 16; m < 64; m <<= 1) {
            two_t other;
            other.o1 = __shfl_xor(o.o1, m);
            other.o2 = __shfl_xor(o.o2, m);
            other.i1 = __shfl_xor(o.i1, m);
            other.i2 = __shfl_xor(o.i2, m);
            o = two_merge(o, other);
        }
        if (lane == 0) {
            s_two[wave] = o;
            if (share == 1u) finish(rec, rec.best, s_two + wave, 1u);
        }
    }
    if (share > 1u) {                        // the same in the whole block: every group had its waves at once
        __syncthreads();
        if ((threadIdx.x & 63) == 0 && wave % share == 0u && wave / share < nopen)
            finish(s_open[wave / share], s_open[wave / share].best, s_two + wave, share);
    }
    __syncthreads();
    if (threadIdx.x < 4) block_counts[4 * blockIdx.x + threadIdx.x] = s_cnt[threadIdx.x];
    // *num_changed through the slots 64 blocks share (see k_rerank)
    if (threadIdx.x == 0 && num_changed) {
        const unsigned first = (blockIdx.x >> 6) << 6;
        const unsigned members = gridDim.x - first < 64u ? gridDim.x - first : 64u;
        const unsigned long long old =
            atomicAdd(&change_slots[(blockIdx.x >> 6) * kSlotStride], (1ull << 40) | (unsigned long long)s_cnt[1]);
        if ((unsigned)(old >> 40) == members - 1u) {
            const unsigned long long total = (old & ((1ull << 40) - 1ull)) + s_cnt[1];
            if (total) atomicAdd(num_changed, total);
        }
    }
}

struct plan_t {
    int NB, k_pad, gblocks, nsplit, P, per_half, ntiles, ncyc, nsu, cpad;
};

plan_t make_plan(const pv_layout *l, int64_t k, bool two_nearest)
{
    plan_t p;
    p.ntiles = (1 << l->nbits) / 32;
    constexpr int cycle = kResidues * kU;    // tiles per residue cycle
    p.ncyc = (p.ntiles + cycle - 1) / cycle; // whole cycles: the table is padded with zero rows
    p.nsu = p.ncyc * kResidues;
    p.cpad = p.nsu * kU * 32;
    p.NB = k >= 4096 ? PV_NBX : 1;
    const int per_block = PV_WAVES * p.NB * 32;
    p.gblocks = (int)((k + per_block - 1) / per_block);
    p.k_pad = p.gblocks * per_block;
    // PV_OCC blocks per compute unit fit (registers, LDS).  Few group blocks: cut the
    // codeword range so that the items fill those slots in ONE round (a 13th split that
    // spills 21 blocks into a second round costs 25 %).  Many group blocks: several short
    // items per slot, handed out dynamically, so the tail is one short item - two to four of
    // them, and a power of two of splits: the splits then cover equal numbers of residue cycles,
    // and the re-rank reads 32 records a group instead of 48 (14336 x 4096 at g = 16, 183 500
    // groups: 4 splits against 6 leave the scoring as it is and take 10 us off the re-rank;
    // 3 and 5 splits cost the scoring 25 to 37 us).
    const int slots = 256 * PV_OCC;
    int want = slots / p.gblocks;
    // The rounding over the two nearest codewords keeps the finer cut (4 items a slot) at g = 8: its
    // cut comes from the second best objective, more keys reach it, and with 32 records a group
    // twice as many groups are left open.  Whole calls, finer / power of two: g = 8, 16 bits, 146 800 groups 363 / 379 us,
    // 73 400 203 / 206, 14 bits, 146 800 170 / 168; g = 16, where the records are what the rounding waits for, 183 500
    // groups, 12 bits 300 / 274, 14 bits 336 / 312, 16 bits 588 / 594 and, far from every codeword, 680 / 660.
    if (want < 4 && two_nearest && l->group_size == 8) want = (4 * slots + p.gblocks - 1) / p.gblocks;
    if (want < 4) {
        const int least = (2 * slots + p.gblocks - 1) / p.gblocks;
        want = 4;
        while (want < least) want *= 2;
    }
    if (want > 8 && slots / p.gblocks < 4) want = 8;
    int max_split = p.nsu * kU / 8;
    if (max_split > p.ncyc) max_split = p.ncyc;
    if (max_split < 1) max_split = 1;
    if (want > max_split) want = max_split;
    if (want > 32) want = 32;
    if (want < 1) want = 1;
    p.nsplit = want;
    // as many residue classes apart as 64 records per group allow: the more partitions, the
    // fewer groups have two keys above the cut in one of them
    p.per_half = kResidues;
    while (p.per_half > 1 && p.nsplit * 2 * p.per_half > 64) p.per_half >>= 1;
    p.P = p.nsplit * 2 * p.per_half;
    return p;
}

// Nothing but matrix instructions: four independent accumulators per wave, four waves per
// SIMD over the whole chip (the matrix-core ceiling of the box at its current clock).
constexpr int kProbeBlocks = 256 * 4;
__global__ __launch_bounds__(kBlock, 4) void k_probe_mfma(float *__restrict__ sink, int64_t iters)
{
    const int lane = threadIdx.x & 63;
    h8 a, b;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        a[e] = (_Float16)(0.001f * (float)(lane + e));
        b[e] = (_Float16)(0.5f + 0.01f * (float)e);
    }
    f16v acc[4];
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[n][r] = 0.0f;
    for (int64_t it = 0; it + 4 <= iters; it += 4) {
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, acc[n], 0, 0, 0);
    }
    if (blockIdx.x < 256) {
        float s = 0.0f;
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) s += acc[n][r];
        sink[((int64_t)blockIdx.x * 16 + (threadIdx.x >> 6)) * 64 + lane] = s;
    }
}

}  // namespace

pv_status pv_launch_probe_mfma(pv_ctx *ctx, int64_t iters, float *sink, int64_t *waves_out)
{
    pv_timed t(ctx, PV_K_PROBE_MFMA);
    hipLaunchKernelGGL(k_probe_mfma, dim3(kProbeBlocks), dim3(kBlock), 0, ctx->stream, sink, iters);
    PV_HIP(ctx, hipGetLastError());
    if (waves_out) *waves_out = (int64_t)kProbeBlocks * (kBlock / 64);
    return PV_OK;
}

bool pv_mfma_supported(const pv_layout *l)
{
    return l->num_codebooks == 1 && (l->group_size == 8 || l->group_size == 16) && l->nbits >= 5;
}

pv_status pv_launch_mfma_search(pv_ctx *ctx, const pv_layout *l, const float *T,
                                const float *codebooks, const float *scales,
                                const int32_t *group_idx, int64_t k, uint16_t *codes,
                                int64_t *num_changed, int32_t power, uint64_t seed)
{
    if (power == 0 && small_codebook(l, k))
        return pv_launch_search_small(ctx, l, T, codebooks, scales, group_idx, k, codes, num_changed);
    plan_t p = make_plan(l, k, power > 0);
    const plan_t dense = p;      // with cells: the plan of the dense contraction, should it be needed
    // Cells (pv_cells.h): g = 8, the nearest codeword, work enough to pay for cutting the codebook.
    const int cbits = l->nbits - kCellLog;
    const bool cells = l->group_size == 8 && power == 0 && l->nbits >= kCellMinBits &&
                       (k << l->nbits) >= kCellMinWork;
    int cell_waves = 8;
    if (cells) {
        const int ncells = 1 << cbits;
        p.cpad = ((1 << l->nbits) + ncells * (kCellPos - 1) + kCellPos - 1) / kCellPos * kCellPos;
        // Waves per block and number of splits (ranges of runs of 16 cells, at most kItemCells cells
        // each): the pair with the least work on the fullest compute unit.  An item costs its groups x
        // its runs, and something besides for each and for itself.  Few splits where that is even: the
        // re-rank reads four records for each.
        const int runs = ncells / 16, least = (ncells + kItemCells - 1) / kItemCells;
        double most = 1e30;
        for (int n = least; n <= 16 && n <= runs; ++n)
            for (int w = kCellWavesMax; w >= 4; --w) {
                const int gb = (int)((k + w * 64 - 1) / (w * 64));
                const int rounds = (gb * n + 255) / 256, most_runs = (runs + n - 1) / n;
                const double work = rounds * ((w + 3.0) * (most_runs + 0.5));
                if (work < most * 0.98) {
                    most = work;
                    p.nsplit = n;
                    cell_waves = w;
                }
            }
        p.gblocks = (int)((k + cell_waves * 64 - 1) / (cell_waves * 64));
        // (the dense contraction takes 512 groups at a time: a list this long has two group tiles a wave)
        p.k_pad = (p.gblocks * cell_waves * 64 + 511) & ~511;
        p.per_half = 2;
        p.P = p.nsplit * 4;
    }
    const int g = l->group_size;
    const int csize = 1 << l->nbits;
    const int gpr = (int)(l->in_features / g);
    const int N = (int)pv_num_groups(l);
    const int nsu_alloc = 2 * p.nsu + 64;    // two norms per super-unit; the scoring kernel stages 64 at a time
    pv_status st;
    // All scratch is one block (each new one costs the first call of a context about 10 us):
    //   bucket counts, cells' counts (zero between calls: cleared once) | the rest of their tables
    //   codebook operand, position -> codeword, norm buckets, bounds of the splits, smallest norm per
    //   super-unit, g = 16: norm per position
    //   groups' operands, bounds, staged targets / scale / code / id, squared reach
    //   records | counters
    size_t used = 0;
    auto take = [&](size_t bytes) {
        const size_t at = used;
        used = (used + bytes + 255) & ~(size_t)255;
        return at;
    };
    const int rr_blocks = (int)((k * rerank_team(l->group_size) + kBlock - 1) / kBlock);
    const int nslots = (rr_blocks + 63) / 64;
    const size_t count_off = take((size_t)kCbCopies * (kNormBins / 2) * 4);
    const size_t cell_count_off = take((size_t)kCbCopies * kCellsMax * 4);
    const size_t zero_head = used;
    const size_t cb_off = take((kCbWords + 8) * 4), cells_off = take(kCellWords * 4);
    const size_t a_off = take((size_t)p.cpad * 32), perm_off = take((size_t)p.cpad * 2);
    const size_t bucket_off = take((size_t)csize * 2), bounds_off = take(256);
    const size_t nmin_off = take((size_t)nsu_alloc * 4), cnorm_off = take((size_t)p.cpad * 4);
    const size_t x_off = take((size_t)p.k_pad * 32), x_meta_off = take((size_t)p.k_pad * 16);
    const size_t stage_off = take((size_t)p.k_pad * (g + 4) * 4), reach_off = take(cells ? (size_t)p.k_pad * 4 : 0);
    const size_t partials_off = take((size_t)p.k_pad * (p.P > dense.P ? p.P : dense.P) * sizeof(int2));
    const size_t fb_off = take(64), rr_off = take((size_t)rr_blocks * 16), slots_off = take((size_t)nslots * kSlotStride * 8);
    if ((st = pv_ensure(ctx, ctx->search, used, zero_head)) != PV_OK) return st;
    char *base = static_cast<char *>(ctx->search.ptr);
    unsigned *rr_counts = reinterpret_cast<unsigned *>(base + rr_off);
    unsigned long long *change_slots = reinterpret_cast<unsigned long long *>(base + slots_off);
    h8 *A = reinterpret_cast<h8 *>(base + a_off);
    uint16_t *perm = reinterpret_cast<uint16_t *>(base + perm_off);
    uint16_t *bucket = reinterpret_cast<uint16_t *>(base + bucket_off);
    float *nmin = reinterpret_cast<float *>(base + nmin_off);
    float *cnorm = reinterpret_cast<float *>(base + cnorm_off);
    h8 *X = reinterpret_cast<h8 *>(base + x_off);
    cb_mem mem;
    mem.part = reinterpret_cast<pv_f4 *>(base + cb_off);
    mem.dpart = reinterpret_cast<float *>(mem.part + kCbParts);
    mem.anchor = mem.dpart + kCbParts;
    mem.cursor = reinterpret_cast<unsigned *>(mem.anchor + 16);
    mem.count = reinterpret_cast<unsigned *>(base + count_off);
    unsigned *cb_meta = mem.cursor + kCbCopies * (kNormBins / 2);
    float *x_meta = reinterpret_cast<float *>(base + x_meta_off);
    float *x_stage = reinterpret_cast<float *>(base + stage_off);
    int2 *partials = reinterpret_cast<int2 *>(base + partials_off);
    unsigned *fb_count = reinterpret_cast<unsigned *>(base + fb_off);          // 4 counters
    unsigned long long *stats = static_cast<unsigned long long *>(ctx->stats.ptr);
    auto nc = reinterpret_cast<unsigned long long *>(num_changed);
    hipStream_t sm = ctx->stream;
    group_args ga;
    ga.T = T;
    ga.scales = scales;
    ga.codebook = codebooks;
    ga.group_idx = group_idx;
    ga.codes = codes;
    ga.k = (int)k;
    ga.k_pad = p.k_pad;
    ga.gpr = gpr;
    ga.N = N;
    ga.csize_mask = csize - 1;
    ga.X = X;
    ga.x_meta = x_meta;
    ga.x_stage = x_stage;
    ga.reach = reinterpret_cast<float *>(base + reach_off);      // cells only
    ctx->rr_blocks_last = rr_blocks;
    ctx->rr_counts = rr_counts;
    clear_args ca;
    ca.stats = stats;
    ca.num_changed = nc;
    ca.change_slots = change_slots;
    ca.fb_count = fb_count;
    ca.nslots = nslots;
    if (cells) {
        const int cb_blocks = csize / kCbChunk;
        unsigned *meta = cb_meta;
        int *su_bounds = reinterpret_cast<int *>(base + bounds_off);
        cell_mem cm;
        cm.part = reinterpret_cast<pv_f4 *>(base + cells_off);
        cm.dpart = reinterpret_cast<float *>(cm.part + kCbParts);
        cm.theta = cm.dpart + kCbParts;
        cm.count = reinterpret_cast<unsigned *>(base + cell_count_off);
        cm.cursor = reinterpret_cast<unsigned *>(cm.theta + 16);
        cm.cell_su = reinterpret_cast<int *>(cm.cursor + kCbCopies * kCellsMax);
        cm.cell_of = reinterpret_cast<uint16_t *>(cm.cell_su + kCellsMax + 8);
        {
            pv_timed t(ctx, PV_K_PREP);
            hipLaunchKernelGGL(k_cells_stats, dim3(cb_blocks + 1), dim3(kBlock), 0, sm, codebooks, csize, cbits, cm,
                               ca, ga);
            hipLaunchKernelGGL(k_cells_prep, dim3(cb_blocks + (p.k_pad + kBlock - 1) / kBlock), dim3(kBlock), 0, sm,
                               codebooks, csize, cbits, cb_blocks, cm, meta, A, perm, su_bounds, p.nsplit, dense.nsplit, ga);
        }
        {
            pv_timed t(ctx, PV_K_SCORE_MFMA);
            const int items = p.gblocks * p.nsplit;
            hipLaunchKernelGGL(k_cells_score, dim3(items < 256 ? items : 256), dim3(cell_waves * 64), 0, sm, A, X,
                               ga.reach, su_bounds, cm, meta, partials, cbits, cb_blocks, p.nsplit, p.gblocks,
                               p.k_pad, fb_count + 1);
            const int ditems = dense.gblocks * dense.nsplit;
            hipLaunchKernelGGL((k_score_mfma<8, PV_NBX>), dim3(ditems < 256 * PV_OCC ? ditems : 256 * PV_OCC),
                               dim3(PV_WAVES * 64), 0, sm, A, X, x_meta, (const float *)nullptr, partials,
                               dense.ncyc, dense.nsplit, dense.per_half, dense.gblocks, p.k_pad, fb_count + 2,
                               cm.theta + 15, cm.dpart, cb_blocks, cm.count, kCbCopies << cbits, meta);
        }
        {
            pv_timed t(ctx, PV_K_RERANK);
            hipLaunchKernelGGL((k_rerank<8, true>), dim3((unsigned)rr_blocks), dim3(kBlock), 0, sm, x_stage, codebooks,
                               (int)k, p.k_pad, partials, p.P, p.per_half, 0, p.nsplit, su_bounds, cm.theta + 15, dense.P,
                               dense.per_half, x_meta, meta, A,
                               cnorm, X, perm, codes, rr_counts, change_slots, nc, l->nbits);
        }
        PV_HIP(ctx, hipGetLastError());
        return PV_OK;
    }
    const int cb_blocks = (p.cpad + kCbChunk - 1) / kCbChunk;
    {
        pv_timed t(ctx, PV_K_PREP);
        const int x_blocks = (p.k_pad + kBlock - 1) / kBlock;
#define PV_PREP(G_, ONE_)                                                                                \
    do {                                                                                           \
        if (!ONE_)                                                                                 \
            hipLaunchKernelGGL(k_cb_stats<G_>, dim3(csize / kCbChunk), dim3(kBlock), 0, sm, codebooks, csize, mem, \
                               bucket, ca);                                                        \
        hipLaunchKernelGGL((k_prep<G_, ONE_>), dim3(cb_blocks + x_blocks), dim3(kBlock), 0, sm, codebooks, csize, p.cpad, \
                           cb_blocks, cb_meta, mem, A, perm, bucket, nmin, cnorm, ga, p.ncyc, p.nsplit, ca); \
    } while (0)
        if (csize <= kOneBlock) {
            if (g == 8) PV_PREP(8, true);
            else PV_PREP(16, true);
        } else {
            if (g == 8) PV_PREP(8, false);
            else PV_PREP(16, false);
        }
#undef PV_PREP
    }
    {
        pv_timed t(ctx, PV_K_SCORE_MFMA);
        const int items = p.gblocks * p.nsplit;
        dim3 grid(items < 256 * PV_OCC ? items : 256 * PV_OCC);
#define PV_SCORE(G_, NB_)                                                                          \
    hipLaunchKernelGGL((k_score_mfma<G_, NB_>), grid, dim3(PV_WAVES * 64), 0, sm, A, X, x_meta, nmin, \
                       partials, p.ncyc, p.nsplit, p.per_half, p.gblocks, p.k_pad, fb_count + 1, (const float *)nullptr, mem.dpart, \
                       cb_blocks, mem.count, G_ == 16 ? kCbCopies * (kNormBins / 2) : 0, cb_meta)
        if (g == 8) {
            if (p.NB == PV_NBX) PV_SCORE(8, PV_NBX);
            else PV_SCORE(8, 1);
        } else {
            if (p.NB == PV_NBX) PV_SCORE(16, PV_NBX);
            else PV_SCORE(16, 1);
        }
#undef PV_SCORE
    }
    {
        pv_timed t(ctx, PV_K_RERANK);
        const dim3 rgrid((unsigned)rr_blocks);
        if (power > 0) {
#define PV_ROUND2(G_)                                                                              \
    hipLaunchKernelGGL(k_round_top2<G_>, rgrid, dim3(kBlock), 0, sm, x_stage, codebooks, (int)k,    \
                       p.k_pad, partials, p.P, p.per_half, p.ncyc, p.nsplit, x_meta, cb_meta, A,    \
                       cnorm, X, perm, codes, rr_counts, change_slots, nc, l->nbits, (int)power,    \
                       (unsigned long long)seed)
            if (g == 8) PV_ROUND2(8);
            else PV_ROUND2(16);
#undef PV_ROUND2
        } else if (g == 8)
            hipLaunchKernelGGL((k_rerank<8, false>), rgrid, dim3(kBlock), 0, sm, x_stage, codebooks, (int)k,
                               p.k_pad, partials, p.P, p.per_half, p.ncyc, p.nsplit, (const int *)nullptr, (const float *)nullptr, 0, 0, x_meta,
                               cb_meta, A, cnorm, X, perm, codes, rr_counts, change_slots, nc, l->nbits);
        else if (k < kWideFrom)
            hipLaunchKernelGGL((k_rerank<16, false>), rgrid, dim3(kBlock), 0, sm, x_stage, codebooks, (int)k,
                               p.k_pad, partials, p.P, p.per_half, p.ncyc, p.nsplit, (const int *)nullptr, (const float *)nullptr, 0, 0, x_meta,
                               cb_meta, A, cnorm, X, perm, codes, rr_counts, change_slots, nc, l->nbits);
        else
            hipLaunchKernelGGL((k_rerank<16, false, true>), rgrid, dim3(kBlock), 0, sm, x_stage, codebooks, (int)k,
                               p.k_pad, partials, p.P, p.per_half, p.ncyc, p.nsplit, (const int *)nullptr, (const float *)nullptr, 0, 0, x_meta,
                               cb_meta, A, cnorm, X, perm, codes, rr_counts, change_slots, nc, l->nbits);
    }
    PV_HIP(ctx, hipGetLastError());
    return PV_OK;
}
