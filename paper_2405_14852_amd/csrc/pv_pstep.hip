// Gradients of the continuous parameters for the P step (Alg. 3, P step: "backprop";
// App. K: codebooks and per-channel scales): the chain rule through
//     W[o, j*g + i] = s_o * sum_m C_m[b(o,j,m), i]
// applied to G = d phi / d W:
//     d phi / d C_m[c, i] = sum over groups n = (o, j) with b(o,j,m) = c of  s_o * G[n, i]
//     d phi / d s_o       = sum_j sum_i G[o, j*g + i] * (C_0[b_0, i] + C_1[b_1, i] + ...)
//
// The codebook gradient is a scatter-add of N * g values into 2^B * g sums.  Floating-point
// atomics would serialise on popular codewords and give run-dependent roundings (and atomics
// on device memory are slow on a part whose L2 is split over several dies); instead the
// groups are SORTED by code with a stable radix sort written for this key width - 8 bits a
// pass, so at most two passes of histogram, prefix sum and scatter, with ranks taken from
// wave ballots and per-wave counters in LDS so that equal codes keep ascending group order
// and no atomic touches device memory - and every codeword's segment is summed by g
// lanes in that order, in double, with exact products: the same sum, in the same order, as a
// plain loop over the groups.  Segments longer than kLong groups are cut into pieces of kLong
// that are summed by the teams of one block and added in piece order (a different
// association from the plain loop: reproducible from run to run, but no longer the sequential
// rounding).  Small codebooks take another route (k_pg_small below), which takes the scale
// gradient along; otherwise that is one block-wide tree sum per row.
#include "pv_internal.h"
#include "pv_dpp.h"
#include "pv_radix.h"

namespace {

constexpr int kBlock = 256;
constexpr int kLong = 128;       // groups per piece: a segment up to this long is summed by one team alone
// the codes of codebook m as sort keys, masked to B bits
struct code_keys {
    const uint16_t *codes;
    int M, m;
    unsigned mask;
    __device__ __forceinline__ unsigned operator()(int64_t e) const
    {
        return (unsigned)(codes[e * M + m] & mask);
    }
};

// start[c] = first position of code c in the sorted order (= position of the next present
// code when c is absent); start[csize] = N.  Also clears the length of the list of long segments.
__global__ __launch_bounds__(kBlock) void k_pg_starts(const uint16_t *__restrict__ sorted, int64_t N,
                                                      int csize, int32_t *__restrict__ start,
                                                      unsigned *__restrict__ nlong)
{
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r == 0) *nlong = 0u;
    if (r >= N) return;
    const int cur = sorted[r];
    const int prev = r == 0 ? -1 : (int)sorted[r - 1];
    for (int c = prev + 1; c <= cur; ++c) start[c] = (int32_t)r;
    if (r == N - 1)
        for (int c = cur + 1; c <= csize; ++c) start[c] = (int32_t)N;
}

// Sum of s_o * G[n, i] over ids[a .. b) in that order, kInFlight gathers issued together.
constexpr int kInFlight = 8;
template <bool HAVE_SCALES, class IDS>
__device__ __forceinline__ double ordered_sum(IDS ids, const float *__restrict__ s_of,
                                              const float *__restrict__ G,
                                              const float *__restrict__ scales, int gpr, int g,
                                              int i, int a, int b, double acc = 0.0)
{
    for (int r0 = a; r0 < b; r0 += kInFlight) {
        float gv[kInFlight], sv[kInFlight];
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const int r = r0 + u < b ? r0 + u : b - 1;
            const int n = ids[r];
            gv[u] = G[(int64_t)n * g + i];
            sv[u] = HAVE_SCALES ? s_of[r] : scales[n / gpr];
        }
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const double next = acc + (double)sv[u] * (double)gv[u];
            acc = r0 + u < b ? next : acc;
        }
    }
    return acc;
}

// Segments of up to kLong groups: one team of TEAM lanes per codeword (TEAM = the group size
// rounded up to a power of two, at least 8).  The team stages the segment's ids and row
// scales in LDS, then lane i sums dimension i in segment order.  A longer segment is put on
// the list for k_pg_long.
template <int TEAM>
__global__ __launch_bounds__(kBlock) void k_pg_short(const int32_t *__restrict__ start,
                                                     const int32_t *__restrict__ order,
                                                     const float *__restrict__ G,
                                                     const float *__restrict__ scales, int gpr, int g,
                                                     int csize, int32_t *__restrict__ long_list,
                                                     unsigned *__restrict__ nlong,
                                                     float *__restrict__ out)
{
    constexpr int kTeams = kBlock / TEAM;
    __shared__ int s_id[kTeams][kLong];
    __shared__ float s_s[kTeams][kLong];
    const int team = threadIdx.x / TEAM, i = threadIdx.x % TEAM;
    const int c = blockIdx.x * kTeams + team;
    int lo = 0, len = 0;
    bool mine = false;
    if (c < csize) {
        lo = start[c];
        len = start[c + 1] - lo;
        mine = len <= kLong;
        if (!mine) {
            len = 0;
            if (i == 0) long_list[atomicAdd(nlong, 1u)] = c;
        }
    }
    for (int r = i; r < len; r += TEAM) s_id[team][r] = order[lo + r];
    __syncthreads();
    // the first kFirst gathers of G and the row scales of the whole segment are requested
    // together: a typical segment costs one round trip here, not one per few groups
    constexpr int kFirst = 32;
    float gv[kFirst];
    const int ii = i < g ? i : 0;
    if (len > 0) {
#pragma unroll
        for (int u = 0; u < kFirst; ++u)
            gv[u] = G[(int64_t)s_id[team][u < len ? u : len - 1] * g + ii];
    }
    for (int r = i; r < len; r += TEAM) s_s[team][r] = scales[s_id[team][r] / gpr];
    __syncthreads();
    if (mine && i < g) {
        double acc = 0.0;
        if (len > 0) {
#pragma unroll
            for (int u = 0; u < kFirst; ++u) {
                const double next = acc + (double)s_s[team][u < len ? u : len - 1] * (double)gv[u];
                acc = u < len ? next : acc;
            }
            if (len > kFirst)
                acc = ordered_sum<true>(s_id[team], s_s[team], G, scales, gpr, g, i, kFirst, len, acc);
        }
        out[(int64_t)c * g + i] = (float)acc;
    }
}

// Segments longer than kLong: one block per segment.  Its teams sum pieces of kLong ids in
// order (piece p of the segment that starts at sorted position lo keeps its sum in
// partial[lo / kLong + p], p >= 1: the ranges of different segments cannot meet; piece 0 stays
// in LDS), and the first g threads add the piece sums in piece order.
template <int TEAM>
__global__ __launch_bounds__(kBlock) void k_pg_long(const int32_t *__restrict__ long_list,
                                                    const unsigned *__restrict__ nlong,
                                                    const int32_t *__restrict__ start,
                                                    const int32_t *__restrict__ order,
                                                    const float *__restrict__ G,
                                                    const float *__restrict__ scales, int gpr, int g,
                                                    double *partial, float *__restrict__ out)
{
    constexpr int kTeams = kBlock / TEAM;
    __shared__ double s_first[64];
    const int team = threadIdx.x / TEAM, i = threadIdx.x % TEAM;
    const int count = (int)*nlong;
    for (int li = blockIdx.x; li < count; li += gridDim.x) {
        const int c = long_list[li];
        const int lo = start[c], len = start[c + 1] - lo;
        const int32_t *ids = order + lo;
        const int pieces = (len + kLong - 1) / kLong;
        double *mine = partial + (int64_t)(lo / kLong) * g;
        for (int p = team; p < pieces; p += kTeams) {
            const int a = p * kLong, b = a + kLong < len ? a + kLong : len;
            if (i < g) {
                const double acc = ordered_sum<false>(ids, nullptr, G, scales, gpr, g, i, a, b);
                if (p == 0) s_first[i] = acc;
                else mine[(int64_t)p * g + i] = acc;
            }
        }
        __syncthreads();
        if ((int)threadIdx.x < g) {
            double acc = s_first[threadIdx.x];
            int p = 1;
            for (; p + 4 <= pieces; p += 4) {          // four loads in flight, added in piece order
                double v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = mine[(int64_t)(p + u) * g + threadIdx.x];
#pragma unroll
                for (int u = 0; u < 4; ++u) acc = acc + v[u];
            }
            for (; p < pieces; ++p) acc = acc + mine[(int64_t)p * g + threadIdx.x];
            out[(int64_t)c * g + threadIdx.x] = (float)acc;
        }
        __syncthreads();
    }
}

// Small codebooks (all M * 2^B * g sums fit one block's LDS): every codeword is shared by
// thousands of groups, so sorting buys nothing.  One pass over G: every wave streams its own
// consecutive vectors, adds s_o * G into the block's LDS table with LDS atomics and, from the same
// registers, the products with the codewords for the scale gradient.
// To make the result independent of the order in which the atomics land, the table is kept in 64-bit
// FIXED POINT: every term is scaled by a power of two that leaves room for the number of terms
// one block can add, and rounded to an integer once; integer addition is associative, so a
// table is a function of the block's inputs only.  The unit comes from the block's FIRST vectors (16
// places spread over its range) instead of a pass of its own: the bound is the block's largest |scale|
// times its largest |G|, 2^ex, and a term keeps kbits = min(62 - headroom, 50) bits below it (48 for 2^14
// groups a block).  Up to twice 2^ex everything still fits 64 bits.  The sweep takes the true bound on
// its way: a block that met more looks for the vectors beyond the room, takes away what they added
// (wrapped integers, but the same ones again), shifts the table to the unit of the true bound, once, and adds them in that.
// 11008 x 4096: no block for bell-shaped gradients, one or two vectors in a third of the blocks for
// Student's t with three degrees of freedom.  Only where they are more than a short list holds or the
// first vectors were all zero the block sweeps its range again.  So no term is
// rounded more coarsely than with the unit of the whole matrix's bound.  The blocks' tables are
// added with the rounding errors carried along, and the total is rounded to fp32.  Gradients or
// scales that are not finite make every entry NaN.  A row's products are summed by the waves that
// meet it, lanes first, and added in order of the waves.
// 11008 x 4096, 2 x 8: vector-ALU issue fills 91 of the kernel's 141 thousand cycles (23.4 M instructions,
// much of it the conversion to integers), the LDS 60 (sixteen 64-bit atomics a group and codebook; 35 of
// them bank conflicts), reading G takes 75; none alone is the bound, their overlap is.  There, with the
// scale gradient (and the maxima) as a kernel of its own that read G first: 98.7 us a step, in one
// pass 73.  Gradients with heavy tails (cubed normal, Student's t): 82 and 86.  Ordering tiles of
// groups by code in LDS and summing in registers, without these atomics, was tried: 112 us, one
// block of 16 waves per compute unit waiting at its barriers.
constexpr int kSmallBlock = 1024;                         // one table serves sixteen waves
constexpr int kSmallWaves = kSmallBlock / 64;
constexpr int kSmallAhead = 2;                            // vectors of a thread in flight
constexpr unsigned kSmallOver = 512;                      // vectors beyond the unit's room that a block lists

struct small_mem {
    long long *partial;  // [blocks][entries]
    double *rows;        // [rows + waves] part of row r that wave w met, at r + w
    double *unit;        // [blocks] what one in `partial` stands for; NaN: some input was not finite
};

// x + 1.5 * 2^52 holds the integer nearest to x (ties to even) in its low mantissa bits for
// |x| < 2^51; the terms stay below 2^50
__device__ __forceinline__ unsigned long long fixed_point_term(double x)
{
    constexpr double kMagic = 6755399441055744.0;
    return (unsigned long long)(__double_as_longlong(x + kMagic) - __double_as_longlong(kMagic));
}

// sums and maxima over a wave through the lane-permute paths of the vector unit; uniform results
__device__ __forceinline__ double wave_lane_f64(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
__device__ __forceinline__ double wave_sum_f64(double v)
{
    pv_team_stages<16>([&](auto c) { v = v + pv_dpp_f64<decltype(c)::value>(v); });
    return (wave_lane_f64(v, 0) + wave_lane_f64(v, 16)) + (wave_lane_f64(v, 32) + wave_lane_f64(v, 48));
}
__device__ __forceinline__ unsigned wave_max_u32(unsigned v)
{
    pv_team_stages<16>([&](auto c) { v = max(v, (unsigned)pv_dpp<decltype(c)::value>((int)v)); });
    const unsigned a = __builtin_amdgcn_readlane((int)v, 0), b = __builtin_amdgcn_readlane((int)v, 16);
    const unsigned d = __builtin_amdgcn_readlane((int)v, 32), e = __builtin_amdgcn_readlane((int)v, 48);
    return max(max(a, b), max(d, e));
}

// largest |scale| times largest |G| of a block, from each wave's own (as bits: NaN > inf > every
// finite value); all threads call this, s_max is 2 * kSmallWaves unsigneds of LDS
__device__ __forceinline__ double block_bound(unsigned gb, unsigned sb, unsigned *s_max)
{
    gb = wave_max_u32(gb);
    sb = wave_max_u32(sb);
    __syncthreads();                                       // the last call's values were read
    if ((threadIdx.x & 63) == 0) {
        s_max[threadIdx.x >> 6] = gb;
        s_max[kSmallWaves + (threadIdx.x >> 6)] = sb;
    }
    __syncthreads();
    gb = sb = 0u;
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) {
        gb = max(gb, s_max[w]);
        sb = max(sb, s_max[kSmallWaves + w]);
    }
    return (double)__uint_as_float(sb) * (double)__uint_as_float(gb);
}

// VPG: 16-byte vectors per group when that is 1, 2 or 4 (a shift finds the group), else 0.
// ROWS: the scale gradient too (rows of at least 64 vectors).  A wave takes `per_wave` consecutive
// vectors, a multiple of 64 that begins with a group.
template <int VPG, bool ROWS>
__global__ __launch_bounds__(kSmallBlock, 8) void k_pg_small(
    const float *__restrict__ G, const uint16_t *__restrict__ codes, const float *__restrict__ codebooks,
    const float *__restrict__ scales, int64_t nvec, int per_wave, int g, int M, int nbits, int gpr,
    int out_features, int kbits, small_mem mem)
{
    extern __shared__ unsigned long long tab[];         // [M][2^B][g]
    __shared__ unsigned s_max[2 * kSmallWaves];
    __shared__ unsigned s_over, s_list[kSmallOver];     // places in the block's range
    const int csize = 1 << nbits;
    const unsigned mask = (unsigned)csize - 1u;
    const int entries = M * csize * g;
    const unsigned vpg = VPG > 0 ? (unsigned)VPG : (unsigned)(g / 4);   // 16-byte vectors per group
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kSmallWaves + (threadIdx.x >> 6)));
    const int64_t v_lo = (int64_t)wave * per_wave;
    const int64_t left = nvec - v_lo;
    const int len = left <= 0 ? 0 : left < per_wave ? (int)left : per_wave;
    // everything inside the wave's range is counted from its first group in 32 bits
    const int64_t n_lo = v_lo / vpg;
    const unsigned row0 = (unsigned)(n_lo / gpr), rem0 = (unsigned)(n_lo - (int64_t)row0 * gpr);
    const double inv_gpr = 1.0 / (double)gpr;
    // vectors of so many groups of a row, as a 32-bit number: a row beyond 2^30 vectors has no end in
    // the wave's range (per_wave is below 2^30: G would not fit the memory otherwise)
    auto row_vecs = [&](int groups) {
        const int64_t n = (int64_t)groups * vpg;
        return n < (1 << 30) ? (int)n : 1 << 30;
    };
    const pv_f4 *G4 = reinterpret_cast<const pv_f4 *>(G) + v_lo;
    const pv_f4 *C4 = reinterpret_cast<const pv_f4 *>(codebooks);
    const uint16_t *codes0 = codes + n_lo * M;
    // Within a codeword's row the elements are permuted by bits of the code (power-of-two
    // groups): for a given element the 64 lanes of an atomic then spread over all LDS banks
    // instead of the few that a row stride of 8 g bytes leaves them.
    const unsigned swm = (g & (g - 1)) == 0 ? (unsigned)g - 1u : 0u;

    // the first vectors of each wave say what to expect; they are read again (from a cache) below
    unsigned gb = 0u, sb = 0u;
    for (int u = 0; u < kSmallAhead; ++u) {
        const int v = lane + u * 64;
        if (v < len) {
            const pv_f4 x = G4[v];
#pragma unroll
            for (int e = 0; e < 4; ++e) gb = max(gb, __float_as_uint(fabsf(x[e])));
            sb = max(sb, __float_as_uint(fabsf(scales[row0 + pv_row_of(rem0 + (unsigned)v / vpg, inv_gpr)])));
        }
    }
    // adds one vector to the table: elements q4 * 4 .. of a group (its first two codes fetched already)
    // (scale and unit in ss: a power of two, exact); NEGATE: takes away what the same call added
    auto add_terms = [&](const pv_f4 &x, double ss, unsigned q4, const unsigned (&c01)[2], const uint16_t *group_codes,
                         bool negate = false) {
        unsigned long long term[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            term[e] = fixed_point_term(ss * (double)x[e]);
            if (negate) term[e] = 0ull - term[e];
        }
        for (int m = 0; m < M; ++m) {
            const unsigned c = m < 2 ? c01[m] : group_codes[m] & mask;
            unsigned long long *row = tab + ((size_t)m * csize + c) * g;
            const unsigned sw = (c >> 2) & swm;
#pragma unroll
            for (int e = 0; e < 4; ++e) atomicAdd(&row[(q4 * 4u + e) ^ sw], term[e]);
        }
    };
    double X = block_bound(gb, sb, s_max);
    int ex = 0;
    double unit = 0.0;
    for (int attempt = 0; attempt < 2; ++attempt) {
        const bool some = X > 0.0 && X < __builtin_huge_val();
        (void)frexp(some ? X : 0.0, &ex);                  // X < 2^ex
        const double up = some ? ldexp(1.0, kbits - ex) : 0.0;
        unit = some ? ldexp(1.0, ex - kbits) : 0.0;
        for (int e = threadIdx.x; e < entries; e += kSmallBlock) tab[e] = 0ull;
        if (threadIdx.x == 0) s_over = 0u;
        __syncthreads();
        const bool rows = ROWS && attempt == 0;
        unsigned cur = row0;
        int row_end = row_vecs(gpr - (int)rem0);           // in vectors from the wave's first
        double acc = 0.0;
        gb = sb = 0u;
        for (int v0 = 0; v0 < len; v0 += 64 * kSmallAhead) {
            pv_f4 gv[kSmallAhead];
            unsigned nl[kSmallAhead], q4[kSmallAhead], c01[kSmallAhead][2];
#pragma unroll
            for (int u = 0; u < kSmallAhead; ++u) {
                const unsigned vc = (unsigned)min(v0 + u * 64 + lane, len - 1);   // clamped: the loads of a batch go out together
                nl[u] = vc / vpg;
                q4[u] = vc - nl[u] * vpg;
                gv[u] = __builtin_nontemporal_load(&G4[vc]);
#pragma unroll
                for (int m = 0; m < 2; ++m) c01[u][m] = m < M ? codes0[(size_t)nl[u] * M + m] & mask : 0u;
            }
#pragma unroll
            for (int u = 0; u < kSmallAhead; ++u) {
                const int at = v0 + u * 64;                // uniform
                if (at >= len) break;
                const bool in = at + lane < len;
                float sf;
                bool next = false;
                if constexpr (ROWS) {                      // at least 64 vectors a row: two rows at most
                    next = at + lane >= row_end;
                    const float sa = scales[cur], sx = scales[min(cur + 1u, (unsigned)out_features - 1u)];
                    sf = next ? sx : sa;
                } else {
                    sf = scales[row0 + pv_row_of(rem0 + nl[u], inv_gpr)];
                }
                gb = max(max(gb, __float_as_uint(fabsf(gv[u].x))), __float_as_uint(fabsf(gv[u].y)));
                gb = max(max(gb, __float_as_uint(fabsf(gv[u].z))), __float_as_uint(fabsf(gv[u].w)));
                sb = max(sb, in ? __float_as_uint(fabsf(sf)) : 0u);
                if (in) add_terms(gv[u], (double)sf * up, q4[u], c01[u], codes0 + (size_t)nl[u] * M);
                if constexpr (ROWS) {
                    const bool ends = at + 64 > row_end;
                    if (rows) {
                        pv_f4 q = C4[c01[u][0] * vpg + q4[u]];
                        for (int m = 1; m < M; ++m) {
                            const unsigned c = m < 2 ? c01[u][m] : codes0[(size_t)nl[u] * M + m] & mask;
                            const pv_f4 cw = C4[((unsigned)m * csize + c) * vpg + q4[u]];
                            q.x = q.x + cw.x;
                            q.y = q.y + cw.y;
                            q.z = q.z + cw.z;
                            q.w = q.w + cw.w;
                        }
                        // a product of two floats is exact in double: one rounding a term
                        double d = (double)gv[u].x * (double)q.x;
                        d = fma((double)gv[u].y, (double)q.y, d);
                        d = fma((double)gv[u].z, (double)q.z, d);
                        d = fma((double)gv[u].w, (double)q.w, d);
                        if (!in) d = 0.0;
                        if (ends) {
                            const double total = wave_sum_f64(acc + (next ? 0.0 : d));
                            if (lane == 0) mem.rows[(size_t)cur + wave] = total;
                            acc = next ? d : 0.0;
                        } else {
                            acc = acc + d;
                        }
                    }
                    if (ends) {
                        ++cur;
                        row_end += row_vecs(gpr);
                    }
                }
            }
        }
        if (ROWS && rows && len > 0) {                     // the row that goes on: zero if none of it was met
            const double total = wave_sum_f64(acc);
            if (lane == 0) mem.rows[(size_t)cur + wave] = total;
        }
        X = block_bound(gb, sb, s_max);                    // what the block did meet
        if (!(X < __builtin_huge_val())) unit = __builtin_nan("");
        // terms up to the limit stay below 2^51 and their sums below 2^63
        if (__builtin_expect(unit != unit || X <= unit * ldexp(1.99, kbits), 1)) break;
        if (some) {
            const double limit = ldexp(1.99, kbits);
            for (int v = lane; v < len; v += 64) {
                const unsigned n = (unsigned)v / vpg;
                const pv_f4 x = G4[v];
                const double ss = (double)scales[row0 + pv_row_of(rem0 + n, inv_gpr)] * up;
                if (fabs(ss) * (double)fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w))) > limit) {
                    const unsigned i = atomicAdd(&s_over, 1u);
                    unsigned c[2];
#pragma unroll
                    for (int m = 0; m < 2; ++m) c[m] = m < M ? codes0[(size_t)n * M + m] & mask : 0u;
                    if (i < kSmallOver) {
                        s_list[i] = (threadIdx.x >> 6) * (unsigned)per_wave + (unsigned)v;
                        add_terms(x, ss, (unsigned)v - n * vpg, c, codes0 + (size_t)n * M, true);
                    }
                }
            }
            __syncthreads();
            const unsigned over = s_over;
            if (over <= kSmallOver) {
                // the unit of the true bound (2^shift of the old): the table is rounded to it, the list added
                int to = 0;
                (void)frexp(X, &to);
                const int shift = to - ex;
                for (int e = threadIdx.x; e < entries; e += kSmallBlock) {
                    const long long t = (long long)tab[e];
                    tab[e] = shift < 64 ? (unsigned long long)((t >> shift) + ((t >> (shift - 1)) & 1)) : 0ull;
                }
                unit = ldexp(1.0, to - kbits);
                __syncthreads();
                for (unsigned i = threadIdx.x; i < over; i += kSmallBlock) {
                    const int64_t v = (int64_t)blockIdx.x * kSmallWaves * per_wave + s_list[i];
                    const int64_t n = v / vpg;
                    unsigned c[2];
#pragma unroll
                    for (int m = 0; m < 2; ++m) c[m] = m < M ? codes[n * M + m] & mask : 0u;
                    const pv_f4 x = reinterpret_cast<const pv_f4 *>(G)[v];
                    add_terms(x, (double)scales[n / gpr] * ldexp(1.0, kbits - to), (unsigned)(v - n * vpg), c, codes + n * M);
                }
                __syncthreads();
                break;
            }
        }
        __syncthreads();                                   // s_over was read
    }
    long long *out = mem.partial + (int64_t)blockIdx.x * entries;
    for (int e = threadIdx.x; e < entries; e += kSmallBlock) {
        const unsigned sw = ((((unsigned)e / (unsigned)g) & mask) >> 2) & swm;   // the code within its codebook, as on the way in
        out[e] = (long long)tab[(unsigned)e ^ sw];
    }
    if (threadIdx.x == 0) mem.unit[blockIdx.x] = unit;
}

// sum + error, the rounding error of the addition kept (Knuth)
__device__ __forceinline__ void add_keeping_error(double &sum, double &error, double v)
{
    const double t = sum + v, b = t - sum;
    error = error + ((sum - (t - b)) + (v - b));
    sum = t;
}

// adds the blocks' tables (16 threads per entry, each a slice of the blocks) and rounds once: upper
// and lower half of an integer are exact as doubles, the upper halves' sum keeps its rounding errors
// and the lower halves' sum has bits to spare.  The blocks from `eblocks` on add the waves' parts of a
// row each thread.
constexpr int kSlices = 16;
__global__ __launch_bounds__(kBlock) void k_pg_small_final(small_mem mem, int blocks, int entries, int eblocks,
                                                           int rows, int64_t row_vecs, int per_wave,
                                                           float *__restrict__ out,
                                                           float *__restrict__ grad_scales)
{
    if ((int)blockIdx.x >= eblocks) {
        const int64_t r = (int64_t)((int)blockIdx.x - eblocks) * kBlock + threadIdx.x;
        if (r >= rows) return;
        const int w1 = (int)(((r + 1) * row_vecs - 1) / per_wave);
        double total = 0.0;
        for (int w = (int)(r * row_vecs / per_wave); w <= w1; ++w) total = total + mem.rows[r + w];
        grad_scales[r] = (float)total;
        return;
    }
    __shared__ double s_sum[kSlices][kBlock / kSlices], s_err[kSlices][kBlock / kSlices];
    const int col = threadIdx.x % (kBlock / kSlices), sl = threadIdx.x / (kBlock / kSlices);
    const int e = blockIdx.x * (kBlock / kSlices) + col;
    double total = 0.0, error = 0.0;
    if (e < entries) {
        for (int b0 = sl; b0 < blocks; b0 += kSlices * 8) {
            long long p[8];
            double unit[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int b = b0 + u * kSlices;
                p[u] = b < blocks ? mem.partial[(int64_t)b * entries + e] : 0;
                unit[u] = b < blocks ? mem.unit[b] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                add_keeping_error(total, error, (double)(int)(p[u] >> 32) * (unit[u] * 4294967296.0));
                error = error + (double)(unsigned)p[u] * unit[u];
            }
        }
    }
    s_sum[sl][col] = total;
    s_err[sl][col] = error;
    __syncthreads();
    if (sl == 0 && e < entries) {
        for (int q = 1; q < kSlices; ++q) {
            add_keeping_error(total, error, s_sum[q][col]);
            error = error + s_err[q][col];
        }
        total = total + error;
        out[e] = total == total ? (float)total : __builtin_nanf("");
    }
}

// one block per output row; VEC: g % 4 == 0, a thread takes 16-byte vectors
template <bool VEC>
__global__ __launch_bounds__(kBlock) void k_pg_scales(const float *__restrict__ G,
                                                      const uint16_t *__restrict__ codes,
                                                      const float *__restrict__ codebooks, int g,
                                                      int M, int nbits, int gpr,
                                                      float *__restrict__ grad_scales)
{
    __shared__ double tmp[kBlock / 64];
    const int64_t o = blockIdx.x;
    const int64_t csize = (int64_t)1 << nbits;
    const unsigned mask = (unsigned)csize - 1u;
    const int64_t in_features = (int64_t)gpr * g;
    double acc = 0.0;
    if constexpr (VEC) {
        const int vpg = g / 4;                                  // vectors per group
        const int64_t nv = in_features / 4;
        const pv_f4 *G4 = reinterpret_cast<const pv_f4 *>(G + o * in_features);
        const pv_f4 *C4 = reinterpret_cast<const pv_f4 *>(codebooks);
        // kAhead vectors of a thread at a time: their codes, then their codewords, are in flight
        // together (a row is only a few vectors per thread: one at a time the kernel is a chain
        // of round trips); the terms are still added in index order
        constexpr int kAhead = 4;
        for (int64_t e0 = threadIdx.x; e0 < nv; e0 += (int64_t)kBlock * kAhead) {
            pv_f4 gv[kAhead], q[kAhead];
            unsigned code[kAhead];
            int q4[kAhead];
            int64_t n[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int64_t e = e0 + (int64_t)u * kBlock;
                const int64_t ec = e < nv ? e : nv - 1;
                n[u] = o * gpr + ec / vpg;
                q4[u] = (int)(ec % vpg);
                gv[u] = __builtin_nontemporal_load(&G4[ec]);
                code[u] = codes[n[u] * M] & mask;
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) q[u] = C4[((int64_t)code[u] * g) / 4 + q4[u]];
            for (int m = 1; m < M; ++m) {
                pv_f4 c[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
                    c[u] = C4[((m * csize + (codes[n[u] * M + m] & mask)) * g) / 4 + q4[u]];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    q[u].x = q[u].x + c[u].x;
                    q[u].y = q[u].y + c[u].y;
                    q[u].z = q[u].z + c[u].z;
                    q[u].w = q[u].w + c[u].w;
                }
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (e0 + (int64_t)u * kBlock < nv) {
                    acc = acc + (double)gv[u].x * (double)q[u].x;
                    acc = acc + (double)gv[u].y * (double)q[u].y;
                    acc = acc + (double)gv[u].z * (double)q[u].z;
                    acc = acc + (double)gv[u].w * (double)q[u].w;
                }
            }
        }
    } else {
        for (int64_t e = threadIdx.x; e < in_features; e += kBlock) {
            const int64_t n = o * gpr + e / g;
            const int i = (int)(e % g);
            float q = codebooks[(int64_t)(codes[n * M] & mask) * g + i];
            for (int m = 1; m < M; ++m)
                q = q + codebooks[(m * csize + (codes[n * M + m] & mask)) * g + i];
            const float gv = G[o * in_features + e];
            acc = acc + (double)gv * (double)q;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc = acc + __shfl_down(acc, off);
    if ((threadIdx.x & 63) == 0) tmp[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) t = t + tmp[w];
        grad_scales[o] = (float)t;
    }
}

inline size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

pv_status pv_launch_codebook_grads(pv_ctx *ctx, const pv_layout *l, const float *G,
                                   const uint16_t *codes, const float *codebooks,
                                   const float *scales, float *grad_codebooks, float *grad_scales)
{
    const int64_t N = pv_num_groups(l);
    const int g = l->group_size, M = l->num_codebooks;
    const int gpr = (int)(l->in_features / g);
    const int csize = 1 << l->nbits;
    const unsigned mask = (unsigned)csize - 1u;
    hipStream_t sm = ctx->stream;

    // small codebooks: per-block LDS tables instead of a sort
    const int64_t entries = (int64_t)M * csize * g;
    if (g % 4 == 0 && entries * 8 <= 64 * 1024 && N / csize >= 64) {
        const int vpg = g / 4;
        const int64_t nvec = N * vpg;
        // Groups of a block: up to 2^20 groups as few thousands as leave at most 256 blocks, one per compute
        // unit (a wave takes whole steps, 1024 groups a block), then 4096.  With 4096 throughout, 256 x 1024 at
        // g = 16 took 22 us (1024 a block: 12), 1024 x 1024 2 x 8 20 (13); with 512
        // blocks of fewer groups at 2^20 27 instead of 21.
        const int64_t groups = N <= 1 << 20 ? ((N + (1 << 18) - 1) >> 18) * 1024 : 4096;
        int64_t blocks64 = (N + groups - 1) / groups;
        if (blocks64 > 512) blocks64 = 512;
        const int blocks = (int)blocks64, waves = blocks * kSmallWaves;
        const int unit = 64 * vpg;
        const int per_wave = (int)((nvec + (int64_t)waves * unit - 1) / ((int64_t)waves * unit)) * unit;
        const int64_t most = (int64_t)per_wave / vpg * kSmallWaves;  // terms one block adds to an entry
        int headroom = 1;
        while (((int64_t)1 << headroom) < (most < N ? most : N)) ++headroom;
        const int kbits = 62 - headroom < 50 ? 62 - headroom : 50;   // bits of a term below the bound
        const bool rows = grad_scales && l->in_features >= 256;      // 64 vectors a row
        const size_t o_rows = align_up((size_t)blocks * entries * 8);
        const size_t o_unit = o_rows + align_up(((size_t)l->out_features + waves) * 8);
        pv_status st2 = pv_ensure(ctx, ctx->pstep, o_unit + (size_t)blocks * 8);
        if (st2 != PV_OK) return st2;
        char *p = static_cast<char *>(ctx->pstep.ptr);
        const small_mem mem{reinterpret_cast<long long *>(p), reinterpret_cast<double *>(p + o_rows),
                            reinterpret_cast<double *>(p + o_unit)};
        pv_timed t(ctx, PV_K_PSTEP);
        if (grad_scales && !rows)
            hipLaunchKernelGGL(k_pg_scales<true>, dim3((unsigned)l->out_features), dim3(kBlock), 0, sm,
                               G, codes, codebooks, g, M, l->nbits, gpr, grad_scales);
#define PV_SMALL(V_)                                                                             \
    do {                                                                                         \
        if (rows)                                                                                \
            hipLaunchKernelGGL((k_pg_small<V_, true>), dim3(blocks), dim3(kSmallBlock), (size_t)entries * 8, \
                               sm, G, codes, codebooks, scales, nvec, per_wave, g, M, l->nbits, gpr, \
                               (int)l->out_features, kbits, mem);                                \
        else                                                                                     \
            hipLaunchKernelGGL((k_pg_small<V_, false>), dim3(blocks), dim3(kSmallBlock), (size_t)entries * 8, \
                               sm, G, codes, codebooks, scales, nvec, per_wave, g, M, l->nbits, gpr, \
                               (int)l->out_features, kbits, mem);                                \
    } while (0)
        if (g == 8) PV_SMALL(2);
        else if (g == 16) PV_SMALL(4);
        else if (g == 4) PV_SMALL(1);
        else PV_SMALL(0);
#undef PV_SMALL
        const int eblocks = (int)((entries + kBlock / kSlices - 1) / (kBlock / kSlices));
        const int rblocks = rows ? (int)((l->out_features + kBlock - 1) / kBlock) : 0;
        hipLaunchKernelGGL(k_pg_small_final, dim3((unsigned)(eblocks + rblocks)), dim3(kBlock), 0, sm, mem, blocks,
                           (int)entries, eblocks, (int)l->out_features, l->in_features / 4, per_wave,
                           grad_codebooks, grad_scales);
        PV_HIP(ctx, hipGetLastError());
        return PV_OK;
    }

    const size_t nn = (size_t)N;
    const int nblocks = (int)((N + kSortTile - 1) / kSortTile);           // tiles of a sorting pass
    const int hist_n = 256 * nblocks;
    size_t o_start = 0;
    size_t o_long = o_start + align_up((size_t)(csize + 1) * 4);
    size_t o_nlong = o_long + align_up((size_t)csize * 4);
    size_t o_total = o_nlong + 256;
    size_t o_hist = o_total + 1024;
    size_t o_base = o_hist + align_up((size_t)hist_n * 4);
    size_t o_keys_a = o_base + align_up((size_t)hist_n * 4);
    size_t o_keys_b = o_keys_a + align_up(nn * 2);
    size_t o_vals_a = o_keys_b + align_up(nn * 2);
    size_t o_order = o_vals_a + align_up(nn * 4);
    size_t o_part = o_order + align_up(nn * 4);
    size_t total = o_part + align_up((size_t)(N / kLong + 2) * g * 8);
    pv_status st = pv_ensure(ctx, ctx->pstep, total);
    if (st != PV_OK) return st;
    char *base = static_cast<char *>(ctx->pstep.ptr);
    int32_t *start = reinterpret_cast<int32_t *>(base + o_start);
    int32_t *long_list = reinterpret_cast<int32_t *>(base + o_long);
    unsigned *nlong = reinterpret_cast<unsigned *>(base + o_nlong);
    unsigned *dig_totals = reinterpret_cast<unsigned *>(base + o_total);
    unsigned *hist = reinterpret_cast<unsigned *>(base + o_hist);
    unsigned *hbase = reinterpret_cast<unsigned *>(base + o_base);
    uint16_t *keys_a = reinterpret_cast<uint16_t *>(base + o_keys_a);
    uint16_t *keys_b = reinterpret_cast<uint16_t *>(base + o_keys_b);
    int32_t *vals_a = reinterpret_cast<int32_t *>(base + o_vals_a);
    int32_t *order = reinterpret_cast<int32_t *>(base + o_order);
    double *partial = reinterpret_cast<double *>(base + o_part);

    pv_timed t(ctx, PV_K_PSTEP);
    int team = 8;
    while (team < g) team <<= 1;      // lanes per work item (g <= 64 checked by the caller)
    const int teams_per_block = kBlock / team;
    const unsigned sblocks = (unsigned)((csize + teams_per_block - 1) / teams_per_block);
    int64_t max_long = N / (kLong + 1);           // segments that can be longer than kLong
    if (max_long > csize) max_long = csize;
    if (max_long > 2048) max_long = 2048;         // blocks stride over the list
    const bool two = l->nbits > 8;
    for (int m = 0; m < M; ++m) {
        // pass over the low 8 bits of the codes (the only one when B <= 8) ...
        uint16_t *k1 = two ? keys_a : keys_b;
        int32_t *v1 = two ? vals_a : order;
        const code_keys ck{codes, M, m, mask};
        hipLaunchKernelGGL(k_digit_hist<code_keys>, dim3(nblocks), dim3(kSortBlock), 0, sm, ck, N, 0,
                           nblocks, hist);
        hipLaunchKernelGGL(k_row_scan, dim3(256), dim3(kRadixBlock), 0, sm, hist, nblocks, hbase, dig_totals);
        hipLaunchKernelGGL((k_digit_scatter<code_keys, uint16_t>), dim3(nblocks), dim3(kSortBlock), 0,
                           sm, ck, (const int32_t *)nullptr, N, 0, nblocks, hbase, dig_totals, k1, v1);
        if (two) {   // ... and over the high ones
            const plain_keys<uint16_t> pk{keys_a};
            hipLaunchKernelGGL(k_digit_hist<plain_keys<uint16_t>>, dim3(nblocks), dim3(kSortBlock), 0,
                               sm, pk, N, 8, nblocks, hist);
            hipLaunchKernelGGL(k_row_scan, dim3(256), dim3(kRadixBlock), 0, sm, hist, nblocks, hbase,
                               dig_totals);
            hipLaunchKernelGGL((k_digit_scatter<plain_keys<uint16_t>, uint16_t>), dim3(nblocks),
                               dim3(kSortBlock), 0, sm, pk, (const int32_t *)vals_a, N, 8, nblocks, hbase,
                               dig_totals, keys_b, order);
        }
        hipLaunchKernelGGL(k_pg_starts, dim3((unsigned)((N + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                           sm, keys_b, N, csize, start, nlong);
        float *out = grad_codebooks + (int64_t)m * csize * g;
#define PV_ACC(TEAM_)                                                                            \
    do {                                                                                         \
        hipLaunchKernelGGL(k_pg_short<TEAM_>, dim3(sblocks), dim3(kBlock), 0, sm, start, order, G, \
                           scales, gpr, g, csize, long_list, nlong, out);                         \
        if (max_long > 0)                                                                        \
            hipLaunchKernelGGL(k_pg_long<TEAM_>, dim3((unsigned)max_long), dim3(kBlock), 0, sm,   \
                               long_list, nlong, start, order, G, scales, gpr, g, partial, out);  \
    } while (0)
        switch (team) {
        case 8: PV_ACC(8); break;
        case 16: PV_ACC(16); break;
        case 32: PV_ACC(32); break;
        default: PV_ACC(64); break;
        }
#undef PV_ACC
    }
    if (grad_scales) {
        if (g % 4 == 0)
            hipLaunchKernelGGL(k_pg_scales<true>, dim3((unsigned)l->out_features), dim3(kBlock), 0, sm,
                               G, codes, codebooks, g, M, l->nbits, gpr, grad_scales);
        else
            hipLaunchKernelGGL(k_pg_scales<false>, dim3((unsigned)l->out_features), dim3(kBlock), 0, sm,
                               G, codes, codebooks, g, M, l->nbits, gpr, grad_scales);
    }
    PV_HIP(ctx, hipGetLastError());
    return PV_OK;
}
