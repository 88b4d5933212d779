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
// groups are put in code order by two launches that exchange 4 bytes a group and, where no bucket is
// overfull, no atomics:
// - k_pg_tiles puts every tile of 8192 groups in the order of up to 512 buckets of codes and writes
//   the tile where it was read, with the places where its buckets start; no
//   counts over the whole matrix are needed.  Blocks of the same launch take the scale gradient,
//   a tree sum per row.
// - k_pg_buckets gives a block to a bucket: it lays the tiles' runs end to end in LDS, puts them in
//   code order there, and sums every codeword's groups by a team of lanes in ascending group order,
//   in double with exact products: the same sum, in the same order, as a plain loop over the
//   groups.  Codewords with more than kLong groups in a chunk of the bucket are summed in pieces that are
//   added in order (a different association from the plain loop: reproducible from run to run,
//   but no longer the sequential rounding).
// - A bucket with far more groups than the others (a codeword that holds many, or several that meet
//   in a bucket) would be one block's work for long: a chunk of 8192 groups takes it 36 us (21 the sums, whose
//   gathers are bound by what one compute unit has in flight).  Its chunks go to blocks of their own, and the last of
//   those to be done adds up.
// Bound by the gathers: 32 bytes of G (g = 8) bring a line of 128, and 2^21 of them in random order
// take 41 us of k_pg_buckets' 54 whatever the kind of load (plain, nontemporal, device scope) and
// whether G was read shortly before.  4096 x 4096, 1 x 16, codes drawn evenly: 107 -> 80 us a call against a radix
// sort of (code, group) in two passes of three kernels, segment starts, sums and scales (nine launches);
// 354 x 384, 1 x 12 41 -> 19; 4096 x 4096, 1 x 12 118 -> 85.  Scales as a launch of their own: 84; beside the
// sums instead of the order: 82.  Buckets of 256 or tiles of 4096 groups: 1 to 8 us more.
// Codes used unevenly, 4096 x 4096, 1 x 16 (the radix sort / buckets of consecutive codes, a block each / this):
// 64 neighbouring codewords hold everything 1390 / 5640 / 131 us, 512 of them 1225 / 1895 / 106; uses that fall
// like 1 / code 705 / 4310 / 172, the same in random order 719 / 730 / 171; one codeword with a third 3370 / 3170 /
// 146; 64 at random places 382 / 389 / 128, 512 151 / 132 / 136; 128 codewords 512 apart 194 / 171 / 170.
// Small codebooks take another route (k_pg_small below), which takes the scale gradient along.
#include "pv_internal.h"
#include "pv_dpp.h"

namespace {

constexpr int kBlock = 256;
constexpr int kLong = 128;       // groups of a codeword in a chunk that one team sums alone, in order

// ---- large codebooks: tiles put in bucket order, then a block for every bucket

// A bucket is 2^low codes, at most 512 buckets a codebook: those whose product with the golden section of 2^B (an odd
// number, so every code has a product of its own) agrees in its high bits.  Neighbouring codes, and codes a power of two
// apart, are spread evenly over the buckets that way, and where few codewords hold most groups they are often
// such (a codebook in order of norm or of use, a part of it in use).  With high bits folded into low ones by
// exclusive or, every 64th code used: 160 us a call, 85 this way; with runs of four codes kept together, whose rows of the
// result share a cache line, 512 neighbours that hold all groups 138, 106 this way, and even use the same.
constexpr int kTileBlock = 1024;
constexpr int kTileWaves = kTileBlock / 64;
constexpr int kTilePer = 8;
constexpr int kTileBits = 13;
constexpr int kTile = 1 << kTileBits;             // groups of a tile
constexpr int kBucketBits = 9;
constexpr int kBuckets = 1 << kBucketBits;
static_assert(kTile == kTileBlock * kTilePer && kBuckets <= kTileBlock, "a tile is one round of a block");

struct bucket_args {
    const uint16_t *codes;
    int64_t N;
    int M, m0;           // codebooks, the first one of this launch
    unsigned mask;       // 2^B - 1
    unsigned mul, inv;   // product of one another: 1 modulo 2^B
    int low, high;       // bits of code * mul within its bucket, bits that name the bucket
    int ntiles;
    uint32_t *entries;   // [codebook of the launch][N] tile by tile: code within the bucket << 16 | place in the tile
    uint16_t *first;     // [codebook of the launch][tile][stride] where a bucket starts in its tile, for buckets + 1
    int stride;          // a multiple of 8
    // buckets with more groups than `overfull`: `spare` chunks in a codebook at most
    unsigned overfull, long_run;         // such a bucket has a tile with more than long_run of its groups
    int mains, spare;                    // blocks with a bucket of their own; then `spare` for each codebook
    unsigned *uneven;                    // [codebook][tile] some bucket has more than long_run groups there
    unsigned *arrived;                   // [codebook][bucket] chunks done
    double *part;                        // [codebook][spare][codes of a bucket][g] their sums
    uint32_t *ids;                       // [codebook][spare][kChunk] their groups in code order
    uint16_t *starts;                    // [codebook][spare][codes of a bucket + 1] where a code's begin
};

// With mul: bucket of a code << low | its number there; with inv: back again.  (16 bits by 16.)
__device__ __forceinline__ unsigned spread_code(unsigned code, unsigned mul, const bucket_args &b)
{
    return (unsigned)__umul24(code, mul) & b.mask;
}

// The lanes of a wave (among `valid`) whose low `bits` bits of d are this lane's: of the lanes with a bit set, those if
// it is set here, else the others.  (The bit spread over a word, and halves of 32: 1 to 3 us a call less than a 64-bit
// choice between the ballot and its complement.)
__device__ __forceinline__ unsigned long long lanes_alike(unsigned d, int bits, bool valid)
{
    const unsigned long long in = __ballot(valid);
    unsigned lo = (unsigned)in, hi = (unsigned)(in >> 32);
#pragma unroll
    for (int bit = 0; bit < kBucketBits; ++bit) {
        if (bit < bits) {                          // uniform
            const unsigned here = (unsigned)((int)(d << (31 - bit)) >> 31);     // all ones if the bit is set
            const unsigned long long has = __ballot(here != 0u);
            lo &= ~((unsigned)has ^ here);
            hi &= ~((unsigned)(has >> 32) ^ here);
        }
    }
    return (unsigned long long)hi << 32 | lo;
}

// Counts of a block's waves per digit become offsets in wave order; start[d] = keys of smaller digits, for d up
// to DIGITS.  All threads call this (at least DIGITS); wcnt[WAVES][DIGITS], start[DIGITS + 1], s_w[DIGITS / 64] in LDS.
template <int WAVES, int DIGITS>
__device__ __forceinline__ void digit_starts(unsigned (*wcnt)[DIGITS], unsigned *start, unsigned *s_w)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned mine = 0, incl = 0;
    __syncthreads();
    if (threadIdx.x < DIGITS) {
        unsigned c[WAVES];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) c[w] = wcnt[w][threadIdx.x];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            wcnt[w][threadIdx.x] = mine;
            mine += c[w];
        }
        incl = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned o = __shfl_up(incl, off);
            if (lane >= off) incl += o;
        }
        if (lane == 63) s_w[wave] = incl;
    }
    __syncthreads();
    if (threadIdx.x < DIGITS) {
        unsigned before = 0;
        for (int w = 0; w < wave; ++w) before += s_w[w];
        start[threadIdx.x] = before + incl - mine;
        if (threadIdx.x == DIGITS - 1) start[DIGITS] = before + incl;
    }
    __syncthreads();
}

// Ranks of `per` rounds of a block's keys (thread's key j: wave * 64 * per + 64 j + lane): a key's place among
// the wave's keys with its digit.  A round finds the lanes with the same digit by one ballot per bit; the wave's
// running count of a digit is in LDS (wcnt, zero at the start), written by the last lane of each set.  Keys with
// equal digits keep their order.
template <int PER, int DIGITS>
__device__ __forceinline__ void digit_ranks(const unsigned (&d)[PER], unsigned (&rank)[PER], int per, int n, int bits,
                                            unsigned (*wcnt)[DIGITS])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (j < per) {                             // uniform
            const bool valid = (wave * per + j) * 64 + lane < n;
            const unsigned long long same = lanes_alike(d[j], bits, valid);
            const unsigned before = valid ? wcnt[wave][d[j]] : 0u;
            rank[j] = before + (unsigned)__popcll(same & below);
            if (valid && lane == 63 - __clzll(same)) wcnt[wave][d[j]] = before + (unsigned)__popcll(same);
        }
    }
}

struct scale_args {
    const float *G;
    const uint16_t *codes;
    const float *codebooks;
    int64_t rows;
    int g, M, nbits, gpr;
    float *grad_scales;
};

// d phi / d s of one output row by a team of kBlock threads (thread t of it; tmp: kBlock / 64 doubles of LDS);
// VEC: g % 4 == 0, a thread takes 16-byte vectors.  All threads of the block call this.
template <bool VEC, int kAhead>
__device__ __forceinline__ void row_scale_grad(const scale_args &a, int64_t o, int t, double *tmp)
{
    const int g = a.g, M = a.M, gpr = a.gpr;
    const int64_t csize = (int64_t)1 << a.nbits;
    const unsigned mask = (unsigned)csize - 1u;
    const int64_t in_features = (int64_t)gpr * g;
    double acc = 0.0;
    if (o < a.rows) {
        if constexpr (VEC) {
            const unsigned vpg = (unsigned)g / 4u;                  // vectors per group
            const double inv_vpg = 1.0 / (double)vpg;
            const int64_t nv = in_features / 4, part = (int64_t)vpg << 24;   // counted in 32 bits: whole groups, whole steps
            const pv_f4 *C4 = reinterpret_cast<const pv_f4 *>(a.codebooks);
            // kAhead vectors of a thread at a time: their codes, then their codewords, are in flight
            // together (a row is only a few vectors per thread: one at a time the kernel is a chain
            // of round trips); the terms are still added in index order
            for (int64_t p0 = 0; p0 < nv; p0 += part) {
                const int cnt = (int)(nv - p0 < part ? nv - p0 : part);
                const pv_f4 *G4 = reinterpret_cast<const pv_f4 *>(a.G + o * in_features) + p0;
                const uint16_t *row_codes = a.codes + (o * gpr + p0 / vpg) * M;
                unsigned code[kAhead];
                auto load_codes = [&](int e0) {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u)
                        code[u] = row_codes[(size_t)pv_row_of((unsigned)min(e0 + u * kBlock, cnt - 1), inv_vpg) * M] & mask;
                };
                load_codes(t);
                for (int e0 = t; e0 < cnt; e0 += kBlock * kAhead) {
                    pv_f4 gv[kAhead], q[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const unsigned e = (unsigned)min(e0 + u * kBlock, cnt - 1);
                        gv[u] = G4[e];
                        q[u] = C4[code[u] * vpg + (e - pv_row_of(e, inv_vpg) * vpg)];
                    }
                    load_codes(e0 + kBlock * kAhead);        // the next ones (past the end: the last one again)
                    for (int m = 1; m < M; ++m) {
                        pv_f4 c[kAhead];
#pragma unroll
                        for (int u = 0; u < kAhead; ++u) {
                            const unsigned e = (unsigned)min(e0 + u * kBlock, cnt - 1), n = pv_row_of(e, inv_vpg);
                            c[u] = C4[((size_t)m * csize + (row_codes[(size_t)n * M + m] & mask)) * vpg + (e - n * vpg)];
                        }
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
                        if (e0 + u * kBlock < cnt) {
                            acc = acc + (double)gv[u].x * (double)q[u].x;
                            acc = acc + (double)gv[u].y * (double)q[u].y;
                            acc = acc + (double)gv[u].z * (double)q[u].z;
                            acc = acc + (double)gv[u].w * (double)q[u].w;
                        }
                    }
                }
            }
        } else {
            for (int64_t e = t; e < in_features; e += kBlock) {
                const int64_t n = o * gpr + e / g;
                const int i = (int)(e % g);
                float q = a.codebooks[(int64_t)(a.codes[n * M] & mask) * g + i];
                for (int m = 1; m < M; ++m)
                    q = q + a.codebooks[(m * csize + (a.codes[n * M + m] & mask)) * g + i];
                acc = acc + (double)a.G[o * in_features + e] * (double)q;
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc = acc + __shfl_down(acc, off);
    if ((t & 63) == 0) tmp[t >> 6] = acc;
    __syncthreads();
    if (t == 0 && o < a.rows) {
        double sum = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) sum = sum + tmp[w];
        a.grad_scales[o] = (float)sum;
    }
}

// one block per output row
template <bool VEC>
__global__ __launch_bounds__(kBlock) void k_pg_scales(scale_args a)
{
    __shared__ double tmp[kBlock / 64];
    row_scale_grad<VEC, 4>(a, blockIdx.x, threadIdx.x, tmp);
}

// The first `sort_blocks` blocks put a tile of groups each in bucket order (stable), the rest take four
// rows of the scale gradient each: the order is a chain of LDS round trips, the gradient a stream.
template <bool VEC>
__global__ __launch_bounds__(kTileBlock, 8) void k_pg_tiles(bucket_args b, scale_args sc, int sort_blocks)
{
    __shared__ unsigned wcnt[kTileWaves][kBuckets];
    __shared__ unsigned s_first[kBuckets + 1], s_w[kBuckets / 64];
    __shared__ unsigned s_out[kTile], s_uneven;
    if ((int)blockIdx.x >= sort_blocks) {
        const int team = threadIdx.x / kBlock;
        row_scale_grad<VEC, 2>(sc, (int64_t)((int)blockIdx.x - sort_blocks) * (kTileBlock / kBlock) + team,
                               threadIdx.x % kBlock, reinterpret_cast<double *>(s_out) + team * (kBlock / 64));
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int mi = (int)blockIdx.x / b.ntiles, tile = (int)blockIdx.x - mi * b.ntiles;
    const int64_t base = (int64_t)tile * kTile;
    const int n = b.N - base < kTile ? (int)(b.N - base) : kTile;
    const int per = (n + kTileBlock - 1) / kTileBlock;
    unsigned code[kTilePer], d[kTilePer], rank[kTilePer];
#pragma unroll
    for (int j = 0; j < kTilePer; ++j) {                  // all loads in flight before the first is used
        const int i = (wave * per + j) * 64 + lane;
        code[j] = b.codes[(base + (i < n ? i : n - 1)) * b.M + b.m0 + mi] & b.mask;
    }
    for (int w = threadIdx.x; w < kTileWaves * kBuckets; w += kTileBlock) (&wcnt[0][0])[w] = 0u;
    if (threadIdx.x == 0) s_uneven = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kTilePer; ++j) {
        code[j] = spread_code(code[j], b.mul, b);
        d[j] = code[j] >> b.low;
    }
    digit_ranks<kTilePer, kBuckets>(d, rank, per, n, b.high, wcnt);
    digit_starts<kTileWaves, kBuckets>(wcnt, s_first, s_w);
#pragma unroll
    for (int j = 0; j < kTilePer; ++j) {
        const int i = (wave * per + j) * 64 + lane;
        if (j < per && i < n)
            s_out[s_first[d[j]] + wcnt[wave][d[j]] + rank[j]] = (code[j] & ((1u << b.low) - 1u)) << 16 | (unsigned)i;
    }
    if ((int)threadIdx.x < 1 << b.high && s_first[threadIdx.x + 1] - s_first[threadIdx.x] > b.long_run) s_uneven = 1u;
    __syncthreads();
    if (b.spare) {
        if (threadIdx.x == 0) b.uneven[mi * b.ntiles + tile] = s_uneven;
        for (int i = tile * kTileBlock + (int)threadIdx.x; i < 1 << b.high; i += b.ntiles * kTileBlock)
            b.arrived[(mi << b.high) + i] = 0u;
    }
    uint32_t *out = b.entries + (int64_t)mi * b.N + base;
    for (int i = threadIdx.x; i < n; i += kTileBlock) out[i] = s_out[i];
    uint16_t *first = b.first + ((int64_t)mi * b.ntiles + tile) * b.stride;
    if ((int)threadIdx.x < 1 << b.high) first[threadIdx.x] = (uint16_t)s_first[threadIdx.x];
    if (threadIdx.x == 0) first[1 << b.high] = (uint16_t)n;
}

// acc[v] += s_o * G[n, i * VEC + v] over the groups ids[a .. b) in that order, as many gathers together as fit
// the registers
template <int VEC, int kInFlight>
__device__ __forceinline__ void ordered_sum(double (&acc)[VEC], const unsigned *ids, int a, int b,
                                            const float *__restrict__ G, const float *__restrict__ scales,
                                            double inv_gpr, int g, int i)
{
    typedef float vec __attribute__((ext_vector_type(VEC)));
    for (int r0 = a; r0 < b; r0 += kInFlight) {
        vec gv[kInFlight];
        float sv[kInFlight];
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const unsigned n = ids[min(r0 + u, b - 1)];
            gv[u] = *reinterpret_cast<const vec *>(G + (int64_t)n * g + i * VEC);
            sv[u] = scales[pv_row_of(n, inv_gpr)];
        }
#pragma unroll
        for (int u = 0; u < kInFlight; ++u)
            if (r0 + u < b) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    acc[v] = acc[v] + (double)sv[u] * (double)gv[u][v];
                }
            }
    }
}

// The tiles' runs of a bucket are laid end to end in LDS (that is group order), put
// in code order (stable), and every codeword's groups are summed by a team of LANES lanes, VEC elements
// each, in ascending group order.  A bucket that does not fit is worked through in chunks, the
// sums going on in device memory (`carry`, written and read by this block alone).  A codeword with more than kLong
// groups in a chunk is cut into pieces that the teams share and that are added in piece order.
// An overfull bucket's chunks are summed by blocks of their own, each of which leaves its sums and the
// groups in code order in device memory.  The block that is done last adds the chunks' sums up, in order, for codewords
// with more than kLong groups altogether, and sums the others from their groups: one after the other, as where
// the bucket is one block's work.
constexpr int kSumBlock = 512;
constexpr int kSumWaves = kSumBlock / 64;
constexpr int kBucketCodes = 1 << (16 - kBucketBits);   // codes of a bucket at most
// With chunks of 5120 groups 2^21 groups spread over the codewords fit as well (54 us), but a codeword that holds a
// twentieth of them costs more than the sort did: 801 us a call against 674, 674 with 8192.
constexpr int kSumPer = 16;
constexpr int kChunk = kSumBlock * kSumPer;
constexpr int kWindow = kSumBlock;                // tiles looked at together
constexpr int kPiece = 32;
constexpr int kRead = 8;                          // groups of a thread that are read together
constexpr int kTilesRel = 4096;                   // tiles that a chunk may span
static_assert(kBucketCodes <= 128 && kTilesRel * kTile <= 1 << 25 && kWindow <= kTilesRel, "an entry in LDS: 7 + 12 + 13 bits");
static_assert(kBuckets == kSumBlock && kBuckets == 64 * 8 && (kSumWaves + 1) * kBuckets < kChunk, "totals of the buckets");
static_assert(kSumBlock % kBucketCodes == 0 && kChunk / kLong <= kBucketCodes, "see the ends of k_pg_buckets");

// inclusive, over the block; a barrier before the next call
__device__ __forceinline__ unsigned block_scan(unsigned v, unsigned *s_scan)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    if (lane == 63) s_scan[wave] = incl;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSumWaves; ++w) incl += w < wave ? s_scan[w] : 0u;
    return incl;
}

// The first blocks have a bucket each.  SPLIT: `spare` more for each codebook have a chunk each of the overfull buckets,
// and return at once where no tile has a run long enough for such a bucket.
template <int LANES, int VEC, bool SPLIT>
__global__ __launch_bounds__(kSumBlock, 4) void k_pg_buckets(bucket_args b, const float *__restrict__ G,
                                                             const float *__restrict__ scales, double inv_gpr, int g,
                                                             double *carry, float *__restrict__ out)
{
    constexpr int kTeams = kSumBlock / LANES;
    __shared__ unsigned s_ent[kChunk];
    __shared__ union {                                // where runs go and counts while a chunk is put in order, then sums of pieces
        struct {
            unsigned cnt[kSumWaves][kBucketCodes], pre[kWindow + 1];
            unsigned short lo[kWindow];
        } order;
        double part[kSumBlock * VEC];
    } s_mem;
    auto &wcnt = s_mem.order.cnt;
    auto &s_pre = s_mem.order.pre;
    auto &s_lo = s_mem.order.lo;
    auto &s_part = s_mem.part;
    __shared__ unsigned s_start[kBucketCodes + 1], s_item[kBucketCodes + 1], s_w4[kBucketCodes / 64], s_scan[kSumWaves], s_fit[kSumWaves], s_pieces;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nb = 1 << b.high, nl = 1 << b.low;
    const int team = threadIdx.x / LANES, i = threadIdx.x % LANES;
    const bool main = !SPLIT || (int)blockIdx.x < b.mains;
    const int mi = main ? (int)blockIdx.x / nb : ((int)blockIdx.x - b.mains) / b.spare;
    int bucket = main ? (int)blockIdx.x - mi * nb : 0;
    int slot = 0, seg = 0, segs = 0;                // chunk `seg` of `segs` of an overfull bucket
    unsigned before = 0, total = 0;                 // groups of the bucket before this block's, and all of them
    const uint16_t *first = b.first + (int64_t)mi * b.ntiles * b.stride;
    if (!main) {
        slot = (int)blockIdx.x - b.mains - mi * b.spare;
        int uneven = 0;
        for (int t = threadIdx.x; t < b.ntiles; t += kSumBlock) uneven |= (int)b.uneven[mi * b.ntiles + t];
        if (!__syncthreads_or(uneven)) return;
        // Every bucket's groups; the chunk that this block's number stands for.  A wave adds up an eighth of the
        // tiles, a lane eight buckets: the sum of where a bucket starts, of which neighbours' difference is the
        // groups.  (Buckets of more than one code are kBuckets.)
        {
            typedef unsigned short us8 __attribute__((ext_vector_type(8)));
            unsigned sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            const us8 *row = reinterpret_cast<const us8 *>(first) + lane;
#pragma unroll 8
            for (int t = wave; t < b.ntiles; t += kSumWaves) {
                const us8 v = row[(int64_t)t * (b.stride / 8)];
#pragma unroll
                for (int q = 0; q < 8; ++q) sum[q] += v[q];
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) s_ent[wave * kBuckets + lane * 8 + q] = sum[q];
            __syncthreads();
            unsigned at = 0;
#pragma unroll
            for (int w = 0; w < kSumWaves; ++w) at += s_ent[w * kBuckets + threadIdx.x];
            s_ent[kSumWaves * kBuckets + threadIdx.x] = at;
            if (threadIdx.x == 0) s_ent[kSumWaves * kBuckets + kBuckets] = (unsigned)b.N;
            __syncthreads();
            total = s_ent[kSumWaves * kBuckets + threadIdx.x + 1] - at;
        }
        const unsigned chunks = total > b.overfull ? (total + kChunk - 1) / kChunk : 0u;
        const unsigned upto = block_scan(chunks, s_scan);
        const bool mine = (unsigned)slot < upto && (unsigned)slot >= upto - chunks;
        if (mine) {
            s_item[0] = threadIdx.x;
            s_item[1] = (unsigned)slot - (upto - chunks);
            s_item[2] = total;
        }
        if (!__syncthreads_or(mine)) return;
        bucket = __builtin_amdgcn_readfirstlane((int)s_item[0]);
        seg = __builtin_amdgcn_readfirstlane((int)s_item[1]);
        total = (unsigned)__builtin_amdgcn_readfirstlane((int)s_item[2]);
        segs = (int)((total + kChunk - 1) / kChunk);
        before = (unsigned)seg * kChunk;
        carry = b.part + ((int64_t)mi * b.spare + slot) * nl * g;
    } else {
        carry += ((int64_t)mi << (b.low + b.high)) * g + (int64_t)bucket * nl * g;
    }
    const uint32_t *entries = b.entries + (int64_t)mi * b.N;
    first += bucket;
    out += ((int64_t)(b.m0 + mi) << (b.low + b.high)) * g;
    if (SPLIT && main && b.ntiles > kWindow) {    // (else the first window has all of it)
        for (int t = threadIdx.x; t < b.ntiles; t += kSumBlock)
            total += (unsigned)first[(int64_t)t * b.stride + 1] - first[(int64_t)t * b.stride];
        block_scan(total, s_scan);
        total = 0;
#pragma unroll
        for (int w = 0; w < kSumWaves; ++w) total += s_scan[w];
        if (total > b.overfull) return;
        __syncthreads();
    }
    bool whole = true;                              // the first chunk: sums start at zero
    int w0 = 0;                                     // the first tile that is not done,
    unsigned skip = 0;                              // and its groups that an earlier chunk took
    // Where the runs of the tiles from w0 on go, and how many of them make `room` groups: n groups in `runs` runs,
    // the last of them perhaps in part (where the window ends first: nothing of the next).  Tiles w .. w + runs;
    // w0 and skip are moved past what was found.
    int runs, n, w;
    auto window = [&](int room) {
        const int t = w0 + (int)threadIdx.x;
        unsigned lo = 0, len = 0;
        if (t < b.ntiles) {
            lo = first[(int64_t)t * b.stride];
            len = first[(int64_t)t * b.stride + 1] - lo;
            if (threadIdx.x == 0) {
                lo += skip;
                len -= skip;
            }
        }
        const unsigned incl = block_scan(len, s_scan);
        s_pre[threadIdx.x] = incl - len;
        s_lo[threadIdx.x] = (unsigned short)lo;
        if (threadIdx.x == kWindow - 1) s_pre[kWindow] = incl;
        const unsigned long long in = __ballot(t < b.ntiles && incl <= (unsigned)room);
        if (lane == 0) s_fit[wave] = (unsigned)__popcll(in);
        __syncthreads();
        int fit = 0;
#pragma unroll
        for (int v = 0; v < kSumWaves; ++v) fit += (int)s_fit[v];
        const bool cut = fit < kWindow && w0 + fit < b.ntiles;
        const int whole_runs = (int)s_pre[fit];
        runs = cut ? fit + 1 : fit;
        n = cut ? room : whole_runs;
        skip = cut ? (fit == 0 ? skip : 0u) + (unsigned)(n - whole_runs) : 0u;
        w = w0;
        w0 += fit;
    };
    while (SPLIT && before > 0) {                            // groups of other blocks
        window((int)before);
        before -= (unsigned)n;
        __syncthreads();
    }
    auto row = [&](int c) { return out + (int64_t)spread_code((unsigned)bucket << b.low | (unsigned)c, b.inv, b) * g + i * VEC; };
    while (w0 < b.ntiles) {
        const int most = SPLIT && segs && seg == segs - 1 ? (int)(total - (unsigned)seg * kChunk) : kChunk;
        const int from = w0;
        int have = 0;
        for (int q = threadIdx.x; q < kSumWaves * kBucketCodes; q += kSumBlock) (&wcnt[0][0])[q] = 0u;
        if (threadIdx.x == 0) s_pieces = 0u;
        for (;;) {
            const bool fresh = w0 == 0 && skip == 0u;
            window(most - have);
            if (SPLIT && main && b.ntiles <= kWindow && fresh && s_pre[kWindow] > b.overfull) return;
            // in LDS: code within the bucket, tile counted from `from`, place in the tile
            auto put = [&](int at, int r, unsigned e) {
                s_ent[have + at] = (e >> 16) << 25 | (unsigned)(w - from + r) << kTileBits | (e & (kTile - 1));
            };
            if (n > runs * 64) {                    // long runs: a thread takes kRead groups at once, wherever they lie
#pragma unroll 1
                for (int q0 = (int)threadIdx.x; q0 - (int)threadIdx.x < n; q0 += kSumBlock * kRead) {
                    unsigned v[kRead];
                    int r[kRead];
#pragma unroll
                    for (int j = 0; j < kRead; ++j) r[j] = 0;
                    for (int step = 1 << (31 - __clz(runs)); step > 0; step >>= 1) {   // the last run that starts at or before it
#pragma unroll
                        for (int j = 0; j < kRead; ++j)
                            if (r[j] + step < runs && (int)s_pre[r[j] + step] <= min(q0 + j * kSumBlock, n - 1)) r[j] += step;
                    }
#pragma unroll
                    for (int j = 0; j < kRead; ++j)
                        v[j] = entries[(unsigned)(w + r[j]) * kTile + s_lo[r[j]] +
                                       (unsigned)(min(q0 + j * kSumBlock, n - 1) - (int)s_pre[r[j]])];
#pragma unroll
                    for (int j = 0; j < kRead; ++j)
                        if (q0 + j * kSumBlock < n) put(q0 + j * kSumBlock, r[j], v[j]);
                }
            } else {                                // a wave a run, eight of them in flight
                constexpr int kRuns = 8;
                for (int r0 = wave; r0 < runs; r0 += kSumWaves * kRuns) {
                    unsigned v[kRuns];
#pragma unroll
                    for (int u = 0; u < kRuns; ++u) {
                        const int r = min(r0 + u * kSumWaves, runs - 1);
                        const int l = min((int)s_pre[r + 1], n) - (int)s_pre[r];
                        v[u] = entries[(unsigned)(w + r) * kTile + s_lo[r] + (lane < l ? lane : 0)];
                    }
#pragma unroll
                    for (int u = 0; u < kRuns; ++u) {
                        const int r = r0 + u * kSumWaves;
                        if (r >= runs) break;
                        const int p = (int)s_pre[r], l = min((int)s_pre[r + 1], n) - p;
                        if (lane < l) put(p + lane, r, v[u]);
                        for (int q = 64 + lane; q < l; q += 64) put(p + q, r, entries[(unsigned)(w + r) * kTile + s_lo[r] + q]);
                    }
                }
            }
            have += n;
            __syncthreads();
            if (have >= most || w0 >= b.ntiles || w0 - from > kTilesRel - kWindow) break;
        }
        n = have;
        const bool last = !(SPLIT && segs) && w0 >= b.ntiles;
        // code order
        const int per = (n + kSumBlock - 1) / kSumBlock;
        {
            unsigned e[kSumPer], d[kSumPer], rank[kSumPer];
#pragma unroll
            for (int j = 0; j < kSumPer; ++j) {
                const int q = (wave * per + j) * 64 + lane;
                e[j] = j < per && q < n ? s_ent[q] : 0u;
                d[j] = e[j] >> 25;
            }
            digit_ranks<kSumPer, kBucketCodes>(d, rank, per, n, b.low, wcnt);
            digit_starts<kSumWaves, kBucketCodes>(wcnt, s_start, s_w4);
#pragma unroll
            for (int j = 0; j < kSumPer; ++j) {
                const int q = (wave * per + j) * 64 + lane;
                if (j < per && q < n)
                    s_ent[s_start[d[j]] + wcnt[wave][d[j]] + rank[j]] =
                        (unsigned)(from + (int)((e[j] >> kTileBits) & (kTilesRel - 1u))) << kTileBits | (e[j] & (kTile - 1));
            }
        }
        // work items: a codeword, or a piece of one
        unsigned clen = 0;
        if ((int)threadIdx.x < nl) clen = s_start[threadIdx.x + 1] - s_start[threadIdx.x];
        if (clen > (unsigned)kLong) s_pieces = 1u;
        __syncthreads();
        const bool pieces = s_pieces != 0u;
        const int piece = max(kPiece, (n + kTeams - 1) / kTeams);
        int items = nl;
        if (pieces) {
            unsigned cnt = (int)threadIdx.x < nl ? (clen > (unsigned)kLong ? (clen + piece - 1) / piece : 1u) : 0u;
            unsigned inc = cnt;
            if (threadIdx.x < kBucketCodes) {
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const unsigned o = __shfl_up(inc, off);
                    if (lane >= off) inc += o;
                }
                if (lane == 63) s_w4[wave] = inc;
            }
            __syncthreads();
            if (threadIdx.x < kBucketCodes) {
                for (int w = 0; w < wave; ++w) inc += s_w4[w];
                s_item[threadIdx.x] = inc - cnt;
                if (threadIdx.x == kBucketCodes - 1) s_item[kBucketCodes] = inc;
            }
            __syncthreads();
            items = (int)s_item[kBucketCodes];
        }
        for (int i0 = 0; i0 < items; i0 += kTeams) {
            const int item = i0 + team;
            int c = item, p = 0, np = 1;
            if (pieces && item < items) {
                int hi = nl;                        // the last codeword whose items start at or before this one
                c = 0;
                while (hi - c > 1) {
                    const int mid = (c + hi) >> 1;
                    if ((int)s_item[mid] <= item) c = mid;
                    else hi = mid;
                }
                p = item - (int)s_item[c];
                np = (int)(s_item[c + 1] - s_item[c]);
            }
            const bool mine = item < items && i * VEC < g;
            double acc[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
            auto finish = [&]() {
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    if (last) row(c)[v] = (float)acc[v];
                    else carry[(int64_t)c * g + i * VEC + v] = acc[v];
                }
            };
            auto go_on = [&]() {
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[v] = carry[(int64_t)c * g + i * VEC + v];
            };
            if (mine) {
                int from = (int)s_start[c], to = (int)s_start[c + 1];
                if (np == 1 && !whole) go_on();
                if (np > 1) {
                    from += p * piece;
                    to = min(to, from + piece);
                }
                ordered_sum<VEC, VEC == 4 ? 8 : 16>(acc, s_ent, from, to, G, scales, inv_gpr, g, i);
                if (np == 1) finish();
            }
            if (pieces) {
                if (mine && np > 1)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) s_part[(team * LANES + i) * VEC + v] = acc[v];
                __syncthreads();
                if (mine && np > 1 && (p == 0 || team == 0)) {   // the codeword's first piece of this round adds up
                    const int more = min(np - p, kTeams - team);
                    int q = 0;
                    if (p > 0 || !whole) go_on();
                    else q = 1;                     // its own is in acc
                    for (; q < more; q += 8) {      // eight reads in flight, added in order
                        double x[8][VEC];
#pragma unroll
                        for (int u = 0; u < 8; ++u)
#pragma unroll
                            for (int v = 0; v < VEC; ++v)
                                x[u][v] = s_part[((team + min(q + u, more - 1)) * LANES + i) * VEC + v];
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            if (q + u < more)
#pragma unroll
                                for (int v = 0; v < VEC; ++v) acc[v] = acc[v] + x[u][v];
                    }
                    if (p + more == np) {
                        finish();
                    } else {
#pragma unroll
                        for (int v = 0; v < VEC; ++v) carry[(int64_t)c * g + i * VEC + v] = acc[v];
                    }
                }
                __syncthreads();
            }
        }
        if (SPLIT && segs) break;
        whole = false;
        __syncthreads();                            // ids, counts and sums of this chunk are done with
    }
    if (!SPLIT || !segs) return;

    // ---- a chunk of an overfull bucket is done: the block that is the last adds up
    const int64_t at = (int64_t)mi * b.spare + slot;
    for (int q = threadIdx.x; q < n; q += kSumBlock) b.ids[at * kChunk + q] = s_ent[q];
    if ((int)threadIdx.x <= nl) b.starts[at * (nl + 1) + threadIdx.x] = (uint16_t)s_start[threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 0) {                         // one wave's fence writes the die's cache back, for all of the block
        __threadfence();
        s_item[0] = atomicAdd(b.arrived + (mi << b.high) + bucket, 1u) + 1u;
        __threadfence();
    }
    __syncthreads();
    if (s_item[0] != (unsigned)segs) return;
    __syncthreads();
    const uint16_t *starts = b.starts + (at - seg) * (nl + 1);
    const double *part = b.part + (at - seg) * nl * g;
    const uint32_t *ids = b.ids + (at - seg) * kChunk;
    constexpr int kShare = kSumBlock / kBucketCodes;
    {                                               // a codeword's groups, by kShare threads
        const int c = (int)threadIdx.x / kShare, p = (int)threadIdx.x % kShare;
        unsigned have = 0;
        if (c < nl)
#pragma unroll 4
            for (int j = p; j < segs; j += kShare)
                have += (unsigned)starts[(int64_t)j * (nl + 1) + c + 1] - starts[(int64_t)j * (nl + 1) + c];
#pragma unroll
        for (int off = 1; off < kShare; off <<= 1) have += __shfl_xor(have, off);
        if (p == 0) s_item[c] = have;
    }
    __syncthreads();
    constexpr int kTogether = 8;
#pragma unroll 1
    for (int c = team; c < nl; c += kTeams)         // more than kLong groups: the chunks' sums in order
        if (s_item[c] > (unsigned)kLong && i * VEC < g) {
            double acc[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
#pragma unroll 1
            for (int j0 = 0; j0 < segs; j0 += kTogether) {
                double x[kTogether][VEC];
#pragma unroll
                for (int u = 0; u < kTogether; ++u)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) x[u][v] = part[((int64_t)min(j0 + u, segs - 1) * nl + c) * g + i * VEC + v];
#pragma unroll
                for (int u = 0; u < kTogether; ++u)
                    if (j0 + u < segs)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) acc[v] = acc[v] + x[u][v];
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v) row(c)[v] = (float)acc[v];
        }
    // up to kLong groups: one after the other, from the chunks' lists
    constexpr int kCodes = kChunk / kLong;          // codewords whose groups fit the list
    constexpr int kLister = kSumBlock / kCodes;     // threads of a codeword, each with some of the chunks
#pragma unroll 1
    for (int c0 = 0; c0 < nl; c0 += kCodes) {
        const int c = c0 + (int)threadIdx.x / kLister, p = (int)threadIdx.x % kLister;
        const int j0 = (int)((int64_t)segs * p / kLister), j1 = (int)((int64_t)segs * (p + 1) / kLister);
        unsigned have = 0;
        if (c < nl && s_item[c] <= (unsigned)kLong)
#pragma unroll 4
            for (int j = j0; j < j1; ++j)
                have += (unsigned)starts[(int64_t)j * (nl + 1) + c + 1] - starts[(int64_t)j * (nl + 1) + c];
        __syncthreads();                            // the lists of the codewords before are done with
        unsigned to = block_scan(have, s_scan) - have;
        if (p == 0) s_start[threadIdx.x / kLister] = to;
        if (threadIdx.x == kSumBlock - 1) s_start[kCodes] = to + have;
        if (have)
            for (int j = j0; j < j1; ++j) {
                const unsigned f = starts[(int64_t)j * (nl + 1) + c], l = starts[(int64_t)j * (nl + 1) + c + 1];
                for (unsigned q = f; q < l; ++q) s_ent[to++] = ids[(int64_t)j * kChunk + q];
            }
        __syncthreads();
#pragma unroll 1
        for (int q = team; q < kCodes && c0 + q < nl; q += kTeams)
            if (s_item[c0 + q] <= (unsigned)kLong && i * VEC < g) {
                double acc[VEC];
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
                ordered_sum<VEC, kTogether>(acc, s_ent, (int)s_start[q], (int)s_start[q + 1], G, scales, inv_gpr, g, i);
#pragma unroll
                for (int v = 0; v < VEC; ++v) row(c0 + q)[v] = (float)acc[v];
            }
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
// 11008 x 4096, 2 x 8: vector-ALU issue fills 84 of the kernel's 138 thousand cycles (21.6 M instructions,
// much of it the conversion to integers), the LDS 60 (sixteen 64-bit atomics a group and codebook; 36 of
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

// s * g + 1.5 * 2^52 holds the integer nearest to s * g (ties to even) in its low mantissa bits for
// |s * g| < 2^51; the terms stay below 2^51.  (s: a scale times a power of two, so the product is exact.)
__device__ __forceinline__ unsigned long long fixed_point_term(double s, float g)
{
    constexpr double kMagic = 6755399441055744.0;
    return (unsigned long long)(__double_as_longlong(fma(s, (double)g, kMagic)) - __double_as_longlong(kMagic));
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
            term[e] = fixed_point_term(ss, x[e]);
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
        float gbf = 0.0f;
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
                // (maxima that keep a NaN: half an instruction an element)
                gbf = __builtin_elementwise_maximum(__builtin_elementwise_maximum(gbf, fabsf(gv[u].x)), fabsf(gv[u].y));
                gbf = __builtin_elementwise_maximum(__builtin_elementwise_maximum(gbf, fabsf(gv[u].z)), fabsf(gv[u].w));
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
        gb = __float_as_uint(gbf) & 0x7FFFFFFFu;
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
    const scale_args sc{G, codes, codebooks, l->out_features, g, M, l->nbits, gpr, grad_scales};

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
            hipLaunchKernelGGL(k_pg_scales<true>, dim3((unsigned)l->out_features), dim3(kBlock), 0, sm, sc);
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

    // Two codebooks at a time: 8 bytes a group of scratch whatever M, and up to 16 for the chunks of overfull buckets.
    const int low = l->nbits > kBucketBits ? l->nbits - kBucketBits : 0, high = l->nbits - low;
    const int nb = 1 << high, stride = (nb + 8) & ~7;
    const unsigned mul = low ? (0x9E3779B9u >> (32 - l->nbits)) | 1u : 1u;     // the golden section of 2^B
    unsigned inv = mul;
    for (int i = 0; i < 4; ++i) inv *= 2u - mul * inv;      // Newton: 3 bits are right to begin with, then 6, 12, 24, 48
    inv &= mask;
    const int64_t ntiles = (N + kTile - 1) / kTile;
    const int at_once = M < 2 ? M : 2;
    // sums that go on from one chunk, or one round of pieces, to the next (a codeword may hold every group)
    const bool chunks = N > kLong;
    // A bucket of more than `overfull` groups is worked through chunk by chunk, by a block each: at least two and a
    // half chunks (128 codewords of 16384 groups, a bucket each: 175 us in two or three chunks one after the other, 210
    // side by side and added up), and three times the average, so that codes drawn evenly have no such bucket.
    const int64_t overfull = 5 * kChunk / 2 > 3 * (N >> high) ? 5 * kChunk / 2 : 3 * (N >> high);
    const int64_t spare = low && N > overfull && ntiles <= kTilesRel ? N / kChunk + N / overfull : 0;
    size_t total = 0;
    auto take = [&](size_t bytes) {
        const size_t at = total;
        total += align_up(bytes);
        return at;
    };
    const size_t o_entries = take((size_t)at_once * N * 4), o_first = take((size_t)at_once * ntiles * stride * 2);
    const size_t o_carry = take(chunks ? (size_t)at_once * csize * g * 8 : 0);
    const size_t o_part = take((size_t)(at_once * spare) * (csize / nb) * g * 8);
    const size_t o_ids = take((size_t)(at_once * spare) * kChunk * 4), o_starts = take((size_t)(at_once * spare) * (csize / nb + 1) * 2);
    const size_t o_uneven = take((size_t)(at_once * ntiles) * 4), o_arrived = take((size_t)at_once * nb * 4);
    pv_status st = pv_ensure(ctx, ctx->pstep, total);
    if (st != PV_OK) return st;
    char *base = static_cast<char *>(ctx->pstep.ptr);
    double *carry = reinterpret_cast<double *>(base + o_carry);
    const double inv_gpr = 1.0 / (double)gpr;

    pv_timed t(ctx, PV_K_PSTEP);
    for (int m0 = 0; m0 < M; m0 += at_once) {
        const int now = M - m0 < at_once ? M - m0 : at_once;
        const bucket_args b{codes, N, M, m0, mask, mul, inv, low, high, (int)ntiles,
                            reinterpret_cast<uint32_t *>(base + o_entries), reinterpret_cast<uint16_t *>(base + o_first), stride,
                            (unsigned)overfull, (unsigned)(overfull / ntiles), nb * now, (int)spare,
                            reinterpret_cast<unsigned *>(base + o_uneven), reinterpret_cast<unsigned *>(base + o_arrived),
                            reinterpret_cast<double *>(base + o_part), reinterpret_cast<uint32_t *>(base + o_ids),
                            reinterpret_cast<uint16_t *>(base + o_starts)};
        const int sort_blocks = (int)(ntiles * now), rows_a_block = kTileBlock / kBlock;
        const int64_t row_blocks = m0 == 0 && grad_scales ? (l->out_features + rows_a_block - 1) / rows_a_block : 0;
        const dim3 grid((unsigned)(sort_blocks + row_blocks));
        if (g % 4 == 0) hipLaunchKernelGGL(k_pg_tiles<true>, grid, dim3(kTileBlock), 0, sm, b, sc, sort_blocks);
        else hipLaunchKernelGGL(k_pg_tiles<false>, grid, dim3(kTileBlock), 0, sm, b, sc, sort_blocks);
#define PV_SUMS(LANES_, VEC_)                                                                                \
    do {                                                                                                     \
        if (spare)                                                                                           \
            hipLaunchKernelGGL((k_pg_buckets<LANES_, VEC_, true>), dim3((unsigned)((nb + spare) * now)),     \
                               dim3(kSumBlock), 0, sm, b, G, scales, inv_gpr, g, carry, grad_codebooks);     \
        else                                                                                                 \
            hipLaunchKernelGGL((k_pg_buckets<LANES_, VEC_, false>), dim3((unsigned)(nb * now)),              \
                               dim3(kSumBlock), 0, sm, b, G, scales, inv_gpr, g, carry, grad_codebooks);     \
    } while (0)
        // lanes that share a codeword: vectors as wide as the group's rows allow, four lanes at least
        if (g == 8) PV_SUMS(4, 2);
        else if (g % 4 == 0 && g <= 16) PV_SUMS(4, 4);
        else if (g % 4 == 0) PV_SUMS(16, 4);
        else if (g <= 8) PV_SUMS(8, 1);
        else PV_SUMS(64, 1);
#undef PV_SUMS
    }
    PV_HIP(ctx, hipGetLastError());
    return PV_OK;
}
