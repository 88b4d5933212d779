// Nearest-codeword search over a small codebook (one codebook, g = 8 or 16) in one launch.
//
// The filter of pv_mfma.hip is three or four dependent launches (the codebook's statistics and operand, the groups' operands,
// the contraction, the decisions), of which each lasts about 5 us for a list of some thousand groups.  A codebook of up
// to 128 KiB fits the LDS, so a block can do all of it for its groups: every wave holds a share of the codewords as
// operand rows in registers, contracts them with the block's groups, and teams of lanes decide
// the groups from the keys, with exact objectives from the codebook in LDS.  Bounds and certificate are those of pv_mfma.hip:
// a team evaluates the 16 U codewords behind the best key, then looks (the objective in single precision, the exact one where
// that is within reach) at those behind every other key that can still reach the best
// objective found, and at all codewords of a partition (wave, half wave) whose runner-up key can; where that is much, a wave
// does it.
// Up to a block a compute unit it is a chain of latencies: load, statistics, operands, contraction, decisions, with four barriers
// (five if a group is left to a wave); beyond, a block goes from one batch of groups to the next, whose targets are requested
// while this one is decided, and the decisions (32 exact objectives a group, double) and the contraction share the vector ALU.
// On 12 988 groups, 4096 codewords, the vector ALU issues on 42 % of the kernel's cycles, the matrix cores work on 5 %, the LDS
// on 21 % (8 % conflicts).  Kernels of a search in a trace, summed, three or four launches (between which there are gaps
// of up to 20 us where the list is short) / this: g = 8, 256 codewords, 104 857 groups 39.0 / 22.1 us; 1024, 12 988
// 20.1 / 12.5, 104 857 53.3 / 33.3; 2048, 12 988 25.4 / 13.5, 104 857 74.4 / 38.0; 4096, 1638 23.2 / 13.2, 12 988
// 28.2 / 15.5, 104 857 77.0 / 53.2; g = 16, 256, 52 428 42.2 / 21.6; 1024 55.5 / 27.5; 2048, 6519 43.7 / 16.8, 52 428
// 71.4 / 40.1.  (The list and codebook of 4096 and 12 988 in a step, whose other kernels take the caches: 16.2.)  Not kept:
// operands in registers from the load on (15 registers spilled, a quarter slower with 4096 codewords, 12 988 groups); a block
// for every 64 groups, without the loop (twice the time with 104 857).
// Slower than several launches: g = 16 and many codewords in tight clusters (1024 in 64 of them 57 / 80 us, 2048 77 / 163): in
// order of their norms, which the LDS has no room to sort, a cluster is behind one key, here behind half of the partitions.
#pragma once

namespace {

template <int G>
struct small_shape {
    static constexpr int kMinBits = 8, kMaxBits = G == 8 ? 12 : 11;     // 128 KiB of codewords at most
};

// Waves of a block (2^bits threads, at most 1024), waves a SIMD that the registers allow (160 of them with g = 16, 8 bits,
// where 128 spill), and so the blocks that are on the chip's 256 compute units at once.
constexpr int small_waves(int nbits) { return nbits >= 10 ? 16 : 1 << (nbits - 6); }
constexpr int small_occupancy(int g, int nbits) { return g == 16 && nbits == 8 ? 3 : 4; }
constexpr int small_blocks(int g, int nbits) { return 256 * (4 * small_occupancy(g, nbits) / small_waves(nbits)); }
static_assert(small_blocks(8, 8) <= kCountedBlocks, "a block's counters have a place");

// Super-units (32 codewords) beside the best key's that a team looks at by itself.  A group with more of them would keep the
// block waiting, and goes to a wave; unless three quarters of a wave's groups have more and none more than twice that, up to
// kAlikeUnits: then no team waits for another.  Whole searches: teams alone, every codeword in double / more than 4 to a wave /
// more than 16 / as it is.  104 857 groups of 8, 4096 codewords, one of them 100 times the others 437 / 134 / 153 / 138 us,
// lengths over three decades 859 / 415 / 429 / 417; 1024 codewords in 64 tight clusters 138 / 159 / 95 / 98; 52 428 groups of
// 16, 2048 codewords over three decades 501 / 160 / 179 / 161, in clusters 252 / 161 / 187 / 163.
constexpr unsigned kTeamUnits = 4, kAlikeUnits = 16;

// SHIFT makes kv non-negative for every codeword that is no farther than D, the smaller of the current codeword's distance and
// of a bound for the smallest one's, so a negative key marks codewords that cannot win.
template <int G, int NBITS>
__global__ __launch_bounds__(64 * small_waves(NBITS), small_occupancy(G, NBITS)) void k_search_small(
    const float *__restrict__ T, const float *__restrict__ cb, const float *__restrict__ scales,
    const int32_t *__restrict__ list, int k, int per_block, int nbatch, uint16_t *__restrict__ codes, unsigned long long *num_changed,
    unsigned long long *stats, pv_counts counts, unsigned *__restrict__ block_counts, int gpr, int N)
{
    constexpr int kCsize = 1 << NBITS, kWaves = small_waves(NBITS), kThreads = kWaves * 64;
    constexpr int kTiles = kCsize / 32 / kWaves;          // codeword tiles of a wave
    constexpr int kSu = kTiles / kU, kParts = 2 * kWaves;
    constexpr int kGroups = kCsize * G >= 1 << 15 ? 64 : 128;
    constexpr int kTeam = kThreads >= 16 * kGroups ? 16 : 8, kRecs = (kParts + kTeam - 1) / kTeam;
    static_assert(kTiles % kU == 0 && kU == 2 && kGroups <= kThreads, "whole super-units, half a wave each; a thread a group");
    __shared__ pv_f4 s_cb[kCsize * (G / 4)];
    __shared__ h8 s_x[kGroups * (G == 8 ? 2 : 3)];        // operand B: x_hi, {-1, -1, -1, pieces of SHIFT}
    __shared__ pv_f4 s_meta[kGroups], s_t[kGroups * (G / 4)], s_tmp[kWaves];
    __shared__ float s_s[kGroups];
    __shared__ double s_oprev[kGroups];
    __shared__ int s_prev[kGroups], s_n[kGroups];
    __shared__ int s_rec[2][kParts][kGroups];
    __shared__ double s_best[kGroups];                    // of a group left open: the best objective so far, its codeword
    __shared__ int s_best_idx[kGroups], s_open[kGroups];
    __shared__ unsigned s_nopen, s_cnt[4];
    static_assert((sizeof(s_cb) + sizeof(s_x) + sizeof(s_meta) + sizeof(s_t) + sizeof(s_tmp) + sizeof(s_s) +
                   sizeof(s_oprev) + sizeof(s_prev) + sizeof(s_n) + sizeof(s_rec) + sizeof(s_best) + sizeof(s_best_idx) +
                   sizeof(s_open) + 64) * (small_blocks(G, NBITS) / 256) <= 160 * 1024, "the LDS holds small_blocks");
    pv_counts_clear(counts);
    // A codeword's parts of 16 bytes: eight lanes that read the same part of the rows that the matrix instruction gives them
    // (0 to 3 and 8 to 11) or of eight rows in turn meet in no bank.
    auto row_at = [](int c, int v) { return (c * (G / 4) + (G == 8 ? (c >> 3) & 1 : (c >> 2) & 3)) ^ v; };
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 4) s_cnt[tid] = 0u;
    // ---- the first groups and the codebook are requested, a row a lane
    int n = -1, code = 0;
    float s = 0.0f;
    pv_f4 tgt[G / 4];
    auto load_id = [&](int batch) {
        const int64_t j = (int64_t)batch * per_block + tid;
        n = tid < per_block && j < k ? list[j] : -1;
        if (n >= N) n = -1;
    };
    auto load_group = [&] {
        const int at = n < 0 ? 0 : n;
        code = (int)codes[at] & (kCsize - 1);
        s = scales[at / gpr];
#pragma unroll
        for (int v = 0; v < G / 4; ++v) tgt[v] = reinterpret_cast<const pv_f4 *>(T)[(int64_t)at * (G / 4) + v];
    };
    if (tid < kGroups) load_id(blockIdx.x);
    const int row0 = wave * kTiles * 32 + lane;           // rows row0 + 64 i are the lane's
    pv_f4 all;
    {
        pv_f4 own[kTiles / 2][G / 4];
#pragma unroll
        for (int i = 0; i < kTiles / 2; ++i)
#pragma unroll
            for (int v = 0; v < G / 4; ++v) own[i][v] = reinterpret_cast<const pv_f4 *>(cb)[(row0 + 64 * i) * (G / 4) + v];
        if (tid < kGroups) load_group();
        cb_stat st;
#pragma unroll
        for (int i = 0; i < kTiles / 2; ++i) {
            stat_add<G>(st, own[i]);
#pragma unroll
            for (int v = 0; v < G / 4; ++v) s_cb[row_at(row0 + 64 * i, v)] = own[i][v];
        }
        all = pv_f4{wave_max_f(st.m), wave_min_f(st.nmin), wave_max_f(st.nmax), __any(st.bad) ? 1.0f : 0.0f};
        if (lane == 0) s_tmp[wave] = all;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const pv_f4 o = s_tmp[w];
        all.x = fmaxf(all.x, o.x);
        all.y = fminf(all.y, o.y);
        all.z = fmaxf(all.z, o.z);
        all.w = fmaxf(all.w, o.w);
    }
    unsigned meta[8];
    meta_words(all, meta);
    bool ok;
    const float P = scale_from_maxabs(meta[0], &ok);
    ok = ok && meta[3] == 0u && meta[1] != 0u;
    const float cmax = P * sqrtf(all.z) * 1.0001f + kNormMargin;      // >= every ||c_hi||
    const float cmin = P * sqrtf(all.y) * 1.0001f + kNormMargin;
    // Operands: every lane rounds one row of a pair of tiles, the halves of the wave then exchange.  (Halves below the normal
    // range: kept or flushed by the matrix core, the operand lies within kNormMargin of P c either way.)
    h8 a[kTiles], an[G == 16 ? kTiles : 1];
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    auto exchange = [](const h8 &x, const h8 &y, h8 &first, h8 &second) {       // {x.low, y.low}, {x.high, y.high}
        const u4 p = __builtin_bit_cast(u4, x), q = __builtin_bit_cast(u4, y);
        u4 f, g;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const auto r = __builtin_amdgcn_permlane32_swap(p[e], q[e], false, false);
            f[e] = r[0];
            g[e] = r[1];
        }
        first = __builtin_bit_cast(h8, f);
        second = __builtin_bit_cast(h8, g);
    };
#pragma unroll
    for (int i = 0; i < kTiles / 2; ++i) {
        h8 c[G / 8], nrm, zero;
        float n2 = 0.0f;
#pragma unroll
        for (int v = 0; v < G / 4; ++v) {
            const pv_f4 cw = s_cb[row_at(row0 + 64 * i, v)];
#pragma unroll
            for (int e = 0; e < 4; ++e) c[v / 2][v % 2 * 4 + e] = (_Float16)(ok ? 2.0f * P * cw[e] : 0.0f);
        }
#pragma unroll
        for (int h = 0; h < G / 8; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const h2 w = {c[h][2 * e], c[h][2 * e + 1]};
                n2 = __builtin_amdgcn_fdot2(w, w, n2, false);
            }
        _Float16 pieces[3];
        split3(0.25f * n2, pieces);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            nrm[e] = e < 3 ? pieces[e] : e < 6 ? (_Float16)1.0f : (_Float16)0.0f;
            zero[e] = (_Float16)0.0f;
        }
        if constexpr (G == 8) {
            exchange(c[0], nrm, a[2 * i], a[2 * i + 1]);
        } else {
            exchange(c[0], c[1], a[2 * i], a[2 * i + 1]);
            exchange(nrm, zero, an[2 * i], an[2 * i + 1]);
        }
    }
    // >= every ||P c - c_hi||: half an fp16 ulp of each element, and what the matrix core flushes (below 2^-15 each)
    const float dC = P * sqrtf(all.z) * 4.8838e-4f + 1.3e-4f;
    for (int batch = blockIdx.x; batch < nbatch; batch += gridDim.x) {
    const int have = min(per_block, k - batch * per_block);
    if (tid < kGroups) {
        pv_f4 m = {0.0f, 0.0f, 0.0f, -1.0f};
        h8 x[G / 8], xs;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            xs[e] = (_Float16)0.0f;
#pragma unroll
            for (int h = 0; h < G / 8; ++h) x[h][e] = (_Float16)0.0f;
        }
        double obj = 0.0;
        if (n >= 0) {
            float xx = 0.0f, e2 = 0.0f, u2 = 0.0f, p2 = 0.0f;
            bool fits = ok && (s != 0.0f) && (fabsf(s) < 3.0e38f);
            const float div = fits ? s : 1.0f;
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const float t = tgt[i >> 2][i & 3], c = s_cb[row_at(code, i >> 2)][i & 3];
                const double r = fma((double)s, (double)c, -(double)t);     // (s * c is exact in double)
                obj = obj + r * r;
                const float u = P * (t / div);
                if (!(fabsf(u) < 240.0f)) fits = false;   // also catches NaN / inf
                const _Float16 hv = to_half_flush(fits ? u : 0.0f);
                const float hf = (float)hv, d = u - hf, dc = P * c - u;
                xx = fmaf(hf, hf, xx);
                e2 = fmaf(d, d, e2);
                u2 = fmaf(u, u, u2);
                p2 = fmaf(dc, dc, p2);
                x[i >> 3][i & 7] = hv;
            }
            if (fits && xx < 57000.0f) {                  // (the bounds: see prep_group)
                const float xn = sqrtf(xx) * 1.0001f;
                const float e1 = 1.01f * (2.0f * kGamma * (cmax + xn) * (cmax + xn) * 1.01f + 5.0e-4f);
                const float dx = sqrtf(e2) * 1.0001f + 2.4e-7f * sqrtf(u2) + 1.0e-30f;
                // fp32 differences of elements up to (32 + |u|), each rounded once
                const float dp = sqrtf(p2) * 1.00001f + 3.0e-7f * (cmax + xn);
                const float D = fminf(dp, (xn + cmin + dx) * 1.0001f);
                // ||P c - u|| <= D makes ||c_hi - x_hi|| <= D + dx + kNormMargin (rounding of a codeword)
                const float want = (D + dx + kNormMargin) * (D + dx + kNormMargin) * 1.0001f + e1 - xx * 0.9999f + 1.0e-3f;
                if (fabsf(want) < 60000.0f) {
                    _Float16 pieces[3];
                    split3(want, pieces);
                    m.x = ((float)pieces[0] + (float)pieces[1]) + (float)pieces[2];
                    m.y = xx;
                    m.z = e1;
                    m.w = dx;
                    xs[0] = xs[1] = xs[2] = (_Float16)-1.0f;
                    xs[3] = pieces[0];
                    xs[4] = pieces[1];
                    xs[5] = pieces[2];
                }
            }
        }
        if (m.w < 0.0f)
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int h = 0; h < G / 8; ++h) x[h][e] = (_Float16)0.0f;
        s_x[tid] = x[0];
        if constexpr (G == 16) s_x[kGroups + tid] = x[1];
        s_x[(G / 8) * kGroups + tid] = xs;
#pragma unroll
        for (int v = 0; v < G / 4; ++v) s_t[tid * (G / 4) + v] = tgt[v];
        s_meta[tid] = m;
        s_s[tid] = s;
        s_prev[tid] = code;
        s_n[tid] = n;
        s_oprev[tid] = obj;
        load_id(batch + gridDim.x);                       // of the next batch (none: -1)
    }
    if (tid == 0) s_nopen = 0u;
    __syncthreads();

    // ---- contraction: the wave's codewords with 32 groups at a time
    unsigned vmask = ~kKeyMask;
    asm volatile("" : "+v"(vmask));   // keep the mask in a vector register
    const f16v z = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int g0 = 0; g0 < have; g0 += 32) {               // uniform
        h8 b, bn;
        if constexpr (G == 8) {
            b = s_x[(half ? kGroups : 0) + g0 + col];
        } else {
            b = s_x[(half ? kGroups : 0) + g0 + col];
            bn = s_x[2 * kGroups + g0 + col];
        }
        int best = kNoKey, second = kNoKey;
#pragma unroll
        for (int su = 0; su < kSu; ++su) {
            int run = kNoKey;
#pragma unroll
            for (int uu = 0; uu < kU; ++uu) {
                f16v acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[su * kU + uu], b, z, 0, 0, 0);
                if constexpr (G == 16) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(an[su * kU + uu], bn, acc, 0, 0, 0);
                run = uu == 0 ? acc_max<true>(acc, kNoKey) : acc_max<false>(acc, run);
            }
            const int key = and_or(run, vmask, (unsigned)su);
            second = imed3(best, second, key);
            best = max(best, key);
        }
        s_rec[0][wave * 2 + half][g0 + col] = best;
        s_rec[1][wave * 2 + half][g0 + col] = second;
    }
    if (tid < kGroups) load_group();                      // its targets, while this one is decided
    __syncthreads();

    // ---- decisions
    // (places worked out here again: kept over the loop they are registers that spill)
    int tid_d = tid;
    asm volatile("" : "+v"(tid_d));
    const int lane_d = tid_d & 63, half_d = lane_d >> 5;
    // The exact objective of codeword c for group g, as everywhere.
    auto exact_at = [&](int g, float sg, int c, cand_t &mine) {
        double obj = 0.0;
#pragma unroll
        for (int v = 0; v < G / 4; ++v) {
            const pv_f4 cw = s_cb[row_at(c, v)], tv = s_t[g * (G / 4) + v];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double r = fma((double)sg, (double)cw[e], -(double)tv[e]);
                obj = obj + r * r;
            }
        }
        if (cand_better(obj, c, mine.obj, mine.idx)) {
            mine.obj = obj;
            mine.idx = c;
        }
    };
    // What an objective in single precision must not exceed, if the exact one is to reach e: its sum has a relative error of at
    // most (G + 2) 2^-24 (product and difference in one rounding), what underflows is below 2e-37.  (NaN, infinity: none does.)
    auto limit_of = [](double e) { return float_above(e) * 1.000002f + 2.0e-37f; };
    auto load_t = [&](int g, pv_f4 (&t)[G / 4]) {
#pragma unroll
        for (int v = 0; v < G / 4; ++v) t[v] = s_t[g * (G / 4) + v];
    };
    auto reaches = [&](const pv_f4 (&t)[G / 4], float sg, int c, float limit) {
        float dd = 0.0f;
#pragma unroll
        for (int v = 0; v < G / 4; ++v) {
            const pv_f4 cw = s_cb[row_at(c, v)];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float r = fmaf(sg, cw[e], -t[v][e]);
                dd = fmaf(r, r, dd);
            }
        }
        return !(dd > limit);
    };
    auto decide = [&](int g, const cand_t &win, unsigned evals, bool scanned) {
        const int prev = s_prev[g];
        int pick = win.idx;
        if (s_oprev[g] <= win.obj || pick == 0x7fffffff) pick = prev;
        if (pick != prev) {
            codes[s_n[g]] = (uint16_t)pick;
            atomicAdd(&s_cnt[1], 1u);
        }
        atomicAdd(&s_cnt[scanned ? 3 : 0], 1u);
        atomicAdd(&s_cnt[2], evals + 1u);
    };
    // A team a group (8 lanes, 16 where there are enough) evaluates what is behind the best key, and looks at what else can
    // reach the objective found, if that is not too much (kTeamUnits).
    const int q = tid_d % kTeam, team_shift = lane_d & ~(kTeam - 1);
    for (int g = tid_d / kTeam; g < have; g += kThreads / kTeam) {
        if (s_n[g] < 0) continue;                         // whole teams
        const pv_f4 m = s_meta[g];
        const float sg = s_s[g];
        const double o_prev = s_oprev[g];
        cand_t mine;
        mine.obj = __builtin_huge_val();
        mine.idx = 0x7fffffff;
        unsigned evals = 0;
        bool open = m.w < 0.0f, scanned = false;          // (not for the filter)
        if (!open) {
            int2 rec[kRecs];
#pragma unroll
            for (int u = 0; u < kRecs; ++u) {
                const int p = q + kTeam * u;
                rec[u] = p < kParts ? make_int2(s_rec[0][p][g], s_rec[1][p][g]) : make_int2(kNoKey, kNoKey);
            }
            long long bk = (long long)0x8000000000000000ull;
#pragma unroll
            for (int u = 0; u < kRecs; ++u) {
                const long long v = ((long long)rec[u].x << 32) | (long long)(unsigned)(63 - (q + kTeam * u));
                bk = v > bk ? v : bk;
            }
            bk = pv_team_max_i64<kTeam>(bk);
            const int best_key = (int)(bk >> 32), best_p = 63 - (int)(bk & 0xFFFFFFFFll);
            double e_star = o_prev;
            if (best_key >= 0) {
                constexpr int kEvalUnroll = G == 8 ? kU : 1;
#pragma unroll kEvalUnroll
                for (int uu = 0; uu < kU; ++uu)
#pragma unroll
                    for (int e = 0; e < 16 / kTeam; ++e) {
                        const int qq = q + kTeam * e;
                        exact_at(g, sg, ((best_p >> 1) * kTiles + (best_key & (int)kKeyMask) * kU + uu) * 32 +
                                            8 * (qq >> 2) + 4 * (best_p & 1) + (qq & 3), mine);
                    }
                evals = 16 * kU / kTeam;                  // a lane
                mine = cand_team_min<kTeam>(mine);
                if (mine.obj < e_star) e_star = mine.obj;
            }
            // what was not evaluated and could still reach E*; never what is behind a negative key
            const key_cut cut(m, reach2_of(e_star, P * fast_rcp(fabsf(sg)), dC, m.w));
            unsigned pending = 0, units = 0;              // bit u: the key of rec[u]; bit 16 + u: all of its partition
#pragma unroll
            for (int u = 0; u < kRecs; ++u) {
                const int p = q + kTeam * u;
                if (rec[u].y >= 0 && cut.open(rec[u].y)) pending |= 1u << (16 + u);
                else if (rec[u].x >= 0 && p != best_p && cut.open(rec[u].x)) pending |= 1u << u;
            }
            if (__ballot(pending != 0u))
                units = pv_team_sum_u32<kTeam>((unsigned)(__popc(pending & 0xFFFFu) + kSu * __popc(pending >> 16)));
            unsigned most = kTeamUnits;
            while (most < kAlikeUnits && __popcll(__ballot(units > most)) >= 48) most *= 2u;
            if (__ballot(units > most)) most = kTeamUnits;
            open = units > most;
            if (open) {                                   // per partition, in place of its second key: 1: its best key, 2: all of it
#pragma unroll
                for (int u = 0; u < kRecs; ++u) {
                    const int p = q + kTeam * u;
                    if (p < kParts) s_rec[1][p][g] = (pending >> (16 + u)) & 1u ? 2 : (int)((pending >> u) & 1u);
                }
            } else if (units) {
                float limit = limit_of(e_star);
                // a lane's rows of a super-unit: of each tile, half of it the partition's, rows q, q + kTeam, ..
                constexpr int kMine = kU * 16 / kTeam;
                auto step_of = [](int i) { return kTeam == 16 ? 32 * i : 32 * (i >> 1) + 16 * (i & 1); };
                pv_f4 t[G / 4];
                load_t(g, t);
                for (;;) {
                    const unsigned team = (unsigned)(__ballot(pending != 0u) >> team_shift) & ((1u << kTeam) - 1u);
                    if (!team) break;
                    const int src = __ffs((int)team) - 1;         // lane of the team with work
                    const int bit = __ffs(__shfl((int)pending, src, kTeam)) - 1, u = bit & 15;
                    int key = 0;
#pragma unroll
                    for (int uu = 0; uu < kRecs; ++uu)
                        if (uu == u) key = rec[uu].x;
                    key = __shfl(key, src, kTeam);
                    const int p = src + kTeam * u;
                    const int su0 = bit >= 16 ? 0 : key & (int)kKeyMask, su1 = bit >= 16 ? kSu : su0 + 1;
                    scanned |= bit >= 16;
                    for (int su = su0; su < su1; ++su) {
                        const int c0 = ((p >> 1) * kTiles + su * kU) * 32 + 4 * (p & 1) + 8 * (q >> 2) + (q & 3);
                        unsigned todo = 0;
#pragma unroll
                        for (int i = 0; i < kMine; ++i) todo |= (unsigned)reaches(t, sg, c0 + step_of(i), limit) << i;
                        if (todo) {
                            evals += (unsigned)__popc(todo);
                            do {
                                const int i = __ffs((int)todo) - 1;
                                exact_at(g, sg, c0 + step_of(i), mine);
                                todo &= todo - 1u;
                            } while (todo);
                            limit = fminf(limit, limit_of(mine.obj));
                        }
                    }
                    if (q == src) pending &= ~(1u << bit);
                }
                mine = cand_team_min<kTeam>(mine);
            }
        }
        evals = pv_team_sum_u32<kTeam>(evals);
        if (q == 0) {
            if (open) {
                s_best[g] = mine.obj;
                s_best_idx[g] = mine.idx;
                s_open[atomicAdd(&s_nopen, 1u)] = g;
                atomicAdd(&s_cnt[2], evals);
            } else {
                decide(g, mine, evals, scanned);
            }
        }
    }
    __syncthreads();
    // The groups left open, a wave each, two partitions at a time.
    const int nopen = __builtin_amdgcn_readfirstlane((int)s_nopen);
    if (nopen == 0) continue;                             // (nothing in LDS is read any more)
    for (int item = wave; item < nopen; item += kWaves) {
        const int g = s_open[item];
        const float sg = s_s[g];
        const bool all_of = s_meta[g].w < 0.0f;
        const double o_prev = s_oprev[g];
        cand_t mine;
        mine.obj = s_best[g];
        mine.idx = s_best_idx[g];
        float limit = limit_of(mine.obj < o_prev ? mine.obj : o_prev);
        pv_f4 t[G / 4];
        load_t(g, t);
        const int what_lane = lane_d >= kParts ? 0 : all_of ? 2 : s_rec[1][lane_d][g];
        const bool scanned = __ballot(what_lane == 2) != 0;
        unsigned evals = 0;
        for (unsigned left = (unsigned)__ballot(what_lane != 0); left;) {
            const int p0 = __ffs((int)left) - 1;
            left &= left - 1u;
            const int p1 = __ffs((int)left) - 1;          // -1: none
            left &= left - 1u;
            const int p = half_d && p1 >= 0 ? p1 : p0;
            const int what = half_d && p1 < 0 ? 0 : all_of ? 2 : s_rec[1][p][g];
            const int su0 = what == 1 ? s_rec[0][p][g] & (int)kKeyMask : 0, su1 = what == 1 ? su0 + 1 : what ? kSu : 0;
            const int c0 = (p >> 1) * kTiles * 32 + 32 * ((lane_d >> 4) & 1) + 4 * (p & 1) + 8 * ((lane_d >> 2) & 3) + (lane_d & 3);
            for (int su = su0; su < su1; ++su) {
                const int c = c0 + su * kU * 32;
                if (reaches(t, sg, c, limit)) {
                    exact_at(g, sg, c, mine);
                    limit = fminf(limit, limit_of(mine.obj));
                    ++evals;
                }
            }
        }
        evals = pv_team_sum_u32<16>(evals);
        evals += (unsigned)__shfl_xor((int)evals, 16);
        evals += (unsigned)__shfl_xor((int)evals, 32);
        cand_t win = cand_team_min<16>(mine);
#pragma unroll
        for (int mask = 16; mask < 64; mask <<= 1) {
            const double o = __shfl_xor(win.obj, mask);
            const int i = __shfl_xor(win.idx, mask);
            if (cand_better(o, i, win.obj, win.idx)) {
                win.obj = o;
                win.idx = i;
            }
        }
        if (lane_d == 0) decide(g, win, evals, scanned);
    }
    __syncthreads();
    }
    if (tid < 4) block_counts[4 * blockIdx.x + tid] = s_cnt[tid];
    if (tid == 0) {
        unsigned long long changed;
        if (pv_counts_arrive(counts.mine, gridDim.x, s_cnt[1], &changed)) {
            if (num_changed) *num_changed = changed;
            for (int i = 0; i < 8; ++i) stats[i] = 0ull;
        }
    }
}

// (Little work is k_search_few's.)
bool small_codebook(const pv_layout *l, int64_t k)
{
    return l->nbits >= 8 && l->nbits <= (l->group_size == 8 ? small_shape<8>::kMaxBits : small_shape<16>::kMaxBits) && k < (1 << 30);
}

pv_status pv_launch_search_small(pv_ctx *ctx, const pv_layout *l, const float *T, const float *codebook, const float *scales,
                                 const int32_t *group_idx, int64_t k, uint16_t *codes, int64_t *num_changed)
{
    unsigned long long *stats;
    pv_counts counts;
    uint32_t *rr_counts;
    const pv_status st = pv_counters(ctx, &stats, &counts, &rr_counts);
    if (st != PV_OK) return st;
    const int g = l->group_size;
    // Groups of a batch: whole tiles of 32, as few as give every compute unit a block, as many as the LDS holds besides the
    // codebook.  Blocks: what is on the chip at once, a batch each or several.  (Four waves a SIMD taken for g = 16, 8 bits too:
    // the last quarter of the blocks began when the others had ended, 183 500 groups 55.2 us, so 49.1; 367 001 93.3, 87.7.)
    const int most = (g << l->nbits) >= 1 << 15 ? 64 : 128;
    int per_block = (int)(((k + 255) / 256 + 31) & ~(int64_t)31);
    if (k > 256 * most) per_block = most;
    const int nbatch = (int)((k + per_block - 1) / per_block);
    const int slots = small_blocks(g, l->nbits);
    const int blocks = nbatch < slots ? nbatch : slots;
    ctx->rr_blocks_last = blocks;
    ctx->rr_counts = rr_counts;
    pv_timed t(ctx, PV_K_SCORE_MFMA);
    auto nc = reinterpret_cast<unsigned long long *>(num_changed);
#define PV_SMALL_CB(G_, B_)                                                                                          \
    case B_:                                                                                                      \
        hipLaunchKernelGGL((k_search_small<G_, B_>), dim3(blocks), dim3(64 * small_waves(B_)), 0, ctx->stream, T, codebook, scales, \
                           group_idx, (int)k, per_block, nbatch, codes, nc, stats, counts, rr_counts, (int)(l->in_features / g),    \
                           (int)pv_num_groups(l));                                                                \
        break
    if (g == 8)
        switch (l->nbits) {
            PV_SMALL_CB(8, 8);
            PV_SMALL_CB(8, 9);
            PV_SMALL_CB(8, 10);
            PV_SMALL_CB(8, 11);
            PV_SMALL_CB(8, 12);
        }
    else
        switch (l->nbits) {
            PV_SMALL_CB(16, 8);
            PV_SMALL_CB(16, 9);
            PV_SMALL_CB(16, 10);
            PV_SMALL_CB(16, 11);
        }
#undef PV_SMALL_CB
    PV_HIP(ctx, hipGetLastError());
    pv_counters_cleared(ctx, counts);
    return PV_OK;
}

}  // namespace
