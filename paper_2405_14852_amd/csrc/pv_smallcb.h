// Nearest-codeword search over a small codebook (one codebook, g = 8 or 16) in one launch.
//
// The filter of pv_mfma.hip is three or four dependent launches (the codebook's statistics and operand, the groups' operands,
// the contraction, the decisions), of which each lasts about 5 us for a list of some thousand groups.  A codebook of up
// to 128 KiB fits the LDS, so a block can do all of it for its groups: every wave holds a share of the codewords as
// operand rows in registers, contracts them with the block's groups, and teams of 8 lanes decide
// the groups from the keys, with exact objectives from the codebook in LDS.  Bounds and certificate are those of pv_mfma.hip:
// a team evaluates the 16 U codewords behind the best key, then those behind every other key that can still reach the best
// objective found, and all codewords of a partition (wave, half wave) whose runner-up key can.
// Latency up to a block a compute unit: load, statistics, operands, contraction, decisions are a chain of five barriers; beyond,
// a block goes from one batch of groups to the next, whose targets are requested while this one is decided, and the
// decisions (32 exact objectives a group, double) and the contraction share the vector ALU.  Whole calls, three or four launches / this:
// g = 8, 256 codewords, 104 857 groups 32.6 / 21.2 us; 1024, 12 988 16.8 / 8.5, 104 857 50.5 / 34.3; 2048, 12 988 20.7 / 9.7,
// 104 857 71.2 / 36.8; 4096, 1638 17.8 / 11.6, 12 988 22.3 / 13.7, 104 857 73.1 / 53.5; g = 16, 256, 52 428 38.2 / 18.7; 1024
// 57.5 / 27.8; 2048, 6519 56.8 / 17.2, 52 428 80.1 / 46.5.  Operands kept in registers from the load on: 15 registers spilled and
// 17.2 us with 4096 codewords, 12 988 groups; a block for every 64 groups, without the loop: 112 us with 104 857.
#pragma once

namespace {

template <int G>
struct small_shape {
    static constexpr int kMinBits = 8, kMaxBits = G == 8 ? 12 : 11;     // 128 KiB of codewords at most
};

// SHIFT makes kv non-negative for every codeword that is no farther than D, the smaller of the current codeword's distance and
// of a bound for the smallest one's, so a negative key marks codewords that cannot win.
template <int G, int NBITS>
__global__ __launch_bounds__(NBITS >= 10 ? 1024 : 1 << NBITS, G == 16 && NBITS == 8 ? 3 : 4) void k_search_small(
    const float *__restrict__ T, const float *__restrict__ cb, const float *__restrict__ scales,
    const int32_t *__restrict__ list, int k, int per_block, int nbatch, uint16_t *__restrict__ codes, unsigned long long *num_changed,
    unsigned long long *stats, pv_counts counts, unsigned *__restrict__ block_counts, int gpr, int N)
{
    constexpr int kCsize = 1 << NBITS, kWaves = NBITS >= 10 ? 16 : 1 << (NBITS - 6), kThreads = kWaves * 64;
    constexpr int kTiles = kCsize / 32 / kWaves;          // codeword tiles of a wave
    constexpr int kSu = kTiles / kU, kParts = 2 * kWaves;
    constexpr int kGroups = kCsize * G >= 1 << 15 ? 64 : 128;
    constexpr int kTeam = 8, kRecs = (kParts + kTeam - 1) / kTeam;
    static_assert(kTiles % kU == 0 && kGroups <= kThreads, "whole super-units; a thread a group");
    __shared__ pv_f4 s_cb[kCsize * (G / 4)];
    __shared__ h8 s_x[kGroups * (G == 8 ? 2 : 3)];        // operand B: x_hi, {-1, -1, -1, pieces of SHIFT}
    __shared__ pv_f4 s_meta[kGroups], s_t[kGroups * (G / 4)], s_tmp[kWaves];
    __shared__ float s_s[kGroups];
    __shared__ double s_oprev[kGroups];
    __shared__ int s_prev[kGroups], s_n[kGroups];
    __shared__ int s_rec[2][kParts][kGroups];
    __shared__ unsigned s_cnt[4];
    pv_counts_clear(counts);
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
            for (int v = 0; v < G / 4; ++v) s_cb[(row0 + 64 * i) * (G / 4) + v] = own[i][v];
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
            const pv_f4 cw = s_cb[(row0 + 64 * i) * (G / 4) + v];
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
                const float t = tgt[i >> 2][i & 3], c = s_cb[code * (G / 4) + (i >> 2)][i & 3];
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
    const int q = tid % kTeam, team_shift = lane & ~(kTeam - 1);
    for (int g = tid / kTeam; g < have; g += kThreads / kTeam) {
        const int ng = s_n[g];
        if (ng < 0) continue;                             // whole teams
        const pv_f4 m = s_meta[g];
        const float sg = s_s[g];
        const double o_prev = s_oprev[g];
        const int prev = s_prev[g];
        pv_f4 t[G / 4];                                   // (g = 16: from LDS as they are needed, the registers are short)
#pragma unroll
        for (int v = 0; v < G / 4; ++v) t[v] = G == 8 ? s_t[g * (G / 4) + v] : pv_f4{0.0f, 0.0f, 0.0f, 0.0f};
        cand_t mine;
        mine.obj = __builtin_huge_val();
        mine.idx = 0x7fffffff;
        unsigned evals = 0;
        auto exact_at = [&](int c) {
            double obj = 0.0;
#pragma unroll
            for (int v = 0; v < G / 4; ++v) {
                const pv_f4 cw = s_cb[c * (G / 4) + v], tv = G == 8 ? t[v] : s_t[g * (G / 4) + v];
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
            ++evals;
        };
        auto team_min = [&](cand_t c) {
            pv_team_stages<kTeam>([&](auto ctrl) {
                constexpr int C = decltype(ctrl)::value;
                const double o = pv_dpp_f64<C>(c.obj);
                const int i = pv_dpp<C>(c.idx);
                if (cand_better(o, i, c.obj, c.idx)) {
                    c.obj = o;
                    c.idx = i;
                }
            });
            return c;
        };
        // the codewords of super-unit su of partition p
        constexpr int kEvalUnroll = G == 8 ? kU : 1;
        auto eval_su = [&](int p, int su) {
#pragma unroll kEvalUnroll
            for (int uu = 0; uu < kU; ++uu)
#pragma unroll
                for (int e = 0; e < 16 / kTeam; ++e) {
                    const int qq = q + kTeam * e;
                    exact_at(((p >> 1) * kTiles + su * kU + uu) * 32 + 8 * (qq >> 2) + 4 * (p & 1) + (qq & 3));
                }
        };
        bool scanned = false;
        if (m.w < 0.0f) {                                 // not for the filter
            for (int c = q; c < kCsize; c += kTeam) exact_at(c);
            scanned = true;
        } else {
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
                eval_su(best_p, best_key & (int)kKeyMask);
                const double o = team_min(mine).obj;
                if (o < e_star) e_star = o;
            }
            // every codeword that was not evaluated and could still reach E* sits behind a key whose upper bound is at
            // least kcut (see rerank), and not behind a negative one
            const float p_over_s = P * fast_rcp(fabsf(sg));
            const float ef = float_above(e_star);
            const float rr = fast_sqrt(ef < 1.2e-38f ? 1.2e-38f : ef) * p_over_s * 1.000002f + kNormMargin + m.w;
            float r2 = rr * rr * 1.000002f;
            if (!(r2 == r2)) r2 = __builtin_huge_valf();
            const float base = m.x + m.y;
            const float kcut = (base * 0.999999f - r2 * 1.000001f) - m.z - 1.0e-6f * (base + r2);
            const bool no_bound = !(kcut > -3.0e38f);
            unsigned pending = 0;                         // bit u: the key of rec[u]; bit 16 + u: all of its partition
#pragma unroll
            for (int u = 0; u < kRecs; ++u) {
                if (rec[u].y >= 0 && (no_bound || key_upper(rec[u].y) >= kcut)) pending |= 1u << (16 + u);
                else if (rec[u].x >= 0 && q + kTeam * u != best_p && (no_bound || key_upper(rec[u].x) >= kcut)) pending |= 1u << u;
            }
            for (;;) {
                const unsigned long long pb = __ballot(pending != 0u);
                const unsigned team = (unsigned)((pb >> team_shift) & ((1ull << kTeam) - 1ull));
                if (!team) break;
                const int src = __ffs(team) - 1;          // lane of the team with work
                const int bit = __ffs(__shfl((int)pending, src, kTeam)) - 1, u = bit & 15;
                int key = 0;
#pragma unroll
                for (int uu = 0; uu < kRecs; ++uu)
                    if (uu == u) key = rec[uu].x;
                key = __shfl(key, src, kTeam);
                if (bit >= 16) {
                    for (int su = 0; su < kSu; ++su) eval_su(src + kTeam * u, su);
                    scanned = true;
                } else {
                    eval_su(src + kTeam * u, key & (int)kKeyMask);
                }
                if (q == src) pending &= ~(1u << bit);
            }
        }
        const cand_t win = team_min(mine);
        evals = pv_team_sum_u32<kTeam>(evals);
        if (q == 0) {
            int pick = win.idx;
            if (o_prev <= win.obj || pick == 0x7fffffff) pick = prev;
            if (pick != prev) {
                codes[ng] = (uint16_t)pick;
                atomicAdd(&s_cnt[1], 1u);
            }
            atomicAdd(&s_cnt[scanned ? 3 : 0], 1u);
            atomicAdd(&s_cnt[2], evals + 1u);
        }
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
    // codebook.  Blocks: what fits the chip at once (four waves a SIMD).
    const int most = (g << l->nbits) >= 1 << 15 ? 64 : 128;
    int per_block = (int)(((k + 255) / 256 + 31) & ~(int64_t)31);
    if (k > 256 * most) per_block = most;
    const int nbatch = (int)((k + per_block - 1) / per_block);
    const int slots = 256 * (l->nbits == 8 ? 4 : l->nbits == 9 ? 2 : 1);       // four waves a SIMD
    static_assert(4 * 256 <= kCountedBlocks, "a block's counters have a place");
    const int blocks = nbatch < slots ? nbatch : slots;
    ctx->rr_blocks_last = blocks;
    ctx->rr_counts = rr_counts;
    pv_timed t(ctx, PV_K_SCORE_MFMA);
    auto nc = reinterpret_cast<unsigned long long *>(num_changed);
#define PV_SMALL_CB(G_, B_)                                                                                          \
    case B_:                                                                                                      \
        hipLaunchKernelGGL((k_search_small<G_, B_>), dim3(blocks), dim3(B_ >= 10 ? 1024 : 1 << B_), 0, ctx->stream, T, codebook, scales, \
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
