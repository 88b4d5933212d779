// Nearest-codeword search that leaves out whole cells of the codebook (one codebook, g = 8).
//
// The weights that are re-encoded stand near a codeword already: the current one.  Its distance
// d_p = ||C[p] - x|| (x = t / s) bounds the distance of the nearest, so a codeword farther than
// d_p need not be scored.  The codebook is cut into cells by one threshold per dimension (two
// more for the last one of a 16-bit codebook): cell bit i says on which side of theta_i the i-th
// coordinate lies.  x is at least |x_i - theta_i| away from every codeword on the other side, so
//     LB(cell)^2 = sum over the bits in which x and the cell differ of (x_i - theta_i)^2
// is a lower bound for the whole cell, separable over the bits, and the cell is left out for the
// group when LB > d_p.  With 512 cells of about 128 codewords and an update of about the distance
// between neighbouring codewords a group keeps some 15 to 20 % of the cells.
//
// k_cells_stats   statistics of the codebook, thresholds (mean of a sample), cell of every
//                 codeword, number of codewords in each cell
// k_cells_prep    codewords placed cell by cell as fp16 operand rows, groups prepared
// k_cells_score   for each block of groups and each range of cells: which groups keep which
//                 cell, then the cell's codewords against those groups only
// Where the current code says little (codes drawn at random, a step of many codeword spacings) a
// group keeps most cells and the dense contraction is faster: k_cells_stats counts the cells that
// 64 groups spread over the list would keep, and above kDenseShare the table is laid out without
// padding and k_score_mfma contracts it, cut into splits as without cells (of the two kernels the one
// that is not needed returns at once; both ways in one kernel left too few registers to either).
// k_rerank        (pv_mfma.hip) decides from the records as it does for the dense contraction
//
// The accumulator is kv = R2 - ||c_hi - x_hi||^2 with R2 a little above (P d_p)^2: a negative kv
// marks a codeword that cannot win, so only non-negative keys are recorded, few of them.
#pragma once

namespace {

constexpr int kCellLog = 7;                   // log2 of the codewords a cell has on average
constexpr int kCellMinBits = 14;              // smallest codebook that is cut into cells
// Groups x codewords from which on cells are used.  Whole search (preparation, scoring, re-rank) against
// the dense contraction alone.  Update of about the codeword spacing: 16 bits 21k groups 77 against 84 us,
// 40k 85 against 114, 56k 87 against 145, 184k 188 against 435; 15 bits 66k 85 against 110; 14 bits 140k 110
// against 122; 13 bits 367k 231 against 243, fewer groups lose.  Current codes that say nothing, so that
// the dense contraction runs after all: 16 bits 40k 121 against 114, 56k 155 against 145, 184k 455 against
// 435; 15 bits 66k 118 against 110 (a launch that does nothing, and the cells' preparation).  The line lies
// above break-even of the first kind for the sake of the second.
constexpr int64_t kCellMinWork = INT64_C(1) << 31;
constexpr int kCellsMax = 1 << (16 - kCellLog);
constexpr int kCellPos = 32 * kU;             // a cell is padded to whole super-units
constexpr int kCellSample = kBlock;           // codewords behind the thresholds
constexpr float kPadNorm = 50000.0f;          // norm of a padding row (a codeword's is at most 8 * 32^2)
constexpr int kCellSuMax = (65536 + kCellsMax * (kCellPos - 1)) / kCellPos + 1;   // super-units of the padded table
constexpr int kCellWavesMax = 16;             // waves of a scoring block, at most
constexpr int kItemCells = 128;               // cells of a work item, at most
constexpr int kSampleGroups = kBlock / 4;     // groups that decide between cells and the dense contraction
constexpr float kDenseShare = 0.45f;          // share of the cells from which on the dense contraction is faster

// v_writelane_b32: lane `lane` of `old` replaced by a value that is the same for the whole wave
// (an LLVM intrinsic without a clang builtin; inline assembly would leave the wait states between a
// comparison and the reading of its result to chance).
extern "C" __device__ int pv_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

// Device scratch of the path (words).
struct cell_mem {
    pv_f4 *part;          // [kCbParts] {max |c|, min norm^2, max norm^2, bad}
    float *dpart;         // [kCbParts] largest rounding error ||P c - c_hi||^2 of a block's codewords
    float *theta;         // [16] thresholds 0..7, then the two outer ones of the last dimension; [15] != 0: dense
    unsigned *count;      // [copies][cells], zero between calls
    unsigned *cursor;     // [copies][cells]
    int *cell_su;         // [cells + 1] first super-unit of a cell
    uint16_t *cell_of;    // [codewords]
};
constexpr size_t kCellWords = kCbParts * 4 + kCbParts + 16 + kCbCopies * kCellsMax +
                              (kCellsMax + 8) + 65536 / 2;     // without `count`

// Bit i of a cell: the side of theta_i.  A 16-bit codebook has nine bits for eight dimensions: two of
// them say between which thresholds of dimension 7 the coordinate lies, and stand at bits 4 and 5, so
// that the splits (equal ranges of cells) differ in signs only and have the same share of the work.
__device__ __forceinline__ int cell_of_codeword(const float (&v)[8], const float *theta, int cbits)
{
    int side[8], cell = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) side[i] = v[i] >= theta[i] ? 1 : 0;
    if (cbits == 9) {
        const int interval = (v[7] >= theta[8] ? 1 : 0) + side[7] + (v[7] >= theta[9] ? 1 : 0);
        return side[0] | side[1] << 1 | side[2] << 2 | side[3] << 3 | interval << 4 | side[4] << 6 | side[5] << 7 | side[6] << 8;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) cell |= side[i] << i;
    return cell & ((1 << cbits) - 1);
}

// The squared lower bounds of one group (coordinates x, in units of theta): low four bits as a
// table, the sum over the others for each run of 16 cells.
struct cell_bounds {
    float low[16], c0[8], c1[8], q0, q1, q2, q3;
    int cbits;
    __device__ __forceinline__ void set(const float (&x)[8], const float *theta, float P, int bits)
    {
        cbits = bits;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float e = x[i] - P * theta[i];
            const float hi = fmaxf(e, 0.0f), lo = fminf(e, 0.0f);
            c0[i] = i < bits ? hi * hi : 0.0f;      // cost of the low side (bit 0)
            c1[i] = i < bits ? lo * lo : 0.0f;
        }
#pragma unroll
        for (int b = 0; b < 16; ++b)
            low[b] = ((b & 1 ? c1[0] : c0[0]) + (b & 2 ? c1[1] : c0[1])) +
                     ((b & 4 ? c1[2] : c0[2]) + (b & 8 ? c1[3] : c0[3]));
        const float a = P * theta[8], b = P * theta[7], c = P * theta[9];
        const float u0 = fmaxf(x[7] - a, 0.0f), u1 = fmaxf(fmaxf(a - x[7], x[7] - b), 0.0f);
        const float u2 = fmaxf(fmaxf(b - x[7], x[7] - c), 0.0f), u3 = fmaxf(c - x[7], 0.0f);
        q0 = u0 * u0;
        q1 = u1 * u1;
        q2 = u2 * u2;
        q3 = u3 * u3;
    }
    // run u holds the cells [16 u, 16 u + 16)   (values first, then the choice: a choice between
    // array elements would put the arrays into memory)
    static __device__ __forceinline__ float pick(int bit, float lo, float hi) { return bit ? hi : lo; }
    __device__ __forceinline__ float run(int u) const
    {
        const float a4 = c0[4], b4 = c1[4], a5 = c0[5], b5 = c1[5], a6 = c0[6], b6 = c1[6], a7 = c0[7], b7 = c1[7];
        if (cbits == 9)
            return pick(u & 2, pick(u & 1, q0, q1), pick(u & 1, q2, q3)) +
                   ((pick(u & 4, a4, b4) + pick(u & 8, a5, b5)) + pick(u & 16, a6, b6));
        return (pick(u & 1, a4, b4) + pick(u & 2, a5, b5)) + (pick(u & 4, a6, b6) + pick(u & 8, a7, b7));
    }
};

// Every block takes the same sample and so the same thresholds.  Results leave as plain stores
// per block (the next kernel adds up 64 of them; atomics of all blocks on one line took 3 us).
__global__ __launch_bounds__(kBlock) void k_cells_stats(const float *__restrict__ cb, int csize, int cbits,
                                                        cell_mem mem, clear_args ca, group_args ga)
{
    __shared__ float s_v[kCellSample * 9];          // row stride 9: conflict-free columns
    __shared__ float s_p[4][2][8];
    __shared__ float s_theta[16];
    __shared__ unsigned s_hist[kCellsMax];
    __shared__ pv_f4 s_tmp[kBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ncells = 1 << cbits;
    const pv_f4 *cb4 = reinterpret_cast<const pv_f4 *>(cb);
    pv_f4 smp[2];       // the codeword of the sample this thread fetches, requested before everything else
    {
        const int c = tid * (csize / kCellSample);
        smp[0] = cb4[c * 2];
        smp[1] = cb4[c * 2 + 1];
    }
    // The last block looks at the groups: thread (sample j, quarter of the cells).
    const bool sampler = blockIdx.x == gridDim.x - 1;
    float sx[8], sreach = -1.0f;
    if (sampler) {
        const int per = ga.k / kSampleGroups;
        const int n = per > 0 || (tid >> 2) < ga.k ? ga.group_idx[(int64_t)(tid >> 2) * (per > 0 ? per : 1)] : -1;
#pragma unroll
        for (int i = 0; i < 8; ++i) sx[i] = 0.0f;
        if (n >= 0 && n < ga.N) {
            const pv_f4 *t4 = reinterpret_cast<const pv_f4 *>(ga.T + (int64_t)n * 8);
            const pv_f4 t0 = t4[0], t1 = t4[1];
            const float inv = 1.0f / ga.scales[n / ga.gpr];
            const int64_t c = (int)ga.codes[n] & ga.csize_mask;
            const pv_f4 c0 = cb4[c * 2], c1 = cb4[c * 2 + 1];
            sreach = 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                sx[i] = (i < 4 ? t0[i & 3] : t1[i & 3]) * inv;
                const float d = (i < 4 ? c0[i & 3] : c1[i & 3]) - sx[i];
                sreach = fmaf(d, d, sreach);
            }
        }
    }
    // the block's codewords are requested first, they arrive while the sample is worked on
    pv_f4 own[4][2];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = (sampler ? 0 : blockIdx.x) * kCbChunk + r * kBlock + tid;   // csize is a multiple of kCbChunk
        own[r][0] = cb4[c * 2];
        own[r][1] = cb4[c * 2 + 1];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) s_v[tid * 9 + e] = smp[e >> 2][e & 3];
    clear_counters(ca, blockIdx.x, gridDim.x);
    for (int i = blockIdx.x * kBlock + tid; i < kCbCopies * ncells; i += gridDim.x * kBlock) mem.cursor[i] = 0u;
    for (int b = tid; b < ncells; b += kBlock) s_hist[b] = 0u;
    __syncthreads();
    {
        // thread (dimension d, run of 8 rows): sum and sum of squares
        const int d = tid & 7, row = (tid >> 3) * 8;
        float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float v = s_v[(row + i) * 9 + d];
            s1 += v;
            s2 = fmaf(v, v, s2);
        }
#pragma unroll
        for (int off = 8; off < 64; off <<= 1) {
            s1 += __shfl_xor(s1, off);
            s2 += __shfl_xor(s2, off);
        }
        if (lane < 8) {
            s_p[wave][0][lane] = s1;
            s_p[wave][1][lane] = s2;
        }
    }
    __syncthreads();
    if (tid < 8) {
        const float inv = 1.0f / kCellSample;
        const float m = (s_p[0][0][tid] + s_p[1][0][tid] + s_p[2][0][tid] + s_p[3][0][tid]) * inv;
        const float q = (s_p[0][1][tid] + s_p[1][1][tid] + s_p[2][1][tid] + s_p[3][1][tid]) * inv;
        // any finite thresholds are right, these balance the cells of a bell-shaped codebook
        const float t = m == m && fabsf(m) < 3.0e37f ? m : 0.0f;
        s_theta[tid] = t;
        if (tid == 7) {
            float w = 0.6745f * sqrtf(fmaxf(q - m * m, 0.0f));
            if (!(w < 3.0e37f)) w = 0.0f;
            s_theta[8] = t - w;
            s_theta[9] = t + w;
        }
    }
    __syncthreads();
    if (sampler) {
        if (tid < 10) mem.theta[tid] = s_theta[tid];
        cell_bounds lb;
        lb.set(sx, s_theta, 1.0f, cbits);
        const int runs = ncells / 16;
        unsigned kept = 0;
        for (int u = tid & 3; u < runs; u += 4) {
            const float room = sreach - lb.run(u);
#pragma unroll
            for (int b = 0; b < 16; ++b) kept += lb.low[b] <= room;
        }
        // (a group that the filter does not take, or whose distance is not a number, keeps nothing here)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) kept += __shfl_xor(kept, off);
        if (lane == 0) s_tmp[wave].x = (float)kept;
        __syncthreads();
        if (tid == 0) {
            const float all = s_tmp[0].x + s_tmp[1].x + s_tmp[2].x + s_tmp[3].x;
            mem.theta[15] = all > kDenseShare * (float)ncells * kSampleGroups ? 1.0f : 0.0f;
        }
        return;
    }
    cb_stat st;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        stat_add<8>(st, own[r]);
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = own[r][i >> 2][i & 3];
        const int cell = cell_of_codeword(v, s_theta, cbits);
        mem.cell_of[blockIdx.x * kCbChunk + r * kBlock + tid] = (uint16_t)cell;
        atomicAdd(&s_hist[cell], 1u);
    }
    const pv_f4 p = stat_block(st, s_tmp);      // its barrier also ends the counting
    if (tid == 0) mem.part[blockIdx.x] = p;
    unsigned *count = mem.count + (blockIdx.x % kCbCopies) * ncells;
    for (int b = tid; b < ncells; b += kBlock) {
        const unsigned v = s_hist[b];
        if (v) atomicAdd(&count[b], v);
    }
}

// Blocks [0, cb_blocks): the chunk of codewords that the same block counted is placed: the
// cell's first super-unit, then the codewords of the copies before this one, then those that
// blocks of this copy placed already, then the rank inside the block.  The order inside a cell
// is of no consequence.  Remaining blocks: one thread per selected group (prep_group).
__global__ __launch_bounds__(kBlock) void k_cells_prep(const float *__restrict__ cb, int csize, int cbits,
                                                       int cb_blocks, cell_mem mem,
                                                       unsigned *__restrict__ meta, h8 *__restrict__ A,
                                                       uint16_t *__restrict__ perm,
                                                       int *__restrict__ su_bounds, int nsplit,
                                                       int dense_splits, group_args ga)
{
    __shared__ unsigned s_meta[8];
    meta_of_parts(mem.part, csize / kCbChunk, s_meta);
    bool ok;
    const float P = scale_from_maxabs(s_meta[0], &ok);
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= cb_blocks) {
        const int j = ((int)blockIdx.x - cb_blocks) * kBlock + tid;
        if (j < ga.k_pad) prep_group<8, true>(ga, j, P, ok && s_meta[3] == 0u && s_meta[1] != 0u, s_meta);
        return;
    }
    constexpr int kPadCells = kCbChunk >> kCellLog;
    __shared__ unsigned s_cnt[kCellsMax], s_base[kCellsMax], s_w[kBlock / 64], s_pad[kPadCells][2];
    const int ncells = 1 << cbits, lane = tid & 63, wave = tid >> 6;
    const int copy = blockIdx.x % kCbCopies;
    const bool dense = mem.theta[15] != 0.0f;   // cells follow one another without padding
    int cell[4];
    unsigned rank[4];
    pv_f4 own[4][2];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = blockIdx.x * kCbChunk + r * kBlock + tid;
        cell[r] = mem.cell_of[c];
        own[r][0] = reinterpret_cast<const pv_f4 *>(cb)[c * 2];
        own[r][1] = reinterpret_cast<const pv_f4 *>(cb)[c * 2 + 1];
    }
    for (int b = tid; b < ncells; b += kBlock) s_cnt[b] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) rank[r] = atomicAdd(&s_cnt[cell[r]], 1u);
    // two cells a thread: their codewords, in all copies and in the copies before this one
    unsigned all[2] = {0u, 0u}, before[2] = {0u, 0u};
    {
        unsigned v[kCbCopies][2];
#pragma unroll
        for (int q = 0; q < kCbCopies; ++q)
#pragma unroll
            for (int e = 0; e < 2; ++e) v[q][e] = 2 * tid + e < ncells ? mem.count[q * ncells + 2 * tid + e] : 0u;
#pragma unroll
        for (int q = 0; q < kCbCopies; ++q)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                before[e] += q < copy ? v[q][e] : 0u;
                all[e] += v[q][e];
            }
    }
    // room of the cells, in positions: whole super-units
    unsigned room[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) room[e] = dense ? all[e] : (all[e] + kCellPos - 1) / kCellPos * kCellPos;
    unsigned inc = room[0] + room[1];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned u = __shfl_up(inc, off);
        if (lane >= off) inc += u;
    }
    if (lane == 63) s_w[wave] = inc;
    __syncthreads();
    unsigned first = inc - room[0] - room[1];
    for (int w = 0; w < wave; ++w) first += s_w[w];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int b = 2 * tid + e;
        if (b < ncells) {
            const unsigned start = first + (e ? room[0] : 0u), end = start + room[e];
            const unsigned mine = s_cnt[b];
            unsigned at = start + before[e];
            if (mine) at += atomicAdd(&mem.cursor[copy * ncells + b], mine);
            s_base[b] = at;
            if (blockIdx.x == 0 && !dense) {
                mem.cell_su[b] = (int)(start / kCellPos);
                if (b == ncells - 1) mem.cell_su[ncells] = (int)(end / kCellPos);
            }
            // the padding rows of every cb_blocks-th cell are this block's
            if (b % cb_blocks == (int)blockIdx.x) {
                s_pad[b / cb_blocks][0] = start + all[e];
                s_pad[b / cb_blocks][1] = end;
            }
            // splits: ranges of runs of 16 cells, or of residue cycles of the dense table
            if (blockIdx.x == 0 && (b & 15) == 0 && !dense)
                for (int i = 0; i < nsplit; ++i)
                    if (split_begin(i, ncells / 16, nsplit) == b / 16) su_bounds[i] = (int)(start / kCellPos);
            if (blockIdx.x == 0 && b == ncells - 1 && !dense) su_bounds[nsplit] = (int)(end / kCellPos);
        }
    }
    if (blockIdx.x == 0 && dense && tid <= dense_splits)
        su_bounds[tid] = split_begin(tid, csize / (kCellPos * kResidues), dense_splits) * kResidues;
    if (blockIdx.x == 0 && tid < 8) meta[tid] = s_meta[tid];
    __syncthreads();
    // cb_blocks = csize / kCbChunk blocks share csize / 2^kCellLog cells: kCbChunk / 2^kCellLog each
    for (int i = tid; i < kPadCells * kCellPos; i += kBlock) {
        const unsigned pos = s_pad[i / kCellPos][0] + i % kCellPos;
        if (pos < s_pad[i / kCellPos][1]) {
            h8 c0, c1;
#pragma unroll
            for (int e = 0; e < 8; ++e) c0[e] = c1[e] = (_Float16)0.0f;
            c1[0] = (_Float16)kPadNorm;
            c1[3] = c1[4] = c1[5] = (_Float16)1.0f;
            const operand_row o = operand_row_of((int)pos);
            A[((int64_t)o.tile * 2 + 0) * 32 + o.row] = c0;
            A[((int64_t)o.tile * 2 + 1) * 32 + o.row] = c1;
            perm[pos] = 0;
        }
    }
    float d2 = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = blockIdx.x * kCbChunk + r * kBlock + tid;
        const int pos = (int)(s_base[cell[r]] + rank[r]);
        h8 chunk[2];
        float n2 = 0.0f, d2c = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float v = ok ? P * own[r][i >> 2][i & 3] : 0.0f;
            const float hf = (float)to_half_flush(v);
            n2 = fmaf(hf, hf, n2);
            const float d = v - hf;
            d2c = fmaf(d, d, d2c);
            chunk[0][i] = (_Float16)(2.0f * hf);
            chunk[1][i] = (_Float16)0.0f;
        }
        d2 = fmaxf(d2, d2c);
        _Float16 pieces[3];
        split3(n2, pieces);
        chunk[1][0] = pieces[0];
        chunk[1][1] = pieces[1];
        chunk[1][2] = pieces[2];
        chunk[1][3] = chunk[1][4] = chunk[1][5] = (_Float16)1.0f;
        const operand_row o = operand_row_of(pos);
#pragma unroll
        for (int u = 0; u < 2; ++u) A[((int64_t)o.tile * 2 + u) * 32 + o.row] = chunk[u];
        perm[pos] = (uint16_t)c;
    }
    __shared__ float s_d[kBlock / 64];
    d2 = wave_max_f(d2);
    if (lane == 0) s_d[wave] = d2;
    __syncthreads();
    if (tid == 0) mem.dpart[blockIdx.x] = fmaxf(fmaxf(s_d[0], s_d[1]), fmaxf(s_d[2], s_d[3]));
}

// One work item: the groups of a block (one a thread) x the cells of one split.
// 1. Every thread takes one group: its operand goes to LDS, the cells it keeps become bits of
//    s_mask (a ballot per cell).
// 2. The bits of each cell become a list of groups, all lists one after the other in LDS (as many
//    cells at a time as there is room for).
// 3. The waves take the super-units of those cells one by one and contract each with 32 listed
//    groups at a time: operand B gathered from LDS, operand A from the L2, one super-unit ahead.
//    A key goes to the group's record by LDS maxima if it is above the second largest there: few
//    lanes have one.
// 4. The records leave: partition = (split, half wave, parity of the super-unit).
// No unit is full: for the Adam step below, vector-ALU issue takes 58 of 109 thousand cycles (14.9 M
// instructions), the LDS 33, the matrix cores 17; the rest are waits at the start of a list and at the
// two barriers of an item.  What a list costs is spread over more groups the larger the block is: up to 16 waves (the launch picks
// the number that fills the chip), one block per compute unit.  56 360 groups, 16 bits: 75 us where the
// update is the codeword spacing of the widest groups (35 us for an Adam step, whose updates are more even)
// against 122 us for the dense contraction.
__global__ __launch_bounds__(kCellWavesMax * 64, kCellWavesMax / 4) void k_cells_score(
    const h8 *__restrict__ A, const h8 *__restrict__ X, const float *__restrict__ reach,
    const int *__restrict__ su_bounds, cell_mem mem, unsigned *__restrict__ meta, int2 *__restrict__ partials,
    int cbits, int cb_parts, int nsplit, int gblocks, int k_pad, unsigned *__restrict__ next_item)
{
    constexpr int kGroupsMax = kCellWavesMax * 64;
    constexpr int kRec = kGroupsMax + 32;               // the group that fills lists up has a record too
    constexpr int kSets = kItemCells / 64;
    constexpr int kListRoom = 24576;                    // entries of all lists together
    static_assert(kCellWavesMax <= 16, "a row of s_share");
    static_assert(kListRoom >= kGroupsMax && kListRoom / 32 <= 1024 && kGroupsMax / 32 < 64, "a list's place and length fit 16 bits");
    __shared__ h8 s_x[(kGroupsMax + 1) * 2];
    __shared__ int s_rec[2][4 * kRec];                  // largest, second largest key: [half wave][parity][group]
    __shared__ uint16_t s_list[kListRoom + 64];         // the last 64: where lanes without an entry write
    __shared__ __attribute__((aligned(16))) uint16_t s_share[kItemCells][16];   // a cell's groups in each wave, then in the waves before
    __shared__ int s_su[kItemCells + 1], s_off[kItemCells], s_cnt[kItemCells];
    __shared__ uint16_t s_unit[kCellSuMax];             // a super-unit's list: place / 32 << 6 | length / 32
    __shared__ int s_next, s_item, s_until;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ncells = 1 << cbits, runs = ncells / 16, waves = blockDim.x >> 6, groups = blockDim.x;
    if (mem.theta[15] != 0.0f) return;      // dense: k_score_mfma does the work, and what follows
    // the counts are done with: zero for the next call; the largest rounding error of the codebook
    for (int i = blockIdx.x * groups + tid; i < kCbCopies * ncells; i += gridDim.x * groups) mem.count[i] = 0u;
    if (blockIdx.x == 0 && tid < 64) {
        const float d = wave_max_f(tid < cb_parts ? mem.dpart[tid] : 0.0f);
        if (tid == 0) meta[2] = __float_as_uint(d);
    }
    if (tid < 2) {   // the filling group: its kv are all negative
        h8 z;
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = (_Float16)(tid == 1 && e < 4 ? -1.0f : 0.0f);
        s_x[kGroupsMax * 2 + tid] = z;
    }
    bool okP;
    const float P = scale_from_maxabs(meta[0], &okP);
    unsigned vmask = ~kKeyMask;
    asm volatile("" : "+v"(vmask));   // keep the mask in a vector register
    const unsigned items = (unsigned)gblocks * (unsigned)nsplit;
    // the next item number (past the end when there are no more); every wave is done with the LDS by then
    auto next = [&]() -> unsigned {
        if (items <= gridDim.x) return items;
        __syncthreads();
        if (tid == 0) s_item = (int)(gridDim.x + atomicAdd(next_item, 1u));
        __syncthreads();
        return (unsigned)s_item;
    };
    for (unsigned item = blockIdx.x; item < items;) {
        const int gb = (int)(item % (unsigned)gblocks), split = (int)(item / (unsigned)gblocks);
        const int su0 = su_bounds[split], su1 = su_bounds[split + 1];
        const int run0 = split_begin(split, runs, nsplit), nruns = split_count(split, runs, nsplit);
        const int per = nruns * 16;
        unsigned mlo[kSets], mhi[kSets];                // lane i: which of the wave's groups keep cell q * 64 + i
        {
            const int j = gb * groups + tid;
            const int64_t xa = (int64_t)(j >> 5) * 64 + (j & 31);
            const h8 x0 = X[xa], x1 = X[xa + 32];
            const float r2 = reach[j];
            s_x[tid * 2] = x0;
            s_x[tid * 2 + 1] = x1;
#pragma unroll
            for (int q = 0; q < 4; ++q) s_rec[0][q * kRec + tid] = s_rec[1][q * kRec + tid] = -1;
            {
                if (tid <= per) s_su[tid] = mem.cell_su[run0 * 16 + tid];
                float x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = (float)x0[i];
                cell_bounds lb;
                lb.set(x, mem.theta, P, cbits);
#pragma unroll
                for (int q = 0; q < kSets; ++q) {
                    int lo = 0, hi = 0;
                    for (int r = 0; r < 4 && q * 4 + r < nruns; ++r) {
                        const float room = r2 - lb.run(run0 + q * 4 + r);
#pragma unroll
                        for (int b = 0; b < 16; ++b) {
                            const unsigned long long m = __ballot(lb.low[b] <= room);
                            lo = pv_writelane((int)m, r * 16 + b, lo);
                            hi = pv_writelane((int)(m >> 32), r * 16 + b, hi);
                        }
                    }
                    mlo[q] = (unsigned)lo;
                    mhi[q] = (unsigned)hi;
                    s_share[q * 64 + lane][wave] = (uint16_t)(__popc(mlo[q]) + __popc(mhi[q]));
                }
            }
        }
        __syncthreads();
        for (int from = 0; from < per;) {
            if (wave == 0) {
                int until = per, at = 0;
                {
                    // lists' lengths and places (whole 32s), one cell a lane; how many cells fit
#pragma unroll
                    for (int q = 0; q < kSets; ++q) {
                        const int c = q * 64 + lane;
                        unsigned n = 0;
                        if (from == 0) {
                            const uint4 *row = reinterpret_cast<const uint4 *>(s_share[c]);
                            uint4 v[2] = {row[0], row[1]};
                            unsigned *p = reinterpret_cast<unsigned *>(v);
#pragma unroll
                            for (int w = 0; w < 8; ++w) {      // counts -> sums of the waves before
                                const unsigned n0 = 2 * w < waves ? p[w] & 0xFFFFu : 0u, n1 = 2 * w + 1 < waves ? p[w] >> 16 : 0u;
                                p[w] = n | (n + n0) << 16;
                                n += n0 + n1;
                            }
                            reinterpret_cast<uint4 *>(s_share[c])[0] = v[0];
                            reinterpret_cast<uint4 *>(s_share[c])[1] = v[1];
                            s_cnt[c] = (int)(c < per ? n : 0u);
                        }
                        const int len = c >= from && c < per ? (s_cnt[c] + 31) & ~31 : 0;
                        int inc = len;
#pragma unroll
                        for (int off = 1; off < 64; off <<= 1) {
                            const int u = __shfl_up(inc, off);
                            if (lane >= off) inc += u;
                        }
                        s_off[c] = at + inc - len;
                        const unsigned long long over = __ballot(at + inc > kListRoom);
                        if (over) {
                            const int first = q * 64 + __ffsll((long long)over) - 1;
                            until = first < until ? first : until;
                        }
                        at += __shfl(inc, 63);
                    }
                }
                if (lane == 0) {
                    s_until = until;
                    s_next = s_su[from] + 2 * waves;     // wave w starts with the w-th and (waves + w)-th
                }
            }
            __syncthreads();
            const int until = s_until;
            {
                // a thread writes its group into the lists of the cells it keeps
#pragma unroll
                for (int q = 0; q < kSets; ++q) {
                    const int c = q * 64 + lane;
                    const bool in = c >= from && c < until;
                    const unsigned lo = in ? mlo[q] : 0u, hi = in ? mhi[q] : 0u;
                    const unsigned place = in ? (unsigned)(s_off[c] + s_share[c][wave]) : 0u;
                    // eight cells at a time without a branch: a lane without an entry writes past the lists
                    for (int i = 0; i < 64 && q * 64 + i < until; i += 8)
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const unsigned l = __builtin_amdgcn_readlane(lo, i + e), h = __builtin_amdgcn_readlane(hi, i + e);
                            const unsigned at = __builtin_amdgcn_readlane(place, i + e);
                            const unsigned pos = __builtin_amdgcn_mbcnt_hi(h, __builtin_amdgcn_mbcnt_lo(l, at));
                            s_list[__builtin_amdgcn_inverse_ballot_w64(((unsigned long long)h << 32) | l) ? pos : kListRoom + lane] =
                                (uint16_t)tid;
                        }
                }
                // ... the last 32 of every list filled up, the super-units' lists noted: 16 lanes a cell
                for (int c = from + wave * 4 + (lane >> 4); c < until; c += waves * 4) {
                    const int off = s_off[c], n = s_cnt[c], len = (n + 31) & ~31, b = s_su[c], e = s_su[c + 1];
                    for (int i = n + (lane & 15); i < len; i += 16) s_list[off + i] = (uint16_t)kGroupsMax;
                    for (int i = b + (lane & 15); i < e; i += 16) s_unit[i - su0] = (uint16_t)((off >> 5) << 6 | len >> 5);
                }
                __syncthreads();
            }
            const int last = s_su[until];
            const unsigned fill = kGroupsMax;
            h8 a0, a1, n0, n1;
            int su = s_su[from] + wave, sn = su + waves;
            unsigned unit = 0, e0 = fill, e1 = fill, e2 = fill;      // list of the super-unit at hand and its first entries
            auto load_a = [&](int i, h8 &p, h8 &q) {
                p = A[(int64_t)(i * 2) * 64 + lane];
                q = A[(int64_t)(i * 2 + 1) * 64 + lane];
            };
            auto first_entries = [&] {
                const uint16_t *l = s_list + (unit >> 6) * 32 + col;
                const unsigned nb = unit & 63u;
                e0 = nb > 0 ? l[0] : fill;
                e1 = nb > 1 ? l[32] : fill;
                e2 = nb > 2 ? l[64] : fill;
            };
            // Contracts super-unit su with operand rows (x0, x1) and requests the next one's (y0, y1).
            // Called with the two pairs of registers in turn: a copy from one to the other would wait
            // for the loads.
            auto contract = [&](const h8 &x0, const h8 &x1, h8 &y0, h8 &y1) {
                unsigned unit_n = 0;
                if (sn < last) {
                    load_a(sn, y0, y1);
                    unit_n = s_unit[sn - su0];
                }
                int s2 = 0;
                if (lane == 0) s2 = __hip_atomic_fetch_add(&s_next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const int nb = __builtin_amdgcn_readfirstlane(unit & 63u);
                const uint16_t *list = s_list + (unit >> 6) * 32 + col;
                const f16v z = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                const int rec = (half * 2 + ((su - su0) & 1)) * kRec;
                // r: the group's place among the records of this half wave and parity
                auto close = [&](const f16v &p, const f16v &q, int *r, int low) {
                    const int run = acc_max<false>(q, acc_max<true>(p, kNoKey));
                    const int key = and_or(run, vmask, (unsigned)su);
                    if (key > low) {
                        const int old = atomicMax(r, key);
                        atomicMax(r + 4 * kRec, old < key ? old : key);
                    }
                };
                auto place = [&](unsigned g) { return &s_rec[0][rec + g]; };
                // list entries are read two steps ahead, operands and records one; past the list's
                // end the filling group stands in
                h8 b0 = s_x[e0 * 2 + half], b1 = s_x[e1 * 2 + half];
                int *r0 = place(e0), *r1 = place(e1);
                int l0 = r0[4 * kRec], l1 = r1[4 * kRec];
                unsigned g2 = e2, g1;
                f16v p0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0, b0, z, 0, 0, 0);
                f16v p1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1, b0, z, 0, 0, 0);
                for (int b = 1; b < nb; b += 2) {
                    const f16v q0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0, b1, z, 0, 0, 0);
                    const f16v q1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1, b1, z, 0, 0, 0);
                    b0 = s_x[g2 * 2 + half];
                    g1 = b + 2 < nb ? (unsigned)list[(b + 2) * 32] : fill;
                    close(p0, p1, r0, l0);
                    r0 = place(g2);
                    l0 = r0[4 * kRec];
                    p0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0, b0, z, 0, 0, 0);
                    p1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1, b0, z, 0, 0, 0);
                    b1 = s_x[g1 * 2 + half];
                    g2 = b + 3 < nb ? (unsigned)list[(b + 3) * 32] : fill;
                    close(q0, q1, r1, l1);
                    r1 = place(g1);
                    l1 = r1[4 * kRec];
                }
                unit = unit_n;
                first_entries();
                close(p0, p1, r0, l0);
                su = sn;
                sn = __builtin_amdgcn_readfirstlane(s2);
            };
            if (su < last) {
                load_a(su, a0, a1);
                unit = s_unit[su - su0];
                first_entries();
            }
            while (su < last) {
                contract(a0, a1, n0, n1);
                if (su >= last) break;
                contract(n0, n1, a0, a1);
            }
            from = until;
            if (from < per) __syncthreads();
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int b1 = s_rec[0][q * kRec + tid], b2 = s_rec[1][q * kRec + tid];
            partials[rec_at(split * 4 + q, (int64_t)gb * groups + tid, nsplit * 4, k_pad)] =
                make_int2(b1 < 0 ? kNoKey : b1, b2 < 0 ? kNoKey : b2);
        }
        item = next();
    }
}

}  // namespace
