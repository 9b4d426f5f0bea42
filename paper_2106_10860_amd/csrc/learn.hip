// The learning step on the GPU: the greedy construction of the hashing trees (Section 4.2,
// Algorithm 2; Appendix C, Algorithms 3 and 4) and the prototypes (bucket means; ridge
// regression, Section 4.3).  Set-up work, run once per problem; what matters here is that
// it takes milliseconds instead of seconds and that its decisions can be checked.
//
// Every decision is the one that fp64 sums with the operations in the order Algorithms 2-4 state
// them lead to - sums over the rows of a bucket sequentially in sorted (or row) order, sums over the
// columns of the subspace in column order - so that the trees are reproducible to the bit and
// do not depend on the launch shape.  Most decisions are made by estimates, sums in any order by all
// threads with a bound of what both can be off; those that are closer than that, and all where
// rows are few, by the sums themselves.  There the parallelism is ACROSS the independent pieces:
// codebooks, candidate columns, buckets and columns.  This file is compiled without floating-point
// contraction.
//
// The serial parts are sums in a given order: chains of additions at the adder's latency over
// operands that other wavefronts have laid side by side in LDS (or no chain, where a sum's bits
// allow any order); products, divisions, comparisons and counting are left to all threads or to
// wavefront ballots.
//
// gather_columns_kernel  the columns of every codebook side by side, rows aligned
// Per level t = 1..4 of all C trees at once:
//   order_rows_kernel    the rows of every bucket listed in row order, the bucket sizes
//   loss_parts_kernel, select_kernel  heuristic_select_idxs by estimates: the four columns with the largest summed loss
//   bucket_loss_kernel   L(j, B) (Section 4.2) for every column j of every bucket, two passes
//                        over the bucket's own rows (the exact losses, where the estimates are unsure)
//   sort_few_kernel, sort_round_kernel, or sort_count_kernel and sort_scatter_kernel  the rows ordered by each candidate column (radix
//                        sort of (value, row) keys: equal values stay in row order)
//   tile_sums_kernel, scan_groups_kernel, split_gains_kernel, choose_by_gain_kernel  Algorithm 3 for every bucket and
//                        Algorithm 2's choice among the candidates by estimates
//   split_chains_kernel (split_chains_small_kernel), split_losses_kernel, choose_kernel  the same where those are unsure:
//                        Algorithm 4's running sums at every 32nd row in both directions, the loss of every split, a
//                        wavefront per 256 rows, the best threshold and loss per bucket
//   apply_kernel         apply_split: the next level's buckets
// Prototypes: cooccurrence_kernel (G^T G), count_codes_kernel, list_codes_kernel and gta_kernel (G^T A~),
// cholesky_panel_kernel, transpose_factor_kernel (the factor by columns), substitution_kernel; or means_kernel.
#include "common.h"
#include "device_common.h"
#include "learn_bounds.h"

namespace maddness {
namespace {

constexpr int kSplitBuckets = 8;   // buckets of the deepest level that is split (level 4 splits 8)
constexpr int kCand = 4;           // candidate columns per level (Section 4.2: n = 4)

struct Bounds {
    int32_t v[2 * MADDNESS_MAX_C];
};

struct LearnArgs {
    const float *A;
    int64_t lda, N;
    int32_t C, dmax;
    int32_t *bounds;      // [C][2] first and one-past-last column of every codebook
    int32_t pitch;        // values of a row of X: dmax rounded up to whole groups of columns
    float *X;             // [C][N + 1][pitch] the codebook's columns of A, then zeros; row N is zeros
    uint8_t *node;        // [C][N] bucket (0-based) of every row in the current level
    double *col_loss;     // [C][8][dmax] L(j, B_i)
    int64_t *bucket_count;  // [C][8]
    int32_t *bucket_start;  // [C][8] where the bucket's rows begin in rows_by_bucket[c]
    int32_t *chunk_count;   // [4][C][kMaxChunks][8] rows of every bucket in every chunk of rows, by level
    int32_t *range_part;  // [C][kRangeParts][2] what a part of the codebook's values span, see any_order()
    int32_t *range;       // [C][2] and what all of them do
    int32_t row_bits;     // N <= 2^row_bits
    uint32_t *varying_part;  // [C][kRangeParts][pitch] the bits in which a part of a column's values differ from its first row's, see gather_columns_kernel and SortDigits
    uint32_t *varying;    // [C][pitch] and in which any of them do
    uint32_t *cand_varying;  // [C][4] those of the candidates
    int32_t look;         // whether the sort goes by them; else by all bits
    int32_t gather_parts; // parts of both that there are
    int32_t *rows_by_bucket;  // [C][N] the rows of bucket 0 in row order, then those of bucket 1, ...
    int32_t *cand;        // [C][4] candidate columns (within the subspace), best first
    int32_t *n_cand;      // [C]
    uint64_t *keys;       // [C][4][N] sorted (value, row) keys
    uint64_t *keys2;      // [C][4][N] the same between digits
    uint32_t *digit_counts;  // [C][4][kMaxSortChunks][kSortBins] keys of every digit in every chunk
    int64_t tile_slots;   // tiles of kSplitRows sorted rows of all buckets of a level, at most
    double *sums;         // [C][4][2][tile_slots][2][dmax] Algorithm 4's running sums before every tile, up and down
    int64_t group_slots;  // groups of kGroupTiles tiles of all buckets of a level, at most
    // what the estimates leave (the tiles' sums lie in `sums`, [C][4][2 tile_slots][2 dmax] or less of it, as [slot][dmax])
    int64_t part_slots;   // parts of kPartRows rows of all buckets of a level, at most
    double *parts;        // [C][part_slots][3][dmax] of a part's values x, the pivot taken off (y): sum y, sum y^2, sum x^2
    int32_t *original;    // [C][dmax] the column that a column is a copy of in all rows, as far as that has been found out; itself
    int64_t *may_compare; // [C] rows that columns may still be compared in (2.5 ns each, less where a row is few columns; a level's exact sums 13)
    double *energy;       // [C][8] the sum of the squares of a bucket's values, or a little more
    int32_t *exact_levels;   // [C][2] on how many levels exact sums chose the candidates, and the split among theirs
    int32_t *unsure;      // [C][2] whether the candidates take exact sums to tell; bit q: whether candidate q's split does, and flags
    double *group_sums;   // [C][4][group_slots][dmax] the sums of the rows of a bucket before every group
    double *totals;       // [C][4][8][dmax] and of all its rows
    double *group_gain;   // [C][4][group_slots][2] the largest gain of a split in the group (-1: no split), the second largest
    int32_t *group_first; // [C][4][group_slots] the bucket's row that the best one comes after
    double *group_loss;   // [C][4][group_slots] loss of the group's best split
    int32_t *group_at;    // [C][4][group_slots][2] the bucket's row it comes after (-1: none); the group's first split
                          // if its loss is not a number (else -1)
    int32_t *chosen;      // [C] the level's column (within the subspace)
    int32_t *split_dims;  // out [C][4]
    float *thresholds;    // out [C][16]
    uint8_t *codes;       // out [N][codes_pitch] or null
    int32_t codes_pitch;
};

// What a.unsure[2 c + 1] holds beside a bit per candidate: the comparison of those takes the bucket's exact losses, which have
// not been summed for the choice of columns; the level's splits have no estimates.
constexpr int kAllCand = (1 << kCand) - 1, kWantsLosses = 1 << kCand, kNoEstimates = 2 << kCand;

__global__ void upload_bounds_kernel(const Bounds b, int32_t n, int32_t *dst)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = b.v[i];
}

__global__ void begin_trees_kernel(const Bounds b, const LearnArgs a, bool estimated)
{
    for (int i = threadIdx.x; i < 2 * a.C; i += blockDim.x) {
        a.bounds[i] = b.v[i];
        a.exact_levels[i] = estimated ? 0 : 4;
        if (!estimated) a.unsure[i] = kAllCand;
    }
}

__global__ void clear_kernel(int32_t *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Sums whose bits allow any order.  Where all values of a codebook are multiples of one power of two, 2^l, and below another,
// 2^t, their sums and the sums of their squares over all rows are exact in fp64 as long as 2 (t - l) + log2(N) <= 53, in
// whatever order they are taken: images, counts, quantised features.  (One bit more of t - l is asked for, so that the same
// holds of differences of two values.)  range[c]: the largest t as an exponent over that of the smallest fp32 number, and
// kLeast - l; both 0 where all values are zeros.
constexpr int kLeast = 512, kNoNumber = 1 << 20, kRangeParts = 256;
__device__ __forceinline__ bool any_order(const LearnArgs &a, int c)
{
    const int top = a.range[2 * c], width = top + a.range[2 * c + 1] - kLeast;
    return top == 0 || 2 * (width + 1) + a.row_bits <= 53;
}

__device__ __forceinline__ void span_of(float x, int &top, int &least)
{
    const uint32_t bits = __float_as_uint(x) & 0x7fffffffu, field = bits >> 23;
    if (bits == 0) return;
    const int e = field ? (int)field : 1;
    const uint32_t m = (bits & 0x7fffffu) | (field ? 0x800000u : 0u);
    top = max(top, field == 255 ? kNoNumber : e + 24);
    least = max(least, kLeast - (e + __ffs((int)m) - 1));
}

// A value as a whole number that compares as the values do (-0 counts as 0, and what is not a number is beyond the infinities).
__device__ __forceinline__ uint32_t ordered_bits(float x)
{
    const uint32_t bits = __float_as_uint(x + 0.0f);
    return (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
}

// The columns of every codebook side by side, each row on a 32-byte (or 64-byte) boundary.  The levels read the rows of a
// bucket in many orders, a codebook's columns at a time: from here they take whole 16-byte pieces, and the rows of a
// codebook fit in an XCD's L2 where A does not.  A 16-byte piece to a thread and turn.
// LOOK: and in which bits a column's values differ, for a sort by digits.  (Fewer rows are sorted by comparing: the trees of 50 rows of 64 columns, 8 codebooks, 164 us,
// 169 with; a thread has the same columns in all turns where there are 8, 16, 32, 64 or 128 of them.)
template <bool LOOK>
__global__ __launch_bounds__(256) void gather_columns_kernel(const LearnArgs a)
{
    const int c = blockIdx.y, pieces = a.pitch / 4, lo = a.bounds[2 * c], d = a.bounds[2 * c + 1] - lo;
    float4 *X = reinterpret_cast<float4 *>(a.X + (size_t)c * (a.N + 1) * a.pitch);
    int top = 0, least = 0;
    // in which bits the columns' values differ from those of the first row
    uint32_t first[4], varying[4] = {};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int col = 4 * (int)(threadIdx.x % pieces) + e;
        first[e] = LOOK ? ordered_bits(col < d ? a.A[lo + col] : 0.0f) : 0u;
    }
    // (four turns' loads ahead of their stores: there are no more workgroups than parts of a range.  2^20 x 128, one codebook:
    // 550 us one by one)
    constexpr int kAhead = 4;
    const int64_t n = (a.N + 1) * pieces, stride = (int64_t)gridDim.x * 256;
    for (int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x; i0 < n; i0 += kAhead * stride) {
        float v[kAhead][4];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t i = min(i0 + u * stride, n - 1), row = i / pieces;
            const int col = 4 * (int)(i - row * pieces);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[u][e] = row < a.N && col + e < d ? a.A[row * a.lda + lo + col + e] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (i0 + u * stride < n) {
                X[i0 + u * stride] = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    span_of(v[u][e], top, least);
                    if (LOOK && i0 + u * stride < a.N * pieces) varying[e] |= ordered_bits(v[u][e]) ^ first[e];
                }
            }
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        top = max(top, __shfl_xor(top, off));
        least = max(least, __shfl_xor(least, off));
    }
    // (one maximum for all, by atomics, took up to 320 us)
    __shared__ int32_t part[4][2];
    __shared__ uint32_t differ[LOOK ? 256 : 1][4];
    if constexpr (LOOK) {
#pragma unroll
        for (int e = 0; e < 4; ++e) differ[threadIdx.x][e] = varying[e];
    }
    if ((threadIdx.x & 63) == 0) {
        part[threadIdx.x >> 6][0] = top;
        part[threadIdx.x >> 6][1] = least;
    }
    __syncthreads();
    if (LOOK && (int)threadIdx.x < a.pitch) {
        uint32_t any = 0;
        for (int t = threadIdx.x / 4; t < 256; t += pieces) any |= differ[t][threadIdx.x & 3];
        a.varying_part[((size_t)c * kRangeParts + blockIdx.x) * a.pitch + threadIdx.x] = any;
    }
    if (threadIdx.x < 2)
        a.range_part[((size_t)c * kRangeParts + blockIdx.x) * 2 + threadIdx.x] =
            max(max(part[0][threadIdx.x], part[1][threadIdx.x]), max(part[2][threadIdx.x], part[3][threadIdx.x]));
}

// The rows of every bucket, in row order (a stable counting sort of the rows by bucket): rows_by_bucket[c]
// holds the rows of bucket 0, then those of bucket 1, ...; bucket_start and bucket_count say where.  A workgroup
// per codebook and chunk of chunk_rows rows; how many rows of each bucket the chunks hold is known (apply_kernel counts
// them as it deals them out), and a row's place among its chunk's comes from wavefront ballots.  (260100 rows, 4
// codebooks: 5.0 ms for the four levels with one workgroup per codebook.)
constexpr int kMaxChunks = 256;
__host__ __device__ constexpr int64_t order_chunk_rows(int64_t N)
{
    const int64_t r = (N + kMaxChunks - 1) / kMaxChunks;
    return r <= 2048 ? 2048 : (r + 255) / 256 * 256;
}

__global__ __launch_bounds__(256) void order_rows_kernel(const LearnArgs a, int level, int n_buckets)
{
    __shared__ int32_t total[kSplitBuckets], before[kSplitBuckets], seen[kSplitBuckets];
    __shared__ int32_t wave_count[2][kSplitBuckets][4];
    const int c = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t N = a.N, chunk_rows = order_chunk_rows(N);
    const int chunk = blockIdx.x, n_chunks = gridDim.x;
    const uint8_t *node = a.node + (size_t)c * N;
    int32_t *out = a.rows_by_bucket + (size_t)c * N;
    if (tid < kSplitBuckets) total[tid] = before[tid] = 0;
    if (level == 0 && chunk == 0 && tid < 128) {
        // (gather_columns_kernel's parts: 64 lanes of a wavefront for either half of a range)
        int most = 0;
        for (int i = lane; i < kRangeParts; i += 64) most = max(most, a.range_part[((size_t)c * kRangeParts + i) * 2 + wave]);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) most = max(most, __shfl_xor(most, off));
        if (lane == 0) a.range[2 * c + wave] = most;
    }
    if (a.look && level == 0 && chunk == 0) {
        for (int col = wave; col < a.pitch; col += 4) {
            uint32_t any = 0;
            for (int i = lane; i < a.gather_parts; i += 64) any |= a.varying_part[((size_t)c * kRangeParts + i) * a.pitch + col];
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) any |= __shfl_xor(any, off);
            if (lane == 0) a.varying[(size_t)c * a.pitch + col] = any;
        }
    }
    __syncthreads();
    if (tid < n_chunks)
        for (int k = 0; k < n_buckets; ++k) {
            const int64_t rows = N - tid * chunk_rows;
            const int32_t here = level == 0 ? (int32_t)(rows < chunk_rows ? rows : chunk_rows)
                                            : a.chunk_count[(((size_t)level * a.C + c) * kMaxChunks + tid) * kSplitBuckets + k];
            if (here) atomicAdd(&total[k], here);
            if (here && tid < chunk) atomicAdd(&before[k], here);
        }
    __syncthreads();
    if (tid == 0) {
        int32_t at = 0;
        for (int k = 0; k < kSplitBuckets; ++k) {
            const int32_t here = k < n_buckets ? total[k] : 0;
            seen[k] = at + before[k];
            if (chunk == 0) {
                a.bucket_start[c * kSplitBuckets + k] = at;
                a.bucket_count[c * kSplitBuckets + k] = here;
            }
            at += here;
        }
    }
    const int64_t first = chunk * chunk_rows, end = first + chunk_rows < N ? first + chunk_rows : N;
    int next_b = first + tid < end ? node[first + tid] : -1;
    __syncthreads();
    int parity = 0;
    for (int64_t n0 = first; n0 < end; n0 += 256, parity ^= 1) {
        const int my_b = next_b;
        next_b = n0 + 256 + tid < end ? node[n0 + 256 + tid] : -1;
        int rank = 0;
        for (int k = 0; k < n_buckets; ++k) {
            const unsigned long long mask = __ballot(my_b == k);
            if (my_b == k) rank = __popcll(mask & ((1ull << lane) - 1ull));
            if (lane == 0) wave_count[parity][k][wave] = __popcll(mask);
        }
        __syncthreads();
        if (my_b >= 0) {
            for (int w = 0; w < wave; ++w) rank += wave_count[parity][my_b][w];
            out[seen[my_b] + rank] = (int32_t)(n0 + tid);
        }
        __syncthreads();
        if (tid < n_buckets)
            seen[tid] += wave_count[parity][tid][0] + wave_count[parity][tid][1] + wave_count[parity][tid][2] + wave_count[parity][tid][3];
    }
}

// The serial sums.  A sum in a given order is one dependent addition per row, and what else is done per row decides how
// near the kernel comes to the adder's latency (5.2 cycles).  A chain sits in a row of 16 lanes of a wavefront: each lane
// holds one of 16 consecutive terms, and v_fmac_f64 with a row broadcast adds them one after the other (times 1.0, which
// rounds as an addition does) without any data movement between the additions; four chains to a wavefront.  (A lane per
// chain that reads its terms from LDS takes twice as long, 12.4 against 6.5 cycles per term for one wavefront.)
// The other wavefronts of the workgroup (helpers) fetch the rows several tiles ahead, NC columns of each, 16 bytes per
// lane, and lay the values out by column in LDS.
constexpr int kChainRows = 256;                              // rows staged at a time (a tile)
constexpr int kChainHelpers = 256;                           // threads that fetch them: one lists a row of a tile
constexpr int kDepth = 4;                                    // tiles whose values are on their way at a time
constexpr int kLists = 8;                                    // lists of row numbers in LDS (a power of two > kDepth + 1)
constexpr int kChainPitch = kChainRows + 4;                  // (a wavefront's writes, 16 rows of every fourth column, meet in no bank; its
                                                             // four chains' reads do: 47 % of split_chains_kernel's LDS cycles)
constexpr int kMaxWidth = 128;                               // widest subspace
static_assert(kChainHelpers == kChainRows, "a helper lists one row of every tile");

#define MADDNESS_ADD_TERM(k) "v_fmac_f64_dpp %0, %1, %2 row_newbcast:" #k " row_mask:0xf bank_mask:0xf\n\t"
// acc += the 16 terms of the lane's row of 16 lanes, first lane's first
__device__ __forceinline__ void add_16_in_order(double &acc, double term, double one)
{
    // (a register that a vector instruction has written may be broadcast two cycles later)
    asm("s_nop 1\n\t" MADDNESS_ADD_TERM(0) MADDNESS_ADD_TERM(1) MADDNESS_ADD_TERM(2) MADDNESS_ADD_TERM(3)
        MADDNESS_ADD_TERM(4) MADDNESS_ADD_TERM(5) MADDNESS_ADD_TERM(6) MADDNESS_ADD_TERM(7) MADDNESS_ADD_TERM(8)
        MADDNESS_ADD_TERM(9) MADDNESS_ADD_TERM(10) MADDNESS_ADD_TERM(11) MADDNESS_ADD_TERM(12) MADDNESS_ADD_TERM(13)
        MADDNESS_ADD_TERM(14) MADDNESS_ADD_TERM(15)
        : "+v"(acc)
        : "v"(term), "v"(one));
}
#undef MADDNESS_ADD_TERM

#define MADDNESS_ADD_TERM(t, k) "v_fmac_f64_dpp %0, " t ", %5 row_newbcast:" #k " row_mask:0xf bank_mask:0xf\n\t"
#define MADDNESS_ADD_TERMS(t)                                                                                              \
    MADDNESS_ADD_TERM(t, 0) MADDNESS_ADD_TERM(t, 1) MADDNESS_ADD_TERM(t, 2) MADDNESS_ADD_TERM(t, 3) MADDNESS_ADD_TERM(t, 4)  \
    MADDNESS_ADD_TERM(t, 5) MADDNESS_ADD_TERM(t, 6) MADDNESS_ADD_TERM(t, 7) MADDNESS_ADD_TERM(t, 8) MADDNESS_ADD_TERM(t, 9)  \
    MADDNESS_ADD_TERM(t, 10) MADDNESS_ADD_TERM(t, 11) MADDNESS_ADD_TERM(t, 12) MADDNESS_ADD_TERM(t, 13)                     \
    MADDNESS_ADD_TERM(t, 14) MADDNESS_ADD_TERM(t, 15)
// The same with four terms to a lane, 64 steps at a stretch.
__device__ __forceinline__ void add_64_in_order(double &acc, const double (&term)[4], double one)
{
    asm("s_nop 1\n\t" MADDNESS_ADD_TERMS("%1") MADDNESS_ADD_TERMS("%2") MADDNESS_ADD_TERMS("%3") MADDNESS_ADD_TERMS("%4")
        : "+v"(acc)
        : "v"(term[0]), "v"(term[1]), "v"(term[2]), "v"(term[3]), "v"(one));
}
#undef MADDNESS_ADD_TERMS
#undef MADDNESS_ADD_TERM

// The chains' part of a tile: `at` is the lane's first value (its 16th of the column's), term(x, i) the term of value x in
// row i of the lane's; before(k) runs before every 32nd row.  Rows from `rows` on (a multiple of 32) are left out.
template <typename Term, typename Before>
__device__ __forceinline__ void add_tile_in_order(double &acc, const float *at, int rows, Term term, Before before)
{
    double one = 1.0;
    asm("" : "+v"(one));
    float x[kChainRows / 16];
#pragma unroll
    for (int i = 0; i < kChainRows / 16; ++i) x[i] = at[16 * i];
#pragma unroll
    for (int i = 0; i < kChainRows / 16; ++i) {
        if (i % 2 == 0 && 16 * i >= rows) break;
        if (i % 2 == 0) before(i / 2);
        add_16_in_order(acc, term(x[i], 16 * i), one);
    }
}

// The workgroup's loop: n_steps tiles of kChainRows rows.  walk(values of tile s, s, rows) runs on the first kWalkers
// wavefronts; meanwhile the helpers lay out tile s + 1, fetch the values of tile s + kDepth + 1 and list the rows of the
// tile after that, whose numbers they asked for kDepth steps before: ask(s, i) reads what tells the number of row i of
// tile s, anything where there is none, and row(read, s, i) is the number, `N` where there is none.  (ask has to read in
// any case: a read under a condition becomes a branch, after which every wait is one for all that is on its way, 600 ns
// a tile.)  X: the codebook's values, from the workgroup's first column on.  n_rows: how many rows there are in all,
// rounded up to a multiple of 32 at most; `rows` is kChainRows, or n_rows where there is one tile alone.
template <int NC>
constexpr size_t stream_lds_bytes() { return sizeof(float) * 2 * NC * kChainPitch + sizeof(int32_t) * kLists * kChainRows; }

template <int NC, int kWalkers, typename Ask, typename Row, typename Walk>
__device__ __forceinline__ void stream_rows(unsigned char *lds, const float *X, int pitch, int n_steps, int n_rows, Ask ask, Row row, Walk walk)
{
    constexpr int kPieces = NC / 4, kStride = kChainHelpers / kPieces, kPer = kChainRows / kStride, kBuffer = NC * kChainPitch;
    float *values = reinterpret_cast<float *>(lds);                        // [2][NC][kChainPitch]
    int32_t *listed = reinterpret_cast<int32_t *>(values + 2 * kBuffer);   // [kLists][kChainRows]
    const int helper = (int)threadIdx.x - 64 * kWalkers, at = helper < 0 ? 0 : helper;
    const int rsub = at / kPieces, piece = at % kPieces;
    const float *src = X + 4 * piece;
    float4 x[kDepth][kPer];
    decltype(ask(0, 0)) next[kDepth];
    auto fetch = [&](int s, int set) __attribute__((always_inline)) {
        const int32_t *rows = listed + (s % kLists) * kChainRows;
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            x[set][u] = *reinterpret_cast<const float4 *>(src + (uint64_t)(uint32_t)rows[rsub + u * kStride] * (uint32_t)pitch);
    };
    auto stash = [&](int s, int set) __attribute__((always_inline)) {
        float *dst = values + (s & 1) * kBuffer + 4 * piece * kChainPitch + rsub;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            dst[u * kStride] = x[set][u].x;
            dst[u * kStride + kChainPitch] = x[set][u].y;
            dst[u * kStride + 2 * kChainPitch] = x[set][u].z;
            dst[u * kStride + 3 * kChainPitch] = x[set][u].w;
        }
    };
    if (n_steps == 1) {
        // a bucket of one tile (many codebooks, few rows): nothing to fetch ahead, and no more rows than there are (the trees
        // of 64 codebooks of 9 columns, 50 rows: 275 us with all that the loop below reads, 227 so)
        const bool walks = __builtin_amdgcn_readfirstlane(helper) < 0;
        if (!walks && helper < n_rows) listed[helper] = row(ask(0, helper), 0, helper);
        __syncthreads();
        if (!walks) {
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (u * kStride < n_rows) {
                    const int r = rsub + u * kStride;
                    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if (r < n_rows) v = *reinterpret_cast<const float4 *>(src + (uint64_t)(uint32_t)listed[r] * (uint32_t)pitch);
                    float *dst = values + 4 * piece * kChainPitch + r;
                    dst[0] = v.x;
                    dst[kChainPitch] = v.y;
                    dst[2 * kChainPitch] = v.z;
                    dst[3 * kChainPitch] = v.w;
                }
        }
        __syncthreads();
        if (walks) walk(values, 0, n_rows);
        __syncthreads();
        return;
    }
    // (Two loops with a barrier a tile in each: in one loop the compiler takes a load for the newest wherever the walkers'
    // side may have come between, and waits for all of them.)
    if (__builtin_amdgcn_readfirstlane(helper) < 0) {
        __syncthreads();
        __syncthreads();
        for (int s = 0; s < n_steps; ++s) {
            walk(values + (s & 1) * kBuffer, s, kChainRows);
            __syncthreads();
        }
        return;
    }
#pragma unroll
    for (int s = 0; s < kDepth + 2; ++s) listed[(s % kLists) * kChainRows + helper] = row(ask(s, helper), s, helper);
    __syncthreads();
    fetch(0, 0);
    stash(0, 0);
#pragma unroll
    for (int s = 1; s <= kDepth; ++s) {
        fetch(s, s % kDepth);
        next[s - 1] = ask(s + kDepth + 1, helper);
    }
    __syncthreads();
    for (int s0 = 0; s0 < n_steps; s0 += kDepth) {
#pragma unroll
        for (int i = 0; i < kDepth; ++i) {
            const int s = s0 + i;
            if (s >= n_steps) return;
            stash(s + 1, (i + 1) % kDepth);
            fetch(s + 1 + kDepth, (i + 1) % kDepth);
            listed[((s + kDepth + 2) % kLists) * kChainRows + helper] = row(next[i], s + kDepth + 2, helper);
            next[i] = ask(s + 2 * kDepth + 2, helper);
            __syncthreads();
        }
    }
}

// A sum in a given order without its chain of roundings: 256 terms at once, 4 to a lane (term 64 k + lane is t[k]), on
// two grounds that are checked for every 256, after which any order gives the same bits.
//   - While a sum s stays in one binade, its ulp u does not change, and adding t rounds s + t to a multiple of u: the
//     step is t rounded to a multiple of u (which adding and subtracting 1.5 times the binade's power of two does), halves
//     going to whichever side makes the sum an even multiple.  Steps are whole multiples of u, so their sum is
//     exact.  A half's side depends on the parity of the sum before it, which the parities of the steps since the last
//     half give (after a half the sum is even): ballots.
//   - If all terms and s are multiples of 2^(E-52) and no partial sum reaches 2^(E+1), every sum is exact.
// Where neither holds (a sum that leaves its binade, some 30 times in a sum of 2^18 squares; data with infinities) the
// 256 terms go through the chain.  (A tile of 256 whole values, both sums: 370 ns each, of which 215 are the rows' way
// into LDS; the chain of either takes 560.)
__device__ __forceinline__ double power_of_two(int field) { return __builtin_bit_cast(double, (uint64_t)field << 52); }

__device__ __forceinline__ double read_lane(double x, int lane)
{
    const uint64_t bits = __builtin_bit_cast(uint64_t, x);
    const uint32_t low = __builtin_amdgcn_readlane((int)(uint32_t)bits, lane), high = __builtin_amdgcn_readlane((int)(bits >> 32), lane);
    return __builtin_bit_cast(double, (uint64_t)high << 32 | low);
}

// the sum over the wavefront's lanes, in any order
__device__ __forceinline__ double wave_sum(double x)
{
    auto rotated = [](double v, auto by) __attribute__((always_inline)) {
        const uint64_t bits = __builtin_bit_cast(uint64_t, v);
        const int low = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)bits, 0x120 + decltype(by)::value, 0xf, 0xf, true);
        const int high = __builtin_amdgcn_update_dpp(0, (int)(bits >> 32), 0x120 + decltype(by)::value, 0xf, 0xf, true);
        return __builtin_bit_cast(double, (uint64_t)(uint32_t)high << 32 | (uint32_t)low);
    };
    x += rotated(x, std::integral_constant<int, 8>{});
    x += rotated(x, std::integral_constant<int, 4>{});
    x += rotated(x, std::integral_constant<int, 2>{});
    x += rotated(x, std::integral_constant<int, 1>{});
    return (read_lane(x, 0) + read_lane(x, 16)) + (read_lane(x, 32) + read_lane(x, 48));
}

__device__ __forceinline__ bool add_in_binade(double &s, const double (&t)[4])      // terms >= 0
{
    const uint64_t bits = __builtin_bit_cast(uint64_t, s);
    const int e = __builtin_amdgcn_readfirstlane((int)(bits >> 52));
    // (zero, or next to the ends of the range: the sum stays only if all terms are 0, as a column of equal values has them)
    if (e < 64 || e > 2000) return !__ballot(t[0] != 0.0 || t[1] != 0.0 || t[2] != 0.0 || t[3] != 0.0);
    const double c = __builtin_bit_cast(double, (uint64_t)e << 52 | 1ull << 51);
    const double ulp = power_of_two(e - 52), half = power_of_two(e - 53), most = power_of_two(e - 1);
    double y[4], steps = 0.0;
    bool fits = true, halves = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        y[k] = t[k] + c;
        const double step = y[k] - c;
        fits &= t[k] < most;
        halves |= fabs(t[k] - step) == half;
        steps += step;
    }
    if (__ballot(!fits)) return false;
    double end = s + wave_sum(steps);
    const double limit = power_of_two(e + 1);
    if (__ballot(halves)) {
        if (!(end + 256.0 * ulp < limit)) return false;
        const int lane = threadIdx.x & 63;
        const unsigned long long below = (1ull << lane) - 1ull;
        int parity = (int)(bits & 1), moved = 0;               // of the sum in units of u; units that halves went the other way
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double left = t[k] - (y[k] - c);
            const bool is_half = fabs(left) == half;
            const unsigned long long odd = __ballot((__builtin_bit_cast(uint64_t, y[k]) & 1) != 0), half_at = __ballot(is_half);
            // the parity before this lane's term: of the steps since the last half, or since the lanes' first
            const unsigned long long before = half_at & below;
            const unsigned long long since = before ? ~((2ull << (63 - __clzll(before))) - 1ull) : ~0ull;
            const bool is_odd = ((__popcll(odd & below & since) + (before ? 0 : parity)) & 1) != 0;
            // (the step as computed is the even one of the two; an odd sum takes the other)
            moved += __popcll(__ballot(is_half && is_odd && left > 0.0)) - __popcll(__ballot(is_half && is_odd && left < 0.0));
            parity = half_at ? __popcll(odd & ~((2ull << (63 - __clzll(half_at))) - 1ull)) & 1 : (parity + __popcll(odd)) & 1;
        }
        end += (double)moved * ulp;
    }
    if (!(end < limit)) return false;
    s = end;
    return true;
}

// room: the least E (as an exponent field) that the terms so far have asked for
__device__ __forceinline__ bool add_exactly(double &s, const double (&t)[4], int &room)
{
    const double m = fmax(fmax(fabs(t[0]), fabs(t[1])), fmax(fabs(t[2]), fabs(t[3])));
    int E = __builtin_amdgcn_readfirstlane(max((int)(__builtin_bit_cast(uint64_t, s) >> 52 & 2047) + 1, room));
    // (256 terms of at most 2^(E-9) each: half a binade)
    while (__ballot(m > power_of_two(E - 9))) {
        room = E = E + 4;
        if (E > 2000) return false;
    }
    if (E > 2000) return false;
    const double scale = power_of_two(2098 - E);               // 2^(52 - E)
    bool whole = s * scale == rint(s * scale);
    double steps = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        whole &= t[k] * scale == rint(t[k] * scale);
        steps += t[k];
    }
    if (__ballot(!whole)) return false;
    s += wave_sum(steps);
    return true;
}

__device__ __forceinline__ void add_chained(double &s, const double (&t)[4])
{
    double one = 1.0;
    asm("" : "+v"(one));
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int row = 0; row < 4; ++row) {
            double acc = s;
            add_16_in_order(acc, t[k], one);
            s = read_lane(acc, 16 * row);
        }
}

// L(j, B_i): the sum, then the squared distances from the mean, over the bucket's rows in row order, a wavefront per
// column, four columns of a bucket to a workgroup.  (Measured, the four levels of 260100 x 27 with 4 codebooks, whole
// values: 1.65 ms; 3.3 ms with four chains to a wavefront and 14.6 ms with a lane per chain that read and converted its
// values itself.  20000 x 512 with 32, of both signs, whose first sum takes the chain: 0.31, 0.39 and 1.75 ms.)
// For the candidates (which: 0), where the estimates are not enough, or where those were and the splits' are not (1): for the
// losses of buckets that some candidate cannot split.
__global__ __launch_bounds__(4 * 64 + kChainHelpers) void bucket_loss_kernel(const LearnArgs a, int which)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int c = blockIdx.x, b = blockIdx.y, col0 = blockIdx.z * 4;
    if (which ? !(a.unsure[2 * c + 1] & kWantsLosses) : !a.unsure[2 * c]) return;
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    if (col0 >= d) return;
    const int count = (int)a.bucket_count[c * kSplitBuckets + b];
    const int32_t *list = a.rows_by_bucket + (size_t)c * a.N + a.bucket_start[c * kSplitBuckets + b];
    const int n_steps = (count + kChainRows - 1) / kChainRows;
    double *out = a.col_loss + ((size_t)c * kSplitBuckets + b) * a.dmax + col0;
    if (count == 0) {
        if (threadIdx.x < 4 && (int)threadIdx.x < d - col0) out[threadIdx.x] = 0.0;
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), cols = min(4, d - col0);
    const float *X = a.X + (size_t)c * (a.N + 1) * a.pitch + col0;
    auto ask = [&](int s, int i) __attribute__((always_inline)) { return list[min(s * kChainRows + i, count - 1)]; };
    auto row = [&](int32_t read, int s, int i) __attribute__((always_inline)) {
        return s * kChainRows + i < count ? read : (int32_t)a.N;
    };
    double sum = 0.0, loss = 0.0;
    int room = 1023;
    stream_rows<4, 4>(lds_raw, X, a.pitch, n_steps, count, ask, row, [&](const float *values, int, int) __attribute__((always_inline)) {
        double t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = (double)values[wave * kChainPitch + 64 * k + lane];
        if (!add_exactly(sum, t, room)) add_chained(sum, t);
    });
    const double mean = sum / (double)count;
    stream_rows<4, 4>(lds_raw, X, a.pitch, n_steps, count, ask, row, [&](const float *values, int s, int) __attribute__((always_inline)) {
        double t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double e = (double)values[wave * kChainPitch + 64 * k + lane] - mean;
            t[k] = s * kChainRows + 64 * k + lane < count ? e * e : 0.0;          // (adding 0 leaves a sum as it is)
        }
        if (!add_in_binade(loss, t)) add_chained(loss, t);
    });
    if (wave < cols && lane == 0) out[wave] = loss;
}

// Estimates, and when they are enough: learn_bounds.h.

// A workgroup per kPartRows rows of a bucket, in row order: what the estimates of L(j, B) take, column by column.  (With
// select_kernel, the four levels of 260100 x 27: 0.11 ms against 1.60 for bucket_loss_kernel; 20000 x 512: 0.10 and 0.31.)
constexpr int kPartRows = 1024, kPartValues = 3;
__device__ __forceinline__ int64_t first_part(int32_t start, int bucket) { return start / kPartRows + bucket; }

template <int NC>
__global__ __launch_bounds__(256) void loss_parts_kernel(const LearnArgs a, int n_buckets)
{
    constexpr int kPieces = NC / 4, kRows = 256 / kPieces, kPer = kPartRows / kRows, kAhead = 8;
    __shared__ double from_wave[4][kPieces][4][kPartValues];
    const int c = blockIdx.x % a.C, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t part = blockIdx.x / a.C;
    int start = 0, count = 0, at = 0;
    for (int k = 0; k < n_buckets; ++k) {
        const int s = a.bucket_start[c * kSplitBuckets + k], n = (int)a.bucket_count[c * kSplitBuckets + k];
        const int64_t first = first_part(s, k);
        if (part >= first && part < first + (n + kPartRows - 1) / kPartRows) {
            start = s;
            count = n;
            at = (int)(part - first) * kPartRows;
        }
    }
    if (count == 0) return;
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c], piece = tid % kPieces;
    const int32_t *list = a.rows_by_bucket + (size_t)c * a.N + start;
    const float *X = a.X + (size_t)c * (a.N + 1) * a.pitch + 4 * piece;
    double *out = a.parts + ((size_t)c * a.part_slots + part) * kPartValues * a.dmax;
    const uint32_t pivot = list[count / 2];
    uint32_t row[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) row[i] = list[min(at + i * kRows + tid / kPieces, count - 1)];
    for (int col0 = 0; col0 < d; col0 += NC) {
        const float4 p4 = *reinterpret_cast<const float4 *>(X + col0 + (uint64_t)pivot * (uint32_t)a.pitch);
        const float p[4] = {p4.x, p4.y, p4.z, p4.w};
        double y1[4] = {}, y2[4] = {}, x2[4] = {};
#pragma unroll
        for (int i0 = 0; i0 < kPer; i0 += kAhead) {
            float4 v[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) v[i] = *reinterpret_cast<const float4 *>(X + col0 + (uint64_t)row[i0 + i] * (uint32_t)a.pitch);
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                const bool here = at + (i0 + i) * kRows + tid / kPieces < count;
                const float x4[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double x = here ? (double)x4[e] : 0.0, y = here ? (double)x4[e] - (double)p[e] : 0.0;
                    y1[e] += y;
                    y2[e] = __builtin_fma(y, y, y2[e]);
                    x2[e] = __builtin_fma(x, x, x2[e]);
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int off = kPieces; off < 64; off <<= 1) {
                y1[e] += __shfl_xor(y1[e], off);
                y2[e] += __shfl_xor(y2[e], off);
                x2[e] += __shfl_xor(x2[e], off);
            }
            if (lane < kPieces) {
                double *to = from_wave[wave][lane][e];
                to[0] = y1[e];
                to[1] = y2[e];
                to[2] = x2[e];
            }
        }
        __syncthreads();
        if (tid < NC * kPartValues) {
            const int value = tid / NC, col = tid % NC;
            double v[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) v[w] = from_wave[w][col / 4][col % 4][value];
            if (col0 + col < d) out[value * a.dmax + col0 + col] = (v[0] + v[1]) + (v[2] + v[3]);
        }
        __syncthreads();
    }
}

// The candidate that is `rank` largest losses down, by one wavefront: total[col] is the loss of column lane + 64 i, taken[i]
// whether a candidate of lower rank has the column (or there is none).  Equal losses: the lower column; a loss that is not a
// number is taken where it is the first column left, as a comparison with it is false.
__device__ __forceinline__ int largest_left(const double (&total)[kMaxWidth / 64], bool (&taken)[kMaxWidth / 64])
{
    const int lane = threadIdx.x & 63;
    int first = kMaxWidth;
#pragma unroll
    for (int i = kMaxWidth / 64 - 1; i >= 0; --i) {
        const unsigned long long open = __ballot(!taken[i]);
        if (open) first = 64 * i + __ffsll(open) - 1;
    }
    const double of_first = first < 64 ? __shfl(total[0], first & 63) : __shfl(total[1], first & 63);
    int best = first;
    if (of_first == of_first) {
        int at = kMaxWidth;
        double mine = 0.0;
#pragma unroll
        for (int i = 0; i < kMaxWidth / 64; ++i)
            if (!taken[i] && total[i] == total[i] && (at == kMaxWidth || total[i] > mine)) {
                mine = total[i];
                at = lane + 64 * i;
            }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double other = __shfl_xor(mine, off);
            const int at2 = __shfl_xor(at, off);
            if (at2 < kMaxWidth && (at == kMaxWidth || other > mine || (other == mine && at2 < at))) {
                mine = other;
                at = at2;
            }
        }
        best = at;
    }
#pragma unroll
    for (int i = 0; i < kMaxWidth / 64; ++i) taken[i] |= lane + 64 * i == best;
    return best;
}

// heuristic_select_idxs from the estimates: the four columns with the largest losses summed over the buckets, largest first,
// and whether the estimates can tell.  A workgroup per codebook, its 8 wavefronts shared out among the buckets.
// Columns next to the one that is chosen may be copies of it: then all their sums are the same, and the first is taken.
// The workgroup compares them row by row and keeps what it finds for choose_by_gain_kernel and the levels that follow.
// (131072 x 64, 8 codebooks of which every column has a copy: the four levels' trees 1964 us, 4268 with exact sums for all
// of them.)
__global__ __launch_bounds__(512) void select_kernel(const LearnArgs a, int level, int n_buckets)
{
    __shared__ int32_t original[kMaxWidth], asked;        // (the column to compare with, or -1)
    __shared__ unsigned long long close[kMaxWidth / 64];  // the columns to compare
    __shared__ uint32_t differ[kMaxWidth / 32];           // those of them that differ
    __shared__ bool hopeless;
    __shared__ double from_wave[8][16][kPartValues], loss[kMaxWidth], error[kMaxWidth], energy[kSplitBuckets], spread[kSplitBuckets];
    const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c], b = wave % n_buckets, share = wave / n_buckets, shares = 8 / n_buckets;
    const int start = a.bucket_start[c * kSplitBuckets + b], count = (int)a.bucket_count[c * kSplitBuckets + b];
    const int n_parts = (count + kPartRows - 1) / kPartRows, col = lane & 15;
    // (used at the end, asked for here)
    const int first_like = tid < d && level > 0 ? a.original[(size_t)c * a.dmax + tid] : tid;
    const double rows_of_lane = lane < n_buckets ? (double)a.bucket_count[c * kSplitBuckets + lane] : 0.0;
    const bool exact_sums = any_order(a, c);
    int64_t left = level == 0 ? (a.pitch <= 32 ? 16 : 8) * a.N : a.may_compare[c];
    if (tid < kMaxWidth) loss[tid] = error[tid] = 0.0;
    if (tid < kSplitBuckets) energy[tid] = spread[tid] = 0.0;
    for (int col0 = 0; col0 < d; col0 += 16) {
        const double *in = a.parts + ((size_t)c * a.part_slots + first_part(start, b)) * kPartValues * a.dmax + min(col0 + col, d - 1);
        double sum[kPartValues] = {};
        // (eight parts asked for at a time: 1024 of 128 columns one by one took 460 us)
        constexpr int kAhead = 8;
        int i = 4 * share + lane / 16;
        for (; i + 4 * shares * (kAhead - 1) < n_parts; i += 4 * shares * kAhead) {
            double x[kAhead][kPartValues];
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int v = 0; v < kPartValues; ++v) x[u][v] = in[((size_t)(i + 4 * shares * u) * kPartValues + v) * a.dmax];
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int v = 0; v < kPartValues; ++v) sum[v] += x[u][v];
        }
        for (; i < n_parts; i += 4 * shares)
#pragma unroll
            for (int v = 0; v < kPartValues; ++v) sum[v] += in[((size_t)i * kPartValues + v) * a.dmax];
#pragma unroll
        for (int v = 0; v < kPartValues; ++v) {
            sum[v] += __shfl_xor(sum[v], 16);
            sum[v] += __shfl_xor(sum[v], 32);
            if (lane < 16) from_wave[wave][lane][v] = sum[v];
        }
        __syncthreads();
        // (a thread per column: the buckets one after the other)
        if (tid < 16 && col0 + tid < d)
            for (int k = 0; k < n_buckets; ++k) {
                const int n = (int)a.bucket_count[c * kSplitBuckets + k];
                if (n == 0) continue;
                double y1 = 0.0, y2 = 0.0, x2 = 0.0;
                for (int w = k; w < 8; w += n_buckets) {
                    y1 += from_wave[w][tid][0];
                    y2 += from_wave[w][tid][1];
                    x2 += from_wave[w][tid][2];
                }
                const int32_t pivot = a.rows_by_bucket[(size_t)c * a.N + a.bucket_start[c * kSplitBuckets + k] + n / 2];
                const double p = (double)a.X[((size_t)c * (a.N + 1) + pivot) * a.pitch + col0 + tid];
                const double here = n > 1 ? fmax(y2 - y1 * y1 / (double)n, 0.0) : 0.0;      // (a row alone: no loss)
                loss[col0 + tid] += here;
                if (n > 1) error[col0 + tid] += loss_error((double)n, y2, p);
                from_wave[k][tid][0] = here;
                from_wave[k][tid][2] = x2;
            }
        __syncthreads();
        if (tid < n_buckets && a.bucket_count[c * kSplitBuckets + tid] > 0)
            for (int k = 0; k < min(16, d - col0); ++k) {
                spread[tid] += from_wave[tid][k][0];
                energy[tid] += from_wave[tid][k][2];
            }
        __syncthreads();
    }
    if (tid < n_buckets) a.energy[c * kSplitBuckets + tid] = energy[tid] * 1.0001;
    if (tid < d) original[tid] = first_like;
    __syncthreads();
    // A bucket whose whole loss is less than what two splits of it have to differ by (little spread far from 0): there will be
    // no telling.  (20000 x 512 of 1000 and a thousandth either way, 32 codebooks: 2976 us with all estimates, 2625 with none.)
    if (wave == 1) {
        const bool here = lane < n_buckets && spread[lane] > 0.0 &&
                          spread[lane] < 2.0 * split_error(rows_of_lane, sqrt(rows_of_lane), (double)a.N, energy[lane], d, exact_sums, true);
        const unsigned long long those = __ballot(here);
        if (lane == 0) hopeless = those != 0;
    }
    const int n_cand = min(kCand, d);
    bool finite = true, sure = true;
    unsigned long long compared[kMaxWidth / 64] = {};     // (columns that others have been compared with)
    for (;;) {
        if (wave == 0) {
            double total[kMaxWidth / 64], off_by[kMaxWidth / 64];
            bool taken[kMaxWidth / 64];
            finite = true;
#pragma unroll
            for (int i = 0; i < kMaxWidth / 64; ++i) {
                taken[i] = lane + 64 * i >= d;
                total[i] = loss[lane + 64 * i];
                off_by[i] = error[lane + 64 * i];
                finite &= total[i] < __builtin_inf() && off_by[i] < __builtin_inf();
            }
            for (int k = 0; k < n_buckets; ++k) finite &= energy[k] < __builtin_inf();
            finite = !__ballot(!finite);
            sure = finite;
            int ask = -1;
            for (int k = 0; k < n_cand; ++k) {
                const int best = largest_left(total, taken) & (kMaxWidth - 1);
                const double least = loss[best] - error[best];
                bool any_close = false, alike = true;             // (the estimates of a copy are the same to the bit)
                unsigned long long those[kMaxWidth / 64];
#pragma unroll
                for (int i = 0; i < kMaxWidth / 64; ++i) {
                    const int col = lane + 64 * i;
                    // (columns of zeros alone have no error: their losses are equal, in column order)
                    const bool less = taken[i] || total[i] + off_by[i] < least || (off_by[i] == 0.0 && error[best] == 0.0) ||
                                      (col > best && original[col] == original[best]);
                    those[i] = __ballot(!less);
                    any_close |= those[i] != 0;
                    alike &= less || (total[i] == loss[best] && off_by[i] == error[best]);
                }
                if (lane == 0) a.cand[c * kCand + k] = best;
                if (!any_close || !sure) continue;
                int pieces = 0;
#pragma unroll
                for (int i = 0; i < kMaxWidth / 64; ++i)
                    pieces += __popcll((those[i] | those[i] >> 1 | those[i] >> 2 | those[i] >> 3) & 0x1111111111111111ull);
                if (__ballot(!alike) || (compared[best / 64] >> (best % 64) & 1) || pieces * a.N > left) {
                    sure = false;
                    continue;
                }
                compared[best / 64] |= 1ull << (best % 64);
                // (64 rows first, by this wavefront: columns of few values tie without being copies)
                const uint32_t *row = reinterpret_cast<const uint32_t *>(a.X) + ((size_t)c * (a.N + 1) + a.N * lane / 64) * a.pitch;
                const uint32_t of_best = row[best];
#pragma unroll
                for (int i = 0; i < kMaxWidth / 64; ++i)
                    for (unsigned long long m = those[i]; m && sure; m &= m - 1)
                        if (__ballot(row[64 * i + __ffsll(m) - 1] != of_best)) sure = false;
                if (!sure) continue;
                ask = best;
                if (lane == 0) {
#pragma unroll
                    for (int i = 0; i < kMaxWidth / 64; ++i) close[i] = those[i];
                }
                break;
            }
            if (lane == 0) asked = ask;
            if (lane < kMaxWidth / 32) differ[lane] = 0;
        }
        __syncthreads();
        const int best = asked;
        if (best < 0) break;
        // a piece of four columns with close ones after the other, its rows until all of them differ
        constexpr int kAhead = 8;
        const uint32_t *X = reinterpret_cast<const uint32_t *>(a.X + (size_t)c * (a.N + 1) * a.pitch);
        for (int piece = 0; 4 * piece < d; ++piece) {
            const uint32_t wanted = (uint32_t)(close[piece / 16] >> (4 * piece % 64)) & 15u;
            if (!wanted) continue;
            for (int64_t row0 = 0; row0 < a.N; row0 += 512 * kAhead) {
                left -= min(a.N - row0, (int64_t)512 * kAhead);
                uint4 v[kAhead];
                uint32_t of_best[kAhead], other = 0;
#pragma unroll
                for (int i = 0; i < kAhead; ++i) {
                    const int64_t row = min(row0 + 512 * i + tid, a.N - 1);
                    v[i] = *reinterpret_cast<const uint4 *>(X + row * a.pitch + 4 * piece);
                    of_best[i] = X[row * a.pitch + best];
                }
#pragma unroll
                for (int i = 0; i < kAhead; ++i)
                    other |= (v[i].x != of_best[i] ? 1u : 0u) | (v[i].y != of_best[i] ? 2u : 0u) | (v[i].z != of_best[i] ? 4u : 0u) |
                             (v[i].w != of_best[i] ? 8u : 0u);
                other &= wanted;
                if (other) atomicOr(&differ[piece / 8], other << (4 * piece % 32));
                __syncthreads();
                const bool all = ((differ[piece / 8] >> (4 * piece % 32)) & wanted) == wanted;
                __syncthreads();                          // (all have read it before the next rows' are added)
                if (all) break;
            }
        }
        __syncthreads();
        if (tid < d && (close[tid / 64] >> (tid % 64) & 1) && !(differ[tid / 32] >> (tid % 32) & 1)) original[tid] = original[best];
        __syncthreads();
    }
    if (tid < d) a.original[(size_t)c * a.dmax + tid] = original[tid];
    if (wave != 0) return;
    if (lane == 0) a.may_compare[c] = left;
    const bool none = hopeless || !finite;
    if (lane == 0) {
        a.n_cand[c] = n_cand;
        a.unsure[2 * c] = sure ? 0 : 1;
        a.unsure[2 * c + 1] = none ? kAllCand | kNoEstimates | (sure ? kWantsLosses : 0) : 0;
        a.exact_levels[2 * c] += sure ? 0 : 1;
        a.exact_levels[2 * c + 1] += none ? 1 : 0;
    }
}

// The same from the exact losses: candidate q.  Every workgroup that sorts a candidate's rows finds out for itself.
__device__ __forceinline__ int select_candidate(const LearnArgs &a, int c, int d, int n_buckets, int q)
{
    const double *cl = a.col_loss + (size_t)c * kSplitBuckets * a.dmax;
    const int lane = threadIdx.x & 63;
    double total[kMaxWidth / 64];
    bool taken[kMaxWidth / 64];
#pragma unroll
    for (int i = 0; i < kMaxWidth / 64; ++i) {
        const int col = min(lane + 64 * i, d - 1);
        total[i] = 0.0;
        for (int b = 0; b < n_buckets; ++b) total[i] += cl[(size_t)b * a.dmax + col];
        taken[i] = lane + 64 * i >= d;
    }
    int best = 0;
    for (int k = 0; k <= q; ++k) best = largest_left(total, taken);
    return best;
}

// (bucket, value, row) keys, 3 + 32 + 29 bits: unsigned order = by bucket, then by value, equal values (-0 counts
// as +0) by row.  The rows of a bucket end up side by side, in the order Algorithm 3 wants them.
constexpr int kKeyRowBits = 29;
__device__ __forceinline__ uint64_t make_key(int bucket, float x, uint32_t row)
{
    return ((uint64_t)bucket << (32 + kKeyRowBits)) | ((uint64_t)ordered_bits(x) << kKeyRowBits) | row;
}
__device__ __forceinline__ float key_value(uint64_t key)
{
    const uint32_t u = (uint32_t)(key >> kKeyRowBits);
    return __uint_as_float((u & 0x80000000u) ? (u ^ 0x80000000u) : ~u);
}
__device__ __forceinline__ int32_t key_row(uint64_t key) { return (int32_t)(key & ((1u << kKeyRowBits) - 1u)); }

// The rows of every (codebook, candidate) sorted by their keys, least significant digit first, up to four digits of nine bits of
// value and bucket (rows that are equal there stay in row order).  Of the value only the bits from the first to the last one in
// which the column's values differ are looked at (SortDigits): whole numbers, bfloat16 and quantised values have few, and the
// launches of the digits that a column does not have end at once (a level of 260100 windows of an image, 4 codebooks: 165 -> 104 us;
// finding the bits out and going by them costs data that uses all bits 2 to 4 per cent below 100000 rows: 20000 rows of 28 columns, 4 codebooks, 548 and 570,
// whole numbers 541 and 487).  A workgroup takes up to 4096 keys at a time (8192 by sort_round_kernel),
// an eighth of them in a row to a wavefront: a key's place among its wavefront's of the same digit comes from nine ballots and a counter in LDS, the
// place of the wavefronts' from those counters, and the keys go through LDS in the digit's order, so that what is written
// are runs.  Up to kSortRound rows are sorted by one launch (sort_round_kernel); more take two a digit: sort_count_kernel counts the
// digits of every chunk of them, sort_scatter_kernel finds where the chunk's begin and moves its keys.  Bound by the
// chain of steps of a round, some 60 instructions a key and digit the longest.  (A level's sort, us: 20000 rows, 32 codebooks 117, 150
// by a bitonic network, 33 passes of 64-bit exchanges over 8192 keys in LDS and the larger distances through memory; 260100,
// 4 codebooks 165 and 262.  Rounds of 8192 keys: 177 and 164; the first digit's keys made from the rows twice, without regard to
// XCDs: 156 and 168.)
constexpr int kSortThreads = 512, kSortWaves = kSortThreads / 64, kSortBits = 9, kSortBins = 1 << kSortBits, kSortDigits = 4;
constexpr int kSortPer = 16, kSortRound = kSortThreads * kSortPer;            // keys of sort_round_kernel
constexpr int kChunkPer = 8, kChunkRound = kSortThreads * kChunkPer, kMaxSortChunks = 64;      // of a chunk's round
static_assert(kSortBins == kSortThreads, "a thread per digit");
static_assert(kSortDigits * kSortBits >= 32 + 3, "value and bucket");
// The digits of a column's keys: the `width` bits of the value from bit `low` on, in which its values differ, then the level's
// bits of the bucket.  Of digit k the lower bits are the value's, from bit `shift` of the key on, and those above them the bucket's.
struct SortDigits {
    int low, width, count;
    int shift, down;
    uint32_t value, bucket;
    __device__ SortDigits(uint32_t varying, int n_buckets)
    {
        low = varying ? __ffs((int)varying) - 1 : 0;
        width = varying ? 32 - __clz((int)varying) - low : 0;
        count = max(1, (width + 31 - __clz(n_buckets) + kSortBits - 1) / kSortBits);
    }
    __device__ void select(int k)
    {
        const int left = min(max(width - kSortBits * k, 0), kSortBits);         // of the value's bits in it
        shift = min(kKeyRowBits + low + kSortBits * k, 63);
        value = (1u << left) - 1u;
        down = 2 * kSortBits - min(max(width - kSortBits * k + kSortBits, 0), 2 * kSortBits);
        bucket = left == kSortBits ? 0u : (uint32_t)kSortBins - 1u;
    }
    __device__ __forceinline__ int of(uint64_t key) const
    {
        return (int)(((uint32_t)(key >> shift) & value) | ((((uint32_t)(key >> (32 + kKeyRowBits)) << kSortBits) >> down) & bucket));
    }
};
// rows of a chunk: even shares of whole rounds, few enough chunks that every workgroup can add up all of their counts
__host__ __device__ constexpr int64_t sort_chunk_rows(int64_t N)
{
    const int64_t rounds = (N + kChunkRound - 1) / kChunkRound, per = (rounds + kMaxSortChunks - 1) / kMaxSortChunks;
    const int64_t chunks = (rounds + per - 1) / per;
    return ((N + chunks - 1) / chunks + kSortThreads - 1) / kSortThreads * kSortThreads;
}

template <int kPer>
struct SortLds {
    uint64_t keys[kSortThreads * kPer];
    uint16_t counts[kSortWaves][kSortBins];        // (two workgroups to a compute unit)
    int32_t to[kSortBins];
    uint32_t of_wave[kSortWaves];
};

// the sum over the workgroup's threads before this one
__device__ __forceinline__ uint32_t sum_before(uint32_t x, uint32_t *of_wave)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t sum = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t other = __shfl_up(sum, off);
        sum += lane >= off ? other : 0u;
    }
    if (lane == 63) of_wave[wave] = sum;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) before += w < wave ? of_wave[w] : 0u;
    return before + sum - x;
}

// One round: the thread's keys (64 i + lane of its wavefront's 64 per_wave; those that do not exist have the last digit and
// come last) go to s.keys in the digit's order.  Returns how many have digit threadIdx.x; *place is where those begin.
template <int kPer>
__device__ __forceinline__ uint32_t sort_round(SortLds<kPer> &s, const uint64_t (&key)[kPer], const int (&digit)[kPer], int per_wave, uint32_t *place)
{
    const int tid = threadIdx.x, wave = tid >> 6;
    uint32_t rank[kPer];
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) s.counts[w][tid] = 0;
    __syncthreads();
    volatile uint16_t *counts = s.counts[wave];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (i < per_wave) {
            const int mine = digit[i];
            uint32_t low = ~0u, high = ~0u;                       // the lanes with the same digit
    #pragma unroll
            for (int b = 0; b < kSortBits; ++b) {
                const int32_t bit = mine << (31 - b) >> 31;
                const unsigned long long m = __ballot(bit != 0);
                low &= ~((uint32_t)m ^ (uint32_t)bit);
                high &= ~((uint32_t)(m >> 32) ^ (uint32_t)bit);
            }
            const uint32_t before = __builtin_amdgcn_mbcnt_hi(high, __builtin_amdgcn_mbcnt_lo(low, 0));
            const uint32_t seen = counts[mine], all = (uint32_t)(__popc(low) + __popc(high));
            if (before + 1 == all) counts[mine] = (uint16_t)(seen + all);
            rank[i] = seen + before;
            wave_lds_fence();
        }
    }
    __syncthreads();
    uint32_t all = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) all += s.counts[w][tid];
    uint32_t at = sum_before(all, s.of_wave);
    *place = at;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        const uint32_t here = s.counts[w][tid];
        s.counts[w][tid] = (uint16_t)at;
        at += here;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i)
        if (i < per_wave) s.keys[s.counts[wave][digit[i]] + rank[i]] = key[i];
    __syncthreads();
    return all;
}

// The column of candidate q, which the workgroup finds out from the exact losses where the estimates were unsure (`shared`: a
// word of LDS); `first` leaves it to the launches that follow.
__device__ __forceinline__ int sort_column(const LearnArgs &a, int c, int q, int d, int n_buckets, bool first, int32_t *shared)
{
    if (!a.unsure[2 * c]) return a.cand[c * kCand + q];
    // (what the estimates left in cand is not read)
    if (threadIdx.x < 64) {
        const int best = select_candidate(a, c, d, n_buckets, q);
        if (threadIdx.x == 0) *shared = best;
        if (threadIdx.x == 0 && first) {
            a.cand[c * kCand + q] = best;
            a.n_cand[c] = min(kCand, d);
        }
    }
    __syncthreads();
    return *shared;
}

__global__ __launch_bounds__(kSortThreads, 4) void sort_round_kernel(const LearnArgs a, int n_buckets)
{
    __shared__ SortLds<kSortPer> s;
    const int c = blockIdx.z, q = blockIdx.y, d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    if (q >= min(kCand, d)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, N = (int)a.N, per_wave = (N + kSortThreads - 1) / kSortThreads;
    const int col = sort_column(a, c, q, d, n_buckets, true, s.to);
    const float *x = a.X + (size_t)c * (a.N + 1) * a.pitch + col;
    const uint8_t *node = a.node + (size_t)c * a.N;
    uint64_t *out = a.keys + ((size_t)c * kCand + q) * a.N;
    uint64_t key[kSortPer];
    int digit[kSortPer];
#pragma unroll
    for (int i = 0; i < kSortPer; ++i) {
        const int p = min(64 * (wave * per_wave + i) + lane, N - 1);
        key[i] = make_key(node[p], x[(int64_t)p * a.pitch], (uint32_t)p);
    }
    SortDigits digits(a.look ? a.varying[(size_t)c * a.pitch + col] : ~0u, n_buckets);
    for (int k = 0; k < digits.count; ++k) {
        digits.select(k);
#pragma unroll
        for (int i = 0; i < kSortPer; ++i) digit[i] = 64 * (wave * per_wave + i) + lane < N ? digits.of(key[i]) : kSortBins - 1;
        uint32_t place;
        sort_round(s, key, digit, per_wave, &place);
        if (k + 1 < digits.count)
#pragma unroll
            for (int i = 0; i < kSortPer; ++i)
                if (i < per_wave) key[i] = s.keys[64 * (wave * per_wave + i) + lane];
    }
    for (int i = tid; i < N; i += kSortThreads) out[i] = s.keys[i];
}

// The same for up to a thread's key each: a key's place is the number of smaller ones, counted by all threads over the keys in
// LDS, two to a read.  (A digit's round takes as long for a few keys as for 512.  The trees of 50 rows of 64 columns, 8
// codebooks: 151 us, 189 by digits; 512 rows 237 and 254.)
__global__ __launch_bounds__(kSortThreads) void sort_few_kernel(const LearnArgs a, int n_buckets)
{
    __shared__ __align__(16) uint64_t keys[kSortThreads];
    __shared__ int32_t shared;
    const int c = blockIdx.z, q = blockIdx.y, d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    if (q >= min(kCand, d)) return;
    const int tid = threadIdx.x, N = (int)a.N, p = min(tid, N - 1);
    const int bucket = a.node[(size_t)c * a.N + p];
    const int col = sort_column(a, c, q, d, n_buckets, true, &shared);
    const uint64_t mine = make_key(bucket, a.X[((size_t)c * (a.N + 1) + p) * a.pitch + col], (uint32_t)p);
    keys[tid] = tid < N ? mine : ~0ull;                   // (smaller than none; whole wavefronts, so there is one where N is odd)
    __syncthreads();
    int before = 0;
    const ulonglong2 *pairs = reinterpret_cast<const ulonglong2 *>(keys);
#pragma unroll 8
    for (int i = 0; i < (N + 1) / 2; ++i) {
        const ulonglong2 two = pairs[i];
        before += (two.x < mine ? 1 : 0) + (two.y < mine ? 1 : 0);
    }
    if (tid < N) a.keys[((size_t)c * kCand + q) * a.N + before] = mine;
}

// the keys as digit k of `count` finds them: after the last one they are in `keys`
__device__ __forceinline__ const uint64_t *sort_source(const LearnArgs &a, int c, int q, int k, int count)
{
    return ((count - k) % 2 ? a.keys2 : a.keys) + ((size_t)c * kCand + q) * a.N;
}

__global__ __launch_bounds__(kSortThreads) void sort_count_kernel(const LearnArgs a, int k, int n_buckets)
{
    __shared__ uint32_t counts[kSortBins];
    __shared__ int32_t shared;
    // (the codebook changes fastest from workgroup to workgroup: those of one codebook meet on few XCDs, whose L2 holds its columns)
    const int c = blockIdx.x % a.C, chunk = blockIdx.x / a.C, q = blockIdx.y, d = a.bounds[2 * c + 1] - a.bounds[2 * c], tid = threadIdx.x;
    if (q >= min(kCand, d)) return;
    counts[tid] = 0;
    const int64_t chunk_rows = sort_chunk_rows(a.N), first = chunk * chunk_rows, end = min(a.N, first + chunk_rows);
    // (the bits of the column are left beside it, where the launches after the first find them without the column's number)
    const int col = k == 0 ? sort_column(a, c, q, d, n_buckets, chunk == 0, &shared) : 0;
    uint32_t varying = ~0u;
    if (a.look) varying = k == 0 ? a.varying[(size_t)c * a.pitch + col] : a.cand_varying[c * kCand + q];
    if (k == 0 && chunk == 0 && tid == 0) a.cand_varying[c * kCand + q] = varying;
    SortDigits digits(varying, n_buckets);
    if (k >= digits.count) return;
    digits.select(k);
    uint64_t *keys = const_cast<uint64_t *>(sort_source(a, c, q, k, digits.count));
    const float *x = a.X + (size_t)c * (a.N + 1) * a.pitch + col;
    const uint8_t *node = a.node + (size_t)c * a.N;
    __syncthreads();
    for (int64_t p0 = first; p0 < end; p0 += kChunkRound) {
        int digit[kChunkPer];
#pragma unroll
        for (int i = 0; i < kChunkPer; ++i) {
            const int64_t p = min(p0 + i * kSortThreads + tid, end - 1);
            // (the first digit's keys are made here)
            const uint64_t key = k == 0 ? make_key(node[p], x[p * a.pitch], (uint32_t)p) : keys[p];
            if (k == 0) keys[p] = key;
            digit[i] = digits.of(key);
        }
#pragma unroll
        for (int i = 0; i < kChunkPer; ++i) {
            // (a value that many rows have, as a ReLU's zeros, would be many additions to one word: the digits of the first two lanes
            // that are left are counted by ballots)
            bool left = p0 + i * kSortThreads + tid < end;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const unsigned long long lanes = __ballot(left);
                if (!lanes) break;
                const int one = __builtin_amdgcn_readlane(digit[i], __ffsll(lanes) - 1);
                const unsigned long long same = __ballot(left && digit[i] == one);
                if ((tid & 63) == __ffsll(lanes) - 1) atomicAdd(&counts[one], (uint32_t)__popcll(same));
                left &= digit[i] != one;
            }
            if (left) atomicAdd(&counts[digit[i]], 1u);
        }
    }
    __syncthreads();
    a.digit_counts[(((size_t)c * kCand + q) * kMaxSortChunks + chunk) * kSortBins + tid] = counts[tid];
}

__global__ __launch_bounds__(kSortThreads, 4) void sort_scatter_kernel(const LearnArgs a, int k, int n_buckets)
{
    __shared__ SortLds<kChunkPer> s;
    const int c = blockIdx.x % a.C, chunk = blockIdx.x / a.C, n_chunks = gridDim.x / a.C, q = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (q >= a.n_cand[c]) return;
    const int64_t chunk_rows = sort_chunk_rows(a.N), first = chunk * chunk_rows, end = min(a.N, first + chunk_rows);
    SortDigits digits(a.look ? a.cand_varying[c * kCand + q] : ~0u, n_buckets);
    if (k >= digits.count) return;
    digits.select(k);
    const uint64_t *keys = sort_source(a, c, q, k, digits.count);
    uint64_t *out = const_cast<uint64_t *>(sort_source(a, c, q, k + 1, digits.count));
    // where the digit threadIdx.x of this chunk goes
    const uint32_t *counts = a.digit_counts + ((size_t)c * kCand + q) * kMaxSortChunks * kSortBins + tid;
    uint32_t all = 0, before = 0;
#pragma unroll 8
    for (int i = 0; i < n_chunks; ++i) {
        const uint32_t here = counts[(size_t)i * kSortBins];
        before += i < chunk ? here : 0u;
        all += here;
    }
    uint32_t at = sum_before(all, s.of_wave) + before;
    const int per_wave = (int)min((int64_t)kChunkPer, chunk_rows / kSortThreads);
    for (int64_t p0 = first; p0 < end; p0 += kSortThreads * per_wave) {
        uint64_t key[kChunkPer];
        int digit[kChunkPer];
#pragma unroll
        for (int i = 0; i < kChunkPer; ++i) key[i] = keys[min(p0 + 64 * (wave * per_wave + i) + lane, end - 1)];
#pragma unroll
        for (int i = 0; i < kChunkPer; ++i) digit[i] = p0 + 64 * (wave * per_wave + i) + lane < end ? digits.of(key[i]) : kSortBins - 1;
        uint32_t place;
        const uint32_t here = sort_round(s, key, digit, per_wave, &place);
        s.to[tid] = (int32_t)(at - place);
        at += here;
        __syncthreads();
        const int n = (int)min((int64_t)kSortThreads * per_wave, end - p0);
        for (int i = tid; i < n; i += kSortThreads) {
            const uint64_t v = s.keys[i];
            out[s.to[digits.of(v)] + i] = v;
        }
        __syncthreads();
    }
}

// Algorithm 3 in two parts.  Algorithm 4's running sums are the one serial thing in it, and a serial sum costs a
// few cycles per row whatever else is done with it, so split_chains_kernel does nothing but add: a chain per
// (candidate, bucket, direction, column, which of the two sums) walks the bucket's rows in sorted order and leaves its
// value at every kSplitRows-th of them.  split_losses_kernel takes it up from there, tile by tile of kSplitRows rows: it
// repeats the few additions in between (the same operations on the same operands), and does the products, divisions,
// differences and comparisons of its rows, all tiles of all buckets at once.  (Measured, the four levels of
// 20000 x 512 with 32 codebooks and of 260100 x 27 with 4: 0.67 + 0.45 and 2.36 + 0.42 ms for the two kernels; 4.8 and
// 34.8 ms as one kernel that did all of it tile after tile.)
constexpr int kSplitRows = 32;
constexpr int kGroupTiles = 8, kGroupRows = kGroupTiles * kSplitRows;     // tiles that a wavefront of split_losses_kernel takes

// the first of the tile slots of a bucket (count rows beginning at `start` take up to count / kSplitRows + 1 of them)
__device__ __forceinline__ int64_t first_slot(int32_t start, int bucket) { return start / kSplitRows + bucket; }
__device__ __forceinline__ int64_t first_group(int32_t start, int bucket) { return start / kGroupRows + bucket; }

// Both sums of up to NC columns to a workgroup, four chains to a wavefront.  Going down (direction 1)
// the tiles are taken last to first, each from its end; what lies past the bucket's last row counts as zeros, which
// leave a sum as it is.  small_too: split_chains_small_kernel takes the buckets of up to kChainRows rows.
template <int NC>
__global__ __launch_bounds__(32 * NC + kChainHelpers) void split_chains_kernel(const LearnArgs a, int small_too)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    // (the codebook changes fastest from workgroup to workgroup: those of one codebook meet on few XCDs)
    const int c = blockIdx.x, b = blockIdx.z, dir = blockIdx.y & 1, q = (blockIdx.y >> 1) & 3, col0 = (blockIdx.y >> 3) * NC;
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    if (q >= a.n_cand[c] || col0 >= d) return;
    const int count = (int)a.bucket_count[c * kSplitBuckets + b], start = a.bucket_start[c * kSplitBuckets + b];
    const int n_tiles = (count + kSplitRows - 1) / kSplitRows;
    if (count <= (small_too ? kChainRows : 1) || !(a.unsure[2 * c + 1] >> q & 1)) return;
    constexpr int kTiles = kChainRows / kSplitRows;
    const int n_steps = (n_tiles + kTiles - 1) / kTiles;
    const uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.N + start;
    const int tid = threadIdx.x, cols = min(NC, d - col0);
    const int chain = (tid / 16) % (2 * NC), l = tid & 15;
    const bool squares = chain >= NC;
    // where the chain's values go: the sums before tile i (of all rows before it, in the direction's order)
    double *out = a.sums + (((size_t)c * kCand + q) * 2 + dir) * a.tile_slots * (2 * a.dmax) +
                  (size_t)first_slot(start, b) * (2 * a.dmax) + (chain / NC) * a.dmax + col0 + chain % NC;
    const bool stored = l == 0 && chain % NC < cols;
    // the place in the sorted order of row i of step s (before the first or after the last: none)
    auto place = [&](int s, int i) __attribute__((always_inline)) {
        const int at = s * kChainRows + i;
        return dir ? n_tiles * kSplitRows - 1 - at : at;
    };
    double acc = 0.0;
    stream_rows<NC, NC / 2>(
        lds_raw, a.X + (size_t)c * (a.N + 1) * a.pitch + col0, a.pitch, n_steps, n_tiles * kSplitRows,
        [&](int s, int i) __attribute__((always_inline)) {
            return static_cast<uint32_t>(keys[max(0, min(place(s, i), count - 1))]);
        },
        [&](uint32_t read, int s, int i) __attribute__((always_inline)) {
            const int p = place(s, i);
            return p >= 0 && p < count ? (int32_t)(read & ((1u << kKeyRowBits) - 1u)) : (int32_t)a.N;
        },
        [&](const float *values, int s, int rows) __attribute__((always_inline)) {
            add_tile_in_order(acc, values + (chain % NC) * kChainPitch + l, rows,
                              [&](float x, int) __attribute__((always_inline)) {
                                  const double v = (double)x;
                                  return squares ? v * v : v;
                              },
                              [&](int t) __attribute__((always_inline)) {
                                  const int tile = kTiles * s + t;
                                  if (stored && tile < n_tiles) out[(size_t)(dir ? n_tiles - 1 - tile : tile) * (2 * a.dmax)] = acc;
                              });
        });
}

// The same for buckets of at most one tile of kChainRows rows, where the other kernel would spend its time on the way in
// and out (a workgroup of 12 wavefronts to a compute unit): both directions and all columns of a group from one reading of
// the rows, a row of 16 lanes per column.  (164 codebooks of 40 columns, 8 rows: a level's chains 8.5 us, 88 there; the trees of
// 64 of 9 columns, 50 rows 185 and 227.)  A bucket of one row has no split.
template <int NC>
__global__ __launch_bounds__(16 * NC) void split_chains_small_kernel(const LearnArgs a)
{
    __shared__ __align__(16) float values[NC][kChainPitch];
    __shared__ int32_t rows[kChainRows];
    const int c = blockIdx.x, b = blockIdx.z, q = blockIdx.y & 3, col0 = (blockIdx.y >> 2) * NC;
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    if (q >= a.n_cand[c] || col0 >= d) return;
    const int count = (int)a.bucket_count[c * kSplitBuckets + b], start = a.bucket_start[c * kSplitBuckets + b];
    if (count < 2 || count > kChainRows || !(a.unsure[2 * c + 1] >> q & 1)) return;
    const int n_tiles = (count + kSplitRows - 1) / kSplitRows, n_rows = n_tiles * kSplitRows, tid = threadIdx.x;
    const uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.N + start;
    const float *X = a.X + (size_t)c * (a.N + 1) * a.pitch + col0;
    for (int i = tid; i < n_rows; i += 16 * NC) rows[i] = i < count ? key_row(keys[i]) : (int32_t)a.N;
    __syncthreads();
    for (int i = tid; i < n_rows * (NC / 4); i += 16 * NC) {
        const int r = i / (NC / 4), piece = i % (NC / 4);
        const float4 v = *reinterpret_cast<const float4 *>(X + (int64_t)rows[r] * a.pitch + 4 * piece);
        values[4 * piece][r] = v.x;
        values[4 * piece + 1][r] = v.y;
        values[4 * piece + 2][r] = v.z;
        values[4 * piece + 3][r] = v.w;
    }
    __syncthreads();
    const int col = tid / 16, l = tid & 15;
    const size_t row_size = 2 * (size_t)a.dmax, down = (size_t)a.tile_slots * row_size;
    double *out = a.sums + ((size_t)c * kCand + q) * 2 * down + (size_t)first_slot(start, b) * row_size + col0 + col;
    double sum[2] = {0.0, 0.0}, squares[2] = {0.0, 0.0}, one = 1.0;
    asm("" : "+v"(one));
    for (int t = 0; t < n_tiles; ++t) {
        if (l == 0 && col0 + col < d)
#pragma unroll
            for (int dir = 0; dir < 2; ++dir) {
                double *at = out + dir * down + (dir ? n_tiles - 1 - t : t) * row_size;
                at[0] = sum[dir];
                at[a.dmax] = squares[dir];
            }
#pragma unroll
        for (int i = 0; i < kSplitRows; i += 16)
#pragma unroll
            for (int dir = 0; dir < 2; ++dir) {
                const int at = t * kSplitRows + i + l;
                const double v = (double)values[col][dir ? n_rows - 1 - at : at];
                add_16_in_order(sum[dir], v, one);
                add_16_in_order(squares[dir], v * v, one);
            }
    }
}

// The estimates' sums, in three steps: tile_sums_kernel adds up every tile by itself, a lane per tile and four columns, and a
// group's tiles with those before them; scan_groups_kernel does the same for the groups of a bucket; split_gains_kernel walks
// every tile from there.  Bound by the fetch of rows in sorted order (32 bytes each for up to 8 columns, mostly from beyond L2
// where a codebook's columns take more than 4 MiB).  The four levels, these three kernels, against the two of exact sums:
// 20000 x 512 with 32 codebooks 0.12 + 0.04 + 0.18 ms, 0.62 + 0.44; 260100 x 27 with 4 0.20 + 0.03 + 0.26, 2.36 + 0.42.
// where the rows of the wavefront's groups come from: the rows of its tiles, listed in LDS, and where the lane's own lie
template <int NC>
struct GroupRows {
    static constexpr int kPieces = NC / 4, kTiles = 64 / kPieces, kGroups = kTiles / kGroupTiles;
    int b, start, count, at, rows;           // the bucket, its first row and its rows (0: no such group), the tile's first, its rows
    int64_t group;
    uint32_t splits;                         // bit i: a split between row i of the tile and the next is one
};

template <int NC>
__device__ __forceinline__ GroupRows<NC> list_group_rows(const LearnArgs &a, int c, int q, int n_buckets, uint32_t (*listed)[kSplitRows + 1])
{
    using G = GroupRows<NC>;
    G g;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, my_tile = lane / G::kPieces, tile = my_tile % kGroupTiles;
    g.group = ((int64_t)(blockIdx.x / a.C) * 4 + wave) * G::kGroups + my_tile / kGroupTiles;
    g.b = g.start = g.count = g.at = 0;
    for (int k = 0; k < n_buckets; ++k) {
        const int s = a.bucket_start[c * kSplitBuckets + k], n = (int)a.bucket_count[c * kSplitBuckets + k];
        const int64_t first = first_group(s, k);
        if (g.group >= first && g.group < first + (n + kGroupRows - 1) / kGroupRows) {
            g.b = k;
            g.start = s;
            g.count = n;
            g.at = (int)(g.group - first) * kGroupRows + tile * kSplitRows;
        }
    }
    g.rows = max(0, min(kSplitRows, g.count - g.at));
    g.splits = 0;
    const uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.N;
    // two tiles' keys to a load
#pragma unroll
    for (int i = 0; i < G::kTiles; i += 2) {
        const int from = (i + lane / kSplitRows) * G::kPieces, r = lane % kSplitRows;
        const int first = __shfl(g.start + g.at, from), left = __shfl(g.count - g.at, from);
        const uint64_t key = keys[r < left ? first + r : 0], next = keys[r + 1 < left ? first + r + 1 : 0];
        listed[i + lane / kSplitRows][r] = r < left ? static_cast<uint32_t>(key) & ((1u << kKeyRowBits) - 1u) : (uint32_t)a.N;
        const unsigned long long here = __ballot(r + 1 < left && key_value(key) < key_value(next));
        if (my_tile == i) g.splits = (uint32_t)here;
        if (my_tile == i + 1) g.splits = (uint32_t)(here >> 32);
    }
    wave_lds_fence();
    return g;
}

template <int NC>
__global__ __launch_bounds__(256) void tile_sums_kernel(const LearnArgs a, int n_buckets)
{
    using G = GroupRows<NC>;
    constexpr int kAhead = 16;
    __shared__ uint32_t listed[4][G::kTiles][kSplitRows + 1];
    const int c = blockIdx.x % a.C, q = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (q >= a.n_cand[c] || a.unsure[2 * c + 1]) return;
    const int piece = lane % G::kPieces, tile = lane / G::kPieces % kGroupTiles;
    const G g = list_group_rows<NC>(a, c, q, n_buckets, listed[wave]);
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    const uint32_t *row = listed[wave][lane / G::kPieces];
    const float *X = a.X + (size_t)c * (a.N + 1) * a.pitch + 4 * piece;
    double *before = a.sums + ((size_t)c * kCand + q) * 4 * a.tile_slots * a.dmax +
                     (size_t)(first_slot(g.start, g.b) + g.at / kSplitRows) * a.dmax + 4 * piece;
    double *all = a.group_sums + (((size_t)c * kCand + q) * a.group_slots + g.group) * a.dmax + 4 * piece;
    for (int col0 = 0; col0 < d; col0 += NC) {
        double sum[4] = {};
#pragma unroll
        for (int i0 = 0; i0 < kSplitRows; i0 += kAhead) {
            float4 v[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) v[i] = *reinterpret_cast<const float4 *>(X + col0 + (uint64_t)row[i0 + i] * (uint32_t)a.pitch);
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                sum[0] += (double)v[i].x;
                sum[1] += (double)v[i].y;
                sum[2] += (double)v[i].z;
                sum[3] += (double)v[i].w;
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double through = sum[e];                               // of the group's tiles up to this one
#pragma unroll
            for (int off = 1; off < kGroupTiles; off <<= 1) {
                const double other = __shfl_up(through, off * G::kPieces);
                through += tile >= off ? other : 0.0;
            }
            if (g.count == 0 || col0 + 4 * piece + e >= d) continue;
            if (g.rows > 0) before[col0 + e] = through - sum[e];
            if (tile == kGroupTiles - 1) all[col0 + e] = through;
        }
    }
}

// A workgroup per (candidate, bucket) and 16 columns; a thread takes up to kScanGroups groups in a row at a time.
constexpr int kScanThreads = 64, kScanGroups = 16;
__global__ __launch_bounds__(16 * kScanThreads) void scan_groups_kernel(const LearnArgs a)
{
    __shared__ double part[kScanThreads + 1][16];
    const int c = blockIdx.x % a.C, q = blockIdx.x / a.C, b = blockIdx.y, col0 = 16 * blockIdx.z;
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    const int side = threadIdx.x & 15, t = threadIdx.x >> 4, col = min(col0 + side, d - 1);
    if (q >= a.n_cand[c] || col0 >= d || a.unsure[2 * c + 1]) return;
    const bool stored = col0 + side < d;
    const int count = (int)a.bucket_count[c * kSplitBuckets + b], start = a.bucket_start[c * kSplitBuckets + b];
    const int n_groups = (count + kGroupRows - 1) / kGroupRows;
    double *sums = a.group_sums + (((size_t)c * kCand + q) * a.group_slots + first_group(start, b)) * a.dmax + col;
    double before = 0.0;
    for (int first = 0; first < n_groups; first += kScanThreads * kScanGroups) {
        const int here = min(n_groups - first, kScanThreads * kScanGroups), per = (here + kScanThreads - 1) / kScanThreads;
        const int lo = first + t * per, left = min(first + here - lo, per);
        double v[kScanGroups], sum = 0.0;
#pragma unroll
        for (int i = 0; i < kScanGroups; ++i) {
            v[i] = sums[(size_t)min(lo + i, n_groups - 1) * a.dmax];
            v[i] = i < left ? v[i] : 0.0;
            sum += v[i];
        }
        __syncthreads();
        part[t][side] = sum;
        __syncthreads();
        if (t == 0) {
            double s = 0.0;
#pragma unroll 16
            for (int i = 0; i < kScanThreads; ++i) {
                const double x = part[i][side];
                part[i][side] = s;
                s += x;
            }
            part[kScanThreads][side] = s;
        }
        __syncthreads();
        double at = before + part[t][side];
        before += part[kScanThreads][side];
        if (stored)
#pragma unroll
            for (int i = 0; i < kScanGroups; ++i)
                if (i < left) {
                    sums[(size_t)(lo + i) * a.dmax] = at;
                    at += v[i];
                }
    }
    if (t == 0 && stored) a.totals[(((size_t)c * kCand + q) * kSplitBuckets + b) * a.dmax + col] = before;
}

// x of the lane whose number differs in bit kBit (of the lowest two)
template <int kBit>
__device__ __forceinline__ double across(double x)
{
    const int64_t bits = __builtin_bit_cast(int64_t, x);
    constexpr int kPerm = kBit == 1 ? 0xb1 : 0x4e;           // lanes 1 0 3 2, or 2 3 0 1
    const int low = __builtin_amdgcn_update_dpp(0, (int)bits, kPerm, 0xf, 0xf, true);
    const int high = __builtin_amdgcn_update_dpp(0, (int)(bits >> 32), kPerm, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (int64_t)high << 32 | (uint32_t)low);
}

// The gain of every split (split_error in learn_bounds.h tells what that is): the lanes of a tile walk its rows together, four columns each, and
// add up what their columns give; lane p of them keeps rows p, p + kPieces, ...
struct Gain {
    double best, second;
    int at;
    __device__ __forceinline__ void add(double g, double g2, int where)
    {
        second = fmax(fmax(second, g2), fmin(best, g));
        at = g > best ? where : at;
        best = fmax(best, g);
    }
};

template <int NC>
__global__ __launch_bounds__(256) void split_gains_kernel(const LearnArgs a, int n_buckets)
{
    using G = GroupRows<NC>;
    constexpr int kPieces = G::kPieces, kAhead = 8, kOwn = kSplitRows / kPieces;
    __shared__ uint32_t listed[4][G::kTiles][kSplitRows + 1];
    const int c = blockIdx.x % a.C, q = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (q >= a.n_cand[c] || a.unsure[2 * c + 1]) return;
    const int piece = lane % kPieces;
    const G g = list_group_rows<NC>(a, c, q, n_buckets, listed[wave]);
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    const uint32_t *row = listed[wave][lane / kPieces];
    const float *X = a.X + (size_t)c * (a.N + 1) * a.pitch + 4 * piece;
    const double *before = a.sums + ((size_t)c * kCand + q) * 4 * a.tile_slots * a.dmax +
                           (size_t)(first_slot(g.start, g.b) + g.at / kSplitRows) * a.dmax;
    const double *all = a.group_sums + (((size_t)c * kCand + q) * a.group_slots + g.group) * a.dmax;
    const double *totals = a.totals + (((size_t)c * kCand + q) * kSplitBuckets + g.b) * a.dmax;
    const double n = (double)max(g.count, 1);
    double squares[kOwn] = {};
    for (int col0 = 0; col0 < d; col0 += NC) {
        double sum[4], mean[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int col = min(col0 + 4 * piece + e, d - 1);
            const bool here = g.rows > 0 && col0 + 4 * piece + e < d;
            sum[e] = here ? all[col] + before[col] : 0.0;
            mean[e] = here ? totals[col] / n : 0.0;
        }
#pragma unroll
        for (int i0 = 0; i0 < kSplitRows; i0 += kAhead) {
            float4 v[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) v[i] = *reinterpret_cast<const float4 *>(X + col0 + (uint64_t)row[i0 + i] * (uint32_t)a.pitch);
#pragma unroll
            for (int i1 = 0; i1 < kAhead; i1 += kPieces) {
                double of[kPieces];
#pragma unroll
                for (int i = 0; i < kPieces; ++i) {
                    const float x[4] = {v[i1 + i].x, v[i1 + i].y, v[i1 + i].z, v[i1 + i].w};
                    const double minus_n1 = -(double)(g.at + i0 + i1 + i + 1);
                    of[i] = 0.0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        sum[e] += (double)x[e];
                        const double w = __builtin_fma(minus_n1, mean[e], sum[e]);
                        of[i] = __builtin_fma(w, w, of[i]);
                    }
                }
                // lane p's row: of[p] of all lanes
                if constexpr (kPieces == 4) {
                    const bool odd = piece & 1, high = piece & 2;
                    const double a0 = (odd ? of[1] : of[0]) + across<1>(odd ? of[0] : of[1]);
                    const double a1 = (odd ? of[3] : of[2]) + across<1>(odd ? of[2] : of[3]);
                    squares[(i0 + i1) / kPieces] += (high ? a1 : a0) + across<2>(high ? a0 : a1);
                } else {
                    const bool odd = piece & 1;
                    squares[(i0 + i1) / kPieces] += (odd ? of[1] : of[0]) + across<1>(odd ? of[0] : of[1]);
                }
            }
        }
    }
    Gain best{-1.0, -1.0, -1};
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const int r = kPieces * i + piece;
        const double n1 = (double)(g.at + r + 1), product = n1 * fmax(n - n1, 1.0);
        double y = __builtin_amdgcn_rcp(product);
        y = __builtin_fma(__builtin_fma(-product, y, 1.0), y, y);
        y = __builtin_fma(__builtin_fma(-product, y, 1.0), y, y);
        const bool splits = g.splits >> r & 1;
        best.add(splits ? squares[i] * n * y : -1.0, -1.0, splits ? g.at + r : -1);
    }
#pragma unroll
    for (int off = 1; off < kPieces * kGroupTiles; off <<= 1) {
        const double b2 = __shfl_xor(best.best, off), s2 = __shfl_xor(best.second, off);
        const int at2 = __shfl_xor(best.at, off);
        best.add(b2, s2, at2);
    }
    if (lane % (kPieces * kGroupTiles) == 0 && g.count > 0) {
        const size_t o = ((size_t)c * kCand + q) * a.group_slots + g.group;
        a.group_gain[2 * o] = best.best;
        a.group_gain[2 * o + 1] = best.second;
        a.group_first[o] = best.at;
    }
}

// (v > l fails where the midpoint rounds to the lower value)
__device__ __forceinline__ float split_value(uint64_t low, uint64_t high)
{
    const float l = key_value(low), h = key_value(high);
    const float v = (float)(((double)l + (double)h) / 2.0);
    return v > l ? v : h;
}

// The best split of every (candidate, bucket) and the best candidate from the gains, where they can tell.  (A candidate that
// cannot split a bucket gains nothing there: L(B) is the constant that the gains are taken off.)
__global__ __launch_bounds__(1024) void choose_by_gain_kernel(const LearnArgs a, int level, int n_buckets)
{
    __shared__ Gain found[kCand][kSplitBuckets];
    __shared__ int32_t chosen;
    const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_cand = a.n_cand[c], d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    if (a.unsure[2 * c + 1]) return;
    // (used by the first wavefront after the loop: a lane per (candidate, bucket), the copies a lane per candidate)
    const int n = lane % kSplitBuckets < n_buckets ? (int)a.bucket_count[c * kSplitBuckets + lane % kSplitBuckets] : 0;
    const double energy = lane % kSplitBuckets < n_buckets ? a.energy[c * kSplitBuckets + lane % kSplitBuckets] : 0.0;
    const bool exact_sums = any_order(a, c), have_losses = a.unsure[2 * c];
    const int first_like = lane < n_cand ? a.original[(size_t)c * a.dmax + a.cand[c * kCand + lane]] : -1 - lane;
    for (int pair = wave; pair < n_cand * n_buckets; pair += 16) {
        const int q = pair / n_buckets, b = pair - q * n_buckets;
        const int start = a.bucket_start[c * kSplitBuckets + b], count = (int)a.bucket_count[c * kSplitBuckets + b];
        const int n_groups = (count + kGroupRows - 1) / kGroupRows;
        const size_t o = ((size_t)c * kCand + q) * a.group_slots + first_group(start, b);
        Gain best{-1.0, -1.0, -1};
#pragma unroll 4
        for (int i = lane; i < n_groups; i += 64)
            best.add(a.group_gain[2 * (o + i)], a.group_gain[2 * (o + i) + 1], a.group_first[o + i]);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double b2 = __shfl_xor(best.best, off), s2 = __shfl_xor(best.second, off);
            const int at2 = __shfl_xor(best.at, off);
            best.add(b2, s2, at2);
        }
        if (lane == 0) found[q][b] = best;
    }
    __syncthreads();
    if (wave == 0) {
        const int q = lane / kSplitBuckets, b = lane % kSplitBuckets;
        const bool here = q < n_cand && b < n_buckets;
        const Gain mine = here ? found[q][b] : Gain{-1.0, -1.0, -1};
        // (of the lanes of a bucket: whether each of the candidates splits it)
        const unsigned long long cannot = __ballot(here && mine.at < 0);
        const bool every_splits = !(cannot & (0x01010101ull << b));
        const double error = n > 1 ? split_error((double)n, sqrt((double)n), (double)a.N, energy, d, exact_sums, every_splits) : 0.0;
        double of_all = error, gain = fmax(mine.best, 0.0);
#pragma unroll
        for (int off = 1; off < kSplitBuckets; off <<= 1) {
            of_all += __shfl_xor(of_all, off);
            gain += __shfl_xor(gain, off);
        }
        // the candidates that may be the best: bits.  (None that splits anything, or no value but 0: all losses are equal, and the
        // first candidate is taken.)
        double most = 0.0;
        int best_q = 0;
#pragma unroll
        for (int i = 0; i < kCand; ++i) {
            const double g = __shfl(gain, i * kSplitBuckets);
            if (i == 0 || (i < n_cand && g > most)) {
                most = g;
                best_q = i;
            }
        }
        const bool any = __ballot(mine.at >= 0), sure_of_sums = !__ballot(!(energy < __builtin_inf()));
        int open = 1 << best_q;
#pragma unroll
        for (int i = 0; i < kCand; ++i)
            if (i < n_cand && any && of_all > 0.0 && !(most - __shfl(gain, i * kSplitBuckets) > 2.0 * of_all)) open |= 1 << i;
        if (!sure_of_sums) open = (1 << n_cand) - 1;
        // (a copy of an earlier candidate has the same losses, and the first of equal ones is taken)
#pragma unroll
        for (int i = 1; i < kCand; ++i)
#pragma unroll
            for (int j = 0; j < i; ++j)
                if (__shfl(first_like, i) == __shfl(first_like, j)) open &= ~(1 << i);
        const bool close = q == best_q && !(mine.second < 0.0 || mine.best - mine.second > 2.0 * error);
        const bool sure = sure_of_sums && open == 1 << best_q && !__ballot(close);
        // (one candidate alone is compared with none, and where all candidates split all buckets no L(B) takes part)
        const bool wants = (open & (open - 1)) && !have_losses && (!sure_of_sums || __ballot(here && (open >> q & 1) && mine.at < 0 && n > 0));
        if (lane == 0) {
            a.unsure[2 * c + 1] = sure ? 0 : open | (wants ? kWantsLosses : 0);
            a.exact_levels[2 * c + 1] += sure ? 0 : 1;
            chosen = sure ? best_q : -1;
            if (sure) {
                const int jj = a.cand[c * kCand + best_q];
                a.chosen[c] = jj;
                a.split_dims[4 * c + level] = a.bounds[2 * c] + jj;
                if (level == 3) a.thresholds[16 * c + 15] = 0.0f;
            }
        }
    }
    __syncthreads();
    const int q = chosen;
    if (q < 0 || tid >= n_buckets) return;
    const int at = found[q][tid].at, count = (int)a.bucket_count[c * kSplitBuckets + tid];
    const uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.N + a.bucket_start[c * kSplitBuckets + tid];
    float v = 0.0f;
    if (at >= 0) v = split_value(keys[at], keys[at + 1]);
    else if (count > 0) v = a.X[((size_t)c * (a.N + 1) + key_row(keys[0])) * a.pitch + a.cand[c * kCand + q]];
    a.thresholds[16 * c + n_buckets - 1 + tid] = v;
}

// A wavefront per kGroupTiles tiles of kSplitRows sorted rows of a bucket, one tile after the other with the next one's
// rows on their way: both running sums of every column and both directions from the values that split_chains_kernel
// left at the tile's ends, a lane per (direction, sum, column); then Algorithm 4's term of every column, summed over the
// columns in column order, a lane per (direction, row); then the loss of the split between every row and the next one
// up, and the best of them (the first of equal ones).
// Bound by the vector ALUs: cx cx / n takes one division per row for all its columns, y = 1 / n, and per column a product
// q = t y and one correction q + (t - n q) y by fused multiply-adds.  That is the correctly rounded quotient, as a
// division gives it: q is off by less than 1.5 ulp and n < 2^29 is whole, so the remainder is exact; what remains
// is off by less than 2^-52 ulp before the last rounding, and t / n is either a double or at least ulp / 2^30 from
// the middle between two (n times such a middle has 54 significant bits or more, t has 53 at most).
// (A loss that is not a number, from data with infinities, gives way to one that is.)
__device__ __forceinline__ bool better(double l2, int at2, double loss, int at)
{
    return at2 >= 0 && (at < 0 || l2 < loss || (loss != loss && l2 == l2) || ((l2 == loss || (l2 != l2 && loss != loss)) && at2 < at));
}

template <int NC>
__global__ __launch_bounds__(64) void split_losses_kernel(const LearnArgs a, int n_buckets)
{
    constexpr int T = kSplitRows, kPitch = T + 4, kSumPitch = T + 1, kChains = 4 * NC;
    constexpr int kPieces = NC / 4, kRows = 64 / kPieces, kPer = T / kRows;
    __shared__ __align__(16) double sums[kChains][kSumPitch];
    __shared__ __align__(16) float xs[2][NC][kPitch];       // the tile's values, first to last and last to first
    const int c = blockIdx.x % a.C, q = blockIdx.y, lane = threadIdx.x;
    if (q >= a.n_cand[c] || !(a.unsure[2 * c + 1] >> q & 1)) return;
    const int64_t group = blockIdx.x / a.C;
    int b = -1, start = 0, count = 0;
    for (int k = 0; k < n_buckets; ++k) {
        const int s = a.bucket_start[c * kSplitBuckets + k], n = (int)a.bucket_count[c * kSplitBuckets + k];
        const int64_t first = first_group(s, k);
        if (group >= first && group < first + (n + kGroupRows - 1) / kGroupRows) {
            b = k;
            start = s;
            count = n;
        }
    }
    if (b < 0) return;
    const int tile0 = (int)(group - first_group(start, b)) * kGroupTiles;                   // of the bucket's tiles
    const int n_tiles = min(kGroupTiles, (count + T - 1) / T - tile0);
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    const uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.N + start;
    const float *X = a.X + (size_t)c * (a.N + 1) * a.pitch + 4 * (lane % kPieces);
    // as the sums are taken: a lane per chain
    const int chain_dir = (lane / (2 * NC)) & 1, which = (lane / NC) & 1, chain_col = lane % NC;
    const double *ends = a.sums + ((((size_t)c * kCand + q) * 2 + chain_dir) * a.tile_slots + first_slot(start, b) + tile0) * (2 * a.dmax) +
                         (size_t)which * a.dmax;
    // as the terms are taken: going up the sums with row k, going down those of the rows after it (what the split after
    // row k leaves above)
    const int k = lane & (T - 1), dir = lane / T, entry = dir ? T - 1 - k : k + 1;

    auto key_of = [&](int t) __attribute__((always_inline)) {       // (one more than the tile's, where there is one)
        const int p = (tile0 + t) * T + lane;
        return t < n_tiles && lane <= T && p < count ? keys[p] : 0;
    };
    auto row_of = [&](int t, uint64_t key) __attribute__((always_inline)) {
        return (tile0 + t) * T + lane < count ? key_row(key) : (int32_t)a.N;
    };
    float4 v[kPer];
    double end;
    auto fetch = [&](int t, int32_t my_row, int col0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            v[u] = *reinterpret_cast<const float4 *>(X + col0 + (int64_t)__shfl(my_row, lane / kPieces + u * kRows) * a.pitch);
        end = ends[(size_t)t * (2 * a.dmax) + min(col0 + chain_col, d - 1)];
    };
    uint64_t key = key_of(0), next_key = key_of(1);
    int32_t my_row = row_of(0, key);
    fetch(0, my_row, 0);
    double best = 0.0;
    int at = -1, first_nan = -1;
    bool have_cand = false;
    for (int t = 0; t < n_tiles; ++t) {
        const int left = count - (tile0 + t) * T;                         // rows from the tile's first to the bucket's last
        const double n = (double)max(dir ? left - (k + 1) : (tile0 + t) * T + k + 1, 1), y = 1.0 / n;
        const uint64_t key_after = key_of(t + 2);
        double sse = 0.0;
        for (int col0 = 0; col0 < d; col0 += NC) {
            if (col0 > 0) fetch(t, my_row, col0);
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int p = lane / kPieces + u * kRows;
                const float x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    xs[0][4 * (lane % kPieces) + e][p] = x[e];
                    xs[1][4 * (lane % kPieces) + e][T - 1 - p] = x[e];
                }
            }
            double acc = end;
            __syncthreads();
            if (col0 + NC >= d) {
                my_row = row_of(t + 1, next_key);
                if (t + 1 < n_tiles) fetch(t + 1, my_row, 0);
            }
            if (lane < kChains) {
                const float *x = xs[chain_dir][chain_col];
                double *dst = sums[lane];          // the sums before the first row, after it, after the second, ...
                *dst = acc;
#pragma unroll
                for (int s = 0; s < T; s += 4) {
                    const float4 f = *reinterpret_cast<const float4 *>(x + s);
                    const float e[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const double w = (double)e[u];
                        acc = acc + w * (which ? w : 1.0);
                        dst[s + u + 1] = acc;
                    }
                }
            }
            __syncthreads();
            const int cols = min(NC, d - col0);
#pragma unroll 4
            for (int col = 0; col < cols; ++col) {
                const double cx = sums[dir * 2 * NC + col][entry], cx2 = sums[dir * 2 * NC + NC + col][entry];
                const double square = cx * cx;
                const double quotient = square * y;
                sse = sse + (cx2 - __builtin_fma(__builtin_fma(-n, quotient, square), y, quotient));
            }
            __syncthreads();
        }
        // a split between row k and the next one: in the same bucket, and their values differ
        const double loss = sse + __shfl_down(sse, T);
        const float value = key_value(key), next_value = __shfl_down(value, 1);
        const bool cand = dir == 0 && k + 1 < left && value < next_value;
        const unsigned long long cands = __ballot(cand);
        if (!have_cand && cands) {
            const int first = __ffsll(cands) - 1;
            const double l = __shfl(loss, first);
            first_nan = l != l ? (tile0 + t) * T + first : -1;
            have_cand = true;
        }
        if (cand && better(loss, (tile0 + t) * T + k, best, at)) {
            best = loss;
            at = (tile0 + t) * T + k;
        }
        key = next_key;
        next_key = key_after;
    }
#pragma unroll
    for (int off = 1; off < T; off <<= 1) {
        const double l2 = __shfl_xor(best, off);
        const int at2 = __shfl_xor(at, off);
        const bool take = better(l2, at2, best, at);
        best = take ? l2 : best;
        at = take ? at2 : at;
    }
    if (lane == 0) {
        const size_t o = ((size_t)c * kCand + q) * a.group_slots + group;
        a.group_loss[o] = best;
        a.group_at[2 * o] = at;
        a.group_at[2 * o + 1] = first_nan;
    }
}

// The best split of every (candidate, bucket) from its groups of tiles, a wavefront each; then Algorithm 2's choice: the
// candidate with the smallest loss summed over the buckets (the first of equal ones), its thresholds into the tree.
// A comparison with a loss that is not a number (data with infinities) is false, as in Algorithm 3: it stays the best
// where it is the bucket's first.
__global__ __launch_bounds__(512) void choose_kernel(const LearnArgs a, int level, int n_buckets)
{
    __shared__ double res_loss[kCand][kSplitBuckets];
    __shared__ float res_v[kCand][kSplitBuckets];
    const int c = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n_cand = a.n_cand[c], d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    const int unsure = a.unsure[2 * c + 1];
    if (!unsure) return;
    for (int pair = wave; pair < n_cand * n_buckets; pair += 8) {
        const int q = pair / n_buckets, b = pair - q * n_buckets;
        if (!(unsure >> q & 1)) continue;
        const int start = a.bucket_start[c * kSplitBuckets + b], count = (int)a.bucket_count[c * kSplitBuckets + b];
        const int n_groups = (count + kGroupRows - 1) / kGroupRows;
        const size_t o = ((size_t)c * kCand + q) * a.group_slots + first_group(start, b);
        double loss = 0.0;
        int at = -1, first = 0x7fffffff;           // (the first group that has a split at all)
        for (int i = lane; i < n_groups; i += 64) {
            const int at2 = a.group_at[2 * (o + i)];
            const double l2 = a.group_loss[o + i];
            if (at2 >= 0 && first == 0x7fffffff) first = i;
            if (better(l2, at2, loss, at)) {
                loss = l2;
                at = at2;
            }
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double l2 = __shfl_xor(loss, off);
            const int at2 = __shfl_xor(at, off);
            first = min(first, __shfl_xor(first, off));
            const bool take = better(l2, at2, loss, at);
            loss = take ? l2 : loss;
            at = take ? at2 : at;
        }
        if (lane == 0) {
            if (at >= 0) {
                const int not_a_number = a.group_at[2 * (o + first) + 1];
                if (not_a_number >= 0) {
                    at = not_a_number;
                    loss = __builtin_nan("");
                }
            }
            const uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.N + start;
            float v = 0.0f;
            if (at >= 0) {
                v = split_value(keys[at], keys[at + 1]);
            } else if (count > 0) {
                // cannot be split: the value of the bucket's first row in sorted order, the loss L(B)
                v = a.X[((size_t)c * (a.N + 1) + key_row(keys[0])) * a.pitch + a.cand[c * kCand + q]];
                const double *cl = a.col_loss + ((size_t)c * kSplitBuckets + b) * a.dmax;
                loss = 0.0;
                for (int jj = 0; jj < d; ++jj) loss += cl[jj];
            }
            res_v[q][b] = v;
            res_loss[q][b] = loss;
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    int best_q = -1;
    double l_min = 0.0;
    for (int q = 0; q < n_cand; ++q) {
        if (!(unsure >> q & 1)) continue;                  // (the estimates tell that it is not the best)
        double l = 0.0;
        for (int b = 0; b < n_buckets; ++b) l += res_loss[q][b];
        if (best_q < 0 || l < l_min) {
            l_min = l;
            best_q = q;
        }
    }
    const int jj = a.cand[c * kCand + best_q];
    a.chosen[c] = jj;
    a.split_dims[4 * c + level] = a.bounds[2 * c] + jj;
    for (int b = 0; b < n_buckets; ++b) a.thresholds[16 * c + n_buckets - 1 + b] = res_v[best_q][b];
    if (level == 3) a.thresholds[16 * c + 15] = 0.0f;
}

// apply_split: below the threshold stays left (2 i), the rest goes right (2 i + 1); the rows that every bucket of the next
// level gets are counted by chunk.
__global__ __launch_bounds__(256) void apply_kernel(const LearnArgs a, int level, int n_buckets)
{
    const int c = blockIdx.y, lane = threadIdx.x & 63;
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int child = -1;
    if (n < a.N) {
        const int j = a.chosen[c];
        const int b = a.node[(size_t)c * a.N + n];
        const float v = a.thresholds[16 * c + n_buckets - 1 + b];
        child = 2 * b + (a.X[((size_t)c * (a.N + 1) + n) * a.pitch + j] >= v ? 1 : 0);
        a.node[(size_t)c * a.N + n] = (uint8_t)child;
        if (level == 3 && a.codes) a.codes[n * a.codes_pitch + c] = (uint8_t)child;
    }
    if (level == 3) return;
    // (a chunk is a whole number of workgroups' rows)
    const int chunk = (int)(((int64_t)blockIdx.x * 256) / order_chunk_rows(a.N));
    int mine = 0;
    for (int k = 0; k < 2 * n_buckets; ++k) {
        const int here = __popcll(__ballot(child == k));
        if (lane == k) mine = here;
    }
    if (mine) atomicAdd(&a.chunk_count[(((size_t)(level + 1) * a.C + c) * kMaxChunks + chunk) * kSplitBuckets + lane], mine);
}

// ---------------------------------------------------------------------------------------
// prototypes
// ---------------------------------------------------------------------------------------

struct ProtoArgs {
    const uint8_t *codes;   // [N][C]
    const float *A;
    int64_t lda, N;
    int32_t D, C, Q;        // Q = 16 C
    int32_t *bounds;
    int32_t *counts;        // [Q][Q] G^T G
    int32_t *range_part;    // [D / 64 and more][kProtoParts][2] what a part of 64 columns' values span
    int32_t *any_order;     // [D / 64 and more] whether their sums may be taken in any order
    int32_t row_bits;       // N <= 2^row_bits
    int32_t shares;         // wavefronts that share a code's rows where any order will do
    double *R_shares;       // [shares - 1][Q][D] what the others than the first add to R
    double *M;              // [Q][Q]: G^T G + lambda I, then M[k][i] = L[i][k]
    double *Lr;             // [Q][Q]: L in tiles of 16 x 16 (factor_at)
    double *R;              // [Q][D]: G^T A~
    int64_t stretch;        // rows of a stretch
    uint32_t *list;         // [C][kListRows + kListSpare] distances in bytes of the stretch's rows, by code
    int32_t *list_count;    // [C][kListChunks][16] how many each of its chunks has of every code
    int32_t *list_start;    // [C][17] where those of a code begin
    float *P;               // out [C][16][D]
};

// G^T A~ where its sums' bits allow any order (as any_order for the trees, 64 columns at a time): workgroups of parts of the
// rows note what those span, and leave it at that as soon as it is too much, for most data after the first rows.  The
// other workgroups clear the counters.
constexpr int kProtoParts = 256, kProtoClear = 256;
__global__ __launch_bounds__(256) void prepare_kernel(const ProtoArgs a)
{
    if (blockIdx.x < kProtoClear) {
        const int64_t QQ = (int64_t)a.Q * a.Q;
        for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < QQ; i += 256 * kProtoClear) a.counts[i] = 0;
        return;
    }
    const int block = (blockIdx.x - kProtoClear) / kProtoParts, part = (blockIdx.x - kProtoClear) % kProtoParts;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = min(64 * block + lane, a.D - 1);
    __shared__ int32_t widest[4][2];
    const int64_t first = a.N * part / kProtoParts, end = a.N * (part + 1) / kProtoParts;
    int top = 0, least = 0;
    constexpr int kAhead = 32;
    for (int64_t n0 = first; n0 < end; n0 += 4 * kAhead) {
        float x[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) x[u] = a.A[min(n0 + 4 * u + wave, end - 1) * a.lda + col];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) span_of(x[u], top, least);
        if (__ballot(top != 0 && top + least - kLeast + a.row_bits > 53)) {
            top = kNoNumber;
            break;
        }
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        top = max(top, __shfl_xor(top, off));
        least = max(least, __shfl_xor(least, off));
    }
    if (lane == 0) {
        widest[wave][0] = top;
        widest[wave][1] = least;
    }
    __syncthreads();
    if (threadIdx.x < 2)
        a.range_part[((size_t)block * kProtoParts + part) * 2 + threadIdx.x] =
            max(max(widest[0][threadIdx.x], widest[1][threadIdx.x]), max(widest[2][threadIdx.x], widest[3][threadIdx.x]));
}

// G^T G: entry (q, q') counts the training rows whose one-hot row has ones at q and q'.  A workgroup takes
// codebook c against kCoGroup codebooks c2 and a stretch of the rows, counts in LDS (16 x 16 counters a pair), and adds
// its 16 x (16 kCoGroup) block to the matrix (whole numbers: in any order).  (One workgroup for all rows of a block left
// the chip empty: 260100 rows, 4 codebooks 0.60 ms.)
constexpr int kCoGroup = 8;
__global__ __launch_bounds__(256) void cooccurrence_kernel(const ProtoArgs a)
{
    __shared__ int32_t hist[kCoGroup][256];
    const int c = blockIdx.x, c2_first = blockIdx.y * kCoGroup, tid = threadIdx.x;
    const int n_c2 = min(kCoGroup, a.C - c2_first);
    for (int i = tid; i < kCoGroup * 256; i += 256) (&hist[0][0])[i] = 0;
    __syncthreads();
    for (int64_t n = (int64_t)blockIdx.z * 256 + tid; n < a.N; n += (int64_t)gridDim.z * 256) {
        const uint8_t *row = a.codes + n * a.C;
        const int k = row[c] & 15;
        uint8_t k2[kCoGroup];
#pragma unroll
        for (int g = 0; g < kCoGroup; ++g) k2[g] = g < n_c2 ? row[c2_first + g] : 0;
#pragma unroll
        for (int g = 0; g < kCoGroup; ++g)
            if (g < n_c2) atomicAdd(&hist[g][16 * k + (k2[g] & 15)], 1);
    }
    __syncthreads();
    for (int i = tid; i < n_c2 * 256; i += 256) {
        const int g = i >> 8, k = (i >> 4) & 15, k2 = i & 15;
        const int32_t here = hist[g][16 * k + k2];
        if (here) atomicAdd(&a.counts[(size_t)(16 * c + k) * a.Q + 16 * (c2_first + g) + k2], here);
    }
}

__global__ __launch_bounds__(256) void ridge_matrix_kernel(const ProtoArgs a, double lambda)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)a.Q * a.Q) return;
    const int r = (int)(i / a.Q), col = (int)(i - (int64_t)r * a.Q);
    a.M[i] = (double)a.counts[i] + (r == col ? lambda : 0.0);
}

// G^T A~: row 16 c + k = the sum, in row order, of the training rows with code k in codebook c.  kListRows rows at a
// time: count_codes_kernel and list_codes_kernel list the rows of every code in row order (as order_rows_kernel does
// for buckets, a workgroup per codebook and kListChunk rows), then a wavefront per (codebook, code, 64 columns) adds
// its rows, 32 fetched ahead.  Every codebook reads all of A; the workgroups of the same columns run on the same XCD
// when their number is a multiple of 8, and all codes' wavefronts walk the rows at about the same pace, so those reads
// meet in its L2.  Bound by the instructions per row (its address, a load, a conversion, an addition):
// 0.20 + 0.02 ms for 20000 x 512 and 32 codebooks, 0.77 + 0.08 ms for 260100 x 27 and 4 (1.0 and 7.5 ms with every thread
// reading all rows; four columns to a lane, for a third of the instructions, gave 0.27 ms: fewer wavefronts, and rows
// four times as long to keep in L2).  Where the sums are exact in any order and these wavefronts leave the chip empty, several share
// a code's rows: 260100 x 27 with 4 0.04 ms instead of 0.75,
// 0.02 for finding out, in a launch that clears the counters as well (data that are not: 5 to 15 us, 131072 x 64, 8 codebooks 447
// without and 459 with it; whole values 1300 and 322).
constexpr int kListRows = 65536;       // rows of a stretch, at most (their distances in bytes from its first fit 32 bits)
constexpr int kGtaAhead = 32;
constexpr int kListSpare = 4 * kGtaAhead;     // entries read past the last (and not used)
constexpr int kListChunk = 2048, kListChunks = kListRows / kListChunk;
__global__ __launch_bounds__(256) void count_codes_kernel(const ProtoArgs a, int64_t first_row)
{
    __shared__ int32_t total[16];
    const int c = blockIdx.x, chunk = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int64_t first = first_row + chunk * kListChunk;
    const int64_t left = min(a.N - first, a.stretch - chunk * kListChunk);
    const int rows = (int)(left < kListChunk ? left : kListChunk);
    const uint8_t *code = a.codes + first * a.C + c;
    if (tid < 16) total[tid] = 0;
    if (a.shares > 1 && first_row == 0)
        for (int block = 4 * (c + a.C * chunk) + (tid >> 6); block < (a.D + 63) / 64; block += 4 * a.C * (int)gridDim.y) {
            const int32_t *range = a.range_part + (size_t)block * kProtoParts * 2;
            int top = 0, least = 0;
#pragma unroll
            for (int i = 0; i < kProtoParts; i += 64) {
                top = max(top, range[2 * (i + lane)]);
                least = max(least, range[2 * (i + lane) + 1]);
            }
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                top = max(top, __shfl_xor(top, off));
                least = max(least, __shfl_xor(least, off));
            }
            if (lane == 0) a.any_order[block] = top == 0 || top + least - kLeast + a.row_bits <= 53;
        }
    __syncthreads();
    int mine = 0;
#pragma unroll
    for (int u = 0; u < kListChunk / 256; ++u) {
        const int k = 256 * u + tid < rows ? code[(int64_t)(256 * u + tid) * a.C] & 15 : -1;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int here = __popcll(__ballot(k == j));
            if (lane == j) mine += here;
        }
    }
    if (mine) atomicAdd(&total[lane], mine);
    __syncthreads();
    if (tid < 16) a.list_count[(c * kListChunks + chunk) * 16 + tid] = total[tid];
}

__global__ __launch_bounds__(256) void list_codes_kernel(const ProtoArgs a, int64_t first_row)
{
    __shared__ int32_t total[16], seen[16], wave_count[kListChunk / 256][16][4];
    const int c = blockIdx.x, chunk = blockIdx.y, n_chunks = gridDim.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t first = first_row + chunk * kListChunk;
    const int64_t left = min(a.N - first, a.stretch - chunk * kListChunk);
    const int rows = (int)(left < kListChunk ? left : kListChunk);
    const uint8_t *code = a.codes + first * a.C + c;
    if (tid < 16) {
        int before = 0, all = 0;
        for (int i = 0; i < n_chunks; ++i) {
            const int here = a.list_count[(c * kListChunks + i) * 16 + tid];
            before += i < chunk ? here : 0;
            all += here;
        }
        total[tid] = all;
        seen[tid] = before;
    }
    int k[kListChunk / 256], rank[kListChunk / 256];
#pragma unroll
    for (int u = 0; u < kListChunk / 256; ++u) {
        k[u] = 256 * u + tid < rows ? code[(int64_t)(256 * u + tid) * a.C] & 15 : -1;
        int mine = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const unsigned long long mask = __ballot(k[u] == j);
            if (k[u] == j) rank[u] = __popcll(mask & ((1ull << lane) - 1ull));
            if (lane == j) mine = __popcll(mask);
        }
        if (lane < 16) wave_count[u][lane][wave] = mine;
    }
    __syncthreads();
    if (tid < 16) {
        int at = 0;
        for (int j = 0; j < tid; ++j) at += total[j];
        if (chunk == 0) {
            a.list_start[c * 17 + tid] = at;
            if (tid == 15) a.list_start[c * 17 + 16] = at + total[15];
        }
        // the place of the first row of every wavefront's 64
        at += seen[tid];
        for (int u = 0; u < kListChunk / 256; ++u)
            for (int w = 0; w < 4; ++w) {
                const int here = wave_count[u][tid][w];
                wave_count[u][tid][w] = at;
                at += here;
            }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kListChunk / 256; ++u)
        if (k[u] >= 0)
            a.list[(size_t)c * (kListRows + kListSpare) + wave_count[u][k[u]][wave] + rank[u]] =
                (uint32_t)(chunk * kListChunk + 256 * u + tid) * (uint32_t)(4 * a.lda);
}

__global__ __launch_bounds__(256) void gta_kernel(const ProtoArgs a, int64_t first_row)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int k = blockIdx.y * 4 + wave, c = blockIdx.z % a.C, share = blockIdx.z / a.C;
    const int col = blockIdx.x * 64 + lane;
    int start = a.list_start[c * 17 + k], count = a.list_start[c * 17 + k + 1] - start;
    const bool shared = a.shares > 1 && a.any_order[blockIdx.x];
    if (share > 0 && !shared) return;
    if (shared) {
        const int per = (count + a.shares - 1) / a.shares;
        start += share * per;
        count = max(0, min(per, count - share * per));
    }
    // (every share has sums of its own, which transpose_factor_kernel adds up: additions to one by several wavefronts would ask
    // for memory that takes atomics of doubles)
    double *out = (share == 0 ? a.R : a.R_shares + (size_t)(share - 1) * a.Q * a.D) + ((size_t)16 * c + k) * a.D + col;
    double sum = first_row > 0 && col < a.D ? *out : 0.0;
    if (count > 0) {
        // (the same for a whole wavefront, and written by a kernel before this one: scalar loads)
        const auto *list = (const __attribute__((address_space(4))) uint32_t *)(a.list + (size_t)c * (kListRows + kListSpare) + start);
        const char *src = reinterpret_cast<const char *>(a.A + first_row * a.lda);
        const uint32_t col_offset = 4 * min(col, a.D - 1);
        float x0[kGtaAhead], x1[kGtaAhead];
        uint32_t r0[kGtaAhead], r1[kGtaAhead];
        auto entries = [&](uint32_t (&r)[kGtaAhead], int at) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < kGtaAhead; ++u) r[u] = list[at + u];
        };
        // (past the last row: row 0 of the stretch, not added)
        auto fetch = [&](float (&v)[kGtaAhead], const uint32_t (&r)[kGtaAhead], int at) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < kGtaAhead; ++u)
                v[u] = *reinterpret_cast<const float *>(src + (uint32_t)((at + u < count ? r[u] : 0u) + col_offset));
        };
        auto add = [&](const float (&v)[kGtaAhead], int at) __attribute__((always_inline)) {
            if (at + kGtaAhead <= count) {
#pragma unroll
                for (int u = 0; u < kGtaAhead; ++u) sum += (double)v[u];
            } else {
#pragma unroll
                for (int u = 0; u < kGtaAhead; ++u) sum += at + u < count ? (double)v[u] : 0.0;
            }
        };
        entries(r0, 0);
        entries(r1, kGtaAhead);
        fetch(x0, r0, 0);
        for (int at = 0; at < count; at += 2 * kGtaAhead) {
            entries(r0, at + 2 * kGtaAhead);
            fetch(x1, r1, at + kGtaAhead);
            __builtin_amdgcn_sched_barrier(0);      // (the loads stay ahead of the additions)
            add(x0, at);
            if (at + kGtaAhead >= count) break;
            entries(r1, at + 3 * kGtaAhead);
            fetch(x0, r0, at + 2 * kGtaAhead);
            __builtin_amdgcn_sched_barrier(0);
            add(x1, at + kGtaAhead);
        }
    }
    if (col < a.D) *out = sum;
}

template <int K>
__device__ __forceinline__ double row_broadcast(double x)
{
    const int64_t bits = __builtin_bit_cast(int64_t, x);
    const int low = __builtin_amdgcn_update_dpp(0, (int)bits, 0x150 + K, 0xf, 0xf, true);
    const int high = __builtin_amdgcn_update_dpp(0, (int)(bits >> 32), 0x150 + K, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (int64_t)high << 32 | (uint32_t)low);
}

// f(0), f(1) .. f(15), the numbers known at compile time (a row broadcast's lane is part of the instruction).
template <typename F>
__device__ __forceinline__ void for_16(F f)
{
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
    f(std::integral_constant<int, 4>{});
    f(std::integral_constant<int, 5>{});
    f(std::integral_constant<int, 6>{});
    f(std::integral_constant<int, 7>{});
    f(std::integral_constant<int, 8>{});
    f(std::integral_constant<int, 9>{});
    f(std::integral_constant<int, 10>{});
    f(std::integral_constant<int, 11>{});
    f(std::integral_constant<int, 12>{});
    f(std::integral_constant<int, 13>{});
    f(std::integral_constant<int, 14>{});
    f(std::integral_constant<int, 15>{});
}

// L is kept in tiles of 16 x 16, as the substitution reads them: of two columns at a time the 16 rows side by side.
__device__ __forceinline__ size_t factor_at(int Q, int r, int k)
{
    return ((size_t)(r >> 4) * (Q >> 4) + (k >> 4)) * 256 + ((k >> 1) & 7) * 32 + (r & 15) * 2 + (k & 1);
}

// Cholesky factorisation M = L L^T: L_jj = sqrt(M_jj - sum_k L_jk^2), L_ij = (M_ij - sum_k L_ik L_jk) / L_jj,
// every sum over k ascending.  M is symmetric, and entry (i, j), i >= j, is kept at M[j][i] (a column side by side).
// One launch per panel of 16 columns J0 .. J0 + 15, which takes the panel's terms off everything to its right: a
// workgroup per 64 x 64 tile of what is left, which works out the panel's rows of L that it needs for itself and then subtracts
// their 16 products from its entries, k ascending as panels and columns go.  A wavefront does its 64 rows of the tile, or of the
// tile's columns, beside the 16 of the diagonal block, of which every row of 16 lanes has one to a lane: what a column
// needs of another row comes by row broadcasts, without barriers.  The tiles of the first column store L; what they read
// stays as it is.  Bound by the chain of 16 roots and divisions per panel, 10.1 us (12.2 with the panel's rows
// in LDS and two barriers to a column).  (Subtracting all columns
// before the panel at once, when the panel's turn comes, takes few workgroups and up to 31 us a launch: 0.65 against
// 0.38 ms for Q = 512.)
constexpr int kCholPanel = 16, kCholTile = 64, kCholPitch = kCholPanel + 1;
__global__ __launch_bounds__(256) void cholesky_panel_kernel(const ProtoArgs a, int J0)
{
    __shared__ double T[2 * kCholTile][kCholPitch];                  // the panel's columns of L: the tile's rows, its columns
    if (blockIdx.y > blockIdx.x) return;                             // (the other triangle)
    const int Q = a.Q, tid = threadIdx.x, l = tid & 15;
    double *M = a.M;
    const int row0 = J0 + kCholPanel + blockIdx.x * kCholTile, col0 = J0 + kCholPanel + blockIdx.y * kCholTile;
    // a tile's entries: four rows of four columns to a thread
    const int tr = 4 * (tid & 15), tc = 4 * (tid >> 4);
    double s[4][4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const int r = row0 + tr + f, c = col0 + tc + e;
            s[e][f] = r < Q && c <= r ? M[(size_t)c * Q + r] : 0.0;
        }
    if (tid < 2 * kCholTile) {
        const int grow = tid < kCholTile ? row0 + tid : col0 + tid - kCholTile;
        double diagonal[kCholPanel], t[kCholPanel];
#pragma unroll
        for (int j = 0; j < kCholPanel; ++j) {
            diagonal[j] = l >= j ? M[(size_t)(J0 + j) * Q + J0 + l] : 0.0;
            t[j] = grow < Q ? M[(size_t)(J0 + j) * Q + grow] : 0.0;
        }
        auto column = [&](auto index) __attribute__((always_inline)) {
            constexpr int j = decltype(index)::value;
            const double root = sqrt(row_broadcast<j>(diagonal[j]));
            diagonal[j] = l == j ? root : diagonal[j] / root;
            t[j] = t[j] / root;
            auto off = [&](auto index2) __attribute__((always_inline)) {
                constexpr int j2 = decltype(index2)::value;
                if constexpr (j2 > j) {
                    const double other = row_broadcast<j2>(diagonal[j]);
                    diagonal[j2] -= diagonal[j] * other;
                    t[j2] -= t[j] * other;
                }
            };
            for_16(off);
        };
        for_16(column);
#pragma unroll
        for (int j = 0; j < kCholPanel; ++j) T[tid][j] = t[j];
        if (blockIdx.y == 0 && tid < kCholTile) {
            if (grow < Q)
#pragma unroll
                for (int j = 0; j < kCholPanel; ++j) a.Lr[factor_at(Q, grow, J0 + j)] = t[j];
            if (blockIdx.x == 0 && tid < kCholPanel)
#pragma unroll
                for (int j = 0; j < kCholPanel; ++j)
                    if (j <= l) a.Lr[factor_at(Q, J0 + l, J0 + j)] = diagonal[j];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kCholPanel; ++k) {
        double li[4], lj[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            li[e] = T[tr + e][k];
            lj[e] = T[kCholTile + tc + e][k];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int f = 0; f < 4; ++f) s[e][f] -= li[f] * lj[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const int r = row0 + tr + f, c = col0 + tc + e;
            if (r < Q && c <= r) M[(size_t)c * Q + r] = s[e][f];
        }
}

// The factor by columns from its tiles; the workgroups after those add the shares of G^T A~ to the first (exact, in whatever order).
__global__ __launch_bounds__(256) void transpose_factor_kernel(const ProtoArgs a)
{
    const int64_t QQ = (int64_t)a.Q * a.Q;
    const unsigned factor = (unsigned)((QQ + 255) / 256);
    if (blockIdx.x >= factor) {
        const int64_t i = (int64_t)(blockIdx.x - factor) * 256 + threadIdx.x, QD = (int64_t)a.Q * a.D;
        if (i >= QD || !a.any_order[(i % a.D) / 64]) return;
        double sum = a.R[i];
#pragma unroll 16
        for (int share = 1; share < a.shares; ++share) sum += a.R_shares[(share - 1) * QD + i];
        a.R[i] = sum;
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= QQ) return;
    const int k = (int)(i / a.Q), r = (int)(i - (int64_t)k * a.Q);
    if (k <= r) a.M[i] = a.Lr[factor_at(a.Q, r, k)];
}

// L y = G^T A~ and L^T P = y, sums over k ascending: y_i = (b_i - sum_{k<i} L_ik y_k) / L_ii, then
// P_i = (y_i - sum_{k>i} L_ki P_k) / L_ii.  A workgroup of 8 wavefronts takes NC columns of A~ and keeps them in LDS for both.
// Forward, a sum ends with the value found last, so 16 rows at a time are solved (a row of 16 lanes per column) and their
// products taken off all rows below: the first wavefront takes the 16 off the next 16 rows and solves those, while the others
// take them off the rows after these.  Backward, a sum BEGINS with the value found just before, and a column's subtractions
// are one chain of Q^2 / 2 steps: the first wavefront subtracts the products, 16 at a time in the lanes of a row, by row
// broadcasts (as in add_16_in_order), while the others form those of the next row, all but the two with the values that
// are just being found; the factor's rows come kSubDepth ahead, and a row's first products are on their way from LDS while
// the value before it is divided.  Bound by that chain, 5.2 cycles a step.
// 512 columns of A~ and Q = 512: 0.55 ms, 0.07 of it forward (0.64 and 0.19 with L by rows, of which a lane's 16 bytes lay in a line each,
// all wavefronts solving and divisions of 15 dependent operations); Q = 1024, 640 columns 1.80 (2.21).  With all seven wavefronts
// laying out the first one shares its turns: 0.67.  Four columns to a workgroup where LDS holds them and two
// rows' products (up to 104 codebooks), else one.
constexpr int kSubDepth = 4, kSubWaves = 8, kSubHelpers = 192, kSubSpare = 128;
constexpr size_t substitution_lds_bytes(int Q, int nc) { return sizeof(double) * (3 * (size_t)nc * (Q + 16) + kSubSpare + 8); }

// a / d, correctly rounded, from r = divisor_reciprocal(d), in 5 dependent operations instead of some 15.  r is the correctly
// rounded 1 / d; a r is within 2 ulps of the quotient, the first correction brings it within one (faithful), and the second
// rounds it correctly (Markstein, "Computation of elementary functions on the IBM RISC System/6000 processor", 1990, theorem on
// the last step of a division).  The theorem wants no underflow in the remainders: quotients and divisors outside
// 2^-200 .. 2^200 (r is not a number there), infinities and not-a-numbers are divided; a zero is its own quotient.
__device__ __forceinline__ double divisor_reciprocal(double d)
{
    return fabs(d) > 0x1p-200 && fabs(d) < 0x1p200 ? 1.0 / d : __builtin_nan("");
}

__device__ __forceinline__ double divide(double a, double d, double r)
{
    const double q0 = a * r;
    const unsigned exponent = ((unsigned)(__builtin_bit_cast(uint64_t, q0) >> 52) & 0x7ffu) - (1023 - 200);
    if (__builtin_amdgcn_ballot_w64(exponent >= 400u && q0 != 0.0)) return a / d;
    const double q1 = __builtin_fma(__builtin_fma(-d, q0, a), r, q0);
    const double q2 = __builtin_fma(__builtin_fma(-d, q1, a), r, q1);
    return q0 == 0.0 ? q0 : q2;
}

template <int NC, int kPer>
__global__ __launch_bounds__(64 * kSubWaves) void substitution_kernel(const ProtoArgs a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    double *X = reinterpret_cast<double *>(lds_raw);      // [NC][Q + 16]
    const int Q = a.Q, D = a.D, tid = threadIdx.x, lane = tid & 63, l = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blocks = Q / 16;
    const int col0 = blockIdx.x * NC;
    for (int idx = tid; idx < Q * NC; idx += 64 * kSubWaves) {
        const int i = idx / NC, cc = idx % NC;
        X[cc * (Q + 16) + i] = col0 + cc < D ? a.R[(size_t)i * D + col0 + cc] : 0.0;
    }
    double *x = X + min(lane >> 4, NC - 1) * (Q + 16);      // (NC = 1: the other rows of lanes do the same)
    __syncthreads();
    // 16 x 16 entries of L: row 16 m + l, columns 16 J .. 16 J + 15
    auto fetch_block = [&](double (&L)[16], int m, int J) __attribute__((always_inline)) {
        const double2 *src = reinterpret_cast<const double2 *>(a.Lr) + ((size_t)min(m, blocks - 1) * blocks + min(J, blocks - 1)) * 128 + l;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double2 v = src[16 * u];
            L[2 * u] = v.x;
            L[2 * u + 1] = v.y;
        }
    };
    // forward
    if (wave == 0) {
        double y[16], below[16];
        auto solve = [&](int J, const double (&L)[16], double diagonal, double acc) __attribute__((always_inline)) {
            const double r = divisor_reciprocal(diagonal);
            auto step = [&](auto index) __attribute__((always_inline)) {
                constexpr int k = decltype(index)::value;
                const double quotient = divide(acc, diagonal, r);
                y[k] = row_broadcast<k>(quotient);
                acc = l > k ? acc - L[k] * y[k] : l == k ? quotient : acc;
            };
            for_16(step);
            x[16 * J + l] = acc;
        };
        auto diagonal_of = [&](int J) __attribute__((always_inline)) {
            const int i = 16 * min(J, blocks - 1) + l;
            return a.Lr[factor_at(Q, i, i)];
        };
        double L0[16], L1[16], d0, d1;
        fetch_block(L0, 0, 0);
        d0 = diagonal_of(0);
        fetch_block(below, 1, 0);
        fetch_block(L1, 1, 1);
        d1 = diagonal_of(1);
        __builtin_amdgcn_sched_barrier(0);
        solve(0, L0, d0, x[l]);
        __syncthreads();
        // rows 16 J .. 16 J + 15, from those above them
        auto turn = [&](int J, double (&L)[16], double &d, double (&next)[16], double &next_d) __attribute__((always_inline)) {
            double acc = x[16 * J + l];
#pragma unroll
            for (int k = 0; k < 16; ++k) acc -= below[k] * y[k];
            fetch_block(below, J + 1, J);
            fetch_block(next, J + 1, J + 1);
            next_d = diagonal_of(J + 1);
            __builtin_amdgcn_sched_barrier(0);
            solve(J, L, d, acc);
            __syncthreads();
        };
        for (int J = 1; J < blocks; J += 2) {
            turn(J, L1, d1, L0, d0);
            if (J + 1 < blocks) turn(J + 1, L0, d0, L1, d1);
        }
    } else {
        double L0[16], L1[16];
        fetch_block(L0, 1 + wave, 0);
        __syncthreads();
        for (int J = 0; J + 1 < blocks; ++J) {
            // the values of rows 16 J .. 16 J + 15 off rows 16 (J + 2) and below
            double y[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) y[u] = x[16 * J + u];
            auto take_off = [&](const double (&L)[16], int m) __attribute__((always_inline)) {
                double v = x[16 * m + l];
#pragma unroll
                for (int k = 0; k < 16; ++k) v -= L[k] * y[k];
                x[16 * m + l] = v;
            };
            int m = J + 1 + wave;
            for (; m < blocks; m += 2 * (kSubWaves - 1)) {
                fetch_block(L1, m + kSubWaves - 1, J);
                __builtin_amdgcn_sched_barrier(0);
                take_off(L0, m);
                if (m + kSubWaves - 1 >= blocks) break;
                fetch_block(L0, m + 2 * (kSubWaves - 1), J);
                __builtin_amdgcn_sched_barrier(0);
                take_off(L1, m + kSubWaves - 1);
            }
            fetch_block(L0, J + 2 + wave, J + 1);
            __syncthreads();
        }
    }
    // backward
    double *products = X + NC * (Q + 16);                          // [2][NC][Q + 16] of row i in products[i & 1]
    double *ends = products + 2 * NC * (Q + 16) + kSubSpare;       // [2][4] row i's diagonal entry, the two beside it, 1 / the first
    const int ht = tid - 64;
    if (ht >= kSubHelpers) {
        for (int i = Q; i >= 0; --i) __syncthreads();               // (beside the first wavefront they would take its turns)
    } else if (ht >= 0) {
        double ring[kSubDepth][kPer];
        // entries i + ht + kSubHelpers u of row i of L^T
        auto fetch_row = [&](int i, double (&L)[kPer]) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < kPer; ++u) L[u] = a.M[(size_t)max(i, 0) * Q + min(max(i, 0) + ht + kSubHelpers * u, Q - 1)];
        };
        auto lay_out = [&](int i, const double (&L)[kPer]) __attribute__((always_inline)) {
            double *dst = products + (i & 1) * NC * (Q + 16);
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int k = i + ht + kSubHelpers * u;
                if (i < 0 || k >= Q) continue;
                if (u == 0 && ht < 3) {
                    ends[4 * (i & 1) + ht] = L[u];
                    if (ht == 0) ends[4 * (i & 1) + 3] = divisor_reciprocal(L[u]);
                    continue;
                }
#pragma unroll
                for (int cc = 0; cc < NC; ++cc) dst[cc * (Q + 16) + k] = L[u] * X[cc * (Q + 16) + k];
            }
        };
#pragma unroll
        for (int u = 0; u < kSubDepth; ++u) fetch_row(Q - 1 - u, ring[u]);
        // (the first two rows have no products but those beside the diagonal)
        lay_out(Q - 1, ring[0]);
        fetch_row(Q - 1 - kSubDepth, ring[0]);
        lay_out(Q - 2, ring[1]);
        fetch_row(Q - 2 - kSubDepth, ring[1]);
        __syncthreads();
        for (int i0 = Q - 1; i0 >= 0; i0 -= kSubDepth) {            // (Q is a multiple of kSubDepth)
#pragma unroll
            for (int u = 0; u < kSubDepth; ++u) {
                const int i = i0 - u;
                __syncthreads();                                    // (row i's subtractions are done, row i + 1 is found)
                lay_out(i - 2, ring[(u + 2) % kSubDepth]);
                fetch_row(i - 2 - kSubDepth, ring[(u + 2) % kSubDepth]);
            }
        }
    } else {
        double minus_one = -1.0, v1 = 0.0, v2 = 0.0;                // rows i + 1 and i + 2
        __builtin_amdgcn_s_setprio(3);
        asm("" : "+v"(minus_one));
        double start, t, p[4], diagonal, beside1, beside2, reciprocal;
        auto row_at = [&](int i) __attribute__((always_inline)) {
            return products + ((i & 1) * NC + min(lane >> 4, NC - 1)) * (Q + 16) + l;
        };
        auto ask = [&](int i) __attribute__((always_inline)) {
            const double *row = row_at(i) + 16 * ((i + 1) >> 4), *end = ends + 4 * (i & 1);
            start = x[i];
            diagonal = end[0]; beside1 = end[1]; beside2 = end[2]; reciprocal = end[3];
            t = row[0];
#pragma unroll
            for (int u = 0; u < 4; ++u) p[u] = row[16 * (1 + u)];        // (past the last block: read, not used)
        };
        __syncthreads();
        ask(Q - 1);
        for (int i = Q - 1; i >= 0; --i) {
            const int first = (i + 1) >> 4, k0 = 16 * first + l;
            const double *row = row_at(i);
            double acc = start;
            if (first < blocks) {
                const double product1 = beside1 * v1, product2 = beside2 * v2;
                t = k0 > i + 2 ? t : k0 == i + 1 ? product1 : k0 == i + 2 ? product2 : 0.0;
                p[0] = k0 + 16 == i + 2 ? product2 : p[0];
                add_16_in_order(acc, t, minus_one);
                // (two sets of products in turn, not moved: a move would cost as much as a step)
                double q[4];
                int m = first + 1;
                auto next = [&](double (&set)[4], int from) __attribute__((always_inline)) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) set[u] = row[16 * (from + u)];
                    __builtin_amdgcn_sched_barrier(0);
                };
                auto rest = [&](const double (&set)[4]) __attribute__((always_inline)) {
                    if (m < blocks) add_16_in_order(acc, set[0], minus_one);
                    if (m + 1 < blocks) add_16_in_order(acc, set[1], minus_one);
                    if (m + 2 < blocks) add_16_in_order(acc, set[2], minus_one);
                };
                while (true) {
                    if (m + 4 > blocks) {
                        rest(p);
                        break;
                    }
                    next(q, m + 4);
                    add_64_in_order(acc, p, minus_one);
                    m += 4;
                    if (m + 4 > blocks) {
                        rest(q);
                        break;
                    }
                    next(p, m + 4);
                    add_64_in_order(acc, q, minus_one);
                    m += 4;
                }
            }
            __syncthreads();                                        // (row i - 1 is laid out)
            const double d = diagonal, r = reciprocal;
            if (i > 0) ask(i - 1);
            __builtin_amdgcn_sched_barrier(0);
            v2 = v1;
            v1 = divide(acc, d, r);
            if (l == 0) x[i] = v1;
        }
    }
    __syncthreads();
    for (int idx = tid; idx < Q * NC; idx += 64 * kSubWaves) {
        const int i = idx / NC, cc = idx % NC;
        if (col0 + cc < D) a.P[(size_t)i * D + col0 + cc] = (float)X[cc * (Q + 16) + i];
    }
}

template <int NC, int kPer>
int launch_substitution(const ProtoArgs &a, hipStream_t stream)
{
    if (int rc = allow_full_lds<substitution_kernel<NC, kPer>>(); rc != MADDNESS_OK) return rc;
    hipLaunchKernelGGL((substitution_kernel<NC, kPer>), dim3((a.D + NC - 1) / NC), dim3(64 * kSubWaves), substitution_lds_bytes(a.Q, NC), stream, a);
    return MADDNESS_OK;
}

// Bucket means on the codebook's own columns, 0 elsewhere and for an empty bucket.
__global__ __launch_bounds__(64) void means_kernel(const ProtoArgs a)
{
    const int c = blockIdx.z, k = blockIdx.y;
    const int col = blockIdx.x * 64 + threadIdx.x;
    if (col >= a.D) return;
    float out = 0.0f;
    if (col >= a.bounds[2 * c] && col < a.bounds[2 * c + 1]) {
        double sum = 0.0;
        int64_t count = 0;
        for (int64_t n = 0; n < a.N; ++n)
            if (a.codes[n * a.C + c] == k) {
                sum += (double)a.A[n * a.lda + col];
                ++count;
            }
        if (count > 0) out = (float)(sum / (double)count);
    }
    a.P[((size_t)c * 16 + k) * a.D + col] = out;
}

size_t align_up(size_t v, size_t al) { return (v + al - 1) / al * al; }

// carves `bytes` (rounded up to 256) off the workspace
struct Carver {
    unsigned char *at;
    size_t used = 0;
    template <typename T>
    T *take(size_t count)
    {
        T *p = reinterpret_cast<T *>(at + used);
        used += align_up(count * sizeof(T), 256);
        return p;
    }
};

void carve_trees(Carver &w, LearnArgs &a)
{
    const size_t C = a.C;
    a.exact_levels = w.take<int32_t>(2 * C);      // (the workspace begins with it: maddness.h)
    a.bounds = w.take<int32_t>(2 * C);
    a.pitch = a.dmax <= 8 ? 8 : (a.dmax + 15) / 16 * 16;
    a.X = w.take<float>(C * (a.N + 1) * a.pitch);
    a.chunk_count = w.take<int32_t>(4 * C * kMaxChunks * kSplitBuckets);
    a.range_part = w.take<int32_t>(2 * C * kRangeParts);
    a.node = w.take<uint8_t>(C * a.N);      // (right behind chunk_count and range_part: all three are cleared together)
    a.range = w.take<int32_t>(2 * C);
    a.varying_part = w.take<uint32_t>(C * kRangeParts * a.pitch);
    a.varying = w.take<uint32_t>(C * a.pitch);
    a.cand_varying = w.take<uint32_t>(C * kCand);
    a.col_loss = w.take<double>(C * kSplitBuckets * a.dmax);
    a.bucket_count = w.take<int64_t>(C * kSplitBuckets);
    a.bucket_start = w.take<int32_t>(C * kSplitBuckets);
    a.rows_by_bucket = w.take<int32_t>(C * a.N);
    a.cand = w.take<int32_t>(C * kCand);
    a.n_cand = w.take<int32_t>(C);
    a.keys = w.take<uint64_t>(C * kCand * a.N);
    if (a.N > kSortRound) {
        a.keys2 = w.take<uint64_t>(C * kCand * a.N);
        a.digit_counts = w.take<uint32_t>(C * kCand * kMaxSortChunks * kSortBins);
    }
    a.tile_slots = a.N / kSplitRows + kSplitBuckets + 1;
    a.sums = w.take<double>(C * kCand * 2 * a.tile_slots * 2 * a.dmax);
    a.group_slots = a.N / kGroupRows + kSplitBuckets + 1;
    a.part_slots = a.N / kPartRows + kSplitBuckets + 1;
    a.parts = w.take<double>(C * a.part_slots * kPartValues * a.dmax);
    a.original = w.take<int32_t>(C * a.dmax);
    a.may_compare = w.take<int64_t>(C);
    a.energy = w.take<double>(C * kSplitBuckets);
    a.unsure = w.take<int32_t>(2 * C);
    a.group_sums = w.take<double>(C * kCand * a.group_slots * a.dmax);
    a.totals = w.take<double>(C * kCand * kSplitBuckets * a.dmax);
    a.group_gain = w.take<double>(C * kCand * a.group_slots * 2);
    a.group_first = w.take<int32_t>(C * kCand * a.group_slots);
    a.group_loss = w.take<double>(C * kCand * a.group_slots);
    a.group_at = w.take<int32_t>(C * kCand * a.group_slots * 2);
    a.chosen = w.take<int32_t>(C);
}

// four wavefronts to a SIMD of 256 compute units in all; at most 2 MiB of their sums
int64_t most_shares(int32_t D, int32_t C) { return std::max<int64_t>(1, 4096 / (((int64_t)D + 63) / 64 * 16 * C)); }

void carve_prototypes(Carver &w, ProtoArgs &a)
{
    const size_t Q = a.Q;
    a.bounds = w.take<int32_t>(2 * (size_t)a.C);
    a.counts = w.take<int32_t>(Q * Q);
    a.range_part = w.take<int32_t>((size_t)(a.D + 63) / 64 * kProtoParts * 2);
    a.any_order = w.take<int32_t>((size_t)(a.D + 63) / 64);
    a.R_shares = w.take<double>((size_t)(most_shares(a.D, a.C) - 1) * Q * a.D);
    a.M = w.take<double>(Q * Q);
    a.Lr = w.take<double>(Q * Q);
    a.R = w.take<double>(Q * a.D);
    a.list = w.take<uint32_t>((size_t)a.C * (kListRows + kListSpare));
    a.list_count = w.take<int32_t>((size_t)a.C * kListChunks * 16);
    a.list_start = w.take<int32_t>((size_t)a.C * 17);
}

}  // namespace

namespace {

size_t batch_bytes(int64_t N, int32_t C, int32_t dmax)
{
    LearnArgs a{};
    a.N = N; a.C = C; a.dmax = dmax;
    Carver w{nullptr};
    carve_trees(w, a);
    return w.used;
}

// Trees do not depend on each other, so the codebooks are taken in batches, one after the other in the same workspace: as
// many as stay within `limit`, one at least.  The codebooks' columns (X) and running sums (sums) take 8 bytes per row and
// column, keys and lists of rows 69 per row and codebook, twice which for all codebooks is the limit above 4 GiB; sums of groups and
// parts of rows a byte for seven columns of a row, the counters up to a megabyte.  Without a limit 2^20 rows of 16 subspaces
// of 128 columns take 17.4 GiB, and one wide subspace makes all others of its batch as wide.  Returns one past the batch's last
// codebook, its widest subspace in *dmax.
int32_t batch_end(int64_t N, int32_t C, const int32_t *bounds, int32_t first, int32_t *dmax)
{
    const size_t limit = std::max<size_t>((size_t)4 << 30, 2 * (size_t)C * 69 * (size_t)N);
    *dmax = 0;
    int32_t end = first;
    for (; end < C; ++end) {
        const int32_t widest = std::max(*dmax, bounds[2 * end + 1] - bounds[2 * end]);
        if (end > first && batch_bytes(N, end + 1 - first, widest) > limit) break;
        *dmax = widest;
    }
    return end;
}

}  // namespace

size_t learn_trees_workspace_bytes(int64_t N, int32_t C, const int32_t *bounds)
{
    size_t bytes = 0;
    for (int32_t c = 0; c < C;) {
        int32_t dmax = 0;
        const int32_t end = batch_end(N, C, bounds, c, &dmax);
        bytes = std::max(bytes, batch_bytes(N, end - c, dmax));
        c = end;
    }
    return bytes;
}

size_t learn_prototypes_workspace_bytes(int32_t D, int32_t C)
{
    ProtoArgs a{};
    a.D = D; a.C = C; a.Q = 16 * C;
    Carver w{nullptr};
    carve_prototypes(w, a);
    return w.used;
}

int learn_max_subspace_width() { return kMaxWidth; }

#define LAUNCH_OK(what)                                                       \
    if (int rc_ = check_hip(hipGetLastError(), what); rc_ != MADDNESS_OK) return rc_

static int launch_learn_batch(LearnArgs a, const int32_t *bounds_host, void *workspace, hipStream_t stream)
{
    const int64_t N = a.N;
    const int32_t C = a.C, dmax = a.dmax;
    Carver w{static_cast<unsigned char *>(workspace)};
    carve_trees(w, a);
    a.row_bits = N > 1 ? 64 - __builtin_clzll((unsigned long long)(N - 1)) : 0;
    const bool narrow = dmax <= 8;
    // (few rows: their chains take no longer than the estimates' seven launches a level, the sooner so the fewer chains there are.
    // The trees of 2048 rows of 64 columns, 8 codebooks: 350 us with estimates, 320 to 333 without; 3000: 366 and 367 to 389; 2100, 4
    // codebooks: 347 and 384 to 402; 2048 of 512, 32 codebooks: 390 and 460)
    const bool estimated = N >= (narrow ? 3072 : 2048);
    Bounds b{};
    for (int i = 0; i < 2 * C; ++i) b.v[i] = bounds_host[i];
    hipLaunchKernelGGL(begin_trees_kernel, dim3(1), dim3(256), 0, stream, b, a, estimated);
    LAUNCH_OK("launch begin_trees_kernel");
    const int64_t clear_words = (a.node + (size_t)C * N - reinterpret_cast<uint8_t *>(a.chunk_count) + 3) / 4;
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)((clear_words + 255) / 256)), dim3(256), 0, stream, a.chunk_count, clear_words);
    LAUNCH_OK("launch clear_kernel");

    const int64_t pieces = (N + 1) * (a.pitch / 4);
    a.gather_parts = (int32_t)std::min<int64_t>((pieces + 255) / 256, kRangeParts);
    a.look = N > kSortThreads && 256 % (a.pitch / 4) == 0 ? 1 : 0;
    if (a.look) hipLaunchKernelGGL(gather_columns_kernel<true>, dim3((unsigned)a.gather_parts, C), dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(gather_columns_kernel<false>, dim3((unsigned)a.gather_parts, C), dim3(256), 0, stream, a);
    LAUNCH_OK("launch gather_columns_kernel");

    for (int level = 0; level < 4; ++level) {
        const int n_buckets = 1 << level;
        hipLaunchKernelGGL(order_rows_kernel, dim3((unsigned)((N + order_chunk_rows(N) - 1) / order_chunk_rows(N)), C), dim3(256), 0,
                           stream, a, level, n_buckets);
        LAUNCH_OK("launch order_rows_kernel");
        const dim3 grid_parts((unsigned)(a.part_slots * C)), grid_bucket_loss(C, n_buckets, a.pitch / 4);
        if (estimated) {
            if (narrow) hipLaunchKernelGGL(loss_parts_kernel<8>, grid_parts, dim3(256), 0, stream, a, n_buckets);
            else hipLaunchKernelGGL(loss_parts_kernel<16>, grid_parts, dim3(256), 0, stream, a, n_buckets);
            LAUNCH_OK("launch loss_parts_kernel");
            hipLaunchKernelGGL(select_kernel, dim3(C), dim3(512), 0, stream, a, level, n_buckets);
            LAUNCH_OK("launch select_kernel");
        }
        hipLaunchKernelGGL(bucket_loss_kernel, grid_bucket_loss, dim3(4 * 64 + kChainHelpers), stream_lds_bytes<4>(), stream, a, 0);
        LAUNCH_OK("launch bucket_loss_kernel");
        if (N <= kSortThreads) {
            hipLaunchKernelGGL(sort_few_kernel, dim3(1, kCand, C), dim3((unsigned)((N + 63) / 64 * 64)), 0, stream, a, n_buckets);
            LAUNCH_OK("launch sort_few_kernel");
        } else if (N <= kSortRound) {
            hipLaunchKernelGGL(sort_round_kernel, dim3(1, kCand, C), dim3(kSortThreads), 0, stream, a, n_buckets);
            LAUNCH_OK("launch sort_round_kernel");
        } else {
            const dim3 chunks((unsigned)((N + sort_chunk_rows(N) - 1) / sort_chunk_rows(N) * C), kCand);
            for (int k = 0; k < kSortDigits; ++k) {
                hipLaunchKernelGGL(sort_count_kernel, chunks, dim3(kSortThreads), 0, stream, a, k, n_buckets);
                LAUNCH_OK("launch sort_count_kernel");
                hipLaunchKernelGGL(sort_scatter_kernel, chunks, dim3(kSortThreads), 0, stream, a, k, n_buckets);
                LAUNCH_OK("launch sort_scatter_kernel");
            }
        }
        // (columns eight or sixteen at a time)
        const int groups = narrow ? 1 : a.pitch / 16;
        if (estimated) {
            const int at_once = narrow ? 16 : 8;              // groups to a workgroup
            const dim3 grid_tiles((unsigned)((a.group_slots + at_once - 1) / at_once * C), kCand);
            if (narrow) hipLaunchKernelGGL(tile_sums_kernel<8>, grid_tiles, dim3(256), 0, stream, a, n_buckets);
            else hipLaunchKernelGGL(tile_sums_kernel<16>, grid_tiles, dim3(256), 0, stream, a, n_buckets);
            LAUNCH_OK("launch tile_sums_kernel");
            hipLaunchKernelGGL(scan_groups_kernel, dim3(C * kCand, n_buckets, groups), dim3(16 * kScanThreads), 0, stream, a);
            LAUNCH_OK("launch scan_groups_kernel");
            if (narrow) hipLaunchKernelGGL(split_gains_kernel<8>, grid_tiles, dim3(256), 0, stream, a, n_buckets);
            else hipLaunchKernelGGL(split_gains_kernel<16>, grid_tiles, dim3(256), 0, stream, a, n_buckets);
            LAUNCH_OK("launch split_gains_kernel");
            hipLaunchKernelGGL(choose_by_gain_kernel, dim3(C), dim3(1024), 0, stream, a, level, n_buckets);
            LAUNCH_OK("launch choose_by_gain_kernel");
            // the codebooks whose splits are unsure and whose exact losses are asked for
            hipLaunchKernelGGL(bucket_loss_kernel, grid_bucket_loss, dim3(4 * 64 + kChainHelpers), stream_lds_bytes<4>(), stream, a, 1);
            LAUNCH_OK("launch bucket_loss_kernel");
        }
        const dim3 chain_groups(C, 8 * groups, n_buckets);
        const dim3 grid_losses((unsigned)(a.group_slots * C), kCand);
        // (where buckets of one tile can be the rule: even shares of the rows are)
        const int small_too = N <= (int64_t)kChainRows * n_buckets;
        const dim3 small_groups(C, 4 * groups, n_buckets);
        if (small_too) {
            if (narrow) hipLaunchKernelGGL(split_chains_small_kernel<8>, small_groups, dim3(16 * 8), 0, stream, a);
            else hipLaunchKernelGGL(split_chains_small_kernel<16>, small_groups, dim3(16 * 16), 0, stream, a);
            LAUNCH_OK("launch split_chains_small_kernel");
        }
        if (N > (small_too ? kChainRows : 1)) {
            if (narrow) hipLaunchKernelGGL(split_chains_kernel<8>, chain_groups, dim3(32 * 8 + kChainHelpers), stream_lds_bytes<8>(), stream, a, small_too);
            else hipLaunchKernelGGL(split_chains_kernel<16>, chain_groups, dim3(32 * 16 + kChainHelpers), stream_lds_bytes<16>(), stream, a, small_too);
            LAUNCH_OK("launch split_chains_kernel");
        }
        if (narrow) hipLaunchKernelGGL(split_losses_kernel<8>, grid_losses, dim3(64), 0, stream, a, n_buckets);
        else hipLaunchKernelGGL(split_losses_kernel<16>, grid_losses, dim3(64), 0, stream, a, n_buckets);
        LAUNCH_OK("launch split_losses_kernel");
        hipLaunchKernelGGL(choose_kernel, dim3(C), dim3(512), 0, stream, a, level, n_buckets);
        LAUNCH_OK("launch choose_kernel");
        hipLaunchKernelGGL(apply_kernel, dim3((unsigned)((N + 255) / 256), C), dim3(256), 0, stream, a, level, n_buckets);
        LAUNCH_OK("launch apply_kernel");
    }
    return MADDNESS_OK;
}

int launch_learn_trees(const float *A, int64_t N, int64_t lda, int32_t C, const int32_t *bounds_host, int32_t *split_dims,
                       float *thresholds, uint8_t *codes, void *workspace, hipStream_t stream)
{
    note_kernel("gather_columns_kernel + order_rows_kernel + loss_parts_kernel + select_kernel + bucket_loss_kernel + sort_few_kernel + sort_round_kernel + sort_count_kernel + sort_scatter_kernel + tile_sums_kernel + scan_groups_kernel + split_gains_kernel + choose_by_gain_kernel + split_chains_small_kernel + split_chains_kernel + split_losses_kernel + choose_kernel + apply_kernel", nullptr);
    for (int32_t c = 0; c < C;) {
        LearnArgs a{};
        const int32_t end = batch_end(N, C, bounds_host, c, &a.dmax);
        a.A = A; a.lda = lda; a.N = N; a.C = end - c;
        a.split_dims = split_dims + 4 * c; a.thresholds = thresholds + 16 * c;
        a.codes = codes ? codes + c : nullptr; a.codes_pitch = C;
        if (int rc = launch_learn_batch(a, bounds_host + 2 * c, workspace, stream); rc != MADDNESS_OK) return rc;
        c = end;
    }
    return MADDNESS_OK;
}

int launch_learn_prototypes(const uint8_t *codes, const float *A, int64_t N, int64_t lda, int32_t D, int32_t C,
                            const int32_t *bounds_host, bool ridge, double lambda, float *prototypes, void *workspace,
                            hipStream_t stream)
{
    ProtoArgs a{};
    a.codes = codes; a.A = A; a.lda = lda; a.N = N; a.D = D; a.C = C; a.Q = 16 * C; a.P = prototypes;
    Carver w{static_cast<unsigned char *>(workspace)};
    carve_prototypes(w, a);
    Bounds b{};
    for (int i = 0; i < 2 * C; ++i) b.v[i] = bounds_host[i];
    hipLaunchKernelGGL(upload_bounds_kernel, dim3(1), dim3(256), 0, stream, b, 2 * C, a.bounds);
    LAUNCH_OK("launch upload_bounds_kernel");
    if (!ridge) {
        note_kernel("means_kernel", nullptr);
        hipLaunchKernelGGL(means_kernel, dim3((D + 63) / 64, 16, C), dim3(64), 0, stream, a);
        LAUNCH_OK("launch means_kernel");
        return MADDNESS_OK;
    }
    note_kernel("prepare_kernel + cooccurrence_kernel + count_codes_kernel + list_codes_kernel + gta_kernel + cholesky_panel_kernel + substitution_kernel", nullptr);
    const int64_t QQ = (int64_t)a.Q * a.Q;
    a.row_bits = N > 1 ? 64 - __builtin_clzll((unsigned long long)(N - 1)) : 0;
    // (each with 64 rows or more)
    a.shares = (int)std::max<int64_t>(1, std::min<int64_t>(most_shares(D, C), std::min<int64_t>(N, kListRows) / 16 / 64));
    hipLaunchKernelGGL(prepare_kernel, dim3((unsigned)(kProtoClear + (a.shares > 1 ? (D + 63) / 64 * kProtoParts : 0))), dim3(256), 0, stream, a);
    LAUNCH_OK("launch prepare_kernel");
    // (stretches of at least 2048 rows, and about four workgroups per compute unit)
    const int co_groups = (C + kCoGroup - 1) / kCoGroup;
    const int64_t stretches = std::max<int64_t>(1, std::min<int64_t>(N / 2048, 4 * device_info().cus / (C * co_groups)));
    hipLaunchKernelGGL(cooccurrence_kernel, dim3(C, co_groups, (unsigned)stretches), dim3(256), 0, stream, a);
    LAUNCH_OK("launch cooccurrence_kernel");
    hipLaunchKernelGGL(ridge_matrix_kernel, dim3((unsigned)((QQ + 255) / 256)), dim3(256), 0, stream, a, lambda);
    LAUNCH_OK("launch ridge_matrix_kernel");
    a.stretch = std::min<int64_t>(kListRows, std::max<int64_t>(1, (1LL << 30) / lda));
    for (int64_t first = 0; first < N; first += a.stretch) {
        const int64_t rows = std::min<int64_t>(N - first, a.stretch);
        const dim3 chunks(C, (unsigned)((rows + kListChunk - 1) / kListChunk));
        hipLaunchKernelGGL(count_codes_kernel, chunks, dim3(256), 0, stream, a, first);
        LAUNCH_OK("launch count_codes_kernel");
        hipLaunchKernelGGL(list_codes_kernel, chunks, dim3(256), 0, stream, a, first);
        LAUNCH_OK("launch list_codes_kernel");
        hipLaunchKernelGGL(gta_kernel, dim3((D + 63) / 64, 4, C * a.shares), dim3(256), 0, stream, a, first);
        LAUNCH_OK("launch gta_kernel");
    }
    for (int J0 = 0; J0 < a.Q; J0 += kCholPanel) {
        const unsigned tiles = std::max(1, (a.Q - J0 - kCholPanel + kCholTile - 1) / kCholTile);
        hipLaunchKernelGGL(cholesky_panel_kernel, dim3(tiles, tiles), dim3(256), 0, stream, a, J0);
        LAUNCH_OK("launch cholesky_panel_kernel");
    }
    const int64_t share_blocks = a.shares > 1 ? ((int64_t)a.Q * D + 255) / 256 : 0;
    hipLaunchKernelGGL(transpose_factor_kernel, dim3((unsigned)((QQ + 255) / 256 + share_blocks)), dim3(256), 0, stream, a);
    LAUNCH_OK("launch transpose_factor_kernel");
    const size_t lds_limit = (size_t)device_info().lds_per_block;
    if (substitution_lds_bytes(a.Q, 1) > lds_limit)
        return fail(MADDNESS_E_UNSUPPORTED, "maddness_learn_prototypes: a column of 16 C values does not fit in LDS");
    // (a helper's registers hold its entries of a row: Q / kSubHelpers of them)
    int rc = MADDNESS_OK;
    if (a.Q <= 3 * kSubHelpers) rc = launch_substitution<4, 3>(a, stream);
    else if (a.Q <= 6 * kSubHelpers) rc = launch_substitution<4, 6>(a, stream);
    else if (substitution_lds_bytes(a.Q, 4) <= lds_limit && a.Q <= 9 * kSubHelpers) rc = launch_substitution<4, 9>(a, stream);
    else rc = launch_substitution<1, 22>(a, stream);
    if (rc != MADDNESS_OK) return rc;
    LAUNCH_OK("launch substitution_kernel");
    return MADDNESS_OK;
}

}  // namespace maddness
