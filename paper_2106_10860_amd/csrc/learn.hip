// The learning step on the GPU: the greedy construction of the hashing trees (Section 4.2,
// Algorithm 2; Appendix C, Algorithms 3 and 4) and the prototypes (bucket means; ridge
// regression, Section 4.3).  Set-up work, run once per problem; what matters here is that
// it takes milliseconds instead of seconds and that its decisions can be checked.
//
// Every quantity a decision depends on (bucket losses, cumulative SSEs, level losses) is
// computed in fp64 with the operations in the order Algorithms 2-4 state them - sums over the
// rows of a bucket run sequentially in sorted (or row) order, sums over the columns of the
// subspace in column order - so that the trees are reproducible to the bit and do not depend
// on the launch shape.  The parallelism is ACROSS the independent pieces: codebooks, candidate
// columns, buckets and columns.  This file is compiled without floating-point contraction.
//
// The serial parts are chains of a few instructions per row on a few lanes, and a wavefront issues
// one vector instruction in four cycles whatever the number of its active lanes: each chain is kept
// to the instructions its sum needs, reads operands that all threads have laid side by side in LDS,
// and leaves products, divisions, comparisons and counting to all threads or to wavefront ballots.
//
// gather_columns_kernel  the columns of every codebook side by side, rows aligned
// Per level t = 1..4 of all C trees at once:
//   order_rows_kernel    the rows of every bucket listed in row order, the bucket sizes
//   bucket_loss_kernel   L(j, B) (Section 4.2) for every column j of every bucket, two passes
//                        over the bucket's own rows
//   select_kernel        heuristic_select_idxs: the four columns with the largest summed loss
//   key_kernel, sort_chunks_kernel, sort_exchange_kernel  the rows ordered by each candidate column (bitonic sort of
//                        (value, row) keys: equal values stay in row order, as a stable sort
//                        of a bucket's rows leaves them)
//   split_chains_kernel, judge_kernel  Algorithm 3 for every bucket of the level: Algorithm 4's
//                        running sums at every 32nd row in both directions, then the loss of
//                        every split, a wavefront per 256 rows
//   choose_kernel        the best threshold and loss per bucket, Algorithm 2's choice among the
//                        candidates
//   apply_kernel         apply_split: the next level's buckets
// Prototypes: cooccurrence_kernel (G^T G), count_codes_kernel, list_codes_kernel and gta_kernel (G^T A~), cholesky_panel_kernel,
// factor by rows, substitution_kernel; or means_kernel.
#include "common.h"

namespace maddness {
namespace {

constexpr int kSplitBuckets = 8;   // buckets of the deepest level that is split (level 4 splits 8)
constexpr int kCand = 4;           // candidate columns per level (Section 4.2: n = 4)
constexpr int kSortChunk = 8192;   // keys sorted in LDS at a time (64 KiB)

struct Bounds {
    int32_t v[2 * MADDNESS_MAX_C];
};

struct LearnArgs {
    const float *A;
    int64_t lda, N, Npad;
    int32_t C, dmax;
    int32_t *bounds;      // [C][2] first and one-past-last column of every codebook
    int32_t pitch;        // values of a row of X: dmax rounded up to whole groups of columns
    float *X;             // [C][N + 1][pitch] the codebook's columns of A, then zeros; row N is zeros
    uint8_t *node;        // [C][N] bucket (0-based) of every row in the current level
    double *col_loss;     // [C][8][dmax] L(j, B_i)
    double *bucket_loss;  // [C][8] L(B_i)
    int64_t *bucket_count;  // [C][8]
    int32_t *bucket_start;  // [C][8] where the bucket's rows begin in rows_by_bucket[c]
    int32_t *chunk_count;   // [4][C][kMaxChunks][8] rows of every bucket in every chunk of rows, by level
    int32_t *rows_by_bucket;  // [C][N] the rows of bucket 0 in row order, then those of bucket 1, ...
    int32_t *cand;        // [C][4] candidate columns (within the subspace), best first
    int32_t *n_cand;      // [C]
    uint64_t *keys;       // [C][4][Npad] sorted (value, row) keys
    int64_t tile_slots;   // tiles of kJudgeRows sorted rows of all buckets of a level, at most
    double *sums;         // [C][4][2][tile_slots][2][dmax] Algorithm 4's running sums before every tile, up and down
    int64_t group_slots;  // groups of kGroupTiles tiles of all buckets of a level, at most
    double *group_loss;   // [C][4][group_slots] loss of the group's best split
    int32_t *group_at;    // [C][4][group_slots][2] the bucket's row it comes after (-1: none); the group's first split
                          // if its loss is not a number (else -1)
    int32_t *chosen;      // [C] the level's column (within the subspace)
    int32_t *split_dims;  // out [C][4]
    float *thresholds;    // out [C][16]
    uint8_t *codes;       // out [N][C] or null
};

__global__ void upload_bounds_kernel(const Bounds b, int32_t n, int32_t *dst)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = b.v[i];
}

__global__ void clear_kernel(int32_t *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// The columns of every codebook side by side, each row on a 32-byte (or 64-byte) boundary.  The levels read the rows of a
// bucket in many orders, a codebook's columns at a time: from here they take whole 16-byte pieces, and the rows of a
// codebook fit in an XCD's L2 where A does not.  A thread per 16-byte piece.
__global__ __launch_bounds__(256) void gather_columns_kernel(const LearnArgs a)
{
    const int c = blockIdx.y, pieces = a.pitch / 4;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t row = i / pieces;
    if (row > a.N) return;
    const int col = 4 * (int)(i - row * pieces), lo = a.bounds[2 * c], d = a.bounds[2 * c + 1] - lo;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = row < a.N && col + e < d ? a.A[row * a.lda + lo + col + e] : 0.0f;
    reinterpret_cast<float4 *>(a.X + (size_t)c * (a.N + 1) * a.pitch)[i] = make_float4(v[0], v[1], v[2], v[3]);
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
constexpr int kChainPitch = kChainRows + 4;                  // (a wavefront's writes, 16 rows of every fourth column, meet in no bank)
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

// The chains' part of a tile: `at` is the lane's first value (its 16th of the column's), term(x, i) the term of value x in
// row i of the lane's; before(k) runs before every 32nd row.
template <typename Term, typename Before>
__device__ __forceinline__ void add_tile_in_order(double &acc, const float *at, Term term, Before before)
{
    double one = 1.0;
    asm("" : "+v"(one));
    float x[kChainRows / 16];
#pragma unroll
    for (int i = 0; i < kChainRows / 16; ++i) x[i] = at[16 * i];
#pragma unroll
    for (int i = 0; i < kChainRows / 16; ++i) {
        if (i % 2 == 0) before(i / 2);
        add_16_in_order(acc, term(x[i], 16 * i), one);
    }
}

// The workgroup's loop: n_steps tiles of kChainRows rows.  walk(values of tile s, s) runs on the first kWalkers
// wavefronts; meanwhile the helpers lay out tile s + 1, fetch the values of tile s + kDepth + 1 and list the rows of the
// tile after that (row_at(s, i): the number of row i of tile s, `N` where there is none), whose numbers they asked for
// kDepth steps before.  X: the codebook's values, from the workgroup's first column on.
template <int NC>
constexpr size_t stream_lds_bytes() { return sizeof(float) * 2 * NC * kChainPitch + sizeof(int32_t) * kLists * kChainRows; }

template <int NC, int kWalkers, typename RowAt, typename Walk>
__device__ __forceinline__ void stream_rows(unsigned char *lds, const float *X, int pitch, int n_steps, RowAt row_at, Walk walk)
{
    constexpr int kPieces = NC / 4, kStride = kChainHelpers / kPieces, kPer = kChainRows / kStride, kBuffer = NC * kChainPitch;
    float *values = reinterpret_cast<float *>(lds);                        // [2][NC][kChainPitch]
    int32_t *listed = reinterpret_cast<int32_t *>(values + 2 * kBuffer);   // [kLists][kChainRows]
    const int helper = (int)threadIdx.x - 64 * kWalkers, at = helper < 0 ? 0 : helper;
    const int rsub = at / kPieces, piece = at % kPieces;
    const float *src = X + 4 * piece;
    float4 x[kDepth][kPer];
    int32_t next[kDepth];
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
    if (helper >= 0)
#pragma unroll
        for (int s = 0; s < kDepth + 2; ++s) listed[(s % kLists) * kChainRows + helper] = row_at(s, helper);
    __syncthreads();
    if (helper >= 0) {
        fetch(0, 0);
        stash(0, 0);
#pragma unroll
        for (int s = 1; s <= kDepth; ++s) {
            fetch(s, s % kDepth);
            next[s - 1] = row_at(s + kDepth + 1, helper);
        }
    }
    __syncthreads();
    for (int s0 = 0; s0 < n_steps; s0 += kDepth) {
#pragma unroll
        for (int i = 0; i < kDepth; ++i) {
            const int s = s0 + i;
            if (s >= n_steps) break;
            if (helper < 0) {
                walk(values + (s & 1) * kBuffer, s);
            } else {
                stash(s + 1, (i + 1) % kDepth);
                fetch(s + 1 + kDepth, (i + 1) % kDepth);
                listed[((s + kDepth + 2) % kLists) * kChainRows + helper] = next[i];
                next[i] = row_at(s + 2 * kDepth + 2, helper);
            }
            __syncthreads();
        }
    }
}

// L(j, B_i): the sum, then the squared distances from the mean, over the bucket's rows in row order, a chain per
// column, up to NC columns of a bucket to a workgroup.  (Measured, level 1 of 260100 x 27 with 4 codebooks, two sums of
// 260100 rows: 1.6 ms, 3 ns a row; 7.1 ms with a lane per chain that read and converted its values itself.  The four
// levels: 3.3 against 14.6 ms, and 0.39 against 1.75 ms for 20000 x 512 with 32 codebooks.)
template <int NC>
__global__ __launch_bounds__(16 * NC + kChainHelpers) void bucket_loss_kernel(const LearnArgs a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int c = blockIdx.x, b = blockIdx.y, col0 = blockIdx.z * NC;
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    if (col0 >= d) return;
    const int count = (int)a.bucket_count[c * kSplitBuckets + b];
    const int32_t *list = a.rows_by_bucket + (size_t)c * a.N + a.bucket_start[c * kSplitBuckets + b];
    const int n_steps = (count + kChainRows - 1) / kChainRows;
    const int tid = threadIdx.x, cols = min(NC, d - col0);
    const int chain = (tid / 16) % NC, l = tid & 15;
    const float *X = a.X + (size_t)c * (a.N + 1) * a.pitch + col0;
    auto row_at = [&](int s, int i) __attribute__((always_inline)) {
        const int p = s * kChainRows + i;
        return p < count ? list[p] : (int32_t)a.N;
    };
    double sum = 0.0, loss = 0.0;
    stream_rows<NC, NC / 4>(lds_raw, X, a.pitch, n_steps, row_at, [&](const float *values, int) __attribute__((always_inline)) {
        add_tile_in_order(sum, values + chain * kChainPitch + l, [](float x, int) { return (double)x; }, [](int) {});
    });
    const double mean = count > 0 ? sum / (double)count : 0.0;
    stream_rows<NC, NC / 4>(lds_raw, X, a.pitch, n_steps, row_at, [&](const float *values, int s) __attribute__((always_inline)) {
        const int left = count - s * kChainRows - l;
        add_tile_in_order(loss, values + chain * kChainPitch + l, [&](float x, int row) __attribute__((always_inline)) {
            const double e = (double)x - mean;
            return row < left ? e * e : 0.0;          // (adding 0 leaves a sum as it is)
        }, [](int) {});
    });
    if (tid < 16 * NC && l == 0 && chain < cols)
        a.col_loss[((size_t)c * kSplitBuckets + b) * a.dmax + col0 + chain] = count > 0 ? loss : 0.0;
}

// heuristic_select_idxs, and L(B_i) = sum over the columns of L(j, B_i).
__global__ __launch_bounds__(64) void select_kernel(const LearnArgs a, int n_buckets)
{
    extern __shared__ double total[];   // [dmax]
    const int c = blockIdx.x;
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    const double *cl = a.col_loss + (size_t)c * kSplitBuckets * a.dmax;
    for (int jj = threadIdx.x; jj < d; jj += 64) {
        double t = 0.0;
        for (int b = 0; b < n_buckets; ++b) t += cl[(size_t)b * a.dmax + jj];
        total[jj] = t;
    }
    if ((int)threadIdx.x < n_buckets) {
        double l = 0.0;
        for (int jj = 0; jj < d; ++jj) l += cl[(size_t)threadIdx.x * a.dmax + jj];
        a.bucket_loss[c * kSplitBuckets + threadIdx.x] = l;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    const int n_cand = d < kCand ? d : kCand;
    int pick[kCand];
    for (int q = 0; q < n_cand; ++q) {
        int best = -1;
        for (int jj = 0; jj < d; ++jj) {
            bool taken = false;
            for (int p = 0; p < q; ++p) taken |= pick[p] == jj;
            if (!taken && (best < 0 || total[jj] > total[best])) best = jj;   // equal losses: the lower column
        }
        pick[q] = best;
        a.cand[c * kCand + q] = best;
    }
    a.n_cand[c] = n_cand;
}

// (bucket, value, row) keys, 3 + 32 + 29 bits: unsigned order = by bucket, then by value, equal values (-0 counts
// as +0) by row.  The rows of a bucket end up side by side, in the order Algorithm 3 wants them.
constexpr int kKeyRowBits = 29;
__device__ __forceinline__ uint64_t make_key(int bucket, float x, uint32_t row)
{
    const uint32_t bits = __float_as_uint(x + 0.0f);
    const uint32_t u = (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
    return ((uint64_t)bucket << (32 + kKeyRowBits)) | ((uint64_t)u << kKeyRowBits) | row;
}
__device__ __forceinline__ float key_value(uint64_t key)
{
    const uint32_t u = (uint32_t)(key >> kKeyRowBits);
    return __uint_as_float((u & 0x80000000u) ? (u ^ 0x80000000u) : ~u);
}
__device__ __forceinline__ int32_t key_row(uint64_t key) { return (int32_t)(key & ((1u << kKeyRowBits) - 1u)); }

__global__ __launch_bounds__(256) void key_kernel(const LearnArgs a)
{
    const int c = blockIdx.z, q = blockIdx.y;
    if (q >= a.n_cand[c]) return;
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= a.Npad) return;
    const int j = a.cand[c * kCand + q];
    a.keys[((size_t)c * kCand + q) * a.Npad + p] =
        p < a.N ? make_key(a.node[(size_t)c * a.N + p], a.X[((size_t)c * (a.N + 1) + p) * a.pitch + j], (uint32_t)p) : ~0ull;
}

// Bitonic sort of Npad keys (a power of two) per (codebook, candidate).  The exchanges at distances below
// kSortChunk run on chunks of kSortChunk keys in LDS, a workgroup per chunk (sort_chunks_kernel: the stages
// k_first .. k_last whole when j_first is 0, else the distances j_first .. 1 of stage k_first); the exchanges
// at larger distances go through memory, a thread per pair (sort_exchange_kernel: one distance of one stage).
__device__ __forceinline__ void exchange(uint64_t &x, uint64_t &y, bool ascending)
{
    if ((x > y) == ascending) {
        const uint64_t t = x;
        x = y;
        y = t;
    }
}

__global__ __launch_bounds__(1024) void sort_chunks_kernel(const LearnArgs a, int64_t k_first, int64_t k_last, int64_t j_first)
{
    extern __shared__ uint64_t chunk[];   // [min(Npad, kSortChunk)]
    const int c = blockIdx.z, q = blockIdx.y;
    if (q >= a.n_cand[c]) return;
    uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.Npad;
    const int64_t n = a.Npad;
    const int64_t m = n < kSortChunk ? n : kSortChunk;   // chunk length
    const int64_t base = (int64_t)blockIdx.x * m;
    const int tid = threadIdx.x;
    for (int64_t i = tid; i < m; i += 1024) chunk[i] = keys[base + i];
    __syncthreads();
    for (int64_t k = k_first; k <= k_last; k <<= 1) {
        for (int64_t j = (k == k_first && j_first) ? j_first : k >> 1; j > 0; j >>= 1) {
            for (int64_t t = tid; t < m / 2; t += 1024) {
                const int64_t i = 2 * t - (t & (j - 1));   // the lower index of pair t at distance j
                exchange(chunk[i], chunk[i + j], ((base + i) & k) == 0);
            }
            __syncthreads();
        }
    }
    for (int64_t i = tid; i < m; i += 1024) keys[base + i] = chunk[i];
}

__global__ __launch_bounds__(256) void sort_exchange_kernel(const LearnArgs a, int64_t k, int64_t j)
{
    const int c = blockIdx.z, q = blockIdx.y;
    if (q >= a.n_cand[c]) return;
    uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.Npad;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= a.Npad / 2) return;
    const int64_t i = 2 * t - (t & (j - 1));
    const uint64_t x = keys[i], y = keys[i + j];
    if ((x > y) == ((i & k) == 0)) {
        keys[i] = y;
        keys[i + j] = x;
    }
}

// Algorithm 3 in two parts.  Algorithm 4's running sums are the one serial thing in it, and a serial sum costs a
// few cycles per row whatever else is done with it, so split_chains_kernel does nothing but add: a chain per
// (candidate, bucket, direction, column, which of the two sums) walks the bucket's rows in sorted order and leaves its
// value at every kJudgeRows-th of them.  judge_kernel takes it up from there, tile by tile of kJudgeRows rows: it
// repeats the few additions in between (the same operations on the same operands), and does the products, divisions,
// differences and comparisons of its rows, all tiles of all buckets at once.  (Measured, the four levels of
// 20000 x 512 with 32 codebooks and of 260100 x 27 with 4: 0.67 + 0.45 and 2.36 + 0.42 ms for the two kernels; 4.8 and
// 34.8 ms as one kernel that did all of it tile after tile.)
constexpr int kJudgeRows = 32;
constexpr int kGroupTiles = 8, kGroupRows = kGroupTiles * kJudgeRows;     // tiles that a wavefront of judge_kernel takes

// the first of the tile slots of a bucket (count rows beginning at `start` take up to count / kJudgeRows + 1 of them)
__device__ __forceinline__ int64_t first_slot(int32_t start, int bucket) { return start / kJudgeRows + bucket; }
__device__ __forceinline__ int64_t first_group(int32_t start, int bucket) { return start / kGroupRows + bucket; }

// The chains are those of bucket_loss_kernel, both sums of up to NC columns to a workgroup.  Going down (direction 1)
// the tiles are taken last to first, each from its end; what lies past the bucket's last row counts as zeros, which
// leave a sum as it is.
template <int NC>
__global__ __launch_bounds__(32 * NC + kChainHelpers) void split_chains_kernel(const LearnArgs a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    // (the codebook changes fastest from workgroup to workgroup: those of one codebook meet on few XCDs)
    const int c = blockIdx.x, b = blockIdx.z, dir = blockIdx.y & 1, q = (blockIdx.y >> 1) & 3, col0 = (blockIdx.y >> 3) * NC;
    const int d = a.bounds[2 * c + 1] - a.bounds[2 * c];
    if (q >= a.n_cand[c] || col0 >= d) return;
    const int count = (int)a.bucket_count[c * kSplitBuckets + b], start = a.bucket_start[c * kSplitBuckets + b];
    const int n_tiles = (count + kJudgeRows - 1) / kJudgeRows;
    if (n_tiles == 0) return;
    constexpr int kTiles = kChainRows / kJudgeRows;
    const int n_steps = (n_tiles + kTiles - 1) / kTiles;
    const uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.Npad + start;
    const int tid = threadIdx.x, cols = min(NC, d - col0);
    const int chain = (tid / 16) % (2 * NC), l = tid & 15;
    const bool squares = chain >= NC;
    // where the chain's values go: the sums before tile i (of all rows before it, in the direction's order)
    double *out = a.sums + (((size_t)c * kCand + q) * 2 + dir) * a.tile_slots * (2 * a.dmax) +
                  (size_t)first_slot(start, b) * (2 * a.dmax) + (chain / NC) * a.dmax + col0 + chain % NC;
    const bool stored = l == 0 && chain % NC < cols;
    double acc = 0.0;
    stream_rows<NC, NC / 2>(
        lds_raw, a.X + (size_t)c * (a.N + 1) * a.pitch + col0, a.pitch, n_steps,
        [&](int s, int i) __attribute__((always_inline)) {
            const int tile = kTiles * s + i / kJudgeRows, in_tile = i % kJudgeRows;
            const int p = dir ? (n_tiles - 1 - tile) * kJudgeRows + kJudgeRows - 1 - in_tile : tile * kJudgeRows + in_tile;
            if (tile >= n_tiles || p >= count) return (int32_t)a.N;
            return (int32_t)(static_cast<uint32_t>(keys[p]) & ((1u << kKeyRowBits) - 1u));
        },
        [&](const float *values, int s) __attribute__((always_inline)) {
            add_tile_in_order(acc, values + (chain % NC) * kChainPitch + l,
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

// A wavefront per kGroupTiles tiles of kJudgeRows sorted rows of a bucket, one tile after the other with the next one's
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
__global__ __launch_bounds__(64) void judge_kernel(const LearnArgs a, int n_buckets)
{
    constexpr int T = kJudgeRows, kPitch = T + 4, kSumPitch = T + 1, kChains = 4 * NC;
    constexpr int kPieces = NC / 4, kRows = 64 / kPieces, kPer = T / kRows;
    __shared__ __align__(16) double sums[kChains][kSumPitch];
    __shared__ __align__(16) float xs[2][NC][kPitch];       // the tile's values, first to last and last to first
    const int c = blockIdx.x % a.C, q = blockIdx.y, lane = threadIdx.x;
    if (q >= a.n_cand[c]) return;
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
    const uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.Npad + start;
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
    const int n_cand = a.n_cand[c];
    for (int pair = wave; pair < n_cand * n_buckets; pair += 8) {
        const int q = pair / n_buckets, b = pair - q * n_buckets;
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
            const uint64_t *keys = a.keys + ((size_t)c * kCand + q) * a.Npad + start;
            float v = 0.0f;
            if (at >= 0) {
                const float l = key_value(keys[at]), h = key_value(keys[at + 1]);
                v = (float)(((double)l + (double)h) / 2.0);
                if (!(v > l)) v = h;
            } else if (count > 0) {
                // cannot be split: the value of the bucket's first row in sorted order, the loss L(B)
                v = a.X[((size_t)c * (a.N + 1) + key_row(keys[0])) * a.pitch + a.cand[c * kCand + q]];
                loss = a.bucket_loss[c * kSplitBuckets + b];
            }
            res_v[q][b] = v;
            res_loss[q][b] = loss;
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    int best_q = 0;
    double l_min = 0.0;
    for (int q = 0; q < n_cand; ++q) {
        double l = 0.0;
        for (int b = 0; b < n_buckets; ++b) l += res_loss[q][b];
        if (q == 0 || l < l_min) {
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
        if (level == 3 && a.codes) a.codes[n * a.C + c] = (uint8_t)child;
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
    double *M;              // [Q][Q]: G^T G + lambda I, then M[k][i] = L[i][k]
    double *Lr;             // [Q][Q]: L by rows
    double *R;              // [Q][D]: G^T A~
    int64_t stretch;        // rows of a stretch
    uint32_t *list;         // [C][kListRows + kListSpare] distances in bytes of the stretch's rows, by code
    int32_t *list_count;    // [C][kListChunks][16] how many each of its chunks has of every code
    int32_t *list_start;    // [C][17] where those of a code begin
    float *P;               // out [C][16][D]
};

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
// four times as long to keep in L2).
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
    const int k = blockIdx.y * 4 + wave, c = blockIdx.z;
    const int col = blockIdx.x * 64 + lane;
    const int start = a.list_start[c * 17 + k], count = a.list_start[c * 17 + k + 1] - start;
    double *out = a.R + ((size_t)16 * c + k) * a.D + col;
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

// Cholesky factorisation M = L L^T: L_jj = sqrt(M_jj - sum_k L_jk^2), L_ij = (M_ij - sum_k L_ik L_jk) / L_jj,
// every sum over k ascending.  M is symmetric, and L_ik is kept at M[k][i] (rows of a column side by side).
// One launch per panel of 16 columns J0 .. J0 + 15; a workgroup takes the 16 rows of the panel's
// diagonal block (every workgroup works them out for itself, the first one stores them) and 48 rows
// below it, four entries of a row per thread.  First the terms of the columns before the panel, in
// chunks of kCholChunk columns staged in LDS, then the panel's own columns one after the other.
constexpr int kCholPanel = 16, kCholRows = 64, kCholChunk = 32;
__global__ __launch_bounds__(256) void cholesky_panel_kernel(const ProtoArgs a, int J0)
{
    __shared__ __align__(16) double Lc[kCholRows][kCholChunk + 2];     // (rows 4 banks apart: 16-byte reads of 16 rows at once)
    __shared__ double T[kCholRows][kCholPanel + 1];
    const int Q = a.Q;
    double *M = a.M;
    const int tid = threadIdx.x;
    auto global_row = [&](int r) {
        return r < kCholPanel ? J0 + r : J0 + kCholPanel + (int)blockIdx.x * (kCholRows - kCholPanel) + (r - kCholPanel);
    };
    const int r = tid >> 2, cg = tid & 3;
    const int gi = global_row(r);
    double s[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = gi < Q ? M[(size_t)(J0 + 4 * cg + e) * Q + gi] : 0.0;

    // staging: thread -> row (tid & 63) of the chunk, columns (tid >> 6) + 4 u
    const int srow = tid & 63, sk = tid >> 6;
    const int sgi = global_row(srow);
    constexpr int kPer = kCholChunk / 4;
    double pre[kPer];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int k = k0 + sk + 4 * u;
            pre[u] = (sgi < Q && k < J0) ? M[(size_t)k * Q + sgi] : 0.0;
        }
    };
    if (J0 > 0) fetch(0);
    for (int k0 = 0; k0 < J0; k0 += kCholChunk) {
        __syncthreads();                      // the chunk before this one has been used
#pragma unroll
        for (int u = 0; u < kPer; ++u) Lc[srow][sk + 4 * u] = pre[u];
        __syncthreads();
        if (k0 + kCholChunk < J0) fetch(k0 + kCholChunk);
        const int kc = min(kCholChunk, J0 - k0);
        for (int kk = 0; kk < kc; kk += 2) {          // (two columns to an LDS read; kc is a multiple of 16)
            const double2 li = *reinterpret_cast<const double2 *>(&Lc[r][kk]);
            double2 lj[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) lj[e] = *reinterpret_cast<const double2 *>(&Lc[4 * cg + e][kk]);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] -= li.x * lj[e].x;
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] -= li.y * lj[e].y;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) T[r][4 * cg + e] = s[e];
    __syncthreads();

    // the panel's own columns: a thread per row (the first wavefront), the row's entries in registers
    double t[kCholPanel];
    const int row = tid, grow = global_row(tid < kCholRows ? tid : 0);
    if (tid < kCholRows)
#pragma unroll
        for (int j = 0; j < kCholPanel; ++j) t[j] = T[row][j];
#pragma unroll
    for (int j = 0; j < kCholPanel; ++j) {
        if (tid < kCholRows) {
#pragma unroll
            for (int k = 0; k < j; ++k) t[j] -= t[k] * T[j][k];
            if (row == j) {
                t[j] = sqrt(t[j]);
                T[j][j] = t[j];
            }
        }
        __syncthreads();
        if (tid < kCholRows && row != j) {
            t[j] = t[j] / T[j][j];
            if (row < kCholPanel) T[row][j] = t[j];     // a row of the diagonal block: read by the rows below
        }
        __syncthreads();
    }
    if (tid < kCholRows && grow < Q && (row >= kCholPanel || blockIdx.x == 0))
#pragma unroll
        for (int j = 0; j < kCholPanel; ++j)
            if (row >= kCholPanel || j <= row) M[(size_t)(J0 + j) * Q + grow] = t[j];
}

__global__ __launch_bounds__(256) void transpose_factor_kernel(const ProtoArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)a.Q * a.Q) return;
    const int r = (int)(i / a.Q), k = (int)(i - (int64_t)r * a.Q);
    a.Lr[i] = k <= r ? a.M[(size_t)k * a.Q + r] : 0.0;
}

// L y = G^T A~ and L^T P = y, sums over k ascending: y_i = (b_i - sum_{k<i} L_ik y_k) / L_ii, then
// P_i = (y_i - sum_{k>i} L_ki P_k) / L_ii.  A workgroup takes NC columns of A~ and keeps them in LDS
// for both sweeps; the first NC threads carry a column each through the sums (in the second sweep the
// sum of a row begins with the value found just before, so a column's subtractions are one chain),
// while all threads fetch the next row of L (first sweep) or of L^T (second sweep, kept at M) through
// registers into the other of two LDS buffers.  A wavefront issues one vector instruction in four
// cycles, so the chain's loop is kept to the two LDS reads, the product and the subtraction of a term:
// NC is a constant (the reads take immediate offsets) and terms go in batches of kSubBatch without a
// bound check.  A batch may run past the row's last term: there the buffer's entry of L is 0 (buffers
// start as zeros, a row's diagonal entry is kept apart, and kSubPad entries and rows follow the last),
// the term is 0 times a finite value, and subtracting 0 changes nothing.
constexpr int kSubMaxPer = MADDNESS_MAX_C * 16 / 256;     // most values of a row a thread fetches
constexpr int kSubBatch = 8;
constexpr int kSubPad = 5 * kSubBatch;                    // the reads run up to five batches past a row's last term
size_t substitution_lds_bytes(int Q, int nc) { return sizeof(double) * ((size_t)(Q + kSubPad) * nc + 2 * (size_t)(Q + kSubPad + 1)); }

template <int NC>
__global__ __launch_bounds__(256) void substitution_kernel(const ProtoArgs a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int Q = a.Q, D = a.D, tid = threadIdx.x;
    const int Qp = Q + kSubPad;
    double *X = reinterpret_cast<double *>(lds_raw);      // [Qp][NC]
    double *rows = X + (size_t)Qp * NC;                   // [2][Qp + 1]: a row of the factor, its diagonal entry last
    const int col0 = blockIdx.x * NC;
    const int ncols = min(NC, D - col0);
    for (int idx = tid; idx < Qp * NC; idx += 256) {
        const int i = idx / NC, cc = idx % NC;
        X[idx] = (i < Q && cc < ncols) ? a.R[(size_t)i * D + col0 + cc] : 0.0;
    }
    for (int idx = tid; idx < 2 * (Qp + 1); idx += 256) rows[idx] = 0.0;
    __syncthreads();
    // step s < Q: row i = s of L, entries 0..i; step s >= Q: row i = 2Q - 1 - s of L^T, entries i..Q-1
    const int n_steps = 2 * Q;
    const int per = (Q + 255) / 256;
    double ahead[kSubMaxPer];
    auto fetch = [&](int s) {
        if (s >= n_steps) return;
        const bool fwd = s < Q;
        const int i = fwd ? s : 2 * Q - 1 - s;
        const double *src = (fwd ? a.Lr : a.M) + (size_t)i * Q;
        const int lo = fwd ? 0 : i, hi = fwd ? i + 1 : Q;
#pragma unroll
        for (int u = 0; u < kSubMaxPer; ++u) {
            const int k = lo + tid + 256 * u;
            if (u < per && k < hi) ahead[u] = src[k];
        }
    };
    auto stash = [&](int s) {
        if (s >= n_steps) return;
        const bool fwd = s < Q;
        const int i = fwd ? s : 2 * Q - 1 - s;
        const int lo = fwd ? 0 : i, hi = fwd ? i + 1 : Q;
        double *dst = rows + (size_t)(s & 1) * (Qp + 1);
#pragma unroll
        for (int u = 0; u < kSubMaxPer; ++u) {
            const int k = lo + tid + 256 * u;
            if (u < per && k < hi) {
                dst[k] = k == i ? 0.0 : ahead[u];
                if (k == i) dst[Qp] = ahead[u];
            }
        }
    };
    fetch(0);
    stash(0);
    __syncthreads();
    for (int s = 0; s < n_steps; ++s) {
        fetch(s + 1);
        if (tid < NC) {
            const bool fwd = s < Q;
            const int i = fwd ? s : 2 * Q - 1 - s;
            const double *Li = rows + (size_t)(s & 1) * (Qp + 1);
            const int lo = fwd ? 0 : i + 1, hi = fwd ? i : Q;
            double v = X[(size_t)i * NC + tid];
            const double *pl = Li + lo, *px = X + (size_t)lo * NC + tid;
            double l0[kSubBatch], x0[kSubBatch], l1[kSubBatch], x1[kSubBatch], l2[kSubBatch], x2[kSubBatch];
            auto read = [&](int at, double *l, double *x) {
#pragma unroll
                for (int u = 0; u < kSubBatch; ++u) {
                    l[u] = pl[at + u];
                    x[u] = px[(at + u) * NC];
                }
            };
            auto subtract = [&](const double *l, const double *x) {
#pragma unroll
                for (int u = 0; u < kSubBatch; ++u) v -= l[u] * x[u];
            };
            read(0, l0, x0);
            read(kSubBatch, l1, x1);
            for (int k = lo; k < hi; k += 3 * kSubBatch) {
                // (the fences keep the compiler from gathering the reads of several batches in one place)
                read(2 * kSubBatch, l2, x2);
                __builtin_amdgcn_sched_barrier(0);
                subtract(l0, x0);
                __builtin_amdgcn_sched_barrier(0);
                read(3 * kSubBatch, l0, x0);
                __builtin_amdgcn_sched_barrier(0);
                subtract(l1, x1);
                __builtin_amdgcn_sched_barrier(0);
                read(4 * kSubBatch, l1, x1);
                __builtin_amdgcn_sched_barrier(0);
                subtract(l2, x2);
                __builtin_amdgcn_sched_barrier(0);
                pl += 3 * kSubBatch;
                px += 3 * kSubBatch * NC;
            }
            X[(size_t)i * NC + tid] = v / Li[Qp];
        }
        stash(s + 1);
        __syncthreads();
    }
    for (int idx = tid; idx < Q * NC; idx += 256) {
        const int i = idx / NC, cc = idx % NC;
        if (cc < ncols) a.P[(size_t)i * D + col0 + cc] = (float)X[idx];
    }
}

template <int NC>
int launch_substitution(const ProtoArgs &a, hipStream_t stream)
{
    if (int rc = allow_full_lds<substitution_kernel<NC>>(); rc != MADDNESS_OK) return rc;
    hipLaunchKernelGGL(substitution_kernel<NC>, dim3((a.D + NC - 1) / NC), dim3(256), substitution_lds_bytes(a.Q, NC), stream, a);
    return MADDNESS_OK;
}

// The substitutions with the products taken out of the chain.  While the first wavefront carries its columns
// through the sum of row i, the other three form the products L_i'k x_k of the NEXT row i' for every k whose x_k
// is known by then (all but the one the chain is just working out) and leave them in LDS; the chain of row i'
// then only reads a product and subtracts it, and forms the one missing product itself - the last term going
// forward, the first going back, so that the terms keep their order.  Same products, same subtractions, a chain
// of half the instructions.  LDS holds the columns, two sets of products and three rows of the factor, so a
// workgroup takes fewer columns than substitution_kernel does; factors too large for that stay with it.
constexpr int kSubHelpers = 192;
constexpr int kSubMaxPerHelper = (MADDNESS_MAX_C * 16 + kSubHelpers - 1) / kSubHelpers;
size_t substitution_products_lds_bytes(int Q, int nc)
{
    return sizeof(double) * (3 * (size_t)(Q + kSubPad) * nc + 3 * (size_t)(Q + kSubPad + 1));
}

template <int NC>
__global__ __launch_bounds__(256) void substitution_products_kernel(const ProtoArgs a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int Q = a.Q, D = a.D, tid = threadIdx.x;
    const int Qp = Q + kSubPad;
    double *X = reinterpret_cast<double *>(lds_raw);      // [Qp][NC]
    double *P = X + (size_t)Qp * NC;                      // [2][Qp][NC] products of the row of step s in P[s & 1]
    double *rows = P + 2 * (size_t)Qp * NC;               // [3][Qp + 1] the row of step s in rows[s % 3], its diagonal entry last
    const int col0 = blockIdx.x * NC;
    const int ncols = min(NC, D - col0);
    for (int idx = tid; idx < Qp * NC; idx += 256) {
        const int i = idx / NC, cc = idx % NC;
        X[idx] = (i < Q && cc < ncols) ? a.R[(size_t)i * D + col0 + cc] : 0.0;
    }
    for (int idx = tid; idx < 2 * Qp * NC + 3 * (Qp + 1); idx += 256) P[idx] = 0.0;     // (products and rows)
    __syncthreads();
    // step s < Q: row i = s of L, entries 0..i; step s >= Q: row i = 2Q - 1 - s of L^T, entries i..Q-1
    const int n_steps = 2 * Q;
    const int ht = tid - 64;                              // helper number (the threads of the other three wavefronts)
    const int per = (Q + kSubHelpers - 1) / kSubHelpers;
    double ahead[kSubMaxPerHelper];
    auto fetch = [&](int s) __attribute__((always_inline)) {
        if (s >= n_steps || ht < 0) return;
        const bool fwd = s < Q;
        const int i = fwd ? s : 2 * Q - 1 - s;
        const double *src = (fwd ? a.Lr : a.M) + (size_t)i * Q;
        const int lo = fwd ? 0 : i, hi = fwd ? i + 1 : Q;
#pragma unroll
        for (int u = 0; u < kSubMaxPerHelper; ++u) {
            const int k = lo + ht + kSubHelpers * u;
            if (u < per && k < hi) ahead[u] = src[k];
        }
    };
    auto stash = [&](int s) __attribute__((always_inline)) {
        if (s >= n_steps || ht < 0) return;
        const bool fwd = s < Q;
        const int i = fwd ? s : 2 * Q - 1 - s;
        const int lo = fwd ? 0 : i, hi = fwd ? i + 1 : Q;
        double *dst = rows + (size_t)(s % 3) * (Qp + 1);
#pragma unroll
        for (int u = 0; u < kSubMaxPerHelper; ++u) {
            const int k = lo + ht + kSubHelpers * u;
            if (u < per && k < hi) {
                dst[k] = ahead[u];
                if (k == i) dst[Qp] = ahead[u];
            }
        }
    };
    // the products of the row of step s, for every k but the one next to the diagonal; zeros after the last
    // (going forward; going back the places after Q - 1 are never written and stay zero)
    auto products = [&](int s) __attribute__((always_inline)) {
        if (s >= n_steps || ht < 0) return;
        const bool fwd = s < Q;
        const int i = fwd ? s : 2 * Q - 1 - s;
        const double *Li = rows + (size_t)(s % 3) * (Qp + 1);
        double *dst = P + (size_t)(s & 1) * Qp * NC;
        const int k_first = fwd ? 0 : i + 2, k_end = fwd ? max(i - 1, 0) : Q;      // [k_first, k_end)
        int idx = k_first * NC + ht;
        const int idx_end = k_end * NC;
        for (; idx + 3 * kSubHelpers < idx_end; idx += 4 * kSubHelpers) {
            double l[4], x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                l[u] = Li[(idx + u * kSubHelpers) / NC];
                x[u] = X[idx + u * kSubHelpers];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) dst[idx + u * kSubHelpers] = l[u] * x[u];
        }
        for (; idx < idx_end; idx += kSubHelpers) dst[idx] = Li[idx / NC] * X[idx];
        if (fwd)
            for (int z = k_end * NC + ht; z < (k_end + 2 * kSubBatch) * NC; z += kSubHelpers) dst[z] = 0.0;
    };
    fetch(0);
    stash(0);
    fetch(1);
    stash(1);
    __syncthreads();
    for (int s = 0; s < n_steps; ++s) {
        fetch(s + 2);
        if (tid < NC) {
            const bool fwd = s < Q;
            const int i = fwd ? s : 2 * Q - 1 - s;
            const double *Li = rows + (size_t)(s % 3) * (Qp + 1);
            const int lo = fwd ? 0 : i + 2, hi = fwd ? i - 1 : Q;       // the terms whose products are in P
            double v = X[(size_t)i * NC + tid];
            if (!fwd && i + 1 < Q) v -= Li[i + 1] * X[(size_t)(i + 1) * NC + tid];
            const double *pp = P + (size_t)(s & 1) * Qp * NC + (size_t)lo * NC + tid;
            double p0[kSubBatch], p1[kSubBatch], p2[kSubBatch];
            auto read = [&](int at, double *t) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < kSubBatch; ++u) t[u] = pp[(at + u) * NC];
            };
            auto subtract = [&](const double *t) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < kSubBatch; ++u) v -= t[u];
            };
            read(0, p0);
            read(kSubBatch, p1);
            for (int k = lo; k < hi; k += 3 * kSubBatch) {
                // (the fences keep the compiler from gathering the reads of several batches in one place; a batch
                // past the last term subtracts zeros, or is read and not used)
                read(2 * kSubBatch, p2);
                __builtin_amdgcn_sched_barrier(0);
                subtract(p0);
                __builtin_amdgcn_sched_barrier(0);
                read(3 * kSubBatch, p0);
                __builtin_amdgcn_sched_barrier(0);
                if (k + kSubBatch < hi) subtract(p1);
                __builtin_amdgcn_sched_barrier(0);
                read(4 * kSubBatch, p1);
                __builtin_amdgcn_sched_barrier(0);
                if (k + 2 * kSubBatch < hi) subtract(p2);
                __builtin_amdgcn_sched_barrier(0);
                pp += 3 * kSubBatch * NC;
            }
            if (fwd && i >= 1) v -= Li[i - 1] * X[(size_t)(i - 1) * NC + tid];
            X[(size_t)i * NC + tid] = v / Li[Qp];
        } else {
            products(s + 1);
        }
        stash(s + 2);
        __syncthreads();
    }
    for (int idx = tid; idx < Q * NC; idx += 256) {
        const int i = idx / NC, cc = idx % NC;
        if (cc < ncols) a.P[(size_t)i * D + col0 + cc] = (float)X[idx];
    }
}

template <int NC>
int launch_substitution_products(const ProtoArgs &a, hipStream_t stream)
{
    if (int rc = allow_full_lds<substitution_products_kernel<NC>>(); rc != MADDNESS_OK) return rc;
    hipLaunchKernelGGL(substitution_products_kernel<NC>, dim3((a.D + NC - 1) / NC), dim3(256),
                       substitution_products_lds_bytes(a.Q, NC), stream, a);
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

int64_t pow2_at_least(int64_t n)
{
    int64_t p = 1;
    while (p < n) p <<= 1;
    return p;
}

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
    a.bounds = w.take<int32_t>(2 * C);
    a.pitch = a.dmax <= 8 ? 8 : (a.dmax + 15) / 16 * 16;
    a.X = w.take<float>(C * (a.N + 1) * a.pitch);
    a.chunk_count = w.take<int32_t>(4 * C * kMaxChunks * kSplitBuckets);
    a.node = w.take<uint8_t>(C * a.N);      // (right behind chunk_count: both are cleared together)
    a.col_loss = w.take<double>(C * kSplitBuckets * a.dmax);
    a.bucket_loss = w.take<double>(C * kSplitBuckets);
    a.bucket_count = w.take<int64_t>(C * kSplitBuckets);
    a.bucket_start = w.take<int32_t>(C * kSplitBuckets);
    a.rows_by_bucket = w.take<int32_t>(C * a.N);
    a.cand = w.take<int32_t>(C * kCand);
    a.n_cand = w.take<int32_t>(C);
    a.keys = w.take<uint64_t>(C * kCand * a.Npad);
    a.tile_slots = a.N / kJudgeRows + kSplitBuckets + 1;
    a.sums = w.take<double>(C * kCand * 2 * a.tile_slots * 2 * a.dmax);
    a.group_slots = a.N / kGroupRows + kSplitBuckets + 1;
    a.group_loss = w.take<double>(C * kCand * a.group_slots);
    a.group_at = w.take<int32_t>(C * kCand * a.group_slots * 2);
    a.chosen = w.take<int32_t>(C);
}

void carve_prototypes(Carver &w, ProtoArgs &a)
{
    const size_t Q = a.Q;
    a.bounds = w.take<int32_t>(2 * (size_t)a.C);
    a.counts = w.take<int32_t>(Q * Q);
    a.M = w.take<double>(Q * Q);
    a.Lr = w.take<double>(Q * Q);
    a.R = w.take<double>(Q * a.D);
    a.list = w.take<uint32_t>((size_t)a.C * (kListRows + kListSpare));
    a.list_count = w.take<int32_t>((size_t)a.C * kListChunks * 16);
    a.list_start = w.take<int32_t>((size_t)a.C * 17);
}

}  // namespace

size_t learn_trees_workspace_bytes(int64_t N, int32_t C, int32_t dmax)
{
    LearnArgs a{};
    a.N = N; a.Npad = pow2_at_least(N); a.C = C; a.dmax = dmax;
    Carver w{nullptr};
    carve_trees(w, a);
    return w.used;
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

int launch_learn_trees(const float *A, int64_t N, int64_t lda, int32_t C, const int32_t *bounds_host, int32_t dmax,
                       int32_t *split_dims, float *thresholds, uint8_t *codes, void *workspace, hipStream_t stream)
{
    LearnArgs a{};
    a.A = A; a.lda = lda; a.N = N; a.Npad = pow2_at_least(N); a.C = C; a.dmax = dmax;
    a.split_dims = split_dims; a.thresholds = thresholds; a.codes = codes;
    Carver w{static_cast<unsigned char *>(workspace)};
    carve_trees(w, a);
    note_kernel("gather_columns_kernel + order_rows_kernel + bucket_loss_kernel + select_kernel + key_kernel + sort_chunks_kernel + sort_exchange_kernel + split_chains_kernel + judge_kernel + choose_kernel + apply_kernel", nullptr);

    Bounds b{};
    for (int i = 0; i < 2 * C; ++i) b.v[i] = bounds_host[i];
    hipLaunchKernelGGL(upload_bounds_kernel, dim3(1), dim3(256), 0, stream, b, 2 * C, a.bounds);
    LAUNCH_OK("launch upload_bounds_kernel");
    const int64_t clear_words = (a.node + (size_t)C * N - reinterpret_cast<uint8_t *>(a.chunk_count) + 3) / 4;
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)((clear_words + 255) / 256)), dim3(256), 0, stream, a.chunk_count, clear_words);
    LAUNCH_OK("launch clear_kernel");

    const int64_t pieces = (N + 1) * (a.pitch / 4);
    hipLaunchKernelGGL(gather_columns_kernel, dim3((unsigned)((pieces + 255) / 256), C), dim3(256), 0, stream, a);
    LAUNCH_OK("launch gather_columns_kernel");

    const size_t sort_lds = sizeof(uint64_t) * (size_t)(a.Npad < kSortChunk ? a.Npad : kSortChunk);
    if (int rc = allow_full_lds<sort_chunks_kernel>(); rc != MADDNESS_OK) return rc;
    const bool narrow = dmax <= 8;
    for (int level = 0; level < 4; ++level) {
        const int n_buckets = 1 << level;
        hipLaunchKernelGGL(order_rows_kernel, dim3((unsigned)((N + order_chunk_rows(N) - 1) / order_chunk_rows(N)), C), dim3(256), 0,
                           stream, a, level, n_buckets);
        LAUNCH_OK("launch order_rows_kernel");
        // (columns eight or sixteen at a time: a wavefront carries them all)
        const int groups = narrow ? 1 : a.pitch / 16;
        const dim3 loss_groups(C, n_buckets, groups);
        if (narrow)
            hipLaunchKernelGGL(bucket_loss_kernel<8>, loss_groups, dim3(16 * 8 + kChainHelpers), stream_lds_bytes<8>(), stream, a);
        else
            hipLaunchKernelGGL(bucket_loss_kernel<16>, loss_groups, dim3(16 * 16 + kChainHelpers), stream_lds_bytes<16>(), stream, a);
        LAUNCH_OK("launch bucket_loss_kernel");
        hipLaunchKernelGGL(select_kernel, dim3(C), dim3(64), sizeof(double) * dmax, stream, a, n_buckets);
        LAUNCH_OK("launch select_kernel");
        hipLaunchKernelGGL(key_kernel, dim3((unsigned)((a.Npad + 255) / 256), kCand, C), dim3(256), 0, stream, a);
        LAUNCH_OK("launch key_kernel");
        const int64_t chunk_len = a.Npad < kSortChunk ? a.Npad : kSortChunk;
        const dim3 chunks((unsigned)(a.Npad / chunk_len), kCand, C), pairs((unsigned)((a.Npad / 2 + 255) / 256), kCand, C);
        hipLaunchKernelGGL(sort_chunks_kernel, chunks, dim3(1024), sort_lds, stream, a, (int64_t)2, chunk_len, (int64_t)0);
        LAUNCH_OK("launch sort_chunks_kernel");
        for (int64_t k = 2 * chunk_len; k <= a.Npad; k <<= 1) {
            for (int64_t j = k >> 1; j >= chunk_len; j >>= 1) {
                hipLaunchKernelGGL(sort_exchange_kernel, pairs, dim3(256), 0, stream, a, k, j);
                LAUNCH_OK("launch sort_exchange_kernel");
            }
            hipLaunchKernelGGL(sort_chunks_kernel, chunks, dim3(1024), sort_lds, stream, a, k, k, chunk_len >> 1);
            LAUNCH_OK("launch sort_chunks_kernel");
        }
        const dim3 chain_groups(C, 8 * groups, n_buckets);
        const dim3 judges((unsigned)(a.group_slots * C), kCand);
        if (narrow) {
            hipLaunchKernelGGL(split_chains_kernel<8>, chain_groups, dim3(32 * 8 + kChainHelpers), stream_lds_bytes<8>(), stream, a);
            LAUNCH_OK("launch split_chains_kernel");
            hipLaunchKernelGGL(judge_kernel<8>, judges, dim3(64), 0, stream, a, n_buckets);
        } else {
            hipLaunchKernelGGL(split_chains_kernel<16>, chain_groups, dim3(32 * 16 + kChainHelpers), stream_lds_bytes<16>(), stream, a);
            LAUNCH_OK("launch split_chains_kernel");
            hipLaunchKernelGGL(judge_kernel<16>, judges, dim3(64), 0, stream, a, n_buckets);
        }
        LAUNCH_OK("launch judge_kernel");
        hipLaunchKernelGGL(choose_kernel, dim3(C), dim3(512), 0, stream, a, level, n_buckets);
        LAUNCH_OK("launch choose_kernel");
        hipLaunchKernelGGL(apply_kernel, dim3((unsigned)((N + 255) / 256), C), dim3(256), 0, stream, a, level, n_buckets);
        LAUNCH_OK("launch apply_kernel");
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
    note_kernel("cooccurrence_kernel + count_codes_kernel + list_codes_kernel + gta_kernel + cholesky_panel_kernel + substitution_kernel", nullptr);
    const int64_t QQ = (int64_t)a.Q * a.Q;
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)((QQ + 255) / 256)), dim3(256), 0, stream, a.counts, QQ);
    LAUNCH_OK("launch clear_kernel");
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
        hipLaunchKernelGGL(gta_kernel, dim3((D + 63) / 64, 4, C), dim3(256), 0, stream, a, first);
        LAUNCH_OK("launch gta_kernel");
    }
    for (int J0 = 0; J0 < a.Q; J0 += kCholPanel) {
        const int below = a.Q - J0 - kCholPanel, per_group = kCholRows - kCholPanel;
        hipLaunchKernelGGL(cholesky_panel_kernel, dim3(std::max(1, (below + per_group - 1) / per_group)), dim3(256), 0,
                           stream, a, J0);
        LAUNCH_OK("launch cholesky_panel_kernel");
    }
    hipLaunchKernelGGL(transpose_factor_kernel, dim3((unsigned)((QQ + 255) / 256)), dim3(256), 0, stream, a);
    LAUNCH_OK("launch transpose_factor_kernel");
    // the kernel that takes the products out of the chain where its LDS layout fits (as many columns of A~ per
    // workgroup as fit, a power of two up to 16); else substitution_kernel (as many columns as LDS holds beside two
    // rows of the factor: a power of two, a wavefront's worth at most)
    const size_t lds_limit = (size_t)device_info().lds_per_block;
    int rc = MADDNESS_OK;
    int npc = 16;
    while (npc > 1 && substitution_products_lds_bytes(a.Q, npc) > lds_limit) npc >>= 1;
    if (substitution_products_lds_bytes(a.Q, npc) <= lds_limit) {
        switch (npc) {
        case 16: rc = launch_substitution_products<16>(a, stream); break;
        case 8: rc = launch_substitution_products<8>(a, stream); break;
        case 4: rc = launch_substitution_products<4>(a, stream); break;
        case 2: rc = launch_substitution_products<2>(a, stream); break;
        default: rc = launch_substitution_products<1>(a, stream); break;
        }
    } else {
        int nc = 64;
        while (nc > 1 && substitution_lds_bytes(a.Q, nc) > lds_limit) nc >>= 1;
        if (substitution_lds_bytes(a.Q, nc) > lds_limit)
            return fail(MADDNESS_E_UNSUPPORTED, "maddness_learn_prototypes: a column of 16 C values does not fit in LDS");
        switch (nc) {
        case 64: rc = launch_substitution<64>(a, stream); break;
        case 32: rc = launch_substitution<32>(a, stream); break;
        case 16: rc = launch_substitution<16>(a, stream); break;
        case 8: rc = launch_substitution<8>(a, stream); break;
        case 4: rc = launch_substitution<4>(a, stream); break;
        case 2: rc = launch_substitution<2>(a, stream); break;
        default: rc = launch_substitution<1>(a, stream); break;
        }
    }
    if (rc != MADDNESS_OK) return rc;
    LAUNCH_OK("launch substitution_kernel");
    return MADDNESS_OK;
}

}  // namespace maddness
