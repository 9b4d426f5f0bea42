// h(B): table construction (Section 3, "Table Construction", with the dense
// prototype matrix of Section 4.3) and 8-bit quantisation (Appendix A).
//
// The contraction T = P B (16 C x D times D x M) is the one dense piece of the
// method and runs on the fp64 matrix cores (v_mfma_f64_16x16x4_f64): products of
// two fp32 numbers are exact in fp64, so the tables differ from an fp64
// reference only by summation order (~1e-16 relative) and the 8-bit entries are
// reproducible to the byte except for values within that distance of a rounding
// boundary.  The contraction is tiny (2 * 16 C D M flops, 0.13 GFLOP at C = 32,
// D = 512, M = 256), so two small launches are enough: one contracts and takes each table's minimum and range from
// its registers, one quantises.
#include "common.h"

namespace maddness {
namespace {

// Workspace of maddness_build_luts_static, the entry point for callers that cannot
// allocate: one array per GPU, held until the process ends.  In host code the name
// `scratch` is only a handle for hipGetSymbolAddress, never a device address.  Which shapes the entry point takes is
// counted without `range` (build_luts_static_bytes); the array has room for it beside the largest of them
// (8 C M bytes, under a seventeenth of what is counted).
static __device__ __align__(256) unsigned char scratch[MADDNESS_STATIC_WORKSPACE_BYTES + MADDNESS_STATIC_WORKSPACE_BYTES / 16];

typedef double double4_t __attribute__((ext_vector_type(4)));

// T and, per codebook and column, the least entry and the range.  A workgroup of eight wavefronts takes RT codebooks
// (16 RT rows of T) and 32 columns.  64 steps of the inner dimension at a time go to LDS, the next 64 on their way
// meanwhile; four wavefronts take each half of the columns, the w-th of them contracts d = 4 (w + 4 i) + 0..3 for its
// RT tiles of 16 x 16, and the partial tiles are added in that order through LDS.
// Operand layout of v_mfma_f64_16x16x4_f64: lane l supplies A[i = l % 16][k = l / 16]
// and B[k = l / 16][j = l % 16]; it receives D[i = 4 r + l / 16][j = l % 16] in
// accumulator element r = 0..3.
// 2 * 16 C D M flops; 1024 x 512 with 64 codebooks: 15 us at the 73 TFLOP/s that a large product reaches; takes 29 us
// there: two wavefronts to a SIMD, each waiting for its operands from LDS, leave the matrix cores busy 38 % of the time (LDS
// 16 %, by the counters; 30 % of that conflicts, of writes).  One codebook and 16 columns to a workgroup, operands straight from memory, took
// 77 us: two loads of 16 rows or 4 rows each per matrix instruction, where staged tiles need 5 reads of LDS for 4 of them.
constexpr int KSPLIT = 4;
constexpr int GEMM_COLS = 32, GEMM_DEPTH = 64, GEMM_THREADS = 128 * KSPLIT;
constexpr int A_PITCH = GEMM_DEPTH + 4, B_PITCH = GEMM_COLS + 16;      // (the reads of an operand's 64 values meet in no LDS bank)

template <int RT>
__global__ __launch_bounds__(GEMM_THREADS) void lut_gemm_kernel(const float *__restrict__ P,
                                                               const float *__restrict__ B, int C, int D, int M,
                                                               int64_t ldb, double *__restrict__ T,
                                                               double *__restrict__ delta, double *__restrict__ range)
{
    constexpr int ROWS = 16 * RT, TILES = 2 * RT;
    constexpr int STAGE = ROWS * A_PITCH + GEMM_DEPTH * B_PITCH;           // floats of one of the two stages
    constexpr size_t PART = sizeof(double) * KSPLIT * TILES * 4 * 64;
    constexpr size_t LDS = sizeof(float) * 2 * STAGE > PART ? sizeof(float) * 2 * STAGE : PART;
    __shared__ __align__(16) unsigned char lds[LDS];
    float *stage = reinterpret_cast<float *>(lds);
    double(*part)[TILES][4][64] = reinterpret_cast<double(*)[TILES][4][64]>(lds);   // once the stages are done with
    const int c0 = blockIdx.x * RT, m0 = blockIdx.y * GEMM_COLS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, w = wave % KSPLIT, half = wave / KSPLIT;
    const int i = lane & 15, kk = lane >> 4;

    constexpr int PER_A = ROWS * GEMM_DEPTH / GEMM_THREADS, PER_B = GEMM_DEPTH * GEMM_COLS / GEMM_THREADS;
    constexpr int A_STEP = GEMM_THREADS / GEMM_DEPTH, B_STEP = GEMM_THREADS / GEMM_COLS;
    // where this thread's first pieces lie; rows and columns that do not exist read the last one and become zeros
    // on their way to LDS (decided at the load, the compiler makes every load a branch of its own, each waited for)
    const int m_own = m0 + tid % GEMM_COLS;
    const float *b_src = B + min(m_own, M - 1);
    float a_next[PER_A], b_next[PER_B];
    auto fetch = [&](int d0) __attribute__((always_inline)) {
        const int d_a = d0 + lane;
        const float *a_src = P + min(d_a, D - 1);
#pragma unroll
        for (int u = 0; u < PER_A; ++u) {
            const int row = 16 * c0 + wave + A_STEP * u;
            a_next[u] = a_src[(size_t)min(row, 16 * C - 1) * D];
        }
#pragma unroll
        for (int u = 0; u < PER_B; ++u) {
            const int d = d0 + tid / GEMM_COLS + B_STEP * u;
            b_next[u] = b_src[(size_t)min(d, D - 1) * ldb];
        }
    };
    double4_t acc[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r] = double4_t{0.0, 0.0, 0.0, 0.0};
    fetch(0);
    int parity = 0;
    for (int d0 = 0; d0 < D; d0 += GEMM_DEPTH, parity ^= 1) {
        float *As = stage + parity * STAGE, *Bs = As + ROWS * A_PITCH;
#pragma unroll
        for (int u = 0; u < PER_A; ++u)
            As[(wave + A_STEP * u) * A_PITCH + lane] = 16 * c0 + wave + A_STEP * u < 16 * C && d0 + lane < D ? a_next[u] : 0.0f;
#pragma unroll
        for (int u = 0; u < PER_B; ++u)
            Bs[(tid / GEMM_COLS + B_STEP * u) * B_PITCH + tid % GEMM_COLS] =
                d0 + tid / GEMM_COLS + B_STEP * u < D && m_own < M ? b_next[u] : 0.0f;
        __syncthreads();
        if (d0 + GEMM_DEPTH < D) fetch(d0 + GEMM_DEPTH);
#pragma unroll
        for (int s = 0; s < GEMM_DEPTH / 16; ++s) {
            const int k = 16 * s + 4 * w + kk;
            const double bv = (double)Bs[k * B_PITCH + 16 * half + i];
#pragma unroll
            for (int r = 0; r < RT; ++r)
                acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)As[(16 * r + i) * A_PITCH + k], bv, acc[r], 0, 0, 0);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[w][2 * r + half][e][lane] = acc[r][e];
    __syncthreads();
    for (int tile = wave; tile < TILES; tile += 2 * KSPLIT) {
        const int c = c0 + tile / 2, m = m0 + 16 * (tile % 2) + i;
        // (an entry that is not a number counts neither way, unless it is the table's first: then minimum and range are
        // none either, as a walk over the sixteen that begins with the first has it)
        double lo = __builtin_inf(), hi = -__builtin_inf(), first = 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double s = part[0][tile][e][lane];
#pragma unroll
            for (int q = 1; q < KSPLIT; ++q) s += part[q][tile][e][lane];
            if (c < C && m < M) T[((size_t)c * 16 + 4 * e + kk) * M + m] = s;
            if (e == 0) first = s;
            lo = s < lo ? s : lo;
            hi = s > hi ? s : hi;
        }
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) {
            const double lo2 = __shfl_xor(lo, off), hi2 = __shfl_xor(hi, off);
            lo = lo2 < lo ? lo2 : lo;
            hi = hi2 > hi ? hi2 : hi;
        }
        if (kk == 0 && c < C && m < M) {
            lo = first == first ? lo : first;
            delta[(size_t)c * M + m] = lo;
            range[(size_t)c * M + m] = hi - lo;
        }
    }
}

// the exponent l of the power-of-two scale for the widest range r
__device__ __forceinline__ int scale_exponent(double r)
{
    if (!(r > 0.0) || !isfinite(r)) return 0;
    // r = f 2^e with f in [0.5, 1); r 2^l <= 255 = (255/256) 2^8
    int e;
    const double f = frexp(r, &e);
    const int l = (f <= 255.0 / 256.0) ? 8 - e : 7 - e;
    return l > 126 ? 126 : (l < -126 ? -126 : l);
}

// A workgroup takes 64 columns and QUANT_CODEBOOKS codebooks: the widest range of every column over all codebooks gives
// the scale's exponent (every workgroup works it out for itself: C values a column), then the entries are quantised.
// The first workgroup of the columns writes scale and offset, the minima added in codebook order (the order the
// definition of beta is written in).
constexpr int QUANT_COLS = 64, QUANT_CODEBOOKS = 2;
constexpr int QUANT_BATCH = 8;       // loads on their way at a time (one by one, 64 codebooks' minima took 15 us)
__global__ __launch_bounds__(256) void lut_quantize_kernel(const double *__restrict__ T, const double *__restrict__ delta,
                                                           const double *__restrict__ range, int C, int M,
                                                           uint8_t *__restrict__ luts, float *__restrict__ scale,
                                                           float *__restrict__ offset)
{
    __shared__ double widest[4][QUANT_COLS];
    const int tx = threadIdx.x % QUANT_COLS, ty = threadIdx.x / QUANT_COLS;
    const int m = blockIdx.x * QUANT_COLS + tx, c0 = blockIdx.y * QUANT_CODEBOOKS;
    double r = 0.0;
    if (m < M)
        for (int c = ty; c < C; c += 4 * QUANT_BATCH) {
            double e[QUANT_BATCH];
#pragma unroll
            for (int u = 0; u < QUANT_BATCH; ++u) e[u] = range[(size_t)min(c + 4 * u, C - 1) * M + m];
#pragma unroll
            for (int u = 0; u < QUANT_BATCH; ++u) r = e[u] > r ? e[u] : r;
        }
    widest[ty][tx] = r;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) r = widest[q][tx] > r ? widest[q][tx] : r;
    if (m >= M) return;
    const int l = scale_exponent(r);
    if (blockIdx.y == 0 && ty == 0) {
        double beta = 0.0;
        for (int c = 0; c < C; c += 2 * QUANT_BATCH) {
            double v[2 * QUANT_BATCH];
#pragma unroll
            for (int u = 0; u < 2 * QUANT_BATCH; ++u) v[u] = delta[(size_t)min(c + u, C - 1) * M + m];
#pragma unroll
            for (int u = 0; u < 2 * QUANT_BATCH; ++u) beta = c + u < C ? beta + v[u] : beta;
        }
        scale[m] = ldexpf(1.0f, -l);
        offset[m] = (float)beta;
    }
    for (int row = ty; row < 16 * QUANT_CODEBOOKS; row += 4) {
        const int c = c0 + row / 16;
        if (c >= C) break;
        const size_t at = ((size_t)c * 16 + row % 16) * M + m;
        double q = rint(ldexp(T[at] - delta[(size_t)c * M + m], l));
        q = (q >= 0.0) ? q : 0.0;  // NaN -> 0
        q = q > 255.0 ? 255.0 : q;
        luts[at] = (uint8_t)q;
    }
}

// Pooled variant (Appendix A as printed), step 1: one block per codebook finds
// the minimum and maximum of the codebook's tables over all columns and entries.
__global__ __launch_bounds__(256) void lut_pooled_minmax_kernel(const double *__restrict__ T, int M,
                                                                double *__restrict__ cb_min,
                                                                double *__restrict__ cb_range)
{
    __shared__ double lo_s[256], hi_s[256];
    const int c = blockIdx.x;
    const double *t = T + (size_t)c * 16 * M;
    const int n = 16 * M;
    double lo = t[0], hi = t[0];
    for (int i = threadIdx.x; i < n; i += 256) {
        const double v = t[i];
        lo = v < lo ? v : lo;
        hi = v > hi ? v : hi;
    }
    lo_s[threadIdx.x] = lo;
    hi_s[threadIdx.x] = hi;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            lo_s[threadIdx.x] = lo_s[threadIdx.x + s] < lo_s[threadIdx.x] ? lo_s[threadIdx.x + s] : lo_s[threadIdx.x];
            hi_s[threadIdx.x] = hi_s[threadIdx.x + s] > hi_s[threadIdx.x] ? hi_s[threadIdx.x + s] : hi_s[threadIdx.x];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        cb_min[c] = lo_s[0];
        cb_range[c] = hi_s[0] - lo_s[0];
    }
}

// Step 2 (one block): the widest range gives the scale, the minima are added in
// codebook order.
__global__ __launch_bounds__(256) void lut_pooled_finish_kernel(const double *__restrict__ cb_min,
                                                                const double *__restrict__ cb_range, int C,
                                                                int M, int *__restrict__ lexp, float *__restrict__ scale,
                                                                float *__restrict__ offset)
{
    // every thread computes the same two numbers, from loads on their way a batch at a time (one by one, 194 codebooks
    // took 25 us, 22 while the compiler still ran ahead; 17 so)
    double r = 0.0, beta = 0.0;
    for (int c = 0; c < C; c += 2 * QUANT_BATCH) {
        double e[2 * QUANT_BATCH], v[2 * QUANT_BATCH];
#pragma unroll
        for (int u = 0; u < 2 * QUANT_BATCH; ++u) {
            e[u] = cb_range[min(c + u, C - 1)];
            v[u] = cb_min[min(c + u, C - 1)];
        }
#pragma unroll
        for (int u = 0; u < 2 * QUANT_BATCH; ++u) {
            r = e[u] > r ? e[u] : r;
            beta = c + u < C ? beta + v[u] : beta;
        }
    }
    const int l = scale_exponent(r);
    for (int m = threadIdx.x; m < M; m += 256) {
        scale[m] = ldexpf(1.0f, -l);
        offset[m] = (float)beta;
    }
    if (threadIdx.x == 0) *lexp = l;
}

__global__ __launch_bounds__(256) void lut_pooled_quantize_kernel(const double *__restrict__ T,
                                                                  const double *__restrict__ cb_min,
                                                                  const int *__restrict__ lexp, int M,
                                                                  uint8_t *__restrict__ luts)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    const int row = blockIdx.y;  // c * 16 + k
    if (m >= M) return;
    double q = rint(ldexp(T[(size_t)row * M + m] - cb_min[row >> 4], *lexp));
    q = (q >= 0.0) ? q : 0.0;  // NaN -> 0
    q = q > 255.0 ? 255.0 : q;
    luts[(size_t)row * M + m] = (uint8_t)q;
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace

// Workspace: T [C][16][M], delta and range [C][M], per-codebook min and range [2][C] and the exponent (pooled variant).
size_t build_luts_workspace_bytes(int32_t D, int32_t C, int32_t M)
{
    (void)D;
    return align_up(sizeof(double) * ((size_t)C * 16 * M + 2 * (size_t)C * M + 2 * (size_t)C) + sizeof(int), 256);
}

// What maddness_build_luts_static holds against MADDNESS_STATIC_WORKSPACE_BYTES.
size_t build_luts_static_bytes(int32_t C, int32_t M)
{
    return align_up(sizeof(double) * ((size_t)C * 16 * M + (size_t)C * M + 2 * (size_t)C) + sizeof(int) * (size_t)M, 256);
}

int launch_build_luts(const maddness_params &p, const float *B, int32_t M, int64_t ldb,
                      uint8_t *luts, float *scale, float *offset, void *workspace, bool pooled,
                      hipStream_t stream)
{
    const int C = p.C;
    double *T = static_cast<double *>(workspace);
    double *delta = T + (size_t)C * 16 * M;
    double *range = delta + (size_t)C * M;
    double *cb_min = range + (size_t)C * M;
    double *cb_range = cb_min + C;
    int *lexp = reinterpret_cast<int *>(cb_range + C);

    note_kernel(pooled ? "lut_gemm_kernel + lut_pooled_minmax_kernel + lut_pooled_finish_kernel + lut_pooled_quantize_kernel"
                       : "lut_gemm_kernel + lut_quantize_kernel", nullptr);
    // as many codebooks to a workgroup as still leave one per compute unit
    const int col_tiles = (M + GEMM_COLS - 1) / GEMM_COLS, cus = device_info().cus;
    auto groups = [&](int rt) { return (C + rt - 1) / rt; };
    if (groups(4) * col_tiles >= cus)
        hipLaunchKernelGGL(lut_gemm_kernel<4>, dim3(groups(4), col_tiles), dim3(GEMM_THREADS), 0, stream, p.prototypes, B, C, p.D, M,
                           ldb, T, delta, range);
    else if (groups(2) * col_tiles >= cus)
        hipLaunchKernelGGL(lut_gemm_kernel<2>, dim3(groups(2), col_tiles), dim3(GEMM_THREADS), 0, stream, p.prototypes, B, C, p.D, M,
                           ldb, T, delta, range);
    else
        hipLaunchKernelGGL(lut_gemm_kernel<1>, dim3(groups(1), col_tiles), dim3(GEMM_THREADS), 0, stream, p.prototypes, B, C, p.D, M,
                           ldb, T, delta, range);
    int rc = check_hip(hipGetLastError(), "launch lut_gemm_kernel");
    if (rc != MADDNESS_OK) return rc;
    if (!pooled) {
        hipLaunchKernelGGL(lut_quantize_kernel,
                           dim3((M + QUANT_COLS - 1) / QUANT_COLS, (C + QUANT_CODEBOOKS - 1) / QUANT_CODEBOOKS), dim3(256), 0,
                           stream, T, delta, range, C, M, luts, scale, offset);
        return check_hip(hipGetLastError(), "launch lut_quantize_kernel");
    }
    hipLaunchKernelGGL(lut_pooled_minmax_kernel, dim3(C), dim3(256), 0, stream, T, M, cb_min, cb_range);
    rc = check_hip(hipGetLastError(), "launch lut_pooled_minmax_kernel");
    if (rc != MADDNESS_OK) return rc;
    hipLaunchKernelGGL(lut_pooled_finish_kernel, dim3(1), dim3(256), 0, stream, cb_min, cb_range, C, M, lexp, scale, offset);
    rc = check_hip(hipGetLastError(), "launch lut_pooled_finish_kernel");
    if (rc != MADDNESS_OK) return rc;
    hipLaunchKernelGGL(lut_pooled_quantize_kernel, dim3((M + 255) / 256, C * 16), dim3(256), 0, stream, T, cb_min, lexp, M, luts);
    return check_hip(hipGetLastError(), "launch lut_pooled_quantize_kernel");
}

// The address of `scratch` on the current device, looked up once per device (every GPU
// holds its own copy of the array at its own address).
int static_workspace(void **workspace)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mutex;
    static void *address[kMaxDevices] = {};
    int dev = -1;
    if (int rc = check_hip(hipGetDevice(&dev), "hipGetDevice"); rc != MADDNESS_OK) return rc;
    if (dev < 0 || dev >= kMaxDevices)
        return fail(MADDNESS_E_UNSUPPORTED, "device ordinal %d: maddness_build_luts_static keeps an address for %d devices",
                    dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(mutex);
    if (!address[dev]) {
        void *ptr = nullptr;
        if (int rc = check_hip(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
            rc != MADDNESS_OK)
            return rc;
        address[dev] = ptr;
    }
    *workspace = address[dev];
    return MADDNESS_OK;
}

}  // namespace maddness
