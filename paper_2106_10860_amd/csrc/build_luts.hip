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
// (16 RT rows of T) and 32 columns; the w-th wavefront contracts d = 16 (w + 8 n) + 0..15 for all 2 RT tiles of 16 x 16, and the
// partial tiles are added in that order through LDS.
// Operand layout of v_mfma_f64_16x16x4_f64: lane l supplies A[i = l % 16][k = l / 16]
// and B[k = l / 16][j = l % 16]; it receives D[i = 4 r + l / 16][j = l % 16] in
// accumulator element r = 0..3.  Which d stand for k = 0..3 is free: here d = 16 (w + 8 n) + 4 k + t in instruction t, so
// that a lane's operands of four instructions lie side by side in a row of P.  Every operand has one reader, so it comes
// straight from memory, the next step's while the matrix cores have this one's, with no barrier before the last step.
// VEC: rows of P are whole 16-byte pieces on 16-byte boundaries.
// 2 * 16 C D M flops; 1024 x 512 with 64 codebooks: 15 us at the 73 TFLOP/s that a large product reaches, 20 here
// (table build 27; 29 and 38 with tiles of both staged in LDS for all wavefronts, whose barriers left the matrix cores idle between
// the steps; staged with 16-byte reads 34).  Two steps ahead: 31, the registers of a second set cost more than they give.
constexpr int KSPLIT = 8;
constexpr int GEMM_COLS = 32, GEMM_DEPTH = 16 * KSPLIT, GEMM_THREADS = 64 * KSPLIT;

template <int RT, bool VEC>
__global__ __launch_bounds__(GEMM_THREADS) void lut_gemm_kernel(const float *__restrict__ P,
                                                               const float *__restrict__ B, int C, int D, int M,
                                                               int64_t ldb, double *__restrict__ T,
                                                               double *__restrict__ delta, double *__restrict__ range)
{
    constexpr int TILES = 2 * RT;
    __shared__ double part[KSPLIT][TILES][4][64];
    const int c0 = blockIdx.x * RT, m0 = blockIdx.y * GEMM_COLS;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, kk = lane >> 4;

    struct Operands {
        float a[RT][4], b[2][4];
    };
    // (rows, columns and depths that do not exist read others; those depths become zeros where they are used)
    const float *a_row[RT], *b_col[2];
#pragma unroll
    for (int r = 0; r < RT; ++r) a_row[r] = P + (size_t)min(16 * (c0 + r) + i, 16 * C - 1) * D;
#pragma unroll
    for (int h = 0; h < 2; ++h) b_col[h] = B + min(m0 + 16 * h + i, M - 1);
    auto fetch = [&](Operands &o, int d0) __attribute__((always_inline)) {
        const int d = d0 + 4 * kk;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if constexpr (VEC) {
                const float4 v = *reinterpret_cast<const float4 *>(a_row[r] + min(d, D - 4));
                o.a[r][0] = v.x;
                o.a[r][1] = v.y;
                o.a[r][2] = v.z;
                o.a[r][3] = v.w;
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) o.a[r][t] = a_row[r][min(d + t, D - 1)];
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t row = (int64_t)min(d + t, D - 1) * ldb;
#pragma unroll
            for (int h = 0; h < 2; ++h) o.b[h][t] = b_col[h][row];
        }
    };
    double4_t acc[RT][2];
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r][0] = acc[r][1] = double4_t{0.0, 0.0, 0.0, 0.0};
    auto contract = [&](Operands &o, int d0) __attribute__((always_inline)) {
        if (d0 + 16 > D) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bool here = d0 + 4 * kk + t < D;
#pragma unroll
                for (int r = 0; r < RT; ++r) o.a[r][t] = here ? o.a[r][t] : 0.0f;
#pragma unroll
                for (int h = 0; h < 2; ++h) o.b[h][t] = here ? o.b[h][t] : 0.0f;
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const double b0 = (double)o.b[0][t], b1 = (double)o.b[1][t];
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const double av = (double)o.a[r][t];
                acc[r][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, b0, acc[r][0], 0, 0, 0);
                acc[r][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, b1, acc[r][1], 0, 0, 0);
            }
        }
    };
    Operands o;
    int d0 = 16 * wave;
    if (d0 < D) fetch(o, d0);
    // (the last step by itself: with the fetch under a condition the compiler waits for all of it at once, 33 us; fetched
    // past the end, the last values are waited for at the barrier)
    for (; d0 + GEMM_DEPTH < D; d0 += GEMM_DEPTH) {
        contract(o, d0);
        fetch(o, d0 + GEMM_DEPTH);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (d0 < D) contract(o, d0);
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[wave][2 * r + h][e][lane] = acc[r][h][e];
    __syncthreads();
    for (int tile = wave; tile < TILES; tile += KSPLIT) {
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
    // (the entries first: they are on their way while the scale is worked out; 30 -> 27 us for the table build above)
    constexpr int PER = 4 * QUANT_CODEBOOKS;          // entry 4 u + ty of the workgroup's
    double entry[PER], least[QUANT_CODEBOOKS];
#pragma unroll
    for (int u = 0; u < PER; ++u) entry[u] = T[(size_t)min(16 * c0 + 4 * u + ty, 16 * C - 1) * M + min(m, M - 1)];
#pragma unroll
    for (int k = 0; k < QUANT_CODEBOOKS; ++k) least[k] = delta[(size_t)min(c0 + k, C - 1) * M + min(m, M - 1)];
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
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (c0 + u / 4 >= C) break;
        double q = rint(ldexp(entry[u] - least[u / 4], l));
        q = (q >= 0.0) ? q : 0.0;  // NaN -> 0
        q = q > 255.0 ? 255.0 : q;
        luts[(size_t)(16 * c0 + 4 * u + ty) * M + m] = (uint8_t)q;
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
    const bool vec = p.D % 4 == 0 && reinterpret_cast<uintptr_t>(p.prototypes) % 16 == 0;
    auto launch = [&](auto rt) {
        constexpr int RT = decltype(rt)::value;
        const dim3 grid(groups(RT), col_tiles);
        if (vec) hipLaunchKernelGGL((lut_gemm_kernel<RT, true>), grid, dim3(GEMM_THREADS), 0, stream, p.prototypes, B, C, p.D, M, ldb, T, delta, range);
        else hipLaunchKernelGGL((lut_gemm_kernel<RT, false>), grid, dim3(GEMM_THREADS), 0, stream, p.prototypes, B, C, p.D, M, ldb, T, delta, range);
    };
    if (groups(4) * col_tiles >= cus) launch(std::integral_constant<int, 4>{});
    else if (groups(2) * col_tiles >= cus) launch(std::integral_constant<int, 2>{});
    else launch(std::integral_constant<int, 1>{});
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
