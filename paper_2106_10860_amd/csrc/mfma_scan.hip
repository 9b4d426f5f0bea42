// The exact table scan on the matrix cores, codes read from memory: a wavefront
// keeps the tables of its output columns in registers for the whole kernel and
// streams over the rows.  See mfma_common.h for the formulation.
#include "mfma_common.h"

#include <algorithm>

namespace maddness {
namespace {

using namespace mfma;

struct MfmaScanArgs {
    const uint8_t *codes;   // [N][C / 2]
    const uint8_t *luts;    // [C][16][M]
    const float *scale;
    const float *offset;
    ScanOut o;
    int64_t N;
    int codebooks;          // the any-shape form: the real number of codebooks (<= the kernel's C); rows of codes
                            // are (codebooks + 1) / 2 bytes
};

// The packed codes of one row as they come from memory (zeros for a row that does not exist), and as the scan takes them:
// rows of any number of bytes are read in (unaligned) words, the last one up to the row's end and moved down afterwards.
// (Put together from bytes where they are loaded, the row has to be waited for there, behind the stores before it:
// M = 250, C = 30, N = 300000 113 us that way, 84 so.)
template <int CW, bool ODD>
__device__ __forceinline__ auto load_row_codes(const MfmaScanArgs &a, int64_t row)
{
    typedef unsigned cvec __attribute__((ext_vector_type(CW)));
    cvec v = {};
    if (row >= a.N) return v;
    if constexpr (ODD) {
        const int bytes = (a.codebooks + 1) / 2;
        const uint8_t *src = a.codes + row * bytes;
        if (bytes < 4) {
            for (int t = 0; t < bytes; ++t) v[0] |= (unsigned)src[t] << (8 * t);
            return v;
        }
        const int past = bytes % 4 ? 4 - bytes % 4 : 0;
#pragma unroll
        for (int q = 0; q < CW; ++q)
            if (4 * q < bytes) {
                uint32_t w;
                __builtin_memcpy(&w, src + 4 * q - (4 * q + 4 > bytes ? past : 0), 4);
                v[q] = w;
            }
    } else {
        // (rows are C / 2 bytes apart and only the base is known to be 16-byte aligned: copied as
        // words, so that no wider alignment than a word's is assumed of a row)
        __builtin_memcpy(&v, reinterpret_cast<const uint32_t *>(a.codes + row * (4 * CW)), sizeof(uint32_t) * CW);
    }
    return v;
}

template <int CW, bool ODD, typename Codes>
__device__ __forceinline__ Codes whole_codes(const MfmaScanArgs &a, Codes v)
{
    if constexpr (ODD) {
        const int bytes = (a.codebooks + 1) / 2;
        if (bytes > 4 && bytes % 4 != 0)
#pragma unroll
            for (int q = 1; q < CW; ++q)
                if (4 * q < bytes && 4 * q + 4 > bytes) v[q] >>= 8 * (4 * q + 4 - bytes);
    }
    return v;
}

// The dequantised results of one step of a workgroup (16 rows, or 32 with NT = 2, times its
// 4 blocks of columns) collected in LDS and written out row by row: a store instruction then
// covers 1 KiB (512 bytes) of one row instead of 256 (128) bytes of four rows.  For outputs
// whose rows do not start on 128-byte lines, where the direct stores end inside lines and run
// at a third to a half of their rate.  All 4 wavefronts take part in every step (barriers).
// ODD: any number of codebooks up to C (the others padded with zero codes and entries), any M,
// any pitch and alignment of codes, tables and outputs: codes and tables are read from any byte on,
// rows are written as ranges of floats in aligned 16-byte pieces (store_dense_rows): the 16 or 32
// consecutive rows of a step as one range when there is no padding between them, else row by row.
template <int KG, int NT, bool ODD = false>
__device__ __forceinline__ void scan_gathered(const MfmaScanArgs &a, const v4i *one_hot, float *tile, int lane, int wave)
{
    constexpr int C = 4 * KG;
    constexpr int CW = C / 8;
    constexpr int SPAN = 16 * NT;
    constexpr int GPS = NT == 2 ? 2 : 1;            // groups of 16 rows per step
    constexpr int TILE_LD = 4 * SPAN + 4;           // floats per tile row (4 of padding)
    typedef float piece __attribute__((ext_vector_type(NT)));
    const int j = lane & 15, g = lane >> 4;
    const int col0 = blockIdx.y * 4 * SPAN;          // first column of the workgroup
    const int col = col0 + wave * SPAN + NT * j;     // first of this lane's NT columns
    const bool col_on = col < a.o.M;
    const bool active = col0 + wave * SPAN < a.o.M;  // the wavefront has columns
    const int n_cols = a.o.M - col0 < 4 * SPAN ? a.o.M - col0 : 4 * SPAN;

    v4i B[NT][KG];
    float sc[NT], of[NT];
    load_tables<KG, NT, 256, ODD>(B, a.luts, a.o.M, col0, 4 * SPAN, wave * SPAN, g, j, reinterpret_cast<unsigned char *>(tile),
                                  threadIdx.x, a.codebooks);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const bool on = ODD ? col + t < a.o.M : col_on;
        sc[t] = on ? a.scale[col + t] : 0.f;
        of[t] = on ? a.offset[col + t] : 0.f;
    }
    const ScanOut acc_only{nullptr, 0, a.o.acc, a.o.M};
    const int64_t n_groups = (a.N + 15) >> 4;
    // rows without padding between them, all columns in this workgroup: the rows of a step are one range of floats
    const bool dense = ODD && a.o.out && a.o.ldo == a.o.M && gridDim.y == 1;
    const float inv_M = 1.0f / (float)a.o.M;
    auto load_codes = [&](int64_t rg) INLINE_LAMBDA { return whole_codes<CW, ODD>(a, load_row_codes<CW, ODD>(a, rg * 16 + j)); };
    // step s of this workgroup: groups GPS (blockIdx.x + s gridDim.x) + 0 .. GPS - 1, i.e. 16 GPS
    // consecutive rows
    for (int64_t rg = (int64_t)GPS * blockIdx.x; rg < n_groups; rg += (int64_t)GPS * gridDim.x) {
        if (active) {
            v4i acc[GPS][NT];
            if constexpr (GPS == 2) scan16x2<KG, NT>(load_codes(rg), load_codes(rg + 1), B, g, one_hot, acc[0], acc[1]);
            else scan16<KG, NT>(load_codes(rg), B, g, one_hot, acc[0]);
            if (col_on) {
#pragma unroll
                for (int q = 0; q < GPS; ++q) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        piece v;
#pragma unroll
                        for (int t = 0; t < NT; ++t) v[t] = fmaf((float)acc[q][t][r], sc[t], of[t]);
                        *reinterpret_cast<piece *>(tile + (q * 16 + 4 * g + r) * TILE_LD + wave * SPAN + NT * j) = v;
                    }
                    if (a.o.acc) {
                        const int64_t r0 = (rg + q) * 16;
                        if constexpr (ODD) {
#pragma unroll
                            for (int r = 0; r < 4; ++r)
#pragma unroll
                                for (int t = 0; t < NT; ++t)
                                    if (r0 + 4 * g + r < a.N && col + t < a.o.M)
                                        a.o.acc[(r0 + 4 * g + r) * a.o.M + col + t] = (uint16_t)acc[q][t][r];
                        } else {
                            store16<NT>(acc_only, acc[q], [r0](int k) { return r0 + k; }, a.N, g, col, sc, of);
                        }
                    }
                }
            }
        }
        __syncthreads();
        // row r of the step goes out through wavefront r % 4, NT columns per lane and instruction
        if (ODD && dense) {
            // the 16 GPS consecutive rows of the step are one range of floats
            const int64_t first = rg * 16, left = a.N - first;
            store_dense_rows(a.o.out + first * a.o.M, left < 16 * GPS ? (int)left : 16 * GPS, a.o.M, inv_M, tile, TILE_LD, 0,
                             (int)threadIdx.x, 256);
        } else
        for (int r = wave; r < 16 * GPS; r += 4) {
            const int64_t row = rg * 16 + r;
            if (row >= a.N) break;
            float *dst = a.o.out + row * a.o.ldo + col0;
            if constexpr (ODD) {
                // a row (its columns of this workgroup) as a range of its own
                if (!a.o.out) continue;
                store_dense_rows<true>(dst, 1, n_cols, 0.f, tile, TILE_LD, r, lane, 64);
            } else {
                for (int c = lane; c < n_cols / NT; c += 64)
                    __builtin_nontemporal_store(*reinterpret_cast<const piece *>(tile + r * TILE_LD + NT * c),
                                                reinterpret_cast<piece *>(dst + NT * c));
            }
        }
        __syncthreads();   // the tile is rewritten in the next step
    }
}

// KG: groups of four codebooks (C = 4 KG); NT: column tiles per wavefront (4 or 2);
// GATHER: results through LDS, whole rows written (above).
template <int KG, int NT, bool GATHER = false, bool ODD = false>
__global__ __launch_bounds__(256, 2) void mfma_scan_kernel(const MfmaScanArgs a)
{
    static_assert(!ODD || GATHER, "the any-shape form writes whole rows through LDS");
    static_assert(NT == 4 || NT == 2, "tiles per wavefront");
    static_assert(KG % 2 == 0, "whole words of packed codes");
    constexpr int C = 4 * KG;
    constexpr int CW = C / 8;          // 32-bit words of packed codes per row
    constexpr int SPAN = 16 * NT;      // output columns per wavefront
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 15, g = lane >> 4;
    __shared__ v4i one_hot[16];
    fill_one_hot_table(one_hot, threadIdx.x);
    __syncthreads();
    if constexpr (GATHER) {
        __shared__ __align__(16) float tile[(NT == 2 ? 32 : 16) * (4 * SPAN + 4)];
        static_assert(sizeof(tile) >= 4 * kTableStage, "the tables pass through it");
        scan_gathered<KG, NT, ODD>(a, one_hot, tile, lane, wave);
        return;
    }
    // blocks of SPAN columns for the 4 wavefronts; with fewer than 4 blocks in all,
    // `share` wavefronts hold the same block and take every share-th group of rows
    const int col_blocks = (a.o.M + SPAN - 1) / SPAN;
    const int share = col_blocks >= 3 ? 1 : (col_blocks == 2 ? 2 : 4);
    const int blocks_here = 4 / share;
    const int c0 = (blockIdx.y * blocks_here + wave % blocks_here) * SPAN;   // first column of this wavefront
    const int col = c0 + NT * j;                    // first of this lane's NT columns
    const bool col_on = col < a.o.M;                // M is a multiple of NT

    v4i B[NT][KG];
    {
        __shared__ __align__(16) unsigned char stage[4 * kTableStage];
        load_tables<KG, NT, 256, false>(B, a.luts, a.o.M, blockIdx.y * blocks_here * SPAN, blocks_here * SPAN,
                                        wave % blocks_here * SPAN, g, j, stage, threadIdx.x, a.codebooks);
    }
    if (c0 >= a.o.M) return;                        // no barriers below
    float sc[NT], of[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        sc[t] = col_on ? a.scale[col + t] : 0.f;
        of[t] = col_on ? a.offset[col + t] : 0.f;
    }

    // rows, 16 at a time; the codes of the next group are fetched ahead
    typedef unsigned cvec __attribute__((ext_vector_type(CW)));
    const int64_t n_groups = (a.N + 15) >> 4;
    auto load_codes = [&](int64_t rg) INLINE_LAMBDA { return load_row_codes<CW, false>(a, rg * 16 + j); };
    int64_t rg = (int64_t)blockIdx.x * share + wave / blocks_here;
    const int64_t stride = (int64_t)gridDim.x * share;
    if constexpr (NT == 2) {
        // two groups per step: four independent accumulation chains for the matrix pipe
        cvec next0 = {}, next1 = {};
        if (rg < n_groups) next0 = load_codes(rg);
        if (rg + stride < n_groups) next1 = load_codes(rg + stride);
        for (; rg + stride < n_groups; rg += 2 * stride) {
            const cvec cw0 = next0, cw1 = next1;
            if (rg + 2 * stride < n_groups) next0 = load_codes(rg + 2 * stride);
            if (rg + 3 * stride < n_groups) next1 = load_codes(rg + 3 * stride);
            v4i acc0[NT], acc1[NT];
            scan16x2<KG, NT>(cw0, cw1, B, g, one_hot, acc0, acc1);
            if (col_on) {
                const int64_t r1 = rg + stride;
                store16<NT>(a.o, acc0, [rg](int k) { return rg * 16 + k; }, a.N, g, col, sc, of);
                store16<NT>(a.o, acc1, [r1](int k) { return r1 * 16 + k; }, a.N, g, col, sc, of);
            }
        }
        if (rg < n_groups) {   // an odd group left over; its codes are in next0
            v4i acc[NT];
            scan16<KG, NT>(next0, B, g, one_hot, acc);
            if (col_on) store16<NT>(a.o, acc, [rg](int k) { return rg * 16 + k; }, a.N, g, col, sc, of);
        }
    } else {
        cvec next = {};
        if (rg < n_groups) next = load_codes(rg);
        for (; rg < n_groups; rg += stride) {
            const cvec cw = next;
            if (rg + stride < n_groups) next = load_codes(rg + stride);
            v4i acc[NT];
            scan16<KG, NT>(cw, B, g, one_hot, acc);
            if (col_on) store16<NT>(a.o, acc, [rg](int k) { return rg * 16 + k; }, a.N, g, col, sc, of);
        }
    }
}

// Rows without padding between them that do not begin on 128-byte lines, whole lines written: a line that two wavefronts
// write a part of each, at different times, costs as much as several whole ones.  Rows whose first floats lie at the same
// place of a line (row mod `classes`) go to the same workgroups, whose blocks of columns begin where the first line
// that begins in such a row does.  The row's last line is filled up with the first columns of the row after it: workgroups
// of their own take it (32 columns to a wavefront, all four the same ones), whose tables go on with column 0 and who scan
// the next rows' codes as well.  Only lines are stored, each by one wavefront, straight from registers.  (Stores alone of
// 512 MB, by rows of 1000, 500, 300 and 250 floats: 5.2, 5.2, 5.1 and 5.5 TB/s; rows from their first float to their last
// 4.4, 3.8, 3.5 and 2.7.  The kernel against the one that gathers rows in LDS: M = 1000, C = 32, N = 131072 148 -> 107 us,
// 4.9 TB/s; M = 999, C = 64 443 -> 305; M = 513, C = 16, N = 262144 237 -> 112; M = 100, C = 32, N = 2^20 181 -> 103.)
constexpr int kLine = 32;

// one group of 16 rows after the other: cls + classes i for 16 values of i
template <int KG, int NT, bool ODD, bool LAST>
__device__ __forceinline__ void scan_lines(const MfmaScanArgs &a, int classes, int cls, int col0, int first, int end, int blocks_here,
                                           int64_t rg, int64_t stride, const v4i *one_hot, unsigned char *stage)
{
    constexpr int C = 4 * KG, CW = C / 8, SPAN = 16 * NT;
    typedef float piece __attribute__((ext_vector_type(NT)));
    const int lane = threadIdx.x & 63, j = lane & 15, g = lane >> 4, M = a.o.M;
    const int col = col0 + first + NT * j;
    v4i B[NT][KG];
    load_tables<KG, NT, 256, ODD, LAST>(B, a.luts, M, col0, blocks_here * SPAN, first, g, j, stage, threadIdx.x, a.codebooks);
    if (col0 + first >= end) return;                // no barriers below
    float sc[NT], of[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int real = min(LAST && col + t >= M ? col + t - M : col + t, M - 1);
        sc[t] = a.scale[real];
        of[t] = a.offset[real];
    }
    const int64_t n_rows = (a.N - cls + classes - 1) / classes, n_groups = (n_rows + 15) >> 4, pitch = (int64_t)classes * M;
    auto load_codes = [&](int64_t group, int after) INLINE_LAMBDA {
        return load_row_codes<CW, ODD>(a, group < n_groups ? cls + (group * 16 + j) * classes + after : a.N);
    };
    auto store = [&](const v4i (&acc)[NT], int64_t group) INLINE_LAMBDA {
        if (col >= end) return;
        const int64_t row0 = cls + (group * 16 + 4 * g) * classes;
        float *dst = a.o.out + row0 * M + col;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            piece v;
#pragma unroll
            for (int t = 0; t < NT; ++t) v[t] = fmaf((float)acc[t][r], sc[t], of[t]);
            const int64_t row = row0 + (int64_t)r * classes;
            if (row + (LAST ? 1 : 0) < a.N) __builtin_nontemporal_store(v, reinterpret_cast<piece *>(dst));
            else if (LAST && row < a.N)                           // (the last row ends inside its last line)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (col + t < M) dst[t] = v[t];
            dst += pitch;
        }
    };
    auto next0 = load_codes(rg, 0);
    if constexpr (LAST) {
        auto next1 = load_codes(rg, 1);
        for (; rg < n_groups; rg += stride) {
            const auto cw0 = whole_codes<CW, ODD>(a, next0), cw1 = whole_codes<CW, ODD>(a, next1);
            next0 = load_codes(rg + stride, 0);
            next1 = load_codes(rg + stride, 1);
            v4i acc[NT], of_next[NT];
            scan16x2<KG, NT>(cw0, cw1, B, g, one_hot, acc, of_next);
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[t][r] = col + t < M ? acc[t][r] : of_next[t][r];
            store(acc, rg);
        }
    } else if constexpr (NT == 2) {
        // two groups per step: four independent accumulation chains for the matrix pipe
        auto next1 = load_codes(rg + stride, 0);
        for (; rg < n_groups; rg += 2 * stride) {
            const auto cw0 = whole_codes<CW, ODD>(a, next0), cw1 = whole_codes<CW, ODD>(a, next1);
            next0 = load_codes(rg + 2 * stride, 0);
            next1 = load_codes(rg + 3 * stride, 0);
            v4i acc0[NT], acc1[NT];
            scan16x2<KG, NT>(cw0, cw1, B, g, one_hot, acc0, acc1);
            store(acc0, rg);
            if (rg + stride < n_groups) store(acc1, rg + stride);
        }
    } else {
        for (; rg < n_groups; rg += stride) {
            const auto cw = whole_codes<CW, ODD>(a, next0);
            next0 = load_codes(rg + stride, 0);
            v4i acc[NT];
            scan16<KG, NT>(cw, B, g, one_hot, acc);
            store(acc, rg);
        }
    }
}

// A class has gridDim.x / classes workgroups (a multiple of 8): `last` of them share out its rows for their last lines, the others
// are `shares` of the rows times `quarters` of the columns before (blocks for four wavefronts).  The workgroups of all
// classes that take the same share lie 8 apart, on one XCD: 128 bytes of codes are rows of up to 8 classes and
// more.
template <int KG, int NT, bool ODD>
__global__ __launch_bounds__(256, 2) void mfma_scan_lines_kernel(const MfmaScanArgs a, int classes, int last, int shares, int share, int quarters)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), M = a.o.M;
    __shared__ v4i one_hot[16];
    __shared__ __align__(16) unsigned char stage[4 * kTableStage];
    fill_one_hot_table(one_hot, threadIdx.x);
    __syncthreads();
    const int cls = (int)blockIdx.x / 8 % classes, unit = (int)blockIdx.x / (8 * classes) * 8 + (int)blockIdx.x % 8;
    const int first_float = (int)(((int64_t)cls * M) % kLine);
    // columns lo .. end - 1 of these rows are whole lines, those from M on of the next row
    const int lo = (kLine - first_float) % kLine, end = M + (kLine - (first_float + M) % kLine) % kLine;
    if (unit < last) {
        scan_lines<KG, 2, ODD, true>(a, classes, cls, end - kLine, 0, end, 1, (int64_t)unit * 4 + wave, (int64_t)last * 4, one_hot, stage);
        return;
    }
    const int blocks_here = 4 / share, y = (unit - last) / shares;
    if (y >= quarters) return;
    scan_lines<KG, NT, ODD, false>(a, classes, cls, lo + y * blocks_here * 16 * NT, wave % blocks_here * 16 * NT, end - kLine, blocks_here,
                                   (int64_t)((unit - last) % shares) * share + wave / blocks_here, (int64_t)shares * share, one_hot, stage);
}

// Whether rows of M columns that begin in `classes` places of a line are written by whole lines; `results`: all rows' columns.
// With less than 48 MB of them caches put the parts of a line together for the other forms (C = 32, M = 1000, N = 16384: 23 us
// there, 19 here, C = 64, M = 250: 16, 31).  What either form measured, this one second (us; Mi: 2^20 results):
//   - 64 columns or less (96 for NT = 2) are mostly last lines, whose results are scanned twice (N = 200000, C = 64, M = 66: 37, 46)
//   - rows that one workgroup's four blocks take whole are written by it in one go (C = 32, N = 300000: M = 248 58, 67; M = 250
//     76, 86; but padded codebooks in up to 8 classes: M = 252, C = 30 83, 62)
//   - every other row begins on a line (two classes): the other form writes at up to 6.0 TB/s, this one at 5 (130 Mi, C = 16:
//     M = 400 92, 114; M = 1040 93, 103), but for up to 144 columns (C = 24, M = 144, 80 Mi 81, 66), a few more than a workgroup takes
//     (C = 16, M = 272, 80 Mi 81, 68) and a few less than a multiple from 1008 on (C = 24, 200 Mi 174, 161), and where results are
//     few and codebooks many (C = 32, M = 528, 13 Mi 19, 16)
//   - few codebooks and 145 to 192 columns (C = 8, M = 164, 200 Mi 144, 172; C = 16, M = 188, 40 Mi 34, 37)
//   - padded codebooks, 16 and 32 classes, 97 to 192 columns (C = 30: M = 170, 13 Mi 27, 35; M = 171, 64 Mi 95, 94; C = 32: M = 183,
//     30 Mi 46, 54; C = 31: M = 125, 16 Mi 33, 39, 64 Mi 102, 92; C = 24: M = 186, 13 Mi 24, 28, 50 Mi 62, 64)
//   - NT = 2 and 16 classes, all the more where the blocks do not fill the workgroups (C = 64: M = 310, 13 Mi 28, 42; M = 322, 50 Mi
//     80, 76; M = 258, 20 Mi 42, 45; M = 162, 64 Mi 116, 134; C = 40: M = 330, 13 Mi 23, 29; M = 258, 50 Mi 77, 51; C = 56, M = 602,
//     30 Mi 59, 41)
inline bool lines_pay(int NT, bool odd, int padded, int C, int M, int classes, bool full, int64_t results)
{
    const int64_t mi = results >> 20;
    if (mi < 12 || M < (NT == 4 ? 64 : 96)) return false;
    if ((M + 16 * NT - 1) / (16 * NT) == 4 && !(odd && classes <= 8)) return false;
    if (NT == 2) {
        if (odd || classes < 16) return true;
        if (M > 160 && M <= 192 && C > 40) return false;
        return mi >= (full || M >= 576 ? 14 + (C - 40) * 7 / 12 : C - 14);
    }
    if (!odd && classes == 2 && !(C > 16 && mi < 24))
        return M < 160 || (M > 256 && M < (C > 16 || (C > 8 && mi < 64) ? 320 : 288)) || (M > 960 && M % 256 >= 240);
    if (!odd && C <= 16 && M > (C > 8 ? 152 : 144) && M <= 192) return mi < 24;
    if (odd && padded == 32 && classes >= 16 && M > 96 && M <= 192) {
        if (M <= 160) return mi >= (C > 30 ? 32 : C > 24 ? 24 : C > 20 ? 16 : 12);
        return mi >= (C > 30 ? 128 : C > 20 ? 64 : 32);
    }
    return true;
}

template <int KG, int NT, bool ODD = false>
int launch_mfma(const MfmaScanArgs &a, hipStream_t stream)
{
    const DeviceInfo &dev = device_info();
    const int span = 16 * NT * 4;                       // columns per workgroup of 4 wavefronts
    const int gy = (a.o.M + span - 1) / span;
    const int col_blocks = (a.o.M + 16 * NT - 1) / (16 * NT);
    int classes = 1;
    while (classes * (int64_t)a.o.M % 32 != 0) classes *= 2;
    // (a row has up to (M + 31) / 32 first floats of a line, its last line's among them)
    const int blocks = (((a.o.M + 31) / 32 - 1) * 32 + 16 * NT - 1) / (16 * NT);
    const int share = blocks >= 3 ? 1 : blocks == 2 ? 2 : 4, quarters = (blocks * share + 3) / 4;
    if (classes > 1 && a.o.out && !a.o.acc && a.o.ldo == a.o.M && aligned_to(a.o.out, 128) && a.N >= 16384 &&
        lines_pay(NT, ODD, 4 * KG, a.codebooks, a.o.M, classes, blocks == 4 / share * quarters, a.N * a.o.M)) {
        // one to four turns of the chip (two workgroups per compute unit; very wide rows: more), whichever leaves the least undone: the last lines take
        // as long as 64 (32) columns
        const double group_us = (KG * NT * 34 + 1000) / 2400.0, table_us = 4.0;
        const int64_t groups = (a.N / classes + 15) / 16;
        int units = 0, shares = 1, last = 1;
        double least = 1e30;
        for (int turns = 1; turns <= 4 || units == 0; ++turns) {       // (units stays 0 until a class has more workgroups than blocks of columns)
            const int u = std::max(8, 2 * dev.cus * turns / classes / 8 * 8);
            const double of_last = NT == 4 ? 0.3 * share : 0.55 * share;
            for (int n = std::max(1, (int)(u / (quarters + of_last))), k = 0; k < 2; ++n, ++k) {
                const int l = u - n * quarters;
                if (l < 1) break;
                const double us = turns * (std::max((double)((groups + (int64_t)n * share - 1) / ((int64_t)n * share)),
                                                    (double)groups * (NT == 4 ? 0.3 : 0.55) / l) * group_us + table_us);
                if (us < least) {
                    least = us;
                    units = u;
                    shares = n;
                    last = l;
                }
            }
        }
        note_kernel("mfma_scan_kernel, whole lines", __PRETTY_FUNCTION__);
        hipLaunchKernelGGL((mfma_scan_lines_kernel<KG, NT, ODD>), dim3((unsigned)(classes * units)), dim3(256), 0, stream, a,
                           classes, last, shares, share, quarters);
        return check_hip(hipGetLastError(), "launch mfma_scan_lines_kernel");
    }
    if constexpr (ODD) {
        const int64_t n_steps = ((a.N + 15) / 16 + (NT == 2 ? 1 : 0)) / (NT == 2 ? 2 : 1);
        int64_t gx = (int64_t)dev.cus * 2 / gy;
        if (gx < 1) gx = 1;
        if (gx > n_steps) gx = n_steps;
        note_kernel("mfma_scan_kernel, any shape", __PRETTY_FUNCTION__);
        hipLaunchKernelGGL((mfma_scan_kernel<KG, NT, true, true>), dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, stream, a);
        return check_hip(hipGetLastError(), "launch mfma_scan_kernel");
    }
    // fp32 output rows that do not start on 128-byte lines, at least 3 blocks of columns (no
    // sharing of blocks among wavefronts): whole rows through LDS
    if (a.o.out && col_blocks >= 3 && (a.o.ldo % 32 != 0 || !aligned_to(a.o.out, 128))) {
        const int64_t n_steps = ((a.N + 15) / 16 + (NT == 2 ? 1 : 0)) / (NT == 2 ? 2 : 1);
        int64_t gx = (int64_t)dev.cus * 2 / gy;
        if (gx < 1) gx = 1;
        if (gx > n_steps) gx = n_steps;
        note_kernel("mfma_scan_kernel, gathered stores", __PRETTY_FUNCTION__);
        hipLaunchKernelGGL((mfma_scan_kernel<KG, NT, true>), dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, stream, a);
        return check_hip(hipGetLastError(), "launch mfma_scan_kernel");
    }
    const int of_block = col_blocks >= 3 ? 1 : (col_blocks == 2 ? 2 : 4);   // wavefronts with the same block, as in the kernel
    const int64_t n_groups = (a.N + 15) / 16;
    int64_t gx = (int64_t)dev.cus * 2 / gy;             // two workgroups per CU in all
    if (gx < 1) gx = 1;
    if (gx * of_block > n_groups) gx = (n_groups + of_block - 1) / of_block;
    note_kernel("mfma_scan_kernel", __PRETTY_FUNCTION__);
    hipLaunchKernelGGL((mfma_scan_kernel<KG, NT>), dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, stream, a);
    return check_hip(hipGetLastError(), "launch mfma_scan_kernel");
}

}  // namespace

// Returns MADDNESS_OK after a launch, 1 if the shape is not covered.
int launch_scan_mfma(int32_t C, int32_t M, const uint8_t *codes, int64_t N, const uint8_t *luts,
                     const float *scale, const float *offset, float *out, int64_t ldo, uint16_t *acc,
                     hipStream_t stream)
{
    // (the tables are read once per workgroup: from which number of rows on that pays depends on what else holds them)
    if (C > 64 || N < matrix_cores_min_rows(C, M, C == 16 || C == 32)) return 1;
    const int NT = C <= 32 ? 4 : 2;
    MfmaScanArgs a{codes, luts, scale, offset, ScanOut{out, ldo, acc, M}, N, C};
    if (C % 8 != 0 || !aligned_to(codes, 16) || M % NT != 0 || !aligned_to(luts, NT) ||
        (out && (ldo % NT != 0 || !aligned_to(out, 4 * NT))) || (acc && !aligned_to(acc, 2 * NT))) {
        // any other shape: padded to 16, 32 or 64 codebooks, everything read and written in the smallest units;
        // worth it from a few blocks of columns on (M = 10 is faster in the general kernel, which does no padded work)
        if (M <= 16) return 1;
        if (C <= 16) return launch_mfma<4, 4, true>(a, stream);
        if (C <= 32) return launch_mfma<8, 4, true>(a, stream);
        return launch_mfma<16, 2, true>(a, stream);
    }
    switch (C) {
    case 8: return launch_mfma<2, 4>(a, stream);
    case 16: return launch_mfma<4, 4>(a, stream);
    case 24: return launch_mfma<6, 4>(a, stream);
    case 32: return launch_mfma<8, 4>(a, stream);
    case 40: return launch_mfma<10, 2>(a, stream);
    case 48: return launch_mfma<12, 2>(a, stream);
    case 56: return launch_mfma<14, 2>(a, stream);
    default: return launch_mfma<16, 2>(a, stream);
    }
}

}  // namespace maddness
