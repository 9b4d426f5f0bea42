// Fused encode + exact scan, and either alone, by blocks of rows and columns, for few and medium numbers of rows.
//
// A call of up to a few thousand rows is bound by latencies: a chain of kernel arguments -> trees, tables and rows -> codes ->
// sums -> stores on a chip that is mostly idle.  So a workgroup (8 wavefronts) takes a block of up to 128 (256) output
// columns and few rows, as many workgroups as the chip holds, and asks for everything at once:
//   1. the tables of its columns come in 16-byte pieces as they lie in memory, a piece per thread and load, all of them on
//      their way together with the first rows and the trees;
//   2. they pass through LDS in blocks of [16 codes][16 columns], from where ds_read_b64_tr_b8 hands every lane the 16
//      entries of one codebook and column, the operand that the matrix instruction wants: no byte is turned round by
//      vector instructions, of which load_tables (mfma_common.h) spends some 90 per 64 bytes;
//   3. a chunk of rows is copied to LDS as the one range of bytes it is in memory (any pitch, any alignment), lane
//      (row, codebook) walks its tree there and leaves 16 times its code in a byte;
//   4. the wavefronts scan the chunk, one or two tiles of 16 columns each, the rows 16 at a time, with the tables as the
//      first operand: a lane ends up with four consecutive columns of one row and stores them at once.  The next chunk's
//      rows are on their way meanwhile.
// Bound by latencies and by the 64 bytes a clock that a compute unit takes in: N = 10000, D = 512, M = 100, C = 32, of 9.1 us
// (11.5 by rows_kernel) the launch takes 1.7, asking for 133 KiB and having them 3.9, the codes 0.9, the tables' way through LDS
// 1.2 and the scan 1.4 (the 100 MHz clock in the first wavefront of every workgroup; vector ALUs busy 23 %, LDS 19 %, matrix cores 4 %).  16 wavefronts to a workgroup were slower (11.6), as were two workgroups to a compute unit
// where one chunk is all the work (11.6), and lanes that read neighbouring codes instead of neighbouring columns of the tables (64
// lines to a load: N = 676, D = 352, M = 737, C = 32 12.4 us, now 6.8).
// From the first row on: a single request takes what a launch and this chain take, there and here, us: N = 2, D = 240, M = 60, C = 48 7.2 and 4.7, N = 7, D = 75, M = 577, C = 15
// 15.3 and 4.4, N = 10, D = 28, M = 4, C = 4 3.7 and 3.3; by columns N = 10, D = 704, M = 30, C = 64, bytes 26 and 9.1; the scan alone N = 7, M = 788, C = 50 9.4 and 5.2;
// averages N = 4, D = 240, M = 242, C = 16 18 and 4.5; of 306 calls of up to 15 rows none was slower.
#include <algorithm>

#include "mfma_common.h"

namespace maddness {
namespace {

using mfma::v4i;
using rows::aligned_to;
using rows::f4;
using rows::kMaxRowBytes;

typedef int v2i __attribute__((ext_vector_type(2)));

constexpr int kBlockWaves = 8, kBlockThreads = 64 * kBlockWaves;

// A block of [16 codes][16 columns] of a codebook's table in LDS, 16 bytes apart: threads that write the same code of
// neighbouring blocks meet in no bank.
constexpr int kTileBytes = 272;

struct BlockArgs {
    const uint8_t *luts;
    const unsigned char *A;   // bytes
    int64_t pitch;            // bytes between rows (A by columns: between columns)
    int64_t N;
    const int32_t *split_dims;
    const float *thresholds;
    const float *scale, *offset;
    float *out;
    int64_t ldo;
    uint16_t *acc;
    uint8_t *codes_out;
    int M, C, D, dtype, row_bytes;
    int tile_shift;           // log2 of the tiles of 16 columns to a block
    int col_blocks;
    int chunk_rows;
    int chunks;               // of the whole matrix
    int row_groups;           // workgroups that share out the chunks, a multiple of 8 where there is more than one block of columns
    unsigned rows_at, tables_at, codes_at;   // in LDS
    int overlay;              // the tables go where the first rows were
    int unit;                 // (codes) bytes to an access: 8, 4 or 1
};

// Units of packed codes that a thread takes of a chunk.
constexpr int kCodeUnits = 4;

constexpr int lanes_per_row(int C) { return C <= 4 ? 4 : C <= 8 ? 8 : C <= 16 ? 16 : C <= 32 ? 32 : 64; }

// KG: groups of four codebooks; NTW: tiles of 16 columns per wavefront; PF: 16-byte pieces of a chunk of rows per thread.
// COLS: A stored by columns.  A chunk is 64 rows, a row to a lane; a wavefront takes every eighth codebook, whose tree is the
// same for all lanes and whose four columns it reads in runs of 64 values.
// AVG (rows): the aggregation by pairwise averages in blocks of 16 codebooks (Appendix D), which is no sum and stays on the vector
// ALUs, with TS = log2 of the tiles of a block of columns.  The tables stay in LDS as they lie in memory, a lane takes four
// columns of one row, and a code is kept as the distance of its entries from the codebook's first, 16 bits, so that a
// lookup takes one addition, one read and one average of four bytes.
// ENC: the codes alone, no tables: a chunk's rows (columns' values) are on their way while the one before is encoded.
// CODES: the scan alone.  A holds packed codes, of which a thread takes up to four units of a chunk and deals them out in LDS.
template <int KG, int NTW, int PF, bool COLS = false, bool AVG = false, int TS = 0, bool CODES = false, bool ENC = false>
__global__ __launch_bounds__(kBlockThreads) void fused_blocks_kernel(const BlockArgs a)
{
    constexpr int LPR = lanes_per_row(4 * KG), RPW = 64 / LPR;    // lanes to a row, rows per wavefront while encoding
    constexpr int KGP = LPR / 4;                                   // bytes of codes per row and lane group
    constexpr int WAVES = kBlockWaves, THREADS = kBlockThreads;
    constexpr int PIECES = (KG * NTW * 8 + WAVES - 1) / WAVES;     // of the tables, per thread, at most
    constexpr int BLOCKS = THREADS / 16;                           // [16][16] blocks of the tables at a time
    constexpr int BOOKS = COLS ? (4 * KG + WAVES - 1) / WAVES : 1; // codebooks of a wavefront

    extern __shared__ __align__(16) unsigned char smem[];
    v4i *one_hot = reinterpret_cast<v4i *>(smem);
    unsigned char *tables = smem + a.tables_at, *stage = smem + a.rows_at, *codes_l = smem + a.codes_at;
    // (all arguments at once: read where they are used, they are a chain of scalar loads before the first vector load)
    asm volatile("" ::"s"(a.luts), "s"(a.A), "s"(a.pitch), "s"(a.N), "s"(a.split_dims), "s"(a.thresholds), "s"(a.scale),
                 "s"(a.offset), "s"(a.out), "s"(a.ldo), "s"(a.acc), "s"(a.codes_out), "s"(a.M), "s"(a.C), "s"(a.D), "s"(a.dtype),
                 "s"(a.row_bytes), "s"(a.tile_shift), "s"(a.col_blocks), "s"(a.chunk_rows), "s"(a.chunks), "s"(a.row_groups),
                 "s"(a.rows_at), "s"(a.tables_at), "s"(a.codes_at), "s"(a.overlay), "s"(a.unit));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;

    // Workgroups b, b + 8, ... run on the same XCD: the blocks of columns of the same rows follow each other there.
    int row_group = blockIdx.x, col_block = 0;
    if (a.col_blocks > 1) {
        const int b = blockIdx.x >> 3;
        col_block = b % a.col_blocks;
        row_group = (b / a.col_blocks) * 8 + (blockIdx.x & 7);
    }
    const int tiles = 1 << a.tile_shift;
    const int col0 = col_block * 16 * tiles;
    if (row_group >= a.chunks) return;

    // ---- everything the block needs is asked for at once, in the order in which it is used ----
    const int c = lane & (LPR - 1);
    const bool real = c < a.C;
    Tree tr;
    if constexpr (!COLS && !CODES) load_tree(tr, a.split_dims + 4 * (real ? c : 0), a.thresholds + 16 * (real ? c : 0), a.D);

    // (by columns: the raw values)
    uint32_t raw[BOOKS][4];
    auto fetch_columns = [&](int chunk) INLINE_LAMBDA {
        const int64_t row = (int64_t)chunk * 64 + lane, at = row < a.N ? row : a.N - 1;
        auto read = [&](auto element) INLINE_LAMBDA {
            typedef decltype(element) Element;
#pragma unroll
            for (int u = 0; u < BOOKS; ++u)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int book = min(wave + WAVES * u, a.C - 1), dim = min(max(a.split_dims[4 * book + t], 0), a.D - 1);
                    raw[u][t] = reinterpret_cast<const Element *>(a.A + dim * a.pitch)[at];
                }
        };
        switch (a.dtype) {
        case kF32: read(uint32_t{}); break;
        case kU8: read(uint8_t{}); break;
        default: read(uint16_t{}); break;
        }
    };
    f4 pre[PF];
    int shift = 0, next_shift = 0;      // of the first row in the staged range
    auto fetch_rows = [&](int chunk) INLINE_LAMBDA {
        const int64_t row0 = (int64_t)chunk * a.chunk_rows;
        const int64_t left = a.N - row0;
        const int n_rows = left < a.chunk_rows ? (int)left : a.chunk_rows;
        const unsigned char *src = a.A + row0 * a.pitch;
        next_shift = (int)(reinterpret_cast<uintptr_t>(src) & 15u);
        // the aligned pieces that cover the range: the first and the last may begin or end up to 15 bytes beyond it, inside
        // the 16 bytes that hold its first or last element
        const unsigned last = (unsigned)(next_shift + (n_rows - 1) * (int)a.pitch + a.row_bytes - 1) >> 4;
        const unsigned char *from = src - next_shift;
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const unsigned p = tid + THREADS * k;
            pre[k] = *reinterpret_cast<const f4 *>(from + 16 * (p < last ? p : last));
        }
    };
    auto write_rows = [&]() INLINE_LAMBDA {
        shift = next_shift;
#pragma unroll
        for (int k = 0; k < PF; ++k) reinterpret_cast<f4 *>(stage)[tid + THREADS * k] = pre[k];
    };
    // (codes: the units of a chunk lie one after another, whatever the rows' bytes)
    const int Cb = (a.C + 1) / 2;
    uint2 packed[kCodeUnits];
    auto fetch_codes = [&](int chunk) INLINE_LAMBDA {
        const int64_t row0 = (int64_t)chunk * a.chunk_rows;
        const int n_rows = a.N - row0 < a.chunk_rows ? (int)(a.N - row0) : a.chunk_rows;
        const unsigned last = (unsigned)(n_rows * Cb - a.unit);
        const unsigned char *from = a.A + row0 * Cb;
#pragma unroll
        for (int k = 0; k < kCodeUnits; ++k) {
            const unsigned at = min((unsigned)((tid + THREADS * k) * a.unit), last);
            if (a.unit == 8) __builtin_memcpy(&packed[k], from + at, 8);
            else if (a.unit == 4) __builtin_memcpy(&packed[k].x, from + at, 4);
            else packed[k].x = from[at];
        }
    };
    auto deal_codes = [&]() INLINE_LAMBDA {
        const unsigned per_row = (unsigned)Cb / (unsigned)a.unit;
#pragma unroll
        for (int k = 0; k < kCodeUnits; ++k) {
            const unsigned at = tid + THREADS * k, r = at / per_row, q = at - r * per_row;
            if ((int)r >= a.chunk_rows) break;
            unsigned char *mine = codes_l + r * LPR;
            const unsigned x = packed[k].x, y = packed[k].y;
            if (a.unit == 8) {
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    // codebooks 16 q + n, + 4, + 8, + 12, 16 times their codes
                    const unsigned lo = (n ? x >> (4 * n - 4) : x << 4) & 0x00F000F0u, hi = (n ? y >> (4 * n - 4) : y << 4) & 0x00F000F0u;
                    *reinterpret_cast<unsigned *>(mine + n * KGP + 4 * q) = __builtin_amdgcn_perm(hi, lo, 0x06040200u);
                }
            } else if (a.unit == 4) {
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    const unsigned lo = (n ? x >> (4 * n - 4) : x << 4) & 0x00F000F0u;
                    *reinterpret_cast<uint16_t *>(mine + n * KGP + 2 * q) = (uint16_t)(lo | lo >> 8);
                }
            } else {
                mine[(2 * q & 3) * KGP + q / 2] = (unsigned char)(x << 4);
                mine[(2 * q + 1 & 3) * KGP + q / 2] = (unsigned char)(x & 0xF0u);
            }
        }
    };
    int chunk = row_group;
    if constexpr (COLS) fetch_columns(chunk);
    else if constexpr (CODES) fetch_codes(chunk);
    else fetch_rows(chunk);

    // ---- encode: the codes of a chunk, times 16, into LDS ----
    auto encode = [&](int64_t row0) INLINE_LAMBDA {
#pragma unroll 1
        for (int r0 = wave * RPW; r0 < a.chunk_rows; r0 += 2 * WAVES * RPW) {
            // two groups of rows at once (the second may be beyond the chunk)
            int r[2];
            float x[2][4];
            const unsigned char *rowp[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                r[h] = r0 + h * WAVES * RPW + lane / LPR;
                rowp[h] = stage + shift + (r[h] < a.chunk_rows ? r[h] : 0) * (int)a.pitch;
            }
            auto read = [&](auto dt) INLINE_LAMBDA {
                constexpr int DT = decltype(dt)::value;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    x[h][0] = widen_at<DT>(rowp[h], tr.j0); x[h][1] = widen_at<DT>(rowp[h], tr.j1);
                    x[h][2] = widen_at<DT>(rowp[h], tr.j2); x[h][3] = widen_at<DT>(rowp[h], tr.j3);
                }
            };
            switch (a.dtype) {
            case kF32: read(std::integral_constant<int, kF32>{}); break;
            case kF16: read(std::integral_constant<int, kF16>{}); break;
            case kBF16: read(std::integral_constant<int, kBF16>{}); break;
            default: read(std::integral_constant<int, kU8>{}); break;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 1 && r0 + WAVES * RPW >= a.chunk_rows) break;
                unsigned code = hash_regs(tr, x[h][0], x[h][1], x[h][2], x[h][3]);
                code = real ? code : 0u;
                if constexpr (AVG) {
                    if (r[h] < a.chunk_rows) reinterpret_cast<uint16_t *>(codes_l)[r[h] * LPR + c] = (uint16_t)(code << (4 + TS));
                } else if constexpr (!ENC) {
                    if (r[h] < a.chunk_rows) codes_l[r[h] * LPR + (c & 3) * KGP + (c >> 2)] = (unsigned char)(code << 4);
                }
                if (a.codes_out && col_block == 0) {
                    // eight codes to a register, the first of eight lanes stores them
                    unsigned q = code | (rows::from_lane_above<1>(code) << 4);
                    q |= rows::from_lane_above<2>(q) << 8;
                    if constexpr (LPR > 4) q |= rows::from_lane_above<4>(q) << 16;
                    constexpr int HELD = LPR > 4 ? 8 : 4;
                    if (c % HELD == 0 && r[h] < a.chunk_rows && row0 + r[h] < a.N) {
                        uint8_t *dst = a.codes_out + (row0 + r[h]) * Cb + c / 2;
                        for (int b = 0; b < HELD / 2; ++b)
                            if (c / 2 + b < Cb) dst[b] = (uint8_t)(q >> (8 * b));
                    }
                }
            }
        }
    };

    auto encode_columns = [&]() INLINE_LAMBDA {
#pragma unroll
        for (int u = 0; u < BOOKS; ++u) {
            const int book = wave + WAVES * u;
            if (book >= 4 * KG) break;
            Tree tree;
            const float *th = a.thresholds + 16 * min(book, a.C - 1);
#pragma unroll
            for (int k = 0; k < 15; ++k) tree.t[k] = th[k];
            float x[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                switch (a.dtype) {
                case kF32: x[t] = __uint_as_float(raw[u][t]); break;
                case kF16: x[t] = (float)__builtin_bit_cast(_Float16, (uint16_t)raw[u][t]); break;
                case kBF16: x[t] = __uint_as_float(raw[u][t] << 16); break;
                default: x[t] = (float)raw[u][t]; break;
                }
            }
            const unsigned code = book < a.C ? hash_regs(tree, x[0], x[1], x[2], x[3]) : 0u;
            codes_l[lane * LPR + (book & 3) * KGP + (book >> 2)] = (unsigned char)(code << 4);
        }
    };
    // (by columns: the packed codes, from where the wavefronts have left them)
    auto store_codes = [&](int64_t row0) INLINE_LAMBDA {
        const int rows = a.N - row0 < 64 ? (int)(a.N - row0) : 64;
        for (int at = tid; at < rows * Cb; at += THREADS) {
            const int r = at / Cb, b = at - r * Cb, c0 = 2 * b, c1 = c0 + 1;
            const unsigned char *mine = codes_l + r * LPR;
            const unsigned low = mine[(c0 & 3) * KGP + (c0 >> 2)] >> 4, high = c1 < a.C ? mine[(c1 & 3) * KGP + (c1 >> 2)] : 0u;
            a.codes_out[row0 * Cb + at] = (uint8_t)(low | high);
        }
    };

    if constexpr (ENC) {
        while (true) {
            const int next = chunk + a.row_groups;
            const bool more = next < a.chunks;
            if constexpr (COLS) {
                encode_columns();
                __syncthreads();
                if (more) fetch_columns(next);
                store_codes((int64_t)chunk * 64);
            } else {
                write_rows();
                __syncthreads();
                if (more) fetch_rows(next);
                encode((int64_t)chunk * a.chunk_rows);
            }
            if (!more) return;
            __syncthreads();
            chunk = next;
        }
    }

    // piece n of a thread: tile tid % tiles (neighbours read neighbouring columns), code (tid / tiles) % 16, codebook
    // tid / (16 tiles) + n BLOCKS / tiles
    const unsigned table_bytes = 16u * (unsigned)a.C * (unsigned)a.M;      // (below 2^31: the launcher)
    const int p_tile = tid & (tiles - 1), p_code = (tid >> a.tile_shift) & 15, p_book = tid >> (4 + a.tile_shift);
    const int book_step = BLOCKS >> a.tile_shift;
    const int n_pieces = ((4 * KG << a.tile_shift) + BLOCKS - 1) / BLOCKS;
    const int last_tile = (a.M - 1 - col0) >> 4;
    const unsigned p_first = (unsigned)(16 * p_book + p_code) * (unsigned)a.M +
                             (unsigned)(col0 + 16 * (p_tile < last_tile ? p_tile : last_tile));
    const unsigned p_step = (unsigned)(16 * book_step) * (unsigned)a.M, p_last = table_bytes - 16;
    uint4 piece[PIECES];
#pragma unroll
    for (int n = 0; n < PIECES; ++n) {
        if (n < n_pieces) {
            // (tiles and codebooks that do not exist read others' entries; the last pieces end where the tables end)
            const unsigned at = p_first + (unsigned)n * p_step;
            __builtin_memcpy(&piece[n], a.luts + (at < p_last ? at : p_last), 16);
        }
    }

    // the wavefront's tiles, and its share of the rows where there are fewer tiles than wavefronts
    constexpr int NTW_SHIFT = NTW == 2 ? 1 : 0;
    const int wave_tiles = tiles >> NTW_SHIFT, tile0 = NTW * (wave & (wave_tiles - 1));
    const int share = wave >> (a.tile_shift - NTW_SHIFT), shares = WAVES >> (a.tile_shift - NTW_SHIFT);
    int col[NTW];
    float sc[NTW][4], of[NTW][4];
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
        col[t] = AVG ? col0 + 4 * (lane & ((4 << TS) - 1)) : col0 + 16 * (tile0 + t) + 4 * g;
        if (col0 + 16 * tiles <= a.M) {
            __builtin_memcpy(sc[t], a.scale + col[t], 16);
            __builtin_memcpy(of[t], a.offset + col[t], 16);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = col[t] + r < a.M ? col[t] + r : a.M - 1;
                sc[t][r] = a.scale[m];
                of[t][r] = a.offset[m];
            }
        }
    }
    if constexpr (!AVG) mfma::fill_one_hot_table(one_hot, tid);

    v4i T[NTW][KG];
    const int first_sum = 128 * a.C;

    // ---- scan: H groups of 16 rows at a time, two chains of sums or more ----
    auto scan = [&](int64_t row0, int r0, auto groups) INLINE_LAMBDA {
        constexpr int H = decltype(groups)::value, CHAINS = H == 1 && NTW == 1 && KG > 1 ? 2 : 1;
        unsigned word[H][(KGP + 3) / 4];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            // (codes of rows that do not exist are any bytes: within the one-hot table)
            const unsigned char *mine = codes_l + (r0 + 16 * shares * h + i) * LPR + g * KGP;
            if constexpr (KGP >= 4) {
#pragma unroll
                for (int q = 0; q < KGP / 4; ++q) word[h][q] = reinterpret_cast<const unsigned *>(mine)[q];
            } else if constexpr (KGP == 2) {
                word[h][0] = *reinterpret_cast<const uint16_t *>(mine);
            } else {
                word[h][0] = *mine;
            }
        }
        v4i sum[H][NTW][CHAINS];
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int t = 0; t < NTW; ++t)
#pragma unroll
                for (int q = 0; q < CHAINS; ++q) {
                    const int start = q == 0 ? first_sum : 0;
                    sum[h][t][q] = v4i{start, start, start, start};
                }
#pragma unroll
        for (int G = 0; G < KG; ++G) {
            v4i oh[H];
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const unsigned at = (word[h][G >> 2] >> (8 * (G & 3))) & 240u;
                oh[h] = *reinterpret_cast<const v4i *>(reinterpret_cast<const unsigned char *>(one_hot) + at);
            }
#pragma unroll
            for (int t = 0; t < NTW; ++t)
#pragma unroll
                for (int h = 0; h < H; ++h)
                    sum[h][t][G % CHAINS] = __builtin_amdgcn_mfma_i32_16x16x64_i8(T[t][G], oh[h], sum[h][t][G % CHAINS], 0, 0, 0);
        }
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const int r = r0 + 16 * shares * h + i;
            const int64_t row = row0 + r;
            if (r < a.chunk_rows && row < a.N) {
#pragma unroll
                for (int t = 0; t < NTW; ++t) {
                    v4i f = sum[h][t][0];
                    if constexpr (CHAINS == 2) f += sum[h][t][1];
                    if (a.out) {
                        float *dst = a.out + row * a.ldo + col[t];
                        f4 v;
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] = fmaf((float)f[q], sc[t][q], of[t][q]);
                        if (col[t] + 3 < a.M) {
                            __builtin_memcpy(dst, &v, 16);
                        } else {
#pragma unroll
                            for (int q = 0; q < 3; ++q)
                                if (col[t] + q < a.M) dst[q] = v[q];
                        }
                    }
                    if (a.acc) {
                        uint16_t *dst = a.acc + row * a.M + col[t];
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (col[t] + q < a.M) dst[q] = (uint16_t)f[q];
                    }
                }
            }
        }
    };

    // ---- averages: 64 / (4 << TS) rows at a time ----
    auto average = [&](int64_t row0) INLINE_LAMBDA {
        constexpr int LANES = 4 << TS, ROWS = 64 / LANES, BOOK = 256 << TS;
        const unsigned char *mine = tables + 4 * (lane & (LANES - 1));
#pragma unroll 1
        for (int r0 = wave * ROWS; r0 < a.chunk_rows; r0 += WAVES * ROWS) {
            const int r = r0 + lane / LANES, rr = r < a.chunk_rows ? r : 0;
            const uint4 *codes = reinterpret_cast<const uint4 *>(codes_l + 2 * rr * LPR);
            uint32_t even = 0, odd = 0;
#pragma unroll
            for (int b = 0; b < KG / 4; ++b) {
                const uint4 q0 = codes[2 * b], q1 = codes[2 * b + 1];
                const uint32_t q[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
                uint32_t y[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const uint32_t at = u % 2 ? q[u / 2] >> 16 : q[u / 2] & 0xffffu;
                    y[u] = *reinterpret_cast<const uint32_t *>(mine + (16 * b + u) * BOOK + at);
                }
#pragma unroll
                for (int span = 1; span < 16; span *= 2)
#pragma unroll
                    for (int u = 0; u < 16; u += 2 * span) y[u] = __builtin_amdgcn_lerp(y[u], y[u + span], 0x01010101u);
                even += y[0] & 0x00FF00FFu;
                odd += __builtin_amdgcn_perm(y[0], y[0], 0x0c030c01u);
            }
            const int64_t row = row0 + r;
            if (r < a.chunk_rows && row < a.N && col[0] < a.M) {
                // 16 times the sum of the blocks' averages, less the excess to be expected of them (Theorem D.1)
                const uint32_t f[4] = {16 * (even & 0xFFFFu), 16 * (odd & 0xFFFFu), 16 * (even >> 16), 16 * (odd >> 16)};
                if (a.out) {
                    float *dst = a.out + row * a.ldo + col[0];
                    f4 v;
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = fmaf((float)((int)f[q] - a.C), sc[0][q], of[0][q]);
                    if (col[0] + 3 < a.M) {
                        __builtin_memcpy(dst, &v, 16);
                    } else {
#pragma unroll
                        for (int q = 0; q < 3; ++q)
                            if (col[0] + q < a.M) dst[q] = v[q];
                    }
                }
                if (a.acc) {
                    uint16_t *dst = a.acc + row * a.M + col[0];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (col[0] + q < a.M) dst[q] = (uint16_t)f[q];
                }
            }
        }
    };

    if constexpr (COLS) {
        encode_columns();
    } else if constexpr (CODES) {
        deal_codes();
    } else {
        write_rows();
        __syncthreads();
        encode((int64_t)chunk * a.chunk_rows);
    }
    // ---- tables: registers -> LDS -> the matrix instruction's operands ----
    if (a.overlay) __syncthreads();
    {
        // (averages: as it lies in memory)
        constexpr int STEP = AVG ? 256 : kTileBytes;
        unsigned char *dst = AVG ? tables + ((p_book * 16 + p_code) << (4 + a.tile_shift)) + 16 * p_tile
                                 : tables + ((p_book << a.tile_shift) + p_tile) * STEP + p_code * 16;
        const unsigned flip = AVG ? 0u : 0x80808080u;            // t - 128 as signed bytes
        if (a.C == 4 * KG && col0 + 16 * tiles <= a.M) {
            // (all there is to them where every column and codebook exists: N = 3490, D = 1024, M = 512, C = 32 10.6 and 9.7 us)
#pragma unroll
            for (int n = 0; n < PIECES; ++n)
                if (n < n_pieces && p_book + n * book_step < 4 * KG)
                    *reinterpret_cast<uint4 *>(dst + n * BLOCKS * STEP) =
                        make_uint4(piece[n].x ^ flip, piece[n].y ^ flip, piece[n].z ^ flip, piece[n].w ^ flip);
        } else {
#pragma unroll
            for (int n = 0; n < PIECES; ++n) {
                if (n < n_pieces) {
                    const int book = p_book + n * book_step;
                    const unsigned at = p_first + (unsigned)n * p_step;
                    if (at > p_last && at < table_bytes) {
                        // the end of the tables: move the bytes down (what moves in stands for columns that do not exist)
                        const unsigned over = 8 * (at - p_last);
                        const uint64_t lo = (uint64_t)piece[n].y << 32 | piece[n].x, hi = (uint64_t)piece[n].w << 32 | piece[n].z;
                        const uint64_t l = over >= 64 ? hi >> (over - 64) : lo >> over | hi << (64 - over), u = over >= 64 ? 0 : hi >> over;
                        piece[n] = make_uint4((uint32_t)l, (uint32_t)(l >> 32), (uint32_t)u, (uint32_t)(u >> 32));
                    }
                    // nothing where there is no codebook
                    const unsigned keep = book < a.C ? ~0u : 0u;
                    const uint4 v = make_uint4((piece[n].x ^ flip) & keep, (piece[n].y ^ flip) & keep, (piece[n].z ^ flip) & keep,
                                               (piece[n].w ^ flip) & keep);
                    if (book < 4 * KG) *reinterpret_cast<uint4 *>(dst + n * BLOCKS * STEP) = v;
                }
            }
        }
    }
    __syncthreads();
    if constexpr (!AVG) {
        typedef __attribute__((address_space(3))) v2i lds_v2i;
        const unsigned char *block = tables + ((g << a.tile_shift) + tile0) * kTileBytes + 8 * i;
        const int step = (4 << a.tile_shift) * kTileBytes;
#pragma unroll
        for (int G = 0; G < KG; ++G)
#pragma unroll
            for (int t = 0; t < NTW; ++t) {
                const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(block + G * step + t * kTileBytes));
                const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(block + G * step + t * kTileBytes + 128));
                T[t][G] = v4i{lo.x, lo.y, hi.x, hi.y};
            }
    }
    if (a.overlay && chunk + a.row_groups < a.chunks) __syncthreads();

    while (true) {
        const int64_t row0 = (int64_t)chunk * a.chunk_rows;
        const int next = chunk + a.row_groups;
        const bool more = next < a.chunks;
        if constexpr (COLS) {
            if (more) fetch_columns(next);
            if (a.codes_out && col_block == 0) store_codes(row0);
        } else if constexpr (CODES) {
            if (more) fetch_codes(next);
        } else {
            if (more) fetch_rows(next);
        }
        if constexpr (AVG) {
            average(row0);
        } else {
#pragma unroll 1
            for (int r0 = 16 * share; r0 < a.chunk_rows; r0 += 32 * shares) {
                if (r0 + 16 * shares < a.chunk_rows) scan(row0, r0, std::integral_constant<int, 2>{});
                else scan(row0, r0, std::integral_constant<int, 1>{});
            }
        }
        if (!more) break;
        chunk = next;
        if constexpr (COLS) {
            __syncthreads();                 // (the codes have been read)
            encode_columns();
        } else if constexpr (CODES) {
            __syncthreads();
            deal_codes();
        } else {
            write_rows();
            __syncthreads();
            encode((int64_t)chunk * a.chunk_rows);
        }
        __syncthreads();
    }
}

template <int KG, int NTW, int PF>
int launch_blocks(const BlockArgs &a, int grid, size_t lds, hipStream_t stream)
{
    if (int rc = allow_full_lds<fused_blocks_kernel<KG, NTW, PF>>(); rc != MADDNESS_OK) return rc;
    note_kernel("fused_blocks_kernel, A by rows", __PRETTY_FUNCTION__);
    hipLaunchKernelGGL((fused_blocks_kernel<KG, NTW, PF>), dim3(grid), dim3(kBlockThreads), lds, stream, a);
    return check_hip(hipGetLastError(), "launch fused_blocks_kernel");
}

template <int KG, int NTW>
int launch_tiles(const BlockArgs &a, int kb, int grid, size_t lds, hipStream_t stream)
{
    return kb == 32   ? launch_blocks<KG, NTW, 4>(a, grid, lds, stream)
           : kb == 64 ? launch_blocks<KG, NTW, 8>(a, grid, lds, stream)
                      : launch_blocks<KG, NTW, 16>(a, grid, lds, stream);
}

template <int KG>
int launch_books(const BlockArgs &a, int ntw, int kb, int grid, size_t lds, hipStream_t stream)
{
    if constexpr (KG <= 8)
        if (ntw == 2) return launch_tiles<KG, 2>(a, kb, grid, lds, stream);
    return launch_tiles<KG, 1>(a, kb, grid, lds, stream);
}

template <int KG>
int launch_columns(const BlockArgs &a, int grid, size_t lds, hipStream_t stream)
{
    if (int rc = allow_full_lds<fused_blocks_kernel<KG, 1, 1, true>>(); rc != MADDNESS_OK) return rc;
    note_kernel("fused_blocks_kernel, A by columns", __PRETTY_FUNCTION__);
    hipLaunchKernelGGL((fused_blocks_kernel<KG, 1, 1, true>), dim3(grid), dim3(kBlockThreads), lds, stream, a);
    return check_hip(hipGetLastError(), "launch fused_blocks_kernel");
}

template <int KG>
int launch_codes(const BlockArgs &a, int grid, size_t lds, hipStream_t stream)
{
    if (int rc = allow_full_lds<fused_blocks_kernel<KG, 1, 1, false, false, 0, true>>(); rc != MADDNESS_OK) return rc;
    note_kernel("fused_blocks_kernel, scan", __PRETTY_FUNCTION__);
    hipLaunchKernelGGL((fused_blocks_kernel<KG, 1, 1, false, false, 0, true>), dim3(grid), dim3(kBlockThreads), lds, stream, a);
    return check_hip(hipGetLastError(), "launch fused_blocks_kernel");
}

template <int KG>
int launch_codes_of_columns(const BlockArgs &a, size_t lds, hipStream_t stream)
{
    note_kernel("fused_blocks_kernel, codes of columns", __PRETTY_FUNCTION__);
    hipLaunchKernelGGL((fused_blocks_kernel<KG, 1, 1, true, false, 0, false, true>), dim3(a.row_groups), dim3(kBlockThreads), lds, stream, a);
    return check_hip(hipGetLastError(), "launch fused_blocks_kernel");
}

template <int KG>
int launch_codes_of_rows(const BlockArgs &a, size_t lds, hipStream_t stream)
{
    note_kernel("fused_blocks_kernel, codes of rows", __PRETTY_FUNCTION__);
    hipLaunchKernelGGL((fused_blocks_kernel<KG, 1, 4, false, false, 0, false, true>), dim3(a.row_groups), dim3(kBlockThreads), lds, stream, a);
    return check_hip(hipGetLastError(), "launch fused_blocks_kernel");
}

template <int KG, int TS>
int launch_averaged(const BlockArgs &a, int kb, int grid, size_t lds, hipStream_t stream)
{
    note_kernel("fused_blocks_kernel, averages", __PRETTY_FUNCTION__);
    if (kb == 32) {
        if (int rc = allow_full_lds<fused_blocks_kernel<KG, 1, 4, false, true, TS>>(); rc != MADDNESS_OK) return rc;
        hipLaunchKernelGGL((fused_blocks_kernel<KG, 1, 4, false, true, TS>), dim3(grid), dim3(kBlockThreads), lds, stream, a);
    } else {
        if (int rc = allow_full_lds<fused_blocks_kernel<KG, 1, 8, false, true, TS>>(); rc != MADDNESS_OK) return rc;
        hipLaunchKernelGGL((fused_blocks_kernel<KG, 1, 8, false, true, TS>), dim3(grid), dim3(kBlockThreads), lds, stream, a);
    }
    return check_hip(hipGetLastError(), "launch fused_blocks_kernel");
}

template <int KG>
int launch_averaged_tiles(const BlockArgs &a, int kb, int grid, size_t lds, hipStream_t stream)
{
    if (a.tile_shift == 1) return launch_averaged<KG, 1>(a, kb, grid, lds, stream);
    if constexpr (KG <= 8)
        if (a.tile_shift == 3) return launch_averaged<KG, 3>(a, kb, grid, lds, stream);
    return launch_averaged<KG, 2>(a, kb, grid, lds, stream);
}

// The options that say how many regions and workgroups the phased kernels take leave this one out: what they are set for is to
// reach those kernels with few rows.
bool left_out() { return option(MADDNESS_OPT_PHASED_ROWS) || option(MADDNESS_OPT_MAX_WORKGROUPS); }

// How a call is cut up.
struct Plan {
    int tile_shift, col_blocks;
    int turns;                // chunks that a workgroup takes
    int64_t groups, rows;     // workgroups to a block of columns, rows of a chunk
    bool shared;              // two workgroups to a compute unit
};

// Kernel sizes: codebooks (at most 64).  Padding, up to half of a size, costs less than what else takes such numbers: by rows N = 2361, D = 57, M = 117, C = 3 7.5 us on the
// general kernel and 3.8, N = 1470, D = 864, M = 3, C = 54, bytes 64 and 5.2, N = 942, D = 720, M = 497, C = 40 26 on the phased kernel and 8.1, N = 395657, D = 198, M = 719, C = 9, bytes
// 428 and 381; by columns (blocks_pay and launch_fused_blocks_cols say where not) 140 calls 3.6 and, of many rows, 2.3 times as fast.
int kernel_codebooks(int C)
{
    for (int s : {4, 8, 16, 24, 32, 48})
        if (s >= C) return s;
    return 64;
}

Plan make_plan(int64_t N, int64_t pitch, bool whole, int M, int KC, int tile_shift, bool shared)
{
    const DeviceInfo &dev = device_info();
    const int wgs = shared ? 2 * dev.cus : dev.cus, kb = shared ? 32 : 128, tiles = (M + 15) / 16;
    Plan q;
    q.tile_shift = tile_shift; q.shared = shared;
    q.col_blocks = (tiles + (1 << tile_shift) - 1) >> tile_shift;
    q.groups = std::max(1, wgs / q.col_blocks);
    if (q.groups > 8 && q.col_blocks > 1) q.groups = q.groups / 8 * 8;
    const int64_t lds = dev.lds_per_block / (shared ? 2 : 1) - 256;
    const int64_t tables = (int64_t)KC * kTileBytes << tile_shift;
    const int64_t most = std::min((kb * 1024 - (whole ? 0 : 16)) / pitch,
                                  (lds - std::max<int64_t>(tables, kb * 1024)) / lanes_per_row(KC) - 16 * (kBlockWaves + 1));
    const int64_t share = std::max<int64_t>(8, (N + q.groups - 1) / q.groups);
    if (most < 1) { q.rows = 0; q.turns = 1 << 30; return q; }
    q.turns = (int)std::min<int64_t>(1 << 30, (share + most - 1) / most);
    q.rows = (share + q.turns - 1) / q.turns;
    return q;
}

Plan choose_plan(int64_t N, int64_t pitch, bool whole, int M, int KC)
{
    int shift = 0;
    while (shift < 3 && (16 << shift) < M) ++shift;
    Plan plan = make_plan(N, pitch, whole, M, KC, shift, false);
    // One chunk, but of so many rows that two workgroups to a compute unit and several smaller chunks, one's on their way while the
    // other has its turn, are faster beside small tables (N = 260100, D = 27, M = 2, C = 4 9.9 and 8.2 us; N = 26900, D = 64, M = 767, C = 8,
    // bfloat16 26.3 and 22.9; N = 44635, D = 120, M = 100, C = 15 12.3 and 11.1; N = 15853, D = 272, M = 100, C = 16, 68 KiB, 7.9 and 8.0).
    if (plan.turns == 1 && !(KC <= 8 && plan.rows * pitch > 32 * 1024) && !(KC == 16 && plan.rows * pitch > 72 * 1024)) return plan;
    // More than one chunk to a workgroup.  Twice the columns to a workgroup are half the rows, which every block of columns
    // reads and encodes again (N = 2941, D = 384, M = 1000, C = 24: 11.9 and 10.2 us); where one block of columns has them all,
    // two workgroups to a compute unit, one with its rows on their way while the other has its turn (N = 131072, D = 128,
    // M = 10, C = 8: 27 and 13.7 us with 128-byte chunks of one workgroup; from 32 codebooks on the tables leave no room:
    // N = 32768, D = 512, M = 5, C = 32 14.5 and 17.6).
    if (KC <= 32 && shift == 3) {
        const Plan wide = make_plan(N, pitch, whole, M, KC, 4, false);
        if (wide.col_blocks < plan.col_blocks && wide.rows > 0) plan = wide;
    }
    if (KC <= 24 && plan.tile_shift <= 3) {
        const Plan shared = make_plan(N, pitch, whole, M, KC, shift, true);
        if (shared.rows > 0) plan = shared;
    }
    return plan;
}

// Up to 8 codebooks the phased kernel pays for padding: N = 131072, D = 128, M = 5, C = 8 26 and 13 us (there and here); N = 382808, D = 119, M = 155, C = 7
// 200 and 115; bytes N = 726104, M = 32 126 and 40.  But it reads a row once for all results, and these blocks once for every 256 of them, of which they
// write parts of lines.  459 calls that either takes, each after one of its own kind: 15 of those that these lines take are slower here by more than 3 %
// (4 to 12), of those that they leave 9 would be faster.
bool few_codebooks_pay(const BlockArgs &a, const Plan &plan)
{
    // a block of columns of at most 128: whatever the rows, to 40 turns (N = 932130, D = 176, M = 53 193 and 152); N = 895395, D = 626, M = 65, C = 2 421 and 470 (135)
    if (plan.tile_shift < 4) return plan.turns <= 64;
    const int M = a.M;
    const int64_t results = a.N * M;
    if (a.dtype == MADDNESS_F32 && a.C == 8 && M % 4 == 0) {
        // There whole registers of four results.  Whole lines: N = 85003, D = 128, M = 608 63 and 54 (5 turns), N = 580419, D = 240, M = 928 523 and 800 (67), N = 127840, D = 168,
        // M = 672 93 and 123 (9), N = 99563, D = 128, M = 320 43 and 52 (4); short rows N = 525885, D = 40, M = 736 385 and 328 (9), N = 583765, D = 88, M = 512 318 and 272.  Others: N = 539796, D = 168, M = 524 637 and 430 (35), N = 309841, D = 32, M = 200 121 and 58;
        // one block of columns, written by 64 bytes there or mostly padding here: N = 210517, D = 244, M = 240 79 and 98 (7), N = 73405, D = 232, M = 156 27 and 32 (3),
        // N = 487872, D = 212, M = 232 1.14 times (13).
        if (M % 32 == 0 && a.ldo % 32 == 0) return plan.turns <= (M <= 320 ? 2 : 4) || a.row_bytes < (M <= 512 ? 384 : 320);
        return plan.turns <= 2 || a.row_bytes < 640 || M > 256 || (M > 160 && M % 16 != 0);
    }
    // There results by lines through LDS, 512 columns to a pass: N = 121293, D = 200, M = 286 63 and 56, N = 340947, D = 224, M = 367 181 and 212 (19 turns), N = 286483, D = 128, M = 463 155 and 178 (9), N = 124696, D = 96, M = 415,
    // binary16 70 and 50; N = 449389, D = 104, M = 617 509 and 353; C = 7 N = 263590, D = 21, M = 984 268 and 310 (259 Mi results).
    if (a.dtype == MADDNESS_F32) return M > 320 && M <= 512 ? plan.turns <= 4 || a.row_bytes < 512 : M <= 900 || results < (200 << 20);
    // Narrow types, from where the results leave the last-level cache: bytes N = 613877, D = 24, M = 485 333 and 513, N = 92976, D = 24, M = 418 61 and 46 (37 Mi); N = 154844, D = 84,
    // M = 886 179 and 211; M = 527, D = 154, binary16 1.52 times, M = 739, D = 184 1.25, M = 612, D = 16 0.89 (508 Mi); bytes M = 308 1.07 (210 Mi), M = 326 0.83 (267 Mi);
    // whole lines N = 577387, D = 44, M = 800 463 and 370.
    if (M % 32 == 0 || results < (100 << 20)) return true;
    return M <= 352 ? results < (250 << 20) : M > 512 && M <= 768 && (a.row_bytes >= 64 || results < (200 << 20));
}

// Whether this kernel is the faster one.  only_if_faster = false: instead of the general kernel, which no other kernel would
// take the call from.  Times in us, this kernel's last.
bool blocks_pay(const BlockArgs &a, int KC, const Plan &plan, bool only_if_faster)
{
    // Rows of many bytes to a codebook are read whole here; the general kernel asks for 64 bytes of them to a split value, which pays where there are
    // many of both: N = 13387, D = 1619, M = 17, C = 1, binary16 6.2 and 10.7, N = 12435, D = 1226, M = 81, C = 2 8.7 and 16.0; N = 12233, D = 1090, M = 79, C = 1, bytes 8.0 and 5.9 (13 MiB),
    // N = 13129, D = 1415, M = 84, C = 5, binary16 11.6 and 11.1 (566 bytes to a codebook).
    // Few entries to add need no line of their own: N = 8192, D = 27, M = 3, C = 4 both take as long as a launch where calls are made one by one, 4.9 and 3.6 in a graph;
    // N = 97583, D = 36, M = 3, C = 9, binary16 14.5 and 7.6, N = 5693, D = 44, M = 3, C = 11, binary16 14.4 and 4.0; none of 455 calls with tables of at most 8 KiB was faster there
    // but for such rows.
    if (a.row_bytes > 600 * a.C && a.N * a.row_bytes > (16 << 20)) return false;
    if (!only_if_faster) return true;
    if (KC <= 8) return few_codebooks_pay(a, plan);
    // One chunk of rows to a workgroup: N = 1891, D = 768, M = 785, C = 48, binary16 45.3 and 11.7; N = 10000, D = 512, M = 100,
    // C = 32 11.5 and 9.1; N = 8192, D = 512, M = 512, C = 32 15.0 and 12.8; N = 4096, D = 512, M = 1005, C = 32 30.6 and 14.5.
    if (plan.turns == 1) return true;
    // Several: the other kernels read a row once for all columns and keep more of it on its way, and the wider and longer the
    // rows the sooner they win.
    // 16 and 24: N = 65536, D = 192, M = 10, C = 24 26 and 13 (2 turns); N = 248254, D = 256, M = 71, C = 16, bfloat16 65 and 46 (4);
    // N = 524288, D = 120, M = 13, C = 15 82 and 54 (8); N = 1048576, D = 320, M = 10, C = 16 230 and 262 (41);
    // two blocks of columns N = 87536, D = 120, M = 474, C = 15, bfloat16 53 and 67; N = 73759, D = 256, M = 256, C = 16 29 and 39.
    if (KC <= 24) return a.M <= 128 ? plan.turns <= 12 : plan.turns <= 2 && plan.tile_shift == 4 && a.C != 16;
    // 32: N = 51479, D = 224, M = 247, C = 32 37 and 30 (2 turns); N = 7417, D = 480, M = 1000, C = 30 27 and 18 (2);
    // N = 65536, D = 352, M = 100, C = 32 33 and 35 (3); N = 262144, D = 256, M = 10, C = 32 74 and 65 (8); N = 175867, D = 512, M = 54 78
    // and 89 (11); N = 75494, D = 256, M = 512 48 and 67 (5).
    if (KC == 32) return plan.turns <= (a.M <= 32 ? 8 : 2);
    // 48 and 64: N = 24287, D = 1024, M = 36, C = 64, bfloat16 21 and 17 (2); N = 63790, D = 528, M = 7, C = 48 40 and 33 (5);
    // N = 126493, D = 384, M = 128, C = 48 70 and 75 (6); N = 31831, D = 704, M = 256, C = 64, binary16 24 and 34 (3).
    return a.M <= 128 && plan.turns <= (a.M <= 32 ? 5 : 2);
}

// The scan alone: whether blocks are faster than what else takes the call.  Times in us, the blocks' last.  `regular`: shapes of which the
// matrix-core kernel without blocks reads and writes 2 to 16 bytes at a time; of others it goes by single bytes and floats.
bool scan_blocks_pay(const BlockArgs &a, int64_t ldo, int KC, int64_t turns)
{
    const int C = a.C, M = a.M, NT = C <= 32 ? 4 : 2;
    const int64_t results = a.N * M;
    const bool regular = C % 8 == 0 && aligned_to(a.A, 16) && M % NT == 0 && aligned_to(a.luts, NT) &&
                         !(a.out && (ldo % NT != 0 || !aligned_to(a.out, 4 * NT))) && !(a.acc && !aligned_to(a.acc, 2 * NT));
    if (M <= 16) {
        // The general kernel, which does no padded work, keeps many rows with next to nothing to add (N = 458095, M = 2, C = 5 7.5 and 9.8;
        // N = 150549, M = 5, C = 5 6.0 and 6.5; with few rows both take as long as a launch), and those that come by single bytes and
        // long chunks (N = 506401, M = 2, C = 30 19.1 and 19.7; N = 1033459, M = 3, C = 12 17 and 20; N = 277910, M = 2 15.1 and 14.1).
        if (C <= 8) return M <= 5 ? a.N <= (1 << 15) : M <= 12 || !regular || results < (3 << 20);
        if (a.unit == 1 && M <= 3) return turns <= 4;
        // (and of more than 48 codebooks, whose chunks are 64 rows: N = 133462, M = 12, C = 61 18.9 and 25.2, N = 1519685, M = 7, C = 60 0.53 times, N = 41505, M = 8, C = 54 0.78, N = 31202,
        // M = 16, C = 53 1.30; results that the general kernel does not add four to a word keep them to where both take as long: N = 134422, M = 10, C = 50 27.8 and 19.1, N = 127361, M = 9,
        // C = 51 28.1 and 19.4; 300000 to 500000 rows 0.99, more 0.77)
        if (a.unit == 1 && C > 48) return turns <= 2 || (M > 8 && M != 12 && a.N <= 300000);
        // N = 334, M = 10, C = 8 4.8 and 4.1; N = 1515582, M = 3, C = 48 100 and 37; N = 2339262, M = 16, C = 15 116 and 43; N = 760602, M = 16, C = 32
        // 25 and 17.  40, 56 and 64 codebooks: N = 90821, M = 10, C = 64 13.1 and 7.3 (2 turns), N = 1231121, M = 8 41 and 51 (10).
        return C <= 32 || C == 48 || !regular || turns <= (C == 56 ? 1 : 3);
    }
    if (!regular) {
        // N = 117, M = 300, C = 32 7.6 and 4.2; N = 3387, M = 785, C = 24 15.9 and 8.2; N = 656328, M = 20, C = 31 212 and 24; N = 376888,
        // M = 100, C = 31 128 and 44: whatever the size, but for results that may be written by whole lines (M = 785, C = 24, N = 117350 91 and 131).
        return results < (12 << 20) || M < 64 || M % 32 == 0 || a.acc || !a.out || ldo != M || !aligned_to(a.out, 128) || a.N < 16384;
    }
    // Rows of results that begin on 128-byte lines: the other kernel's blocks of columns are as good, and what counts is how much of the blocks
    // here is padding.  C = 8: N = 38200, M = 64 5.6 and 5.8 (2.3 Mi results); 16: N = 153, M = 512 16.6 and 4.2, N = 29654, M = 192 8.3 and 9.8 (5.4, 7.2 with
    // padding), N = 8922, M = 640 8.0 and 8.5 (5.4), N = 22553, M = 256 8.3 and 8.2 (5.5); 24: N = 45793, M = 128 9.5 and 9.2 (5.6); 32: N = 88025, M = 64
    // 11.0 and 9.2 (5.4), N = 42606, M = 192 12.1 and 13.4 (7.8, 10.4), N = 165055, M = 64 13.1 and 13.8 (10); 48 and 64: N = 1341, M = 256 6.0 and 5.6, N = 5420,
    // M = 512 8.6 and 8.6 (2.6), N = 6197, M = 640 11.2 and 12.0 (3.8), N = 97347, M = 32 9.1 and 8.9 (3), N = 152246, M = 32 12.7 and 16.0 (4.6).
    const int64_t padded = a.N * 16 * ((int64_t)a.col_blocks << a.tile_shift);
    const bool on_lines = ldo % 32 == 0;
    if (on_lines) {
        if (C <= 32) return padded < (C == 8 ? 2 << 20 : C == 16 ? 4 << 20 : C == 24 ? 5 << 20 : 7 << 20);
        if (C == KC) return M <= 64 ? turns <= 2 && padded < (4 << 20) : turns == 1 && 2 * padded < (5 << 20);
    }
    // Others: N = 109905, M = 36, C = 8 7.4 and 7.9 (3.8); N = 18831, M = 300, C = 16 11.0 and 9.7 (5.4), N = 35862, M = 200 11.3 and 10.4 (6.8); N = 319639, M = 36,
    // C = 32 22.5 and 19.8 (11).  48 and 64: N = 28337, M = 200, C = 64 18.2 and 17.0 (1 turn), N = 112329, M = 36, C = 48 14.1 and 12.8 (2), N = 46504, M = 200, C = 64
    // 22.6 and 23.6 (2, 9 Mi).
    if (C <= 24) return results < (C == 8 ? 3 << 20 : 7 << 20);
    if (C <= 32) return results < (12 << 20);
    // 40 and 56, padded here: N = 1341, M = 256, C = 56 6.0 and 5.6; N = 14178, M = 512, C = 40 10.8 and 14.5.
    if (C != KC) return results < (1 << 20);
    return turns == 1 || (turns == 2 && results < (5 << 20));
}

// A stored by columns, 16, 32 or 64 codebooks: whether blocks are faster than the kernels that take whole rows of results, the phased
// one (to 2^17 rows a row to a lane, beyond, where columns lie on four elements, four) and, of more rows, cols_kernel.  Lines drawn through 1085 calls with 1
// to 1024 results, columns used once and many times; of 612 others, each after one of its own kind, 10 that they take are slower here by more than 3 % (4 to 17),
// 21 that they leave would be faster.  There and here, us; what counts is how many workgroups the blocks of 64 rows and columns make, beside 256 compute units.
bool columns_pay(const BlockArgs &a, int64_t ld, int turns)
{
    const int C = a.C, M = a.M, cus = device_info().cus;
    const bool full = M % 64 == 0, wide = a.dtype == MADDNESS_F32;
    const int64_t blocks = (int64_t)a.chunks * a.col_blocks;
    if ((a.N & ~(int64_t)3) > (1 << 17)) {             // (they take whole runs of four rows)
        // cols_kernel: N = 341509, M = 84, C = 16 112 and 59; N = 275568, M = 200, C = 16, bytes 121 and 62; N = 432774, M = 96, C = 32 1.83 times; but N = 380782,
        // M = 256, C = 16 128 and 146, bytes N = 495291 135 and 177, N = 468621, M = 256, C = 32 206 and 242; M = 192, C = 16, binary16 1.2 to 1.6 times, where columns
        // lie on four elements 0.93
        if (C == 16 || ld % 4 != 0) return C == 64 || !full || M < (ld % 4 != 0 ? 256 : 192) || (C == 32 && !wide);
        // Four rows to a lane, which pays from some 200000 rows on.  C = 32: N = 149808, M = 32 43 and 35, N = 159528, M = 192 1.38 times, N = 191260, M = 256 0.97, N = 275892, M = 300
        // 0.94; narrow types N = 172236, M = 64 1.16, N = 199600, M = 256 1.20, N = 255872, M = 64 0.80, N = 285633, M = 192 0.76, N = 172216, M = 512 0.79; results that end
        // within a line N = 431384, M = 100, bytes 1.23 (14 turns), N = 251772, M = 300 185 and 155 (24).
        if (C == 32) return M < 512 && (a.N <= (wide ? 170000 : 200000) || (!wide && M > 32 && M % 32 != 0 && turns <= 24));
        // C = 64: N = 152220, M = 128 1.22 times, N = 267568 0.78, narrow types N = 176504 1.23, N = 228484 0.96; N = 138328, M = 64 0.98, N = 186772, M = 256 0.68
        return M > 64 && M <= 128 && a.N <= 190000;
    }
    // 16: N = 102000, M = 100 1.3 times, N = 70039, M = 892 111 and 69; N = 24222, M = 320, bytes 1.25 times, N = 20958, M = 512 19.7 and 22.3, N = 57664,
    // binary16 34 and 45; N = 104887, M = 100 1.3 times, N = 123476, M = 128 27 and 31
    if (C == 16) return !full || blocks <= 5 * cus || (M <= 128 && (!wide || 2 * blocks <= 13 * cus));
    // 32: N = 67775, M = 32 1.16 times, N = 95988, M = 128 0.84; N = 17637, M = 200 1.23, N = 49770 27.7 and 32.3; N = 15120, M = 320 1.19, N = 30591, M = 384 0.82;
    // N = 68555, M = 300 1.12 (7 turns); narrow types N = 206915, M = 128 2.1, N = 121416, M = 384 1.12, N = 8774, M = 512 21.1 and 15.6, N = 63868 52 and 63; a column or
    // less to a codebook, of which that kernel's reads meet in the caches, N = 17656, M = 192 1.23, N = 78969, M = 320 0.75
    if (C == 32 && !wide) return !full || M <= 128 || (M < 512 ? a.D > C || blocks <= 4 * cus : turns <= 4);
    if (C == 32) return !full && M > 256 ? turns <= 16 : blocks <= (M <= 128 || !full ? 5 : 3) * cus;
    // 64: N = 13785, M = 256 18.3 and 22.9 (2 turns), N = 28047, M = 64 0.85; narrow types N = 108204, M = 64 81 and 60 (4), N = 118359, M = 128 99 and 76 (8),
    // N = 14582, M = 300 34 and 31 (3), N = 15912, M = 512 34 and 42 (4); a column or less to a codebook N = 24988, M = 192, bytes 0.69, N = 88229, D = 64, M = 64, binary16 1.13,
    // N = 40555, D = 50, M = 64, bytes 0.82
    if (a.D <= C) return blocks <= (wide || M > 128 || a.D < C ? 1 : 6) * cus;
    return wide ? turns <= 1 && (M > 64 || blocks <= cus) : turns <= (M <= 128 ? 8 : 3);
}

}  // namespace

int launch_fused_blocks(const maddness_params &p, const MatrixA &A, int64_t N, int32_t M, const uint8_t *luts,
                        const float *scale, const float *offset, float *out, int64_t ldo, uint16_t *acc,
                        uint8_t *codes, bool only_if_faster, hipStream_t stream)
{
    const int es = A.elem_bytes(), C = p.C;
    if (A.col_major || C > 64 || (int64_t)p.D * es > kMaxRowBytes || 16 * (int64_t)C * M >= (1LL << 31)) return 1;
    if (left_out()) return 1;
    BlockArgs a{};
    a.A = static_cast<const unsigned char *>(A.data); a.pitch = A.ld * es; a.row_bytes = p.D * es; a.D = p.D; a.dtype = A.dtype;
    a.N = N;
    a.split_dims = p.split_dims; a.thresholds = p.thresholds;
    a.luts = luts; a.scale = scale; a.offset = offset; a.M = M; a.C = C;
    a.out = out; a.ldo = ldo; a.acc = acc; a.codes_out = codes;
    // the range of a chunk is read whole: rows without much between them
    if (a.pitch > a.row_bytes + a.row_bytes / 8 + 64) return 1;
    const int KC = kernel_codebooks(C);
    // every row begins on a 16-byte boundary, or the range of a chunk takes up to a piece more (rows of more than 4 KiB N = 372, D = 1963, M = 4, C = 48 35 and 4.9 us, N = 6846, D = 1097,
    // M = 683, C = 48 47 and 36)
    const bool whole = a.pitch % 16 == 0 && aligned_to(A.data, 16);
    const Plan plan = choose_plan(N, a.pitch, whole, M, KC);
    if (plan.rows < 1 || N / plan.rows >= (1 << 30)) return 1;
    if (!blocks_pay(a, KC, plan, only_if_faster)) return 1;

    a.tile_shift = plan.tile_shift; a.col_blocks = plan.col_blocks;
    const int tiles = 1 << plan.tile_shift, ntw = plan.tile_shift == 4 ? 2 : 1;
    a.chunk_rows = (int)plan.rows;
    a.chunks = (int)((N + plan.rows - 1) / plan.rows);
    int64_t groups = std::min<int64_t>(plan.groups, a.chunks);
    if (a.col_blocks > 1) groups = (groups + 7) / 8 * 8;
    a.row_groups = (int)groups;
    const int stage_bytes = (int)(plan.rows * a.pitch + (whole ? 0 : 16));
    const int kb = stage_bytes <= 32 * 1024 ? 32 : stage_bytes <= 64 * 1024 ? 64 : 128;
    const size_t table_lds = (size_t)KC * tiles * kTileBytes, rows_lds = (size_t)kb * 1024;
    // (the scan reads the codes of up to a turn of its wavefronts beyond the last row)
    const size_t code_lds = (size_t)((plan.rows + 15) / 16 * 16 + 16 * (kBlockWaves * ntw / tiles)) * lanes_per_row(KC);
    const size_t room = device_info().lds_per_block / (plan.shared ? 2 : 1);
    a.overlay = 256 + table_lds + rows_lds + code_lds > room ? 1 : 0;
    a.rows_at = 256;
    a.tables_at = 256 + (a.overlay ? 0 : (unsigned)rows_lds);
    a.codes_at = (unsigned)(a.overlay ? 256 + std::max(table_lds, rows_lds) : 256 + table_lds + rows_lds);
    const size_t lds = a.codes_at + code_lds;
    if (lds > room) return 1;
    const int grid = a.row_groups * a.col_blocks;
    switch (KC) {
    case 4: return launch_books<1>(a, ntw, kb, grid, lds, stream);
    case 8: return launch_books<2>(a, ntw, kb, grid, lds, stream);
    case 16: return launch_books<4>(a, ntw, kb, grid, lds, stream);
    case 24: return launch_books<6>(a, ntw, kb, grid, lds, stream);
    case 32: return launch_books<8>(a, ntw, kb, grid, lds, stream);
    case 48: return launch_books<12>(a, ntw, kb, grid, lds, stream);
    default: return launch_books<16>(a, ntw, kb, grid, lds, stream);
    }
}

// A stored by columns: 64 rows to a chunk, as many blocks of columns as leave a workgroup for every compute unit.  Instead of the
// general kernel (only_if_faster = false) whatever the rows: that one reads the split values a lane for itself and walks large tables tile by tile (us,
// there and here: N = 554, M = 1000, C = 48, binary16 349 and 9; N = 14231, M = 512, C = 48, binary16 214 and 31; N = 9407, M = 122, C = 24 21 and 7.6;
// N = 524288, M = 4, C = 48, bfloat16 621 and 172; of 484 calls of 16, 32 and 64 codebooks none was faster there); instead of the others, which take 16, 32 and 64
// codebooks, by columns_pay.
int launch_fused_blocks_cols(const maddness_params &p, const MatrixA &A, int64_t N, int32_t M, const uint8_t *luts,
                             const float *scale, const float *offset, float *out, int64_t ldo, uint16_t *acc,
                             uint8_t *codes, bool only_if_faster, hipStream_t stream)
{
    const int es = A.elem_bytes(), C = p.C;
    if (!A.col_major || C > 64 || N >= (1LL << 36) || 16 * (int64_t)C * M >= (1LL << 31)) return 1;
    if (left_out() || option(MADDNESS_OPT_COLS_RUN)) return 1;
    const int KC = kernel_codebooks(C);
    BlockArgs a{};
    a.A = static_cast<const unsigned char *>(A.data); a.pitch = A.ld * es; a.D = p.D; a.dtype = A.dtype;
    a.N = N;
    a.split_dims = p.split_dims; a.thresholds = p.thresholds;
    a.luts = luts; a.scale = scale; a.offset = offset; a.M = M; a.C = C;
    a.out = out; a.ldo = ldo; a.acc = acc; a.codes_out = codes;
    a.chunk_rows = 64;
    a.chunks = (int)((N + 63) / 64);
    const DeviceInfo &dev = device_info();
    const int all_tiles = (M + 15) / 16;
    int shift = 0;
    while (shift < 3 && (1 << shift) < all_tiles) ++shift;
    auto blocks = [&](int sh) { return (all_tiles + (1 << sh) - 1) >> sh; };
    while (shift > 0 && (int64_t)a.chunks * blocks(shift - 1) <= dev.cus) --shift;
    const int tiles = 1 << shift;
    a.tile_shift = shift; a.col_blocks = blocks(shift);
    const int lpr = lanes_per_row(KC);
    const size_t table_lds = (size_t)KC * tiles * kTileBytes, code_lds = (size_t)(64 + 16 * (kBlockWaves / tiles)) * lpr;
    a.rows_at = a.tables_at = 256;
    a.codes_at = (unsigned)(256 + table_lds);
    const size_t lds = a.codes_at + code_lds;
    if (lds > (size_t)dev.lds_per_block) return 1;
    // (three workgroups to a compute unit where they are small, else two: N = 524288, M = 3, C = 16, binary16 37 and 44 us; N = 178739, M = 128,
    // C = 32, binary16 50 and 43)
    const int per_cu = (int)std::min<size_t>(KC <= 16 ? 3 : 2, dev.lds_per_block / lds), wgs = dev.cus * per_cu;
    int64_t groups = std::max(1, wgs / a.col_blocks);
    if (groups > 8 && a.col_blocks > 1) groups = groups / 8 * 8;
    groups = std::min<int64_t>(groups, a.chunks);
    if (a.col_blocks > 1) groups = (groups + 7) / 8 * 8;
    a.row_groups = (int)groups;
    const int grid = a.row_groups * a.col_blocks;
    const int turns = (a.chunks + a.row_groups - 1) / a.row_groups;
    if (only_if_faster && (C == 16 || C == 32 || C == 64) && !columns_pay(a, A.ld, turns)) return 1;
    // Next to nothing to read and to add for many rows, half of it padding: the general kernel (N = 774266, M = 2, C = 2 16 and 34, N = 88197, M = 3, C = 1, binary16 5.0 and 6.0;
    // N = 150580, M = 6, C = 3 7.7 and 9.0, N = 625847, M = 7, C = 4 28 and 35, N = 675992, M = 1, C = 6 27 and 34; one turn N = 26413, M = 3, C = 2 5.5 and 3.7; N = 137365, M = 9, C = 2 14.1 and 8.7; N = 529582, M = 4, C = 6, bytes
    // 31 and 27).
    if (M <= 8 && (C <= 2 ? turns > 1 : turns > 3 && (C == 3 || (C <= 6 && A.dtype == MADDNESS_F32)))) return 1;
    switch (KC) {
    case 4: return launch_columns<1>(a, grid, lds, stream);
    case 8: return launch_columns<2>(a, grid, lds, stream);
    case 16: return launch_columns<4>(a, grid, lds, stream);
    case 24: return launch_columns<6>(a, grid, lds, stream);
    case 32: return launch_columns<8>(a, grid, lds, stream);
    case 48: return launch_columns<12>(a, grid, lds, stream);
    default: return launch_columns<16>(a, grid, lds, stream);
    }
}

// The aggregation by averages (fp32 rows, 16, 32, 48 or 64 codebooks): blocks of up to 64 KiB of tables, which stay in LDS.  There
// (the general kernel, and those for tables in LDS or in tiles of it) and here, us (turns): one turn N = 695, D = 512, M = 1000, C = 32 254
// and 6.8, N = 1824, D = 1024, M = 128, C = 64 80 and 6.3, N = 4096, D = 512, M = 100, C = 32 7.9 and 6.0; one block of columns N = 128647, D = 256,
// M = 107, C = 16 85 and 48 (8), N = 390133, D = 1024, M = 45, C = 64 454 and 332 (95); several N = 9845, D = 1024, M = 128, C = 64 81 and 17 (5),
// N = 119634, D = 128, M = 256, C = 16 66 and 57 (8), N = 129570, D = 256, M = 512, C = 16 139 and 152 (32), N = 172750, D = 512, M = 128, C = 64 120 and
// 171 (43); C = 32 with tables in LDS for rows_kernel N = 8192, D = 512, M = 256 9.3 and 10.2 (2), N = 50246 31 and 54 (13), N = 524288, M = 128 218
// and 272 (64), and without, where the general kernel walks the tables tile by tile and blocks read every row once for each, N = 58664, D = 256, M = 791 297 and 135 (29),
// N = 262070, M = 303 344 and 283 (52), N = 161770, M = 772 286 and 423 (79), N = 126359, D = 512, M = 656 281 and 370 (99), N = 534525, M = 984 1155 and 1958 (522); rows of 512
// bytes N = 403599, D = 128, M = 646 902 and 668 (79), N = 683104, M = 915 1674 and 1409 (167).
int launch_averaged_blocks(const maddness_params &p, const MatrixA &A, int64_t N, int32_t M, const uint8_t *luts,
                           const float *scale, const float *offset, float *out, int64_t ldo, uint16_t *acc,
                           uint8_t *codes, hipStream_t stream)
{
    const int C = p.C;
    if (!A.plain() || C > 64 || C % 16 != 0 || (int64_t)p.D * 4 > kMaxRowBytes || 16 * (int64_t)C * M >= (1LL << 31)) return 1;
    if (left_out()) return 1;
    BlockArgs a{};
    a.A = static_cast<const unsigned char *>(A.data); a.pitch = A.ld * 4; a.row_bytes = p.D * 4; a.D = p.D; a.dtype = A.dtype;
    a.N = N;
    a.split_dims = p.split_dims; a.thresholds = p.thresholds;
    a.luts = luts; a.scale = scale; a.offset = offset; a.M = M; a.C = C;
    a.out = out; a.ldo = ldo; a.acc = acc; a.codes_out = codes;
    if (a.pitch > a.row_bytes + a.row_bytes / 8 + 64) return 1;
    const bool whole = a.pitch % 16 == 0 && aligned_to(A.data, 16);
    const DeviceInfo &dev = device_info();
    int shift = 1;
    while (shift < (C <= 32 ? 3 : 2) && (16 << shift) < M) ++shift;
    a.tile_shift = shift;
    a.col_blocks = (M + (16 << shift) - 1) >> (4 + shift);
    const int64_t tables = (int64_t)256 * C << shift, codes_row = 2 * lanes_per_row(C);
    int64_t groups = std::max(1, dev.cus / a.col_blocks);
    if (groups > 8 && a.col_blocks > 1) groups = groups / 8 * 8;
    const int64_t most = std::min<int64_t>((64 * 1024 - (whole ? 0 : 16)) / a.pitch,
                                           (dev.lds_per_block - 256 - tables - 64 * 1024) / codes_row);
    if (most < 1) return 1;
    const int64_t share = std::max<int64_t>(8, (N + groups - 1) / groups), turns = (share + most - 1) / most;
    const int64_t rows = (share + turns - 1) / turns;
    if (N / rows >= (1 << 30)) return 1;
    const bool held = C == 32 && p.D <= 512 && p.D % 4 == 0 && whole && maddness::rows::tables_ok(C, M, luts, scale, offset, out, ldo, acc);
    // (to 100 turns for up to 90000 rows by four blocks of columns or more, beside which the general kernel walks most tables: N = 46431, D = 863, M = 1000 329 and 252 (81),
    // N = 34478, D = 1361, M = 793 374 and 262 (90), N = 19214, D = 1834, M = 847 365 and 141 (76), N = 82756, D = 1024, M = 531 327 and 334 (108); N = 124436, D = 512, M = 556 232 and 301 (82))
    const int64_t most_turns = a.col_blocks >= 4 && N < 90000 ? 100 : 64;
    if (turns > 1 && (held || (a.col_blocks > 1 && (C != 32 ? turns > 16 : turns > most_turns && a.row_bytes >= 1024)))) return 1;
    a.chunk_rows = (int)rows;
    a.chunks = (int)((N + rows - 1) / rows);
    groups = std::min<int64_t>(groups, a.chunks);
    if (a.col_blocks > 1) groups = (groups + 7) / 8 * 8;
    a.row_groups = (int)groups;
    const int kb = rows * a.pitch + (whole ? 0 : 16) <= 32 * 1024 ? 32 : 64;
    a.rows_at = 256;
    a.tables_at = 256 + kb * 1024;
    a.codes_at = (unsigned)(a.tables_at + tables);
    const size_t lds = a.codes_at + (size_t)(rows * codes_row);
    if (lds > (size_t)dev.lds_per_block) return 1;
    const int grid = a.row_groups * a.col_blocks;
    switch (C) {
    case 16: return launch_averaged_tiles<4>(a, kb, grid, lds, stream);
    case 32: return launch_averaged_tiles<8>(a, kb, grid, lds, stream);
    case 48: return launch_averaged_tiles<12>(a, kb, grid, lds, stream);
    default: return launch_averaged_tiles<16>(a, kb, grid, lds, stream);
    }
}

// The scan alone: 256 rows to a chunk at most, as many blocks of columns as leave a workgroup for every compute unit where rows are few.
// N = 1205, M = 300, C = 16 3.7 us (the general kernel 13.0), N = 4070 5.2 (13.5).
int launch_scan_blocks(int32_t C, int32_t M, const uint8_t *codes, int64_t N, const uint8_t *luts, const float *scale,
                       const float *offset, float *out, int64_t ldo, uint16_t *acc, hipStream_t stream)
{
    if (C > 64 || N >= (1LL << 36) || 16 * (int64_t)C * M >= (1LL << 31)) return 1;
    if (left_out()) return 1;
    const int KC = kernel_codebooks(C);
    BlockArgs a{};
    a.A = codes; a.N = N;
    a.luts = luts; a.scale = scale; a.offset = offset; a.M = M; a.C = C;
    a.out = out; a.ldo = ldo; a.acc = acc;
    const int Cb = (C + 1) / 2;
    a.unit = Cb % 8 == 0 ? 8 : Cb % 4 == 0 ? 4 : 1;
    const DeviceInfo &dev = device_info();
    const int all_tiles = (M + 15) / 16, lpr = lanes_per_row(KC);
    int shift = 0;
    while (shift < 3 && (1 << shift) < all_tiles) ++shift;
    auto blocks = [&](int sh) { return (all_tiles + (1 << sh) - 1) >> sh; };
    // (eight chunks of rows or a multiple, one to a die: with fewer the other dies have nothing to do, N = 454, M = 640, C = 64 8.1 us so, 5.5 with two tiles to a block)
    while (shift > 0 && ((N + 127) / 128 + 7) / 8 * 8 * blocks(shift - 1) <= dev.cus) --shift;
    const int tiles = 1 << shift;
    a.tile_shift = shift; a.col_blocks = blocks(shift);
    const size_t table_lds = (size_t)KC * tiles * kTileBytes;
    const int64_t most = std::min(256, kCodeUnits * kBlockThreads * a.unit / Cb);
    const size_t code_lds = (size_t)((most + 15) / 16 * 16 + 16 * (kBlockWaves / tiles)) * lpr;
    a.tables_at = a.rows_at = 256;
    a.codes_at = (unsigned)(256 + table_lds);
    const size_t lds = a.codes_at + code_lds;
    if (lds > (size_t)dev.lds_per_block) return 1;
    // (two workgroups to a compute unit where one would take several turns: N = 33000, M = 200, C = 30 13.5 and 15.6 us; beside one
    // turn they read the tables twice: N = 450, M = 200, C = 64 8.0 and 5.1; 64 codebooks N = 90821, M = 10 9.3 and 7.3)
    int64_t groups, share, turns;
    for (int per_cu = 1;; ++per_cu) {
        groups = std::max(1, dev.cus * per_cu / a.col_blocks);
        if (groups > 8 && a.col_blocks > 1) groups = groups / 8 * 8;
        share = std::max<int64_t>(16, (N + groups - 1) / groups);
        turns = (share + most - 1) / most;
        if (per_cu == 2 || turns <= (KC == 64 ? 2 : 1) || 2 * lds > (size_t)dev.lds_per_block) break;
    }
    if (!scan_blocks_pay(a, ldo, KC, turns)) return 1;
    const int64_t rows = std::min(most, ((share + turns - 1) / turns + 15) / 16 * 16);
    a.chunk_rows = (int)rows;
    a.chunks = (int)((N + rows - 1) / rows);
    groups = std::min<int64_t>(groups, a.chunks);
    if (a.col_blocks > 1) groups = (groups + 7) / 8 * 8;
    a.row_groups = (int)groups;
    const int grid = a.row_groups * a.col_blocks;
    switch (KC) {
    case 4: return launch_codes<1>(a, grid, lds, stream);
    case 8: return launch_codes<2>(a, grid, lds, stream);
    case 16: return launch_codes<4>(a, grid, lds, stream);
    case 24: return launch_codes<6>(a, grid, lds, stream);
    case 32: return launch_codes<8>(a, grid, lds, stream);
    case 48: return launch_codes<12>(a, grid, lds, stream);
    default: return launch_codes<16>(a, grid, lds, stream);
    }
}

// The codes alone, for what would else be the general kernel's, in which a lane asks for the split values of its row and pair of
// codebooks one by one.  There and here, us: by rows N = 13471, D = 240, C = 24 5.9
// and 4.6, N = 12485, D = 1728, C = 32, binary16 13.6 and 8.2, N = 762885, D = 96, C = 24, bfloat16 121 and 48, N = 344094, D = 1000, C = 15, binary16 245 and 118;
// by columns N = 26139, C = 30, bfloat16 14.2 and 6.6, N = 353958, C = 48 179 and 77, N = 1294803, C = 63, bytes 701 and 332.
int launch_encode_blocks(const maddness_params &p, const MatrixA &A, int64_t N, uint8_t *codes, hipStream_t stream)
{
    const int es = A.elem_bytes(), C = p.C;
    if (C > 64 || N >= (1LL << 36)) return 1;
    if (left_out()) return 1;
    const int KC = kernel_codebooks(C);
    BlockArgs a{};
    a.A = static_cast<const unsigned char *>(A.data); a.pitch = A.ld * es; a.row_bytes = p.D * es; a.D = p.D; a.dtype = A.dtype;
    a.N = N; a.C = C; a.col_blocks = 1;
    a.split_dims = p.split_dims; a.thresholds = p.thresholds;
    a.codes_out = codes;
    a.rows_at = a.codes_at = a.tables_at = 256;
    const DeviceInfo &dev = device_info();
    if (A.col_major) {
        // Next to no codes to a row (N = 1154410, C = 4, bfloat16 33 and 36; N = 481716, C = 8 18.6 and 20.1, N = 816156, C = 9 44 and 52; bytes N = 101212, C = 8 11.2 and 5.7),
        // nor few rows, of which a wavefront here takes several codebooks in turn (N = 5527, C = 64, bfloat16 6.4 and 8.1, N = 3980, C = 23, bytes 3.9 and 4.3; fp32 N = 6119, C = 9 2.7 and 3.2,
        // N = 8793, C = 15 4.1 and 3.7, N = 7801, C = 26 4.3 and 5.2, N = 11712, C = 24 6.1 and 4.7, N = 5491, C = 8 2.9 and 2.7, N = 6227, C = 48 7.2 and 6.8).
        const bool wide = A.dtype == MADDNESS_F32;
        if (KC == 4 || (wide && ((KC == 8 && N > (1 << 17)) || (C <= 12 && N > (1 << 18))))) return 1;
        if (N < (wide && C != 8 && KC <= 32 ? (KC <= 16 ? 8192 : 9216) : (KC == 24 ? 192 : 128) * KC)) return 1;
        // workgroups to a compute unit, with 4 and as here: N = 440208, C = 24, bytes 45.7 and 42.6; N = 353958, C = 48 88 and 77; N = 132534, C = 63 39.3
        // and 38.0; fewer for C = 15 lose (N = 302525, bytes 19.8 with 4, 22.1 with 3)
        const int64_t wgs = (int64_t)dev.cus * (KC <= 16 ? 4 : KC < 64 ? 3 : 2);
        a.chunk_rows = 64;
        a.chunks = (int)((N + 63) / 64);
        a.row_groups = (int)std::min<int64_t>(wgs, a.chunks);
        const size_t lds = 256 + 64 * (size_t)lanes_per_row(KC);
        switch (KC) {
        case 8: return launch_codes_of_columns<2>(a, lds, stream);
        case 16: return launch_codes_of_columns<4>(a, lds, stream);
        case 24: return launch_codes_of_columns<6>(a, lds, stream);
        case 32: return launch_codes_of_columns<8>(a, lds, stream);
        case 48: return launch_codes_of_columns<12>(a, lds, stream);
        default: return launch_codes_of_columns<16>(a, lds, stream);
        }
    }
    if ((int64_t)p.D * es > kMaxRowBytes || a.pitch > a.row_bytes + a.row_bytes / 8 + 64) return 1;
    const bool whole = a.pitch % 16 == 0 && aligned_to(A.data, 16);
    // Few codes: the launch here is the longer one, by a tenth (fp32 N = 70, C = 1 1.9 and 2.6, N = 2650, C = 14 2.7 and 3.5, N = 4279, C = 28 3.8 and 3.9, N = 7829, C = 28 4.1 and 4.1,
    // N = 14754, C = 24 6.4 and 4.6; the other types, which take longer there, from where the rows here make two workgroups to a compute unit: bytes N = 1887, C = 20 3.5 and 2.9,
    // N = 4702, C = 3 3.2 and 3.7, N = 14523, C = 6 3.5 and 3.7, N = 7210, C = 19 4.1 and 3.7), but for powers of two, where there every lane has a pair of codebooks and workgroups are
    // fewest (N = 240, D = 64, C = 8 3.3 and 2.6, N = 72, C = 32 3.0 and 2.7; from there on N = 4796, C = 8 2.8 and 3.6, binary16 N = 2173, C = 16 3.7 and 3.4).
    // (fp32 N = 16500 to 24500, C = 8 5.3 and 4.0, C = 16, 32 and 64 1.06 times, below 128 Ki codes 0.83)
    const bool few = N <= 8 * dev.cus, power = C >= 8 && (C & (C - 1)) == 0;
    if (A.dtype == MADDNESS_F32 ? N * C < ((power ? 128 : 192) << 10) && !(few && power) : N * C < (88 << 10) && !few && !power) return 1;
    // (whole rows are read here, 64 bytes for each split value there: N = 20680, D = 512, C = 4, binary16 5.8 and 6.1)
    const int64_t most = (32 * 1024 - (whole ? 0 : 16)) / a.pitch;
    if (most < 1 || a.row_bytes > 192 * C) return 1;
    // two workgroups to a compute unit where that makes one chunk to each (N = 27487, D = 120, C = 30 4.6 us, 5.7 with four), else four (N = 240545, D = 192,
    // C = 48 42.8, 46.3 with two, 49.1 with two and chunks of 64 KiB)
    int64_t wgs = 2 * (int64_t)dev.cus;
    if ((N + wgs - 1) / wgs > most) wgs *= 2;
    const int64_t share = std::max<int64_t>(8, (N + wgs - 1) / wgs), turns = (share + most - 1) / most, rows = (share + turns - 1) / turns;
    if (N / rows >= (1 << 30)) return 1;
    a.chunk_rows = (int)rows;
    a.chunks = (int)((N + rows - 1) / rows);
    a.row_groups = (int)std::min<int64_t>(wgs, a.chunks);
    const size_t lds = 256 + 32 * 1024;
    switch (KC) {
    case 4: return launch_codes_of_rows<1>(a, lds, stream);
    case 8: return launch_codes_of_rows<2>(a, lds, stream);
    case 16: return launch_codes_of_rows<4>(a, lds, stream);
    case 24:
    case 32: return launch_codes_of_rows<8>(a, lds, stream);
    default: return launch_codes_of_rows<16>(a, lds, stream);
    }
}

}  // namespace maddness
