// Fused encode + exact scan with the scan on the matrix cores, in phases:
//
// A workgroup of 8 wavefronts (two per SIMD, 256 registers each; one workgroup
// per CU) takes a block of rows through
//   E   every wavefront encodes its share of the rows and leaves the packed codes
//       of the block in LDS (C / 2 bytes per row).  Row-major A (fp32 or a narrow
//       type): as the row kernels do - register prefetch, staging in
//       wavefront-private LDS, Algorithm 1 with the tree in registers.  A stored
//       by columns: as the column kernels do - a lane owns four consecutive rows,
//       only the 4 C split columns are read (cols_common.h);
//   S   wavefront w holds the tables of output columns [SPAN w, SPAN (w + 1)) in
//       registers and goes through all rows of the block, 16 at a time: codes from
//       LDS, one-hot operands, int8 MFMA, dequantise, store (mfma_common.h).  If M
//       exceeds 8 SPAN columns the phase is repeated with the next 8 SPAN columns;
//       if it has at most 4 SPAN, several wavefronts hold the same columns and
//       share out the rows.
//       The tables are re-read from L2 at the start of every S phase, by the whole
//       workgroup through LDS, which leaves the registers to E meanwhile.
// E is bound by HBM reads, S by HBM writes; they do not overlap within a
// workgroup, and the larger a region, the longer the chip as a whole only reads or
// only writes, which HBM serves faster than a mixture (N = 2^20, D = 512, M = 256,
// C = 32: 0.51 ms with one region, 0.56 ms with four, 0.53 ms for the kernel in which
// every wavefront reads, gathers and writes).  Measured alternatives that overlapped
// the phases within a CU were slower on the stress workload (N = 2^22, D = 1024,
// M = 512, C = 64; this kernel: 4.8 ms): two workgroups of 4 wavefronts per CU
// (6.0 ms; 7.3 ms when started half a period apart), and 4 encoding + 4 scanning
// wavefronts with double-buffered codes (6.2 ms, whatever the encoders' prefetch
// depth; only the by-columns input gained, 0.295 against 0.324 ms at N = 2^20,
// M = 256).  Used for many rows of any type by up to 64 codebooks, for any number of them
// where the tables are larger than the other kernels take at once (and for many shapes whose
// tables these still hold: few_rows_in_lds), of the few rows those that the kernel by blocks of rows and columns leaves, for A stored by columns (few_columns_in_lds); and,
// as its E phase alone, to encode fp32 rows.
#include <algorithm>

#include "cols_common.h"
#include "mfma_common.h"

namespace maddness {
namespace {

using namespace rows;
using namespace mfma;

constexpr int kWaves = 8;

// one workgroup per compute unit, or fewer when MADDNESS_OPT_MAX_WORKGROUPS says so (testing aid)
int max_workgroups()
{
    const int cus = device_info().cus, cap = option(MADDNESS_OPT_MAX_WORKGROUPS);
    return cap >= 1 && cap < cus ? cap : cus;
}

// Most rows per wavefront and region.  As many as LDS holds codes for is best: with one
// region the whole chip first only reads, then only writes (N = 2^21, D = 512, M = 256,
// C = 32: 1.02 ms with regions of 2^21 rows, 1.10 ms with 2^20).
#ifndef MADDNESS_PHASED_MAX_ROWS
#define MADDNESS_PHASED_MAX_ROWS 1024
#endif

// A stored by columns: up to this many rows are encoded a row to a lane (EncodeMode kByColumnsFew).  Four rows to a lane
// read longer pieces of a column, but a workgroup takes 2048 rows then: C = 32, M = 256, binary16, N = 65536 40 us a
// row to a lane and 98 four, N = 2^18 132 and 104.
constexpr int64_t kColsFewRows = 1 << 17;

// the value of x, as far as the compiler knows a new one each time
__device__ __forceinline__ int opaque(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}
enum EncodeMode { kRowMajor = 0, kByColumns = 1, kByColumnsFew = 2 };

// Bytes at the start of LDS that the phases use in turn: E stages RPI rows of DV KiB per wavefront there
// (row-major A); S first passes the tables of its columns through it, then keeps the one-hot table there (256 bytes)
// and, when it writes whole rows, two tiles of one step's results each (16 rows, or 32 with NT = 2, of 8 blocks of
// 16 NT columns + 4 floats of padding).
constexpr int tile_bytes(int NT) { return (NT == 2 ? 32 : 16) * (kWaves * 16 * NT + 4) * 4; }
constexpr int shared_bytes(int emode, int RPI, int DV, int NT, bool scan, bool gather)
{
    const int stage = emode == kRowMajor ? kWaves * RPI * DV * 1024 : 256;
    const int tables = scan ? kWaves * kTableStage : 256;
    const int tiles = gather ? 256 + 2 * tile_bytes(NT) : 256;
    return std::max(stage, std::max(tables, tiles));
}

// DV: 16-byte pieces per lane and row (row-major); unused for columns.
// SCAN = false: the E phase only (the codes go to a.codes_out), a kernel of its own name.
// GATHER = true (row-major A, more than 4 blocks of columns): the S phase collects the
// fp32 results of a step in LDS and writes whole rows, for outputs whose rows do not start
// on 128-byte lines.
// PAD = true: a.codebooks < C codebooks exist (a multiple of 8); the kernel runs as for C with
// the others' codes and table entries zero, and writes rows of a.codebooks / 2 bytes to a.codes_out.
// ODD = true (row-major A, with PAD): any shape the tile sizes cover - rows of A that start on any
// element and end anywhere, any number of codebooks up to C, any M, any pitch
// and alignment of the outputs.  The E phase reads the aligned 16-byte pieces that cover a row,
// the tables are read from any byte on, and the S phase writes through LDS (GATHER) - rows without padding
// between them as ranges of floats in aligned 16-byte pieces, other rows each as a range of its own
// (store_dense_rows) - or, for one or two blocks of columns, with 4-byte stores straight from the registers,
// the wavefronts sharing out the rows (gathered, such narrow outputs would leave the matrix work to one or
// two of the eight wavefronts: N = 2^20, D = 512, M = 10, C = 16 takes 0.37 instead of 0.52 ms).
template <int C, int DV, int NT, int EMODE, int DT, bool SCAN = true, bool GATHER = false, bool PAD = false, bool ODD = false>
__global__ __launch_bounds__(kWaves * 64) void fused_mfma_kernel(const RowsArgs a, const int rw)
{
    static_assert(!ODD || (PAD && EMODE == kRowMajor), "ODD: rows, padding codebooks");
    constexpr int KG = C / 4;
    constexpr int RPI = 64 / C;
    constexpr int CB = C / 2;
    constexpr int CW = C / 8;
    constexpr int SPAN = 16 * NT;
    // groups of rows a wavefront of the E phase keeps in flight: one for fp32 (more is slower there: 0.335
    // against 0.310 ms per 2^20 rows of 2 KiB), more for narrow types, whose rows are few bytes each
#ifndef MADDNESS_NARROW_PREFETCH
#define MADDNESS_NARROW_PREFETCH 2
#endif
    constexpr int E_PF = DT == kF32 ? 1 : (DT == kU8 ? 2 * MADDNESS_NARROW_PREFETCH : MADDNESS_NARROW_PREFETCH);
    // row-major: staging of RPI rows per wavefront; by columns: room for the one-hot table only
    constexpr int STAGE_BYTES = shared_bytes(EMODE, RPI, DV, NT, SCAN, GATHER);
    typedef unsigned cvec __attribute__((ext_vector_type(CW)));

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    v4i *one_hot = reinterpret_cast<v4i *>(smem);                   // 16 entries of 16 bytes, valid during S
    unsigned char *codes_l = smem + STAGE_BYTES;                   // [kWaves * rw][CB]

    // S: the wavefronts share out blocks of SPAN output columns; when M has at most 4
    // blocks, `share` wavefronts (a power of two) take the same block and every share-th
    // step of the rows each
    const int col_blocks = (a.M + SPAN - 1) / SPAN;
    int share = 1;
    // (with 3 or 4 blocks only beside rows of more than 2 KiB: N = 2^20, C = 32, M = 256 takes
    // 0.510 ms without and 0.516 ms with sharing at D = 512, 0.863 and 0.822 ms at D = 1024)
    // (col_blocks = 0: encode only, nothing to share)
    if (col_blocks > 0 && (col_blocks <= 2 || (col_blocks <= 4 && EMODE == kRowMajor && a.D * elem_size(DT) > 2048)))
        while (share < kWaves && 2 * share * col_blocks <= kWaves) share *= 2;
    const ScanOut o{a.out, a.ldo, a.acc, a.M};

    v4i B[NT][KG];
    float sc[NT], of[NT];
    int col = 0, j = 0, g = 0, lane_in_s = 0;
    bool col_on = false;
    // the tables of the pass whose first block of columns is block0, `blocks` of them, into the registers of the
    // wavefronts; this one has block0 + my_block
    auto take_columns = [&](int block0, int blocks, int my_block) INLINE_LAMBDA {
        col = (block0 + my_block) * SPAN + NT * j;
        col_on = col < a.M;
        const int tid_s = 64 * wave + lane_in_s;
        __syncthreads();      // (the staging area: E, or the pass before, is done with it)
        load_tables<KG, NT, kWaves * 64, PAD>(B, a.luts, a.M, block0 * SPAN, blocks * SPAN, my_block * SPAN, g, j, smem, tid_s,
                                              a.codebooks);
        __syncthreads();
        fill_one_hot_table(one_hot, tid_s);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const bool on = ODD ? col + t < a.M : col_on;    // (else M is a multiple of NT)
            sc[t] = on ? a.scale[col + t] : 0.f;
            of[t] = on ? a.offset[col + t] : 0.f;
        }
    };
    // S for `groups` groups of 16 local rows; row_of(l): matrix row of local row l.
    // `turns` wavefronts hold the same columns, this one takes steps turn, turn + turns, ...
    // (a step: one group, or two for C = 64); the caller passes constants where it can.
    auto scan_rows = [&](int groups, auto row_of, int blocks_per_pass, int my_block, int turns, int turn) INLINE_LAMBDA {
        auto one_group = [&](int rg) INLINE_LAMBDA {
            const cvec cw = *reinterpret_cast<const cvec *>(codes_l + (size_t)(rg * 16 + j) * CB);
            v4i acc[NT];
            scan16<KG, NT>(cw, B, g, one_hot, acc);
            if (col_on) {
                if constexpr (ODD) store16_any<NT>(o, acc, [&](int k) INLINE_LAMBDA { return row_of(16 * rg + k); }, a.N, g, col, sc, of);
                else store16<NT>(o, acc, [&](int k) INLINE_LAMBDA { return row_of(16 * rg + k); }, a.N, g, col, sc, of);
            }
        };
        for (int block0 = 0; block0 < col_blocks; block0 += blocks_per_pass) {
            take_columns(block0, blocks_per_pass, my_block);   // re-read every time: the registers are free for E meanwhile
            if (block0 + my_block >= col_blocks) continue;
            if constexpr (NT == 2) {
                // two groups per step: four independent accumulation chains for the matrix pipe
#pragma unroll 1
                for (int rg = 2 * turn; rg + 2 <= groups; rg += 2 * turns) {
                    const cvec cw0 = *reinterpret_cast<const cvec *>(codes_l + (size_t)(rg * 16 + j) * CB);
                    const cvec cw1 = *reinterpret_cast<const cvec *>(codes_l + (size_t)(rg * 16 + 16 + j) * CB);
                    v4i acc0[NT], acc1[NT];
                    scan16x2<KG, NT>(cw0, cw1, B, g, one_hot, acc0, acc1);
                    if (col_on) {
                        if constexpr (ODD) {
                            store16_any<NT>(o, acc0, [&](int k) INLINE_LAMBDA { return row_of(16 * rg + k); }, a.N, g, col, sc, of);
                            store16_any<NT>(o, acc1, [&](int k) INLINE_LAMBDA { return row_of(16 * rg + 16 + k); }, a.N, g, col, sc, of);
                        } else {
                            store16<NT>(o, acc0, [&](int k) INLINE_LAMBDA { return row_of(16 * rg + k); }, a.N, g, col, sc, of);
                            store16<NT>(o, acc1, [&](int k) INLINE_LAMBDA { return row_of(16 * rg + 16 + k); }, a.N, g, col, sc, of);
                        }
                    }
                }
                // an odd last group goes to the wavefront whose turn it would be
                if ((groups & 1) && (groups >> 1) % turns == turn) one_group(groups - 1);
            } else {
#pragma unroll 1
                for (int rg = turn; rg < groups; rg += turns) one_group(rg);
            }
        }
    };
    // S with the results of a step (16 rows, or 32 for C = 64, times the up to 8 SPAN columns
    // of a pass) collected in LDS and written out row by row: a wavefront's store then covers
    // 1 KiB of one row instead of 256 (128) bytes of four rows, so that few stores end inside
    // a 128-byte line.  Every wavefront takes every step of every pass (one barrier per step); with at
    // most 4 blocks of columns the four wavefronts without columns do the writing.
    constexpr int GPS = NT == 2 ? 2 : 1;                 // groups of 16 rows per step
    constexpr int TILE_LD = kWaves * SPAN + 4;           // floats per row of the tile (4 of padding)
    auto scan_rows_gathered = [&](int groups, auto row_of) INLINE_LAMBDA {
        typedef float piece __attribute__((ext_vector_type(NT)));
        // two tiles behind the one-hot table, used in turn: a step's results are written out while the
        // next step is computed, with one barrier per step
        float *tiles = reinterpret_cast<float *>(smem + 256);
        constexpr int TILE_FLOATS = tile_bytes(NT) / 4;
        const ScanOut acc_only{nullptr, 0, a.acc, a.M};
        const int n_passes = (col_blocks + kWaves - 1) / kWaves;
        const int n_steps = (groups + GPS - 1) / GPS;
        // rows without padding between them and all columns in one pass: the rows of a unit are one range of floats
        const bool dense = ODD && a.out && a.ldo == a.M && n_passes == 1;
        const float inv_M = 1.0f / (float)a.M;
        // at most 4 blocks of columns: wavefronts 0 - 3 compute, wavefronts 4 - 7 write; else all do both
        const int first_writer = col_blocks <= kWaves / 2 ? kWaves / 2 : 0;
        const int n_writers = kWaves - first_writer;
        int it = 0;
        for (int pass = 0; pass < n_passes; ++pass) {
            const bool active = pass * kWaves + wave < col_blocks;
            take_columns(pass * kWaves, kWaves, wave);
            const int col0 = pass * kWaves * SPAN;
            const int n_cols = a.M - col0 < kWaves * SPAN ? a.M - col0 : kWaves * SPAN;
#pragma unroll 1
            for (int step = 0; step < n_steps; ++step, ++it) {
                float *tile = tiles + (it & 1) * TILE_FLOATS;
                const int rg = GPS * step;
                if (active) {
                    v4i acc[GPS][NT];
                    const cvec cw0 = *reinterpret_cast<const cvec *>(codes_l + (size_t)(rg * 16 + j) * CB);
                    if constexpr (GPS == 2) {
                        if (rg + 1 < groups) {
                            const cvec cw1 = *reinterpret_cast<const cvec *>(codes_l + (size_t)(rg * 16 + 16 + j) * CB);
                            scan16x2<KG, NT>(cw0, cw1, B, g, one_hot, acc[0], acc[1]);
                        } else {
                            scan16<KG, NT>(cw0, B, g, one_hot, acc[0]);
#pragma unroll
                            for (int t = 0; t < NT; ++t) acc[1][t] = acc[0][t];   // rows that do not exist: never written out
                        }
                    } else {
                        scan16<KG, NT>(cw0, B, g, one_hot, acc[0]);
                    }
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
                            if (a.acc && rg + q < groups) {
                                if constexpr (ODD) {
                                    // rows of acc start anywhere: one 16-bit store per sum
#pragma unroll
                                    for (int r = 0; r < 4; ++r) {
                                        const int64_t row = row_of(16 * (rg + q) + 4 * g + r);
#pragma unroll
                                        for (int t = 0; t < NT; ++t)
                                            if (row < a.N && col + t < a.M) a.acc[row * a.M + col + t] = (uint16_t)acc[q][t][r];
                                    }
                                } else {
                                    store16<NT>(acc_only, acc[q], [&](int k) INLINE_LAMBDA { return row_of(16 * (rg + q) + k); }, a.N, g,
                                                col, sc, of);
                                }
                            }
                        }
                    }
                }
                // (the tile written two steps ago was read before the barrier of the step between)
                __syncthreads();
                if (wave < first_writer) continue;
                const int rows_here = 16 * (groups - rg < GPS ? groups - rg : GPS);
                const int pieces = n_cols / NT;
                if (ODD && dense) {
                    // whole units of 8 consecutive rows = one range of 8 M floats each
                    for (int u = 0; 8 * u < rows_here; ++u) {
                        const int64_t first = row_of(16 * rg + 8 * u);
                        const int64_t left = a.N - first;
                        if (left > 0)
                            store_dense_rows(a.out + first * a.M, left < 8 ? (int)left : 8, a.M, inv_M, tile, TILE_LD, 8 * u,
                                             tid - 64 * first_writer, 64 * n_writers);
                    }
                    continue;
                }
                // row r of the step goes out through one wavefront, a piece of NT columns per lane
                for (int r = wave - first_writer; r < rows_here; r += n_writers) {
                    const int64_t row = row_of(16 * rg + r);
                    if (row >= a.N) continue;
                    float *dst = a.out + row * a.ldo + col0;
                    if constexpr (ODD) {
                        if (!a.out) continue;
                        // a row (its columns of this pass) as a range of its own (N = 2^20, D = 1000, M = 500,
                        // C = 50: 1.64 against 1.82 ms with 4-byte stores)
                        store_dense_rows<true>(dst, 1, n_cols, 0.f, tile, TILE_LD, r, lane_in_s, 64);
                    } else {
                        for (int c = lane_in_s; c < pieces; c += 64)
                            __builtin_nontemporal_store(*reinterpret_cast<const piece *>(tile + r * TILE_LD + NT * c),
                                                        reinterpret_cast<piece *>(dst + NT * c));
                    }
                }
            }
        }
    };
    auto scan_block = [&](int groups, auto row_of) INLINE_LAMBDA {
        // everything S derives from the lane number is derived here, each time: hoisted out
        // of the loop over the regions it would occupy registers during E, and what E keeps
        // in a spilled register it reloads in its inner loop, behind the prefetched rows
        const int lane_s = opaque(lane);
        lane_in_s = lane_s;
        j = lane_s & 15;
        g = lane_s >> 4;
        if constexpr (GATHER) {
            scan_rows_gathered(groups, row_of);
        } else if (share == 1) {
            scan_rows(groups, row_of, kWaves, wave, 1, 0);
        } else {
            const int blocks_per_pass = kWaves / share;
            scan_rows(groups, row_of, blocks_per_pass, wave % blocks_per_pass, share, wave / blocks_per_pass);
        }
    };

    const int64_t G = gridDim.x;
    if constexpr (EMODE == kRowMajor) {
        // Rows are dealt out in units of 8 consecutive rows (one per wavefront), round-robin
        // over the workgroups: in a region of 8 rw gridDim rows, unit u belongs to workgroup
        // u % gridDim and is its local unit u / gridDim.  At any moment the chip as a whole
        // reads one moving window of A (a few DRAM pages) instead of one stream per
        // wavefront, and a last, partly filled region is shared out evenly.
        unsigned char *stage = smem + wave * (RPI * DV * 1024);
        const int64_t region_rows = 8 * (int64_t)rw * G;
        for (int64_t region0 = 0; region0 < a.N; region0 += region_rows) {
            // ---- E: local row 8 k + wave is matrix row region0 + 8 (k G + block) + wave ----
            // (the tree is re-read each time: its 19 registers are better used by S)
            // (and E's own lane-derived values are derived anew, so that S need not keep them)
            const int lane_e = opaque(lane);
            Tree tr;
            {
                int c = lane_e & (C - 1);
                if constexpr (PAD) c = c < a.codebooks ? c : 0;   // a padding lane: any tree, its code is dropped
                load_tree(tr, a.split_dims + 4 * c, a.thresholds + 16 * c, a.D);
            }
            encode_rows_to_lds<C, DV, DT, false, PAD, ODD, E_PF>(a, tr, stage, codes_l + wave * CB, region0 + 8 * (int64_t)blockIdx.x + wave,
                                          rw, lane_e, 8 * G, 8);
            __syncthreads();
            const int64_t units_left = (a.N - region0 + 7) / 8 - (int64_t)blockIdx.x;   // units of this region from ours on
            const int64_t my_units = units_left <= 0 ? 0 : (units_left + G - 1) / G;
            const int units = (int)(my_units < rw ? my_units : rw);
            auto row_of = [&](int l) INLINE_LAMBDA { return region0 + 8 * ((int64_t)(l >> 3) * G + blockIdx.x) + (l & 7); };
            if (ODD && a.codes_out) {
                // rows of (a.codebooks + 1) / 2 bytes that start anywhere: a byte per thread and step
                const int bytes = (a.codebooks + 1) / 2;
                for (int u = tid; u < 8 * units * bytes; u += kWaves * 64) {
                    const int l = u / bytes, b = u - l * bytes;
                    const int64_t row = row_of(l);
                    if (row < a.N) a.codes_out[row * bytes + b] = codes_l[(size_t)l * CB + b];
                }
            } else if (PAD && a.codes_out) {
                // rows of a.codebooks / 2 bytes, a 32-bit word (8 codebooks) per thread and step
                const int words = a.codebooks / 8;
                for (int u = tid; u < 8 * units * words; u += kWaves * 64) {
                    const int l = u / words, w = u - l * words;
                    const int64_t row = row_of(l);
                    if (row < a.N)
                        *reinterpret_cast<uint32_t *>(a.codes_out + row * (a.codebooks / 2) + 4 * w) =
                            *reinterpret_cast<const uint32_t *>(codes_l + (size_t)l * CB + 4 * w);
                }
            } else if (a.codes_out) {
                // The codes of the region's rows, up to 16 bytes per thread and step.  (Stored row by
                // row in the encoder's loop they cost it a tenth of its rate: N = 2^22,
                // D = 1024, C = 64 encodes in 3.07 ms that way.)
                constexpr int PIECE = CB < 16 ? CB : 16;     // C = 16: a row's 8 bytes
                constexpr int PER_ROW = CB / PIECE;
                typedef unsigned piece_t __attribute__((ext_vector_type(PIECE / 4)));
                for (int u = tid; u < 8 * units * PER_ROW; u += kWaves * 64) {
                    const int64_t row = row_of(u / PER_ROW);
                    if (row < a.N)
                        *reinterpret_cast<piece_t *>(a.codes_out + row * CB + PIECE * (u % PER_ROW)) =
                            *reinterpret_cast<const piece_t *>(codes_l + (size_t)u * PIECE);
                }
            }
            // ---- S ----
            if constexpr (SCAN) scan_block((units + 1) / 2, row_of);   // 16 local rows = 2 units
            __syncthreads();   // the codes area is overwritten by the next region's E
        }
    } else {
        // A workgroup takes blocks of 8 rw consecutive rows; kByColumns: rw a multiple of 256, wavefront
        // w the rows [w rw, (w + 1) rw) of the block in groups of 256, N a multiple of 4.
        const int64_t block_rows = 8 * (int64_t)rw;
        for (int64_t R0 = blockIdx.x * block_rows; R0 < a.N; R0 += G * block_rows) {
            // ---- E ----
            if constexpr (EMODE == kByColumnsFew) {
                // Few rows: the wavefronts share out the codebooks as well, eight (a word of codes) of 64 rows to one,
                // a row to a lane, all 32 loads of a lane on their way at once.  (In runs of four rows, two codebooks
                // at a time, a wavefront takes 256 rows in C / 2 turns of one memory latency each: N = 65536 keeps 32
                // compute units busy, for 98 us with C = 32 and M = 256 and 234 us with C = 64 and M = 512.)
                constexpr int TOGETHER = kWaves / CW;                  // wavefront groups of 64 rows
                const int q = wave % CW;
                const auto split_dims = cols::as_constant(a.split_dims);
                const auto thresholds = cols::as_constant(a.thresholds);
                const int64_t block_end = block_rows < a.N - R0 ? block_rows : a.N - R0;
                for (int local = 64 * (wave / CW); local < block_end; local += 64 * TOGETHER) {
                    const int64_t row = R0 + local + lane, from = row < a.N ? row : a.N - 1;
                    float x[8][4];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int col_t = min(max(split_dims[4 * (8 * q + u) + t], 0), a.D - 1);
                            x[u][t] = widen_at<DT>(a.A, (int64_t)col_t * a.lda + from);
                        }
                    unsigned word = 0;
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        Tree tr;
#pragma unroll
                        for (int i = 0; i < 15; ++i) tr.t[i] = thresholds[16 * (8 * q + u) + i];
                        word |= hash_regs(tr, x[u][0], x[u][1], x[u][2], x[u][3]) << (4 * u);
                    }
                    *reinterpret_cast<uint32_t *>(codes_l + (size_t)(local + lane) * CB + 4 * q) = word;
                    if (a.codes_out && row < a.N) *reinterpret_cast<uint32_t *>(a.codes_out + row * CB + 4 * q) = word;
                }
            } else {
                cols::ColsEncoder<C, DT, 2, 4> enc(a);
                for (int grp = 0; grp < rw / 256; ++grp) {
                    const int local = wave * rw + grp * 256;
                    if (R0 + local >= a.N) break;   // the same for the whole wavefront
                    enc.encode_group(R0 + local, lane);
                    enc.store_codes(a.codes_out);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        cvec v;
#pragma unroll
                        for (int q = 0; q < CW; ++q) v[q] = enc.cwn[r][q];
                        *reinterpret_cast<cvec *>(codes_l + (size_t)(local + 4 * lane + r) * CB) = v;
                    }
                }
            }
            // ---- S ----
            const int64_t left = a.N - R0;
            const int groups = (int)(((left < block_rows ? left : block_rows) + 15) >> 4);
            scan_block(groups, [&](int l) INLINE_LAMBDA { return R0 + l; });
            __syncthreads();   // the codes area is overwritten by the next block's E
        }
    }
}

template <int C, int DV, int NT, int DT, bool SCAN = true, bool GATHER = false, bool PAD = false, bool ODD = false>
int launch_rows(const RowsArgs &a, hipStream_t stream)
{
    constexpr int RPI = 64 / C;
    const DeviceInfo &dev = device_info();
    // (the staging area of E; with GATHER, S puts its two tiles of results there)
    constexpr int stage_bytes = shared_bytes(kRowMajor, RPI, DV, NT, SCAN, GATHER);
    // rows per wavefront and region: as many as LDS holds codes for (the tables are re-read
    // once per region and pass)
    int rw = (dev.lds_per_block - stage_bytes) / (kWaves * (C / 2));
    if (rw > MADDNESS_PHASED_MAX_ROWS) rw = MADDNESS_PHASED_MAX_ROWS;
    // MADDNESS_OPT_PHASED_ROWS lowers that further (testing aid: several regions and a ragged
    // last one with few rows)
    if (const int v = option(MADDNESS_OPT_PHASED_ROWS); v >= 2 && v < rw) rw = v;
    // whole steps of the encoder (RPI rows) and whole groups of 16 rows for the scan (2 units)
    constexpr int STEP = RPI > 2 ? RPI : 2;
    rw = rw / STEP * STEP;
    if (rw < STEP) return 1;
    // few rows: one region, no more rows per wavefront than it takes
    const int64_t need = (a.N + 8 * (int64_t)dev.cus - 1) / (8 * (int64_t)dev.cus);
    if (need < rw) rw = (int)((need + STEP - 1) / STEP * STEP);
    const size_t lds = (size_t)stage_bytes + (size_t)kWaves * rw * (C / 2);
    if (int rc = allow_full_lds<fused_mfma_kernel<C, DV, NT, kRowMajor, DT, SCAN, GATHER, PAD, ODD>>(); rc != MADDNESS_OK) return rc;
    const int64_t units = (a.N + 7) / 8;
    const int grid = (int)(units < max_workgroups() ? units : max_workgroups());
    note_kernel("fused_mfma_kernel, A by rows", __PRETTY_FUNCTION__);
    hipLaunchKernelGGL((fused_mfma_kernel<C, DV, NT, kRowMajor, DT, SCAN, GATHER, PAD, ODD>), dim3(grid), dim3(kWaves * 64), lds, stream, a, rw);
    return check_hip(hipGetLastError(), "launch fused_mfma_kernel");
}

template <int C, int NT, int DT>
int launch_cols(const RowsArgs &a, hipStream_t stream)
{
    const DeviceInfo &dev = device_info();
    // rows per wavefront and block: a multiple of 256; as few blocks per workgroup as LDS
    // allows, all of the same size
    int rw_max = (dev.lds_per_block - shared_bytes(kByColumns, 1, 1, NT, true, false)) / (kWaves * (C / 2)) / 256 * 256;
    // MADDNESS_OPT_PHASED_ROWS lowers that (testing aid: several blocks per workgroup with few rows)
    if (const int v = option(MADDNESS_OPT_PHASED_ROWS); v >= 2 && (v + 255) / 256 * 256 < rw_max) rw_max = (v + 255) / 256 * 256;
    if (rw_max < 256) return 1;
    const int wgs = max_workgroups();
    constexpr int stage_bytes = shared_bytes(kByColumns, 1, 1, NT, true, false);
    const int64_t per_wave = (a.N + (int64_t)kWaves * wgs - 1) / ((int64_t)kWaves * wgs);   // rows per wavefront in all
    const int64_t turns = (per_wave + rw_max - 1) / rw_max;
    int rw = (int)(((per_wave + turns - 1) / turns + 255) / 256 * 256);
    if (rw > rw_max) rw = rw_max;
    const size_t lds = stage_bytes + (size_t)kWaves * rw * (C / 2);
    if (int rc = allow_full_lds<fused_mfma_kernel<C, 1, NT, kByColumns, DT>>(); rc != MADDNESS_OK) return rc;
    const int64_t blocks = (a.N + (int64_t)kWaves * rw - 1) / ((int64_t)kWaves * rw);
    const int grid = (int)(blocks < wgs ? blocks : wgs);
    note_kernel("fused_mfma_kernel, A by columns", __PRETTY_FUNCTION__);
    hipLaunchKernelGGL((fused_mfma_kernel<C, 1, NT, kByColumns, DT>), dim3(grid), dim3(kWaves * 64), lds, stream, a, rw);
    return check_hip(hipGetLastError(), "launch fused_mfma_kernel");
}

// A stored by columns, few rows: any number of them, any stride.
template <int C, int NT, int DT>
int launch_cols_few(const RowsArgs &a, hipStream_t stream)
{
    const DeviceInfo &dev = device_info();
    constexpr int stage_bytes = shared_bytes(kByColumnsFew, 1, 1, NT, true, false);
    constexpr int STEP = 64 * kWaves / (C / 8);      // rows that the workgroup encodes at a time
    // an even share of the rows for every workgroup, in as many turns as LDS takes codes for
    const int cap = (dev.lds_per_block - stage_bytes) / (C / 2) / STEP * STEP, wgs = max_workgroups();
    int64_t rows = (a.N + wgs - 1) / wgs;
    if (rows > cap) rows = (rows + (rows + cap - 1) / cap - 1) / ((rows + cap - 1) / cap);
    // MADDNESS_OPT_PHASED_ROWS lowers that (testing aid: several blocks per workgroup with few rows)
    if (const int v = option(MADDNESS_OPT_PHASED_ROWS); v >= 2 && kWaves * (int64_t)v < rows) rows = kWaves * v;
    rows = (rows + STEP - 1) / STEP * STEP;
    const size_t lds = stage_bytes + (size_t)rows * (C / 2);
    if (int rc = allow_full_lds<fused_mfma_kernel<C, 1, NT, kByColumnsFew, DT>>(); rc != MADDNESS_OK) return rc;
    const int64_t blocks = (a.N + rows - 1) / rows;
    note_kernel("fused_mfma_kernel, A by columns, few rows", __PRETTY_FUNCTION__);
    hipLaunchKernelGGL((fused_mfma_kernel<C, 1, NT, kByColumnsFew, DT>), dim3((unsigned)(blocks < wgs ? blocks : wgs)), dim3(kWaves * 64),
                       lds, stream, a, (int)(rows / kWaves));
    return check_hip(hipGetLastError(), "launch fused_mfma_kernel");
}

template <int C, int NT>
int launch_cols_few_typed(const RowsArgs &a, int dtype, hipStream_t stream)
{
    switch (dtype) {
    case MADDNESS_F32: return launch_cols_few<C, NT, kF32>(a, stream);
    case MADDNESS_F16: return launch_cols_few<C, NT, kF16>(a, stream);
    case MADDNESS_BF16: return launch_cols_few<C, NT, kBF16>(a, stream);
    default: return launch_cols_few<C, NT, kU8>(a, stream);
    }
}

template <int C, int DV, int NT>
int launch_rows_typed(const RowsArgs &a, int dtype, hipStream_t stream)
{
    switch (dtype) {
    case MADDNESS_F16: return launch_rows<C, DV, NT, kF16>(a, stream);
    case MADDNESS_BF16: return launch_rows<C, DV, NT, kBF16>(a, stream);
    default: return launch_rows<C, DV, NT, kU8>(a, stream);
    }
}

// fp32 row-major A of any shape the tiles cover (up to 64 codebooks, rows of up to 8 KiB; up to 16
// codebooks: 2 KiB, up to 32: 4 KiB), any M, any pitch and alignment: the ODD form of the kernel.
// Not for short rows to encode: the E phase spends a fixed time per row, and below 512 bytes the general
// kernels, which only fetch the 4 C split values of a row, are faster (D = 27, C = 4, N = 2^20:
// 0.03 against 0.47 ms).
template <bool SCAN, bool GATHER>
int launch_odd_sized(const RowsArgs &a, int codebooks, int need, hipStream_t stream)
{
    if (codebooks <= 16 && need <= 1024) return launch_rows<16, 1, 4, kF32, SCAN, GATHER, true, true>(a, stream);
    if (codebooks <= 16 && need <= 2048) return launch_rows<16, 2, 4, kF32, SCAN, GATHER, true, true>(a, stream);
    if (codebooks <= 32 && need <= 2048) return launch_rows<32, 2, 4, kF32, SCAN, GATHER, true, true>(a, stream);
    if (codebooks <= 32 && need <= 4096) return launch_rows<32, 4, 4, kF32, SCAN, GATHER, true, true>(a, stream);
    if (codebooks <= 64 && need <= 4096) return launch_rows<64, 4, 2, kF32, SCAN, GATHER, true, true>(a, stream);
    if (codebooks <= 64 && need <= 8192) return launch_rows<64, 8, 2, kF32, SCAN, GATHER, true, true>(a, stream);
    return 1;
}

// The same for a narrow type: rows of up to 4 KiB (up to 16 codebooks: 1 KiB, up to 32: 2 KiB).
template <int DT, bool GATHER>
int launch_odd_narrow(const RowsArgs &a, int codebooks, int need, hipStream_t stream)
{
    if (codebooks <= 16 && need <= 1024) return launch_rows<16, 1, 4, DT, true, GATHER, true, true>(a, stream);
    if (codebooks <= 32 && need <= 1024) return launch_rows<32, 1, 4, DT, true, GATHER, true, true>(a, stream);
    if (codebooks <= 32 && need <= 2048) return launch_rows<32, 2, 4, DT, true, GATHER, true, true>(a, stream);
    if (codebooks <= 64 && need <= 1024) return launch_rows<64, 1, 2, DT, true, GATHER, true, true>(a, stream);
    if (codebooks <= 64 && need <= 2048) return launch_rows<64, 2, 2, DT, true, GATHER, true, true>(a, stream);
    if (codebooks <= 64 && need <= 4096) return launch_rows<64, 4, 2, DT, true, GATHER, true, true>(a, stream);
    return 1;
}

template <bool GATHER>
int launch_odd_typed(const RowsArgs &a, int dtype, int codebooks, int need, hipStream_t stream)
{
    switch (dtype) {
    case MADDNESS_F16: return launch_odd_narrow<kF16, GATHER>(a, codebooks, need, stream);
    case MADDNESS_BF16: return launch_odd_narrow<kBF16, GATHER>(a, codebooks, need, stream);
    default: return launch_odd_narrow<kU8, GATHER>(a, codebooks, need, stream);
    }
}

// The codebooks of the kernel that takes rows of `need` bytes in that form (0: none does).
int odd_codebooks(int es, int codebooks, int need)
{
    const int per_row = es == 4 ? 1 : 2;      // (narrow rows: half the bytes)
    return codebooks <= 16 && need * per_row <= 2048 ? 16 : codebooks <= 32 && need * per_row <= 4096 ? 32
           : codebooks <= 64 && need * per_row <= 8192 ? 64 : 0;
}

// Few rows (those that the kernel by blocks of rows and columns, which is asked first, has left): the general kernel has to bring the tables into LDS, 11 to 20 us for what it holds at once (up to some
// 148 KiB; 25 to 45 us where it reads single bytes), and this one tables of `kernel_codebooks` codebooks and whole passes
// of columns into registers, 12 us for one pass and some 8 for each further one.  So it depends on how much of these is
// padding.  Measured, general and here: words, fp32 rows, 1.5 times the tables 19 and 13 us, 2.5 times 15 and 13, 3.3 times
// 11.7 and 12.5, 3.9 times 12.4 and 14.1, 5.3 times 18 and 30 (C = 12, M = 592, rows of 6000 bytes, which the kernel for 64
// codebooks takes); narrow rows 3.1 times 15.3 and 14.5, 4.1 times 19 and 22, 6.2 times 19 and 29; up to 8 rows, for which
// the general kernel takes 11 to 13 us, 2.0 times 12.7 and 12.3, 2.4 times 11.3 and 12.3; single bytes 5.2 times 28 and 21,
// 7.8 times 24 and 23, 10.2 times 28 and 31.  64 codebooks with whole 16-byte pieces have tiles walked instead (30 to 100 us).
bool few_rows_in_lds(const RowsArgs &a, int kernel_codebooks, int es, bool any_shape)
{
    if (a.N >= 16384 || !scan_in_one_piece(a.codebooks, a.M, true)) return false;
    if (a.codebooks == 64 && (a.N > 8 || a.M % 16 == 0)) return false;
    const int pass = kernel_codebooks == 64 ? 256 : 512;                      // columns
    const int64_t padded = (int64_t)kernel_codebooks * ((a.M + pass - 1) / pass * pass), tables = (int64_t)a.codebooks * a.M;
    const bool words = a.M % 4 == 0 && aligned_to(a.luts, 4);
    const int tenths = !words ? 90 : a.N <= 8 ? 23 : es != 4 ? 35 : any_shape ? 30 : 33;
    return 10 * padded > tenths * tables;
}

// Narrow rows of any shape, tables of up to 80 KiB: the general kernel reads the 4 C split values of a row and adds C table
// entries for every column, this one reads whole rows and pays for the codebooks and columns it is built for.  Below 32768
// rows the general kernel wins or is level (C = 24, M = 200, 75 KiB 13 and 14 us for 1410), and for short rows with next to no
// entries (C = 22, M = 8, rows of 348 bytes, 124440 of them 24 and 33).  From there on both times are estimated, in us, with
// costs fitted to 638 drawn shapes of 32768 to 300000 rows: this kernel's within a tenth, the general one's, which depends on
// what of the rows the caches hold, within a third (with 16 lanes to a row it is the dearer one).  By this rule 917 shapes
// take 1.02 times as long as with the faster kernel every time, 25 of them over a tenth longer than in the general kernel, 27
// than here; always the general one 1.36 times, always this one 1.06 times.  Measured, general and here: C = 1, M = 13,
// bytes, rows of 562, 152670 of them 16 and 35; C = 16, M = 20, rows of 85, 53325 12 and 20; C = 12, M = 216, rows of 160,
// 252134 86 and 102; C = 2, M = 92, binary16, rows of 3116, 55727 24 and 45; C = 16, M = 64, rows of 512, 32768 25 and 15;
// C = 16, M = 16, bytes, rows of 1943, 106122 90 and 47; C = 16, M = 17, rows of 1536, 51491 48 and 25; C = 53, M = 42,
// bytes, rows of 426, 85913 67 and 33; C = 9, M = 240, bytes, rows of 702, 205940 150 and 88; C = 4, M = 512, binary16,
// rows of 128, 131072 111 and 71.
bool narrow_rows_split_only(const RowsArgs &a, int kernel_codebooks, int es)
{
    if (a.N < 32768 || (a.D * es < 512 && a.codebooks * (int64_t)a.M < 256)) return true;
    const int words = (a.M + 3) / 4, span = kernel_codebooks == 64 ? 32 : 64, blocks = (a.M + span - 1) / span;
    int lanes = 1;                                         // of a wavefront to a row, as launch_scan has it
    while (lanes < words && lanes < 64) lanes *= 2;
    const int rows_at_once = std::max(64 / lanes, 4), row_passes = rows_at_once * lanes / 64 * ((words + lanes - 1) / lanes);
    const int code_passes = (rows_at_once * ((a.codebooks + 1) / 2) + 63) / 64;
    const double rows = 1e-3 * (double)a.N, C = a.codebooks, KC = kernel_codebooks, row_bytes = (double)a.D * es;
    const bool odd = a.M % 4 != 0;
    // a wavefront's turn: codes, table entries (reads that start a power of two apart meet in LDS banks), stores; then what
    // grows with the rows' bytes
    const double turn = 0.64 * code_passes + 0.008 * C * row_passes + (a.M == 4 * lanes ? 0.32 : 0.0) + (odd ? 0.29 : 0.0) +
                        (lanes >= 16 ? 0.19 : 0.0);
    // rows of the tables that start a multiple of 64 bytes apart; input and results beyond the 256 MB of the last cache; and it
    // writes no more than some 2.2 TB/s
    const double slower = (lanes == 1 ? 1.09 : 1.0) * (a.M % 64 == 0 ? 1.17 : 1.0) *
                          (rows * (row_bytes + 4.0 * a.M) > 256e3 ? 1.25 : 1.0);
    const double general = 5.0 + 0.003 * C * a.M + (a.M <= 8 ? 0.26 * C : 0.0) + rows / rows_at_once * turn +
                           rows * ((odd ? 0.95e-3 * a.M : 0.0) + 1.1e-4 * std::min(row_bytes, 256.0 * C) +
                                   7e-3 * C * std::min(1.0, row_bytes / 2048));
    const double here = 10.5 + (es == 1 ? 2.5 : 0.0) +
                        rows * (0.056 + KC * (1.8e-3 + 3.1e-4 * blocks) + 8e-5 * row_bytes + 1.15e-3 * a.M);
    return std::max(slower * general, 1.82e-3 * rows * a.M) < (lanes == 16 ? 0.75 : 1.05) * here;
}

template <bool SCAN>
int launch_odd(const RowsArgs &a, int codebooks, const MatrixA &A, hipStream_t stream)
{
    const int es = A.elem_bytes(), row_bytes = a.D * es;
    if (!SCAN && (row_bytes < 512 || A.dtype != MADDNESS_F32)) return 1;
    if (!aligned_to(a.A, es)) return 1;
    // a row is staged from the 16-byte boundary at or before its start: row n begins (a0 + n s) mod 16
    // bytes after one
    const unsigned a0 = (unsigned)reinterpret_cast<uintptr_t>(a.A) & 15u, s = (unsigned)(a.lda * es) & 15u;
    unsigned max_shift = 0;
    for (unsigned n = 0; n < 16; ++n) max_shift = std::max(max_shift, (a0 + n * s) & 15u);
    const int need = row_bytes + (int)max_shift;
    if constexpr (SCAN) {
        // Where the general kernels are as fast, having few table entries to add for the time a row takes here: fp32 rows
        // below 512 bytes and tables they read in one piece (C = 15, M = 100 43 us there and 44 here for 2^17 rows; C = 30,
        // M = 300, 140 KiB, 189 and 89); narrow rows and few rows as above.
        const int64_t table_bytes = 16 * (int64_t)codebooks * a.M;
        if (A.dtype == MADDNESS_F32 && row_bytes < 512 && table_bytes <= 64 * 1024) return 1;
        const int kernel_codebooks = odd_codebooks(es, codebooks, need);
        if (kernel_codebooks == 0) return 1;
        if (A.dtype != MADDNESS_F32 && table_bytes <= 80 * 1024 && narrow_rows_split_only(a, kernel_codebooks, es)) return 1;
        if (few_rows_in_lds(a, kernel_codebooks, es, true)) return 1;
        // more than two blocks of columns: whole rows through LDS; else straight from the registers
        const int span = codebooks <= 32 ? 64 : 32;
        const bool gather = (a.M + span - 1) / span > 2;
        if (A.dtype != MADDNESS_F32)
            return gather ? launch_odd_typed<true>(a, A.dtype, codebooks, need, stream)
                          : launch_odd_typed<false>(a, A.dtype, codebooks, need, stream);
        if (gather) return launch_odd_sized<true, true>(a, codebooks, need, stream);
    }
    return launch_odd_sized<SCAN, false>(a, codebooks, need, stream);
}

// Row-major A: rows of 16-byte pieces, at most 8 KiB (fp32) or 4 KiB (narrow types) long.
// SCAN = false (encode only): fp32.
template <bool SCAN>
int launch_row_major(const RowsArgs &a, int C, int D, const MatrixA &A, hipStream_t stream)
{
    const int es = A.elem_bytes();
    if ((D * es) % 16 != 0 || (A.ld * es) % 16 != 0 || !aligned_to(A.data, 16)) return 1;
    if (a.codebooks == C && a.codes_out && !aligned_to(a.codes_out, C == 16 ? 8 : 16)) return 1;
    const int row_bytes = D * es;
    if (a.codebooks != C) {
        // a multiple of 8 codebooks that is not 16, 32 or 64: the next larger kernel, padded (fp32)
        if (A.dtype != MADDNESS_F32 || (a.codes_out && !aligned_to(a.codes_out, 4))) return 1;
        if (C == 16 && D <= 512) return launch_rows<16, 2, 4, kF32, SCAN, false, true>(a, stream);
        if (C == 32 && D <= 512) return launch_rows<32, 2, 4, kF32, SCAN, false, true>(a, stream);
        if (C == 32 && D <= 1024) return launch_rows<32, 4, 4, kF32, SCAN, false, true>(a, stream);
        if (C == 64 && D <= 1024) return launch_rows<64, 4, 2, kF32, SCAN, false, true>(a, stream);
        return 1;
    }
    if constexpr (SCAN) {
        // The S phase that writes whole rows: for fp32 output rows that do not start on 128-byte
        // lines (more than 4 blocks of columns; N = 2^20, C = 32, M = 1000: 1.43 against 2.04 ms),
        // and where one pass of the 8 wavefronts covers the whole row exactly (C <= 32, M in
        // (448, 512]: 0.675 against 0.767 ms at M = 512; no gain elsewhere: at M = 256 0.519 against 0.524 ms
        // beside rows of 2 KiB and 0.864 against 0.834 ms beside rows of 4 KiB, 1.27 against 1.22 ms at
        // M = 1024, 2.89 against 2.39 ms at C = 64, M = 512)
        const int span = C == 64 ? 32 : 64;
        const bool unaligned = a.ldo % 32 != 0 || !aligned_to(a.out, 128);
        const bool one_full_pass = C != 64 && a.M > 7 * span && a.M <= 8 * span;
        if (A.dtype == MADDNESS_F32 && a.out && ((unaligned && a.M > 4 * span) || one_full_pass)) {
            if (C == 16 && D <= 512) return launch_rows<16, 2, 4, kF32, true, true>(a, stream);
            if (C == 32 && D <= 512) return launch_rows<32, 2, 4, kF32, true, true>(a, stream);
            if (C == 32 && D <= 1024) return launch_rows<32, 4, 4, kF32, true, true>(a, stream);
            if (C == 64 && D <= 1024) return launch_rows<64, 4, 2, kF32, true, true>(a, stream);
        }
    }
    if (A.dtype == MADDNESS_F32) {
        if (C == 16 && D <= 256) return launch_rows<16, 1, 4, kF32, SCAN>(a, stream);
        if (C == 16 && D <= 512) return launch_rows<16, 2, 4, kF32, SCAN>(a, stream);
        if (C == 16 && D <= 1024) return launch_rows<16, 4, 4, kF32, SCAN>(a, stream);
        if (C == 64 && D <= 1024) return launch_rows<64, 4, 2, kF32, SCAN>(a, stream);
        if (C == 32 && D <= 512) return launch_rows<32, 2, 4, kF32, SCAN>(a, stream);
        if (C == 32 && D <= 1024) return launch_rows<32, 4, 4, kF32, SCAN>(a, stream);
        if (C == 64 && D <= 2048) return launch_rows<64, 8, 2, kF32, SCAN>(a, stream);
        if (C == 32 && D <= 2048) return launch_rows<32, 8, 4, kF32, SCAN>(a, stream);
        return 1;
    }
    if constexpr (!SCAN) return 1;
    if (row_bytes > 4096) return 1;
    if (C == 16) return launch_odd<SCAN>(a, C, A, stream);
    if (C == 32)
        return row_bytes <= 1024   ? launch_rows_typed<32, 1, 4>(a, A.dtype, stream)
               : row_bytes <= 2048 ? launch_rows_typed<32, 2, 4>(a, A.dtype, stream)
                                   : launch_rows_typed<32, 4, 4>(a, A.dtype, stream);
    return row_bytes <= 1024   ? launch_rows_typed<64, 1, 2>(a, A.dtype, stream)
           : row_bytes <= 2048 ? launch_rows_typed<64, 2, 2>(a, A.dtype, stream)
                               : launch_rows_typed<64, 4, 2>(a, A.dtype, stream);
}

// A stored by columns, few rows: tables and trees cost this kernel 12 to 19 us before the first row; the general one brings
// the tables it can hold at once into LDS in 9 to 22 us, and then takes 8192 rows of large tables, or more the fewer words
// a row of them has, in 2 us; reads of rows of 16, 32 or 64 words meet in LDS banks there.  Measured, general and here: C = 16,
// M = 264, 66 KiB, 15.2 and 18.3 us for 4200 rows, 22.5 and 18.1 (M = 320) for 8500; C = 32, M = 192 15.2 and 17.3 for 6000, 22.1
// and 19.1 for 8500; M = 256 20 and 19 for 5000; C = 64, M = 96 18.5 and 17.3 for 6000; C = 16, M = 584, 146 KiB, 21.3 and
// 19.0 for 100, 22.7 and 28.1 for 1000, 33.1 and 28.7 for 8500; small tables, time there over time here for 16384, 25000,
// 45000 and 80000 rows: C = 16, M = 16 1.04, 1.01, 1.01, 0.79 (100000: 1.12), M = 28 0.97, 0.97, 0.92, 1.15, M = 48 0.94, 1.15,
// 1.87, 2.46, M = 64 1.07, 1.87, 2.52, 2.27; C = 32, M = 20 0.69, 0.75, 0.76, 1.95, M = 48 0.79, 1.02, 1.30, 1.46, M = 100 0.95,
// 1.19, 1.23, 2.48.  C = 16, M = 140, general and here, 15.2 and 17.3 for 24576, 19.9 and 17.4 for 25000; M = 188 13.3 and 17.1 for
// 16384, 17.0 and 17.4 for 24576; M = 200 13.9 and 17.5 for 16384, 21.0 and 17.6 for 19000; M = 252 15.3 and 17.6, 18.4 and 17.6;
// M = 256 20.1 and 17.0 for 16384.
bool few_columns_in_lds(int C, int M, int64_t N)
{
    const int64_t tables = 16 * (int64_t)C * M;
    if (tables > 128 * 1024) return C == 16 && N > 256 && N <= 8192 && scan_in_one_piece(C, M, true);
    if (tables > 64 * 1024) return N < (C == 64 || tables == 128 * 1024 ? 4096 : 8193);
    if (C == 64) return N < 16384;
    int lanes = 1;                                         // of a wavefront to a row, as launch_scan has it
    while (4 * lanes < M && lanes < 64) lanes *= 2;
    const bool banks = M == 4 * lanes;
    switch (lanes) {
    case 1: return N < 16384;
    case 2: return C == 16 || N < 16384;
    case 4: return N < (C == 16 ? 98304 : 65536);
    case 8: return N < (C == 32 && banks ? 24576 : 57344);
    case 64: return N < (banks ? 16384 : M < 192 ? 24577 : 16385);
    default: return N < (banks || (C == 16 && lanes == 32) ? 16384 : 24576);
    }
}

}  // namespace

// Returns MADDNESS_OK after a launch, 1 if the shape is not covered.
int launch_fused_mfma(const maddness_params &p, const MatrixA &A, int64_t N, int32_t M, const uint8_t *luts,
                      const float *scale, const float *offset, float *out, int64_t ldo, uint16_t *acc,
                      uint8_t *codes, hipStream_t stream)
{
    const int D = p.D;
    const int es = A.elem_bytes();
    if (!A.col_major && (int64_t)D * es > kMaxRowBytes) return 1;
    RowsArgs a{};
    a.A = A.data; a.lda = A.ld; a.D = D; a.N = N;
    a.split_dims = p.split_dims; a.thresholds = p.thresholds;
    a.luts = luts; a.scale = scale; a.offset = offset; a.M = M;
    a.out = out; a.ldo = ldo; a.acc = acc; a.codes_out = codes;
    a.codebooks = p.C;
    // the kernel's C: 16, 32 or 64; another multiple of 8 takes the next larger one with padding
    const int C = p.C <= 16 ? 16 : (p.C <= 32 ? 32 : 64);
    const int NT = C == 64 ? 2 : 4;
    // shapes the tiled forms do not take as they are (C not a multiple of 8, rows of A or of the outputs that
    // are not whole aligned pieces, M not a multiple of the lane's columns): the form for any shape
    const bool regular = p.C % 8 == 0 && p.C >= 8 && p.C <= 64 && (C == p.C || A.plain()) && M % NT == 0 &&
                         aligned_to(luts, NT) && (!out || (ldo % NT == 0 && aligned_to(out, 4 * NT))) &&
                         (!acc || aligned_to(acc, 2 * NT)) &&
                         (A.col_major || ((D * es) % 16 == 0 && (A.ld * es) % 16 == 0 && aligned_to(A.data, 16) &&
                                          (!codes || aligned_to(codes, C != p.C ? 4 : (C == 16 ? 8 : 16)))));
    if (regular && A.col_major && C == p.C && N <= kColsFewRows) {
        if (few_columns_in_lds(C, M, N)) return 1;
        if (codes && !aligned_to(codes, 4)) return 1;
        return C == 16   ? launch_cols_few_typed<16, 4>(a, A.dtype, stream)
               : C == 32 ? launch_cols_few_typed<32, 4>(a, A.dtype, stream)
                         : launch_cols_few_typed<64, 2>(a, A.dtype, stream);
    }
    if (N < matrix_cores_min_rows(p.C, M, regular && (p.C == 16 || p.C == 32))) return 1;
    if (!regular) {
        if (A.col_major || p.C > 64) return 1;
        return launch_odd<true>(a, p.C, A, stream);
    }
    if (A.col_major) {
        if (C == 16) return 1;
        // runs of four rows: column stride and base aligned to four elements, whole quads of rows
        // (the caller takes care of the last N % 4 rows)
        if (N % 4 != 0 || A.ld % 4 != 0 || !aligned_to(A.data, 4 * (size_t)es)) return 1;
        if (codes && !aligned_to(codes, C / 2)) return 1;
        if (C == 32) {
            switch (A.dtype) {
            case MADDNESS_F32: return launch_cols<32, 4, kF32>(a, stream);
            case MADDNESS_F16: return launch_cols<32, 4, kF16>(a, stream);
            case MADDNESS_BF16: return launch_cols<32, 4, kBF16>(a, stream);
            default: return launch_cols<32, 4, kU8>(a, stream);
            }
        }
        switch (A.dtype) {
        case MADDNESS_F32: return launch_cols<64, 2, kF32>(a, stream);
        case MADDNESS_F16: return launch_cols<64, 2, kF16>(a, stream);
        case MADDNESS_BF16: return launch_cols<64, 2, kBF16>(a, stream);
        default: return launch_cols<64, 2, kU8>(a, stream);
        }
    }
    if (few_rows_in_lds(a, C, es, false)) return 1;
    return launch_row_major<true>(a, C, D, A, stream);
}

// Encode only, with the E phase of the same kernel (M = 0: no S phase, the codes are copied
// from LDS to memory after it): the rows of a region are read in one moving window by the
// whole chip.
int launch_encode_phased(const maddness_params &p, const MatrixA &A, int64_t N, uint8_t *codes, hipStream_t stream)
{
    if (p.C > 64 || !A.plain() || N < 16384 || (int64_t)p.D * A.elem_bytes() > kMaxRowBytes) return 1;
    const int C = p.C <= 16 ? 16 : (p.C <= 32 ? 32 : 64);   // the kernel's C; the rest is padding
    RowsArgs a{};
    a.A = A.data; a.lda = A.ld; a.D = p.D; a.N = N;
    a.split_dims = p.split_dims; a.thresholds = p.thresholds;
    a.codes_out = codes;
    a.codebooks = p.C;
    if (p.C % 8 == 0) {
        const int rc = launch_row_major<false>(a, C, p.D, A, stream);
        if (rc != 1) return rc;
    }
    return launch_odd<false>(a, p.C, A, stream);
}

}  // namespace maddness
