// Internal tables shared by the host planner and the device kernels.
// Plain structs only: they are copied byte-for-byte to the GPU.
#ifndef PSGD_INTERNAL_H
#define PSGD_INTERNAL_H

#include <stdint.h>
#include <string>
#include <vector>

#include "psgd.h"

namespace psgd {

constexpr int kWave = 64;          // gfx950 wavefront
constexpr int kBlock = 256;        // threads per workgroup in the streaming kernels (4 waves)
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kAlignElems = 64;    // every matrix starts on a multiple of this many elements
constexpr int kMaxVecPerLaneK1 = 2;  // column vectors a lane owns per row in the P = M Q kernel
constexpr int kMaxVecPerLaneK3 = 2;  // column vectors a lane owns in the Q = M^T P and decompress kernels
constexpr int kOrthoBlock = 256;   // threads of the single-workgroup Gram-Schmidt kernel
constexpr int kValuMaxRank = 8;    // ranks up to this run on the vector-ALU kernels
constexpr int kPanelFloats = 12288;  // n*r up to this: Gram-Schmidt by one workgroup with the panel in LDS (48 KB)
constexpr int kGramRows = 256;     // rows per workgroup of the Gram / apply kernels (Cholesky-QR over row blocks)
constexpr int kPreReduceParts = 16; // more partial-P slices than this: a reduction kernel runs before the orthogonalisation
constexpr int kOrthoMaxRows = 1024; // largest value of the tuning key ortho_rows: panels with more rows always take the multi-workgroup route
// Streaming kernels: from this many workers on, on sets of at least kMeanElems elements (kMeanElemsPerWorker for every worker above
// sixteen workers) with 15 in 16 of them in rows that are multiples of 4, the products are taken of the mean over the workers.
// Whole steps, us, each worker by itself / the mean first: ResNet18-shaped set, rank 4, 16 workers 730 / 670, 8 workers 372 / 348, 4
// workers 215 / 205; 24 matrices of 9 M elements, 5 workers 205 / 191; two transformer layers (42 M elements), 4 workers 729 / 657, bf16
// gradients, rank 2 643 / 590; 1.1 M elements (ResNet18-shaped), 8 workers 76.6 / 68.0, 4 workers 44.2 / 44.2, 16 workers 153.7 / 153.5.
// The other side of the line: two workers save no bytes (24 M elements 219 / 244); narrower accesses lose at 20 M elements in odd
// rows (3 workers, 294 / 341) and in the LSTM-shaped set's rows of 650 (4 workers, 719 / 756); on small sets the serial walk over many
// workers is too long (32 workers: 1.1 M elements 287 / 293 and 149 / 158, 2.0 M 255 / 278, but 2.1 M 471 / 457, 2.8 M 487 / 416).  Three
// workers (ResNet18-shaped 168 / 157, with the update 198 / 193) and sets below 2^20 elements (0.7 M, 4 workers 38.7 / 35.8; five matrices,
// 16 workers 36.5 / 36.9) have not been measured over a range, and stay with each worker by itself.  Sets that build_one_sweep
// takes (rank <= 4, rows that fit a workgroup, one_sweep_pays) are walked once instead: the line holds for the others.
constexpr int kMeanWorkers = 4;
constexpr int64_t kMeanElems = int64_t(1) << 20;
constexpr int64_t kMeanElemsPerWorker = int64_t(1) << 16;
constexpr int kFlatTileElems = 1024;        // baselines: elements of a flattened matrix per workgroup of the elementwise sweep (one 16-byte access per
                                            // lane and array: the smallest slices were the fastest, 8192 -> 1024: 34.7 -> 28.7 us on the ResNet18 set)
constexpr int kFactorAlignElems = 4;        // P and Q of a matrix start at multiples of 4 floats (vector loads of factor rows)
constexpr int kHrGramTileRows = 128;       // matrix-core path: rows per workgroup of the mean-P / Gram / apply kernels
constexpr int64_t kHrMaxRows = 1 << 22;   // matrix-core path: tallest matrix (an n x 64 factor is addressed with 31-bit byte offsets)
constexpr int64_t kHrMaxCols = 1 << 20;   // matrix-core path: longest row (tiles of <= 256 rows are addressed with 31-bit byte offsets)
constexpr int64_t kStreamHintBytes = int64_t(320) << 20;   // update matrices of all workers above this (the 256 MB memory-side
                                                           // cache and a margin): the sweeps after the first treat M as a stream

// One matrix of the model.
struct MatDesc {
    int64_t off;        // element offset in the matrix region
    int64_t p_off;      // float offset in packed P
    int64_t q_off;      // float offset in packed Q
    int64_t ppart_off;  // float offset in the workspace: partial P, [W * n_cchunk][n][r]
    int64_t qpart_off;  // float offset in the workspace: partial Q, [W * n_rblock][m][r]
    int64_t gram_off;   // Cholesky-QR panels: offset (in doubles) of the Gram partials, [n_gblock][r*r]
    int32_t n, m, r;    // rows, columns, effective rank
    int32_t vec;        // elements per vector access along a row (4, 2 or 1)
    int32_t n_cchunk;   // column chunks of the P = M Q kernel (partials to sum)
    int32_t n_rblock;   // row blocks of the Q = M^T P kernel (partials to sum)
    int32_t tensor;     // index in the caller's shape list
    int32_t n_gblock;   // row blocks of the Gram / apply kernels; 0 = panel orthogonalised by one workgroup in LDS (k_ortho)
    int32_t pad_[2];
    int64_t chol_off;   // matrix-core path: offset (in doubles) of this matrix's Cholesky factor, r*r + r values
    int64_t kept_off;   // Random Block / Random K baselines: offset of this matrix's kept values (and indices) in their packed buffers
    int64_t kept;       // ... and their number, min((n + m) * rank, n * m)
};

// One workgroup's share of a streaming kernel.
struct Tile {
    int32_t mat;    // matrix index; -1: a slice of the vector region
    int32_t row0;   // first row (vector tiles: unused)
    int32_t nrows;  // rows
    int32_t vec0;   // first column vector (units of MatDesc::vec elements);
                    // vector tiles: first element / 4 is not assumed, see elem0 below
    int32_t nvec;   // column vectors
    int32_t part;   // which partial buffer slice this tile writes
    int64_t elem0;  // vector tiles and Q-reduce tiles: first element
    int64_t nelem;  // vector tiles and Q-reduce tiles: element count
};

// Resident path: one wavefront keeps one tile of M in registers through the whole step.
constexpr int kResRows = 32;         // most rows of a resident tile (registers: rows * vec floats per lane) ...
constexpr int res_rows_for_rank(int r) { return r <= 2 ? 32 : 24; }   // ... fewer when the rank needs the registers
constexpr int kResMinRows = 8;       // strips are not made thinner than this
constexpr int kResMaxN = 512;        // tallest matrix the single-wavefront Gram-Schmidt handles (8 rows per lane)
constexpr int kResMaxRank = 4;
constexpr int kResCUs = 256;         // MI355X compute units: the planner's provisional figure (it runs without a device); the
                                     // tiling is laid out again for the device's own count when the tables are uploaded
constexpr int kResBlocksPerCU = 2;   // 256-thread workgroups per compute unit (8 wavefronts, 2 per SIMD)
// Resident step fused with the update: from this many elements on momentum and parameters go around the caches (stream_hints < 0).
// Four states of a set in turn, us, ordinary / around: ResNet18-shaped, 11.2 M elements, rank 2 / 4 70.4 / 80.8 and 62.7 / 72.5; 6.3 M,
// rank 1 45.9 and 39.4; 3.9 M, rank 2 32.1 and 34.9; 2.8 M, rank 4 34.5 and 36.8; five matrices 15.9 and 16.8.  What else runs between the steps
// decides on either side of the line.  One state behind 512 MB of other work: 11.2 M, rank 1 / 2 / 4 68.8 / 73.0 / 85.9 and 67.3 / 71.7 / 83.2, 6.3 M 46.6 / 49.7 / 60.2 and
// 44.7 / 46.8 / 57.7, 3.9 M 41.5 / 42.0 / 52.8 and 38.8 / 40.2 / 48.4, 2.1 M 35.5 / 36.6 / 41.2 and 32.9 / 34.2 / 39.8, 0.7 M 25.4 / 26.7 / 31.2 and 24.8 / 26.1 / 30.4; with nothing in between, where the
// memory-side cache holds it: 11.2 M 58.0 / 61.3 / 70.5 and 61.8 / 65.2 / 75.5, 6.3 M 39.3 / 42.4 / 52.1 and 41.6 / 45.4 / 55.0, 3.9 M 31.8 / 35.2 / 43.8 and 33.0 / 37.3 / 46.4, 2.1 M 24.3 / 28.0 / 37.3 and
// 24.6 / 28.8 / 38.6; behind 96 MB, rank 2, 11.2 M 66.1 / 63.9, 8.5 M 51.3 / 54.2, 3.9 M 34.9 / 36.8, 0.7 M 20.8 / 21.2.  Small sets go with small networks and little
// other work, large ones with much, so the line stays between them.
constexpr int64_t kResAroundElems = 4000000;
constexpr int kResTracePoints = 16;  // diagnostic timestamps per workgroup of the resident kernel

// One wavefront's share of the resident kernel.
struct RTile {
    int32_t mat;         // matrix index; -1: slice of the vector region; -2: idle slot
    int32_t row0, nrows; // strip of rows (nrows <= kResRows)
    int32_t vec0, nvec;  // column vectors (nvec <= 64)
    int32_t ppart;       // column-chunk index = slice of partial P this tile writes; the wavefront with
                         // ppart == 0 adds the chunks of its strip, the one that also has row0 == 0
                         // orthogonalises the matrix
    int32_t nstrips_mat; // strips of this matrix
    int32_t qrun_len;    // > 0: first of a run of consecutive wavefronts of the workgroup that hold strips of
                         // the same column chunk; it adds the run's sums in LDS and writes one partial Q
    int32_t qpart;       // slot of that partial; the run with qpart == 0 adds the chunk's partials
    int32_t nqparts;     // partial-Q slots of this column chunk
    int32_t cntq;        // running index of this column chunk over the model
    int32_t cnts;        // running index of this strip over the model
    int32_t pad_;
    int64_t elem0, nelem;  // vector tiles: slice of the vector region
};

// P = M Q and S = M^T P in one walk over M (k_one_sweep, k_solve)
constexpr int kOneMaxRank = 4;
constexpr int kOneMaxWaves = 8;     // wavefronts of a workgroup, and of a row
constexpr int kOneRows = 2;         // rows of a step
constexpr int kOneStepWorkers = 8;  // from this many workers on small sets have groups of a single step (one_sweep_blocks)
constexpr int64_t kOneStepElems = int64_t(1) << 19;
constexpr int64_t kOneMaxBytes = int64_t(64) << 20;   // plan-owned partial sums
// psgd_step_iterations on a plan that takes the one walk: above this many elements of all workers the mean is stored and every further
// iteration reads it twice (8 bytes an element) instead of every worker's M once (4 W).  Whole calls, us, mean / one walk: 4 workers,
// two and four iterations, ResNet18-shaped, 1.1 M elements 60 / 52 and 106 / 100, 2.8 M 83 / 79 and 138 / 139, 8.5 M 187 / 189 and 272 / 294, LSTM-shaped, rows of 648,
// 31.6 M 609 / 645 and 781 / 880, rows of 300, 5.2 M (20.6 M in all) 156 / 131 and 229 / 191; 40 of 256 x 1024 187 / 195 and 269 / 276; 8 workers, three iterations, ResNet18-shaped 1.1 M 111 / 103,
// 2.8 M 190 / 200, 8.5 M 363 / 444; 16 workers, four, 1.1 M 218 / 213, 2.8 M 333 / 382, rows of 300 540 / 624.
constexpr int64_t kIterMeanElems = int64_t(20) << 20;
// Lines of one_sweep_pays, in elements of a worker, and in bytes of partial S
constexpr int64_t kOneMeanWorkers = 8;
constexpr int64_t kOneThinElems = int64_t(1) << 19, kOneThin4Elems = int64_t(1) << 22;
constexpr int64_t kOnePartialBytes = 3500000, kOnePartialElems = int64_t(7) << 19, kOnePartialElems4 = int64_t(1) << 23;
// Column vectors a lane owns (12 columns; fewer with several workers, whose steps take the registers of two more sets of rows, and of
// rows that are read element by element), and steps whose loads are in flight: what 256 registers hold beside the lane's fp64
// sums (rank 4: 96 of them).  LSTM-shaped set, rank 4, k_one_sweep: 12 columns, one step 69 us; 6 columns and two wavefronts to a
// row, three steps 78.  24 matrices, three workers, two iterations: 8 / 6 / 8 columns, two steps 182 us a pass, 12 and one step 196.
constexpr int one_nv(int v, bool mean) { return (v == 1 ? 8 : (!mean ? 12 : (v == 2 ? 6 : 8))) / v; }
constexpr int one_depth(int r, bool mean) { return mean || r <= 2 ? 2 : 1; }
// k_one_sweep_wide: column vectors (of four) a lane owns, rows whose loads are in flight, and shared memory: Q of a row as floats, after it
// one column vector's sums of every lane
constexpr int kOneWideNV = 4, kOneWideDepth = 2;
constexpr int kOneWideLds = kOneMaxWaves * kWave * kOneWideNV * 4 * kOneMaxRank * 4;
static_assert(4 * kOneMaxRank * (kOneMaxWaves * kWave + 1) * 8 <= kOneWideLds, "the sums fit where Q was");
// floats of Q a lane needs, in sets of four
constexpr int one_q_floats(int r, int v, bool mean) { return (one_nv(v, mean) * v * r + 3) / 4 * 4; }
// column vectors of a lane whose sums are added over the workgroup's groups at a time (at most 16 doubles a lane)
constexpr int one_deposit(int r, int v, bool mean) {
    int n = 16 / (v * r) < 1 ? 1 : 16 / (v * r);
    while (one_nv(v, mean) % n) --n;
    return n;
}
struct OneMat {
    int64_t off, p_off, q_off;   // as in MatDesc
    int64_t s_off, g_off;        // in doubles: [n_blocks][m][r] of partial S, [n_blocks][R (R + 1) / 2] of partial Gram matrices
    int32_t n, m, r, vec;
    int32_t n_blocks;            // row blocks
    int32_t waves_log2;          // wavefronts that share a row
};
struct OneTile {
    int32_t mat, row0, nrows, block;
};
struct SolveTile {
    int32_t mat;
    int32_t first, count;        // rows of P (`rows`), else rows of Q
    int16_t rows, cols_log2;     // rows of Q per workgroup, 2^cols_log2
};

struct Tuning {
    int64_t one_sweep = -1; // P = M Q and Q = M^T P_hat in one walk over M: -1 by the rule at build_one_sweep, 0 never, 1 also where another key
                            // asks for a kernel of the two walks
    int64_t k1_rows = 0;    // rows per workgroup tile, P = M Q; 0: by the access width of the matrix (16 / 32 / 64; twice
                            // that for small sets)
    int64_t k1_nv = 2;      // column vectors per lane (<= kMaxVecPerLaneK1); products of the mean over the workers: always one
    int64_t worker_mean = -1;  // products of the mean over the workers: -1 by the rule at kMeanWorkers, 0 never, 1 with any two workers
    int64_t k3_rows = 0;    // rows per workgroup tile, Q = M^T P; 0: 128, or 1024 for matrices >= 2048 x 2048
    int64_t k3_nv = 1;      // column vectors per lane (<= kMaxVecPerLaneK3)
    int64_t k4_rows = 0;    // rows per workgroup tile, decompress + residual; 0: 16 (32 for small sets)
    int64_t k4_nv = 1;
    int64_t hr_k3_rows = 2048;  // matrix-core Q = M^T P: rows per workgroup (four strips)
    int64_t hr_k4_rows = 0;     // matrix-core decompression: rows per workgroup (four strips of 16-row steps); 0 = by rank
    int64_t hr_k1_rows = 128;   // matrix-core P = M Q: rows per workgroup (multiple of 64, at most 256)
    int64_t hr_k1_cols = 2048;  // matrix-core P = M Q: columns per workgroup (multiple of 64); longer rows are split and their partial P summed
    int64_t stream_hints = -1;  // sweeps 2 and 3 of the streaming path: non-temporal loads of M and stores of the error
                                // memory (and temporal instead of non-temporal stores of Delta'); matrix-core path:
                                // non-temporal loads of M in sweep 2.
                                // -1: when M of all workers exceeds kStreamHintBytes; 0: never; 1: always
    int64_t gram_fused = -1; // Cholesky-QR panels of the two walks: 1 = Gram matrices and factorisation in one launch when the device holds a matrix's
                            // row blocks at once; 0 = always the two launches; 2 = one launch whatever the device holds
                            // (diagnostic: the waits may time out, which psgd_plan_check then reports); -1 as 1, and one walk may be taken instead
    int64_t gram_spin = 1 << 18;   // polls of one slot in that launch before a wait gives up
    int64_t ortho_rows = 0;        // panels of at most this many rows (and kPanelFloats values) are orthogonalised by one workgroup
                                   // with Gram-Schmidt in LDS (k_ortho), the others by Cholesky-QR over row blocks; 0: none (a
                                   // launch of its own for the short panels costs more than it saves: ResNet18-shaped set,
                                   // streaming, rank 2 / 4 / 8: 61.9 / 73.1 / 110.4 us with 1024, 59.6 / 67.0 / 100.9 us with 0)
    int64_t bf16_valu = -1; // bf16 gradients / output at rank <= 8: 1 = the streaming (vector-ALU) kernels, 0 = the matrix-core kernels,
                            // -1 = the matrix-core kernels at rank >= 4 on a set beyond the memory-side cache whose shapes they take
    int64_t resident = 1;   // 1: psgd_step keeps M on chip when the model fits; 0: always stream; 2: as 1 without the check
                            // against the device at upload (diagnostic, with res_max_blocks: lets a test see the waits give up)
    int64_t res_spin = 1 << 21;      // polls before a wait of the resident kernel gives up
    int64_t res_max_blocks = 0;      // 0: the device's capacity; else the most workgroups the resident tiling may use (diagnostic)
    int64_t res_rows = 0;   // 0: smallest strip height that fits; else forced strip height
    int64_t res_trace = 0;  // 1: the resident kernel records phase timestamps (diagnostic)
    int64_t xcd_order = -1;    // tile lists are ordered so that each accelerator die (own L2) works on one contiguous range of
                               // tiles: 1 = of the whole list; k >= 2 = of each group of consecutive matrices, a group being
                               // closed once it holds k tiles (a large matrix is then spread over all dies by itself); 0 = off;
                               // -1 = the planner's choice (groups sized by the worker count)
};

struct DeviceTables {
    OneMat* one_mats = nullptr;
    OneTile* one_tiles = nullptr;
    SolveTile* solve_tiles = nullptr;
    MatDesc* mats = nullptr;
    MatDesc* mats_mean = nullptr;
    Tile* tiles1 = nullptr;
    Tile* tiles1m = nullptr;
    Tile* tiles3 = nullptr;
    Tile* tiles4 = nullptr;
    Tile* tiles4u = nullptr;   // decompression fused with the update: tiles of its own, or null (then tiles4)
    Tile* tilesq = nullptr;
    Tile* tiles_gram = nullptr;
    Tile* tilesp = nullptr;
    Tile* hr_tiles1 = nullptr;
    Tile* hr_tiles3 = nullptr;
    Tile* hr_tiles4 = nullptr;
    int64_t* flat_first = nullptr;         // baselines: per matrix the index of its first slice of kFlatTileElems elements
    int32_t* kept_slice_mat = nullptr;     // baselines: per slice of kBlock kept entries, its matrix ...
    int64_t* kept_slice_first = nullptr;   // ... and its first entry within that matrix
    int32_t* mat_tensor = nullptr;         // per matrix: index in the caller's tensor list
    int32_t* small_mats = nullptr;
    unsigned* gram_sync = nullptr;              // k_gram_chol: error word, epoch, finished-workgroup count
    unsigned long long* gram_mail = nullptr;    // k_gram_chol: the row blocks' Gram matrices as {value, epoch} slots
    MatDesc* res_mats = nullptr;
    RTile* res_tiles = nullptr;
    unsigned* res_sync = nullptr;  // error word, epoch, finished-workgroup count
    unsigned long long* res_mail = nullptr;  // mailbox of {value, epoch} slots
    unsigned long long* res_trace = nullptr;  // only with tuning res_trace = 1
    void* base = nullptr;   // the one allocation holding all of the above
};

}  // namespace psgd

struct psgd_plan {
    int32_t rank = 0;
    int32_t workers = 0;
    psgd_dtype grad_dtype = PSGD_F32;
    psgd_dtype out_dtype = PSGD_F32;
    psgd_sizes sizes{};
    std::vector<psgd_shape> shapes;
    std::vector<int64_t> tensor_flat_off;   // per tensor
    std::vector<int32_t> tensor_mat;        // per tensor: matrix index or -1
    std::vector<psgd::MatDesc> mats;
    std::vector<psgd::Tile> tiles1, tiles3, tiles4, tilesq;
    std::vector<psgd::Tile> tiles4u;        // third sweep when fused with the update, if its tiles differ (else empty)
    std::vector<psgd::Tile> tiles_gram;     // row blocks of the panels orthogonalised by Cholesky-QR
    std::vector<int64_t> flat_first;        // baselines (Appendix G): running count of the slices of the flattened matrices
    int64_t flat_tiles = 0;                 //   (n_matrices + 1 entries), their total, and the slices of the vector region
    int64_t flat_vec_tiles = 0;
    std::vector<int32_t> kept_slice_mat;    // baselines: slices of kBlock kept entries (matrix, first entry)
    std::vector<int64_t> kept_slice_first;
    std::vector<int32_t> mat_tensor;
    int64_t kept_slices = 0;
    std::vector<int32_t> small_mats;        // matrices orthogonalised by one workgroup (Gram-Schmidt in LDS)
    int64_t ws_gram_doubles = 0;            // workspace: Gram partials, after the float regions
    // matrix-core path (rank > 8, or bf16 gradients / output)
    bool hr = false;
    int32_t hr_nt = 1;                      // 16-wide rank tiles
    std::vector<psgd::Tile> hr_tiles1, hr_tiles3, hr_tiles4;
    int64_t ws_chol_doubles = 0;
    std::vector<psgd::Tile> tilesp;         // 64-element slices of the n x r panels (pre-reduction of partial P)
    bool p_pre_reduce = false;              // some matrix has more than kPreReduceParts partial-P slices
    bool p_pre_reduce_mean = false;         // the same for the products of the mean over the workers
    std::vector<psgd::Tile> tiles1m;        // mean_first: the first sweep's tiles, one column vector per lane ...
    std::vector<psgd::MatDesc> mats_mean;   // ... and the same matrices with their column chunks
    float* mbar = nullptr;                  // device, N floats: mean over the workers of M (mean_first)
    bool mean_first = false;                // streaming kernels: the planner's choice of the mean (taken where mbar is there and gram_fused holds)
    bool update_around = false;             // fused update: momentum and parameters go around the memory-side cache
    bool stream_hints = false;              // see Tuning::stream_hints
    bool gram_fused = false;                // Cholesky-QR panels: one launch (k_gram_chol) instead of two (set at upload)
    int32_t max_n = 0;
    int64_t ws_ppart_floats = 0;            // workspace: partial P region (floats)
    int64_t ws_qpart_floats = 0;            // workspace: partial Q region, starts after partial P
    psgd::Tuning tuning;
    // one walk over M per iteration
    bool one_sweep = false;                 // taken (after the upload: the partial sums' memory is there)
    bool one_wide = false;                  // matrix-core plans: psgd_step's own walk (k_one_sweep_wide)
    bool iter_mean = false;                 // psgd_step_iterations, more than one: two walks over the mean, held in mbar, instead
    int32_t one_waves = 0;                  // wavefronts of a workgroup
    int32_t one_lds_bytes = 0;
    int64_t one_s_doubles = 0, one_bytes = 0;   // partial S, and partial S and Gram matrices: plan-owned
    double* one_part = nullptr;             // device
    std::vector<psgd::OneMat> one_mats;
    std::vector<psgd::OneTile> one_tiles;
    std::vector<psgd::SolveTile> solve_tiles;
    // resident path
    bool resident_ok = false;               // planner found a tiling that fits the chip
    int32_t res_strip_rows = 0;
    int32_t res_blocks = 0;
    int32_t res_vec_class = 0;
    std::vector<psgd::MatDesc> res_mats;    // same matrices, partial-sum layout of the resident tiling
    std::vector<psgd::RTile> res_tiles;     // res_blocks * 4 entries
    int32_t res_n_cntq = 0;                 // column-chunk arrival counters
    int32_t res_n_cnts = 0;                 // strip arrival counters
    int64_t res_ws_floats = 0;
    int64_t res_sync_words = 0;
    int64_t res_mail_slots = 0;             // 64-bit mailbox slots (plan-owned device memory)
    bool tables_built = false;
    bool uploaded = false;
    int device = -1;
    void* static_ws = nullptr;              // the library-owned workspace on that device (psgd_step_static)
    psgd::DeviceTables dev;
    std::string last_error;
    // per-kernel timing (benchmarks only)
    bool profiling = false;
    bool compress_marked = false;            // a compress call has recorded its events since profiling was switched on
    void* events[PSGD_N_KERNELS + 2] = {};   // hipEvent_t: before/after each kernel
    double kernel_ms[PSGD_N_KERNELS] = {};
    int64_t profiled_steps = 0;
};

namespace psgd {
// Algorithm 2's last two lines fused into the decompression: m <- lambda m + Delta', x <- x - gamma (Delta' + m),
// on buffers laid out like `out` (fp32); Delta' itself is then not stored.  mom == nullptr: plain decompression.
struct UpdateArgs {
    float* mom = nullptr;
    float* param = nullptr;
    float lr = 0.f;
    float lam = 0.f;
};
// host planner (psgd_plan.cpp)
psgd_status build_tables(psgd_plan* plan);
// lays the resident tiling out for a device that holds `max_blocks` workgroups at once (sets plan->resident_ok)
void build_resident(psgd_plan* plan, int64_t max_blocks);
// device side (psgd_kernels.hip)
psgd_status upload_tables(psgd_plan* plan);
void free_tables(psgd_plan* plan);
// add = false: one more subspace iteration on the update already held in err (grad is not read, err not written);
// with grad = nullptr the same right after a compress or iteration of the same call, on the same M
psgd_status launch_compress(psgd_plan* plan, const void* grad, float* err, float* q, float* p,
                            void* workspace, void* stream, bool add = true);
psgd_status launch_decompress(psgd_plan* plan, const float* p, const float* q, float* err,
                              const void* grad, void* out, void* workspace, void* stream,
                              const UpdateArgs& upd = UpdateArgs());
// psgd_compress in two walks over M, on a plan whose tables are on the device; grad = nullptr: M is what the call before left
psgd_status launch_two_walks(psgd_plan* plan, const void* grad, float* err, float* q, float* p, void* workspace, void* stream, bool add);
// P and the partial S and Gram matrices, then P_hat and Q from them (one walk over M)
psgd_status launch_one_sweep(psgd_plan* plan, const void* grad, float* err, const float* q, float* p, void* stream, bool add);
psgd_status launch_solve(psgd_plan* plan, float* q, float* p, const double* spart, const double* gpart, void* stream);
psgd_status launch_one_sweep_wide(psgd_plan* plan, const void* grad, float* err, const float* q, float* p, double* spart, double* gpart,
                                  void* stream);
psgd_status hr_step_wide(psgd_plan* plan, const void* grad, float* err, float* q, float* p, void* out, void* workspace, void* stream);
psgd_status one_sweep_prepare(psgd_plan* plan);   // once per plan, at the upload
psgd_status set_profiling(psgd_plan* plan, bool enable);
// workers: those that have partial Q of their own
psgd_status launch_q_reduce(psgd_plan* plan, float* ws, float* q, void* stream, int workers);
psgd_status finish_profiled_step(psgd_plan* plan);
psgd_status hr_compress(psgd_plan* plan, const void* grad, float* err, float* q, float* p, void* workspace,
                        void* stream, bool add);
psgd_status hr_decompress(psgd_plan* plan, const float* p, const float* q, float* err, const void* grad, void* out,
                          void* stream, const UpdateArgs& upd, bool add_g = false);
psgd_status launch_vector_mean(psgd_plan* plan, const void* grad, void* out, void* stream, const UpdateArgs& upd);
psgd_status check_plan(psgd_plan* plan, void* stream);
psgd_status static_workspace(psgd_plan* plan, void** ws);
// Appendix G baselines (psgd_sparse.hip): starts != nullptr: Random Block, else Random K with `indices`
psgd_status launch_sparse_step(psgd_plan* plan, const void* grad, float* err, const int64_t* starts,
                               const int64_t* indices, float* vals, void* out, void* stream);
psgd_status read_trace(psgd_plan* plan, uint64_t* out, int64_t capacity, int64_t* n_written);
psgd_status resident_check_device(psgd_plan* plan);
// Every whole step that is not the calls in sequence: the resident kernel; a matrix-core plan's one walk that stores no M (no update, one
// iteration, buffers that let it); several iterations on the stored mean.  What a plan has none of for this call runs as the calls do.
psgd_status launch_resident_step(psgd_plan* plan, const void* grad, float* err, float* q, float* p, void* out,
                                 void* workspace, void* stream, const UpdateArgs& upd = UpdateArgs(), int iterations = 1);
// The resident kernel's synchronisation words (units of unsigned), one 256-byte line each: an error word
// (a wait gave up), the epoch that tags this step's mailbox slots, the count of finished workgroups.
constexpr int kSyncLineWords = 64;
constexpr int64_t res_sync_err() { return 1 * kSyncLineWords; }
constexpr int64_t res_sync_epoch() { return 2 * kSyncLineWords; }
constexpr int64_t res_sync_done() { return 3 * kSyncLineWords; }
constexpr int64_t kResSyncWords = 4 * kSyncLineWords;
}  // namespace psgd

#endif
