// Internal declarations shared by the host scheduler and the kernel files.
// Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <vector>

#include "ng.h"

namespace ng {

typedef unsigned short bf16_t;   // raw bfloat16 bits

constexpr int kMaxS = 64;        // history slots
constexpr int kDotPartsMax = 256; // per-matrix partial sums of the Gram-row reduction
constexpr int kAdamPatchCols = 128; // columns of one transform+Adam workgroup patch (32 rows)
constexpr int kDynChunk = 96;    // per-step table entries uploaded per launch (by kernel argument)
constexpr int kSkinnyMaxRank = 16;   // fp32 layer sets with ranks up to this take the vector-ALU projection / update
constexpr int kSkinnyRows = 128;     // rows and columns of the gradient / weight one of their workgroups takes
constexpr int kSkinnyCols = 256;
constexpr int kStatePanelCols = 2048;   // columns per panel of a wide M, V or history slot (see state_panel)
// bits of the device's sticky status word: 1 solve (pivot / non-finite), 2 transform+Adam (non-finite),
// 4 Cholesky pivot of the refresh, 8 Ritz value among the leading r not positive (zero or NaN: the rows it is the norm
// of come from a factor of T plus a shift, so a gradient of too low a rank shows as a pivot, bit 4)
constexpr int kStatusNotConverged = 16;   // the Jacobi eigen-solve of a refresh ran out of sweeps
constexpr int kFactorMax = 256;   // largest order whose inverse Cholesky factor one workgroup computes in registers
constexpr int kJacobiBlock = 16;  // rows per block of the blocked Jacobi (a visit rotates a pair of blocks)

// Static per-matrix description, lives in the workspace (device) and in the handle (host).
struct MatDev {
    // m, n: dimensions of the problem the kernels see: the weight's for NG_SIDE_LEFT, swapped for
    // NG_SIDE_RIGHT (the transposed problem); ld_w / ld_g always describe the caller's row-major arrays
    int m, n, r, ldn;
    int side;
    int l;            // refresh sketch width
    int ldk;          // contraction length of PbT (m rounded up to 32)
    int ldr;          // contraction length of Pb (r rounded up to 32)
    int roct;         // ceil(r/8): octets of N in the bf16 layout
    long long ld_w, ld_g;
    long long slot_elems;   // elements from one history slot to the next: r * state_cols(ldn, pw)
    int pw;           // columns per panel of M, V and every history slot (== ldn: one panel, plain row-major)
    float* P;
    float* M;
    float* V;
    float* H;         // history ring; bf16 elements when StepScalars::hist_bf16 (same element offsets)
    double* K;        // s*s Gram
    double* w64;      // s
    float* w32;       // s
    void* N;
    bf16_t* Pb;       // [ldr/32][m][32]  bf16 copy of P,   k-blocked: (i, rho) at ((rho/32) m + i) 32 + rho%32
    bf16_t* PbT;      // [ldk/32][r][32]  bf16 copy of P^T, k-blocked: (rho, i) at ((i/32) r + rho) 32 + i%32
                      // (operands of the update / projection GEMMs: the 64 bytes one row gives to a 32-deep
                      // stage lie next to its neighbours', so a tile's stage is one run of whole cache lines)
    // Scratch of one step lies behind the per-step table (MatDyn[n_mats]) in one block: the three
    // offsets below are in bytes from the start of that table (the `dyn` argument of the kernels),
    // -1 where a matrix has none.  The block is the front of the caller's workspace for ng_step and
    // the library's own static device array for ng_step_static.
    long long dot_parts_off;   // double [kDotPartsMax][s]: partial sums of the Gram-row reduction
    int dot_nparts;      // workgroups of the Gram-row reduction for this matrix
    int dot_iters;       // grid-stride iterations per workgroup
    // refresh scratch (all in the workspace)
    float* Ya;        // [max(m,n)][l]
    float* Yb;        // [max(m,n)][l]
    float* Yc;        // [max(m,n)][l]
    bf16_t* Yp;       // third plane of the last basis (null: the matrix's gradient products run on the fp32 GEMM)
    long long yp_plane, yp_last;   // elements from one sketch plane to the next, those of the last basis (see sketch_plane)
    float* Bm;        // [l][ldn]   B = Q^T G; later the l x r rotation
    double* T;        // [lp][lp]   Gram matrix / Cholesky factor of orders above kFactorMax
    float* Linv;      // [lp][lp]   inverse Cholesky factor (float); during the Rayleigh-Ritz step the rows
                      //            that the Jacobi rotates
    double* ritz;     // [lp]
    int* order;       // [lp]
    int* jflag;       // [64] rotations of each Jacobi sweep
    float* carry;     // [r][ldn] scratch of the history carry-over (null unless enabled)
    // fp32 projection in row chunks (proj_chunks > 0): R is the sum of proj_chunks float planes
    // [proj_rows][ldn], which the Gram row adds up in chunk order on its way (or k_reduce_parts does)
    long long proj_parts_off;
    int proj_chunks, proj_rows;
    long long tail8_off;   // 8 bf16: the last gradient row's columns from the last multiple of 8 on,
                           // zero-padded (rewritten every step, see launch_upload_dyn)
    int lp;           // l rounded up to a whole number of Jacobi block pairs: order and row pitch of T, Linv
    // k_history: place of the matrix's HistoryLines in the step's scratch, and its tiles (0: see k_gram_row)
    long long hist_sync_off;
    int hist_tiles;
    unsigned long long clear_off;   // 16-byte units of the history rings before this matrix's, in the table's order (see ClearShare)
};

// Per-step values: uploaded into the step's scratch block by a tiny kernel that receives them by value.
struct MatDyn {
    const void* g;
    void* w;
    int head;      // slot written by this step
    int count;     // valid slots after the push
    float bc1, bc2;   // Adam bias corrections 1/(1-beta1^t), 1/sqrt(1-beta2^t)
};

struct DynChunk {
    MatDyn e[kDynChunk];
};

constexpr size_t kStaticScratchBytes = NG_STATIC_SCRATCH_BYTES;   // the library's own step scratch (ng_step_static)

// M, V and every history slot hold their r x ldn elements as column panels of pw columns: panel p
// (columns p pw .. p pw + pw - 1) is a row-major r x pw block, and the panels lie one after the other.
// pw == ldn is the plain row-major array.  Otherwise pw = kStatePanelCols, a multiple of every tile and
// patch width (a tile lies in one panel), and the last panel's columns from ldn on are padding: zero,
// never written, and skipped by the kernels that read an array flat.  A 2048-column panel gives 4-byte
// elements a row pitch of 8 KB, at which the streaming kernels run fastest (transform+Adam: 6.6 TB/s on
// 2048-column states against 5.8 TB/s on row-major 5472-column ones and 5.1 TB/s at a 5.5 KB pitch).
struct StatePanel {
    unsigned base;   // element offset of the panel inside the array
    int pitch;       // its row pitch
    int col0;        // its first column
    __host__ __device__ unsigned at(int row, int col) const { return base + (unsigned)row * (unsigned)pitch + (unsigned)(col - col0); }
};
__host__ __device__ inline StatePanel state_panel(int r, int pw, int col) {
    StatePanel sp;
    const int p = col / pw;
    sp.col0 = p * pw;
    sp.pitch = pw;
    sp.base = (unsigned)p * (unsigned)r * (unsigned)pw;
    return sp;
}
// columns an array of ldn columns occupies in panels of pw
__host__ __device__ inline int state_cols(int ldn, int pw) { return (ldn + pw - 1) / pw * pw; }

// The same arrays read flat, V elements per 16-byte vector: the r * ldn / V vectors that hold the
// columns below ldn, numbered in storage order; position q lies at vector at(q) of the array.
struct FlatState {
    unsigned whole;      // vectors before the last panel (stored without gaps)
    unsigned row_valid;  // vectors per row of the last panel that hold columns below ldn
    unsigned row_pitch;  // vectors per stored row of the last panel
    unsigned count;      // r * ldn / V
    __host__ __device__ unsigned at(unsigned q) const {
        if (q < whole || row_valid == row_pitch) return q;
        const unsigned k = q - whole, row = k / row_valid;
        return whole + row * row_pitch + (k - row * row_valid);
    }
};
__host__ __device__ inline FlatState flat_state(int r, int ldn, int pw, int V) {
    FlatState f;
    const int last0 = (ldn - 1) / pw * pw;   // first column of the last panel
    f.whole = (unsigned)last0 / (unsigned)V * (unsigned)r;
    f.row_valid = (unsigned)(ldn - last0) / (unsigned)V;
    f.row_pitch = (unsigned)pw / (unsigned)V;
    f.count = (unsigned)r * (unsigned)ldn / (unsigned)V;
    return f;
}

// address inside the step's scratch block, which starts with the per-step table
template <typename T>
__device__ __forceinline__ T* step_scratch(const MatDyn* dyn, long long off) {
    return reinterpret_cast<T*>(reinterpret_cast<char*>(const_cast<MatDyn*>(dyn)) + off);
}

// What the workgroups of one matrix share in k_history, kHistoryLines lines per matrix; zeroed at the start of every step, as
// are the bits behind them (one per tile: left to the workgroup that solves).  A workgroup counts itself in and looks for w
// in line (tile mod kHistoryLines): hundreds of them on one line took turns there (4 to 9 ns a tile for the count alone).
struct HistoryLine {
    unsigned long long w[16];         // solved weights: the float, marked by a 1 above it (3: tiles have been left)
    unsigned long long arrived_late;  // tiles of this line whose partial sums are in memory, and above, whether one was left
    unsigned full;                    // line 0: lines whose tiles have all arrived
    unsigned state;                   // line 0: kSolverGone or kAllThere, whichever came first
    unsigned started;                 // workgroups of this line's tiles (and in line 0 the solver) that have started
    unsigned pad[27];
};
static_assert(sizeof(HistoryLine) == 256, "two cache lines");
constexpr int kHistoryLines = 8;
constexpr unsigned kSolverGone = 1, kAllThere = 2;
constexpr unsigned kHistoryWait = 10000;   // 100 us, several times what the largest matrix takes to arrive
constexpr unsigned kHistoryPatience = 100; // times that end any wait
// Whether a tile that waits is left at its look number `looks` (from 0): see wait_for_weights in k_history.hip
__host__ __device__ inline bool history_leaves(unsigned tile, unsigned not_started, unsigned looks) {
    return looks + 1 >= kHistoryPatience || tile < not_started << (looks < 16 ? looks : 16);
}
// Items of k_history (TileRef): a tile (its first row and column, and in `pad` log2(bands) << 2 | tile << 4), or the solver of a
// matrix.
enum { kHistoryTile = 0, kHistorySolve = 1 };

struct StepScalars {
    float lambda;
    float beta1, beta2, eps;
    float lr_scale, lr_wd;
    int adam_mode;
    int s;               // slots read by the kernels (>= 1; the s = 0 case uses one scratch slot)
    int use_fisher;      // 0 when hparams.s == 0
    int hist_bf16;       // history slots are bf16 (else float)
    int norm_count;      // Fisher normaliser 1/count (valid slots) instead of 1/s
    int slot;            // history slot an OP_CARRY_SLOT product works on
    int planes;          // sketch planes that an OP_APPLY_* product stores (sketch_plane); 0: none
    int planes_only;     // ... and not its float result
};

// Plane q of the sketch that a product with the gradient reads, [rows / 8][l][8] bf16, rows past the last zero.  The planes lie
// in sketch buffers that are free while they live: two of the random matrix or of a basis inside the subspace iteration in Yc,
// the third in Bm, which the product B = Q^T G fills later.  The last basis comes from Yc and goes to Ya as floats too, and
// that product reads its planes: they lie in Yb, the third behind the others where Yb is long enough (n from about 3/2 m
// on), else in memory of its own, 2 bytes per element of Q.  (Planes of their own took 6 bytes per element of
// max(m, n) x l, 35 % of the workspace; this is 4 to 8 %.)
__host__ __device__ inline bf16_t* sketch_plane(const MatDev& md, bool last, int q) {
    if (q == 2) return last ? md.Yp : (bf16_t*)md.Bm;
    return last ? (bf16_t*)md.Yb + q * md.yp_last : (bf16_t*)md.Yc + q * md.yp_plane;
}

// Grouped-launch work item: which matrix and which tile / part of it a workgroup takes.
// mat < 0 marks a padding entry (the workgroup exits).
struct TileRef {
    int mat;
    int ti, tj;
    int pad;
};

// Host side: the order in which a grouped GEMM launch's tile table lists the tiles (ng_api.hip).
void xcd_order(const std::vector<TileRef>& logical, const std::vector<int>& cost, std::vector<TileRef>* out);

// Left-side projection tiles of a gradient with at least 8 columns take the direct-to-LDS kernel.  It
// reads whole 16-byte chunks; the one chunk per row that straddles the last column (n % 8 != 0) reads up
// to 7 elements past the row's end, which is the start of the next row or its padding: inside the
// caller's buffer for every row but the last, whose chunk comes from MatDev::tail8 instead.
__host__ __device__ inline bool projection_tile_direct(int n) { return n >= 8; }

// ---------------------------------------------------------------- launchers
// Every launcher enqueues on `stream` and returns hipGetLastError().

// mats != null: also refresh MatDev::tail8 of the left-side matrices from the bf16 gradients in the chunk
// zero_bytes (a multiple of 16) from byte zero_off of the block that the table starts are cleared
hipError_t launch_upload_dyn(MatDyn* table, const DynChunk& chunk, int first, int n, const MatDev* mats,
                             size_t zero_off, size_t zero_bytes, hipStream_t stream);
hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t stream);   // bytes % 4 == 0
// zero the history ring and the Gram block of every matrix (buffer sizes as ng_query_sizes reports them)
hipError_t launch_clear_history(const MatDev* mats, int n_mats, int s, int h_elem_bytes, size_t k_bytes,
                                hipStream_t stream);

// fp32 grouped GEMM with selectable operands (k_gemm_f32.hip)
enum GemmOp {
    OP_PROJECT_F32 = 0,   // R(slot head) = P^T G                     (step, NG_F32)
    OP_UPDATE_F32,        // W -= lr*(scale * P N + wd W)             (step, NG_F32)
    OP_G_B2A,             // Ya = G Yb     (m x l)
    OP_G_C2A,             // Ya = G Yc
    OP_GT_C2B,            // Yb = G^T Yc   (n x l)
    OP_GRAM_A,            // Ya^T Ya   (rows m) -> partial planes, see sym_planes
    OP_GRAM_B,            // Yb^T Yb   (rows n)
    OP_GRAM_CA,           // Yc^T Yc   (rows m)
    OP_GRAM_CB,           // Yc^T Yc   (rows n)
    OP_APPLY_A2C,         // Yc = Ya Linv^T (rows m)
    OP_APPLY_B2C,         // Yc = Yb Linv^T (rows n)
    OP_APPLY_C2A,         // Ya = Yc Linv^T (rows m)
    OP_APPLY_C2B,         // Yb = Yc Linv^T (rows n)
    OP_QT_G,              // Bm = Ya^T G   (l x ldn)
    OP_B_BT,              // Bm Bm^T   (l x l) -> partial planes
    OP_ROTATE,            // P = Ya * Urot (m x r), Urot (l x r floats) staged in Bm
    OP_GRAM_P,            // P^T P (r x r) -> partial planes
    OP_APPLY_P2A,         // Ya[m][r] = P Linv^T
    OP_T_CARRY,           // Linv (r x r, float) = P^T Yc, Yc holding the previous projector
    OP_CARRY_SLOT,        // carry (r x ldn) = Linv * H[slot]
    OP_COUNT
};
void gemm_f32_dims(int op, const MatDev& md, int* M, int* N, int* K);

// A symmetric product C = X^T X is left as `count` float planes [order][order], `pitch` apart, one per run of the
// contraction, lower tiles only: C(i, j) is their sum, which the kernel that reads it forms in fp64.  A run is
// about `chunk` long and never longer than half of the contraction, whatever else is in the layer set: one run of
// 2048 rows instead of two of 1024 left the column norms of the 1.1B set's projectors 6.4e-7 from 1 (rms) instead of
// 4.0e-7, one of 600 instead of 304 (600 x 600, rank 512) 3.3e-7 instead of 1.8e-7.
// The planes lie in the sketch buffer that is free at that point of the refresh ([max(m,n)][l] floats): Ya
// while Yb is orthonormalised and for the new projector's Gram matrix, Yb otherwise.  An order above half of its
// rows leaves room for one plane there; the second then goes to the head of another buffer that is free: the sketch
// buffer that the next product fills (while an orthonormalisation runs), Yc for B B^T, and Bm once the
// rotation staged in it has been applied.  Each holds at least order^2 floats, because order <= l <= m, n.
constexpr int kSymPlanesMax = 8;
constexpr int kSymStep = 16;       // runs are whole multiples of this; a contraction up to this long is not cut
struct SymPlanes {
    float* p;
    int order, count;
    long long pitch;               // floats from one plane to the next
};
// planes that a contraction of length k is cut into where there is room
inline int sym_plane_count(int k, int chunk) {
    const int least = k > kSymStep ? 2 : 1, want = (k + chunk - 1) / chunk;
    return want < least ? least : want < kSymPlanesMax ? want : kSymPlanesMax;
}
inline SymPlanes sym_planes(int op, const MatDev& md, int chunk) {
    SymPlanes s;
    s.p = (op == OP_GRAM_B || op == OP_GRAM_CB || op == OP_GRAM_P) ? md.Ya : md.Yb;
    s.order = op == OP_GRAM_P ? md.r : md.l;
    const int k = (op == OP_GRAM_A || op == OP_GRAM_CA || op == OP_GRAM_P) ? md.m : md.n;
    const int rows = md.m > md.n ? md.m : md.n;
    const int room = rows / s.order;       // (order <= l: at least this many)
    s.count = sym_plane_count(k, chunk);
    s.pitch = (long long)s.order * s.order;
    if (s.count > room && room > 1) s.count = room;
    if (s.count > room) {
        const float* second = op == OP_GRAM_P ? md.Bm : op == OP_GRAM_CA ? md.Ya : op == OP_GRAM_CB ? md.Yb : md.Yc;
        s.count = 2;
        s.pitch = second - s.p;
    }
    return s;
}
// The kernels read it from a table [kSymOps][n_mats] in the workspace, `sym` being a product's row of it.  (Formed in the
// kernels, the divisions and the choice of buffers were 7 us of a refresh of the 60M set; as members of MatDev, its
// longer stride was 0.5 us of the step of three mid-size matrices.)
constexpr int kSymOps = 6;
inline int sym_index(int op) {      // -1: not a symmetric product
    return op >= OP_GRAM_A && op <= OP_GRAM_CB ? op - OP_GRAM_A : op == OP_B_BT ? 4 : op == OP_GRAM_P ? 5 : -1;
}

// whether a product takes the 128 x 128 tile; arguments as launch_gemm_f32
bool f32_tile_large(GemmOp op, int max_m, int max_n, int max_k, long long tiles, int max_split);

// max_m, max_n, max_k: largest dimensions of the product over the layer set, tiles: its 128 x 128 tiles, each piece of a cut
// contraction counted (grid and tile choice)
// max_split: largest number of pieces that a matrix's contraction is cut into, 0 or 1 for none (symmetric products:
// SymPlanes::count, the projection: MatDev::proj_chunks); sym: symmetric products only
// planeless: only the matrices without sketch planes (a product with the gradient, the others having gone through
// launch_sketch_product; the dimensions are then theirs)
hipError_t launch_gemm_f32(GemmOp op, const MatDev* mats, const MatDyn* dyn, int n_mats,
                           int max_m, int max_n, int max_k, long long tiles, int grad_dtype, StepScalars sc,
                           int max_split, const SymPlanes* sym, int sides, bool planeless, hipStream_t stream);

// bf16 MFMA GEMMs of the step (k_gemm_bf16.hip)
// which: 0 projection (direct-to-LDS kernel), 1 update, 2 projection (register-staged kernel)
// tiles4: 256 x 256 tiles of the left-side projection over the layer set
void bf16_tile_shape(int which, int max_r, long long tiles4, int* bm, int* bn);
// zero16: 16 bytes of zeros in device memory (fetched in place of out-of-range operand chunks)
// The projection's tile table has three runs, each with its own kernel: n_direct left-side tiles for
// the direct-to-LDS kernel (see projection_tile_direct), then n_staged other left-side tiles, then
// n_right right-side tiles.
hipError_t launch_project_bf16(const MatDev* mats, const MatDyn* dyn, const TileRef* tiles, int n_direct,
                               int n_staged, int n_right, int max_r, long long tiles4, int hist_bf16,
                               const void* zero16, hipStream_t stream);
// sides: bit 0 = left-side matrices present, bit 1 = right-side ones (one kernel instance each)
hipError_t launch_update_bf16(const MatDev* mats, const MatDyn* dyn, const TileRef* tiles, int n_tiles,
                              StepScalars sc, const void* zero16, int sides, hipStream_t stream);

// Refresh products of a bf16 gradient with an fp32 sketch matrix Y, held as bf16 planes (sketch_plane), on the bf16 MFMA;
// left side, at least 8 columns.  form 1: Ya = G Y, form 2: Yb = G^T Y, form 3: Bm = Y^T G; planes: how many of Y's three
// planes enter (form 1: 1 to 3, form 2: 2 or 3, form 3: 3).  tiles: ti counts kSketchTileG rows or columns of the
// gradient, tj kSketchTileL sketch columns.
constexpr int kSketchTileG = 128, kSketchTileL = 128;
hipError_t launch_sketch_product(int form, int planes, const MatDev* mats, const MatDyn* dyn, const TileRef* tiles,
                                 int n_tiles, const void* zero16, hipStream_t stream);

// Projection and update of fp32 layer sets with ranks <= kSkinnyMaxRank, left side (k_skinny.hip).
// tiles: one entry per kSkinnyRows x kSkinnyCols block of the m x ldn range of every matrix; rk: 4, 8
// or 16, at least the largest rank of the set (the rows of a chunk, MatDev::proj_rows).
// stream_past: gradient and weight are read and written past the caches
hipError_t launch_project_skinny(const MatDev* mats, const MatDyn* dyn, const TileRef* tiles, int n_tiles, int rk,
                                 bool stream_past, hipStream_t stream);
// ring slot `head` of every matrix <- the sum of its projection's row chunks
hipError_t launch_reduce_parts(const MatDev* mats, const MatDyn* dyn, int n_mats, int max_ldn, int max_r, hipStream_t stream);
hipError_t launch_update_skinny(const MatDev* mats, const MatDyn* dyn, const TileRef* tiles, int n_tiles, int rk,
                                StepScalars sc, bool stream_past, hipStream_t stream);

// Gram row, solve, fused transform + Adam (k_elementwise.hip)
// parts: the projection left row chunks (MatDev::proj_chunks), which this kernel adds up into the slot
// row_override >= 0: the Gram row of that slot instead of the step's head (history carry-over);
// launch_solve then only stores the row and column of K and skips the solve
hipError_t launch_gram_row(const MatDev* mats, const MatDyn* dyn, const TileRef* chunks, int n_chunks,
                           int s, int hist_bf16, bool parts, int row_override, hipStream_t stream);
hipError_t launch_solve(const MatDev* mats, const MatDyn* dyn, int first, int n_mats, StepScalars sc,
                        int row_override, int* status, hipStream_t stream);
// Both passes over the history in one launch, s <= 16 (k_history.hip).  wait_ticks: 100 MHz ticks that a workgroup waits for
// its matrix's weights before it leaves its tile to the one that solves.
// history_shape: rows of a lane, columns of a wavefront, and the most tiles of a matrix that goes this way
void history_shape(int s, int hist_bf16, int bf16_n, int* lane_rows, int* wave_cols, int* most_tiles);
hipError_t launch_history(const MatDev* mats, const MatDyn* dyn, const TileRef* items, int n_items, StepScalars sc,
                          int grad_dtype, unsigned wait_ticks, int* status, hipStream_t stream);
hipError_t launch_save_projector(const MatDev* mats, int n_mats, hipStream_t stream);   // Yc <- P
hipError_t launch_carry_store(const MatDev* mats, int n_mats, int slot, int hist_bf16, hipStream_t stream);
hipError_t launch_transform_adam(const MatDev* mats, const MatDyn* dyn, const TileRef* patches, int n_patches,
                                 StepScalars sc, int grad_dtype, int* status, hipStream_t stream);
hipError_t launch_make_bf16_copies(const MatDev* mats, int n_mats, int max_m, int max_r, hipStream_t stream);

// Ritz value from the sum of its row's squares; -1 for NaN (non-finite gradient), behind every number, so that the places
// are a permutation whatever the rows hold and every entry of the order written from them is an index (with NaN
// comparing false, all NaN values had place 0 and the other entries kept what the workspace held).
__host__ __device__ inline double ritz_value(double sum) { return sum >= 0.0 ? sqrt(sum) : -1.0; }
// Place of value i among n, largest first and equal ones by index.
__host__ __device__ inline int ritz_place(const double* v, int n, int i, int first = 0, int step = 1) {
    const double vi = v[i];
    int place = 0;
    for (int j = first; j < n; j += step) {
        const double vj = v[j];
        place += (vj > vi) || (vj == vi && j < i);
    }
    return place;
}

// Part `part` of `parts` of clearing the history ring of every matrix (and, in the first, the Gram blocks), done by extra
// workgroups of a launch that leaves units and memory idle; parts == 0: none.  units: 16-byte units of all rings.
struct ClearShare {
    int part, parts, blocks;
    unsigned long long units, k_bytes;
};
// The units [lo, hi) that workgroup `block` of a part clears: all rings in a row, cut evenly, whatever the matrices' sizes, at
// whole cache lines (refresh of the 350M set 11.99 ms, cut anywhere 12.19).
__host__ __device__ inline void clear_range(const ClearShare& cs, int block, unsigned long long* lo, unsigned long long* hi) {
    const unsigned long long a = cs.units * (unsigned)cs.part / (unsigned)cs.parts, n = cs.units * (unsigned)(cs.part + 1) / (unsigned)cs.parts - a;
    *lo = (a + n * (unsigned)block / (unsigned)cs.blocks) & ~15ull;
    *hi = (a + n * (unsigned)(block + 1) / (unsigned)cs.blocks) & ~15ull;
}

// refresh helpers (k_refresh.hip)
// fills Yb (n x l), or, where a matrix has sketch planes, the first of them with the same values rounded to bf16
hipError_t launch_fill_gaussian(const MatDev* mats, int n_mats, int max_rows, bool planes, unsigned long long seed,
                                unsigned long long call_id, hipStream_t stream);
// Linv = inverse Cholesky factor of the symmetric product `op` (its planes, plus shift_rel * trace on the
// diagonal).  clear: beside orders up to kFactorMax only
hipError_t launch_inverse_factor(GemmOp op, const MatDev* mats, const SymPlanes* sym, int n_mats, int max_order,
                                 double shift_rel, ClearShare clear, int* status, hipStream_t stream);
// X <- X L^{-T}, X^T X + shift_rel * trace on the diagonal = L L^T, for sketches of up to 32 columns and kOrthoRows rows
// in one launch: Ya or Yb into Yc (passes 1) or, by a second, unshifted pass, back into Ya (passes 2); P into Ya.  planes:
// sketch planes of a result, which take the place of a single pass's floats (matrices that have them)
enum { kOrthoA, kOrthoB, kOrthoP };
// A workgroup takes a matrix's rows 256 at a time: against the three launches per pass, whose products have a workgroup for
// every 64 rows, refreshes of one n x n matrix at l = 32 took 280 us for 342 (256 x 512) and 464 for 471 (n = 1024), of
// 72 of n = 768 at l = 16 679 for 762; beyond, 693 for 662 (n = 2048) and 1206 for 1048 (n = 4096), with fp32 in every basis.
constexpr int kOrthoRows = 1024;
hipError_t launch_orthonormalise_small(int which, int passes, double shift_rel, int planes, const MatDev* mats, int n_mats,
                                       ClearShare clear, int* status, hipStream_t stream);
// extra workgroups of those launches that clearing is to have, bytes in each launch; 0 where it is better elsewhere
int clear_share_blocks(int n_mats, int max_order, int max_pairs, unsigned long long bytes);
// the rows that the Jacobi starts from: L^T of T = B B^T = L L^T (planes of OP_B_BT)
hipError_t launch_jacobi_prepare(const MatDev* mats, const SymPlanes* sym, int n_mats, int max_l, int max_lp, int* status,
                                 hipStream_t stream);
// up to `sweeps` (1 .. 64) sweeps over every matrix, each matrix until one of its sweeps rotates nothing
// clear.parts != 0: something is to be cleared; *cleared tells whether it was
hipError_t launch_jacobi(const MatDev* mats, int n_mats, int max_pairs, int sweeps, ClearShare clear, bool* cleared, hipStream_t stream);
hipError_t launch_jacobi_finish(const MatDev* mats, int n_mats, int sweeps, int* status, hipStream_t stream);
// whether the kernel that fixes the signs also makes the bf16 copies (of a bf16 layer set)
bool sign_fix_copies(int n_mats, int max_m, int max_r);
hipError_t launch_sign_fix(const MatDev* mats, int n_mats, int max_r, bool copies, hipStream_t stream);

// micro-benchmarks (k_microbench.hip)
hipError_t launch_mb_copy(const void* src, void* dst, size_t bytes, hipStream_t stream);
hipError_t launch_mb_read(const void* src, size_t bytes, void* sink, hipStream_t stream);
hipError_t launch_mb_mfma(int iters, int waves_per_simd, bool random_operands, void* sink, double* flops,
                          hipStream_t stream);

}  // namespace ng
