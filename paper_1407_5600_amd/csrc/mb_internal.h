// Internal state of the multiblob library: grid handle, spring table, FFT
// plans, tile geometry and the per-kernel timing hooks.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "../../include/multiblob.h"

namespace mb {

// Stable kernel ids (reported by the timing interface).
enum KernelId : int {
    K_BIN_COUNT = 0,
    K_SCAN_REDUCE,
    K_SCAN_APPLY,
    K_SPRINGS_SCATTER,
    K_BIN_SCATTER,
    K_SPRINGS,
    K_SPREAD,
    K_FFT_X_FWD,
    K_FFT_Y_FWD,
    K_FFT_Z_SPECTRAL,
    K_FFT_Y_INV,
    K_FFT_X_INV,
    K_INTERP,
    K_INTERP_STEP,
    K_U0,    // particle means and reordering at the end of a call
    K_DIAG,  // the same with the diagnostics
    K_FOLD,
    K_INTERP_GRAD,
    K_SPRINGS_ADJ,
    K_FFT_XY_INV,
    K_NUM
};

// Spring table of the particle template on the device: the pair list and,
// per blob, its incident pairs with the pair's other blob.
struct SpringsDev {
    const int* pa;          // [npairs]
    const int* pb;          // [npairs]
    const double* r0;       // [npairs]
    const int* adj_start;   // [nb + 1]
    const int* adj_pair;    // [2 * npairs] pair << 8 | other blob of the pair
    double k;
    int nb;
    int npairs;
    int ppb;                // particles per block of the springs kernels
};

// Tile geometry for spreading and interpolation.
// Tiles are numbered box-tile major: the 2^(lfx+lfy+lfz) tiles of one
// spreading box tile (2^lfx along x, ...) are consecutive, x fastest within
// it, and the box tiles (nbx x nby x ...) follow one another x fastest, so a
// box tile's blobs form one range of the tile-sorted records.  For the box
// tiles themselves (and any tiles not grouped) lfx = lfy = lfz = 0, nbx =
// ntx, nby = nty: plain x-fastest order.
struct Tiles {
    int tx, ty, tz;     // tile extent in cells
    int ntx, nty, ntz;  // tiles per axis
    int n;              // tiles per box
    int remap;          // 1: XCD-aware block -> tile mapping
    int nbox;           // boxes of the grid (a batch of equal boxes)
    int lfx, lfy, lfz;  // log2 of the tiles per box tile along each axis
    int nbx, nby;       // box tiles along x and y
};


// Tile shapes (tx, ty, tz) with instantiated spreading and interpolation
// kernels: the LDS of the float32 interpolation (three components of the
// (tx+3)(ty+3)(tz+3) box) stays under 64 KB.
#define MB_TILE_SHAPES(X) X(16, 8, 8) X(8, 8, 8) X(32, 8, 8) X(16, 16, 8) X(16, 8, 16) X(8, 16, 16)

bool tile_shape_supported(int tx, int ty, int tz);
// A spreading kernel exists for box tiles of sx x sy x sz cells made of
// binning tiles of tx x ty x tz.
bool box_shape_supported(int sx, int sy, int sz, int tx, int ty, int tz);

struct TimerPair {
    hipEvent_t a, b;
    int id;
};

}  // namespace mb

struct mb_springs {
    int nb;
    int npairs;
    int ppb;
    double k;
    int device;
    int* d_pa;
    int* d_pb;
    double* d_r0;
    int* d_adj_start;
    int* d_adj_pair;
};

struct mb_grid {
    mb_grid_desc d;
    int device;
    // workspace: every O(N) and O(M) scratch buffer below (tables to force
    // partials and the non-finite flag) lies in this one region
    void* ws;           // null until a workspace is set (external_workspace)
    size_t ws_bytes;
    size_t zero_off;    // the workspace is zeroed from here on
    bool ws_owned;      // allocated by the library (freed at destroy)
    int* d_flag;        // [0] non-finite flag (check_finite; bit 2: a springs
                        // block gave up waiting for the offsets), [1] the
                        // fused scan's published launch number
    uint32_t scan_epoch;  // launches of kernels with the fused scan
    bool scan_unchecked;  // one since the flag was last read
    double* d_qint;     // [max_blobs][3] positions in the step calls' particle order
    double* d_pint;     // [max_blobs][3] per-particle forces, same order
    int* d_order;       // [max_blobs] caller's particle of each internal particle
    int ntiles_cap;     // tiles per box the workspace holds (all shapes)
    int L, NC;          // cells per side, complex columns L/2 + 1
    int64_t N;          // L^3 (cells of one box)
    size_t fsz;         // bytes per scalar (8 or 4)
    // FFT
    void* d_tw;         // twiddles W_L^k, k < L (cplx<T>)
    void* d_dsym;       // D symbol per mode index: (1 - e^{-2 pi i m / L}) / h
    void* d_d2;         // |D symbol|^2 per mode index (T)
    void* d_spec;       // [3][L(z)][NC(kx)][L(ky)] cplx<T>
    int nblk_x;         // blocks of an x pass
    unsigned char* d_act;  // [nbox][L] z planes holding a force: set by the binning of a
                           // masked steady solve, cleared by its last pass
    double* d_psum;     // [nblk_x][2] per-block sums of v and f (float64)
    // binning (by tile)
    int* d_count;       // [tiles] (kept zeroed between uses)
    int* d_offs;        // [tiles + 1]
    int* d_bsum;        // scan block sums
    int nscan;          // scan blocks
    int* d_tile;        // [max_blobs] tile of each blob; small boxes: blob of each record
    int* d_rank;        // [max_blobs] place among its tile's blobs; small boxes: [nbox] exponent
                        // of each box's fixed-point force sums
    int* d_perm;        // [max_blobs] blob of each sorted record
    int64_t perm_m;     // d_perm is a permutation of [0, perm_m) (-1: none; small boxes leave it)
    bool own_capture;   // mb_step_graph is capturing a step
    bool replayed;      // a caller captured a call: its replays write d_perm unseen
    bool binned_small;  // the last binning was by box (small_boxes)
    void* d_rec;        // [max_blobs] records
    size_t rec_size;
    mb::Tiles tiles;       // binning, spreading and interpolation tiles
    mb::Tiles btiles;      // spread box tiles: whole numbers of tiles per axis
    void* d_box;           // [3][tiles][box nodes] spread boxes of the step
    double* d_u;           // [max_blobs][3] blob velocities of the last step
    double* d_adj;         // reverse-step scratch (allocated on first use)
    double* d_adj_part;    // per-block k / r0 derivative sums (deterministic)
    size_t adj_part_cap;   // doubles in d_adj_part
    double* d_mid;         // midpoint scheme: q* and a velocity per blob (first use)
    int scheme;            // mb_scheme of the steps
    double* d_tile_part;   // [tiles][4]  (sum v_a, max |Dv|)
    double* d_force_part;  // [force blocks][3]
    // timing
    uint32_t timing;    // bit mask of timed kernel ids
    std::vector<mb::TimerPair> pending;
    std::vector<hipEvent_t> free_events;
    double acc_ms[mb::K_NUM];
    int64_t acc_n[mb::K_NUM];
};

namespace mb {

// Timing of a launch of kernel `id` (when timing is enabled for it): two
// events, queued for mb_grid_kernel_times, that the launch itself records
// at its start and end (hipExtLaunchKernel), so the duration is the
// kernel's execution without the gaps around it.  False: not timed.
bool timer_pair(mb_grid* g, int id, hipEvent_t* start, hipEvent_t* stop);

#define MB_LAUNCH(g, id, s, kern, grid, block, shm, ...)                          \
    do {                                                                          \
        hipEvent_t a_ = nullptr, b_ = nullptr;                                    \
        if (::mb::timer_pair((g), (id), &a_, &b_))                                \
            hipExtLaunchKernelGGL(kern, dim3(grid), dim3(block), (shm), (s), a_, b_, \
                                  0, __VA_ARGS__);                                \
        else                                                                      \
            hipLaunchKernelGGL(kern, dim3(grid), dim3(block), (shm), (s),         \
                               __VA_ARGS__);                                      \
    } while (0)

// Blocks of an x pass of the FFT solve (one float64 partial sum pair each).
int fft_x_blocks(int L, int precision);

// Workspace set-up on stream s: the FFT twiddle and symbol tables (computed
// on the device), zeroed tile counts, partial sums and non-finite flag.
hipError_t init_workspace(mb_grid* g, hipStream_t s);
// Zero n 32-bit words at p (a kernel, never a memset node in a graph).
hipError_t zero_words(void* p, size_t n, hipStream_t s);

// Launchers (templated on the field scalar type, float or double).  Each
// returns hipSuccess or the launch error.
// Tile, rank and counting sort of the blobs at q; with counted the counts,
// tiles and ranks are already in place (the previous step's interpolation
// binned these positions) and only the scan runs.
// scan: also the scan of the counts into offsets (else the springs kernel
// of the step does it: scatter_springs with scan).
template <typename T>
hipError_t bin_blobs(mb_grid* g, int64_t M, const double* q, hipStream_t s,
                     bool counted = false, bool scan = true);
// Binning and records of the blobs at q (tiles false: records of small boxes
// need not be by tile) with forces F (nullable: none) scaled
// by fscale (h^-3 when fscale <= 0: a force density); with Fsum the forces
// are F2 + f2scale F (F2 nullable), also stored there.
template <typename T>
hipError_t bin_records(mb_grid* g, int64_t M, const double* q, const double* F, hipStream_t s,
                       bool tiles, double fscale = 0.0, const double* F2 = nullptr, double f2scale = 0.0,
                       double* Fsum = nullptr);
// Boxes of so few blobs (and tiles) that one block bins a box in LDS, the
// solve forms their force from the records without spreading, and the
// interpolation gathers from the field directly; with sp also the box's
// particles have to fit a block of the springs kernels.  More than a blob to four
// cells is not few (only an 8^3 box: 512 of them with 247 blobs each, steady
// flow, 89 us a step against 74 through the boxes of tiles).  Independent of the
// number of boxes, so that a batch steps as its boxes would alone.
constexpr int kSmallBlobs = 256;
constexpr int kSmallTiles = 4096;  // 16 KB of LDS counts
constexpr int kMaxTileCells = 2048;  // largest of MB_TILE_SHAPES
// Edges whose boxes can be small (up to 192): only they have the kernels of the path.
constexpr bool small_edge(int L) { return (int64_t)L * L * L <= (int64_t)kSmallTiles * kMaxTileCells; }
constexpr int kExpNonfinite = 1 << 20;  // box exponent: a force of the box is not finite
bool small_boxes(const mb_grid* g, int64_t M, const SpringsDev* sp);
// Springs and records of small boxes, with tiles by tile (for the spreading and
// the interpolation that forms sums over the tiles); mark: also the z planes
// their nodes lie in (d_act).
template <typename T>
hipError_t bin_springs(mb_grid* g, const SpringsDev& sp, int64_t P, const double* q,
                       const double* Fext, hipStream_t s, const double* Gblob, bool force_sums,
                       bool tiles, bool mark);
// Non-finite flag of the grid's checks (null unless check_finite).
inline int* finite_flag(mb_grid* g) { return g->d.check_finite ? g->d_flag : nullptr; }
// Springs and records; force_sums: also the per-block sums of the blob
// forces read by the diagnostics.
// scan: block 0 of the kernel first scans the tile counts (left by the
// binning, bin_blobs with scan = false) into the offsets the others wait for;
// only where fused_scan_ok.
template <typename T>
hipError_t scatter_springs(mb_grid* g, const SpringsDev& sp, int64_t P,
                           const double* q, const double* Fext, hipStream_t s,
                           const double* Gblob = nullptr, bool force_sums = true,
                           bool scan = false);
// The scan can ride in the kernel that places the records: at most `tiles`
// tiles (kFusedTiles, a single scan block's worth, in the springs kernel, whose
// blocks have forces to form meanwhile; kFusedScatterTiles in the scattering
// kernel, where the others wait for all of it: 1,300 blobs in each of 48 32^3
// boxes, 1,536 tiles, an interpolation 32.3 -> 31.4 us, 64 boxes 38.9 -> 40.1;
// 128^3, 2,048 tiles, 79,000 blobs 28.2 -> 30.6) and a stream not being captured
// (a captured launch would replay its launch number; d_flag[1] is zeroed with the
// workspace, launch numbers start at 1).
constexpr int kFusedTiles = 4096;
constexpr int kFusedScatterTiles = 1536;
bool fused_scan_ok(mb_grid* g, hipStream_t s, int tiles);
// Called (by fused_scan_ok) before a binning by tile: whether the stream is being
// captured.  Where it is, by the caller, the order of the blobs that the grid keeps
// is no more used: each replay writes d_perm, for its number of blobs, without the
// grid seeing it, and an order taken into the graph would be read there whatever has
// become of it by then.  (The graph of mb_step_graph lives within its call.)
bool note_capture(mb_grid* g, hipStream_t s);
// Blob of each record of the last binning.
inline int* record_blobs(mb_grid* g) { return g->binned_small ? g->d_tile : g->d_perm; }
hipError_t spring_forces(const SpringsDev& sp, int64_t P, const double* q,
                         const double* Fext, double* F, hipStream_t s,
                         mb_grid* timing_grid, const double* Gblob = nullptr);
// qbar += (dF/dq)^T Fbar; kbar, r0bar (nullable) accumulate the k and rest
// length parts; fsum (nullable) += Fbar.
hipError_t springs_adjoint(const SpringsDev& sp, int64_t P, const double* q,
                           const double* Fbar, double* qbar, double* kbar,
                           double* r0bar, hipStream_t s, mb_grid* timing_grid,
                           double* part = nullptr, double* fsum = nullptr);
// Doubles of per-block partial sums springs_adjoint writes to `part`
// (then summed in block order) instead of its float64 atomics.
size_t springs_adjoint_part_size(const SpringsDev& sp, int64_t P);
// out = (a ? a : 0) + sc b; y += x (n doubles).
hipError_t blob_axpy(int64_t n, const double* a, double sc, const double* b, double* out,
                     hipStream_t s);
hipError_t blob_add(int64_t n, const double* x, double* y, hipStream_t s);
// y = (rho/dt) x + (eta/2) L_h x (explicit half of Crank-Nicolson).
template <typename T>
hipError_t apply_cn(mb_grid* g, const T* x, T* y, hipStream_t s);
// Spreading into the per-tile boxes (g->d_box), and the field from them.
template <typename T>
hipError_t spread_boxes(mb_grid* g, hipStream_t s);
template <typename T>
hipError_t fold_boxes(mb_grid* g, T* f, hipStream_t s);
// Force of a fluid solve.
template <typename T>
struct SolveForce {
    enum Src { FIELD, BOXES, RECORDS };
    Src src = FIELD;
    // FIELD: the force density.  Else (nullable) a force density added to the
    // blobs', which is the sum of the boxes of the last spreading, or (small
    // boxes, mbox blobs each) formed from the records of the last binning.
    const T* f = nullptr;
    int mbox = 0;
    // the explicit half is left out (v_in = 0, unread)
    bool rhs_only = false;
    // RECORDS in steady flow without f: the binning marked the z planes that
    // hold nodes of the blobs, and the transforms pass over the others; marked:
    // about how many of a box
    bool planes = false;
    int marked = 0;
    // with planes: only these are written to v_out, for a field that is
    // interpolated at those blobs and then overwritten; the interpolation
    // then clears the marks (else the solve does)
    bool planes_out = false;
};
template <typename T>
hipError_t fluid_solve(mb_grid* g, const T* v_in, const SolveForce<T>& force, T* v_out,
                       hipStream_t s);
// Elements of the box array: 3 components x tiles x (tx+3)(ty+3)(tz+3).
size_t box_elems(const Tiles& t);
// Interpolation of v at the binned blobs (u_out, q_update += dt u, both
// nullable; diag: per-tile partial sums); bin_next (with q_update): also
// bin the moved blobs into the counts of the next binning; clear_planes
// (small boxes): after a solve with planes_out.
template <typename T>
hipError_t interpolate(mb_grid* g, int64_t M, const T* v, double* u_out,
                       double* q_update, int diag, hipStream_t s, double uscale = 1.0,
                       bool bin_next = false, bool clear_planes = false);
// gout += wscale sum_a W_a grad_q (J v)_a per blob, on the binned records;
// u_out (nullable): also uscale J v.
template <typename T>
hipError_t interpolate_grad(mb_grid* g, int64_t M, const T* v, const double* W, double wscale,
                            double* gout, hipStream_t s, double* u_out = nullptr,
                            double uscale = 1.0);
// Particle order of a step call: particles counting-sorted by the tile of
// their last blob (the centre of the icosahedral template) into d_order
// (internal particle -> caller's particle), and the positions q and forces
// Fext (nullable) gathered into d_qint and d_pint in that order.
hipError_t order_particles(mb_grid* g, int64_t P, int nb, const double* q,
                           const double* Fext, hipStream_t s);
// End of a step call: with reordered, positions back into q in the caller's
// order and the blob velocities u into u_out (nullable); the particle
// velocities U0 (nullable) as means of u, in the caller's order; the
// diagnostics (nullable) from their partials.
hipError_t finish_call(mb_grid* g, int64_t P, int nb, bool reordered, double* q, const double* u,
                       double* u_out, double* U0, int force_blocks, double* diag,
                       hipStream_t s);
size_t record_size(int precision);
// Blocks and dynamic LDS bytes of the springs kernels for P particles.
int springs_blocks(const SpringsDev& sp, int64_t P);
size_t springs_lds(const SpringsDev& sp);

}  // namespace mb
