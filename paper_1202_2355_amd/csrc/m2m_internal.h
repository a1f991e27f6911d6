// Internal device-side structures shared by the HIP kernels (m2m_kernels.hip)
// and the host side of the C ABI (m2m_api.cpp). Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace m2m {

constexpr int kMaxGH = 8;          // largest Gauss-Hermite order
constexpr int kMaxLOSVD = 256;     // largest LOSVD bin count
constexpr int kMaxLM = 8;          // largest degree l of the a_lm density observables
constexpr int kMaxCells = 4096;    // largest n_E * n_x
constexpr int kLcTable = 8192;     // entries of the ln r_c(ln zeta) table
constexpr int kFinCols = 64;       // columns (bins or cells) per finalize block
constexpr int kFinThreads = 1024;  // finalize block: 16 waves over the tiles
constexpr int kFinWaves = kFinThreads / 64;  // row groups of the fixed reduction order
constexpr int kSmoothMaxSide = 128;   // prior smoothing: at most this many cells per axis
constexpr int kSmoothMaxCells = 2048; // and per smoothed grid
constexpr int kSmoothMaxPoints = 256; // and at most this many first-stage search points
constexpr int kGcvSlots = 5;          // lambda points a wave scores in one pass over the cells
constexpr int kHistCap = 8192;     // chi^2 history ring per fit
constexpr int kSegAlign = 64;      // tile boundaries are multiples of 64 particles
constexpr int kMaxScfNodes = 64;   // largest node count of the self-consistent potential

// kernel launch modes (bit set)
enum : int32_t {
    kModeStep = 1,       // a full M2M step: (assign) FOC, push, deposit, (cells)
    kModeInit = 2,       // deposit the current state; finalize sets ytilde = y
    kModeObserve = 4,    // deposit the current state into obs_out only
    kModeCells = 8,      // accumulate the prior cells of the current state only
    kModeWriteThrough = 16,  // step: particle stores write through L2 (small fits)
    kModePot = 32,       // rebuild the self-consistent potential from the current state only
    kModeStream = 64,    // batch step: nontemporal particle loads and stores (large states)
    kModeInterleave = 128,  // one fit: tiles take interleaved chunks of particles (large states)
    kModeBack = 256,     // with kModeInterleave: the chunks from the last to the first
};

// Particle state up to this size is stepped with write-through stores: it
// stays in the memory-side cache, and no dirty particle lines are left in L2
// for the write-back at the end of the step kernel.
constexpr size_t kWriteThroughMax = size_t(64) << 20;

// The particle state of a batch launch above this size is streamed with
// nontemporal loads and stores (the batch step kernels of the lean kinds of
// observables, FP32 state): it does not fit the memory-side cache anyway, and with the
// hint on both the loads and the stores the 64-fit batch of 1.16 GB stepped
// 11 % faster; either hint alone gained nothing, and a state that stays in
// the cache (3.2e7 bytes) stepped 6 % slower with them.
constexpr size_t kStreamMin = size_t(128) << 20;

// The step kernel of one fit whose particle state exceeds kStreamMin takes
// its particles interleaved (kModeInterleave): chunks of one block's width,
// dealt to the tiles in turn, so that the blocks in flight read and write a
// narrow window of each array. At 8e6 particles (480 MB) the step kernel ran
// 10 % faster so; at 1e6 (in the memory-side cache) 2-4 % slower, and the
// 64-fit batch (many fits of about 24 tiles each) gained nothing. Every
// other step takes the chunks in the opposite order (kModeBack): the step
// begins with the particles that the one before it touched last, which are still
// in the 256 MB memory-side cache. LOSVD step, us, always forward and in
// turn: 8e6 particles (256 MB) 98.3 / 93.5, 1.6e7 211 / 187, 3.2e7 412 / 378,
// 6e6 71.1 / 71.0. Batches gained nothing: streamed with nontemporal accesses,
// which leave little in the cache, 3 % slower at 16 fits of 1e6 particles.

// Dynamic per-fit state, device resident, written only by the kernels (and by
// the host between launches, on the fit's stream).
struct FitState {
    int64_t kstep;           // correction steps done (prior schedule)
    int64_t tstep;           // all steps done (chi^2 history index)
    int32_t steps_left;      // steps still to run; kernels skip the fit at 0
    int32_t correct;         // force of change on (1) or relaxation (0)
    int32_t assign_pending;  // fresh cell priors wait to be assigned
    int32_t error;           // bit 0: non-finite chi^2 seen, bit 1: a run did not complete
    uint32_t ticket;         // finalize: blocks done this launch
    uint32_t mticket;        // the same in observe mode
    double chi2;             // chi^2 after the last step
};

// Static per-fit description (device copy). Pointers are device addresses.
struct FitDev {
    // particle state (float or double, SoA)
    void *x, *y, *z, *vx, *vy, *vz, *u, *uh;
    int64_t n;
    // potential: Hernquist G M upsilon, a; NFW G M200 / f(c), r_s; Phi(0)
    double GMh, a, GMn, rs, phi0;
    // observables
    int32_t n_r, n_R, kin, nk, J, n_v, gh_nmax, C;
    int32_t jk0;             // index of the first kinematic observable
    int32_t l_max;           // a_lm degree; n_r then counts mesh intervals
    double lr0, lrs;         // radial bin guess: (log2(r^2) - lr0) * lrs
    double lR0, lRs;         // annulus bin guess
    double vmin, vidv;       // LOSVD bin guess: (v - vmin) * vidv
    void *redge2, *Redge2, *vedge, *Vp, *isp, *rp;  // tables in the state dtype
    void* rmesh;             // a_lm mesh radii (n_r + 1, state dtype)
    double *Y, *sigma, *yv, *ytil, *delta, *obs_out;
    double *partials;        // tile rows of row_len doubles
    int32_t row_len;         // J + 2 C (+ scf_P)
    int32_t kpriv;           // private copies of the in-tile bins (power of 2)
    int32_t smooth;          // thin-plate smoothing of the prior grid at refreshes
    int32_t n_bin_jobs;      // ceil(J / kFinCols)
    int32_t n_cell_jobs;     // ceil(C / kFinCols)
    int32_t entropy;
    // priors
    int32_t n_E, n_x, prior_every, pad1;
    double E_lo, E_hi, E_scale;  // E_scale = n_E / (E_hi - E_lo)
    // energy coordinate of the cells: (e - cell_e0) * cell_es with e = E, or
    // e = exp(E) (cell_flags bit 1); bit 0: particles with L_z < 0 take cell
    // cell_half + k n_x + l
    double cell_e0, cell_es;
    int32_t cell_flags, cell_half;
    void *ucell, *lctab;         // C values; kLcTable values of ln r_c(ln zeta)
    uint16_t *cidx;              // n values: cell of each particle at the last refresh
    // prior grid in FP64: cell data of the last refresh (means, or the
    // previous prior of empty cells) and the current priors
    double *cdata, *gprior;
    // smoothing: the log10(lambda) search range, the cell width along energy
    double sm_plo, sm_phi, sm_hE;
    int32_t sm_k1, pad3;         // points of the first search stage
    // eigenvalues and parity-block eigenvectors of the smoothing penalty
    // (smooth_basis below), FP64
    double* sm_basis;
    double lz0, ilz;             // ln zeta of entry 0, 1 / step in ln zeta
    double hv2, hr02, hiq2;      // logarithmic halo: v0^2 (0: none), r0^2, 1/q^2
    // step constants
    double dt, w0, foc_mu, foc_cs, foc_chi, q;  // foc_mu = eps dt mu, foc_chi = eps dt w0
    double *chi2_hist;
    double *chi2_part;           // one per bin job
    FitState *st;
    // self-consistent stellar potential (last, so that the fields before keep
    // their offsets in the kernel arguments) (scf_nr = 0: none): a multipole
    // expansion to degree scf_lmax with node values at scf_nr radii
    // log-spaced from scf_rho[0]; the tile rows carry its scf_P interval sums
    // from column scf_col0 (after the cell columns), reduced by n_pot_jobs
    // finalize jobs on the steps that rebuild it (every scf_every steps)
    int32_t scf_nr, scf_lmax, scf_every, scf_col0, scf_P, n_pot_jobs;
    double scf_ls0, scf_ih;      // ln rho_0, 1 / node spacing in ln r
    double scf_c;                // G upsilon M / N: Phi scale per unit weight u
    double *scf_rho;             // node radii (FP64)
    double *scf_sum;             // interval sums of the last rebuild (scf_P)
    double *scf_tab;             // nodes x (l, m): Phi_lm(rho_k), r dPhi_lm/dr there
};

// One tile: a contiguous particle range of one fit, owned by one block.
struct Tile {
    int32_t fit;     // index into the launch's fit table
    int32_t row;     // tile row in the fit's partials
    int64_t begin, end;
    int32_t n_rows;  // tiles of this fit in the launch
    int32_t pad;
};

// Tile t of count tiles over n particles (tile rows row0 + t of fit `fit`):
// boundaries at n t / count rounded down to a multiple of kSegAlign, the
// last tile ending at n. The host builds its tile tables with it, and the
// one-fit step kernel finds its own tile with it.
__host__ __device__ inline Tile tile_of(int64_t n, int t, int count, int fit, int row0) {
    int64_t b = n * t / count, e = n * (t + 1) / count;
    b = b / kSegAlign * kSegAlign;
    e = (t == count - 1) ? n : e / kSegAlign * kSegAlign;
    return Tile{fit, row0 + t, b, e, count, 0};
}

// One finalize block: kFinCols columns of one fit, or (kind kFinWholeFit)
// every column of one fit and the end of its step.
constexpr int32_t kFinWholeFit = 3;
struct FinJob {
    int32_t fit;
    int32_t kind;  // 0: observable and cell columns, 1: cell columns, 2: potential columns, 3: all
    int32_t col0;
    int32_t n_tiles;  // rows of the fit to reduce
};

// Fits whose cell columns have jobs of their own (kind 1, after those of kind 0), and
// the observable and cell jobs of a fit.
__host__ __device__ inline bool cells_apart(int32_t prior_every) { return prior_every == 1; }
__host__ __device__ inline int column_jobs(int nbj, int ncj, int32_t prior_every) {
    return cells_apart(prior_every) ? nbj + ncj : (nbj > ncj ? nbj : ncj);
}

// ---- run kernel (m2m_run.h): several steps of one fit in one launch ---------
constexpr int kRunCols = 16;        // columns per reduction job
constexpr int kRunMaxSteps = 256;   // steps per launch
constexpr int kRunMaxBlocks = 256;  // one block per compute unit
constexpr size_t kRunStaticLds = 2 * 16 * kRunCols * 8 + 256;  // its static LDS (16 waves), rounded up
constexpr uint32_t kRunWait = 1000000000; // 10 s (100 MHz counter): a wait within a run that failed
// How long a launch waits for blocks that have not started: 50 ms, and 0.1 ms times
// the blocks wanted for each that runs after a launch that was called off.
constexpr uint32_t kRunStart = 5000000, kRunAgain = 10000;

// Counters of the launches of a context, in its workspace.
struct RunSync {
    // low half: blocks that have started, over all launches, and kRunOff once this
    // launch is called off; high half: the blocks that had started by then
    uint64_t start;
    uint32_t start0;    // the low half before this launch
    uint32_t left;      // blocks that have left a launch that was called off
    uint32_t wait;      // longest wait within a run, 100 MHz ticks (0: kRunWait)
    uint32_t patience;  // 1 + kRunAgain after a launch that was called off, 0 after another
};
// After a launch that ends beyond this many blocks the count begins again.
constexpr uint32_t kRunStartMax = 0x40000000u;
__host__ __device__ inline uint32_t run_start_after(uint32_t start0, uint32_t blocks) {
    return start0 + blocks > kRunStartMax ? 0u : start0 + blocks;
}

// Exchange areas of a run, in memory of its stream: 64-bit words of 32 data and 32
// tag bits (m2m_run.h).
struct RunArgs {
    int32_t keep_at, keep_bytes;  // LDS offset and size of the kept kernels (0: not kept)
    int32_t n_jobs, n_cell_jobs;  // ceil(J / kRunCols), ceil(C / kRunCols)
    RunSync* sync;
    uint64_t *rows;   // blocks x (J + 2 C) sums, 2 words each
    uint64_t *res;    // J entries of the force table, 1 word (FP32) or 2
    uint64_t *cell;   // C cell priors, the same
    // kRunMaxSteps x n_jobs parts of chi^2, 2 words each; where the priors are
    // smoothed 6 C words and 2 + 6 kSmoothMaxPoints per grid half follow
    uint64_t *parts;
};
// LDS offset of the prior smoothing's two grids (FP64)
__host__ __device__ inline int run_smooth_at(const RunArgs& a) {
    return (a.keep_at + a.keep_bytes + 7) & ~7;
}

// What one launch does: n_steps steps with the force of change on or off (a fit
// of a batch: as many of them as it has left, with its own setting), their tags
// from tag0 + 1. known: start0 is the counter's value before the launch, else the
// kernel reads it.
struct RunCall {
    int32_t n_steps, correct, known;
    uint32_t start0, tag0;
};

// one block of a run of many fits: block b of nb of fit `fit`
struct RunTile {
    int32_t fit, b, nb, pad;
};

// Blocks and threads per block of a run over n particles of J observables: at
// most one block per compute unit, and at least one per reduction job. FP32:
// 8 waves a block up to 2^15 particles, above that 16. FP64: 8 waves (16 would
// leave 128 registers a lane and spill 45 to 65), half of them idle up to 2^15
// particles. Measured us a step, Gauss-Hermite (blocks x threads): FP32 16384
// particles 32x512 4.8, 16x1024 5.7, 64x256 5.7, 256x256 9.8; 131072 128x1024
// 6.0, 256x1024 6.5, 256x512 7.5; 10^6 256x1024 12.3, 256x512 17.8. FP64 16384
// 64x512 6.0, 32x512 6.2, 256x256 10.8; 65536 128x512 7.2, 256x512 8.4.
struct RunShape {
    int block, blocks;
};
inline RunShape run_shape(int64_t n, bool f64, int J) {
    const bool small = n <= 32768;
    const int block = small || f64 ? 512 : 1024, per = f64 && small ? 256 : block;
    const int64_t jobs = (J + kRunCols - 1) / kRunCols;
    int64_t b = (n + per - 1) / per;
    b = b > 16 ? b : 16;
    b = b > jobs ? b : jobs;
    return RunShape{block, (int)(b < kRunMaxBlocks ? b : kRunMaxBlocks)};
}

// steps (at most kRunMaxSteps) of one fit over `blocks` blocks, or (tiles) of the
// fits of a table, each up to the steps it has left; done (or NULL): an event
// that the launch itself completes
hipError_t launch_run_f32(int block, int kin, const FitDev& fd, const RunArgs& ra, int blocks,
                          size_t lds, const RunCall& call, hipStream_t s, hipEvent_t done);
hipError_t launch_run_f64(int block, int kin, const FitDev& fd, const RunArgs& ra, int blocks,
                          size_t lds, const RunCall& call, hipStream_t s, hipEvent_t done);
// the same of a fit whose priors are smoothed
hipError_t launch_run_smooth_f32(int block, int kin, const FitDev& fd, const RunArgs& ra, int blocks,
                                 size_t lds, const RunCall& call, hipStream_t s, hipEvent_t done);
hipError_t launch_run_smooth_f64(int block, int kin, const FitDev& fd, const RunArgs& ra, int blocks,
                                 size_t lds, const RunCall& call, hipStream_t s, hipEvent_t done);
hipError_t launch_runs_f32(int block, int kin, const FitDev* fits, const RunArgs* ras,
                           const RunTile* tiles, int blocks, size_t lds, int n_steps, uint32_t tag0,
                           hipStream_t s, hipEvent_t done);
hipError_t launch_runs_f64(int block, int kin, const FitDev* fits, const RunArgs* ras,
                           const RunTile* tiles, int blocks, size_t lds, int n_steps, uint32_t tag0,
                           hipStream_t s, hipEvent_t done);

// ---- launchers (m2m_kernels.hip) ------------------------------------------
// kin: kinematic kind of every fit in the launch, from kin_class()
hipError_t launch_step(bool f64, bool acc64, int block, int kin, const FitDev* fits,
                       const Tile* tiles, int n_tiles, size_t lds_bytes, int32_t mode,
                       hipStream_t s);
// the column jobs of the fits of the table (n_fits of them)
// scf: the fits have the self-consistent potential (kin_scf of their kin class)
// smooth: some fit of the launch smooths its prior grid (the variant with the
// smoothing's LDS grids); whole: every job is a whole-fit job (one block per
// fit, the kernel with small blocks), else every job is a column job
// wide: column jobs of 16 waves (else 4)
hipError_t launch_finalize(bool f64, const FitDev* fits, const FinJob* jobs, int n_jobs, int32_t mode,
                           hipStream_t s, bool scf, bool smooth, bool whole, bool wide);
bool kin_scf(int kin);
// the step kernel of one particle-state / in-tile-sum type pair (one == nullptr:
// over the fit and tile tables, else over that one fit); m2m_step_*.hip
hipError_t launch_step_f64(int block, int kin, const FitDev* fits, const Tile* tiles,
                           const FitDev* one, int n_tiles, size_t lds, int32_t mode, hipStream_t s);
hipError_t launch_step_f32d(int block, int kin, const FitDev* fits, const Tile* tiles,
                            const FitDev* one, int n_tiles, size_t lds, int32_t mode, hipStream_t s);
hipError_t launch_step_f32f(int block, int kin, const FitDev* fits, const Tile* tiles,
                            const FitDev* one, int n_tiles, size_t lds, int32_t mode, hipStream_t s);
// one fit, fd (a host copy of its description) passed by value: the step
// over n_tiles tiles as tile_of splits it; the finalize jobs of that fit
// (bin and cell columns, then potential columns) over n_rows tile rows
hipError_t launch_step1(bool f64, bool acc64, int block, int kin, const FitDev& fd, int n_tiles,
                        size_t lds, int32_t mode, hipStream_t s);
hipError_t launch_finalize1(bool f64, const FitDev& fd, int n_rows, int32_t mode, hipStream_t s);

// ---- prior smoothing basis (m2m_smooth.cpp) -------------------------------
// Doubles of the eigendecomposition of the thin-plate penalty of an
// n_E x n_x grid: n_E n_x eigenvalues, then the eigenvectors of its four
// reflection-parity blocks.
size_t smooth_basis_len(int nE, int nx);
// Compute it (or take it from the process-wide cache of grid shapes) into
// out; false if the eigen-iteration does not converge.
bool smooth_basis(int nE, int nx, double hE, double hx, double* out);
hipError_t launch_assign(bool f64, const FitDev* fit, int blocks, hipStream_t s);
hipError_t launch_weights(bool f64, const void* u, void* w, int64_t n, double scale,
                          hipStream_t s);
hipError_t launch_poke(FitState* st, int32_t steps_left, int32_t correct, hipStream_t s);
hipError_t launch_gather(const FitDev* fits, int n, int32_t* out, hipStream_t s);
hipError_t launch_residuals(bool f64, const FitDev* fit, hipStream_t s);
size_t step_lds_bytes(bool f64, bool acc64, int J, int n_r, int n_R, int n_v, int kpriv, int C,
                      int scf_nr, int scf_lmax);
int kin_class(int kin, int gh_nmax, int dens, bool scf);
int private_copies(int J, size_t bytes);

}  // namespace m2m
