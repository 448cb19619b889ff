// Device-side data structures shared by the kernels and the host driver.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace kkt {

constexpr int kRestartMax = 64;        // largest supported FGMRES restart length
constexpr int kStreamBlock = 256;      // threads per block of the streaming kernels
constexpr int kStreamGridMax = 1024;   // blocks of the streaming kernels (partial-sum rows)
constexpr int kCoopBlock = 256;        // threads per block of the refactorization
constexpr int kTileThreads = 256;      // threads per block of the triangular solves
constexpr int kTileRows = 2048;        // rows of a multi-level solve tile (values in LDS)
constexpr int kTileLds = 32768;        // default LDS bytes of a staged solve tile
constexpr int kTileLdsMin = 16 * 1024;  // smallest and largest tile budgets (gfx950: 160 KiB of LDS
constexpr int kTileLdsMax = 150 * 1024; // per compute unit, the rest for the kernel's own arrays)
// Wavefronts the refactorization keeps resident on an MI355X: 3 blocks of 4 per compute unit,
// 256 compute units.
constexpr int kResidentRefactorWaves = 3 * 4 * 256;
constexpr int kRefactorLds = 1024;     // factor entries staged in LDS per wavefront
constexpr int kRefTileLds = 32512;     // LDS bytes of a refactorization tile
constexpr int64_t kSolSmallRows = 250000;  // fewer rows: solve tiles of 12 KiB, else 16 KiB
constexpr int64_t kDirectResidRows = 400000;  // kkt_residual gathers x in its own launch beyond
constexpr int kMaxBatch = 8;           // systems of one pattern refactored by one launch
constexpr int kWorkQueues = 8;         // hand-out queues of the refactorization and the solve tiles
// Spin limit of one dependency wait (iterations of a short sleep, a few seconds in all);
// exceeding it marks Control::hang and lets every wave run to completion.
constexpr unsigned int kSpinLimit = 1u << 22;

// Hand-out counters of the triangular solves (device memory, zeroed before a launch): the window
// kernels' next tile of each sweep, and the tile kernel's queues, each on a 256-byte line of its
// own (one counter hands out about 85 tasks per microsecond: 18,600 tasks at 2M unknowns
// took most of a 340 us launch).
struct SolveWork {
    unsigned int lower, upper;
    unsigned int pad[62];
    unsigned int queue[kWorkQueues * 64];
};
__device__ __forceinline__ void reset_work(SolveWork *w) {
    w->lower = 0;
    w->upper = 0;
    for (int q = 0; q < kWorkQueues; ++q) w->queue[q * 64] = 0;
}

// ||w - V h||, h = V^T w, from ww = ||w||^2 and hh = ||h||^2 (V's columns are orthonormal), where w has
// been through one Gram-Schmidt pass: h is then rounding, about 1e-16 of the vector before that
// pass, so nothing cancels unless w is that small too, and there the breakdown test (the norm
// against 1e-14 of it) ends the cycle.  A NaN stays one.
__device__ __forceinline__ double second_pass_norm(double ww, double hh) {
    const double d2 = ww - hh;
    return d2 < 0.0 ? 0.0 : sqrt(d2);
}

// Scalars shared between kernels of one refactor/solve (device memory).
struct Control {
    unsigned long long knorm_bits;  // max_i sum_j |K_ij| as the bits of a non-negative double
    unsigned int nonfinite;         // a non-finite matrix value was ingested
    unsigned int guard_fail;        // a guarded pivot under the FAIL policy
    unsigned long long nguard;      // guarded (perturbed) pivots
    unsigned int counter;           // arrivals of complete groups (last_arrival)
    int stop;                       // current FGMRES cycle has ended
    int jdone;                      // Arnoldi steps completed in the current cycle
    int breakdown;                  // happy breakdown in the current cycle
    int nonfinite_b;                // non-finite right-hand side
    unsigned int hang;              // a dependency wait exceeded its spin limit
    double beta;                    // ||rho|| at the start of the cycle
    double inner_tol;               // stop when the estimated residual <= inner_tol
    double est;                     // estimated residual |g_{j+1}|
    double wnorm_in;                // ||K z_j|| before orthogonalization
    double hn;                      // ||w|| after CGS2
    double rnorm2, xnorm2, bnorm2;  // sums of squares from the residual kernel
    double rinf, xinf;              // max |rho_i|, max |x_i| from the residual kernel
    double h1[kRestartMax + 1];     // first CGS pass coefficients
    double g[kRestartMax + 1];      // g[j]: right-hand side entry j before rotation j is applied
    double gr[kRestartMax];         // gr[j]: entry j after rotation j (the least-squares rhs); kept
                                    // apart from g so that no block of the normalization kernel
                                    // reads a value block 0 rewrites in the same launch
    double cs[kRestartMax], sn[kRestartMax];
    double y[kRestartMax];          // least-squares solution of the cycle
    double H[(kRestartMax + 1) * kRestartMax];  // rotated Hessenberg (upper triangular), column-major
    double Hbar[(kRestartMax + 1) * kRestartMax];  // DCGS2: final columns before rotation
    double hp[2][kRestartMax + 1];  // DCGS2: one-pass column j in hp[j & 1] (read by step j + 1)
    // Refactorization hand-out: kWorkQueues counters, one per 256-byte line; queue q hands out
    // items q, q + kWorkQueues, ... (next_task; first_queue says where a block starts).
    unsigned int work_refactor[kWorkQueues * 64];
    SolveWork work;                 // hand-out of the triangular solves
    unsigned int arrive[kWorkQueues * 64];  // arrivals of the blocks of each group, a line each
};

// What the host needs after each Arnoldi step, written by the normalization kernel into
// pinned host memory (one record per step of the cycle).
struct StepRecord {
    int stop;
    unsigned int hang;
    int jdone;
    int pad;
    double est;
    unsigned long long token;  // written last (release): identifies the step the record is for
};

// Signalling-NaN bit patterns no arithmetic result takes: "not written yet" in the exchange vectors.
// (A value of the caller's may: it is changed before it is stored there.)
constexpr unsigned long long kSent64 = 0x7FF4DEADBEEF0001ull;
constexpr unsigned int kSent32 = 0x7FA0BEEFu;

// What a caller inside the library arms before direct_solve_armed: n sentinels of the factors'
// precision in each of y and z, *work reset.
struct SolveScratch {
    int64_t n;
    bool f32;
    void *y, *z;
    SolveWork *work;
};

// Host-visible summary copied back once per cycle.
struct ControlSummary {
    unsigned long long knorm_bits;
    unsigned int nonfinite;
    unsigned int guard_fail;
    unsigned long long nguard;
    unsigned int counter;
    int stop, jdone, breakdown, nonfinite_b;
    unsigned int hang;
    double beta, inner_tol, est, wnorm_in, hn, rnorm2, xnorm2, bnorm2, rinf, xinf;
};

}  // namespace kkt
