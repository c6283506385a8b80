// walker.hpp -- device state and kernel launchers of the host-driven walkers
// (look-ahead ratio, its gradient, accept with bordering).
#pragma once
#include "dsu_internal.hpp"

namespace dsu {

// Blocks of a look-ahead launch at most.
constexpr int kLaBlocks = 32;
// Host result words before a launch: a signalling NaN no arithmetic produces.
constexpr unsigned long long kLaPending = 0x7FF4A5C35A3C1E0Full;
constexpr int kLaWords = 4;

// Device state of a host-driven walker.  Element type T (float, double, or
// interleaved complex double2) and K x K type S (double or double2).
struct LaDev {
    void *bt;       // np x np, T
    void *u;        // kp x np, T
    void *vg;       // kp x np, T
    void *a;        // np x np, S: Slater matrix
    void *phi;      // np, T: pending proposal row
    void *phi64;    // np, S: the same before rounding to T (phi itself if T = S)
    void *cinv;     // kp x ldc, S: C_k^{-1} in pending order
    void *cinvt;    // kp x ldc, S: its transpose
    void *t;        // kp, S: C_k^{-1} q of the pending proposal
    void *b;        // kp, S: p^T C_k^{-1}
    void *ratio;    // S: device copy of R
    void *part;     // kLaBlocks x ldp, S: the blocks' partial sums
    double *words;  // kLaWords mapped pinned host words: results (R; grad R or the drift in 1..3)
    int *idx;       // kp pending electrons
    unsigned *counter;  // blocks finished (last-block reduction)
    int ldc;        // kp + 1
    int ldp;        // partial sums a block leaves
};

// Where a launch reads the proposed rows: FP64 host rows in mapped pinned
// memory (stride np, zero padded), or one device row of n elements of T.
struct LaSource {
    const void *host;
    const void *dev;
};

// Multideterminant state of an FP64 walker (single-reference expansion).
struct MdDev {
    double *v;      // np x m: virtual orbitals, row i = electron i (zero rows past n)
    double *t;      // np x m: table T = A^{-1} V (row j = occupied orbital j)
    double *vphi;   // m: virtual row of the proposal
    const double *vphi_host;  // the same in mapped pinned host memory
    double *x;      // m: (vphi - phi T) / R
    int *order;     // ndet: substitutions per determinant (0..4)
    int *occ;       // ndet x 4: occupied orbitals replaced
    int *occ_u;     // ndet x 4: their places in uocc
    int *virt;      // ndet x 4: virtual orbitals put in their place
    int *uocc;      // nu: the occupied orbitals the expansion replaces, each once
    double *cu;     // nu: column e of the current inverse (look-ahead corrected) at uocc
    double *coef;   // ndet
    double *q;      // [0]: sum_I c_I det S_I of the pending proposal; [1]: of the present state
    int m, ndet, nu;
};

// Partial sums per block at delay kp: four x rows against BT[e] and Vg, then q
// (and m columns of phi T).
inline int la_ldp(int kp) { return 4 * (kp + 1) + kp; }

// Single-walker look-ahead ratio and accept (bordering); lookahead.hpp.
// grad_mode 0: ratio; 1: ratio and its gradient; 2: gradient of the present
// row only (m = pending slot held by e, or -1).
template <typename T>
hipError_t launch_walker_propose(const LaDev &w, const LaSource &src, int n, int np, int k, int e, int grad_mode, int m,
                                 hipStream_t s);
template <typename T> hipError_t launch_walker_accept(const LaDev &w, int n, int np, int k, int e, hipStream_t s);
// Multideterminant steps (FP64).  table: T = BT^T V.  propose: the look-ahead
// and Q' = sum_I c_I det(S_I + c_J x_V); words 0..2 = (R Q' / Q, R, Q').
// init: Q = sum_I c_I det S_I of the present table -> q[1] and word 2.
// accept: the acceptance, T += c x, V[e] = vphi, Q = Q'.
hipError_t launch_md_table(const LaDev &w, const MdDev &md, int n, int np, hipStream_t s);
hipError_t launch_md_propose(const LaDev &w, const LaSource &src, const MdDev &md, int n, int np, int k, int e,
                             hipStream_t s);
hipError_t launch_md_init(const LaDev &w, const MdDev &md, hipStream_t s);
hipError_t launch_md_accept(const LaDev &w, const MdDev &md, int n, int np, int k, int e, hipStream_t s);

// Host side of the result words: la_arm marks `count` of them pending before
// the launch, la_wait returns once each holds a result (after 2 s without one
// the stream is synchronised instead, which reports a failed kernel).
void la_arm(double *words, int first, int count);
int la_wait(const double *words, int first, int count, hipStream_t s);

}  // namespace dsu
