// dsu_api.hip -- the host-driven single walker of the C ABI (include/dsu.h):
// a host state machine around three kernels (look-ahead ratio, accept with
// bordering, flush) plus the FP64 Gauss-Jordan recompute.  A move is one
// look-ahead launch the host waits for and one accept launch it does not.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "host_common.hpp"
#include "walker.hpp"

using namespace dsu;

using dsu::dalloc;
using dsu::dev_alloc;
using dsu::dfree;
using dsu::fail;
using dsu::GjDesc;
using dsu::GjWork;
using dsu::kpad;
using dsu::make_stream;

// ==========================================================================
// Single walker
// ==========================================================================
struct dsu_walker {
    int n = 0, np = 0, K = 0, kp = 0, prec = 0, policy = 0, flush_mode = DSU_FLUSH_AUTO;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    LaDev wd{};
    void *flush_y = nullptr, *flush_w = nullptr;  // scratch of the matrix-core flush
    double **a_ptr = nullptr;       // device array {a}
    void **bt_ptr = nullptr;        // device array {bt}
    double *inv_tmp = nullptr;      // n x n FP64 for dsu_get_inverse
    double *row_stage = nullptr;    // mapped pinned host staging: proposal row, then its 3 gradient rows
    const double *row_stage_dev = nullptr;  // its device address
    double *words_h = nullptr;      // pinned host words the look-ahead kernel writes R and grad R into
    GjWork gj;
    // host mirror of the state machine
    int k = 0, slots = 0;
    // multideterminant expansion (FP64 walkers): table, excitations, Q
    MdDev md{};
    bool md_on = false, prop_md = false;
    double md_q = 1.0, md_q_pending = 1.0;
    double *vphi_stage = nullptr;           // mapped pinned staging of the virtual row
    char *md_block = nullptr;               // device memory of md and md_part
    void *md_part = nullptr;                // partial sums with the expansion's m columns
    int md_ldp = 0;
    std::vector<int> idx;
    bool has_prop = false;
    int prop_e = -1;
    double prop_r = 0.0;
    double logdet = 0.0;
    int sign = 1;
};

static size_t elem(int prec) { return dsu::elem_size(prec); }

static void walker_md_free(dsu_walker *w) {
    dfree(w->md_block);
    w->md_block = nullptr;
    if (w->vphi_stage) (void)hipHostFree(w->vphi_stage);
    w->vphi_stage = nullptr;
    w->md_part = nullptr;
    w->md = MdDev{};
    w->md_on = w->prop_md = false;
}

static void walker_free(dsu_walker *w) {
    if (w->wd.phi != w->wd.phi64) dfree(w->wd.phi);  // FP64 walkers share one row buffer
    for (void *p : {w->wd.bt, w->wd.u, w->wd.vg, w->wd.a, w->wd.phi64, w->wd.cinv, w->wd.cinvt, w->wd.part, w->wd.t, w->wd.b,
                    w->wd.ratio, (void *)w->wd.idx, (void *)w->wd.counter, w->flush_y, w->flush_w, (void *)w->a_ptr, (void *)w->bt_ptr, (void *)w->inv_tmp})
        dfree(p);
    if (w->words_h) (void)hipHostFree(w->words_h);
    if (w->row_stage) (void)hipHostFree(w->row_stage);
    walker_md_free(w);
    w->gj.release();
    if (w->own_stream && w->stream) (void)hipStreamDestroy(w->stream);
}

// Fresh inverse of the n x n matrix `slater_host` (which becomes A) or of A.
static int walker_recompute(dsu_walker *w, const double *slater_host, double *fresh_logdet, int *fresh_sign) {
    if (slater_host) {
        // up in one piece into a buffer the inversion overwrites: a pitched
        // copy of pageable rows goes row by row
        HIPCHK(hipMemcpyAsync(w->gj.m2, slater_host, sizeof(double) * w->n * w->n, hipMemcpyHostToDevice, w->stream));
        HIPCHK(launch_pad_rows(w->gj.m2, (double *)w->wd.a, w->n, w->np, w->stream));
    }
    HIPCHK(launch_load_transpose(w->a_ptr, w->gj.mptr, 1, w->n, w->np, w->np, w->stream));
    const GjDesc *res = nullptr;
    HIPCHK(w->gj.invert(1, w->n, w->stream, &res));
    if (w->prec == DSU_FP64)
        HIPCHK(launch_cast_perm<double>(res, reinterpret_cast<double *const *>(w->bt_ptr), 1, w->n, w->np,
                                        w->stream));
    else
        HIPCHK(launch_cast_perm<float>(res, reinterpret_cast<float *const *>(w->bt_ptr), 1, w->n, w->np,
                                       w->stream));
    double ld = 0.0;
    int sg = 0, st = 0;
    HIPCHK(hipMemcpyAsync(&ld, w->gj.logdet, sizeof(double), hipMemcpyDeviceToHost, w->stream));
    HIPCHK(hipMemcpyAsync(&sg, w->gj.sign, sizeof(int), hipMemcpyDeviceToHost, w->stream));
    HIPCHK(hipMemcpyAsync(&st, w->gj.status, sizeof(int), hipMemcpyDeviceToHost, w->stream));
    HIPCHK(hipStreamSynchronize(w->stream));
    if (st != 0) return fail(DSU_ESINGULAR, "Slater matrix is singular");
    *fresh_logdet = ld;
    *fresh_sign = sg;
    return DSU_OK;
}

extern "C" int dsu_walker_create(int32_t n, int32_t k_delay, int32_t precision, int32_t policy,
                                 const double *slater_host, void *hip_stream, dsu_walker **out) {
    if (!out) return fail(DSU_EINVAL, "out is NULL");
    *out = nullptr;
    if (n < 1 || n > 32768) return fail(DSU_EINVAL, "n = %d out of range [1, 32768]", n);
    if (k_delay < 1 || k_delay > DSU_MAX_K) return fail(DSU_EINVAL, "k_delay = %d out of range [1, %d]", k_delay, DSU_MAX_K);
    if (precision != DSU_FP64 && precision != DSU_FP32_MIXED) return fail(DSU_EINVAL, "bad precision %d", precision);
    if (policy != DSU_FLUSH_K_ACCEPTED && policy != DSU_FLUSH_K_PROPOSED) return fail(DSU_EINVAL, "bad policy %d", policy);
    if (!slater_host) return fail(DSU_EINVAL, "slater matrix is NULL");
    dsu_walker *w = new dsu_walker();
    w->n = n;
    w->np = round_up(n, 64);
    w->K = k_delay;
    w->kp = kpad(k_delay);
    w->prec = precision;
    w->policy = policy;
    int rc = DSU_OK;
    const size_t s = elem(precision), np = w->np, kp = w->kp;
#define TRY(x)                 \
    do {                       \
        rc = (x);              \
        if (rc != DSU_OK) {    \
            walker_free(w);    \
            delete w;          \
            return rc;         \
        }                      \
    } while (0)
    TRY(make_stream(hip_stream, &w->stream, &w->own_stream));
    TRY(dev_alloc(&w->wd.bt, np * np * s));
    TRY(dev_alloc(&w->wd.u, kp * np * s));
    TRY(dev_alloc(&w->wd.vg, kp * np * s));
    TRY(dev_alloc(&w->wd.a, np * np * sizeof(double)));
    TRY(dev_alloc(&w->wd.phi64, np * sizeof(double)));
    if (precision == DSU_FP64) w->wd.phi = w->wd.phi64;
    else TRY(dev_alloc(&w->wd.phi, np * s));
    w->wd.ldp = la_ldp((int)kp);
    TRY(dev_alloc(&w->wd.part, (size_t)kLaBlocks * w->wd.ldp * sizeof(double)));
    TRY(dev_alloc(&w->wd.cinv, kp * (kp + 1) * sizeof(double)));
    TRY(dev_alloc(&w->wd.cinvt, kp * (kp + 1) * sizeof(double)));
    TRY(dev_alloc(&w->wd.t, kp * sizeof(double)));
    TRY(dev_alloc(&w->wd.b, kp * sizeof(double)));
    TRY(dev_alloc(&w->wd.ratio, sizeof(double)));
    TRY(dalloc(&w->wd.idx, kp));
    TRY(dalloc(&w->wd.counter, 1));
    w->wd.ldc = (int)kp + 1;
    // coherent: the host watches the result words while the kernel runs
    if (hipHostMalloc((void **)&w->words_h, kLaWords * sizeof(double), hipHostMallocMapped | hipHostMallocCoherent) !=
        hipSuccess)
        TRY(fail(DSU_ENOMEM, "hipHostMalloc failed"));
    std::memset(w->words_h, 0, kLaWords * sizeof(double));
    if (hipHostMalloc((void **)&w->row_stage, 4 * np * sizeof(double), hipHostMallocMapped | hipHostMallocCoherent) !=
        hipSuccess)
        TRY(fail(DSU_ENOMEM, "hipHostMalloc failed"));
    {
        void *dptr = nullptr;
        if (hipHostGetDevicePointer(&dptr, w->row_stage, 0) != hipSuccess)
            TRY(fail(DSU_EDEVICE, "hipHostGetDevicePointer failed"));
        w->row_stage_dev = static_cast<const double *>(dptr);
    }
    {
        void *dptr = nullptr;
        if (hipHostGetDevicePointer(&dptr, w->words_h, 0) != hipSuccess)
            TRY(fail(DSU_EDEVICE, "hipHostGetDevicePointer failed"));
        w->wd.words = static_cast<double *>(dptr);
    }
    // pointer tables for the batched-style launchers
    TRY(dalloc(&w->a_ptr, 1));
    TRY(dalloc(&w->bt_ptr, 1));
    if (hipMemcpy(w->a_ptr, &w->wd.a, sizeof(double *), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(w->bt_ptr, &w->wd.bt, sizeof(void *), hipMemcpyHostToDevice) != hipSuccess)
        TRY(fail(DSU_EDEVICE, "pointer table upload failed"));
    TRY(dev_alloc(&w->flush_y, s * (precision == DSU_FP64 ? flush_scratch_elems<double>(w->np, w->np, w->kp)
                                                          : flush_scratch_elems<float>(w->np, w->np, w->kp))));
    TRY(dev_alloc(&w->flush_w, np * kp * s));
    TRY(w->gj.alloc(1, w->np, n));
    TRY(walker_recompute(w, slater_host, &w->logdet, &w->sign));
    w->idx.assign(w->kp, -1);
#undef TRY
    *out = w;
    return DSU_OK;
}

extern "C" int dsu_walker_destroy(dsu_walker *w) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    (void)hipStreamSynchronize(w->stream);
    walker_free(w);
    delete w;
    return DSU_OK;
}

template <typename T> static hipError_t walker_flush_t(dsu_walker *w, bool valu) {
    const FlushArgs<T> fa{(T *)w->wd.bt, (const T *)w->wd.u, (const T *)w->wd.vg, (const double *)w->wd.cinv,
                          (const double *)w->wd.cinvt, w->wd.idx, w->wd.ldc, (T *)w->flush_y, (T *)w->flush_w};
    return valu ? launch_flush_valu<T>(fa, w->np, w->k, w->stream)
                : launch_flush_mfma<T, 1>(fa, w->np, w->k, w->stream);
}

static int walker_do_flush(dsu_walker *w) {
    if (w->k > 0) {
        // The vector ALUs read BT, U and Vg once per slot group and cost about
        // k np; the matrix cores one launch (small n) or three, the same up to 16
        // slots.  A flush and the next look-ahead, us, vector / matrix.  FP64: k =
        // 1 24.5 / 31 at n = 1024, 75 / 89 at 4096; k = 2 32.5 / 33.9 at 960, 31.4 / 31.0 at
        // 1024, 99 / 89 at 4096; k = 3 27.8 / 29.8 at 448, 26.9 / 26.7 at 512; k = 4 28.5 /
        // 28.6 at 384, 31.4 / 29.9 at 448.  FP32: k = 2 16.3 / 16.8 at 100, 32 / 34.5 at
        // 1024, 90 / 97 at 4096; k = 3 18.1 / 16.9 at 128, 22.8 / 22.1 at 256, 22.4 / 23.6 at
        // 320, 26.7 / 27.3 at 448, 28.4 / 27.3 at 512; k = 4 19.4 / 16.9 at 128, 29.7 / 27.3 at
        // 448
        const int k = w->k, np = w->np;
        const bool line = w->prec == DSU_FP64 ? k == 1 || (k == 2 && np < 1024) || (k <= 4 && k * np <= 1536)
                                              : k <= 2 || (k == 3 && np > 256 && np < 512);
        const bool valu = w->flush_mode == DSU_FLUSH_VALU || (w->flush_mode == DSU_FLUSH_AUTO && line);
        if (w->prec == DSU_FP64) HIPCHK(walker_flush_t<double>(w, valu));
        else HIPCHK(walker_flush_t<float>(w, valu));
    }
    w->k = 0;
    w->slots = 0;
    std::fill(w->idx.begin(), w->idx.end(), -1);
    return DSU_OK;
}

extern "C" int dsu_flush(dsu_walker *w) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    return walker_do_flush(w);
}

// Look-ahead of the row(s) in `src` against electron e; the proposal becomes pending.
static int walker_propose_common(dsu_walker *w, const LaSource &src, int e, double *ratio_out,
                                 double *grad_out = nullptr) {
    // an electron may hold at most one pending move: apply the window first
    for (int j = 0; j < w->k; ++j)
        if (w->idx[j] == e) {
            CHK(walker_do_flush(w));
            break;
        }
    const int gm = grad_out ? 1 : 0, words = grad_out ? 4 : 1;
    la_arm(w->words_h, 0, words);
    if (w->prec == DSU_FP64)
        HIPCHK(launch_walker_propose<double>(w->wd, src, w->n, w->np, w->k, e, gm, -1, w->stream));
    else HIPCHK(launch_walker_propose<float>(w->wd, src, w->n, w->np, w->k, e, gm, -1, w->stream));
    CHK(la_wait(w->words_h, 0, words, w->stream));
    const volatile double *h = w->words_h;
    const double r = h[0];
    w->has_prop = true;
    w->prop_e = e;
    w->prop_r = r;
    if (ratio_out) *ratio_out = r;
    if (grad_out)
        for (int a = 0; a < 3; ++a) grad_out[a] = h[1 + a];
    return DSU_OK;
}

// Copy `nrows` host rows (n FP64 each) into the pinned staging rows the
// look-ahead kernel reads, zero padded to np.  Every earlier look-ahead was
// waited for, so the rows are free.
static LaSource walker_stage_rows(dsu_walker *w, int nrows, const double *const *rows) {
    const size_t np = w->np;
    for (int r = 0; r < nrows; ++r) {
        double *st = w->row_stage + r * np;
        std::memcpy(st, rows[r], sizeof(double) * w->n);
        std::memset(st + w->n, 0, sizeof(double) * (np - w->n));
    }
    return LaSource{w->row_stage_dev, nullptr};
}

extern "C" int dsu_propose_ratio(dsu_walker *w, int32_t electron, const double *phi_host, double *ratio_out) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (w->md_on) return fail(DSU_ESTATE, "multideterminant walker: propose with dsu_propose_ratio_md");
    if (electron < 0 || electron >= w->n) return fail(DSU_EINVAL, "electron %d out of range", electron);
    if (!phi_host) return fail(DSU_EINVAL, "row is NULL");
    return walker_propose_common(w, walker_stage_rows(w, 1, &phi_host), electron, ratio_out);
}

extern "C" int dsu_propose_ratio_grad(dsu_walker *w, int32_t electron, const double *phi_host, const double *dphi_host,
                                      double *ratio_out, double *grad_out) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (w->md_on) return fail(DSU_ESTATE, "multideterminant walker: propose with dsu_propose_ratio_md");
    if (electron < 0 || electron >= w->n) return fail(DSU_EINVAL, "electron %d out of range", electron);
    if (!phi_host || !dphi_host || !grad_out) return fail(DSU_EINVAL, "NULL argument");
    const double *rows[4] = {phi_host, dphi_host, dphi_host + w->n, dphi_host + 2 * (size_t)w->n};
    return walker_propose_common(w, walker_stage_rows(w, 4, rows), electron, ratio_out, grad_out);
}

extern "C" int dsu_eval_grad(dsu_walker *w, int32_t electron, const double *dphi_host, double *grad_out) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (electron < 0 || electron >= w->n) return fail(DSU_EINVAL, "electron %d out of range", electron);
    if (!dphi_host || !grad_out) return fail(DSU_EINVAL, "NULL argument");
    const double *rows[3] = {dphi_host, dphi_host + w->n, dphi_host + 2 * (size_t)w->n};
    const LaSource src = walker_stage_rows(w, 3, rows);
    int m = -1;  // pending slot holding this electron's accepted move, if any
    for (int j = 0; j < w->k; ++j)
        if (w->idx[j] == electron) m = j;
    la_arm(w->words_h, 1, 3);
    if (w->prec == DSU_FP64)
        HIPCHK(launch_walker_propose<double>(w->wd, src, w->n, w->np, w->k, electron, 2, m, w->stream));
    else HIPCHK(launch_walker_propose<float>(w->wd, src, w->n, w->np, w->k, electron, 2, m, w->stream));
    CHK(la_wait(w->words_h, 1, 3, w->stream));
    const volatile double *h = w->words_h;
    for (int a = 0; a < 3; ++a) grad_out[a] = h[1 + a];
    return DSU_OK;
}

extern "C" int dsu_propose_ratio_dev(dsu_walker *w, int32_t electron, const void *phi_dev, double *ratio_out) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (w->md_on) return fail(DSU_ESTATE, "multideterminant walker: propose with dsu_propose_ratio_md");
    if (electron < 0 || electron >= w->n) return fail(DSU_EINVAL, "electron %d out of range", electron);
    if (!phi_dev) return fail(DSU_EINVAL, "row is NULL");
    return walker_propose_common(w, LaSource{nullptr, phi_dev}, electron, ratio_out);
}

static int walker_slot_used(dsu_walker *w) {
    ++w->slots;
    const bool full = w->policy == DSU_FLUSH_K_ACCEPTED ? (w->k >= w->K) : (w->slots >= w->K);
    if (full) return walker_do_flush(w);
    return DSU_OK;
}

extern "C" int dsu_accept(dsu_walker *w) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (!w->has_prop) return fail(DSU_ESTATE, "no pending proposal");
    const double r = w->prop_r;
    const double floor = w->prec == DSU_FP64 ? RatioFloor<double>::value : RatioFloor<float>::value;
    if (!(std::fabs(r) > floor) || !std::isfinite(r)) return fail(DSU_ESINGULAR, "ratio %g cannot be accepted", r);
    if (w->prop_md && !(std::fabs(w->md_q_pending) > 0.0 && std::isfinite(w->md_q_pending)))
        return fail(DSU_ESINGULAR, "the expansion vanishes at the proposed configuration");
    if (w->prop_md) {
        HIPCHK(launch_md_accept(w->wd, w->md, w->n, w->np, w->k, w->prop_e, w->stream));
        w->md_q = w->md_q_pending;
        w->prop_md = false;
    } else if (w->prec == DSU_FP64) {
        HIPCHK(launch_walker_accept<double>(w->wd, w->n, w->np, w->k, w->prop_e, w->stream));
    } else {
        HIPCHK(launch_walker_accept<float>(w->wd, w->n, w->np, w->k, w->prop_e, w->stream));
    }
    w->idx[w->k] = w->prop_e;
    ++w->k;
    w->logdet += std::log(std::fabs(r));
    if (r < 0) w->sign = -w->sign;
    w->has_prop = false;
    return walker_slot_used(w);
}

extern "C" int dsu_reject(dsu_walker *w) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (!w->has_prop) return fail(DSU_ESTATE, "no pending proposal");
    w->has_prop = false;
    w->prop_md = false;
    if (w->policy == DSU_FLUSH_K_PROPOSED) return walker_slot_used(w);
    return DSU_OK;
}

static int walker_md_refresh(dsu_walker *w);

extern "C" int dsu_recompute_inverse(dsu_walker *w, const double *slater_host_or_null, double *logdet_out,
                                     int32_t *sign_out, double *drift_out) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    double ld;
    int sg;
    CHK(walker_recompute(w, slater_host_or_null, &ld, &sg));
    if (w->md_on) {
        if (slater_host_or_null) {
            walker_md_free(w);  // the virtual rows belong to the old configuration
        } else {
            CHK(walker_md_refresh(w));
        }
    }
    if (drift_out) *drift_out = w->logdet - ld;
    w->logdet = ld;
    w->sign = sg;
    w->k = 0;
    w->slots = 0;
    w->has_prop = false;
    std::fill(w->idx.begin(), w->idx.end(), -1);
    if (logdet_out) *logdet_out = ld;
    if (sign_out) *sign_out = sg;
    return DSU_OK;
}

extern "C" int dsu_get_inverse(dsu_walker *w, double *out_host) {
    if (!w || !out_host) return fail(DSU_EINVAL, "NULL argument");
    CHK(walker_do_flush(w));
    if (!w->inv_tmp) CHK(dalloc(&w->inv_tmp, (size_t)w->n * w->n));
    if (w->prec == DSU_FP64) HIPCHK(launch_untranspose<double>((const double *)w->wd.bt, w->inv_tmp, w->n, w->np, w->stream));
    else HIPCHK(launch_untranspose<float>((const float *)w->wd.bt, w->inv_tmp, w->n, w->np, w->stream));
    HIPCHK(hipMemcpyAsync(out_host, w->inv_tmp, sizeof(double) * w->n * w->n, hipMemcpyDeviceToHost, w->stream));
    HIPCHK(hipStreamSynchronize(w->stream));
    return DSU_OK;
}

extern "C" int dsu_get_logdet(dsu_walker *w, double *logdet, int32_t *sign) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (logdet) *logdet = w->logdet;
    if (sign) *sign = w->sign;
    return DSU_OK;
}

extern "C" int dsu_walker_pending(dsu_walker *w, int32_t *k_out) {
    if (!w || !k_out) return fail(DSU_EINVAL, "NULL argument");
    *k_out = w->k;
    return DSU_OK;
}

extern "C" int dsu_walker_set_flush_kernel(dsu_walker *w, int32_t mode) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (mode < DSU_FLUSH_AUTO || mode > DSU_FLUSH_MFMA) return fail(DSU_EINVAL, "bad flush mode %d", mode);
    if (mode == DSU_FLUSH_VALU && w->K > 64) return fail(DSU_EINVAL, "VALU flush supports k <= 64");
    w->flush_mode = mode;
    return DSU_OK;
}


// ==========================================================================
// Multideterminant expansion on a single reference (FP64 walkers)
// ==========================================================================
// Table T = A^{-1} V from the present (flushed) inverse, and Q of the present table.
static int walker_md_refresh(dsu_walker *w) {
    HIPCHK(launch_md_table(w->wd, w->md, w->n, w->np, w->stream));
    la_arm(w->words_h, 2, 1);
    HIPCHK(launch_md_init(w->wd, w->md, w->stream));
    CHK(la_wait(w->words_h, 2, 1, w->stream));
    const double q = ((const volatile double *)w->words_h)[2];
    if (!(std::fabs(q) > 0.0) || !std::isfinite(q)) return fail(DSU_ESINGULAR, "the expansion vanishes (Q = %g)", q);
    w->md_q = q;
    return DSU_OK;
}

extern "C" int dsu_walker_set_multidet(dsu_walker *w, int32_t m, const double *virt_host, int32_t ndet,
                                       const int32_t *order, const int32_t *occ, const int32_t *virt,
                                       const double *coef) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (w->prec != DSU_FP64) return fail(DSU_EINVAL, "multideterminant expansions need an FP64 walker");
    if (m < 1 || m > 4096) return fail(DSU_EINVAL, "m = %d out of range [1, 4096]", m);
    if (ndet < 1 || ndet > (1 << 20)) return fail(DSU_EINVAL, "ndet = %d out of range", ndet);
    if (!virt_host || !order || !occ || !virt || !coef) return fail(DSU_EINVAL, "NULL argument");
    for (int d = 0; d < ndet; ++d) {
        const int o = order[d];
        if (o < 0 || o > 4) return fail(DSU_EINVAL, "determinant %d: order %d outside [0, 4]", d, o);
        for (int a = 0; a < o; ++a) {
            const int j = occ[4 * d + a], v = virt[4 * d + a];
            if (j < 0 || j >= w->n || v < 0 || v >= m) return fail(DSU_EINVAL, "determinant %d: index out of range", d);
            for (int b = 0; b < a; ++b)
                if (occ[4 * d + b] == j || virt[4 * d + b] == v)
                    return fail(DSU_EINVAL, "determinant %d: repeated orbital", d);
        }
    }
    walker_md_free(w);
    CHK(walker_do_flush(w));
    w->has_prop = false;
    const size_t np = w->np;
    int rc = DSU_OK;
#define MDTRY(x)                  \
    do {                          \
        rc = (x);                 \
        if (rc != DSU_OK) {       \
            walker_md_free(w);    \
            return rc;            \
        }                         \
    } while (0)
    // the occupied orbitals the expansion replaces, each once
    std::vector<int> place(w->n, -1), uocc, occ_u(4 * (size_t)ndet, 0);
    for (int d = 0; d < ndet; ++d)
        for (int a = 0; a < order[d]; ++a) {
            const int j = occ[4 * d + a];
            if (place[j] < 0) {
                place[j] = (int)uocc.size();
                uocc.push_back(j);
            }
            occ_u[4 * (size_t)d + a] = place[j];
        }
    w->md.nu = (int)uocc.size();
    uocc.push_back(0);  // never empty
    w->md_ldp = la_ldp(w->kp) + m;
    // one device block, its pieces 256-byte aligned, the caller's lists last and
    // uploaded together (a block and a copy each: 345 us a call at n = 64, m = 4; so 130)
    std::vector<char> lists;
    size_t bytes = 0;
    std::vector<std::pair<void **, size_t>> pieces;
    auto piece = [&](auto **p, size_t count) {
        pieces.push_back({(void **)p, bytes});
        bytes += (count * sizeof(**p) + 255) & ~(size_t)255;
    };
    auto list = [&](auto **p, const auto *host, size_t count) {
        const size_t at = lists.size();
        piece(p, count);
        lists.resize(at + ((count * sizeof(**p) + 255) & ~(size_t)255));
        std::memcpy(lists.data() + at, host, count * sizeof(**p));
    };
    double *part = nullptr;
    piece(&w->md.v, np * m);
    piece(&w->md.t, np * m);
    piece(&part, (size_t)kLaBlocks * w->md_ldp);
    piece(&w->md.cu, uocc.size());
    piece(&w->md.vphi, (size_t)m);
    piece(&w->md.x, (size_t)m);
    piece(&w->md.q, 2);
    const size_t lists_at = bytes;
    list(&w->md.uocc, uocc.data(), uocc.size());
    list(&w->md.occ_u, occ_u.data(), occ_u.size());
    list(&w->md.order, order, (size_t)ndet);
    list(&w->md.occ, occ, 4 * (size_t)ndet);
    list(&w->md.virt, virt, 4 * (size_t)ndet);
    list(&w->md.coef, coef, (size_t)ndet);
    MDTRY(dalloc(&w->md_block, bytes));
    for (auto &q : pieces) *q.first = w->md_block + q.second;
    w->md_part = part;
    if (hipHostMalloc((void **)&w->vphi_stage, sizeof(double) * m, hipHostMallocMapped | hipHostMallocCoherent) !=
        hipSuccess)
        MDTRY(fail(DSU_ENOMEM, "hipHostMalloc failed"));
    {
        void *dptr = nullptr;
        if (hipHostGetDevicePointer(&dptr, w->vphi_stage, 0) != hipSuccess)
            MDTRY(fail(DSU_EDEVICE, "hipHostGetDevicePointer failed"));
        w->md.vphi_host = static_cast<const double *>(dptr);
    }
    w->md.m = m;
    w->md.ndet = ndet;
    if (hipMemcpy(w->md.v, virt_host, sizeof(double) * w->n * m, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(w->md_block + lists_at, lists.data(), lists.size(), hipMemcpyHostToDevice) != hipSuccess)
        MDTRY(fail(DSU_EDEVICE, "expansion upload failed"));
    MDTRY(walker_md_refresh(w));
#undef MDTRY
    w->md_on = true;
    return DSU_OK;
}

extern "C" int dsu_propose_ratio_md(dsu_walker *w, int32_t electron, const double *phi_host, const double *vphi_host,
                                    double *ratio_out, double *ratio_ref_out) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (!w->md_on) return fail(DSU_ESTATE, "no multideterminant expansion set");
    if (electron < 0 || electron >= w->n) return fail(DSU_EINVAL, "electron %d out of range", electron);
    if (!phi_host || !vphi_host) return fail(DSU_EINVAL, "row is NULL");
    const LaSource src = walker_stage_rows(w, 1, &phi_host);
    std::memcpy(w->vphi_stage, vphi_host, sizeof(double) * w->md.m);
    // an electron may hold at most one pending move: apply the window first
    for (int j = 0; j < w->k; ++j)
        if (w->idx[j] == electron) {
            CHK(walker_do_flush(w));
            break;
        }
    LaDev wd = w->wd;  // with room for the expansion's columns in the partial sums
    wd.part = w->md_part;
    wd.ldp = w->md_ldp;
    la_arm(w->words_h, 0, 3);
    HIPCHK(launch_md_propose(wd, src, w->md, w->n, w->np, w->k, electron, w->stream));
    CHK(la_wait(w->words_h, 0, 3, w->stream));
    const volatile double *h = w->words_h;
    const double total = h[0], r = h[1], q = h[2];
    w->has_prop = true;
    w->prop_e = electron;
    w->prop_r = r;
    w->prop_md = true;
    w->md_q_pending = q;
    if (ratio_out) *ratio_out = total;
    if (ratio_ref_out) *ratio_ref_out = r;
    return DSU_OK;
}

extern "C" int dsu_walker_md_value(dsu_walker *w, double *logabs, int32_t *sign) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (!w->md_on) return fail(DSU_ESTATE, "no multideterminant expansion set");
    if (logabs) *logabs = w->logdet + std::log(std::fabs(w->md_q));
    if (sign) *sign = w->md_q < 0 ? -w->sign : w->sign;
    return DSU_OK;
}
