// k_walker.hip -- the real host-driven walker's look-ahead kernels
// (lookahead.hpp instantiated for float and double) and the set-up steps of
// the multideterminant expansion.
#include "lookahead.hpp"

#include <chrono>
#include <cstring>

#include "host_common.hpp"

namespace dsu {

template <typename T>
hipError_t launch_walker_propose(const LaDev &w, const LaSource &src, int n, int np, int k, int e, int grad_mode, int m,
                                 hipStream_t s) {
    const MdDev none{};
    if (grad_mode == 0) return la_propose<T, 0>(w, src, n, np, k, e, -1, none, s);
    if (grad_mode == 1) return la_propose<T, 1>(w, src, n, np, k, e, -1, none, s);
    return la_propose<T, 2>(w, src, n, np, k, e, m, none, s);
}
template <typename T> hipError_t launch_walker_accept(const LaDev &w, int n, int np, int k, int e, hipStream_t s) {
    return la_accept<T>(w, n, np, k, e, MdDev{}, s);
}
template hipError_t launch_walker_propose<float>(const LaDev &, const LaSource &, int, int, int, int, int, int,
                                                 hipStream_t);
template hipError_t launch_walker_propose<double>(const LaDev &, const LaSource &, int, int, int, int, int, int,
                                                  hipStream_t);
template hipError_t launch_walker_accept<float>(const LaDev &, int, int, int, int, hipStream_t);
template hipError_t launch_walker_accept<double>(const LaDev &, int, int, int, int, hipStream_t);

// ------------------------------------------------------------------------
// Multideterminant expansion on a single reference (FP64 walker).
// Psi = sum_I c_I det(A_I): A_I is A with occupied columns J_I replaced by
// virtual columns V_I, and det(A_I) / det(A) = det S_I, S_I = T[J_I][V_I]
// with the table T = A^{-1} V.  Moving electron e (rows phi, vphi) changes T
// by a rank-1 term: T' = T + c x^T, c = A^{-1}[:, e] (the delayed inverse's
// column, i.e. BT[e] corrected by the pending moves as in the look-ahead),
// x = (vphi - phi T) / R with R the reference ratio.
// ------------------------------------------------------------------------

// T[j][v] = sum_i BT[i][j] V[i][v], j < n (rows past n stay zero).
__global__ void k_md_table(const double *bt, MdDev md, int n, int np) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x, v = blockIdx.y;
    if (j >= n) return;
    double s = 0.0;
    for (int i = 0; i < n; ++i) s += bt[(size_t)i * np + j] * md.v[(size_t)i * md.m + v];
    md.t[(size_t)j * md.m + v] = s;
}

// Q = sum_I c_I det S_I of the present table (one workgroup).
__global__ __launch_bounds__(kLaThreads) void k_md_init(MdDev md, double *words) {
    __shared__ double sbuf[kLaWaves];
    double s = 0.0;
    for (int d = threadIdx.x; d < md.ndet; d += kLaThreads) s += md.coef[d] * md_det(md, d, false);
    s = la_block_sum(s, sbuf);
    if (threadIdx.x == 0) {
        md.q[1] = s;
        la_report(words + 2, s);
    }
}

hipError_t launch_md_table(const LaDev &w, const MdDev &md, int n, int np, hipStream_t s) {
    hipLaunchKernelGGL(k_md_table, dim3((n + 255) / 256, md.m), dim3(256), 0, s, (const double *)w.bt, md, n, np);
    return hipGetLastError();
}

hipError_t launch_md_propose(const LaDev &w, const LaSource &src, const MdDev &md, int n, int np, int k, int e,
                             hipStream_t s) {
    return la_propose<double, 0, true>(w, src, n, np, k, e, -1, md, s);
}

hipError_t launch_md_init(const LaDev &w, const MdDev &md, hipStream_t s) {
    hipLaunchKernelGGL(k_md_init, dim3(1), dim3(kLaThreads), 0, s, md, w.words);
    return hipGetLastError();
}

hipError_t launch_md_accept(const LaDev &w, const MdDev &md, int n, int np, int k, int e, hipStream_t s) {
    return la_accept<double, true>(w, n, np, k, e, md, s);
}

// ------------------------------------------------------------------------
// Result words, host side.
// ------------------------------------------------------------------------
void la_arm(double *words, int first, int count) {
    volatile unsigned long long *h = reinterpret_cast<unsigned long long *>(words);
    for (int i = first; i < first + count; ++i) h[i] = kLaPending;
}

int la_wait(const double *words, int first, int count, hipStream_t s) {
    const volatile unsigned long long *h = reinterpret_cast<const unsigned long long *>(words);
    auto done = [&] {
        for (int i = first; i < first + count; ++i)
            if (h[i] == kLaPending) return false;
        return true;
    };
    const auto t0 = std::chrono::steady_clock::now();
    for (unsigned spin = 0;; ++spin) {
        if (done()) return DSU_OK;
        if ((spin & 4095u) == 4095u && std::chrono::steady_clock::now() - t0 > std::chrono::seconds(2)) break;
    }
    HIPCHK(hipStreamSynchronize(s));
    if (!done()) return fail(DSU_EDEVICE, "look-ahead kernel did not report");
    return DSU_OK;
}

}  // namespace dsu
