// lookahead.hpp -- the two kernels of a host-driven move, for the real walker
// (T = float or double) and the complex one (T = double2): the look-ahead
// ratio of Sec. II, eq. (3), and the acceptance with its bordering.
//
// With k accepted moves pending (electrons e_1..e_k, new rows U, stale BT rows
// Vg) the ratio for moving electron e to the row phi is
//     R = r0 - p^T C_k^{-1} q,  r0 = phi.BT[e],  p_j = phi.Vg[j],  q_j = U[j].BT[e]
// (the Schur complement of C_{k+1} = [[C_k, q], [p^T, r0]]; plain transposes
// over the complex field too), and an accepted move borders C_k^{-1}:
//     t = C^{-1} q,  b^T = p^T C^{-1},
//     C_{k+1}^{-1} = [[C^{-1} + t b^T / R, -t / R], [-b^T / R, 1 / R]].
//
// A move is one propose launch the host waits for and one accept launch it
// does not.  Both move at most a few MB and are bound by latency: of the host
// link (the proposed row in, the ratio out), of a launch and its instruction
// fetch, and of each dependent step of the reduction.  So the work is cut to
// have few of them, in little code:
//  * propose: a block owns a range of columns of every row, at most kLaBlocks
//    blocks.  It reads its part of the proposed rows from the host's pinned
//    buffer itself (once over the link; no staging launch).  All products are
//    one skinny matrix product on 16x16x4 matrix cores, the 2 k + 1 rows of
//    BT[e], Vg, U against at most five columns (the x rows and BT[e]), which
//    sums over the lanes without exchanges; complex rows enter as real rows
//    of twice the length against (re, -im) and (im, re).  The last block to
//    finish adds the blocks' partial sums and forms t and b, C^{-1} and its
//    transpose both stored so that each is a sum over coalesced rows.
//  * the results go to pinned host words that the host set to kLaPending
//    before the launch: a word that changed is a result, so neither a fence
//    towards the host nor a completion tag follows them.
//  * accept: b and t are known, so every entry of the bordered inverse and
//    every copied row element is independent: one grid of small blocks.
// Per launch on MI355X, propose then accept, before (row staging + one dot
// product per block + a serial tail; one accept block) and now: N = 64, K = 16
// FP64 9.7 + 4.0 -> 6.8 + 2.8 us; N = 1024, K = 64 FP64 19.2 + 9.3 -> 10.7 +
// 3.0 us; N = 4096, K = 128 FP32 36.4 + 21.6 -> 13.7 + 3.2 us; complex N = 500,
// K = 16 11.1 + 4.9 -> 9.4 + 2.9 us; multideterminant N = 1024, K = 64, 16
// virtuals 38.1 + 12.4 -> 15.3 + 4.8 us.  Of the 10.7 us about 2 are the link,
// 1 the products, 1 the count-off, 1.5 the partial sums, 2 the t and b
// products; instruction fetch is part of each (every line runs once a launch:
// a 20 KB form of this kernel with the loads of all phases in flight together
// measured 15 us, this one has 5 to 6.4 KB, 13 for the expansion).
#pragma once
#include "dsu_internal.hpp"
#include "tiles.hpp"
#include "walker.hpp"

namespace dsu {

constexpr int kLaThreads = 512, kLaWaves = kLaThreads / 64;

// Arithmetic of the three element types; S is the type of everything K x K, R the real element.
template <typename T> struct LaNum { typedef double S; typedef T R; };
template <> struct LaNum<double2> { typedef double2 S; typedef double R; };
__device__ __forceinline__ double la_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ double2 la_fma(double2 a, double2 b, double2 c) {
    return make_double2(__builtin_fma(a.x, b.x, __builtin_fma(-a.y, b.y, c.x)),
                        __builtin_fma(a.x, b.y, __builtin_fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ double la_add(double a, double b) { return a + b; }
__device__ __forceinline__ double2 la_add(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double la_sub(double a, double b) { return a - b; }
__device__ __forceinline__ double2 la_sub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double la_neg_mul(double a, double b) { return -(a * b); }
__device__ __forceinline__ double2 la_neg_mul(double2 a, double2 b) {
    return make_double2(a.y * b.y - a.x * b.x, -(a.x * b.y + a.y * b.x));
}
__device__ __forceinline__ double la_mul(double a, double b) { return a * b; }
__device__ __forceinline__ double2 la_mul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double la_inv(double a) { return 1.0 / a; }
__device__ __forceinline__ double2 la_inv(double2 a) {
    const double d = a.x * a.x + a.y * a.y;
    return make_double2(a.x / d, -a.y / d);
}
template <typename T> __device__ __forceinline__ T la_zero() { return T(0); }
template <> __device__ __forceinline__ double2 la_zero<double2>() { return make_double2(0.0, 0.0); }
template <typename T> __device__ __forceinline__ T la_one() { return T(1); }
template <> __device__ __forceinline__ double2 la_one<double2>() { return make_double2(1.0, 0.0); }
template <typename T> __device__ __forceinline__ typename LaNum<T>::S la_wide(T v) { return double(v); }
template <> __device__ __forceinline__ double2 la_wide<double2>(double2 v) { return v; }
template <typename T> __device__ __forceinline__ T la_shfl_xor(T v, int o) { return __shfl_xor(v, o, 64); }
template <> __device__ __forceinline__ double2 la_shfl_xor<double2>(double2 v, int o) {
    return make_double2(__shfl_xor(v.x, o, 64), __shfl_xor(v.y, o, 64));
}

typedef double la_d2 __attribute__((ext_vector_type(2)));
template <typename T> __device__ __forceinline__ T la_load(const T *p) { return *gmem(p); }
template <> __device__ __forceinline__ double2 la_load<double2>(const double2 *p) {
    const la_d2 x = *(DSU_GLOBAL const la_d2 *)p;
    return make_double2(x[0], x[1]);
}

template <typename T> __device__ __forceinline__ T la_wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = la_add(v, la_shfl_xor(v, o));
    return v;
}

// A result word for the host (any bit pattern but kLaPending).
__device__ __forceinline__ void la_report(double *word, double v) {
    unsigned long long b = (unsigned long long)__double_as_longlong(v);
    if (b == kLaPending) b |= 1ull << 51;  // the quiet NaN of the same payload
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(word), b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void la_report_s(double *word, double v) { la_report(word, v); }
__device__ __forceinline__ void la_report_s(double *word, double2 v) {
    la_report(word, v.x);
    la_report(word + 1, v.y);
}

// Element c of proposed row r: the host's FP64 rows (stride np, zero padded),
// or one device row of n elements of T.
template <typename T>
__device__ __forceinline__ typename LaNum<T>::S la_source(const LaSource &src, int r, int c, int n, int np) {
    typedef typename LaNum<T>::S S;
    if (src.host) return la_load(static_cast<const S *>(src.host) + (size_t)r * np + c);
    return c < n ? la_wide(la_load(static_cast<const T *>(src.dev) + c)) : la_zero<S>();
}

// Sum of an FP64 value over the block, for every thread.
__device__ __forceinline__ double la_block_sum(double v, double *sbuf) {
    v = la_wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sbuf[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kLaWaves; ++q) s += sbuf[q];
    return s;
}

// det of the order x order matrix S[a][b] = T[J_a][V_b] (+ c[J_a] x[V_b] with
// the proposal's rank-1 term): Gaussian elimination with partial pivoting.
// Singles and doubles, the bulk of an expansion, in a few instructions; the
// rest on the matrix bordered to 4 x 4 with the identity (every index fixed,
// so it stays in registers).
__device__ __forceinline__ double md_det(const MdDev &md, int d, bool with_x) {
    const int o = md.order[d];
    auto entry = [&](int a, int b) {
        const int j = md.occ[4 * d + a], v = md.virt[4 * d + b];
        return md.t[(size_t)j * md.m + v] + (with_x ? md.cu[md.occ_u[4 * d + a]] * md.x[v] : 0.0);
    };
    if (o == 0) return 1.0;
    if (o == 1) return entry(0, 0);
    if (o == 2) {
        const double a = entry(0, 0), b = entry(0, 1), c = entry(1, 0), e = entry(1, 1);
        const bool up = fabs(c) > fabs(a);
        const double p = up ? c : a;
        if (p == 0.0) return 0.0;
        const double r = (up ? b : e) - (up ? a : c) / p * (up ? e : b);
        return up ? -p * r : p * r;
    }
    double s[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) s[a][b] = a < o && b < o ? entry(a, b) : (a == b ? 1.0 : 0.0);
    double det = 1.0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
        for (int a = p + 1; a < 4; ++a) {  // the largest entry of column p to row p
            const bool up = fabs(s[a][p]) > fabs(s[p][p]);
            if (up) det = -det;
#pragma unroll
            for (int b = p; b < 4; ++b) {
                const double x = s[p][b], y = s[a][b];
                s[p][b] = up ? y : x;
                s[a][b] = up ? x : y;
            }
        }
        if (s[p][p] == 0.0) return 0.0;
        det *= s[p][p];
#pragma unroll
        for (int a = p + 1; a < 4; ++a) {
            const double f = s[a][p] / s[p][p];
#pragma unroll
            for (int b = p + 1; b < 4; ++b) s[a][b] -= f * s[p][b];
        }
    }
    return det;
}

// Look-ahead products of a set of x rows against one electron.  R(x) =
// x.BT[e] - sum_j (x.Vg[j]) t_j is linear in x, so the ratio (x = phi) and its
// gradient (x = d phi / d r_a) share q and t; so does the drift grad_e ln|det|
// at the present position (x = gradient rows of the present row).
//   GR = 0: x = {phi};  GR = 1: x = {phi, dphi_x, dphi_y, dphi_z};
//   GR = 2: x = {dphi_x, dphi_y, dphi_z}: results to words 1..3 only, the
//           pending proposal (phi, t, b, ratio) untouched.  If e itself holds
//           pending slot m, row e of the delayed matrix is U[m], and the
//           lemma's right-hand side becomes q - 1_m.
//   MD (GR = 0, FP64): the multideterminant ratio as well.  Besides the
//           look-ahead each block forms its columns' part of phi T; the last
//           block then has x = (vphi - phi T) / R, c = A^{-1}[:, e] at the
//           occupied orbitals the expansion names, and
//           Q' = sum_I c_I det(S_I + c_J x_V).
// Block b takes columns b * cb .. + cb of every row, as real columns (cb a
// multiple of 64; np and cb count two for a complex element).
template <typename T, int GR, bool MD>
__global__ __launch_bounds__(kLaThreads) void k_lookahead(LaDev w, LaSource src, int n, int np, int cb, int k, int e,
                                                          int m, MdDev md) {
    typedef typename LaNum<T>::S S;
    typedef typename LaNum<T>::R R;               // real element of a row
    constexpr int Z = sizeof(T) / sizeof(R);      // reals per element
    constexpr int NX = GR == 0 ? 1 : (GR == 1 ? 4 : 3), NB = Z * (NX + 1);
    constexpr int X0 = GR == 1 ? 1 : 0;           // first gradient row
    constexpr int VEC = 16 / (int)sizeof(R);
    typedef typename Vec16<R>::type vec_t;
    extern __shared__ __attribute__((aligned(16))) char s_dyn[];
    R *s_x = reinterpret_cast<R *>(s_dyn);        // NB columns of the block's cb rows: the x rows, then BT[e]
    __shared__ S s_d[NX * (DSU_KMAX_LDS + 1) + DSU_KMAX_LDS];  // x.BT[e], x.Vg[j] per x row; then q
    __shared__ S s_t[DSU_KMAX_LDS], s_p[kLaWaves][64];
    __shared__ double s_red[kLaWaves];
    __shared__ S s_r;
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int ldr = Z * np, c0 = blockIdx.x * cb, cols = ldr - c0 < cb ? ldr - c0 : cb;
    const int rows = 2 * k + 1, ld = k + 1, nd = NX * ld + k, ldx = cb + VEC;
    const R *bte = static_cast<const R *>(w.bt) + (size_t)e * ldr;
    const R *u = static_cast<const R *>(w.u), *vg = static_cast<const R *>(w.vg);
    // tiles of 16 rows: A operand row lr, columns 4 lk .. + 3 of each 16 (the
    // contraction's order is free), B operand column lr (repeated past NB).
    // A group is 64 columns of a tile; each group's rows are loaded before the
    // products of the one before, the first ones before the x rows arrive.
    const int gpt = cols / 64, groups = ((rows + 15) / 16 - wave + kLaWaves - 1) / kLaWaves * gpt;
    vec_t y[16 / VEC];
    auto load = [&](int g) __attribute__((always_inline)) {
        const int r = 16 * (wave + kLaWaves * (g / gpt)) + lr;
        const R *yp =
            (r == 0 || r >= rows ? bte : (r <= k ? vg + (size_t)(r - 1) * ldr : u + (size_t)(r - 1 - k) * ldr)) + c0 +
            64 * (g % gpt) + 4 * lk;
#pragma unroll
        for (int h = 0; h < 16 / VEC; ++h)
            y[h] = *(DSU_GLOBAL const vec_t *)gmem(yp + 16 * (h / (4 / VEC)) + VEC * (h % (4 / VEC)));
    };
    if (groups > 0) load(0);
    // the product's columns: x row r (complex: (re, -im), then (im, re)); row NX is BT[e]
    for (int v = tid; v < (NX + 1) * (cols / Z); v += kLaThreads) {
        const int r = v / (cols / Z), c = v % (cols / Z);
        S x;
        if (r == NX) x = la_wide(la_load(reinterpret_cast<const T *>(bte + c0) + c));
        else x = la_source<T>(src, r, c0 / Z + c, n, np);
        if constexpr (Z == 2) {
            R *o = s_x + (size_t)(2 * r) * ldx + 2 * c;
            o[0] = x.x;
            o[1] = -x.y;
            o[ldx] = x.y;
            o[ldx + 1] = x.x;
        } else {
            s_x[r * ldx + c] = R(x);
        }
        if (GR != 2 && r == 0) {  // kept for the acceptance
            static_cast<S *>(w.phi64)[c0 / Z + c] = x;
            if constexpr (sizeof(T) != sizeof(S)) static_cast<T *>(w.phi)[c0 + c] = T(x);
        }
    }
    if (MD && blockIdx.x == 0)
        for (int v = tid; v < md.m; v += kLaThreads) md.vphi[v] = md.vphi_host[v];
    __syncthreads();
    double *part = static_cast<double *>(w.part) + (size_t)blockIdx.x * Z * w.ldp;
    const R *xb = s_x + (size_t)(lr < NB ? lr : NB - 1) * ldx + 4 * lk;
    // FP64: the sums of four columns that a matrix instruction makes are added in
    // pairs, the rounding errors of a chain as long as the row being 1.2 to 1.9
    // times as large in R; FP32 products in chains of 16 columns, added up in FP64
    f64x4 acc{0, 0, 0, 0};
    for (int g = 0; g < groups; ++g) {
        vec_t cur[16 / VEC];
#pragma unroll
        for (int h = 0; h < 16 / VEC; ++h) cur[h] = y[h];
        if (g + 1 < groups) load(g + 1);
        f64x4 sum[16 / VEC];
#pragma unroll
        for (int h = 0; h < 16 / VEC; ++h) {
            const vec_t bv = *reinterpret_cast<const vec_t *>(xb + 64 * (g % gpt) + 16 * (h / (4 / VEC)) +
                                                              VEC * (h % (4 / VEC)));
            if constexpr (sizeof(R) == 8) {
                sum[h] = Mma<R>::mma(cur[h][0], bv[0], f64x4{0, 0, 0, 0}) + Mma<R>::mma(cur[h][1], bv[1], f64x4{0, 0, 0, 0});
            } else {
                f32x4 part32{0, 0, 0, 0};
#pragma unroll
                for (int q = 0; q < VEC; ++q) part32 = Mma<R>::mma(cur[h][q], bv[q], part32);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] += (double)part32[i];
            }
        }
        if constexpr (sizeof(R) == 8) {
#pragma unroll
            for (int o = 8 / VEC; o > 0; o /= 2)
#pragma unroll
                for (int h = 0; h < o; ++h) sum[h] += sum[h + o];
            acc += sum[0];
        }
        if (g % gpt != gpt - 1) continue;
        const int r0 = 16 * (wave + kLaWaves * (g / gpt));
        // x rows: value of x row lr / Z at Vg row r; q rows: the products with BT[e]
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ro = r0 + Mma<R>::row0(lane) + i * Mma<R>::row_step, a = lr / Z;
            if (ro <= k ? a < NX : (a == NX && ro < rows))
                part[Z * (ro <= k ? a * ld + ro : NX * ld + ro - 1 - k) + lr % Z] = acc[i];
        }
        acc = f64x4{0, 0, 0, 0};
    }
    if constexpr (MD) {
        // this block's rows of T, tiles of 16 virtual orbitals: A = T^T, B = phi
        for (int v0 = 16 * wave; v0 < md.m; v0 += 16 * kLaWaves) {
            const int v = v0 + lr < md.m ? v0 + lr : md.m - 1;
            const double *t = md.t + (size_t)(c0 + lk) * md.m + v;
            f64x4 acc{0, 0, 0, 0};
            for (int j = 0; j < cols; j += 32) {  // (added in pairs, as above)
                f64x4 sum[8];
#pragma unroll
                for (int h = 0; h < 8; ++h)
                    sum[h] = Mma<double>::mma(la_load(t + (size_t)(j + 4 * h) * md.m), (double)s_x[j + 4 * h + lk],
                                              f64x4{0, 0, 0, 0});
#pragma unroll
                for (int o = 4; o > 0; o /= 2)
#pragma unroll
                    for (int h = 0; h < o; ++h) sum[h] += sum[h + o];
                acc += sum[0];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int vo = v0 + lk + 4 * i;
                if (lr == 0 && vo < md.m) part[nd + vo] = acc[i];
            }
        }
    }
    const int nblk = gridDim.x;
    __syncthreads();  // the block's partial sums are written
    if (nblk > 1) {
        if (tid == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            s_last = __hip_atomic_fetch_add(w.counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nblk - 1u;
        }
        __syncthreads();
        if (!s_last) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    const S *pt = static_cast<const S *>(w.part);
    for (int v = tid; v < (MD ? nd + md.m : nd); v += kLaThreads) {
        S s = la_zero<S>();
        for (int q = 0; q < nblk; q += 8) {  // (in pairs, as above)
            S a[8];
            if (q + 8 <= nblk) {
#pragma unroll
                for (int i = 0; i < 8; ++i) a[i] = la_load(pt + (size_t)(q + i) * w.ldp + v);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    a[i] = q + i < nblk ? la_load(pt + (size_t)(q + i) * w.ldp + v) : la_zero<S>();
            }
#pragma unroll
            for (int o = 4; o > 0; o /= 2)
#pragma unroll
                for (int i = 0; i < o; ++i) a[i] = la_add(a[i], a[i + o]);
            s = la_add(s, a[0]);
        }
        if (GR == 2 && m >= 0 && v == NX * ld + m) s = la_sub(s, la_one<S>());
        if constexpr (MD) {
            if (v >= nd) md.x[v - nd] = md.vphi[v - nd] - s;  // (to be divided by R)
            else s_d[v] = s;
        } else {
            s_d[v] = s;
        }
    }
    __syncthreads();
    // t = C^{-1} q from the rows of C^{-T} (waves 0-3) and b = C^{-T} p from
    // those of C^{-1} (waves 4-7), 64 entries at a time: lane l entry l, wave
    // w every fourth row
    const bool is_b = wave >= kLaWaves / 2;
    const S *mat = static_cast<const S *>(is_b ? w.cinv : w.cinvt), *vec = is_b ? s_d + 1 : s_d + NX * ld;
    for (int h = 0; h < k; h += 64) {
        const S *mh = mat + (h + lane < k ? h + lane : 0);
        S s = la_zero<S>();
#pragma unroll 8
        for (int r = wave & 3; r < k; r += 4) s = la_fma(la_load(mh + (size_t)r * w.ldc), vec[r], s);
        s_p[wave][lane] = s;
        __syncthreads();
        if (tid < 128 && h + lane < k) {
            const S *q = &s_p[4 * wave][lane];
            const S v = la_add(la_add(q[0], q[64]), la_add(q[128], q[192]));
            if (wave == 0) s_t[h + lane] = v;
            if (GR != 2) static_cast<S *>(wave ? w.b : w.t)[h + lane] = v;
        }
        __syncthreads();
    }
    // wave a: result a = x_a.BT[e] - sum_i (x_a.Vg[i]) t_i
    if (wave < NX) {
        S s = la_zero<S>();
        for (int i = lane; i < k; i += 64) s = la_fma(s_d[wave * ld + 1 + i], s_t[i], s);
        s = la_wave_sum(s);
        if (lane == 0) {
            const S r = la_sub(s_d[wave * ld], s);
            if (GR != 2 && wave == 0) {
                *static_cast<S *>(w.ratio) = r;
                if (!MD) la_report_s(w.words, r);
                s_r = r;
            } else {
                la_report_s(w.words + 1 + wave - X0, r);
            }
        }
    }
    if (tid == 0) *w.counter = 0u;
    if constexpr (MD) {
        for (int a = wave - 1; a < md.nu; a += kLaWaves - 1) {  // beside wave 0's R
            if (a < 0) break;
            const int j = md.uocc[a];
            double s = 0.0;
            for (int l = lane; l < k; l += 64) s = __builtin_fma(s_t[l], la_load(vg + (size_t)l * np + j), s);
            s = la_wave_sum(s);
            if (lane == 0) md.cu[a] = bte[j] - s;
        }
        __syncthreads();
        const double r = s_r;
        for (int v = tid; v < md.m; v += kLaThreads) md.x[v] /= r;
        __syncthreads();
        double s = 0.0;
        for (int d = tid; d < md.ndet; d += kLaThreads) s += md.coef[d] * md_det(md, d, true);
        s = la_block_sum(s, s_red);
        if (tid == 0) {
            md.q[0] = s;
            la_report(w.words, r * s / md.q[1]);
            la_report(w.words + 1, r);
            la_report(w.words + 2, s);
        }
    }
}

// Acceptance of the pending proposal as slot k.  Blocks 0 .. nrow - 1: rows of
// the bordered inverse, one per wave, and of its transpose; the next ncopy:
// 256 columns each of the rows appended to U and Vg and of A's new row; with
// MD the rest: 64 rows each of the table, T += c x^T with c = BT[e] - sum_l
// t_l Vg[l].  No block writes what another reads.
template <typename T, bool MD>
__global__ __launch_bounds__(kThreads) void k_la_accept(LaDev w, int n, int np, int k, int e, int nrow, int ncopy,
                                                        MdDev md) {
    typedef typename LaNum<T>::S S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int blk = blockIdx.x;
    if (blk < nrow) {
        // row i of C^{-1}: column j gets t_i (b_j / R); of C^{-T}: t_j (b_i / R)
        const bool tr = blk >= nrow / 2;
        const int i = 4 * (tr ? blk - nrow / 2 : blk) + wave;
        if (i > k) return;
        const S rinv = la_inv(*static_cast<const S *>(w.ratio));
        const S *t = static_cast<const S *>(w.t), *b = static_cast<const S *>(w.b);
        S *c = static_cast<S *>(tr ? w.cinvt : w.cinv) + (size_t)i * w.ldc;
        for (int j = lane; j <= k; j += 64) {
            const int ti = tr ? j : i, bi = tr ? i : j;  // indices of t and b
            if (ti == k) c[j] = bi == k ? rinv : la_neg_mul(b[bi], rinv);
            else if (bi == k) c[j] = la_neg_mul(t[ti], rinv);
            else c[j] = la_fma(t[ti], la_mul(b[bi], rinv), c[j]);
        }
        return;
    }
    blk -= nrow;
    const T *bte = static_cast<const T *>(w.bt) + (size_t)e * np;
    if (blk < ncopy) {
        const int c = blk * kThreads + tid;
        if (c < np) {
            const T x = static_cast<const T *>(w.phi)[c];
            static_cast<T *>(w.u)[(size_t)k * np + c] = x;
            static_cast<T *>(w.vg)[(size_t)k * np + c] = bte[c];
            static_cast<S *>(w.a)[(size_t)e * np + c] = static_cast<const S *>(w.phi64)[c];
        }
        if (c == 0) w.idx[k] = e;
        return;
    }
    blk -= ncopy;
    if constexpr (MD) {
        __shared__ double s_c[4][64];
        const int j0 = 64 * blk;
        double s = 0.0;
#pragma unroll 4
        for (int l = wave; l < k; l += 4)
            s = __builtin_fma(static_cast<const double *>(w.t)[l],
                              static_cast<const double *>(w.vg)[(size_t)l * np + j0 + lane], s);
        s_c[wave][lane] = s;
        __syncthreads();
        if (wave == 0) s_c[0][lane] = bte[j0 + lane] - (s_c[0][lane] + s_c[1][lane] + s_c[2][lane] + s_c[3][lane]);
        __syncthreads();
        double *t = md.t + (size_t)j0 * md.m;
        for (int v = tid; v < 64 * md.m && j0 + v / md.m < n; v += kThreads)
            t[v] = __builtin_fma(s_c[0][v / md.m], md.x[v % md.m], t[v]);
        if (blk == 0) {
            for (int v = tid; v < md.m; v += kThreads) md.v[(size_t)e * md.m + v] = md.vphi[v];
            if (tid == 0) md.q[1] = md.q[0];
        }
    }
}

template <typename T, int GR, bool MD = false>
static hipError_t la_propose(const LaDev &w, const LaSource &src, int n, int np, int k, int e, int m, const MdDev &md,
                             hipStream_t s) {
    // 64 real columns a block while that makes at most kLaBlocks blocks, then
    // as many more: the last block reads every block's partial sums
    typedef typename LaNum<T>::R R;
    constexpr int Z = sizeof(T) / sizeof(R), NB = Z * (GR == 0 ? 2 : (GR == 1 ? 5 : 4));
    const int ldr = Z * np, cb = 64 * ((ldr + 64 * kLaBlocks - 1) / (64 * kLaBlocks));
    const size_t lds = (size_t)NB * (cb + 16 / sizeof(R)) * sizeof(R);
    hipLaunchKernelGGL((k_lookahead<T, GR, MD>), dim3((ldr + cb - 1) / cb), dim3(kLaThreads), lds, s, w, src, n, np, cb,
                       k, e, m, md);
    return hipGetLastError();
}

template <typename T, bool MD = false>
static hipError_t la_accept(const LaDev &w, int n, int np, int k, int e, const MdDev &md, hipStream_t s) {
    const int nrow = 2 * (k / 4 + 1), ncopy = (np + kThreads - 1) / kThreads;
    hipLaunchKernelGGL((k_la_accept<T, MD>), dim3(nrow + ncopy + (MD ? np / 64 : 0)), dim3(kThreads), 0, s, w, n, np, k,
                       e, nrow, ncopy, md);
    return hipGetLastError();
}

}  // namespace dsu
