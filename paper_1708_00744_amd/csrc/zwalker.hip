// zwalker.hip -- the host-driven single walker with complex orbitals
// (twisted boundary conditions), FP64 complex arithmetic throughout.
//
// The method carries over unchanged: the determinant lemma and the Woodbury
// identity hold over the complex field with plain (not conjugate) transposes,
// so the look-ahead ratio of Sec. II, eq. (3), is R = r0 - p^T C_k^{-1} q,
// C_k^{-1} is bordered on each acceptance, and the flush is eq. (4):
// Y = BT U^T, Y[e_j][j] -= 1, W = Y C^{-T}, BT -= W Vg.  BT = (A^{-1})^T.
// The Metropolis weight is |R|^2; the walker tracks log|det A| and arg det A.
// Complex values are stored interleaved (re, im) as double2.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <vector>

#include "host_common.hpp"
#include "lookahead.hpp"

namespace dsu {

typedef double2 zc;

__device__ __forceinline__ zc zmul(zc a, zc b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ __forceinline__ zc zfma(zc a, zc b, zc c) {
    return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ zc zsub(zc a, zc b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ zc zinv(zc a) {
    const double d = a.x * a.x + a.y * a.y;
    return make_double2(a.x / d, -a.y / d);
}

// Beside the look-ahead state: the flush's and the inversion's work arrays.
struct ZWalkerDev {
    zc *bt;            // np x np
    zc *u;             // kp x np: new rows of the pending moves
    zc *vg;            // kp x np: stale BT rows of the pending electrons
    zc *a;             // np x np: Slater matrix
    zc *cinv;          // kp x (kp + 1): C_k^{-1} in pending order
    int *idx;          // kp pending electrons
    zc *w;             // np x (kp + 1): flush scratch W
    zc *work;          // np x np: the inversion's other buffer; also dsu_zget_inverse's output
    zc *panel;         // np x 16: a group's factored columns
    zc *mult;          // 16 x np: a group's multipliers, a column of M each as its pivot found it
    zc *pval;          // np: pivots
    zc *pinv;          // np: their reciprocals
    int *slot;         // np: the pivot a row was taken for
    int *piv;          // np: the row taken for a pivot
    double *stat;      // log|det|, arg det without the row order's sign, 1 if singular to working precision
    int ldc;           // kp + 1
};

// C[M x N] = (or -=) A[M x Kd] op(B); op(B) = B^T with B stored N x Kd when
// TRANSB, else B stored Kd x N.  64 x 64 tile per workgroup, 4 x 4 per thread.
template <bool TRANSB, bool SUB>
__global__ __launch_bounds__(kThreads) void k_zgemm(const zc *__restrict__ A, int lda, const zc *__restrict__ B, int ldb,
                                                    zc *C, int ldc, int M, int N, int Kd) {
    constexpr int TM = 64, TN = 64, TK = 8;
    __shared__ zc sa[TK][TM + 1], sb[TK][TN + 1];
    const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
    zc acc[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = make_double2(0.0, 0.0);
    for (int k0 = 0; k0 < Kd; k0 += TK) {
        for (int v = tid; v < TM * TK; v += kThreads) {
            const int i = v / TK, kk = v % TK, m = m0 + i, kx = k0 + kk;
            sa[kk][i] = (m < M && kx < Kd) ? A[(size_t)m * lda + kx] : make_double2(0.0, 0.0);
        }
        for (int v = tid; v < TN * TK; v += kThreads) {
            if (TRANSB) {
                const int j = v / TK, kk = v % TK, n = n0 + j, kx = k0 + kk;
                sb[kk][j] = (n < N && kx < Kd) ? B[(size_t)n * ldb + kx] : make_double2(0.0, 0.0);
            } else {
                const int kk = v / TN, j = v % TN, n = n0 + j, kx = k0 + kk;
                sb[kk][j] = (n < N && kx < Kd) ? B[(size_t)kx * ldb + n] : make_double2(0.0, 0.0);
            }
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < TK; ++kk) {
            zc a[4], bb[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) a[r] = sa[kk][ty + 16 * r];
#pragma unroll
            for (int c = 0; c < 4; ++c) bb[c] = sb[kk][tx + 16 * c];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[r][c] = zfma(a[r], bb[c], acc[r][c]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int m = m0 + ty + 16 * r, n = n0 + tx + 16 * c;
            if (m < M && n < N) {
                zc *p = C + (size_t)m * ldc + n;
                *p = SUB ? zsub(*p, acc[r][c]) : acc[r][c];
            }
        }
}

template <bool TRANSB, bool SUB>
static hipError_t zgemm(const zc *A, int lda, const zc *B, int ldb, zc *C, int ldc, int M, int N, int Kd, hipStream_t s) {
    const dim3 grid((N + 63) / 64, (M + 63) / 64);
    hipLaunchKernelGGL((k_zgemm<TRANSB, SUB>), grid, dim3(kThreads), 0, s, A, lda, B, ldb, C, ldc, M, N, Kd);
    return hipGetLastError();
}

// Flush, first half, one wave per row of BT (4 rows per workgroup): the
// row's look-ahead products y_j = BT[i] . U[j] (16 slots at a time, lanes
// striding the columns, then a wave reduction), y_j -= 1 where e_j = i, and
// the row of W = (Y - E) C^{-T}: w_j = sum_l y_l Cinv[j][l].  Bound by U's loads from
// L2: four slots' are in flight together, and each workgroup starts at a column of
// its own (all of them at the same columns of rows np elements apart meet in a
// quarter of L2's channels).  Slot by slot from column 0 a launch took 304 to 523
// us at n = 512, k = 200, by how far the waves drift apart; a flush with the next
// move's look-ahead, before and so: n = 512, k = 200 394 to 612 -> 310 us, n = 1000
// 863 to 1050 -> 392, n = 256, k = 130 200 to 260 -> 167, n = 1000, k = 8 61 to 69 -> 42.
__global__ __launch_bounds__(kThreads) void k_zflush_w(ZWalkerDev w, int np, int k) {
    __shared__ zc s_y[4][DSU_KMAX_LDS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 4 + wave;  // np is a multiple of 64: every wave has a row
    const zc *bt = w.bt + (size_t)i * np;
    for (int j0 = 0; j0 < k; j0 += 16) {
        const int nj = k - j0 < 16 ? k - j0 : 16;
        zc acc[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[j] = make_double2(0.0, 0.0);
        for (int t = 0, c = lane + 64 * (blockIdx.x % (np / 64)); t < np; t += 64, c = c + 64 < np ? c + 64 : lane) {
            const zc b = la_load(bt + c);
#pragma unroll
            for (int q = 0; q < 16; q += 4) {
                if (q >= nj) break;
                zc u[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) u[j] = la_load(w.u + (size_t)(q + j < nj ? j0 + q + j : j0) * np + c);
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[q + j] = zfma(b, u[j], acc[q + j]);
            }
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            zc v = acc[j];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                v.x += __shfl_xor(v.x, o, 64);
                v.y += __shfl_xor(v.y, o, 64);
            }
            if (lane == 0 && j < nj) s_y[wave][j0 + j] = make_double2(v.x - (w.idx[j0 + j] == i ? 1.0 : 0.0), v.y);
        }
    }
    __syncthreads();
    for (int j = lane; j < k; j += 64) {
        zc s = make_double2(0.0, 0.0);
        for (int l = 0; l < k; ++l) s = zfma(s_y[wave][l], w.cinv[(size_t)j * w.ldc + l], s);
        w.w[(size_t)i * w.ldc + j] = s;
    }
}

// ---------------------------------------------------------------------------
// Fresh inverse: in-place Gauss-Jordan on M = A^T with partial pivoting, WS
// columns (a group) at a time.  A launch pair per column with the rows moved
// in memory cost 12 us a column, the matrix's pitched upload 5 ms; now a launch
// pair per group (38 + 12 us at n = 600) and one flat upload.  New matrix in,
// inverse out: 11.7 -> 2.2 ms at n = 600, 45.9 -> 10.4 ms at n = 1500.
//  * k_zgj_group, one workgroup, thread t holds rows t + NT r of the group's
//    columns in registers, so a pivot step is one exchange through LDS and one
//    barrier;
//  * k_zgj_update applies the group's steps to all other columns, from one
//    buffer to another (the pivot rows it needs are those of the old one).  Every
//    element gets what one elimination step after the other gives it, with the
//    steps' own multipliers.  A product by the group's inverse (its factored
//    columns on the untouched pivot rows, the real part and the imaginary part
//    each accumulated from the old element) takes 6 us instead of 12 and 1.77 ms
//    instead of 2.18 in all, but its inverses' rms errors were 1.42 times those
//    of the elimination (1000 twisted-wave matrices of n = 100 and 130); these
//    are 1.00 times (+- 0.014).
// Rows are not interchanged: slot[i] names the pivot row i was taken for (-1:
// none yet).  With row p_j taken for pivot j the result holds, in row p_i and
// column j, element (i, p_j) of the inverse; k_zgj_gather puts it in place.
// The pivot is the largest in modulus, by its square, which its reciprocal needs anyway.
// ---------------------------------------------------------------------------

// M[i][j] = A[j][i] for i, j < n (zero elsewhere up to np), through LDS; slots
// cleared.  A: `in`, rows of ldi; where that is the caller's own n x n matrix
// (ldi = n), also copied to a (rows of np; its padding is zero already).
__global__ __launch_bounds__(kThreads) void k_zgj_load(const zc *in, int ldi, zc *a, zc *m, int *slot, int n, int np) {
    __shared__ zc t[32][33];
    const int x = threadIdx.x & 31, y = threadIdx.x >> 5, i0 = blockIdx.y * 32, j0 = blockIdx.x * 32;
#pragma unroll
    for (int q = 0; q < 32; q += 8) {
        const int r = j0 + y + q, c = i0 + x;  // row r, column c of A
        const bool on = r < n && c < n;
        const zc v = on ? la_load(in + (size_t)r * ldi + c) : make_double2(0.0, 0.0);
        t[y + q][x] = v;
        if (in != a && on) a[(size_t)r * np + c] = v;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 32; q += 8) m[(size_t)(i0 + y + q) * np + j0 + x] = t[x][y + q];
    if (blockIdx.x == 0 && threadIdx.x < 32) slot[i0 + threadIdx.x] = -1;
}

// Pivots k0 .. k0 + w - 1 on the group's columns; factored columns to panel
// (np x WS), the steps' multipliers to mult, pivots and their reciprocals to pval
// and pinv, the rows taken to piv and slot.  A pivot step
// is bound by its serial chain (search, exchange, reciprocal) and by 6 WS RPT
// FP64 operations a thread, on one compute unit, so:
//  * WS RPT = 32 complex values a thread on as few waves as hold the rows: what
//    a wave does once a step serves RPT rows of each lane;
//  * the pivot row sits one column a lane (in each 16 lanes) and enters the
//    multiply-adds as row broadcasts;
//  * the columns rotate by one a step (the multiply-adds write one register to
//    the left), so the pivot column is always the first, every index is fixed
//    and the body of one step stays in the instruction cache.
template <int WS, int RPT>
__global__ __launch_bounds__(512) void k_zgj_group(const zc *__restrict__ m, zc *__restrict__ panel,
                                                   zc *__restrict__ mult, int *slot, int *piv, zc *pval, zc *pinv,
                                                   int np, int n, int k0, int w) {
    __shared__ zc s_row[WS];
    __shared__ double s_key[8];
    __shared__ int s_at[8];
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
    double ax[RPT][WS], ay[RPT][WS];  // re, im
    int mine[RPT];                    // the pivot each row was taken for; -2: no row
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int i = tid + nt * r;
        const bool in = i < n;
        mine[r] = in ? slot[i] : -2;
        const zc *src = m + (size_t)(in ? i : 0) * np + k0;
#pragma unroll
        for (int c = 0; c < WS; ++c) {
            const zc v = la_load(src + c);
            ax[r][c] = in ? v.x : 0.0;
            ay[r][c] = in ? v.y : 0.0;
        }
    }
#pragma unroll 1
    for (int s = 0; s < WS; ++s) {
        double fx[RPT], fy[RPT];
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            fx[r] = ax[r][0];
            fy[r] = ay[r][0];
        }
        if (s >= w) {  // past the last column: only the rotation
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
#pragma unroll
                for (int c = 1; c < WS; ++c) {
                    ax[r][c - 1] = ax[r][c];
                    ay[r][c - 1] = ay[r][c];
                }
                ax[r][WS - 1] = fx[r];
                ay[r][WS - 1] = fy[r];
            }
            continue;
        }
        // this wave's candidate (a NaN ranks below every number, a row already taken below NaN)
        double best = -1.0;
        int bi = tid;
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const double v = __builtin_fma(fx[r], fx[r], fy[r] * fy[r]), key = mine[r] != -1 ? -1.0 : (v == v ? v : -0.5);
            if (key > best) {
                best = key;
                bi = tid + nt * r;
            }
        }
        const double top = wave_max(best);
        if (lane == __builtin_ctzll(__ballot(best == top))) {
            s_key[wave] = top;
            s_at[wave] = bi;
        }
        __syncthreads();
        // every wave picks the winner (same values, same result)
        const double key = (lane & 7) < nw ? s_key[lane & 7] : -1.0;
        const int at = s_at[lane & 7];
        const double all = lane_f64(group_max<8>(key), 0);
        const int p = __builtin_amdgcn_readlane(at, __builtin_ctzll(__ballot(key == all)));
        bool own[RPT];
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            own[r] = p == tid + nt * r;
            if (own[r])
#pragma unroll
                for (int c = 0; c < WS; ++c) s_row[c] = make_double2(ax[r][c], ay[r][c]);
        }
        __syncthreads();
        const zc rv = s_row[lane & (WS - 1)];
        const double px = row_bcast_f64<0>(rv.x), py = row_bcast_f64<0>(rv.y);
        const double d = __builtin_fma(px, px, py * py), ix = px / d, iy = -py / d;
        const double sx = __builtin_fma(rv.x, ix, -(rv.y * iy)), sy = __builtin_fma(rv.x, iy, rv.y * ix);
        if (tid == 0) {
            pval[k0 + s] = make_double2(px, py);
            pinv[k0 + s] = make_double2(ix, iy);
            piv[k0 + s] = p;
        }
#pragma unroll
        for (int r = 0; r < RPT; ++r)
            if (mine[r] != -2) (mult + (size_t)s * np + nt * r)[tid] = make_double2(fx[r], fy[r]);
#pragma unroll
        for (int r = 0; r < RPT; ++r)
            if (own[r]) {  // the pivot row itself: scaled
                mine[r] = k0 + s;
                fx[r] = fy[r] = 0.0;
#pragma unroll
                for (int c = 1; c < WS; ++c) {
                    const double x = ax[r][c], y = ay[r][c];
                    ax[r][c] = __builtin_fma(x, ix, -(y * iy));
                    ay[r][c] = __builtin_fma(x, iy, y * ix);
                }
            }
        static_for(std::make_integer_sequence<int, WS - 1>{}, [&](auto c_c) __attribute__((always_inline)) {
            constexpr int c = decltype(c_c)::value + 1;
            const double qx = row_bcast_f64<c>(sx), qy = row_bcast_f64<c>(sy);
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                ax[r][c - 1] = ax[r][c] - __builtin_fma(fx[r], qx, -(fy[r] * qy));
                ay[r][c - 1] = ay[r][c] - __builtin_fma(fx[r], qy, fy[r] * qx);
            }
        });
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            ax[r][WS - 1] = own[r] ? ix : __builtin_fma(fy[r], iy, -(fx[r] * ix));
            ay[r][WS - 1] = own[r] ? iy : -__builtin_fma(fx[r], iy, fy[r] * ix);
        }
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int i = tid + nt * r;
        if (i >= n) continue;
        if (mine[r] >= k0) slot[i] = mine[r];
        zc *dst = panel + (size_t)i * WS;
#pragma unroll
        for (int c = 0; c < WS; ++c) dst[c] = make_double2(ax[r][c], ay[r][c]);
    }
}

// a - f q, as in k_zgj_group's steps: the product first, so that one rounding at a's size is taken, not two.
__device__ __forceinline__ zc zgj_step(zc a, zc f, zc q) {
    return make_double2(a.x - __builtin_fma(f.x, q.x, -(f.y * q.y)), a.y - __builtin_fma(f.x, q.y, f.y * q.x));
}

// The group's steps on the columns outside it, panel[i][c - k0] in its own.  A
// workgroup: 16 rows x 64 columns, four rows a thread; all loads are issued before
// the products.  Its first wave takes the pivot rows through the group's steps (q_s,
// pivot row s as step s leaves it), then every row takes a - f_s q_s, s in order; a
// row taken at step t starts from q_t.
template <int WS>
__global__ __launch_bounds__(kThreads) void k_zgj_update(const zc *__restrict__ src, zc *__restrict__ dst,
                                                         const zc *__restrict__ panel, const zc *__restrict__ mult,
                                                         const int *__restrict__ slot, const int *__restrict__ piv,
                                                         const zc *__restrict__ pinv, int np, int n, int k0, int w) {
    __shared__ zc s_f[16][WS], s_fp[WS][WS], s_q[WS][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = blockIdx.x * 64 + lane, i0 = blockIdx.y * 16;
    zc v[WS], o[4];
    int at[4];
    if (wave == 0)
#pragma unroll
        for (int t = 0; t < WS; ++t) v[t] = la_load(src + (size_t)piv[k0 + (t < w ? t : 0)] * np + c);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = i0 + wave + 4 * r;
        at[r] = i < n ? __builtin_amdgcn_readfirstlane(slot[i]) - k0 : -1;  // the step that takes the row (< 0: none)
        o[r] = i < n && at[r] < 0 ? la_load(src + (size_t)i * np + c) : make_double2(0.0, 0.0);
    }
    for (int q = tid; q < 16 * WS; q += kThreads) {
        const int i = q % 16, j = q / 16;
        s_f[i][j] = i0 + i < n && j < w ? la_load(mult + (size_t)j * np + i0 + i) : make_double2(0.0, 0.0);
    }
    for (int q = tid; q < WS * WS; q += kThreads) {
        const int t = q % WS, j = q / WS;
        s_fp[t][j] = t < w && j < w ? la_load(mult + (size_t)j * np + piv[k0 + t]) : make_double2(0.0, 0.0);
    }
    __syncthreads();
    if (wave == 0)
        static_for(std::make_integer_sequence<int, WS>{}, [&](auto s_c) __attribute__((always_inline)) {
            constexpr int s = decltype(s_c)::value;
            if (s >= w) return;  // uniform
            const zc f = la_load(pinv + k0 + s), x = v[s];
            const zc q = make_double2(__builtin_fma(x.x, f.x, -(x.y * f.y)), __builtin_fma(x.x, f.y, x.y * f.x));
            s_q[s][lane] = q;
#pragma unroll
            for (int t = s + 1; t < WS; ++t) v[t] = zgj_step(v[t], s_fp[t][s], q);
        });
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (at[r] >= 0) o[r] = s_q[at[r]][lane];
#pragma unroll 4
    for (int s = 0; s < w; ++s) {
        const zc q = s_q[s][lane];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (s > at[r]) o[r] = zgj_step(o[r], s_f[wave + 4 * r][s], q);
    }
    const bool own = c >= k0 && c < k0 + w;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = i0 + wave + 4 * r;
        if (i >= n) continue;
        if (own) o[r] = la_load(panel + (size_t)i * WS + c - k0);
        dst[(size_t)i * np + c] = o[r];
    }
}

// BT[i][c] = M[p_i][slot c] for i, c < n, zero elsewhere up to np.
__global__ __launch_bounds__(kThreads) void k_zgj_gather(const zc *__restrict__ m, zc *__restrict__ bt,
                                                         const int *__restrict__ slot, const int *__restrict__ piv,
                                                         int n, int np) {
    const int c = blockIdx.x * kThreads + threadIdx.x, i = blockIdx.y;
    if (c >= np) return;
    bt[(size_t)i * np + c] = i < n && c < n ? la_load(m + (size_t)piv[i] * np + slot[c]) : make_double2(0.0, 0.0);
}

// stat[0] = sum log|p|, stat[1] = sum arg p; stat[2] = 1 if a pivot's modulus
// is at or below n 2^-52 times the largest up to it (or no number).  One
// workgroup, thread t the pivots t cnt .. + cnt.
__global__ __launch_bounds__(1024) void k_zgj_stat(const zc *__restrict__ pval, double *stat, int n) {
    __shared__ double s_mx[2][1024];
    __shared__ double s_sum[2][16];
    __shared__ int s_bad;
    const int tid = threadIdx.x, cnt = (n + 1023) / 1024, q0 = tid * cnt, q1 = q0 + cnt < n ? q0 + cnt : n;
    double ld = 0.0, ph = 0.0, mx = 0.0;
    if (tid == 0) s_bad = 0;
    for (int q = q0; q < q1; ++q) {
        const zc p = pval[q];
        const double v = hypot(p.x, p.y);
        ld += log(v);
        ph += atan2(p.y, p.x);
        mx = fmax(mx, v);
    }
    s_mx[0][tid] = mx;
    int b = 0;
    for (int o = 1; o < 1024; o *= 2, b ^= 1) {  // inclusive prefix maxima
        __syncthreads();
        s_mx[b ^ 1][tid] = tid >= o ? fmax(s_mx[b][tid], s_mx[b][tid - o]) : s_mx[b][tid];
    }
    __syncthreads();
    mx = tid > 0 ? s_mx[b][tid - 1] : 0.0;
    for (int q = q0; q < q1; ++q) {
        const double v = hypot(pval[q].x, pval[q].y);
        mx = fmax(mx, v);
        if (!(v > (double)n * 0x1p-52 * mx)) s_bad = 1;
    }
    ld = la_wave_sum(ld);
    ph = la_wave_sum(ph);
    if ((tid & 63) == 0) {
        s_sum[0][tid >> 6] = ld;
        s_sum[1][tid >> 6] = ph;
    }
    __syncthreads();
    if (tid == 0) {
        ld = ph = 0.0;
        for (int q = 0; q < 16; ++q) {
            ld += s_sum[0][q];
            ph += s_sum[1][q];
        }
        stat[0] = ld;
        stat[1] = ph;
        stat[2] = s_bad ? 1.0 : 0.0;
    }
}

// One inversion, of the n x n matrix `host` (which becomes A) or of A: M starts in the buffer from which an even or odd
// number of updates ends in `work`, and is gathered from there into BT.
template <int WS, int RPT>
static hipError_t zgj_invert(const zc *host, const ZWalkerDev &d, int n, int np, hipStream_t s) {
    zc *a = d.a, *bt = d.bt, *work = d.work, *panel = d.panel, *mult = d.mult, *pval = d.pval, *pinv = d.pinv;
    int *slot = d.slot, *piv = d.piv;
    double *stat = d.stat;
    const int groups = (n + WS - 1) / WS;
    zc *src = groups % 2 ? bt : work, *dst = groups % 2 ? work : bt;
    if (host) {  // up in one piece (a pitched copy of pageable rows goes row by row: 3 ms at n = 600)
        const hipError_t e = hipMemcpyAsync(dst, host, sizeof(zc) * n * n, hipMemcpyHostToDevice, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_zgj_load, dim3(np / 32, np / 32), dim3(kThreads), 0, s, (const zc *)(host ? dst : a),
                       host ? n : np, a, src, slot, n, np);
    const int nt = round_up((n + RPT - 1) / RPT, 64);
    for (int k0 = 0; k0 < n; k0 += WS) {
        const int w = n - k0 < WS ? n - k0 : WS;
        hipLaunchKernelGGL((k_zgj_group<WS, RPT>), dim3(1), dim3(nt), 0, s, (const zc *)src, panel, mult, slot, piv, pval,
                           pinv, np, n, k0, w);
        hipLaunchKernelGGL((k_zgj_update<WS>), dim3(np / 64, (n + 15) / 16), dim3(kThreads), 0, s, (const zc *)src, dst,
                           (const zc *)panel, (const zc *)mult, (const int *)slot, (const int *)piv, (const zc *)pinv, np,
                           n, k0, w);
        zc *t = src;
        src = dst;
        dst = t;
    }
    hipLaunchKernelGGL(k_zgj_gather, dim3((np + kThreads - 1) / kThreads, np), dim3(kThreads), 0, s, (const zc *)work, bt,
                       (const int *)slot, (const int *)piv, n, np);
    hipLaunchKernelGGL(k_zgj_stat, dim3(1), dim3(1024), 0, s, (const zc *)pval, stat, n);
    return hipGetLastError();
}

// out[i][j] = BT[j][i] (A^{-1}, n x n).
__global__ void k_zuntranspose(const zc *bt, zc *out, int n, int np) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x, i = blockIdx.y;
    if (j < n) out[(size_t)i * n + j] = bt[(size_t)j * np + i];
}

}  // namespace dsu

using namespace dsu;

struct dsu_zwalker {
    int n = 0, np = 0, K = 0, kp = 0, policy = 0;
    // scratch of the matrix-core flush (real embedding, for delays with 2k <= 256)
    double *flush_y = nullptr, *flush_w = nullptr;
    int flush_mode = DSU_FLUSH_AUTO;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    ZWalkerDev wd{};
    LaDev la{};                             // look-ahead state (shares bt, u, vg, a, cinv, idx)
    double *words_h = nullptr;              // pinned host words the look-ahead kernel writes R into
    double *row_stage = nullptr;            // mapped pinned host staging of a proposal row
    const double *row_stage_dev = nullptr;  // its device address
    std::vector<int> piv_h;                 // host copy of the pivot rows
    int k = 0, slots = 0;
    std::vector<int> idx;
    bool has_prop = false;
    int prop_e = -1;
    double prop_re = 0.0, prop_im = 0.0;
    double logabs = 0.0, phase = 0.0;
};

static double wrap_phase(double p) {
    p = std::fmod(p, 2.0 * M_PI);
    if (p > M_PI) p -= 2.0 * M_PI;
    if (p <= -M_PI) p += 2.0 * M_PI;
    return p;
}

static void zwalker_free(dsu_zwalker *w) {
    for (void *p : {(void *)w->wd.bt, (void *)w->wd.u, (void *)w->wd.vg, (void *)w->wd.a, w->la.phi,
                    (void *)w->wd.cinv, w->la.cinvt, w->la.part, w->la.t, w->la.b, w->la.ratio, (void *)w->wd.idx,
                    (void *)w->la.counter, (void *)w->wd.w, (void *)w->wd.work, (void *)w->wd.panel,
                    (void *)w->wd.mult, (void *)w->wd.pval, (void *)w->wd.pinv, (void *)w->wd.slot, (void *)w->wd.piv, (void *)w->wd.stat, (void *)w->flush_y, (void *)w->flush_w})
        dfree(p);
    if (w->words_h) (void)hipHostFree(w->words_h);
    if (w->row_stage) (void)hipHostFree(w->row_stage);
    if (w->own_stream && w->stream) (void)hipStreamDestroy(w->stream);
}

// Fresh inverse from A: BT = (A^T)^{-1} by in-place Gauss-Jordan on A^T.
static int zwalker_recompute(dsu_zwalker *w, const double *slater_host, double *logabs, double *phase) {
    const int n = w->n, np = w->np;
    const ZWalkerDev &d = w->wd;
    // 32 complex values a thread, on at most 512 threads
    auto invert = n <= 1024   ? zgj_invert<16, 2>
                  : n <= 2048 ? zgj_invert<8, 4>
                  : n <= 4096 ? zgj_invert<4, 8>
                  : n <= 8192 ? zgj_invert<2, 16>
                              : zgj_invert<1, 32>;
    HIPCHK(invert(reinterpret_cast<const zc *>(slater_host), d, n, np, w->stream));
    double st[3];
    w->piv_h.resize(n);
    HIPCHK(hipMemcpyAsync(st, d.stat, sizeof(st), hipMemcpyDeviceToHost, w->stream));
    HIPCHK(hipMemcpyAsync(w->piv_h.data(), d.piv, sizeof(int) * n, hipMemcpyDeviceToHost, w->stream));
    HIPCHK(hipStreamSynchronize(w->stream));
    if (st[2] != 0.0) return fail(DSU_ESINGULAR, "Slater matrix is singular");
    // the sign of the row order: n minus its number of cycles (an element seen is marked ~)
    int odd = n & 1;
    for (int i = 0; i < n; ++i) {
        if (w->piv_h[i] < 0) continue;
        odd ^= 1;
        for (int q = i; w->piv_h[q] >= 0;) {
            const int to = w->piv_h[q];
            w->piv_h[q] = ~to;
            q = to;
        }
    }
    *logabs = st[0];
    *phase = wrap_phase(st[1] + (odd ? M_PI : 0.0));
    return DSU_OK;
}

static int zwalker_flush(dsu_zwalker *w) {
    const int k = w->k, np = w->np;
    if (k > 0) {
        // on the matrix cores through the real embedding when its width fits
        // (2k <= 256), else W row by row and the complex product on the vector ALUs
        // (us, vector / matrix: k = 1 16 / 14 at n = 64, 30 / 27 at 1024; k = 16 52 / 26 at 500)
        const bool mfma = 2 * k <= 256 && w->flush_mode != DSU_FLUSH_VALU;
        if (mfma) {
            const FlushArgs<double> fa{(double *)w->wd.bt, (const double *)w->wd.u, (const double *)w->wd.vg,
                                       (const double *)w->wd.cinv, (const double *)w->la.cinvt, w->wd.idx, w->wd.ldc,
                                       w->flush_y, w->flush_w};
            HIPCHK((launch_flush_mfma<double, 2>(fa, np, k, w->stream)));
        } else {
            hipLaunchKernelGGL(k_zflush_w, dim3(np / 4), dim3(kThreads), 0, w->stream, w->wd, np, k);
            HIPCHK(hipGetLastError());
            HIPCHK((zgemm<false, true>(w->wd.w, w->wd.ldc, w->wd.vg, np, w->wd.bt, np, np, np, k, w->stream)));
        }
    }
    w->k = 0;
    w->slots = 0;
    std::fill(w->idx.begin(), w->idx.end(), -1);
    return DSU_OK;
}

extern "C" int dsu_zwalker_set_flush_kernel(dsu_zwalker *w, int32_t mode) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (mode != DSU_FLUSH_AUTO && mode != DSU_FLUSH_VALU && mode != DSU_FLUSH_MFMA)
        return fail(DSU_EINVAL, "bad flush kernel %d", mode);
    w->flush_mode = mode;
    return DSU_OK;
}

extern "C" int dsu_zwalker_create(int32_t n, int32_t k_delay, int32_t policy, const double *slater_host,
                                  void *hip_stream, dsu_zwalker **out) {
    if (!out) return fail(DSU_EINVAL, "out is NULL");
    *out = nullptr;
    if (n < 1 || n > 16384) return fail(DSU_EINVAL, "n = %d out of range [1, 16384]", n);
    if (k_delay < 1 || k_delay > DSU_MAX_K) return fail(DSU_EINVAL, "k_delay = %d out of range [1, %d]", k_delay, DSU_MAX_K);
    if (policy != DSU_FLUSH_K_ACCEPTED && policy != DSU_FLUSH_K_PROPOSED) return fail(DSU_EINVAL, "bad policy %d", policy);
    if (!slater_host) return fail(DSU_EINVAL, "slater matrix is NULL");
    dsu_zwalker *w = new dsu_zwalker();
    w->n = n;
    w->np = round_up(n, 64);
    w->K = k_delay;
    w->kp = kpad(k_delay);
    w->policy = policy;
    const size_t np = w->np, kp = w->kp;
    int rc = DSU_OK;
#define TRY(x)              \
    do {                    \
        rc = (x);           \
        if (rc != DSU_OK) { \
            zwalker_free(w); \
            delete w;       \
            return rc;      \
        }                   \
    } while (0)
    TRY(make_stream(hip_stream, &w->stream, &w->own_stream));
    TRY(dalloc(&w->wd.bt, np * np));
    TRY(dalloc(&w->wd.u, kp * np));
    TRY(dalloc(&w->wd.vg, kp * np));
    TRY(dalloc(&w->wd.a, np * np));
    TRY(dalloc(&w->wd.cinv, kp * (kp + 1)));
    TRY(dalloc(&w->wd.idx, kp));
    TRY(dev_alloc(&w->la.cinvt, kp * (kp + 1) * sizeof(zc)));
    TRY(dev_alloc(&w->la.phi, np * sizeof(zc)));
    TRY(dev_alloc(&w->la.t, kp * sizeof(zc)));
    TRY(dev_alloc(&w->la.b, kp * sizeof(zc)));
    TRY(dev_alloc(&w->la.ratio, sizeof(zc)));
    w->la.ldp = la_ldp((int)kp);
    TRY(dev_alloc(&w->la.part, (size_t)kLaBlocks * w->la.ldp * sizeof(zc)));
    TRY(dalloc(&w->la.counter, 1));
    w->la.bt = w->wd.bt;
    w->la.u = w->wd.u;
    w->la.vg = w->wd.vg;
    w->la.a = w->wd.a;
    w->la.phi64 = w->la.phi;
    w->la.cinv = w->wd.cinv;
    w->la.idx = w->wd.idx;
    TRY(dalloc(&w->wd.w, np * (kp + 1)));
    TRY(dalloc(&w->wd.work, np * np));
    TRY(dalloc(&w->wd.panel, np * 16));
    TRY(dalloc(&w->wd.mult, np * 16));
    TRY(dalloc(&w->wd.pval, np));
    TRY(dalloc(&w->wd.pinv, np));
    TRY(dalloc(&w->wd.slot, np));
    TRY(dalloc(&w->wd.piv, np));
    TRY(dalloc(&w->wd.stat, 3));
    const int kp2 = std::min<int>(256, 2 * (int)kp);  // padded real slots
    TRY(dalloc(&w->flush_y, flush_scratch_elems<double>(w->np, 2 * w->np, kp2)));
    TRY(dalloc(&w->flush_w, np * kp2));
    w->wd.ldc = w->la.ldc = (int)kp + 1;
    // coherent: the host watches the result words while the kernel runs
    if (hipHostMalloc((void **)&w->words_h, kLaWords * sizeof(double), hipHostMallocMapped | hipHostMallocCoherent) !=
        hipSuccess)
        TRY(fail(DSU_ENOMEM, "hipHostMalloc failed"));
    std::memset(w->words_h, 0, kLaWords * sizeof(double));
    if (hipHostMalloc((void **)&w->row_stage, 2 * np * sizeof(double), hipHostMallocMapped | hipHostMallocCoherent) !=
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
        w->la.words = static_cast<double *>(dptr);
    }
    TRY(zwalker_recompute(w, slater_host, &w->logabs, &w->phase));
    w->idx.assign(w->kp, -1);
#undef TRY
    *out = w;
    return DSU_OK;
}

extern "C" int dsu_zwalker_destroy(dsu_zwalker *w) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    (void)hipStreamSynchronize(w->stream);
    zwalker_free(w);
    delete w;
    return DSU_OK;
}

extern "C" int dsu_zpropose_ratio(dsu_zwalker *w, int32_t electron, const double *phi_host, double *ratio_out) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (electron < 0 || electron >= w->n) return fail(DSU_EINVAL, "electron %d out of range", electron);
    if (!phi_host) return fail(DSU_EINVAL, "row is NULL");
    // an electron may hold at most one pending move: apply the window first
    for (int j = 0; j < w->k; ++j)
        if (w->idx[j] == electron) {
            CHK(zwalker_flush(w));
            break;
        }
    // every earlier look-ahead was waited for, so the staging row is free
    std::memcpy(w->row_stage, phi_host, sizeof(double) * 2 * w->n);
    std::memset(w->row_stage + 2 * w->n, 0, sizeof(double) * 2 * (w->np - w->n));
    la_arm(w->words_h, 0, 2);
    HIPCHK((la_propose<zc, 0>(w->la, LaSource{w->row_stage_dev, nullptr}, w->n, w->np, w->k, electron, -1, MdDev{},
                              w->stream)));
    CHK(la_wait(w->words_h, 0, 2, w->stream));
    const volatile double *h = w->words_h;
    w->prop_re = h[0];
    w->prop_im = h[1];
    w->has_prop = true;
    w->prop_e = electron;
    if (ratio_out) {
        ratio_out[0] = w->prop_re;
        ratio_out[1] = w->prop_im;
    }
    return DSU_OK;
}

static int zwalker_slot_used(dsu_zwalker *w) {
    ++w->slots;
    const bool full = w->policy == DSU_FLUSH_K_ACCEPTED ? (w->k >= w->K) : (w->slots >= w->K);
    if (full) return zwalker_flush(w);
    return DSU_OK;
}

extern "C" int dsu_zaccept(dsu_zwalker *w) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (!w->has_prop) return fail(DSU_ESTATE, "no pending proposal");
    const double mod = std::hypot(w->prop_re, w->prop_im);
    if (!(mod > RatioFloor<double>::value) || !std::isfinite(mod))
        return fail(DSU_ESINGULAR, "ratio (%g, %g) cannot be accepted", w->prop_re, w->prop_im);
    HIPCHK((la_accept<zc>(w->la, w->n, w->np, w->k, w->prop_e, MdDev{}, w->stream)));
    w->idx[w->k] = w->prop_e;
    ++w->k;
    w->logabs += std::log(mod);
    w->phase = wrap_phase(w->phase + std::atan2(w->prop_im, w->prop_re));
    w->has_prop = false;
    return zwalker_slot_used(w);
}

extern "C" int dsu_zreject(dsu_zwalker *w) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (!w->has_prop) return fail(DSU_ESTATE, "no pending proposal");
    w->has_prop = false;
    if (w->policy == DSU_FLUSH_K_PROPOSED) return zwalker_slot_used(w);
    return DSU_OK;
}

extern "C" int dsu_zflush(dsu_zwalker *w) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    return zwalker_flush(w);
}

extern "C" int dsu_zrecompute_inverse(dsu_zwalker *w, const double *slater_host_or_null, double *logabs_out,
                                      double *phase_out, double *drift_out) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    double la, ph;
    CHK(zwalker_recompute(w, slater_host_or_null, &la, &ph));
    if (drift_out) *drift_out = w->logabs - la;
    w->logabs = la;
    w->phase = ph;
    w->k = 0;
    w->slots = 0;
    w->has_prop = false;
    std::fill(w->idx.begin(), w->idx.end(), -1);
    if (logabs_out) *logabs_out = la;
    if (phase_out) *phase_out = ph;
    return DSU_OK;
}

extern "C" int dsu_zget_inverse(dsu_zwalker *w, double *out_host) {
    if (!w || !out_host) return fail(DSU_EINVAL, "NULL argument");
    CHK(zwalker_flush(w));
    hipLaunchKernelGGL(k_zuntranspose, dim3((w->n + 255) / 256, w->n), dim3(256), 0, w->stream, (const zc *)w->wd.bt,
                       w->wd.work, w->n, w->np);
    HIPCHK(hipGetLastError());
    HIPCHK(hipMemcpyAsync(out_host, w->wd.work, sizeof(zc) * w->n * w->n, hipMemcpyDeviceToHost, w->stream));
    HIPCHK(hipStreamSynchronize(w->stream));
    return DSU_OK;
}

extern "C" int dsu_zget_logdet(dsu_zwalker *w, double *logabs, double *phase) {
    if (!w) return fail(DSU_EINVAL, "walker is NULL");
    if (logabs) *logabs = w->logabs;
    if (phase) *phase = w->phase;
    return DSU_OK;
}

extern "C" int dsu_zwalker_pending(dsu_zwalker *w, int32_t *k_out) {
    if (!w || !k_out) return fail(DSU_EINVAL, "NULL argument");
    *k_out = w->k;
    return DSU_OK;
}
