// k_linalg.hip -- matrix kernels of libdsu for gfx950.
//
//  * k_flush_y / k_flush_w / k_flush_bt: the host-driven walker's en-bloc update
//    of the inverse, Sherman-Morrison-Woodbury, eq. (4) of arXiv:1708.00744,
//    written for the transposed inverse BT:
//        Y  = BT U^T            (np x k)   U   = accepted new orbital rows
//        Y' = Y - E             E[idx_j][j] = 1
//        W  = Y' C^{-T}         C^{-1}     = inverse of I_k + V'A^{-1}U (eq. (3))
//        BT = BT - W Vg         Vg         = stale BT rows of the moved electrons
//    on matrix cores (v_mfma_*_16x16x4), one launch per product.
//  * k_flush_valu: the same update with vector ALUs, one wave per row (small k).
//  * k_gj_update: the trailing update of the Gauss-Jordan inversion,
//    M' = (row-interchanged M) - W Q, on matrix cores.
//  * Gauss-Jordan inversion with partial pivoting in FP64, blocked by panels of
//    nb columns: the O(N^3) explicit route the paper uses for direct checks.
#include "dsu_internal.hpp"
#include "tiles.hpp"

namespace dsu {

// ---------------------------------------------------------------------------
// The flush of one determinant, real (Z = 1) or complex (Z = 2, interleaved:
// the real embedding, each complex product as its four real ones).  One
// workgroup per 64 rows doing the three products back to back left all but
// N / 64 compute units idle (161 us at N = 1024, K = 64 in FP64, 644 us at N =
// 4096, K = 128 in FP32), so each product has the launch its shape asks for:
//  * Y: 64 rows x 32 slots a workgroup and, in FP64, the columns in up to 8
//    parts where the rows leave the GPU idle (partial sums, added by W's
//    launch; FP32 keeps one chain of additions per element).  Operands go from
//    global memory straight into fragments, four 128-byte steps ahead;
//  * W: a wave per 16 rows x 32 slots, C^{-T} coalesced;
//  * BT: 64 x 64 tiles, V through LDS.
// Measured, the three launches: N = 1024, K = 64 FP64 161 -> 32 us, N = 1000, K =
// 32 105 -> 25, N = 4096, K = 128 FP32 644 -> 199, complex N = 500, K = 16 51 ->
// 25 (there against W row by row on the vector units, an embedding and an update).
// ---------------------------------------------------------------------------
// Y[part][row][slot], slots kb .. kb + NT 16: real columns c of BT's row and U's
// rows.  For Z = 2 slot 2 j is (re, -im) and 2 j + 1 (im, re) of U[j].
template <typename T, int NT, int Z>
__global__ __launch_bounds__(kThreads) void k_flush_y(FlushArgs<T> fa, int np, int ldr, int kp, int nkb, int cols) {
    typedef typename Vec16<T>::type vec_t;
    constexpr int VEC = 16 / (int)sizeof(T), E = 2 * VEC, CW = 4 * E, D = 4;  // E columns a lane and step, D steps ahead
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int kb = (b % nkb) * 16 * NT, rb = (b / nkb) % (np / 64), part = b / nkb / (np / 64);
    const int c0 = part * cols, c1 = c0 + cols < ldr ? c0 + cols : ldr;
    DSU_GLOBAL const T *ap = gmem<const T>(fa.bt) + (size_t)(64 * rb + 16 * wave + lr) * ldr + E * lk;
    DSU_GLOBAL const T *bp[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) bp[t] = gmem(fa.u) + (size_t)((kb + 16 * t + lr) / Z) * ldr + E * lk;
    typename Mma<T>::acc_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = typename Mma<T>::acc_t{0, 0, 0, 0};
    vec_t a[D][2], bv[D][NT][2];
    auto load = [&](int d, int c) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            a[d][h] = *(DSU_GLOBAL const vec_t *)(ap + c + h * VEC);
#pragma unroll
            for (int t = 0; t < NT; ++t) bv[d][t][h] = *(DSU_GLOBAL const vec_t *)(bp[t] + c + h * VEC);
        }
    };
    // Z = 2: a step's four matrix instructions, and the ring's steps, are added in
    // pairs (one chain along the row made the update's errors 1.2 to 1.7 times those
    // of sums over lanes in a tree)
    const typename Mma<T>::acc_t zero{0, 0, 0, 0};
    typename Mma<T>::acc_t sum[D][NT];
    auto mul = [&](int d) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if constexpr (Z == 2) {  // (kb and 16 t are even: lr's parity is the slot's)
                typename Mma<T>::acc_t m[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const T re = bv[d][t][h][0], im = bv[d][t][h][1];
                    m[h] = Mma<T>::mma(a[d][h][0], lr & 1 ? im : re, zero) +
                           Mma<T>::mma(a[d][h][1], lr & 1 ? re : -im, zero);
                }
                sum[d][t] = m[0] + m[1];
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int q = 0; q < VEC; ++q) acc[t] = Mma<T>::mma(a[d][h][q], bv[d][t][h][q], acc[t]);
            }
        }
    };
    // c1 - c0 is a multiple of CW; D steps loaded ahead, in a ring
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, c0 + d * CW < c1 ? c0 + d * CW : c0);
    for (int c = c0; c < c1; c += D * CW) {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (c + d * CW < c1) {
                mul(d);
                const int cn = c + (D + d) * CW;
                load(d, cn < c1 ? cn : c0);
            } else {
#pragma unroll
                for (int t = 0; t < NT; ++t) sum[d][t] = zero;
            }
        if constexpr (Z == 2)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] += (sum[0][t] + sum[1][t]) + (sum[2][t] + sum[3][t]);
    }
    T *y = fa.y + ((size_t)part * np + 64 * rb + 16 * wave + Mma<T>::row0(lane)) * kp + kb + lr;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) y[(size_t)i * Mma<T>::row_step * kp + 16 * t] = acc[t][i];
}

// W[row][l] = sum_j (Y - E)[row][j] C^{-1}[l][j] for 16 NT of the (real) slots
// l, one wave per 16 rows; C^{-1} taken as zero beyond kslots (complex) slots.
// The row's Y values (sums of the parts) are in registers before the products.
template <typename T, int KP, int NT, int Z>
__global__ __launch_bounds__(64) void k_flush_w(FlushArgs<T> fa, int np, int parts, int kslots) {
    constexpr int S = KP / 4, nkb = KP / (16 * NT);
    const int lane = threadIdx.x, lr = lane & 15, lk = lane >> 4;
    const int kb = (blockIdx.x % nkb) * 16 * NT, row = blockIdx.x / nkb * 16 + lr;
    DSU_GLOBAL const T *y = gmem<const T>(fa.y) + (size_t)row * KP + lk;
    DSU_GLOBAL const double *ct = gmem(fa.cinvt);
    DSU_GLOBAL const int *idx = gmem(fa.idx);
    T a[S];
    int e[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        a[s] = y[4 * s];
        e[s] = idx[(4 * s + lk) / Z < kslots ? (4 * s + lk) / Z : 0];
    }
#pragma unroll 2
    for (int q = 1; q < parts; ++q)
#pragma unroll
        for (int s = 0; s < S; ++s) a[s] += y[(size_t)q * np * KP + 4 * s];
    typename Mma<T>::acc_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = typename Mma<T>::acc_t{0, 0, 0, 0};
    constexpr int B = S < 16 ? S : 16;  // steps whose C^{-T} loads are in flight together
#pragma unroll
    for (int s0 = 0; s0 < S; s0 += B) {
        if (4 * s0 >= Z * kslots) break;
        double c[B][NT];
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int j = 4 * (s0 + b) + lk, l = kb + 16 * t + lr, jz = j / Z, lz = l / Z;
                const bool in = jz < kslots && lz < kslots;
                DSU_GLOBAL const double *p = ct + (size_t)Z * (in ? (size_t)jz * fa.ldc + lz : 0);
                if constexpr (Z == 2) {
                    // (y_re, y_im) times (c_re, c_im): re takes c_re, -c_im; im takes c_im, c_re
                    const double v = p[(l ^ j) & 1];
                    c[b][t] = !in ? 0.0 : ((l & 1) < (j & 1) ? -v : v);
                } else {
                    c[b][t] = in ? p[0] : 0.0;
                }
            }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int j = 4 * (s0 + b) + lk;
            T v = a[s0 + b];
            if (j / Z >= kslots) v = T(0);
            else if (j % Z == 0 && e[s0 + b] == row) v -= T(1);
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = Mma<T>::mma(v, T(c[b][t]), acc[t]);
        }
    }
    T *w = fa.w + (size_t)(blockIdx.x / nkb * 16 + Mma<T>::row0(lane)) * KP + kb + lr;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) w[(size_t)i * Mma<T>::row_step * KP + 16 * t] = acc[t][i];
}

// One 64 x 64 tile of BT -= W Vg (real columns; Z = 2: row 2 j of the embedded
// Vg is (re, im) of Vg[j], row 2 j + 1 (-im, re)).
template <typename T, int KP, int Z>
__global__ __launch_bounds__(kThreads) void k_flush_bt(FlushArgs<T> fa, int ldr, int ncb) {
    typedef Phase3Cfg<T, KP> C;
    typedef typename Vec16<T>::type vec_t;
    constexpr int CW = C::CW, LDV = C::LDV, VEC = 16 / (int)sizeof(T), RS = Mma<T>::row_step;
    constexpr int NV = KP * (CW / VEC) / kThreads;
    __shared__ __attribute__((aligned(16))) T lds[KP * LDV];
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int r0 = (b / ncb) * 64, cb = (b % ncb) * 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    DSU_GLOBAL const T *wr = gmem<const T>(fa.w) + (size_t)(r0 + 16 * wave + (lane & 15)) * KP + (lane >> 4);
    DSU_GLOBAL T *rp = gmem(fa.bt) + (size_t)(r0 + 16 * wave + Mma<T>::row0(lane)) * ldr + cb + (lane & 15);
    DSU_GLOBAL const T *vg = gmem(fa.vg) + cb;
    T wa[KP / 4];
#pragma unroll
    for (int s = 0; s < KP / 4; ++s) wa[s] = -wr[4 * s];
    for (int c0 = 0; c0 < 64; c0 += CW) {
        vec_t sv[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int v = tid + q * kThreads, r = v / (CW / VEC), cc = (v % (CW / VEC)) * VEC;
            sv[q] = *(DSU_GLOBAL const vec_t *)(vg + (size_t)(r / Z) * ldr + c0 + cc);
            if constexpr (Z == 2)
                if (r & 1) sv[q] = vec_t{-sv[q][1], sv[q][0]};
        }
        typename Mma<T>::acc_t acc[CW / 16];
#pragma unroll
        for (int t = 0; t < CW / 16; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[t][i] = rp[(size_t)(i * RS) * ldr + c0 + 16 * t];
        if (c0 > 0) __syncthreads();
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int v = tid + q * kThreads, r = v / (CW / VEC), cc = (v % (CW / VEC)) * VEC;
            *reinterpret_cast<vec_t *>(lds + r * LDV + cc) = sv[q];
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < KP / 4; ++s) {
            const T *bp = lds + (4 * s + (lane >> 4)) * LDV + (lane & 15);
#pragma unroll
            for (int t = 0; t < CW / 16; ++t) acc[t] = Mma<T>::mma(wa[s], bp[16 * t], acc[t]);
        }
#pragma unroll
        for (int t = 0; t < CW / 16; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) rp[(size_t)(i * RS) * ldr + c0 + 16 * t] = acc[t][i];
    }
}

// Column parts of Y's launch: FP64 only, up to 8, while the launch has fewer
// than 256 workgroups and a part at least 128 columns.
template <typename T> static int flush_parts(int np, int ldr, int kp) {
    int p = 1;
    if (sizeof(T) == 8)
        while (p < 8 && (np / 64) * (kp / (kp > 16 ? 32 : 16)) * p < 256 && ldr / (2 * p) >= 128) p *= 2;
    return p;
}

template <typename T> size_t flush_scratch_elems(int np, int ldr, int kp_max) {
    size_t most = 0;
    for (int kp = 16; kp <= kp_max; kp *= 2) {
        const size_t e = (size_t)flush_parts<T>(np, ldr, kp) * np * kp;
        most = e > most ? e : most;
    }
    return most;
}
template size_t flush_scratch_elems<float>(int, int, int);
template size_t flush_scratch_elems<double>(int, int, int);

template <typename T, int KP> struct FlushLds {
    static constexpr int LDY = KP + 16 / (int)sizeof(T);
    static constexpr int p1 = KP * (128 / (int)sizeof(T) + 16 / (int)sizeof(T));
    static constexpr int p2 = 64 * LDY + WCfg<T, KP>::elems;  // Y' block + staged C chunk
    static constexpr int p3 = KP * Phase3Cfg<T, KP>::LDV;
    static constexpr int m12 = p1 > p2 ? p1 : p2;
    static constexpr int elems = m12 > p3 ? m12 : p3;
};

// ---------------------------------------------------------------------------
// The three products of eq. (4) in one launch, 64 rows per workgroup: for
// matrices of at most FusedRows padded rows, where two launches fewer count
// more than idle compute units.  A flush and the next move's look-ahead, us, one
// launch against three, at 16 / 32 / 64 / 128 slots.  FP64: np = 64 15.6 / 17.5 / 22.9 /
// - and 20.1 / 23.6 / 26.9 / -, 128 21.7 / 24.8 / 34.7 / 70 and 23.9 / 28.2 / 31.6 / 38,
// 192 26.5 / 31.6 / 45.9 / 92 and 26.5 / 31.8 / 35.4 / 42.  FP32: np = 128 16.7 / 18.7 / 24.6
// / 39 and 22.0 / 28.0 / 34.0 / 43, 192 19 / 22 / 31 / 51 and 24 / 30 / 36 / 48, 256 22 / 26 /
// 37 / 61 and 25 / 31 / 38 / 52, 320 24 / 29 / 42 / 72 and 26 / 33 / 40 / 51, 448 29 / 36 / 54 / 92
// and 28 / 37 / 43 / 57.
// ---------------------------------------------------------------------------
template <typename T, int KP> struct FusedRows {
    static constexpr int value = sizeof(T) == 8 ? (KP <= 32 ? 128 : 64) : (KP <= 32 ? 320 : (KP == 64 ? 256 : 128));
};

template <typename T, int KP>
__global__ __launch_bounds__(kThreads) void k_flush_fused(FlushArgs<T> fd, int ld, int kslots) {
    __shared__ __attribute__((aligned(16))) T lds[FlushLds<T, KP>::elems];
    constexpr int LDY = FlushLds<T, KP>::LDY;
    const int r0 = blockIdx.x * kRowBlock;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    typename Mma<T>::acc_t acc[KP / 16];
    rowblock_times_ut<T, KP>(fd.bt + (size_t)r0 * ld, ld, kRowBlock, fd.u, ld, 0, ld, lds, acc);

    // Y block -> LDS, subtract E, then W = Y' C^{-T} on matrix cores.
#pragma unroll
    for (int t = 0; t < KP / 16; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) lds[(16 * wave + Mma<T>::row0(lane) + i * Mma<T>::row_step) * LDY + 16 * t + (lane & 15)] = acc[t][i];
    __syncthreads();
    for (int j = tid; j < kslots; j += kThreads) {
        const int e = fd.idx[j];
        if (e >= r0 && e < r0 + kRowBlock) lds[(e - r0) * LDY + j] -= T(1);
    }
    __syncthreads();
    typename Mma<T>::acc_t wacc[KP / 16];
    w_from_y<T, KP>(lds, LDY, fd.cinv, fd.ldc, kslots, lds + 64 * LDY, wacc);
#pragma unroll
    for (int t = 0; t < KP / 16; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) lds[(16 * wave + Mma<T>::row0(lane) + i * Mma<T>::row_step) * LDY + 16 * t + (lane & 15)] = wacc[t][i];
    __syncthreads();
    T wa[KP / 4];
#pragma unroll
    for (int s = 0; s < KP / 4; ++s) wa[s] = -lds[(16 * wave + (lane & 15)) * LDY + 4 * s + (lane >> 4)];
    __syncthreads();
    rowblock_plus_wv<T, KP>(fd.bt + (size_t)r0 * ld, ld, ld, fd.vg, ld, wa, lds);
}

template <typename T, int KP, int Z>
static hipError_t flush_mfma(const FlushArgs<T> &fa, int np, int kslots, hipStream_t s) {
    if constexpr (Z == 1)
        if (np <= FusedRows<T, KP>::value) {
            hipLaunchKernelGGL((k_flush_fused<T, KP>), dim3(np / kRowBlock), dim3(kThreads), 0, s, fa, np, kslots);
            return hipGetLastError();
        }
    constexpr int NT = KP > 16 ? 2 : 1;
    const int ldr = Z * np, nkb = KP / (16 * NT), parts = flush_parts<T>(np, ldr, KP);
    // whole steps of 128 bytes a part
    const int step = 128 / (int)sizeof(T), cols = ((ldr + parts - 1) / parts + step - 1) / step * step;
    hipLaunchKernelGGL((k_flush_y<T, NT, Z>), dim3((np / 64) * nkb * parts), dim3(kThreads), 0, s, fa, np, ldr, KP, nkb,
                       cols);
    hipLaunchKernelGGL((k_flush_w<T, KP, NT, Z>), dim3((np / 16) * nkb), dim3(64), 0, s, fa, np, parts, kslots);
    hipLaunchKernelGGL((k_flush_bt<T, KP, Z>), dim3((np / 64) * (ldr / 64)), dim3(kThreads), 0, s, fa, ldr, ldr / 64);
    return hipGetLastError();
}

template <typename T, int Z> hipError_t launch_flush_mfma(const FlushArgs<T> &fa, int np, int kslots, hipStream_t s) {
    if (kslots <= 0) return hipSuccess;
    const int kr = Z * kslots;
    if (kr <= 16) return flush_mfma<T, 16, Z>(fa, np, kslots, s);
    if (kr <= 32) return flush_mfma<T, 32, Z>(fa, np, kslots, s);
    if (kr <= 64) return flush_mfma<T, 64, Z>(fa, np, kslots, s);
    if (kr <= 128) return flush_mfma<T, 128, Z>(fa, np, kslots, s);
    if (kr <= 256) return flush_mfma<T, 256, Z>(fa, np, kslots, s);
    return hipErrorInvalidValue;
}
template hipError_t launch_flush_mfma<float, 1>(const FlushArgs<float> &, int, int, hipStream_t);
template hipError_t launch_flush_mfma<double, 1>(const FlushArgs<double> &, int, int, hipStream_t);
template hipError_t launch_flush_mfma<double, 2>(const FlushArgs<double> &, int, int, hipStream_t);

// ---------------------------------------------------------------------------
// VALU flush: one wave per row of BT, k <= KMAX slots in registers.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

template <typename T, int KMAX>
__global__ __launch_bounds__(kThreads) void k_flush_valu(FlushArgs<T> fd, int np, int kslots) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = blockIdx.x * 4 + wave;
    T *bt = fd.bt + (size_t)row * np;
    T y[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) y[j] = T(0);
    for (int c = lane; c < np; c += 64) {
        const T x = bt[c];
#pragma unroll
        for (int j = 0; j < KMAX; ++j)
            if (j < kslots) y[j] += x * fd.u[(size_t)j * np + c];
    }
    T w[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        y[j] = wave_sum(y[j]);
        if (j < kslots && fd.idx[j] == row) y[j] -= T(1);
    }
#pragma unroll
    for (int l = 0; l < KMAX; ++l) {
        T s = T(0);
#pragma unroll
        for (int j = 0; j < KMAX; ++j)
            if (l < kslots && j < kslots) s += T(fd.cinv[(size_t)l * fd.ldc + j]) * y[j];
        w[l] = s;
    }
    for (int c = lane; c < np; c += 64) {
        T x = bt[c];
#pragma unroll
        for (int l = 0; l < KMAX; ++l)
            if (l < kslots) x -= w[l] * fd.vg[(size_t)l * np + c];
        bt[c] = x;
    }
}

template <typename T> hipError_t launch_flush_valu(const FlushArgs<T> &fa, int np, int kslots, hipStream_t s) {
    if (kslots <= 0) return hipSuccess;
#define DSU_VALU(KM)                                                                                   \
    if (kslots <= KM) {                                                                                \
        hipLaunchKernelGGL((k_flush_valu<T, KM>), dim3(np / 4), dim3(kThreads), 0, s, fa, np, kslots); \
        return hipGetLastError();                                                                      \
    }
    DSU_VALU(1) DSU_VALU(2) DSU_VALU(4) DSU_VALU(8) DSU_VALU(16) DSU_VALU(32) DSU_VALU(64)
#undef DSU_VALU
    return hipErrorInvalidValue;
}
template hipError_t launch_flush_valu<float>(const FlushArgs<float> &, int, int, hipStream_t);
template hipError_t launch_flush_valu<double>(const FlushArgs<double> &, int, int, hipStream_t);

// ---------------------------------------------------------------------------
// Blocked Gauss-Jordan inversion (FP64, in place, partial pivoting).
// For a panel of columns R = [k0, k1): factor the panel with the unblocked
// in-place Gauss-Jordan step (pivot = largest |entry| among rows >= k, lowest
// index on ties), recording the row swaps.  The panel then holds the columns
// R of the accumulated elimination matrix T.  The other columns follow from
// the swapped pivot rows Q = M[R, :] as  M <- M - (E_R - T) Q.
// After the last panel, column swaps in reverse pivot order unscramble the
// inverse.  logdet = sum ln|pivot|, sign = swap parity * prod sign(pivot).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void argmax_combine(double &v, int &i, double v2, int i2) {
    if (v2 > v || (v2 == v && i2 < i)) { v = v2; i = i2; }
}

// One workgroup per determinant.  The panel P is column-major (P[j*np + i]).
__global__ __launch_bounds__(kThreads) void k_gj_panel(const GjDesc *__restrict__ descs, int n, int np, int nb, int k0,
                                                       int k1) {
    __shared__ double s_v[kThreads / 64];
    __shared__ int s_i[kThreads / 64];
    __shared__ double s_row[64];
    __shared__ int s_p;
    const GjDesc g = descs[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int w = k1 - k0;
    double *P = g.panel;
    for (int v = tid; v < np * w; v += kThreads) {
        const int j = v / np, i = v % np;
        P[(size_t)j * np + i] = g.m[(size_t)i * np + k0 + j];
    }
    if (k0 == 0 && tid == 0) { *g.logdet = 0.0; *g.sign = 1; *g.status = 0; *g.pmax = 0.0; }
    __syncthreads();
    for (int kk = 0; kk < w; ++kk) {
        const int k = k0 + kk;
        const double *pc = P + (size_t)kk * np;
        double best = -1.0;
        int bi = n;
        for (int i = k + tid; i < n; i += kThreads) argmax_combine(best, bi, fabs(pc[i]), i);
        for (int o = 32; o > 0; o >>= 1) {
            const double v2 = __shfl_xor(best, o, 64);
            const int i2 = __shfl_xor(bi, o, 64);
            argmax_combine(best, bi, v2, i2);
        }
        if (lane == 0) { s_v[wave] = best; s_i[wave] = bi; }
        __syncthreads();
        if (tid == 0) {
            double bv = s_v[0];
            int bidx = s_i[0];
            for (int q = 1; q < kThreads / 64; ++q) argmax_combine(bv, bidx, s_v[q], s_i[q]);
            // singular when the best pivot is at rounding level of the largest one
            const double pm = fmax(*g.pmax, bv);
            *g.pmax = pm;
            if (!(bv > (double)n * 2.220446049250313e-16 * pm)) { *g.status = -3; bidx = k; }
            s_p = bidx;
            g.piv[k] = bidx;
        }
        __syncthreads();
        const int p = s_p;
        if (p != k && tid < w) {
            double *col = P + (size_t)tid * np;
            const double t = col[k];
            col[k] = col[p];
            col[p] = t;
        }
        __syncthreads();
        const double d = P[(size_t)kk * np + k];
        if (tid == 0) {
            if (d != 0.0) *g.logdet += log(fabs(d));
            int sg = *g.sign;
            if (p != k) sg = -sg;
            if (d < 0.0) sg = -sg;
            *g.sign = sg;
        }
        const double dinv = d != 0.0 ? 1.0 / d : 0.0;
        if (tid < w) s_row[tid] = tid == kk ? dinv : P[(size_t)tid * np + k] * dinv;
        __syncthreads();
        // each thread owns whole rows: read the multiplier first, then update
        for (int i = tid; i < np; i += kThreads) {
            if (i == k) {
                for (int j = 0; j < w; ++j) P[(size_t)j * np + i] = s_row[j];
                continue;
            }
            const double f = P[(size_t)kk * np + i];
            for (int j = 0; j < w; ++j) {
                if (j == kk) P[(size_t)j * np + i] = -f * dinv;
                else P[(size_t)j * np + i] -= f * s_row[j];
            }
        }
        __syncthreads();
    }
}

// The row whose old contents end up at row x after the interchanges k0 + q <->
// piv[q], q = 0 .. w - 1, in that order.
__device__ __forceinline__ int gj_trace(int x, const int *piv, int k0, int w) {
    for (int q = w - 1; q >= 0; --q) x = x == k0 + q ? piv[q] : (x == piv[q] ? k0 + q : x);
    return x;
}

// Compose the interchanges `piv` (of rows k0 .. k0 + w - 1, in LDS) into the
// running map of all interchanges so far: perm[r] = the row of the first matrix
// whose contents row r holds now.  src = gj_trace of row r, thread tid < 2 w.
__device__ __forceinline__ void gj_total_map(int *perm, int r, int src, bool on) {
    const int from = on ? perm[src] : 0;
    __syncthreads();  // every source read before any row changes
    if (on) perm[r] = from;  // rows named twice get the same value
}

// The panel's row interchanges, composed: rowsrc[i] = the row of M whose
// contents row i holds after the swaps k <-> piv[k], k = k0 .. k1-1, in order
// (one workgroup per determinant).  At most 2 (k1 - k0) rows move, each traced
// by its own thread; the rest stay i.
__global__ __launch_bounds__(kThreads) void k_gj_rowsrc(const GjDesc *__restrict__ descs, int np, int k0, int k1) {
    __shared__ int s_piv[64];
    const GjDesc g = descs[blockIdx.x];
    const int w = k1 - k0, tid = threadIdx.x;
    if (tid < w) s_piv[tid] = g.piv[k0 + tid];
    for (int i = tid; i < np; i += kThreads) {
        g.rowsrc[i] = i;
        if (k0 == 0) g.perm[i] = i;
    }
    __syncthreads();
    const bool on = tid < 2 * w;
    const int r = on ? (tid < w ? k0 + tid : s_piv[tid - w]) : 0, x = on ? gj_trace(r, s_piv, k0, w) : 0;
    if (on) g.rowsrc[r] = x;
    gj_total_map(g.perm, r, x, on);
}

// Trailing update with the row interchanges folded in, into the other buffer:
//     m2[i][c] = m[rowsrc[i]][c] - sum_j W[i][j] Q[j][c]     (c outside the panel)
//     m2[i][c] = T[i][c - k0]                                 (the panel's columns)
// One workgroup per 64 RT rows (wave w: RT row tiles of 16 rows, their W
// fragments in registers), FP64 16x16x4 matrix cores, the columns in chunks
// of CW = 32 or 64 (two or four 16-wide tiles; 16 for a pair, whose Q chunk then
// takes 32 KB of LDS and leaves room for three workgroups a compute unit instead
// of two: 362 -> 328 us a launch at N = 1024, 64 determinants, 52 TFLOP/s):
//  * Q chunks go global -> LDS directly (no registers), double-buffered in two
//    arrays the compiler can tell apart, so the next chunk's copy stays in
//    flight while the current chunk's products read the other array; each B
//    operand read from LDS serves the wave's RT row tiles;
//  * two accumulator sets serve even and odd chunks: while one set runs a
//    chunk's products, the other is stored (the previous chunk's results) and
//    reloaded with the next chunk's source rows, so every global access has a
//    chunk of products to complete in before the barrier that waits for it.
// PAIR: two 64-column panels R1 = [k0, k0 + 64) and R2 = [k0 + 64, k0 + 128)
// in one pass (KP = 128).  With P1, P2 the panels' interchanges, T1, T2 their
// factored columns and Q1 = (P1 M)[R1], Q2 = (P2 M1)[R2] the pivot rows
// before each panel's update (M1 = M after the first panel):
//     m2 = P2 P1 M + P2 (T1 - E1) Q1 + (T2 - E2) Q2
// outside R1 and R2; rowsrc holds P2 P1, rowsrc_b P2, qrow the rows of M
// that are Q1, q2 the rows Q2.  R2's columns are T2 (the tail below), R1's
// are written afterwards by k_gj_pair_fix.
template <int KP, int RT, int CW, bool PAIR = false>
__global__ __launch_bounds__(kThreads, PAIR ? 3 : 2) void k_gj_update(const GjDesc *__restrict__ descs, int np,
                                                                      int nblk, int parts, int k0, int w) {
    constexpr int NT = CW / 16, RB = 64 * RT;
    constexpr int PIECES = KP * CW / 2;         // 16-byte pieces of one Q chunk
    constexpr int IPW = PIECES / kThreads;      // direct copies per wave per chunk (64 pieces each)
    static_assert(IPW >= 1 && IPW * kThreads == PIECES, "copy split");
    static_assert(!PAIR || KP == 128, "a pair is two 64-column panels");
    __shared__ __attribute__((aligned(16))) double q_even[KP * CW];
    __shared__ __attribute__((aligned(16))) double q_odd[KP * CW];
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int d = b / (nblk * parts), r0 = (b % nblk) * RB;
    // this workgroup's columns: a part of whole chunk pairs
    const int cols = (np / (2 * CW) + parts - 1) / parts * (2 * CW), cbeg = b / nblk % parts * cols;
    const int cend = cbeg + cols < np ? cbeg + cols : np;
    if (cbeg >= cend) return;
    const GjDesc g = descs[d];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lk = lane >> 4;
    DSU_GLOBAL const double *msrc = gmem(g.m);
    DSU_GLOBAL double *mdst = gmem(g.m2);
    // -W = T - E_R from the factored panel T (column-major), zero beyond its width
    double wa[RT][KP / 4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int ra = r0 + 16 * (RT * wave + rt) + lr;
        DSU_GLOBAL const double *tp = gmem(g.panel) + ra;
        if constexpr (PAIR) {
            // steps s < 16 are the first panel's columns j < 64 (row P2[ra] of T1 - E1),
            // the rest the second panel's (row ra of T2 - E2)
            const int rb = g.rowsrc_b[ra];
            DSU_GLOBAL const double *tb = gmem(g.panel_b) + rb;
#pragma unroll
            for (int s = 0; s < KP / 4; ++s) {
                const int j = 4 * s + lk;
                wa[rt][s] = s < KP / 8 ? tb[(size_t)j * np] - (rb == k0 + j ? 1.0 : 0.0)
                                       : tp[(size_t)(j - KP / 2) * np] - (ra == k0 + j ? 1.0 : 0.0);
            }
        } else {
#pragma unroll
            for (int s = 0; s < KP / 4; ++s) {
                const int j = 4 * s + lk;
                wa[rt][s] = j < w ? tp[(size_t)j * np] - (ra == k0 + j ? 1.0 : 0.0) : 0.0;
            }
        }
    }
    // Q row j = row k0 + j after the interchanges = M[rowsrc[k0 + j]] (rows
    // j >= w meet zero columns of W; the panel's own columns of the result
    // are replaced below).  This lane's copy pieces: piece p = (wave * IPW +
    // i) * 64 + lane lands at LDS byte 16 p, i.e. Q row p / (CW / 2), columns
    // 2 (p % (CW / 2)) + {0, 1} of the chunk
    // (a pair's Q rows 64.. are the rows of q2)
    size_t qoff[IPW];
    DSU_GLOBAL const double *qbase[IPW];
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
        const int p = (wave * IPW + i) * 64 + lane, qr = p / (CW / 2);
        if constexpr (PAIR) {
            qbase[i] = qr < KP / 2 ? msrc : gmem<const double>(g.q2);
            qoff[i] = (size_t)(qr < KP / 2 ? g.qrow[qr] : qr - KP / 2) * np + 2 * (p % (CW / 2));
        } else {
            qbase[i] = msrc;
            qoff[i] = (size_t)g.rowsrc[k0 + qr] * np + 2 * (p % (CW / 2));
        }
    }
    auto copy_q = [&](int c0, double *dstl) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < IPW; ++i)
            __builtin_amdgcn_global_load_lds((const DSU_GLOBAL void *)(qbase[i] + qoff[i] + c0),
                                             (__attribute__((address_space(3))) void *)(dstl + (wave * IPW + i) * 128),
                                             16, 0, 0);
    };
    // result rows of this lane (FP64 tile layout: row (lane / 16) + 4 i), column lr of each tile
    int row[RT][4];
    DSU_GLOBAL const double *src[RT][4];
    DSU_GLOBAL double *dst[RT][4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            row[rt][i] = r0 + 16 * (RT * wave + rt) + Mma<double>::row0(lane) + i * Mma<double>::row_step;
            src[rt][i] = msrc + (size_t)g.rowsrc[row[rt][i]] * np + lr;
            dst[rt][i] = mdst + (size_t)row[rt][i] * np + lr;
        }
    typedef Mma<double>::acc_t acc_set[RT][NT];
    acc_set acc_e, acc_o;
    copy_q(cbeg, q_even);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc_e[rt][t][i] = src[rt][i][cbeg + 16 * t];
    // chunk c0 runs its products on `cur` (loaded with its source rows) and Q
    // in q_cur; `oth` holds chunk c0 - CW's results (c0 > cbeg), is stored, and
    // takes chunk c0 + CW's source rows (the last chunk re-reads its own rows,
    // so the load is unconditional)
    auto chunk = [&](int c0, const double *q_cur, double *q_nxt, acc_set &cur, acc_set &oth)
        __attribute__((always_inline)) {
        // chunk c0's Q is in q_cur (the barrier waits for this wave's copies,
        // and with them for everything issued before); every wave is done
        // reading q_nxt
        __syncthreads();
        if (c0 > cbeg)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) dst[rt][i][c0 - CW + 16 * t] = oth[rt][t][i];
        const int c1 = c0 + CW;
        if (c1 < cend) copy_q(c1, q_nxt);
        const int cl = c1 < cend ? c1 : c0;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) oth[rt][t][i] = src[rt][i][cl + 16 * t];
        __builtin_amdgcn_sched_barrier(0);  // stores and next loads issued before the products
        const double *qb = q_cur + lk * CW + lr;
#pragma unroll
        for (int s = 0; s < KP / 4; ++s)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const double bq = qb[4 * s * CW + 16 * t];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) cur[rt][t] = Mma<double>::mma(wa[rt][s], bq, cur[rt][t]);
            }
    };
    // np is a multiple of 2 CW (the launcher's choice of CW): chunks come in
    // pairs, and the loop body is straight-line code over fixed register sets
    for (int c0 = cbeg; c0 < cend; c0 += 2 * CW) {
        chunk(c0, q_even, q_odd, acc_e, acc_o);
        chunk(c0 + CW, q_odd, q_even, acc_o, acc_e);
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[rt][i][cend - CW + 16 * t] = acc_o[rt][t][i];
    // The panel's columns (a pair's second panel): the lane that stored each of
    // them overwrites it with the factored panel (same thread, same address:
    // program order holds).
    const int tk0 = PAIR ? k0 + KP / 2 : k0, tw = PAIR ? KP / 2 : w;
    const int tbeg = tk0 - tk0 % CW, tend = tk0 + tw < cend ? tk0 + tw : cend;
    for (int c0 = tbeg > cbeg ? tbeg : cbeg; c0 < tend; c0 += CW)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int c = c0 + 16 * t + lr;
            if (c >= tk0 && c < tk0 + tw)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        dst[rt][i][c - lr] = g.panel[(size_t)(c - tk0) * np + row[rt][i]];
        }
}

// ---------------------------------------------------------------------------
// Two-level panel factorisation (same algebra one level down): the panel's
// columns are factored WS at a time by one workgroup per determinant
// (k_gj_group), and each group's rank-WS update reaches the panel's other
// columns through k_gj_apply, spread over many workgroups.
// ---------------------------------------------------------------------------

// P[j][i] = M[i][k0 + j] for the panel's w columns (64-row tiles through LDS,
// every load of a thread in flight at once).
__global__ __launch_bounds__(kThreads) void k_gj_gather(const GjDesc *__restrict__ descs, int np, int k0, int w) {
    __shared__ double t[64][65];
    const GjDesc g = descs[blockIdx.y];
    const int r0 = blockIdx.x * 64, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    DSU_GLOBAL const double *m = gmem<const double>(g.m) + (size_t)r0 * np + k0 + lane;
    DSU_GLOBAL double *P = gmem(g.panel) + r0 + lane;
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = lane < w ? m[(size_t)(wave + 4 * q) * np] : 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) t[wave + 4 * q][lane] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q)
        if (wave + 4 * q < w) P[(size_t)(wave + 4 * q) * np] = t[lane][wave + 4 * q];
}

// Of the lanes in `mask` (not empty) the one that holds the smallest idx.
__device__ __forceinline__ int lowest_lane(unsigned long long mask, int idx) {
    int l = __builtin_ctzll(mask);
    for (unsigned long long m = mask & (mask - 1); m; m &= m - 1) {  // (ties only)
        const int o = __builtin_ctzll(m);
        if (__builtin_amdgcn_readlane(idx, o) < __builtin_amdgcn_readlane(idx, l)) l = o;
    }
    return l;
}

// One group of WS panel columns, factored in registers: thread t owns rows
// t + NT r (r < RPT).  What bounds it: the pivots are a serial chain on one
// compute unit, N x WS multiply-adds each.  So:
//  * WS RPT = 64 values a thread on as few waves as hold the rows (NT = 256
//    or 512): barriers span 4 or 8 waves, and what a wave does once a pivot
//    serves RPT rows of each lane;
//  * rows are interchanged in name only: a thread keeps its rows and the
//    position each one has, which the interchanges and the ties of the pivot
//    search go by; the positions are used when the columns are stored.  Only
//    the pivot row's owner does anything of its own in a step (it scales its
//    row in place);
//  * the scaled pivot row sits one column a lane (one LDS read and one
//    multiply) and enters the multiply-adds from scalar registers (readlane);
//    every wave reading it from LDS as broadcasts cost 16 reads of 16 bytes a
//    wave and bound the step;
//  * four pivots per loop body, then the columns rotate by four through the
//    registers: every register index is fixed, and the body of a few KB stays
//    in the instruction cache (a step unrolled per column fetches each line
//    once, from memory);
//  * logarithms of the pivots after the loop, one per lane.
// Every element gets the operations of one plain elimination step in the same
// order, whatever NT and RPT.  Per launch (N = 1024, 32 columns, 64
// determinants): 152 -> 61 us; N = 2048, 16 columns: 81 -> 36; N = 4096, 8
// columns: 48 -> 30 us (32 determinants); N = 512: 267 -> 79 us (512).
// Afterwards the workgroup moves the group's row interchanges through the
// panel's other columns (a permutation of at most 2 ws rows, one round of
// loads and stores) and leaves the pivot rows of those columns in g.w for
// k_gj_apply: Q[j][c] at w[64 j + c].
template <int NT, int WS, int RPT>
__global__ __launch_bounds__(NT) void k_gj_group(const GjDesc *__restrict__ descs, int n, int np, int k0, int j0,
                                                 int ws, int w) {
    constexpr int NW = NT / 64;
    __shared__ double s_prow[WS + 1];
    __shared__ double s_cv[NW], s_d[WS];
    __shared__ int s_ci[NW], s_p[WS], s_src[2 * WS];
    const GjDesc g = descs[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb = k0 + j0;
    DSU_GLOBAL double *P = gmem(g.panel) + (size_t)j0 * np;
    double sv[RPT][WS];
    int pos[RPT];  // the position of each row after the interchanges so far
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int i = tid + NT * r;
        pos[r] = i;
        DSU_GLOBAL const double *pi = P + (i < np ? i : 0);
        if (ws == WS) {
#pragma unroll
            for (int j = 0; j < WS; ++j) sv[r][j] = pi[(size_t)j * np];
        } else {
#pragma unroll
            for (int j = 0; j < WS; ++j) sv[r][j] = j < ws ? pi[(size_t)j * np] : 0.0;
        }
    }
    double pmax = 0.0;
    int status = 0;
    if (kb != 0) {
        pmax = *g.pmax;
        status = *g.status;
    }
    const double tiny = (double)n * 2.220446049250313e-16;
    auto step = [&](auto q_c, int kk) __attribute__((always_inline)) {
        constexpr int q = decltype(q_c)::value;
        if (kk >= ws) return;  // uniform
        const int k = kb + kk;
        // the wave's candidate: largest |entry| of column kk at positions k .. n - 1, lowest position on ties
        double best = -1.0;
        int bp = n;
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const double a = fabs(sv[r][q]);
            if (pos[r] >= k && pos[r] < n && (a > best || (a == best && pos[r] < bp))) {
                best = a;
                bp = pos[r];
            }
        }
        const double wm = wave_max(best);
        // (a wave without a candidate: any lane, position n)
        const int wl = wm >= 0.0 ? lowest_lane(__ballot(best == wm), bp) : 0;
        if (lane == wl) {
            s_cv[wave] = wm;
            s_ci[wave] = bp;
        }
        __syncthreads();
        // every wave combines the candidates (same values, same result)
        const double cv = s_cv[lane & (NW - 1)];
        const int ci = s_ci[lane & (NW - 1)];
        const double bv = lane_f64(group_max<NW>(cv), 0);
        int p = __builtin_amdgcn_readlane(ci, lowest_lane(__ballot(cv == bv) & ((1ull << NW) - 1), ci));
        pmax = fmax(pmax, bv);
        // singular when the best pivot is at rounding level of the largest
        // one: flagged, and no interchange
        if (!(bv > tiny * pmax)) {
            status = -3;
            p = k;
        }
        // the owner publishes the pivot row
        bool own[RPT];
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            own[r] = pos[r] == p;
            if (own[r])
#pragma unroll
                for (int j = 0; j < WS; ++j) s_prow[j] = sv[r][j];
            pos[r] = pos[r] == p ? k : (pos[r] == k ? p : pos[r]);
        }
        __syncthreads();
        // column j of the row in lane j of each row of 16 lanes
        constexpr int NR = (WS + 15) / 16;
        double rp[NR];
#pragma unroll
        for (int h = 0; h < NR; ++h) rp[h] = s_prow[(16 * h + (lane & 15)) & (WS - 1)];
        const double d = row_bcast_f64<q>(rp[0]);
        const double dinv = d != 0.0 ? 1.0 / d : 0.0;
#pragma unroll
        for (int h = 0; h < NR; ++h) rp[h] *= dinv;
        if (tid == 0) {
            s_p[kk] = p;
            s_d[kk] = d;
        }
        double f[RPT];
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            f[r] = own[r] ? 0.0 : -sv[r][q];
            if (own[r])
#pragma unroll
                for (int j = 0; j < WS; ++j) sv[r][j] *= dinv;
        }
        static_for(std::make_integer_sequence<int, WS>{}, [&](auto j_c) __attribute__((always_inline)) {
            constexpr int j = decltype(j_c)::value;
            if constexpr (j != q) {
                const double pj = row_bcast_f64<j % 16>(rp[j / 16]);
#pragma unroll
                for (int r = 0; r < RPT; ++r) sv[r][j] = __builtin_fma(f[r], pj, sv[r][j]);
            }
        });
#pragma unroll
        for (int r = 0; r < RPT; ++r) sv[r][q] = own[r] ? dinv : f[r] * dinv;
    };
    int turned = 0;  // columns rotated so far
#pragma unroll 1
    for (; turned < ws; turned += 4) {
        step(std::integral_constant<int, 0>{}, turned);
        step(std::integral_constant<int, 1>{}, turned + 1);
        step(std::integral_constant<int, 2>{}, turned + 2);
        step(std::integral_constant<int, 3>{}, turned + 3);
        if constexpr (WS > 4)
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                const double t0 = sv[r][0], t1 = sv[r][1], t2 = sv[r][2], t3 = sv[r][3];
#pragma unroll
                for (int j = 0; j < WS - 4; ++j) sv[r][j] = sv[r][j + 4];
                sv[r][WS - 4] = t0;
                sv[r][WS - 3] = t1;
                sv[r][WS - 2] = t2;
                sv[r][WS - 1] = t3;
            }
    }
    // column j now sits at place j + WS - turned; rows go to their positions
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        if (tid + NT * r >= np) continue;
        DSU_GLOBAL double *po = P + pos[r];
        if (ws == WS) {
#pragma unroll
            for (int j = 0; j < WS; ++j) po[(size_t)j * np] = sv[r][j];
        } else {
#pragma unroll
            for (int q = 0; q < WS; ++q) {
                const int j = q - (WS - turned);
                if (j >= 0 && j < ws) po[(size_t)j * np] = sv[r][q];
            }
        }
    }
    __syncthreads();  // s_p, s_d
    if (tid < ws) {
        const double d = s_d[tid];
        s_d[tid] = d != 0.0 ? log(fabs(d)) : 0.0;
        int flips = (s_p[tid] != kb + tid ? 1 : 0) ^ (d < 0.0 ? 1 : 0);
        const int odd = __popcll(__ballot(flips != 0)) & 1;
        g.piv[kb + tid] = s_p[tid];
        if (tid == 0) {
            double ld = kb != 0 ? *g.logdet : 0.0;
            for (int q = 0; q < ws; ++q) ld += s_d[q];
            const int sign = kb != 0 ? *g.sign : 1;
            *g.logdet = ld;
            *g.sign = odd ? -sign : sign;
            *g.status = status;
            *g.pmax = pmax;
        }
    }
    if (w <= ws) return;
    // the interchanges k <-> p, in order, put old row s_0(s_1(...(r))) at row r
    if (tid < 2 * ws) {
        int x = tid < ws ? kb + tid : s_p[tid - ws];
        for (int q = ws - 1; q >= 0; --q) x = x == kb + q ? s_p[q] : (x == s_p[q] ? kb + q : x);
        s_src[tid] = x;
    }
    __syncthreads();
    constexpr int NM = (2 * WS * (64 - WS) + NT - 1) / NT;  // moved values a thread, at most
    const int oc = w - ws, cnt = 2 * ws * oc;
    DSU_GLOBAL double *A = gmem(g.panel), *Q = gmem(g.w);
    double mv[NM];
#pragma unroll
    for (int q = 0; q < NM; ++q) {
        const int v = tid + NT * q, c = v / (2 * ws), t = v % (2 * ws);
        if (v < cnt) mv[q] = A[(size_t)(c < j0 ? c : c + ws) * np + s_src[t]];
    }
    __syncthreads();  // every value read before any row changes
#pragma unroll
    for (int q = 0; q < NM; ++q) {
        const int v = tid + NT * q, c = v / (2 * ws), t = v % (2 * ws);
        if (v < cnt) {
            const int cc = c < j0 ? c : c + ws;
            A[(size_t)cc * np + (t < ws ? kb + t : s_p[t - ws])] = mv[q];  // rows named twice receive the same value
            if (t < ws) Q[64 * t + cc] = mv[q];
        }
    }
}

// The group's update of the panel's other columns, P_c += (S - E) Q_c, as
// matrix-core tiles: a wave takes 16 rows and, transposed (D' = Q^T (S - E)^T,
// so that a lane's result lies along the column-major panel), the columns in
// tiles of 16.  One workgroup per 64 rows: the few MB it moves and 2 N ws w
// flops are a few microseconds on any number of determinants, so it is bound by
// its launch or by the panel's bytes (N = 1024, 32 columns, 64 determinants: 44
// -> 13 us; N = 512, 512 determinants: 143 -> 39; N = 4096, 8 columns, 32: 37
// -> 22; one determinant of N = 1024: 9 -> 6; the first figures with one or four
// columns per workgroup on the vector units).  A matrix-core step adds its four
// products in ascending order, so each element gets the chain of multiply-adds
// of the vector form.
__global__ __launch_bounds__(kThreads) void k_gj_apply(const GjDesc *__restrict__ descs, int np, int k0, int j0, int ws,
                                                       int w) {
    const GjDesc g = descs[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
    const int row = blockIdx.x * 64 + 16 * wave + lr;
    DSU_GLOBAL double *P = gmem(g.panel);
    DSU_GLOBAL const double *S = P + (size_t)j0 * np, *Q = gmem<const double>(g.w);
    double b[8];  // (S - E)[row][lk + 4 s]
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int j = lk + 4 * s;
        b[s] = j < ws ? S[(size_t)j * np + row] - (row == k0 + j0 + j ? 1.0 : 0.0) : 0.0;
    }
    for (int c0 = 0; c0 < w; c0 += 16) {
        if (c0 >= j0 && c0 + 16 <= j0 + ws) continue;
        f64x4 acc;
        double a[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = c0 + lk + 4 * i;
            acc[i] = c < w ? P[(size_t)c * np + row] : 0.0;
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) a[s] = lk + 4 * s < ws && c0 + lr < w ? Q[64 * (lk + 4 * s) + c0 + lr] : 0.0;
#pragma unroll
        for (int s = 0; s < 8; ++s)
            if (4 * s < ws) acc = Mma<double>::mma(a[s], b[s], acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = c0 + lk + 4 * i;
            if (c < w && !(c >= j0 && c < j0 + ws)) P[(size_t)c * np + row] = acc[i];
        }
    }
}

// ---------------------------------------------------------------------------
// Panel pairs: the pieces of the fused two-panel step around k_gj_update's
// PAIR form (same notation: R1, R2, P1, P2, T1, T2, Q1, Q2, M1).
// ---------------------------------------------------------------------------

// In the three pair kernels a wave takes 16 of a block's 64 rows (columns in
// k_gj_pair_q2) and forms the 64-term products on matrix cores, one operand in
// registers from global memory, the other in LDS.  On the vector units, 16
// results a thread with one operand broadcast from LDS, the LDS reads bound
// them.  A matrix-core step adds its four products in ascending order, so each
// element keeps its chain of multiply-adds.  Per launch (N = 1024, 64
// determinants), before and after: slab 35 -> 28 us, q2 51 -> 41, fix 56 -> 37.

// After the first panel: R2's columns of M1 = P1 M + (T1 - E1) Q1 become the
// second panel, and T1 moves to panel_b.  One block per 64 rows; a wave rewrites
// the rows it read.  Transposed (D' = Q1^T (T1 - E1)^T) so that results lie along
// the column-major panel; operand row m of a tile is column pair_col(m), so that
// a lane's four results are neighbours in their row of P1 M.
__device__ __forceinline__ int pair_col(int m) { return 4 * (m & 3) + (m >> 2); }
constexpr int kPairLd = 80;  // doubles a row of an LDS operand [l][64]: lanes of l and l + 1 in different banks
__global__ __launch_bounds__(kThreads, 3) void k_gj_pair_slab(const GjDesc *__restrict__ descs, int np, int k0) {
    __shared__ double s_q[64 * kPairLd];  // Q1[l][R2 column j]
    const GjDesc g = descs[blockIdx.y];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lk = lane >> 4;
    const int row = blockIdx.x * 64 + 16 * wave + lr;
    DSU_GLOBAL const double *m = gmem<const double>(g.m);
    DSU_GLOBAL double *pb = gmem(g.panel_b), *pa = gmem(g.panel);
    double tv[16], qv[16];
    int qr[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) qr[q] = g.rowsrc[k0 + wave + 4 * q];
    DSU_GLOBAL const double *mr = m + (size_t)g.rowsrc[row] * np + k0 + 64 + 4 * lk;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        tv[q] = pa[(size_t)(4 * q + lk) * np + row];
        qv[q] = m[(size_t)qr[q] * np + k0 + 64 + lane];
    }
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[t][i] = mr[16 * t + i];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        pb[(size_t)(4 * q + lk) * np + row] = tv[q];
        s_q[(wave + 4 * q) * kPairLd + lane] = qv[q];
        tv[q] -= row == k0 + 4 * q + lk ? 1.0 : 0.0;
    }
    __syncthreads();
    const double *qp = s_q + lk * kPairLd + pair_col(lr);
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = Mma<double>::mma(qp[4 * q * kPairLd + 16 * t], tv[q], acc[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) pa[(size_t)(16 * t + 4 * lk + i) * np + row] = acc[t][i];
}

// After the second panel: rowsrc_b = P2 (its own swaps), rowsrc = P2 P1 (row
// i of the result <- row rowsrc[i] of M), qrow[l] = P1's source of row k0 + l.
// One workgroup per determinant; P1's map in dynamic LDS (4 np bytes) while
// rowsrc is overwritten.
__global__ __launch_bounds__(kThreads) void k_gj_pair_rowsrc(const GjDesc *__restrict__ descs, int np, int k0) {
    extern __shared__ int s_r1[];
    __shared__ int s_piv[64];
    const GjDesc g = descs[blockIdx.x];
    const int tid = threadIdx.x, kb = k0 + 64;
    if (tid < 64) s_piv[tid] = g.piv[kb + tid];
    for (int i = tid; i < np; i += kThreads) {
        s_r1[i] = g.rowsrc[i];
        g.rowsrc_b[i] = i;
    }
    __syncthreads();
    const bool on = tid < 128;
    const int r = on ? (tid < 64 ? kb + tid : s_piv[tid - 64]) : 0, x = on ? gj_trace(r, s_piv, kb, 64) : 0;
    if (on) {
        g.rowsrc_b[r] = x;
        g.rowsrc[r] = s_r1[x];
    }
    if (tid < 64) g.qrow[tid] = s_r1[k0 + tid];
    gj_total_map(g.perm, r, x, on);
}

// Q2[j] = M1[P2 row k0 + 64 + j] = M[rowsrc[k0 + 64 + j]] + (T1 - E1)[r_j] Q1,
// r_j = rowsrc_b[k0 + 64 + j], for all columns (R1's and R2's are not used).
// One block per 64 columns.
__global__ __launch_bounds__(kThreads) void k_gj_pair_q2(const GjDesc *__restrict__ descs, int np, int k0) {
    __shared__ double s_q[64 * kPairLd];  // Q1[l][c0 + c]
    const GjDesc g = descs[blockIdx.y];
    const int c0 = blockIdx.x * 64, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lk = lane >> 4;
    DSU_GLOBAL const double *m = gmem<const double>(g.m), *pb = gmem<const double>(g.panel_b);
    double wv[16], qv[16];
    int qr[16], sr[4];
    const int r = g.rowsrc_b[k0 + 64 + 16 * wave + lr];  // r_j of this lane's operand row
#pragma unroll
    for (int q = 0; q < 16; ++q) qr[q] = g.qrow[wave + 4 * q];
#pragma unroll
    for (int i = 0; i < 4; ++i) sr[i] = g.rowsrc[k0 + 64 + 16 * wave + lk + 4 * i];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        qv[q] = m[(size_t)qr[q] * np + c0 + lane];
        wv[q] = pb[(size_t)(4 * q + lk) * np + r];
    }
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[t][i] = m[(size_t)sr[i] * np + c0 + 16 * t + lr];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        s_q[(wave + 4 * q) * kPairLd + lane] = qv[q];
        wv[q] -= r == k0 + 4 * q + lk ? 1.0 : 0.0;
    }
    __syncthreads();
    const double *qp = s_q + lk * kPairLd + lr;
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = Mma<double>::mma(wv[q], qp[4 * q * kPairLd + 16 * t], acc[t]);
    DSU_GLOBAL double *q2 = gmem(g.q2) + (size_t)(16 * wave + lk) * np + c0 + lr;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) q2[(size_t)(4 * i) * np + 16 * t] = acc[t][i];
}

// R1's columns of the pair's result: m2[i][k0 + j] = (P2 T1)[i][j] +
// (T2 - E2)[i] (P2 T1)[R2][j] (T1 is M1's R1 block, Q2's R1 columns are its
// rows at P2's pivots).  Runs after the update, which leaves those columns
// to it.  One block per 64 rows; the LDS array first holds the block's rows of
// P2 T1, then R2's, both at [j][row] (rows of 66: column reads spread over the
// banks).
__global__ __launch_bounds__(kThreads) void k_gj_pair_fix(const GjDesc *__restrict__ descs, int np, int k0) {
    constexpr int LD = 66;
    __shared__ double s_x[64 * LD];
    const GjDesc g = descs[blockIdx.y];
    const int r0 = blockIdx.x * 64, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lk = lane >> 4;
    DSU_GLOBAL const double *pa = gmem<const double>(g.panel), *pb = gmem<const double>(g.panel_b);
    const int row = r0 + 16 * wave + lr, rb = g.rowsrc_b[r0 + lane], rz = g.rowsrc_b[k0 + 64 + lane];
    double av[16], x1[16], x2[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int a = wave + 4 * q;
        x1[q] = pb[(size_t)a * np + rb];
        av[q] = pa[(size_t)(4 * q + lk) * np + row];
        x2[q] = pb[(size_t)a * np + rz];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) s_x[(wave + 4 * q) * LD + lane] = x1[q];
    __syncthreads();
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[t][i] = s_x[(16 * t + lr) * LD + 16 * wave + lk + 4 * i];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        s_x[(wave + 4 * q) * LD + lane] = x2[q];
        av[q] -= row == k0 + 64 + 4 * q + lk ? 1.0 : 0.0;
    }
    __syncthreads();
    const double *zp = s_x + lr * LD + lk;
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = Mma<double>::mma(av[q], zp[16 * t * LD + 4 * q], acc[t]);
    DSU_GLOBAL double *dst = gmem(g.m2) + (size_t)(r0 + 16 * wave + lk) * np + k0 + lr;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) dst[(size_t)(4 * i) * np + 16 * t] = acc[t][i];
}

// Column parts of an update launch: doubled while the launch has fewer than 512
// workgroups (two a compute unit) and a part keeps 128 columns or more.  One part
// left most units idle for few determinants.  An inverse, one part and so: N =
// 1024, one determinant 3.08 -> 2.53 ms, 4 of them 3.17 -> 2.70; N = 2048, one 8.65
// -> 6.49, 4 9.07 -> 7.77; N = 4096, 2 29.6 -> 23.7; from 512 workgroups on nothing
// changes (N = 1024, 64: 6.4 ms).
static int gj_update_parts(int ndesc, int np) {
    int parts = 1;
    while (ndesc * (np / 64) * parts < 512 && np / (2 * parts) >= 128) parts *= 2;
    return parts;
}

template <int RT, int CW>
static void launch_gj_update(const GjDesc *descs_dev, int ndesc, int np, int nb, int k0, int w, hipStream_t s) {
    const int nblk = np / (64 * RT), parts = gj_update_parts(ndesc, np);
    const dim3 grid(ndesc * nblk * parts);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, descs_dev, np, nblk, parts, k0, w);
    };
    if (nb == 16) launch(k_gj_update<16, RT, CW>);
    else if (nb == 32) launch(k_gj_update<32, RT, CW>);
    else launch(k_gj_update<64, RT, CW>);
}

// Factor the panel [k0, k0 + w); gather = false: the panel buffer already
// holds the panel's columns (a pair's second panel).
template <int NT, int WS, int RPT>
static void launch_gj_panel(const GjDesc *descs_dev, int ndesc, int n, int np, int k0, int w, hipStream_t s,
                            bool gather) {
    if (gather) hipLaunchKernelGGL(k_gj_gather, dim3(np / 64, ndesc), dim3(kThreads), 0, s, descs_dev, np, k0, w);
    for (int j0 = 0; j0 < w; j0 += WS) {
        const int ws = j0 + WS <= w ? WS : w - j0;
        hipLaunchKernelGGL((k_gj_group<NT, WS, RPT>), dim3(ndesc), dim3(NT), 0, s, descs_dev, n, np, k0, j0, ws, w);
        if (w > ws)
            hipLaunchKernelGGL(k_gj_apply, dim3(np / 64, ndesc), dim3(kThreads), 0, s, descs_dev, np, k0, j0, ws, w);
    }
}

// Final column permutation: the swaps k <-> piv[k] undone on the columns, last
// one first, put column perm[j] at place j, perm = the inverse of the map of
// all row interchanges that the panels composed in g.perm.  (Following the n
// swaps on one thread took 78 us at n = 1024.)  g.rowsrc is scratch here.
__global__ __launch_bounds__(1024) void k_gj_perm(const GjDesc *__restrict__ descs, int np) {
    const GjDesc g = descs[blockIdx.x];
    for (int r = threadIdx.x; r < np; r += 1024) g.rowsrc[r] = g.perm[r];
    __syncthreads();
    for (int r = threadIdx.x; r < np; r += 1024) g.perm[g.rowsrc[r]] = r;
}

GjTiles gj_tiles_default(int n, int np) {
    // measured on MI355X: 64-column panels from N = 512 (512: 7.0 ms against
    // 9.2 with 32 columns for 512 inverses), in pairs from 1024 (4096: 119 ms
    // against 139 for 32 inverses, 2048: 32.9 against 37.0 ms for 64, 1024:
    // 18.6 against 20.4 ms for 256; at 512 7.1 against 7.0); 64-column update
    // chunks where np pairs them up (4096, single panels: 139 against 146 ms; 512:
    // 7.4 against 7.0)
    GjTiles t;
    t.nb = n >= 1024 && np <= 4096 ? 128 : (n >= 512 ? 64 : (n >= 64 ? 32 : 16));
    t.cw = np % 128 == 0 ? 64 : 32;
    t.cpb = np >= 2048 ? 4 : 1;  // reported back, without effect
    return t;
}

hipError_t launch_gj_invert(const GjDesc *set_a, const GjDesc *set_b, int ndesc, int n, int np, const GjTiles &tiles,
                            hipStream_t s, const GjDesc **final_set) {
    const int nb = tiles.nb, cw = tiles.cw;  // (tiles.cpb has no effect)
    if (nb != 16 && nb != 32 && nb != 64 && nb != 128) return hipErrorInvalidValue;
    if (np % 64) return hipErrorInvalidValue;  // the trailing update takes column chunks in pairs
    if (!(cw == 32 || (cw == 64 && np % 128 == 0))) return hipErrorInvalidValue;
    const int pw = nb == 128 ? 64 : nb;  // columns factored at a time
    // factor the panel [k0, k0 + w): groups of 32 .. 4 columns in registers up to np = 8192 (64 values a thread),
    // beyond that one column at a time
    auto factor = [&](const GjDesc *d, int k0, int w, bool gather) {
        if (np <= 256) launch_gj_panel<256, 32, 1>(d, ndesc, n, np, k0, w, s, gather);
        else if (np <= 512) launch_gj_panel<256, 32, 2>(d, ndesc, n, np, k0, w, s, gather);
        else if (np <= 1024) launch_gj_panel<512, 32, 2>(d, ndesc, n, np, k0, w, s, gather);
        else if (np <= 2048) launch_gj_panel<512, 16, 4>(d, ndesc, n, np, k0, w, s, gather);
        else if (np <= 4096) launch_gj_panel<512, 8, 8>(d, ndesc, n, np, k0, w, s, gather);
        else if (np <= 8192) launch_gj_panel<512, 4, 16>(d, ndesc, n, np, k0, w, s, gather);
        else hipLaunchKernelGGL(k_gj_panel, dim3(ndesc), dim3(kThreads), 0, s, d, n, np, pw, k0, k0 + w);
    };
    const GjDesc *cur = set_a, *nxt = set_b;
    for (int k0 = 0; k0 < n;) {
        const int k1 = k0 + pw < n ? k0 + pw : n;
        // two whole 64-column panels share one trailing update (both row maps
        // in LDS: np <= 4096); otherwise one panel at a time
        const bool pair = nb == 128 && k0 + 128 <= n && np <= 4096;
        factor(cur, k0, k1 - k0, true);
        // row interchanges, then the trailing update into the other buffer
        hipLaunchKernelGGL(k_gj_rowsrc, dim3(ndesc), dim3(kThreads), 0, s, cur, np, k0, k1);
        if (pair) {
            hipLaunchKernelGGL(k_gj_pair_slab, dim3(np / 64, ndesc), dim3(kThreads), 0, s, cur, np, k0);
            factor(cur, k0 + 64, 64, false);
            hipLaunchKernelGGL(k_gj_pair_rowsrc, dim3(ndesc), dim3(kThreads), (size_t)np * sizeof(int), s, cur, np, k0);
            hipLaunchKernelGGL(k_gj_pair_q2, dim3(np / 64, ndesc), dim3(kThreads), 0, s, cur, np, k0);
            const int parts = gj_update_parts(ndesc, np);
            hipLaunchKernelGGL((k_gj_update<128, 1, 16, true>), dim3(ndesc * (np / 64) * parts), dim3(kThreads), 0, s,
                               cur, np, np / 64, parts, k0, 64);
            hipLaunchKernelGGL(k_gj_pair_fix, dim3(np / 64, ndesc), dim3(kThreads), 0, s, cur, np, k0);
            k0 += 128;
        } else {
            // (128-row workgroups, RT = 2, measured no faster than 64-row ones)
            if (cw == 64)
                launch_gj_update<1, 64>(cur, ndesc, np, pw, k0, k1 - k0, s);
            else
                launch_gj_update<1, 32>(cur, ndesc, np, pw, k0, k1 - k0, s);
            k0 = k1;
        }
        const GjDesc *t = cur;
        cur = nxt;
        nxt = t;
    }
    hipLaunchKernelGGL(k_gj_perm, dim3(ndesc), dim3(1024), 0, s, cur, np);
    if (final_set) *final_set = cur;
    return hipGetLastError();
}

// BT[i][j] = T(M[i][perm[j]]) inside n x n, zero padding.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_cast_perm(const GjDesc *__restrict__ gj, T *const *__restrict__ bt, int n,
                                                        int np) {
    const int d = blockIdx.z;
    const GjDesc g = gj[d];
    T *out = bt[d];
    const int j = blockIdx.x * kThreads + threadIdx.x;
    const int i = blockIdx.y;
    if (j >= np) return;
    out[(size_t)i * np + j] = (i < n && j < n) ? T(g.m[(size_t)i * np + g.perm[j]]) : T(0);
}

// The same with the row staged in LDS first (one row per workgroup, dynamic
// LDS of np doubles): the permuted gather then reads LDS instead of scattered
// global lines; the row comes in with 16-byte loads and leaves four columns a
// thread (np is a multiple of 64).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_cast_perm_row(const GjDesc *__restrict__ gj, T *const *__restrict__ bt,
                                                            int n, int np) {
    extern __shared__ double s_row[];
    typedef double d2 __attribute__((ext_vector_type(2)));
    const GjDesc g = gj[blockIdx.y];
    T *out = bt[blockIdx.y] + (size_t)blockIdx.x * np;
    const int i = blockIdx.x;
    const d2 *src = reinterpret_cast<const d2 *>(g.m + (size_t)i * np);
    for (int j = threadIdx.x; j < np / 2; j += kThreads) reinterpret_cast<d2 *>(s_row)[j] = src[j];
    __syncthreads();
    for (int j4 = threadIdx.x; j4 < np / 4; j4 += kThreads) {
        const int j = 4 * j4;
        const int4 pv = reinterpret_cast<const int4 *>(g.perm)[j4];
        const int pj[4] = {pv.x, pv.y, pv.z, pv.w};
        T v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (i < n && j + e < n) ? T(s_row[pj[e]]) : T(0);
        if constexpr (sizeof(T) == 4) {
            *reinterpret_cast<float4 *>(out + j) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
            reinterpret_cast<d2 *>(out + j)[0] = d2{(double)v[0], (double)v[1]};
            reinterpret_cast<d2 *>(out + j)[1] = d2{(double)v[2], (double)v[3]};
        }
    }
}

template <typename T>
hipError_t launch_cast_perm(const GjDesc *gj_dev, T *const *bt_dev, int ndesc, int n, int np, hipStream_t s) {
    if (np <= 8192)
        hipLaunchKernelGGL((k_cast_perm_row<T>), dim3(np, ndesc), dim3(kThreads), (size_t)np * sizeof(double), s,
                           gj_dev, bt_dev, n, np);
    else
        hipLaunchKernelGGL((k_cast_perm<T>), dim3((np + kThreads - 1) / kThreads, np, ndesc), dim3(kThreads), 0, s,
                           gj_dev, bt_dev, n, np);
    return hipGetLastError();
}
template hipError_t launch_cast_perm<float>(const GjDesc *, float *const *, int, int, int, hipStream_t);
template hipError_t launch_cast_perm<double>(const GjDesc *, double *const *, int, int, int, hipStream_t);

// M = A^T padded with the identity (32 x 32 tiles through LDS).
__global__ __launch_bounds__(kThreads) void k_load_transpose(const double *const *__restrict__ a_all,
                                                             double *const *__restrict__ m_all, int n, int np, int lda) {
    __shared__ double tile[32][33];
    const double *a = a_all[blockIdx.z];
    double *m = m_all[blockIdx.z];
    const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
    for (int r = ty; r < 32; r += 8) {
        const int i = by + r, j = bx + tx;  // read A[i][j]
        tile[r][tx] = (i < n && j < n) ? a[(size_t)i * lda + j] : (i == j ? 1.0 : 0.0);
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int j = bx + r, i = by + tx;  // write M[j][i] = A[i][j]
        if (j < np && i < np) m[(size_t)j * np + i] = tile[tx][r];
    }
}

hipError_t launch_load_transpose(const double *const *a_dev, double *const *m_dev, int ndesc, int n, int np, int lda,
                                 hipStream_t s) {
    hipLaunchKernelGGL(k_load_transpose, dim3(np / 32, np / 32, ndesc), dim3(kThreads), 0, s, a_dev, m_dev, n, np, lda);
    return hipGetLastError();
}

// a[i][j] = in[i][j], rows of n to rows of np.
__global__ __launch_bounds__(kThreads) void k_pad_rows(const double *__restrict__ in, double *__restrict__ a, int n,
                                                       int np) {
    const int j = blockIdx.x * kThreads + threadIdx.x, i = blockIdx.y;
    if (j < n) a[(size_t)i * np + j] = in[(size_t)i * n + j];
}

hipError_t launch_pad_rows(const double *in, double *a, int n, int np, hipStream_t s) {
    hipLaunchKernelGGL(k_pad_rows, dim3((n + kThreads - 1) / kThreads, n), dim3(kThreads), 0, s, in, a, n, np);
    return hipGetLastError();
}

// out[i][j] = BT[j][i], n x n FP64.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_untranspose(const T *__restrict__ bt, double *__restrict__ out, int n,
                                                          int np) {
    __shared__ double tile[32][33];
    const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int r = ty; r < 32; r += 8) {
        const int i = by + r, j = bx + tx;
        tile[r][tx] = (i < n && j < n) ? double(bt[(size_t)i * np + j]) : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int j = bx + r, i = by + tx;
        if (j < n && i < n) out[(size_t)j * n + i] = tile[tx][r];
    }
}

template <typename T>
hipError_t launch_untranspose(const T *bt, double *out, int n, int np, hipStream_t s) {
    hipLaunchKernelGGL((k_untranspose<T>), dim3(np / 32, np / 32), dim3(kThreads), 0, s, bt, out, n, np);
    return hipGetLastError();
}
template hipError_t launch_untranspose<float>(const float *, double *, int, int, hipStream_t);
template hipError_t launch_untranspose<double>(const double *, double *, int, int, hipStream_t);

}  // namespace dsu
