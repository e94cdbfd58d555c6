// A Cholesky-QR pass after its Gram matrix: the factor R of S = R^T R (M x M,
// FP64) and X <- X R^{-1} for the tall row-major block.
//
// Panels of 128 columns, left to right: X_j <- (X_j - sum_{k<j} X_k R_kj) R_jj^{-1},
// with the diagonal blocks inverted beforehand in FP64.  A wave owns 32 or 16 rows and
// walks all panels, so the solve is one launch without a barrier; its operands
// come straight from memory, 16 bytes along k per lane and load (a lane's values
// go to successive products, which permutes k alike on both sides).  R and the
// inverses are laid out beforehand as operands, 1 KB per 16 columns and
// group of k: from their column-major form a load takes half of 16 cache lines,
// more than the L1 holds until the other halves are wanted.
//
// Measured against the library's triangular solve (ms): 440,000 x 1024 FP32
// 5.8 -> 4.7, 440,000 x 600 FP64 6.1 -> 3.5, 120,000 x 128 FP64 0.17 -> 0.068.
// Bound by the matrix cores: 64 FP32 (32 FP64) products, 2048 cycles, per 10
// loads of 1 KB.  128 columns because the rows' earlier panels, too many to stay in
// an L2, are read again for each panel: (M / 128 - 1) / 2 times in all.
#include <algorithm>

#include "internal.hpp"
#include "kernels.hpp"

namespace chf {

namespace {

constexpr int kTriBlock = 128;
constexpr int kTriPitch = kTriBlock + 2;

template <class T>
using Acc = T __attribute__((ext_vector_type(4)));

__device__ inline Acc<float> mfma(float a, float b, Acc<float> c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ inline Acc<double> mfma(double a, double b, Acc<double> c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// row of the 16 x 16 result held by (register, lane); the column is lane % 16
template <class T>
__device__ inline int result_row(int reg, int lane) {
    return sizeof(T) == 4 ? 4 * (lane >> 4) + reg : 4 * reg + (lane >> 4);
}

template <class T>
struct alignas(16) Piece16 {
    static constexpr int N = 16 / int(sizeof(T));
    T e[N];
};
// 16 bytes from an element-aligned address
template <class T>
__device__ inline Piece16<T> load16(const T* p) {
    Piece16<T> v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

// values of one operand (64 lanes), and the operand order of an upper triangle
// of 16-column tiles and `groups` groups of k per tile: element e of lane l of
// tile t and group g is R[k][j], j = 16 t + l % 16, and k = g KG + N (l / 16) + e
// where the other operand comes from memory, whose pieces lie along k.  The
// inverses take k = g KG + 4 e + l / 16 instead, so that the products add k in
// ascending order and the largest term, the diagonal's, last: out of order the
// sums after it round at its size (FP64, 128 columns, in units of 2^-53 beside the
// columns' common factors: 1.11 against 1.05, the library 1.05; the whole error of 97
// FP32 columns with an FP64 Gram, in units of 2^-24: 0.97 against 0.74, library 0.92).
template <class T>
struct Packed {
    static constexpr int N = Piece16<T>::N, KG = 4 * N, V = 64 * N;
    __device__ static void where(int64_t idx, int groups, bool ascending, int* k, int* j) {
        const int e = int(idx % N), l = int(idx / N % 64);
        const int64_t op = idx / V;
        *k = int(op % groups) * KG + (ascending ? 4 * e + (l >> 4) : N * (l >> 4) + e);
        *j = int(op / groups) * 16 + (l & 15);
    }
};

}  // namespace

// P = -R in operand order
template <class T>
__global__ void __launch_bounds__(256) pack_upper_kernel(int m, int groups, int64_t n, const double* __restrict__ R,
                                                         T* __restrict__ P) {
    const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (idx >= n) return;
    int k, j;
    Packed<T>::where(idx, groups, false, &k, &j);
    P[idx] = k <= j && j < m ? -T(R[int64_t(j) * m + k]) : T(0);
}

// the value of one lane (a constant) on all lanes
__device__ inline double from_lane(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The upper triangular kTriBlock square in M (rows of kTriPitch) by its inverse,
// by 512 threads: 16 x 16 blocks by back substitution, one column per thread,
// then doubled with Z12 = -Z11 (R12 Z22) in place, up to the w columns that are not
// those of the identity.
__device__ inline void invert_upper(double* M, int w) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    double z[16];
    double* const D = M + (t >> 4) * 16 * (kTriPitch + 1);
    if (t < kTriBlock) {
#pragma unroll
        for (int i = 15; i >= 0; --i) {
            double v = i == (t & 15) ? 1.0 : 0.0;
#pragma unroll
            for (int k = i + 1; k < 16; ++k) v = fma(-D[i * kTriPitch + k], z[k], v);
            z[i] = v / D[i * kTriPitch + i];
        }
    }
    __syncthreads();
    if (t < kTriBlock)
#pragma unroll
        for (int i = 0; i < 16; ++i) D[i * kTriPitch + (t & 15)] = z[i];
    for (int s = 16; s < w; s *= 2) {
        const int q = s / 16, tiles = kTriBlock / (2 * s) * q * q;
        // side 0: W = R12 Z22 over R12;  side 1: Z12 = -Z11 W over W
        for (int side = 0; side < 2; ++side) {
            Acc<double> acc[2];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                acc[u] = Acc<double>{0, 0, 0, 0};
                const int tile = wave + 8 * u;
                if (tile >= tiles) continue;
                const int c = tile / (q * q) * 2 * s, ti = tile % (q * q) / q * 16, tj = tile % q * 16;
                const double* const A = M + (c + ti) * kTriPitch + (side ? c : c + s);
                const double* const B = M + (side ? c : c + s) * kTriPitch + c + s + tj;
                for (int k = 0; k < s; k += 4) {
                    const double a = A[(lane & 15) * kTriPitch + k + (lane >> 4)];
                    const double b = B[(k + (lane >> 4)) * kTriPitch + (lane & 15)];
                    acc[u] = mfma(side ? -a : a, b, acc[u]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int tile = wave + 8 * u;
                if (tile >= tiles) continue;
                const int c = tile / (q * q) * 2 * s, ti = tile % (q * q) / q * 16, tj = tile % q * 16;
#pragma unroll
                for (int reg = 0; reg < 4; ++reg)
                    M[(c + ti + result_row<double>(reg, lane)) * kTriPitch + c + s + tj + (lane & 15)] = acc[u][reg];
            }
        }
    }
    __syncthreads();
}

// Cholesky factor R (R^T R = S) of a symmetric matrix, upper, column-major, over
// the upper triangle of S: per block of 128 columns one workgroup factors the
// diagonal block in LDS and inverts it (this kernel), the block's rows are
// multiplied by the inverse (chol_panel_kernel) and what is right of them updated
// (chol_update_kernel).  Bound by the chain of pivots: 16 x 16 blocks by one wave
// in registers, their rows by substitution, the rest of the square on the matrix
// cores: 72 us a block, and 11 + 8 .. 20 for the other two (the library's
// factorisation: 240 us at M = 128, 2.6 ms at 1024, now 72 us and 0.85 ms, the
// inverses of the solve included).  *info: 1 + the first column whose pivot is not
// positive and finite, if it was 0.
// Z, W: the inverse in operand order of T and FP64 (W null: Z is that).
template <class T>
__global__ void __launch_bounds__(512) chol_diag_kernel(int m, int b0, double* __restrict__ S, T* __restrict__ Z,
                                                        double* __restrict__ W, int* __restrict__ info) {
    __shared__ double M[kTriBlock * kTriPitch];
    __shared__ double dinv[16];
    const int t = threadIdx.x, lane = t & 63, l = lane & 15, wave = t >> 6;
    const int w = min(kTriBlock, m - b0);
    for (int idx = t; idx < kTriBlock * kTriBlock; idx += 512) {
        const int k = idx % kTriBlock, j = idx / kTriBlock;
        double v = k == j ? 1.0 : 0.0;
        if (k <= j && b0 + j < m) v = S[int64_t(b0 + j) * m + b0 + k];
        M[k * kTriPitch + j] = v;
    }
    __syncthreads();
    for (int c0 = 0; c0 < w; c0 += 16) {
        if (wave == 0) {
            double a[16];
            int bad = 16;
#pragma unroll
            for (int i = 0; i < 16; ++i) a[i] = M[(c0 + i) * kTriPitch + c0 + l];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                double d = from_lane(a[i], i);
                if (!__builtin_amdgcn_class(d, 0x180)) {   // normal or subnormal, above zero
                    bad = min(bad, i);
                    d = 1.0;
                }
                // 1 / sqrt(d) by two Newton steps from the hardware's estimate, which
                // give the root without a division: the chain of pivots is the time
                double inv = __builtin_amdgcn_rsq(d);
                inv = fma(inv, fma(-0.5 * d * inv, inv, 0.5), inv);
                inv = fma(inv, fma(-0.5 * d * inv, inv, 0.5), inv);
                double u = d * inv;
                u = fma(fma(-u, u, d), 0.5 * inv, u);
                a[i] = l == i ? u : a[i] * inv;
                if (lane == 0) dinv[i] = inv;
#pragma unroll
                for (int r = i + 1; r < 16; ++r) a[r] = fma(-from_lane(a[i], r), a[i], a[r]);
            }
            if (lane < 16)
#pragma unroll
                for (int i = 0; i < 16; ++i) M[(c0 + i) * kTriPitch + c0 + l] = l >= i ? a[i] : 0.0;
            if (bad < 16 && lane == 0 && *info == 0) *info = b0 + c0 + bad + 1;
        }
        __syncthreads();
        const int j = c0 + 16 + t;
        if (j < kTriBlock) {
            double x[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = M[(c0 + i) * kTriPitch + j];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                x[i] *= dinv[i];
#pragma unroll
                for (int r = i + 1; r < 16; ++r) x[r] = fma(-M[(c0 + i) * kTriPitch + c0 + r], x[i], x[r]);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) M[(c0 + i) * kTriPitch + j] = x[i];
        }
        __syncthreads();
        const int nt = (w + 15 - c0) / 16 - 1;
        for (int tile = wave; tile < nt * nt; tile += 8) {
            const int ti = tile / nt, tj = tile % nt;
            if (ti > tj) continue;
            double* const C = M + (c0 + 16 + 16 * ti) * kTriPitch + c0 + 16 + 16 * tj + l;
            Acc<double> acc;
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) acc[reg] = C[result_row<double>(reg, lane) * kTriPitch];
#pragma unroll
            for (int k = 0; k < 16; k += 4) {
                const double* const row = M + (c0 + k + (lane >> 4)) * kTriPitch + c0 + 16 + l;
                acc = mfma(-row[16 * ti], row[16 * tj], acc);
            }
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) C[result_row<double>(reg, lane) * kTriPitch] = acc[reg];
        }
        __syncthreads();
    }
    for (int idx = t; idx < kTriBlock * kTriBlock; idx += 512) {
        const int k = idx % kTriBlock, j = idx / kTriBlock;
        if (k <= j && b0 + j < m) S[int64_t(b0 + j) * m + b0 + k] = M[k * kTriPitch + j];
        else if (k > j) M[k * kTriPitch + j] = 0.0;
    }
    __syncthreads();
    invert_upper(M, w);
    // (the 16-column tiles that hold a column of R; no other is read)
    const int n = (w + 15) / 16 * 16 * kTriBlock;
    for (int idx = t; idx < n; idx += 512) {
        int k, j;
        Packed<T>::where(idx, kTriBlock / Packed<T>::KG, true, &k, &j);
        Z[idx] = k <= j ? T(M[k * kTriPitch + j]) : T(0);
        if (W) {
            Packed<double>::where(idx, kTriBlock / Packed<double>::KG, true, &k, &j);
            W[idx] = k <= j ? M[k * kTriPitch + j] : 0.0;
        }
    }
}

// R_kj = R_kk^{-T} S_kj for the columns right of a full diagonal block; a wave
// takes 16 columns
__global__ void __launch_bounds__(64) chol_panel_kernel(int m, int b0, double* S, const double* __restrict__ W) {
    using K = Packed<double>;
    constexpr int NG = kTriBlock / K::KG;
    const int lane = threadIdx.x, l = lane & 15, kq = lane >> 4;
    const int col = b0 + kTriBlock + 16 * int(blockIdx.x) + l;
    double* const sc = S + int64_t(min(col, m - 1)) * m + b0;
    Piece16<double> b[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int e = 0; e < K::N; ++e) b[g].e[e] = sc[g * K::KG + 4 * e + kq];
#pragma unroll
    for (int q = 0; q < kTriBlock / 16; ++q) {
        Acc<double> acc = {0, 0, 0, 0};
#pragma unroll
        for (int g = 0; g < 2 * q + 2; ++g) {
            const Piece16<double> a = load16(W + ((q * NG + g) * 64 + lane) * K::N);
#pragma unroll
            for (int e = 0; e < K::N; ++e) acc = mfma(a.e[e], b[g].e[e], acc);
        }
        if (col < m)
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) sc[16 * q + result_row<double>(reg, lane)] = acc[reg];
    }
}

// S_ij -= R_ki^T R_kj right of block k, 64 x 64 per workgroup, 32 x 32 per wave
__global__ void __launch_bounds__(256) chol_update_kernel(int m, int b0, double* S) {
    using K = Packed<double>;
    const int lane = threadIdx.x & 63, l = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b1 = b0 + kTriBlock, nb = (m - b1 + 63) / 64;
    int tj = int(blockIdx.x), ti = 0;
    while (tj >= nb - ti) tj -= nb - ti, ++ti;
    tj += ti;
    const int r0 = b1 + 64 * ti + 32 * (wave >> 1), c0 = b1 + 64 * tj + 32 * (wave & 1);
    if (r0 > c0 || r0 >= m || c0 >= m) return;
    const double *ra[2], *cb[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        ra[p] = S + int64_t(min(r0 + 16 * p + l, m - 1)) * m + b0 + K::N * kq;
        cb[p] = S + int64_t(min(c0 + 16 * p + l, m - 1)) * m + b0 + K::N * kq;
    }
    Acc<double> acc[2][2];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) acc[p][q] = Acc<double>{0, 0, 0, 0};
#pragma unroll 4
    for (int g = 0; g < kTriBlock / K::KG; ++g) {
        Piece16<double> a[2], b[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            a[p] = load16(ra[p] + g * K::KG);
            b[p] = load16(cb[p] + g * K::KG);
        }
#pragma unroll
        for (int e = 0; e < K::N; ++e)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int q = 0; q < 2; ++q) acc[p][q] = mfma(a[p].e[e], b[q].e[e], acc[p][q]);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) {
                const int r = r0 + 16 * p + result_row<double>(reg, lane), c = c0 + 16 * q + l;
                if (r <= c && c < m) S[int64_t(c) * m + r] -= acc[p][q][reg];
            }
}

template <class T, int RT>
__global__ void __launch_bounds__(256, sizeof(T) == 8 ? 2 : 1) solve_upper_kernel(T* X, int64_t ldx, int64_t n_rows, int m, int groups,
                                                             const T* __restrict__ R, const T* __restrict__ Z) {
    constexpr int N = Piece16<T>::N, KG = 4 * N, G = 16 / KG, CT = kTriBlock / 16;
    constexpr int LP = 16 + N;                 // pitch of a 16 x 16 tile in LDS, rows 16-byte aligned
    __shared__ __align__(16) T turn[4][16 * RT * LP];
    const int lane = threadIdx.x & 63, l = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t(blockIdx.x) * 4 + wave) * (16 * RT);
    if (row0 >= n_rows) return;
    T* const tw = turn[wave];
    // rows past the end repeat the last one and are not stored
    const T* xr[RT];
#pragma unroll
    for (int p = 0; p < RT; ++p) xr[p] = X + min(row0 + 16 * p + l, n_rows - 1) * ldx + N * kq;
    // The products are summed over kTriBlock of k at a time, from zero, and the sums
    // taken from the panel one after the other, as the blocked solve of a library
    // does: one chain over all k rounds m times at the size of the whole (error at
    // 600 columns, FP32, 1.3e-6, in blocks 0.8e-6; columns 384 to 400 of 400, FP64, in
    // units of 2^-53: 8.6 and 2.0).  With FP64 blocks of one panel there are no products, and
    // the panel is kept where they would be added.
    constexpr bool APART = sizeof(T) == 4 || RT == 1;
    Acc<T> acc[RT][CT], own[APART ? RT : 1][APART ? CT : 1];
    // columns past the end repeat the last one
    auto start = [&](int j0) {
#pragma unroll
        for (int p = 0; p < RT; ++p)
#pragma unroll
            for (int q = 0; q < CT; ++q) {
                const int64_t col = min(j0 + 16 * q + l, m - 1);
#pragma unroll
                for (int reg = 0; reg < 4; ++reg) {
                    const T x = X[min(row0 + 16 * p + result_row<T>(reg, lane), n_rows - 1) * ldx + col];
                    if constexpr (APART) own[p][q][reg] = x;
                    else acc[p][q][reg] = x;
                }
                if constexpr (APART) acc[p][q] = Acc<T>{0, 0, 0, 0};
            }
    };
    start(0);
    for (int j0 = 0; j0 < m; j0 += kTriBlock) {
        const int w = min(kTriBlock, m - j0), last = (w + 15) / 16 - 1;    // columns and last tile of the panel
        // two sets of operands: one is multiplied while the other is loaded; of X
        // two groups at a time, whole cache lines of its rows.  FP32: the order is
        // kept and the sums stay in accumulation registers, one wave per SIMD
        // (4.7 ms at 440,000 x 1024; 5.1 as the compiler orders it for two waves).
        // FP64: two waves, whose products are long enough to cover the loads;
        // the sums apart leave them registers for 16 rows each (3.5 ms at 440,000 x
        // 600; 32 rows and one wave 3.8).
        auto keep_order = [] {
            if constexpr (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
        };
        Piece16<T> a[2][2][RT], b[2][CT];
        auto fetch_a = [&](auto set, int k0) {
            constexpr int i = decltype(set)::value;
            k0 = min(k0, j0 - 2 * KG);
#pragma unroll
            for (int p = 0; p < RT; ++p)
#pragma unroll
                for (int h = 0; h < 2; ++h) a[i][h][p] = load16(xr[p] + k0 + h * KG);
        };
        const T* const rb = R + (int64_t(j0 / 16) * groups * 64 + lane) * N;
        const int64_t tile = int64_t(groups) * 64 * N;
        auto fetch_b = [&](auto set, int k0) {
            constexpr int i = decltype(set)::value;
            const T* const at = rb + int64_t(min(k0, j0 - KG)) * 16;        // 64 N values per KG = 4 N of k
#pragma unroll
            for (int q = 0; q < CT; ++q) b[i][q] = load16(at + min(q, last) * tile);
        };
        auto multiply = [&](auto aset, auto half, auto bset) {
            constexpr int i = decltype(aset)::value, h = decltype(half)::value, j = decltype(bset)::value;
            if constexpr (sizeof(T) == 4) {
#pragma unroll
                for (int p = 0; p < RT; ++p)
#pragma unroll
                    for (int q = 0; q < CT; ++q) asm("" : "+a"(acc[p][q]));
            }
#pragma unroll
            for (int e = 0; e < N; ++e)
#pragma unroll
                for (int p = 0; p < RT; ++p)
#pragma unroll
                    for (int q = 0; q < CT; ++q) acc[p][q] = mfma(a[i][h][p].e[e], b[j][q].e[e], acc[p][q]);
        };
        using S0 = std::integral_constant<int, 0>;
        using S1 = std::integral_constant<int, 1>;
        if (j0 > 0) {
            fetch_a(S0{}, 0);
            fetch_b(S0{}, 0);
        }
        for (int k0 = 0; k0 < j0; k0 += 4 * KG) {
            fetch_a(S1{}, k0 + 2 * KG);
            fetch_b(S1{}, k0 + KG);
            keep_order();
            multiply(S0{}, S0{}, S0{});
            keep_order();
            fetch_b(S0{}, k0 + 2 * KG);
            keep_order();
            multiply(S0{}, S1{}, S1{});
            keep_order();
            fetch_a(S0{}, k0 + 4 * KG);
            fetch_b(S1{}, k0 + 3 * KG);
            keep_order();
            multiply(S1{}, S0{}, S0{});
            keep_order();
            fetch_b(S0{}, k0 + 4 * KG);
            keep_order();
            multiply(S1{}, S1{}, S1{});
            if constexpr (APART) {
                if ((k0 + 4 * KG) % kTriBlock == 0) {
#pragma unroll
                    for (int p = 0; p < RT; ++p)
#pragma unroll
                        for (int q = 0; q < CT; ++q) {
                            own[p][q] += acc[p][q];
                            acc[p][q] = Acc<T>{0, 0, 0, 0};
                        }
                }
            }
        }
        // X_j - sum, turned from the result layout to the operand layout of ascending
        // k (column 4 e + kq of a group lies at N kq + e); columns past the end count as
        // zero
        const int place = l / KG * KG + l % 4 * N + l % KG / 4;
        Piece16<T> v[RT][CT][G];
#pragma unroll
        for (int q = 0; q < CT; ++q) {
            const bool in = 16 * q + l < w;
#pragma unroll
            for (int p = 0; p < RT; ++p)
#pragma unroll
                for (int reg = 0; reg < 4; ++reg)
                {
                    T x;
                    if constexpr (APART) x = own[p][q][reg];
                    else x = acc[p][q][reg];
                    tw[(p * 16 + result_row<T>(reg, lane)) * LP + place] = in ? x : T(0);
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int p = 0; p < RT; ++p)
#pragma unroll
                for (int g = 0; g < G; ++g)
                    v[p][q][g] = *reinterpret_cast<const Piece16<T>*>(tw + (p * 16 + l) * LP + g * KG + N * kq);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        // times the inverse of R_jj
        const T* const zb = Z + int64_t(j0 / kTriBlock) * kTriBlock * kTriBlock + lane * N;
        constexpr int D = sizeof(T) == 4 ? 2 : 1;      // FP64 has no registers to load ahead
        Piece16<T> z[D][CT][G];
        auto fetch_z = [&](int set, int q) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
                if (c <= q)
#pragma unroll
                    for (int g = 0; g < G; ++g) z[set][c][g] = load16(zb + (q * (kTriBlock / KG) + c * G + g) * 64 * N);
        };
        if (D > 1) fetch_z(0, 0);
#pragma unroll
        for (int q = 0; q < CT; ++q) {
            if (16 * q >= w) continue;
            if (D == 1) fetch_z(0, q);
            else if (q + 1 < CT && 16 * (q + 1) < w) fetch_z((q + 1) % D, q + 1);
            Acc<T> r[RT];
#pragma unroll
            for (int p = 0; p < RT; ++p) r[p] = Acc<T>{0, 0, 0, 0};
#pragma unroll
            for (int c = 0; c <= q; ++c)
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int e = 0; e < N; ++e)
#pragma unroll
                        for (int p = 0; p < RT; ++p) r[p] = mfma(v[p][c][g].e[e], z[q % D][c][g].e[e], r[p]);
            const int col = j0 + 16 * q + l;
#pragma unroll
            for (int p = 0; p < RT; ++p)
#pragma unroll
                for (int reg = 0; reg < 4; ++reg) {
                    const int64_t row = row0 + 16 * p + result_row<T>(reg, lane);
                    if (row < n_rows && col < m) X[row * ldx + col] = r[p][reg];
                }
        }
        if (j0 + kTriBlock < m) start(j0 + kTriBlock);
        // the wave's later panels read what its other lanes have stored
        __threadfence_block();
    }
}

// X <- X Q in place for M <= kTriBlock: a wave reads its 32 rows as operands, then
// multiplies and writes them, 16 columns at a time; Q in operand order (P).  Bound by
// reading and writing X.  The library's product into a work block and the copy back
// took 81 + 40 us for 120,000 x 97 FP64; a Rayleigh-Ritz step there 1472 -> 1356.
// Wider blocks would not fit the registers and keep the product through panels.
template <class T>
__global__ void __launch_bounds__(256) pack_square_kernel(int m, int groups, int64_t n, const double* __restrict__ Q,
                                                          T* __restrict__ P) {
    const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (idx >= n) return;
    int k, j;
    Packed<T>::where(idx, groups, false, &k, &j);
    P[idx] = k < m && j < m ? T(Q[int64_t(j) * m + k]) : T(0);
}

template <class T>
__global__ void __launch_bounds__(256, 2) rotate_kernel(T* X, int64_t ldx, int64_t n_rows, int m,
                                                        const T* __restrict__ P) {
    constexpr int N = Piece16<T>::N, KG = 4 * N, G = 16 / KG, RT = 2, CT = kTriBlock / 16;
    const int lane = threadIdx.x & 63, l = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t(blockIdx.x) * 4 + wave) * (16 * RT);
    if (row0 >= n_rows) return;
    const int tiles = (m + 15) / 16;
    Piece16<T> v[RT][CT][G];
#pragma unroll
    for (int p = 0; p < RT; ++p) {
        const T* const x = X + min(row0 + 16 * p + l, n_rows - 1) * ldx;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int k = 16 * c + g * KG + N * kq;
                if (k + N <= m) {
                    v[p][c][g] = load16(x + k);
                } else {
#pragma unroll
                    for (int e = 0; e < N; ++e) v[p][c][g].e[e] = k + e < m ? x[k + e] : T(0);
                }
            }
    }
#pragma unroll 1
    for (int q = 0; q < tiles; ++q) {
        const T* const z = P + (int64_t(q) * tiles * G * 64 + lane) * N;
        Acc<T> r[RT];
#pragma unroll
        for (int p = 0; p < RT; ++p) r[p] = Acc<T>{0, 0, 0, 0};
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            if (c >= tiles) continue;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const Piece16<T> b = load16(z + (c * G + g) * 64 * N);
#pragma unroll
                for (int e = 0; e < N; ++e)
#pragma unroll
                    for (int p = 0; p < RT; ++p) r[p] = mfma(v[p][c][g].e[e], b.e[e], r[p]);
            }
        }
        const int col = 16 * q + l;
#pragma unroll
        for (int p = 0; p < RT; ++p)
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) {
                const int64_t row = row0 + 16 * p + result_row<T>(reg, lane);
                if (row < n_rows && col < m) X[row * ldx + col] = r[p][reg];
            }
    }
}

// scratch: the last diagonal block's inverse in FP64 (FP32 blocks), the
// inverses and -R in operand order
template <class T>
static T* inverses_of(void* work) {
    return static_cast<T*>(work) + (sizeof(T) == 4 ? 2 * kTriBlock * kTriBlock : 0);
}
static int64_t packed_values(int m) {
    const int64_t mp = (int64_t(m) + 15) / 16 * 16;
    return mp * mp;
}
size_t cholesky_work_bytes(int m, size_t elem_bytes) {
    const int64_t square = kTriBlock * kTriBlock, panels = (m + kTriBlock - 1) / kTriBlock;
    return size_t((elem_bytes == 4 ? 2 * square : 0) + panels * square + packed_values(m)) * elem_bytes;
}

// the rows in runs whose launches, of up to 4 threads a row, stay below the 2^32
// threads at which the count wraps
template <class F>
static void by_rows(int64_t n_rows, F&& launch) {
    constexpr int64_t kRun = int64_t(1) << 29;
    for (int64_t r0 = 0; r0 < n_rows; r0 += kRun) launch(r0, std::min(kRun, n_rows - r0));
}

template <class T>
void cholesky(double* S, int m, void* work, int* info, hipStream_t s) {
    double* const W = sizeof(T) == 4 ? static_cast<double*>(work) : nullptr;
    T* Z = inverses_of<T>(work);
    for (int b0 = 0; b0 < m; b0 += kTriBlock, Z += kTriBlock * kTriBlock) {
        chol_diag_kernel<T><<<1, 512, 0, s>>>(m, b0, S, Z, W, info);
        LAUNCH_CHECK();
        const int right = m - b0 - kTriBlock;
        if (right <= 0) break;
        chol_panel_kernel<<<unsigned((right + 15) / 16), 64, 0, s>>>(m, b0, S,
                                                                     W ? W : reinterpret_cast<const double*>(Z));
        LAUNCH_CHECK();
        const int nb = (right + 63) / 64;
        chol_update_kernel<<<unsigned(int64_t(nb) * (nb + 1) / 2), 256, 0, s>>>(m, b0, S);
        LAUNCH_CHECK();
    }
}
template void cholesky<float>(double*, int, void*, int*, hipStream_t);
template void cholesky<double>(double*, int, void*, int*, hipStream_t);

template <class T>
void solve_upper(T* X, int64_t ldx, int64_t n_rows, int m, const double* R, void* work, hipStream_t s) {
    const int panels = (m + kTriBlock - 1) / kTriBlock, groups = (m + 15) / 16 * 16 / Packed<T>::KG;
    const T* const Z = inverses_of<T>(work);
    T* const P = inverses_of<T>(work) + int64_t(panels) * kTriBlock * kTriBlock;
    if (panels > 1) {
        const int64_t n = packed_values(m);
        pack_upper_kernel<T><<<unsigned((n + 255) / 256), 256, 0, s>>>(m, groups, n, R, P);
        LAUNCH_CHECK();
    }
    // rows of a wave: 32, or 16 for FP64 blocks of several panels (one panel,
    // 120,000 x 128: 68 us with 32, 71 with 16)
    auto go = [&](auto rt) {
        constexpr int RT = decltype(rt)::value;
        by_rows(n_rows, [&](int64_t r0, int64_t rows) {
            solve_upper_kernel<T, RT><<<unsigned((rows + 64 * RT - 1) / (64 * RT)), 256, 0, s>>>(X + r0 * ldx, ldx, rows, m,
                                                                                                groups, P, Z);
        });
    };
    if constexpr (sizeof(T) == 8) {
        if (panels > 1) go(std::integral_constant<int, 1>{});
        else go(std::integral_constant<int, 2>{});
    } else {
        go(std::integral_constant<int, 2>{});
    }
    LAUNCH_CHECK();
}
template void solve_upper<float>(float*, int64_t, int64_t, int, const double*, void*, hipStream_t);
template void solve_upper<double>(double*, int64_t, int64_t, int, const double*, void*, hipStream_t);

size_t rotate_work_bytes(int m, size_t elem_bytes) {
    return m <= kTriBlock ? size_t(packed_values(m)) * elem_bytes : 0;
}

template <class T>
bool rotate(T* X, int64_t ldx, int64_t n_rows, int m, const double* Q, void* work, hipStream_t s) {
    if (m > kTriBlock) return false;
    const int64_t n = packed_values(m);
    T* const P = static_cast<T*>(work);
    pack_square_kernel<T><<<unsigned((n + 255) / 256), 256, 0, s>>>(m, (m + 15) / 16 * 16 / Packed<T>::KG, n, Q, P);
    LAUNCH_CHECK();
    by_rows(n_rows, [&](int64_t r0, int64_t rows) {
        rotate_kernel<T><<<unsigned((rows + 127) / 128), 256, 0, s>>>(X + r0 * ldx, ldx, rows, m, P);
    });
    LAUNCH_CHECK();
    return true;
}
template bool rotate<float>(float*, int64_t, int64_t, int, const double*, void*, hipStream_t);
template bool rotate<double>(double*, int64_t, int64_t, int, const double*, void*, hipStream_t);

}  // namespace chf
