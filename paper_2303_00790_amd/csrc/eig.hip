// Symmetric eigenproblem of the projected Hamiltonian for M <= kEigMax: own
// reduction to tridiagonal form and back-transformation around the library's
// divide and conquer.
//
// The reduction is a chain of M - 2 steps, each a matrix-vector product with and
// a rank-2 update of what is left, so it is bound by the latency of a step (two
// sums, a root and a division, 1.5 us with no matrix at all).  One workgroup
// keeps the whole matrix in its registers, 8 threads to a row, and a step costs
// two barriers: every wave forms the step's sums for itself from the column in
// LDS.  Larger blocks go to the library, whose reduction keeps the matrix in
// memory: 192 x 192 doubles are 144 registers of each of 512 threads, and the
// next multiple would not leave two waves per SIMD the registers they work with.
// M = 97: 215 us (the library's reduction there: 626 for the largest of its kernels),
// back-transformation 27.  A whole Rayleigh-Ritz at 1.1 nm (FP64, full work block),
// with the library's reduction, Gram product and rotation -> now: M = 24 1112 -> 499
// us, 64 2337 -> 918, 97 2347 -> 1326, 128 3053 -> 1640, 192 5020 -> 2596; 200, through
// the library, 5317 -> 5273.  Eigenvalues against 80 bits over 8 to 192 states:
// 0.88 to 1.39 units of 2^-53 of the norm, the library's 1.01 to 1.34.
#include <algorithm>

#include "internal.hpp"
#include "kernels.hpp"

namespace chf {

namespace {

template <int CTRL>
__device__ inline double dpp(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// sum over aligned groups of 8 and 16 lanes, the same on all of them: lane ^ 1,
// lane ^ 2, the mirrored half row, the row rotated by 8
__device__ inline double sum8(double v) {
    v += dpp<0xB1>(v);
    v += dpp<0x4E>(v);
    v += dpp<0x141>(v);
    return v;
}
__device__ inline double sum16(double v) {
    v = sum8(v);
    v += dpp<0x128>(v);
    return v;
}

}  // namespace

// Q^T S Q = T: diagonal D[m], off-diagonal E[m - 1], Q = H_0 H_1 .. H_{m-3} with
// H_k = 1 - tau_k y_k y_k^T, y_k in V[k m ..] (zero up to k).
// Thread (ti, tj) = (t / 8, t % 8) holds rows ti + TI r, columns 16 b + 2 tj + {0, 1}.
template <int TI, int RA, int CB>
__global__ void __launch_bounds__(8 * TI) tridiag_kernel(int m, const double* __restrict__ S, double* __restrict__ D,
                                                         double* __restrict__ E, double* __restrict__ V,
                                                         double* __restrict__ tau) {
    constexpr int W = 16 * CB, WAVES = TI / 8;
    static_assert(TI * RA == W, "rows and columns of the same padded matrix");
    __shared__ __align__(16) double ys[2][W], ps[2][W];
    __shared__ double big[WAVES], diag[2];
    const int t = threadIdx.x, tj = t & 7, ti = t >> 3, l16 = t & 15;
    double a[RA][2 * CB];
    double amax = 0.0;
#pragma unroll
    for (int r = 0; r < RA; ++r)
#pragma unroll
        for (int c = 0; c < 2 * CB; ++c) {
            const int i = ti + TI * r, j = c / 2 * 16 + 2 * tj + c % 2;
            a[r][c] = i < m && j < m ? S[int64_t(i) * m + j] : 0.0;
            amax = fmax(amax, fabs(a[r][c]));
        }
    // a power of two brings the entries to the order of one, so that no square
    // over- or underflows
    for (int off = 32; off > 0; off >>= 1) amax = fmax(amax, __shfl_xor(amax, off, 64));
    if ((t & 63) == 0) big[t >> 6] = amax;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WAVES; ++i) amax = fmax(amax, big[i]);
    int ex = 0;
    if (amax > 0.0 && isfinite(amax)) (void)frexp(amax, &ex);
#pragma unroll
    for (int r = 0; r < RA; ++r)
#pragma unroll
        for (int c = 0; c < 2 * CB; ++c) a[r][c] = ldexp(a[r][c], -ex);
    // column k to LDS from the threads that hold it: what is below the diagonal,
    // zero up to it
    auto publish = [&](int k) {
#pragma unroll
        for (int b = 0; b < CB; ++b)
            if (b == k >> 4 && tj == (k & 15) >> 1)
#pragma unroll
                for (int r = 0; r < RA; ++r) {
                    const int i = ti + TI * r;
                    const double v = k & 1 ? a[r][2 * b + 1] : a[r][2 * b];
                    ys[k & 1][i] = i > k ? v : 0.0;
                    if (i == k) diag[k & 1] = v;
                }
    };
    publish(0);
    for (int k = 0; k + 2 < m; ++k) {
        __syncthreads();
        const double* const y = ys[k & 1];
        // y = column below the diagonal, with y_{k+1} = al - beta;  tau = 2 / |y|^2
        const double al = y[k + 1];
        double sg = 0.0;
#pragma unroll
        for (int c = 0; c < CB; ++c) sg = fma(y[16 * c + l16], y[16 * c + l16], sg);
        sg = sum16(l16 == ((k + 1) & 15) ? fma(-al, al, sg) : sg);
        // (the column's square without al^2: summed again where that cancels)
        if (!(sg > 0.25 * al * al)) {
            sg = 0.0;
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                const double v = 16 * c + l16 == k + 1 ? 0.0 : y[16 * c + l16];
                sg = fma(v, v, sg);
            }
            sg = sum16(sg);
        }
        double beta = al, tk = 0.0, y1 = 0.0;
        if (!(sg < 1e-280)) {
            beta = -copysign(sqrt(fma(al, al, sg)), al);
            y1 = al - beta;
            tk = -1.0 / (beta * y1);
        }
        double p[RA];
#pragma unroll
        for (int r = 0; r < RA; ++r) p[r] = 0.0;
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            if (16 * b + 15 <= k) continue;
            const int j = 16 * b + 2 * tj;
            double2 yj = *reinterpret_cast<const double2*>(y + j);
            if (b == (k + 1) >> 4) {
                yj.x = j == k + 1 ? y1 : yj.x;
                yj.y = j + 1 == k + 1 ? y1 : yj.y;
            }
#pragma unroll
            for (int r = 0; r < RA; ++r) p[r] = fma(a[r][2 * b + 1], yj.y, fma(a[r][2 * b], yj.x, p[r]));
        }
        double yi[RA];
#pragma unroll
        for (int r = 0; r < RA; ++r) {
            const int i = ti + TI * r;
            p[r] = sum8(p[r]);
            yi[r] = i == k + 1 ? y1 : y[i];
            if (tj == 0) ps[k & 1][i] = p[r];
            if (tj == 1 && i < m) V[int64_t(k) * m + i] = yi[r];
        }
        if (t == 0) {
            D[k] = ldexp(diag[k & 1], ex);
            E[k] = ldexp(beta, ex);
            tau[k] = tk;
        }
        __syncthreads();
        // w = tau p - (tau^2 / 2) (y.p) y;  A -= y w^T + w y^T
        const double* const q = ps[k & 1];
        double yp = 0.0;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int i = 16 * c + l16;
            double v = y[i];
            if (c == (k + 1) >> 4) v = i == k + 1 ? y1 : v;
            yp = fma(q[i], v, yp);
        }
        const double h = tk * (tk * sum16(yp));
        double wi[RA];
#pragma unroll
        for (int r = 0; r < RA; ++r) {
            wi[r] = fma(h, yi[r], -tk * p[r]);
            yi[r] = -tk * yi[r];
        }
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            if (16 * b + 15 <= k) continue;
            const int j = 16 * b + 2 * tj;
            double2 yj = *reinterpret_cast<const double2*>(y + j);
            const double2 qj = *reinterpret_cast<const double2*>(q + j);
            if (b == (k + 1) >> 4) {
                yj.x = j == k + 1 ? y1 : yj.x;
                yj.y = j + 1 == k + 1 ? y1 : yj.y;
            }
#pragma unroll
            for (int r = 0; r < RA; ++r) {
                a[r][2 * b] = fma(wi[r], yj.x, fma(yi[r], qj.x, a[r][2 * b]));
                a[r][2 * b + 1] = fma(wi[r], yj.y, fma(yi[r], qj.y, a[r][2 * b + 1]));
            }
        }
        publish(k + 1);
    }
    __syncthreads();
    // what is left: the last two diagonal entries and the one beside them
    const int k = max(m - 2, 0);
    if (t == 0) {
        D[k] = ldexp(diag[k & 1], ex);
        if (m > 1) E[k] = ldexp(ys[k & 1][k + 1], ex);
    }
    if (m > 1) publish(m - 1);
    __syncthreads();
    if (t == 0 && m > 1) D[m - 1] = ldexp(diag[(m - 1) & 1], ex);
}

// Z <- H_0 H_1 .. H_{m-3} Z (columns, column-major): 16 lanes per column, 4
// columns per wave
template <int CB>
__global__ void __launch_bounds__(64) back_transform_kernel(int m, const double* __restrict__ V,
                                                            const double* __restrict__ tau, double* __restrict__ Z) {
    const int l = threadIdx.x & 15, col = int(blockIdx.x) * 4 + int(threadIdx.x >> 4);
    const bool in = col < m;
    double* const zc = Z + int64_t(in ? col : 0) * m;
    constexpr int AHEAD = 4;
    double z[CB], v[AHEAD][CB], tk[AHEAD];
#pragma unroll
    for (int c = 0; c < CB; ++c) z[c] = 16 * c + l < m ? zc[16 * c + l] : 0.0;
    for (int k0 = m - 3; k0 >= 0; k0 -= AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int k = max(k0 - u, 0);
            tk[u] = k0 - u >= 0 ? tau[k] : 0.0;
#pragma unroll
            for (int c = 0; c < CB; ++c) v[u][c] = 16 * c + l < m ? V[int64_t(k) * m + 16 * c + l] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            double s = 0.0;
#pragma unroll
            for (int c = 0; c < CB; ++c) s = fma(v[u][c], z[c], s);
            s = tk[u] * sum16(s);
#pragma unroll
            for (int c = 0; c < CB; ++c) z[c] = fma(-s, v[u][c], z[c]);
        }
    }
#pragma unroll
    for (int c = 0; c < CB; ++c)
        if (in && 16 * c + l < m) zc[16 * c + l] = z[c];
}

size_t eig_work_bytes(int m) {
    return m <= kEigMax ? (size_t(m) * m + size_t(m)) * sizeof(double) : 0;
}

void sym_eig(chf_ctx* ctx, int m, double* S, double* evals, double* E, double* work, int* info, hipStream_t s) {
    ROCBLAS_CHECK(rocblas_set_stream(ctx->blas, s));
    if (m > kEigMax) {
        ROCBLAS_CHECK(rocsolver_dsyevd(ctx->blas, rocblas_evect_original, rocblas_fill_upper, m, S, m, evals, E, info));
        return;
    }
    double* const V = work;
    double* const tau = work + size_t(m) * m;
    auto go = [&](auto threads, auto width) {
        constexpr int TI = decltype(threads)::value / 8, W = decltype(width)::value;
        tridiag_kernel<TI, W / TI, W / 16><<<1, 8 * TI, 0, s>>>(m, S, evals, E, V, tau);
        LAUNCH_CHECK();
        ROCBLAS_CHECK(rocsolver_dstedc(ctx->blas, rocblas_evect_tridiagonal, m, evals, E, S, m, info));
        back_transform_kernel<W / 16><<<unsigned((m + 3) / 4), 64, 0, s>>>(m, V, tau, S);
        LAUNCH_CHECK();
    };
    using std::integral_constant;
    // threads: 229 us with 256 and 214 with 512 at M = 97, 84 with 256 and 93 with 128 at 64
    if (m <= 64) go(integral_constant<int, 256>{}, integral_constant<int, 64>{});
    else if (m <= 128) go(integral_constant<int, 512>{}, integral_constant<int, 128>{});
    else go(integral_constant<int, 512>{}, integral_constant<int, kEigMax>{});
}

}  // namespace chf
