// Hamiltonian application and the Chebyshev filter on gfx950.
//
// Paper: ChFSI's efficiency rests on sparse H-times-wavefunction products;
// the grid points are stored along blockwise Hilbert space-filling curves so
// that these products touch memory with good locality.  H = -1/2 L (12th-
// order FD stencil) + V_eff + sum_a |beta_a> h_l <beta_a| (KB form).
//
// Kernels
//  * vloc_kernel      V_loc on every row (FP64, all atoms, erf screening).
//  * kb_gather        C[a][lm][v] = h^3 sum_q beta_alm(q) X(q, v) per projector atom.
//  * hx_generic       per-row neighbour-table stencil + V + KB scatter, with
//                     the Chebyshev three-term update fused into the store:
//                     Y = alpha (H X - c X) - beta Z  (Z may alias Y).
//  * hx_tile          the same operator on the Hilbert-blocked layout: one
//                     workgroup per (8^3 block, 32-float / 16-double vector
//                     chunk), z-march with a register window per column, x/y
//                     halos and the block atoms' KB coefficients staged in
//                     LDS, the KB term as MFMA products inside the march.
//  * hx_narrow        the same operator for one row piece of at most 16 bytes
//                     (1 or 2 FP64, 2 or 4 FP32 vectors), one thread per point.
//  * hx_tiled         a tile of the same shape without staging, for Hamiltonians
//                     with a block touched by more than kMaxBlockAtoms projector
//                     atoms and those without projectors.
#include <atomic>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "internal.hpp"
#include "kernels.hpp"
#include "reduce.hpp"

namespace chf {

// ---------------------------------------------------------------------------
// local potential
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) vloc_kernel(int64_t n_rows, const int32_t* __restrict__ row_ijk4, double h,
                                                   int n_atoms, const double4* __restrict__ atoms,
                                                   const double* __restrict__ width, double* __restrict__ vloc) {
    __shared__ double4 sa[256];
    __shared__ double sw[256];
    const int64_t row = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const bool live = row < n_rows && row_ijk4[4 * row + 3] != 0;
    double x = 0, y = 0, z = 0;
    if (live) {
        x = double(row_ijk4[4 * row + 0]) * h;
        y = double(row_ijk4[4 * row + 1]) * h;
        z = double(row_ijk4[4 * row + 2]) * h;
    }
    double v = 0.0;
    const double two_over_sqrt_pi = 1.1283791670955126;
    for (int base = 0; base < n_atoms; base += 256) {
        __syncthreads();
        if (base + threadIdx.x < n_atoms) {
            sa[threadIdx.x] = atoms[base + threadIdx.x];
            sw[threadIdx.x] = width[base + threadIdx.x];
        }
        __syncthreads();
        const int cnt = min(256, n_atoms - base);
        if (live) {
            for (int t = 0; t < cnt; ++t) {
                const double4 a = sa[t];
                const double dx = x - a.x, dy = y - a.y, dz = z - a.z;
                const double d = sqrt(dx * dx + dy * dy + dz * dz);
                const double w = sw[t];
                double term;
                if (d < 1e-8)
                    term = a.w * two_over_sqrt_pi / w;
                else if (d > 6.0 * w)   // erf(x) rounds to exactly 1 in FP64 for x > 5.93
                    term = a.w / d;
                else
                    term = a.w * erf(d / w) / d;
                v -= term;
            }
        }
    }
    if (row < n_rows) vloc[row] = live ? v : 0.0;
}

void launch_vloc(chf_ham* H, const double4* atoms, const double* width, int n_atoms, hipStream_t s) {
    const int64_t n = H->grid.n_rows;
    vloc_kernel<<<dim3(unsigned((n + 255) / 256)), dim3(256), 0, s>>>(n, H->row_ijk4.as<int32_t>(), H->h, n_atoms,
                                                                      atoms, width, H->vloc.as<double>());
    LAUNCH_CHECK();
}

__global__ void cast_veff_kernel(int64_t n, const double* __restrict__ src, const uint8_t* __restrict__ inside,
                                 double* __restrict__ d64, float* __restrict__ d32, int* __restrict__ bad) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double v = inside[i] ? src[i] : 0.0;
    if (!isfinite(v)) {
        atomicOr(bad, 1);
        return;
    }
    if (d64) d64[i] = v;
    if (d32) d32[i] = float(v);
}

void launch_cast_veff(chf_ham* H, const double* src, double* d64, float* d32, int* bad_dev, hipStream_t s) {
    const int64_t n = H->grid.n_rows;
    cast_veff_kernel<<<dim3(unsigned((n + 255) / 256)), dim3(256), 0, s>>>(n, src, H->row_inside.as<uint8_t>(),
                                                                          d64, d32, bad_dev);
    LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// generic neighbour-table H X with fused recurrence epilogue
// ---------------------------------------------------------------------------
template <class T>
struct StepCoef {
    T c[7];        // -1/2 c_k / h^2 (c[0] already multiplied by 3: three axes)
    T alpha, shift, beta;
    // the same step with alpha folded in (tiled kernel):
    //   y = sum_k ac[k] (X(p+k) + X(p-k)) + (d0 + alpha V(p)) X(p) + alpha KB - beta Z
    T ac[7];       // alpha c[k], k >= 1 (ac[0] unused)
    T d0;          // alpha (c[0] - shift)
};

template <class T>
__global__ void __launch_bounds__(256) hx_generic_kernel(int64_t row0, int64_t n_rows, int nvec, int nvc,
                                                         const int32_t* __restrict__ nbr,
                                                         const uint8_t* __restrict__ inside,
                                                         const T* __restrict__ veff,
                                                         const int64_t* __restrict__ ent_off,
                                                         const int32_t* __restrict__ ent_atom,
                                                         const T* __restrict__ ent_beta, const T* __restrict__ C,
                                                         const T* __restrict__ X, int64_t ldx, T* Y, int64_t ldy,
                                                         const T* Z, int64_t ldz, StepCoef<T> k) {
    const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t r = gid / nvc, row = row0 + r;
    const int vc = int(gid - r * nvc);
    if (row >= n_rows) return;
    constexpr int VPT = 4;
    const int v0 = vc * VPT;
    if (!inside[row]) {
        for (int e = 0; e < VPT; ++e)
            if (v0 + e < nvec) Y[row * ldy + v0 + e] = T(0);
        return;
    }
    T xc[VPT], acc[VPT];
    const T* xr = X + row * ldx;
    for (int e = 0; e < VPT; ++e) {
        xc[e] = (v0 + e < nvec) ? xr[v0 + e] : T(0);
        acc[e] = k.c[0] * xc[e];
    }
    const int32_t* nb = nbr + row * kNbr;
#pragma unroll
    for (int col = 0; col < kNbr; ++col) {
        const int32_t r = nb[col];
        const int kk = (col % 12) < 6 ? 6 - (col % 12) : (col % 12) - 5;
        if (r >= 0) {
            const T* q = X + int64_t(r) * ldx;
            for (int e = 0; e < VPT; ++e)
                if (v0 + e < nvec) acc[e] += k.c[kk] * q[v0 + e];
        }
    }
    if (veff) {
        const T vr = veff[row];
        for (int e = 0; e < VPT; ++e) acc[e] += vr * xc[e];
    }
    if (ent_off)
    for (int64_t en = ent_off[row]; en < ent_off[row + 1]; ++en) {
        const int64_t a = ent_atom[en];
        const T* b = ent_beta + 4 * en;
        const T* ca = C + a * 4 * nvec;
        for (int e = 0; e < VPT; ++e)
            if (v0 + e < nvec)
                acc[e] += b[0] * ca[v0 + e] + b[1] * ca[nvec + v0 + e] + b[2] * ca[2 * nvec + v0 + e] +
                          b[3] * ca[3 * nvec + v0 + e];
    }
    for (int e = 0; e < VPT; ++e) {
        if (v0 + e >= nvec) continue;
        T y = k.alpha * (acc[e] - k.shift * xc[e]);
        if (Z) y -= k.beta * Z[row * ldz + v0 + e];
        Y[row * ldy + v0 + e] = y;
    }
}

template <class T>
StepCoef<T> make_coef(const chf_ham* H, double alpha, double shift, double beta) {
    StepCoef<T> k;
    k.c[0] = T(3.0 * H->coef[0]);
    for (int i = 1; i < 7; ++i) k.c[i] = T(H->coef[i]);
    k.alpha = T(alpha);
    k.shift = T(shift);
    k.beta = T(beta);
    k.ac[0] = T(0);
    for (int i = 1; i < 7; ++i) k.ac[i] = T(alpha * H->coef[i]);
    k.d0 = T(alpha * (3.0 * H->coef[0] - shift));
    return k;
}

template <class T>
static const T* veff_of(const chf_ham* H) {
    return std::is_same<T, double>::value ? H->veff64.as<T>() : H->veff32.as<T>();
}
template <class T>
static const T* ent_beta_of(const chf_ham* H) {
    return std::is_same<T, double>::value ? H->ent_beta64.as<T>() : H->ent_beta32.as<T>();
}

template <class T>
void launch_hx_generic(chf_ham* H, const T* X, int64_t ldx, T* Y, int64_t ldy, const T* Z, int64_t ldz, int nvec,
                       const T* C, double alpha, double shift, double beta, hipStream_t s, bool lap_only) {
    const int nvc = (nvec + 3) / 4;
    // (a launch holds fewer than 2^32 threads: runs of rows of at most half of that)
    const int64_t n = H->grid.n_rows, run = std::max<int64_t>(1, (int64_t(1) << 31) / nvc);
    for (int64_t row0 = 0; row0 < n; row0 += run) {
        const int64_t end = std::min(n, row0 + run), total = (end - row0) * nvc;
        hx_generic_kernel<T><<<dim3(unsigned((total + 255) / 256)), dim3(256), 0, s>>>(
            row0, end, nvec, nvc, H->nbr_rows.as<int32_t>(), H->row_inside.as<uint8_t>(),
            lap_only ? nullptr : veff_of<T>(H), lap_only ? nullptr : H->ent_off.as<int64_t>(),
            H->ent_atom.as<int32_t>(), ent_beta_of<T>(H), C, X, ldx, Y, ldy, Z, ldz,
            make_coef<T>(H, alpha, shift, beta));
        LAUNCH_CHECK();
    }
}

// ---------------------------------------------------------------------------
// KB gather: C[a][lm][v] = sum_j (h^3 beta_alm(row_j)) X[row_j][v]
//
// One workgroup per (projector atom, chunk of QL pieces of QN vectors).  The
// support's rows are dealt to kSlots row slots (row j to slot j mod kSlots);
// each slot sums its rows in order and the slots are added as a binary tree,
// lowest slot bit first: over the RL = 64 / QL row lanes of a wave, then over
// the WV = kSlots / RL waves.  So the sums do not depend on how a width is
// spread over lanes: a vector's coefficients are the same bits in a block of
// any width, and on every run.
//
// What bounds it: the re-reads of the support rows (~1,350 per atom, each row
// in ~2.9 supports).  Chunks of 256 bytes keep the rows that the atoms in
// flight on an XCD share in its 4 MB L2; the chunks run one after the other.
// Against one workgroup of 4 waves per 1024-byte chunk, which also left a wave
// 338 rows in series (us per launch, before -> now): 5 nm, 256 FP32 vectors
// 690 -> 582 (7.6 TB/s of rows); 2.5 nm 219 -> 84; 5 nm, 128 FP64 870 -> 704;
// 1.1 nm, 128 FP64 191 -> 24; 3 nm, 2 FP64 161 -> 20.  Chunks of 512 bytes
// took 817 us at 5 nm FP32, of 128 bytes 614.
// ---------------------------------------------------------------------------
constexpr int kSlots = 64;

template <class T, int QN>
struct alignas(sizeof(T) * QN) Piece {
    T e[QN];
};

template <class T, int QN, int QL>
__global__ void __launch_bounds__(kSlots * QL) kb_gather_kernel(const int64_t* __restrict__ sup_off,
                                                                const int32_t* __restrict__ sup_row,
                                                                const T* __restrict__ sup_beta,
                                                                const T* __restrict__ X, int64_t ldx, int nvec,
                                                                T* __restrict__ C, int n_proj) {
    using V = Piece<T, QN>;
    using B4 = Piece<T, 4>;
    constexpr int RL = 64 / QL, WV = kSlots / RL;
    // rows of a slot loaded together: 4, or 2 where the FP64 operands of 4
    // would halve the waves that the registers allow (886 against 704 us at 5 nm)
    constexpr int DEEP = sizeof(T) == 8 && QL >= 16 ? 2 : 4;
    __shared__ V part[WV][4][QL];
    // XCD-aware order (grid = 8 * per_xcd): consecutive atoms, which share
    // support rows (the device numbers atoms along the Hilbert curve), run on
    // the same XCD and read the shared rows from its L2
    const int per_xcd = int(gridDim.x / 8);
    const int a = int(blockIdx.x % 8) * per_xcd + int(blockIdx.x / 8);
    if (a >= n_proj) return;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int q = lane % QL;
    const int v = (int(blockIdx.y) * QL + q) * QN;
    const bool ok = v < nvec;
    const int64_t j0 = sup_off[a], j1 = sup_off[a + 1];
    const B4* beta = reinterpret_cast<const B4*>(sup_beta);
    V s[4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int e = 0; e < QN; ++e) s[m].e[e] = T(0);
    auto row = [&](int64_t j) {
        V x;
#pragma unroll
        for (int e = 0; e < QN; ++e) x.e[e] = T(0);
        if (ok) x = *reinterpret_cast<const V*>(X + int64_t(sup_row[j]) * ldx + v);
        return x;
    };
    auto add = [&](const B4& b, const V& x) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int e = 0; e < QN; ++e) s[m].e[e] = fma(b.e[m], x.e[e], s[m].e[e]);
    };
    // slot wave RL + row lane: the rows that a wave loads together are
    // consecutive, and so are their indices and weights
    int64_t j = j0 + wave * RL + lane / QL;
    for (; j + (DEEP - 1) * kSlots < j1; j += DEEP * kSlots) {
        V x[DEEP];
        B4 b[DEEP];
#pragma unroll
        for (int d = 0; d < DEEP; ++d) {
            x[d] = row(j + d * kSlots);
            b[d] = beta[j + d * kSlots];
        }
#pragma unroll
        for (int d = 0; d < DEEP; ++d) add(b[d], x[d]);
    }
    for (; j < j1; j += kSlots) add(beta[j], row(j));
#pragma unroll
    for (int off = QL; off < 64; off *= 2)
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int e = 0; e < QN; ++e) s[m].e[e] += __shfl_xor(s[m].e[e], off, 64);
    if (lane < QL)
#pragma unroll
        for (int m = 0; m < 4; ++m) part[wave][m][q] = s[m];
    __syncthreads();
    for (int t = threadIdx.x; t < 4 * QL; t += 64 * WV) {
        const int lm = t / QL, qq = t % QL;
        const int vv = (int(blockIdx.y) * QL + qq) * QN;
        if (vv >= nvec) continue;
        V r[WV];
#pragma unroll
        for (int w = 0; w < WV; ++w) r[w] = part[w][lm][qq];
#pragma unroll
        for (int h = 1; h < WV; h *= 2)
#pragma unroll
            for (int w = 0; w < WV; w += 2 * h)
#pragma unroll
                for (int e = 0; e < QN; ++e) r[w].e[e] += r[w + h].e[e];
        *reinterpret_cast<V*>(C + (int64_t(a) * 4 + lm) * nvec + vv) = r[0];
    }
}

template <class T, int QN>
static void gather_launch(chf_ham* H, const T* beta, const T* X, int64_t ldx, int nvec, T* C, hipStream_t s) {
    const int n = int(H->proj.n_proj), pieces = nvec / QN;
    int ql = 16;
    while (ql > 1 && ql / 2 >= pieces) ql /= 2;
    const dim3 grid(unsigned(8 * ((n + 7) / 8)), unsigned((pieces + ql - 1) / ql));
    auto go = [&](auto qlc) {
        constexpr int QL = decltype(qlc)::value;
        kb_gather_kernel<T, QN, QL><<<grid, dim3(kSlots * QL), 0, s>>>(
            H->sup_off.as<int64_t>(), H->sup_row.as<int32_t>(), beta, X, ldx, nvec, C, n);
    };
    if (ql == 16) go(std::integral_constant<int, 16>{});
    else if (ql == 8) go(std::integral_constant<int, 8>{});
    else if (ql == 4) go(std::integral_constant<int, 4>{});
    else if (ql == 2) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 1>{});
    LAUNCH_CHECK();
}

// pieces of 16 bytes where the width, the leading dimension and the base
// address allow, else of 8 (FP32), else single elements
template <class T>
void launch_kb_gather(chf_ham* H, const T* X, int64_t ldx, int nvec, T* C, hipStream_t s) {
    if (H->proj.n_proj == 0) return;
    constexpr int Q16 = 16 / int(sizeof(T));
    const T* beta = std::is_same<T, double>::value ? H->sup_beta64.as<T>() : H->sup_beta32.as<T>();
    const auto fits = [&](int qn) { return nvec % qn == 0 && ldx % qn == 0 && uintptr_t(X) % (qn * sizeof(T)) == 0; };
    if (fits(Q16)) gather_launch<T, Q16>(H, beta, X, ldx, nvec, C, s);
    else if (Q16 == 4 && fits(2)) gather_launch<T, 2>(H, beta, X, ldx, nvec, C, s);
    else gather_launch<T, 1>(H, beta, X, ldx, nvec, C, s);
}

// 8-byte lane values of the tiled kernel: two floats or one double
template <class T>
struct Lane;
template <>
struct Lane<float> {
    using V = float2;
    static constexpr int N = 2;
};
template <>
struct Lane<double> {
    using V = double;
    static constexpr int N = 1;
};
__device__ inline void lzero(float2& v) { v = make_float2(0.f, 0.f); }
__device__ inline void lzero(double& v) { v = 0.0; }
__device__ inline float2 lfma(float s, float2 a, float2 c) { return make_float2(fmaf(s, a.x, c.x), fmaf(s, a.y, c.y)); }
__device__ inline double lfma(double s, double a, double c) { return fma(s, a, c); }
__device__ inline float2 ladd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ inline double ladd(double a, double b) { return a + b; }
__device__ inline float2 lscale(float s, float2 a) { return make_float2(s * a.x, s * a.y); }
__device__ inline double lscale(double s, double a) { return s * a; }

template <class V>
__device__ inline V lz() {
    V v;
    lzero(v);
    return v;
}

// raw buffer access (vector memory through a 128-bit resource descriptor)
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, int(bytes), 0x00020000);
}
template <class V>
__device__ inline V bload(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
template <class V>
__device__ inline void bstore(V v, __amdgpu_buffer_rsrc_t r, unsigned off) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, 0);
}

// Unstaged tile kernel: one workgroup per tile (one 8^3 block x one 128-byte
// vector chunk), 1024 threads = 64 columns (x, y) x 16 lanes; a lane holds 8
// bytes (2 floats or 1 double) of the chunk.  It serves the Hamiltonians that the
// staged tile kernel below does not take: with a block touched by more than
// kMaxBlockAtoms projector atoms, and without projectors.  Each thread keeps
// X(x, y, z-6 .. z+13) of its column and lane in registers and marches z = 0..7; the
// x/y neighbours of plane z (the plane and its 6-deep halos from the -x/+x/-y/+y
// blocks) are staged in LDS as a 20 x 20 square, double-buffered so that one
// barrier per plane suffices.  The eight output rows wait in registers, and the KB
// term is added after the march from the coefficients in global memory.  Rows
// outside the sphere are stored as zero; on input they must hold zero (the layout
// contract), so they enter the stencil as the zero boundary.
constexpr int kMaxBlockAtoms = 64;
constexpr int kLanes = 16;

template <class T>
__global__ void __launch_bounds__(64 * kLanes) hx_tiled_kernel(int64_t n_blocks, int n_chunks, const int32_t* __restrict__ bnb,
                                                         const uint64_t* __restrict__ bmask, const T* __restrict__ veff,
                                                         const int32_t* __restrict__ ent_off,
                                                         const int32_t* __restrict__ ent_atom,
                                                         const T* __restrict__ ent_beta, const T* __restrict__ C,
                                                         int nvec, const T* __restrict__ X, int64_t ldx, T* Y,
                                                         int64_t ldy, const T* Z, int64_t ldz, StepCoef<T> k) {
    using V = typename Lane<T>::V;
    constexpr int LANES = kLanes;
    constexpr int LN = Lane<T>::N;       // elements per lane
    constexpr int CH = LANES * LN;       // vectors per chunk
    constexpr int LSH = 4;
    constexpr int CPW = 64 / LANES;      // columns per wave
    // LDS plane: the full 20 x 20 square x in [-6, 14), y in [-6, 14) (corners
    // unused) so every neighbour is a constant offset from the centre
    __shared__ V plane[2][400][LANES];

    // XCD-aware tile order: workgroup ids are dealt round-robin to the 8
    // XCDs; give each XCD a contiguous run of the tile sequence (blocks in
    // Hilbert order, the vector chunks of a block adjacent) so that
    // neighbouring blocks share its L2 and the chunks of a block share the
    // block's tables (KB entries, V_eff, masks).
    const int64_t ntiles = n_blocks * n_chunks;
    const int64_t per_xcd = (ntiles + 7) / 8;
    const int64_t tile = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (tile >= ntiles) return;

    const int t = threadIdx.x;
    const int p = t & (LANES - 1);       // lane within the chunk
    const int col = t >> LSH;            // column 0..63
    const int cx = col & 7, cy = col >> 3;
    const int wave = t >> 6;
    const unsigned es = sizeof(T);
    const unsigned blk_bytes = unsigned(kBlockPts) * unsigned(ldx) * es;
    constexpr unsigned kOOB = 0x80000000u;
    const unsigned plane_x = 64u * unsigned(ldx) * es;
    const unsigned plane_z = 64u * unsigned(ldz) * es;
    const unsigned plane_y = 64u * unsigned(ldy) * es;
    const int ctr = (cy + 6) * 20 + (cx + 6);
    auto res_x = [&](int32_t nb) {
        return make_rsrc(nb >= 0 ? X + int64_t(nb) * kBlockPts * ldx : X, nb >= 0 ? blk_bytes : 0u);
    };

    const int64_t blk = tile / n_chunks;
    const int chunk = int(tile - blk * n_chunks);
    int32_t nbs[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) nbs[f] = bnb[6 * blk + f];
    const int vbase = chunk * CH + p * LN;
    const bool vok = vbase < nvec;
    const unsigned off_x = vok ? (unsigned(cx + 8 * cy) * unsigned(ldx) + unsigned(vbase)) * es : kOOB;
    const unsigned off_z = vok ? (unsigned(cx + 8 * cy) * unsigned(ldz) + unsigned(vbase)) * es : kOOB;
    const __amdgpu_buffer_rsrc_t rOwn = res_x(int32_t(blk));
    const __amdgpu_buffer_rsrc_t rZm = res_x(nbs[4]);
    const __amdgpu_buffer_rsrc_t rZp = res_x(nbs[5]);
    const __amdgpu_buffer_rsrc_t rZ =
        make_rsrc(Z ? Z + blk * kBlockPts * ldz : X, Z ? unsigned(kBlockPts) * unsigned(ldz) * es : 0u);
    // Halo slot u of a wave covers CPW consecutive halo rows, all on one side
    // of the block (48 rows per side), so the side is wave-uniform.
    int hrow[3];
    __amdgpu_buffer_rsrc_t rH[3];
    unsigned hoff[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        const int hr0 = CPW * wave + 64 * u;
        const int side = __builtin_amdgcn_readfirstlane(hr0 / 48);
        const int hr = col + 64 * u;
        const int rem = hr - 48 * side;
        int lx, ly, x, y, nb;
        if (side < 2) {
            const int c6 = rem % 6;
            ly = rem / 6;
            lx = side == 0 ? 2 + c6 : c6;
            x = side == 0 ? c6 - 6 : 8 + c6;
            y = ly;
            nb = side == 0 ? nbs[0] : nbs[1];
        } else {
            const int r6 = rem / 8;
            lx = rem % 8;
            ly = side == 2 ? 2 + r6 : r6;
            x = lx;
            y = side == 2 ? r6 - 6 : 8 + r6;
            nb = side == 2 ? nbs[2] : nbs[3];
        }
        hrow[u] = (y + 6) * 20 + (x + 6);
        rH[u] = res_x(__builtin_amdgcn_readfirstlane(nb));
        hoff[u] = vok ? (unsigned(lx + 8 * ly) * unsigned(ldx) + unsigned(vbase)) * es : kOOB;
    }
    auto load_plane = [&](int zz) -> V {
        if (zz < 0) return bload<V>(rZm, off_x + unsigned(zz + 8) * plane_x);
        if (zz >= 8) return bload<V>(rZp, off_x + unsigned(zz - 8) * plane_x);
        return bload<V>(rOwn, off_x + unsigned(zz) * plane_x);
    };
    auto load_halo = [&](int z, V* hv) {
#pragma unroll
        for (int u = 0; u < 3; ++u) hv[u] = bload<V>(rH[u], hoff[u] + unsigned(z) * plane_x);
    };
    auto store_halo = [&](int b, const V* hv) {
#pragma unroll
        for (int u = 0; u < 3; ++u) plane[b][hrow[u]][p] = hv[u];
    };
    auto load_z = [&](int z) -> V { return bload<V>(rZ, off_z + unsigned(z) * plane_z); };

    const int64_t base = blk * kBlockPts;
    const int lrow = cx + 8 * cy;             // this column's row in plane 0
    // the X window of this column, the first two halo planes and Y_{k-1} of
    // plane 0
    V w[20];
#pragma unroll
    for (int i = 0; i < 14; ++i) w[i] = load_plane(i - 6);
    V hv0[3], hv[3];
    load_halo(0, hv0);
    load_halo(1, hv);
    V zcur = load_z(0);
    store_halo(0, hv0);
    plane[0][ctr][p] = w[6];
    __syncthreads();

    const __amdgpu_buffer_rsrc_t rY = make_rsrc(Y + base * ldy, unsigned(kBlockPts) * unsigned(ldy) * es);
    const unsigned off_y = vok ? (unsigned(lrow) * unsigned(ldy) + unsigned(vbase)) * es : kOOB;
    V r[8];
    const T* vr = veff + base;
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        const int b = z & 1;
        // stage plane z + 1 (its loads were issued one plane ago), then
        // issue the loads for planes further ahead
        if (z < 7) {
            store_halo(b ^ 1, hv);
            plane[b ^ 1][ctr][p] = w[z + 7];
        }
        if (z < 6) load_halo(z + 2, hv);
        V znext = lz<V>();
        if (z < 7) znext = load_z(z + 1);
        if (z < 6) w[z + 14] = load_plane(z + 8);

        // unscaled stencil (c_0 x + sum_s c_s (six neighbours at distance s))
        V acc = lscale(k.c[0], w[z + 6]);
#pragma unroll
        for (int s = 1; s <= 6; ++s) {
            V sum = ladd(w[z + 6 - s], w[z + 6 + s]);
            sum = ladd(sum, plane[b][ctr - s][p]);
            sum = ladd(sum, plane[b][ctr + s][p]);
            sum = ladd(sum, plane[b][ctr - 20 * s][p]);
            sum = ladd(sum, plane[b][ctr + 20 * s][p]);
            acc = lfma(k.c[s], sum, acc);
        }
        const V xc = w[z + 6];
        acc = lfma(vr[lrow + 64 * z], xc, acc);
        V y = lscale(k.alpha, lfma(-k.shift, xc, acc));
        if (Z) y = lfma(-k.beta, zcur, y);
        r[z] = y;
        zcur = znext;
        __syncthreads();
    }

    // KB scatter after the march, in rounds so that the entry loads of all
    // eight rows are in flight together
    if (ent_off && vok) {
        int e0[8], e1[8];
        int nmax = 0;
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            const int64_t row = base + lrow + 64 * z;
            e0[z] = ent_off[row];
            e1[z] = ent_off[row + 1];
            nmax = max(nmax, e1[z] - e0[z]);
        }
        for (int j = 0; j < nmax; ++j) {
#pragma unroll
            for (int z = 0; z < 8; ++z) {
                const int en = e0[z] + j;
                if (en < e1[z]) {
                    const T* bb = ent_beta + 4 * int64_t(en);
                    const T* ca = C + int64_t(ent_atom[en]) * 4 * int64_t(nvec) + vbase;
                    V acc = lscale(bb[0], *reinterpret_cast<const V*>(ca));
                    acc = lfma(bb[1], *reinterpret_cast<const V*>(ca + nvec), acc);
                    acc = lfma(bb[2], *reinterpret_cast<const V*>(ca + 2 * nvec), acc);
                    acc = lfma(bb[3], *reinterpret_cast<const V*>(ca + 3 * nvec), acc);
                    r[z] = lfma(k.alpha, acc, r[z]);
                }
            }
        }
    }
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        const bool in = (bmask[8 * blk + z] >> lrow) & 1;
        bstore<V>(in ? r[z] : lz<V>(), rY, off_y + unsigned(z) * plane_y);
    }
}

// ---------------------------------------------------------------------------
// Staged tile kernel: the Hilbert-blocked H X + recurrence with the KB term
// from coefficients staged in LDS (blocks touched by at most kMaxBlockAtoms
// projector atoms).  One workgroup per (8^3 block, 128-byte vector chunk), 512
// threads = 64 columns x 8 lanes of 16 bytes; a wave is one x line (8 columns)
// of the block's plane.  Per plane of the z-march: the x/y neighbours come
// from the plane and its 6-deep halos in LDS (a 20 x 20 square), the z
// neighbours from the column's register window.
//
// KB term of a plane: out[row][vec] += sum over slots and channels of
// beta[row][slot][lm] C[slot][lm][vec], a matrix product.  Rows are taken in
// groups of 16 (two x lines); for each atom that touches a group a 16 x 4
// matrix of weights (zero outside the support) is kept in memory in operand
// order, the 4 x 16 coefficients are read from LDS, and one 16x16x4 MFMA (FP32
// or FP64, full precision) adds the atom.  The product is transposed (rows of
// the result = vectors), so a lane ends up with 4 vectors of one row; it goes
// through LDS to the lanes that hold that row.  Coefficients that are Inf or NaN
// would reach rows through zero weights; they are kept out of the products and
// added entry by entry after the march (5 nm, 256 FP32 vectors of which all are Inf
// or NaN: 2.4 -> 8.8 ms; others: no change).
//
// The plane is single-buffered (two barriers per plane), which keeps a
// workgroup within half of the 160 KB of LDS and its threads within 128
// registers: two workgroups run on a CU, one marching while the other loads.
//
// What bounds it: the traffic behind the L2 (14.3 GB per 5 nm FP32 launch in 2.36
// ms = 6.1 TB/s, twice the two blocks read and the one written, for the halos; the
// same rate for FP64) and the latency of a plane.  One 1024-thread workgroup per CU,
// whose KB term was applied entry by entry on the VALU, took 21.9 us per tile at
// every size, 7.8 of them before the first plane; now 15.4.  us per launch,
// before -> now: 5 nm, 256 FP32 vectors 3337 -> 2360; 5 nm, 128 FP64 3389 -> 2561;
// 3 nm, 128 FP64 1011 -> 751; 2.5 nm, 256 FP32 674 -> 476; 1.1 nm, 128 FP64
// 154 -> 102; 2 nm, 97 FP64 (rows on 8 bytes) 470 -> 343, 474 with every 16 bytes in
// two pieces of 8.
// PB: what a row starts on and is a multiple of, 128 bytes (cache lines), 16 or 8.
// ---------------------------------------------------------------------------
constexpr int kSlotBytes = 512;      // staged coefficients of an atom: 4 channels x 128 bytes
constexpr int kRowGroup = 16;        // rows of a KB weight matrix
constexpr int kGroups = kBlockPts / kRowGroup;
constexpr int kKbStep = 4;           // a group's atom list is padded to this multiple
constexpr int kKbAhead = 2 * kKbStep;  // entries of a plane whose weights are fetched ahead
// slots of the half-LDS variant (the 1.1 to 5 nm Si clusters have at most 23 atoms to
// a block); a Hamiltonian with a block touched by more takes the one with
// kMaxBlockAtoms slots, one workgroup per CU.  An H X with up to 56 atoms to a block
// (256 Si in a sphere of 18 bohr), one 1024-thread workgroup that adds entry by entry
// -> this variant: 128 FP64 vectors 287 -> 208 us, 97 323 -> 207, 16 153 -> 43, 256
// FP32 292 -> 190; with up to 37 atoms (203 Si), two workgroups: 284 -> 156, 321 ->
// 159, 153 -> 38, 287 -> 146.
constexpr int kFewSlots = 40;
// a row's 16-byte pieces lie kKbPitch apart in the KB plane: 16 rows and 32
// bytes, so that the 8 pieces of two rows fall on different banks
constexpr int kKbPitch = 16 * 16 + 32;
constexpr int kKbBytes = (kBlockPts / 8) / kRowGroup * 8 * kKbPitch;
constexpr int kPlaneBytes = 400 * 128;

typedef float mf4 __attribute__((ext_vector_type(4)));
typedef double md4 __attribute__((ext_vector_type(4)));
template <class T>
struct Wide;
template <>
struct Wide<float> {
    static constexpr int N = 4;
    using A = mf4;
};
template <>
struct Wide<double> {
    static constexpr int N = 2;
    using A = md4;
};
__device__ inline mf4 mfma4(float a, float b, mf4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ inline md4 mfma4(double a, double b, md4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes from any multiple of 4.  policy 2 = non-temporal: Y_{k-1} is read and
// Y_{k+1} written once per launch, so they should not displace the X rows that
// neighbouring tiles read again as halos (5 nm, 256 FP32: 2481 -> 2361 us with the
// reads so, 2429 without the writes so).  Not where two chunks share a cache line,
// which would be fetched twice (2 nm, 97 FP64: 377 against 343 us; 1.1 nm, 33 FP64
// 62 against 41).
template <class V, int POLICY>
__device__ inline V bload16(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, voff, int(soff), POLICY));
}

// tables that the tile kernel needs only for coefficients that are Inf or NaN
template <class T>
struct TileRare {
    const int32_t *ent_off, *ent_soff, *blk_atom_off, *blk_atoms;
    const T* ent_beta;
};

template <class T, int PB, int SLOTS>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(SLOTS <= kFewSlots ? 4 : 2)))
hx_tile_kernel(int n_blocks, int n_chunks, int group, const int32_t* __restrict__ bnb, const uint64_t* __restrict__ bmask,
               const T* __restrict__ veff, const int32_t* __restrict__ rg_off, const int32_t* __restrict__ rg_slot,
               const T* __restrict__ rg_beta, const int32_t* __restrict__ blk_atom_off,
               const int32_t* __restrict__ blk_atoms, const T* __restrict__ C, int nvec, const T* __restrict__ X,
               int64_t ldx, T* Y, int64_t ldy, const T* Z, int64_t ldz, const TileRare<T>* rare, StepCoef<T> k) {
    constexpr int N = Wide<T>::N;
    using V = Piece<T, N>;
    using A = typename Wide<T>::A;
    constexpr int CH = 8 * N;                 // vectors of a chunk
    constexpr bool f32 = sizeof(T) == 4;
    __shared__ __align__(16) char lds[SLOTS * kSlotBytes + kPlaneBytes + kKbBytes];
    __shared__ int odd[8];                    // whether a wave staged a coefficient that is Inf or NaN
    char* const lds_kb = lds + SLOTS * kSlotBytes;
    V (*plane)[8] = reinterpret_cast<V (*)[8]>(lds + SLOTS * kSlotBytes + kKbBytes);

    // XCD-aware tile order: workgroup ids are dealt round-robin to the 8 XCDs; an
    // XCD takes a contiguous run of blocks, `group` chunks of all of them after the
    // other: fewer chunks at a time leave more neighbouring blocks, whose halos
    // overlap, in its L2, more share a block's tables and whole cache lines.
    const unsigned per_xcd = (unsigned(n_blocks) + 7) / 8;
    const unsigned id = blockIdx.x / 8, first = id / (per_xcd * group) * group;
    const unsigned wide = min(unsigned(group), unsigned(n_chunks) - first), rest = id - per_xcd * first;
    const int blk = int(blockIdx.x % 8 * per_xcd + rest / wide), chunk = int(first + rest % wide);
    if (rest >= per_xcd * wide || blk >= n_blocks) return;

    const int t = threadIdx.x;
    const int p = t & 7;
    const int col = t >> 3;
    const int cx = col & 7;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);   // = the y line of this wave's columns
    const int lane = t & 63;
    constexpr unsigned es = sizeof(T);
    constexpr unsigned kOOB = 0x80000000u;
    // bytes of a block from its first to its last vector.  The last 16 bytes of a
    // ragged row's last lane may reach past the row (PB 8), of the block's last row
    // past this; the range that holds for certain is that of the vector offset, so
    // the last plane's offset is added to it.
    auto blk_bytes = [&](int64_t ld) { return (unsigned(kBlockPts - 1) * unsigned(ld) + unsigned(nvec)) * es; };
    const unsigned plane_x = 64u * unsigned(ldx) * es;
    const unsigned plane_z = 64u * unsigned(ldz) * es;
    const unsigned plane_y = 64u * unsigned(ldy) * es;
    const int ctr = (wave + 6) * 20 + (cx + 6);
    auto res_x = [&](int32_t nb) {
        return make_rsrc(nb >= 0 ? X + int64_t(nb) * kBlockPts * ldx : X, nb >= 0 ? blk_bytes(ldx) : 0u);
    };
    int32_t nbs[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) nbs[f] = bnb[6 * int64_t(blk) + f];
    const int vbase = chunk * CH + p * N;
    const bool vok = vbase < nvec;
    const unsigned vbytes = unsigned(vbase) * es;
    const unsigned off_x = vok ? unsigned(col) * unsigned(ldx) * es + vbytes : kOOB;
    const unsigned off_z = vok ? unsigned(col) * unsigned(ldz) * es + vbytes : kOOB;
    const unsigned off_y = vok ? unsigned(col) * unsigned(ldy) * es + vbytes : kOOB;
    const __amdgpu_buffer_rsrc_t rOwn = res_x(blk);
    const __amdgpu_buffer_rsrc_t rZm = res_x(nbs[4]);
    const __amdgpu_buffer_rsrc_t rZp = res_x(nbs[5]);
    const __amdgpu_buffer_rsrc_t rZ =
        make_rsrc(Z ? Z + int64_t(blk) * kBlockPts * ldz : X, Z ? blk_bytes(ldz) : 0u);
    const __amdgpu_buffer_rsrc_t rY = make_rsrc(Y + int64_t(blk) * kBlockPts * ldy, blk_bytes(ldy));
    // halo slot u of a wave: 8 consecutive halo rows, all on one side (48 rows
    // per side)
    int hrow[3];
    __amdgpu_buffer_rsrc_t rH[3];
    unsigned hoff[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        const int side = (8 * wave + 64 * u) / 48;
        const int rem = col + 64 * u - 48 * side;
        int lx, ly, x, y;
        if (side < 2) {
            const int c6 = rem % 6;
            ly = rem / 6;
            lx = side == 0 ? 2 + c6 : c6;
            x = side == 0 ? c6 - 6 : 8 + c6;
            y = ly;
        } else {
            const int r6 = rem / 8;
            lx = rem % 8;
            ly = side == 2 ? 2 + r6 : r6;
            x = lx;
            y = side == 2 ? r6 - 6 : 8 + r6;
        }
        hrow[u] = (y + 6) * 20 + (x + 6);
        rH[u] = res_x(side == 0 ? nbs[0] : side == 1 ? nbs[1] : side == 2 ? nbs[2] : nbs[3]);
        hoff[u] = vok ? unsigned(lx + 8 * ly) * unsigned(ldx) * es + vbytes : kOOB;
    }
    auto load = [](auto policy, __amdgpu_buffer_rsrc_t r, unsigned off, int z, unsigned plane) -> V {
        constexpr int P = decltype(policy)::value;
        const unsigned o = unsigned(z) * plane;
        return PB == 8 && z == 7 ? bload16<V, P>(r, off + o, 0) : bload16<V, P>(r, off, o);
    };
    constexpr std::integral_constant<int, 0> often;
    constexpr std::integral_constant<int, PB == 128 ? 2 : 0> once;
    auto load_plane = [&](int zz) -> V {
        return load(often, zz < 0 ? rZm : zz >= 8 ? rZp : rOwn, off_x, zz & 7, plane_x);
    };

    // the X window of this column, the halos of plane 0, Y_{k-1} and V_eff
    V w[20], hv[3];
#pragma unroll
    for (int i = 0; i < 13; ++i) w[i] = load_plane(i - 6);
#pragma unroll
    for (int u = 0; u < 3; ++u) hv[u] = load(often, rH[u], hoff[u], 0, plane_x);

    // KB coefficients of the block's atoms, alpha applied: 16 slots a round.  One that
    // is Inf or NaN is staged as zero, since the zero weights of the rows outside its
    // atom's support would make it NaN there; its own rows get it at the end.
    const int a0 = blk_atom_off[blk];
    const int na = min(blk_atom_off[blk + 1] - a0, SLOTS);
    bool bad = false;
    for (int sl = t >> 5; sl < na; sl += 16) {
        const int lm = (t >> 3) & 3;
        const T* src = C + (int64_t(blk_atoms[a0 + sl]) * 4 + lm) * nvec + vbase;
        V c;
#pragma unroll
        for (int e = 0; e < N; ++e) c.e[e] = T(0);
        if constexpr (PB >= 16) {
            if (vok) c = *reinterpret_cast<const V*>(src);
        } else {
#pragma unroll
            for (int e = 0; e < N; ++e)
                if (vbase + e < nvec) c.e[e] = src[e];
        }
#pragma unroll
        for (int e = 0; e < N; ++e) {
            c.e[e] *= k.alpha;
            if (!isfinite(c.e[e])) {
                c.e[e] = T(0);
                bad = true;
            }
        }
        *reinterpret_cast<V*>(lds + sl * kSlotBytes + lm * 128 + p * 16) = c;
    }
    bad = __any(bad);
    if (lane == 0) odd[wave] = bad;
    auto stage = [&](int z) {
#pragma unroll
        for (int u = 0; u < 3; ++u) plane[hrow[u]][p] = hv[u];
        plane[ctr][p] = w[z + 6];
    };
    stage(0);

    // KB product of a plane.  FP32: 4 row groups x 2 halves of the chunk, one
    // for each wave.  FP64: 4 row groups, taken by waves 0-3 for even planes
    // and 4-7 for odd ones.
    const int grp = f32 ? wave >> 1 : wave & 3;
    const int lk = lane >> 4, li = lane & 15;
    // operand A of a slot: coefficient lm = lk of result row li, which is
    // vector li of the half (FP32), or 4 (li % 4) + li / 4 (FP64, so that a
    // lane's four result rows are consecutive vectors)
    const int a_off = lk * 128 + (f32 ? (wave & 1) * 64 + li * 4 : (4 * (li & 3) + (li >> 2)) * 8);
    auto kb_mine = [&](int z) { return f32 || (wave >> 2) == (z & 1); };
    // this wave's entries, plane after plane (one row group's 8 planes are
    // consecutive): the weights of the first kKbAhead entries of a plane are
    // fetched ahead (kb_fetch), while the plane before it is worked on, also where
    // its list is shorter; behind the last list lie as many that nothing uses
    int e_off[9];
    const int64_t rg0 = int64_t(blk) * kGroups + grp * 8;
#pragma unroll
    for (int z = 0; z < 9; ++z) e_off[z] = rg_off[rg0 + z];
    const __amdgpu_buffer_rsrc_t rW =
        make_rsrc(rg_beta + int64_t(e_off[0]) * 64, unsigned(e_off[8] - e_off[0]) * 64u * es);
    T kb_b[kKbAhead];
    auto weight = [&](int e) {
        const unsigned o = unsigned(e - e_off[0]) * 64u * es;
        if constexpr (f32) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rW, unsigned(lane) * es, int(o), 0));
        else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rW, unsigned(lane) * es, int(o), 0));
    };
    auto kb_fetch = [&](int z, int part) {
        if (!kb_mine(z)) return;
#pragma unroll
        for (int u = part * kKbStep; u < (part + 1) * kKbStep; ++u) kb_b[u] = weight(e_off[z] + u);
    };
    auto kb_step = [&](A acc, int e, const T* b) {
        T a[kKbStep];
#pragma unroll
        for (int u = 0; u < kKbStep; ++u) a[u] = *reinterpret_cast<const T*>(lds + rg_slot[e + u] + a_off);
#pragma unroll
        for (int u = 0; u < kKbStep; ++u) acc = mfma4(a[u], b[u], acc);
        return acc;
    };
    auto kb_plane = [&](int z) {
        A acc = {0, 0, 0, 0};
        if (!kb_mine(z)) return acc;
        const int e0 = e_off[z], e1 = e_off[z + 1];
        if (e0 < e1) acc = kb_step(acc, e0, kb_b);
        if (e0 + kKbStep < e1) acc = kb_step(acc, e0 + kKbStep, kb_b + kKbStep);
        for (int e = e0 + kKbAhead; e < e1; e += kKbStep) {
            T b[kKbStep];
#pragma unroll
            for (int u = 0; u < kKbStep; ++u) b[u] = weight(e + u);
            acc = kb_step(acc, e, b);
        }
        return acc;
    };
    // row li of the group, pieces lk (FP32: of this half) or 2 lk, 2 lk + 1
    char* const kb_w = lds_kb + (grp * 8 + (f32 ? (wave & 1) * 4 + lk : 2 * lk)) * kKbPitch + li * 16;
    auto kb_store = [&](int z, A acc) {
        if (!kb_mine(z)) return;
        if constexpr (f32) {
            *reinterpret_cast<A*>(kb_w) = acc;
        } else {
            *reinterpret_cast<V*>(kb_w) = V{{acc[0], acc[1]}};
            *reinterpret_cast<V*>(kb_w + kKbPitch) = V{{acc[2], acc[3]}};
        }
    };
    const char* const kb_r = lds_kb + ((col >> 4) * 8 + p) * kKbPitch + (col & 15) * 16;
    kb_fetch(0, 0);
    __syncthreads();
    kb_fetch(0, 1);
    kb_store(0, kb_plane(0));
    __syncthreads();

    const int64_t base = int64_t(blk) * kBlockPts;
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        // loads of this plane's update and of the next plane
        const V zc = load(once, rZ, off_z, z, plane_z);   // zero without Z (empty buffer)
        const T vr = veff[base + col + 64 * z];
        if (z < 7) {
#pragma unroll
            for (int u = 0; u < 3; ++u) hv[u] = load(often, rH[u], hoff[u], z + 1, plane_x);
            w[z + 13] = load_plane(z + 7);
        }

        // alpha-scaled off-diagonal stencil; the diagonal is added last
        V acc = *reinterpret_cast<const V*>(kb_r);
#pragma unroll
        for (int s = 1; s <= 6; ++s) {
            const V xm = plane[ctr - s][p], xp = plane[ctr + s][p], ym = plane[ctr - 20 * s][p],
                    yp = plane[ctr + 20 * s][p];
#pragma unroll
            for (int e = 0; e < N; ++e) {
                T sum = w[z + 6 - s].e[e] + w[z + 6 + s].e[e];
                sum += xm.e[e];
                sum += xp.e[e];
                sum += ym.e[e];
                sum += yp.e[e];
                acc.e[e] = fma(k.ac[s], sum, acc.e[e]);
            }
        }
        const T dg = fma(k.alpha, vr, k.d0);
        // rows outside the sphere are stored as zero
        const bool in = (unsigned(bmask[8 * int64_t(blk) + z] >> (8 * wave)) >> cx) & 1u;
        V y;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const T v = fma(-k.beta, zc.e[e], fma(dg, w[z + 6].e[e], acc.e[e]));   // beta = 0 without Z
            y.e[e] = in ? v : T(0);
        }
        // The plane's offset is part of the vector offset: a 128-bit store with
        // a scalar offset register was seen to lose its last dword when the
        // next instruction overwrites the data register; the compiler keeps
        // that distance only for stores without one.
        const u32x4 yb = __builtin_bit_cast(u32x4, y);
        const unsigned oy = off_y + unsigned(z) * plane_y;
        if constexpr (PB >= 16) {
            __builtin_amdgcn_raw_buffer_store_b128(yb, rY, oy, 0, PB == 128 ? 2 : 0);
        } else {
            // a row's last piece may be half inside
            const bool whole = vbase + N / 2 < nvec;
            __builtin_amdgcn_raw_buffer_store_b128(yb, rY, whole ? oy : kOOB, 0, 0);
            if (nvec % N) __builtin_amdgcn_raw_buffer_store_b64(u32x2{yb.x, yb.y}, rY, whole ? kOOB : oy, 0, 0);
        }
        if (z < 7) {
            // (the weights are not fetched above the stencil, whose operands
            // take the registers)
            __builtin_amdgcn_sched_barrier(0);
            kb_fetch(z + 1, 0);
            if (f32) kb_fetch(z + 1, 1);
            __syncthreads();
            stage(z + 1);
            if (!f32) kb_fetch(z + 1, 1);
            kb_store(z + 1, kb_plane(z + 1));
            __syncthreads();
        }
    }

    int any = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) any |= odd[i];
    if (!__builtin_amdgcn_readfirstlane(any)) return;
    // (everything is formed anew, so that nothing is kept for this in the march)
    __threadfence_block();               // a thread reads its rows again
    const int me = int(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)));
    const int my_col = 8 * wave + (me >> 3), v0 = chunk * CH + (me & 7) * N;
    const int32_t* const atoms = rare->blk_atoms + rare->blk_atom_off[blk];
    for (int z = 0; z < 8; ++z) {
        const int64_t row = int64_t(blk) * kBlockPts + my_col + 64 * z;
        for (int en = rare->ent_off[row]; en < rare->ent_off[row + 1]; ++en)
            for (int vec = v0; vec < min(v0 + N, nvec); ++vec) {
                T sum = T(0);
                for (int lm = 0; lm < 4; ++lm) {
                    const T v = C[(int64_t(atoms[rare->ent_soff[en] / kSlotBytes]) * 4 + lm) * nvec + vec] * k.alpha;
                    if (!isfinite(v)) sum += rare->ent_beta[4 * int64_t(en) + lm] * v;
                }
                T* const y = Y + row * ldy + vec;
                if (!(sum == T(0))) *y += sum;
            }
    }
}

// weights of the KB row groups in MFMA operand order: lane 16 k + j of entry e
// holds channel k of row j of the group, zero where the row is outside the
// atom's support or the entry only pads the list
template <class T>
__global__ void __launch_bounds__(64) rg_beta_kernel(const int32_t* __restrict__ rg_off,
                                                     const int32_t* __restrict__ rg_slot,
                                                     const int32_t* __restrict__ rg_len,
                                                     const int32_t* __restrict__ ent_off,
                                                     const int32_t* __restrict__ ent_soff,
                                                     const T* __restrict__ ent_beta, T* __restrict__ rg_beta,
                                                     int64_t n_rg) {
    const int lane = threadIdx.x;
    // (in turns: a wave for each group of 2^30 rows would be 2^32 threads, which a
    // launch does not hold)
    for (int64_t rg = blockIdx.x; rg < n_rg; rg += gridDim.x) {
        const int64_t row = rg / kGroups * kBlockPts + rg % 8 * 64 + rg / 8 % 4 * kRowGroup + (lane & 15);
        const int e0 = rg_off[rg], e1 = rg_off[rg + 1], n = rg_len[rg];
        for (int e = e0; e < e1; ++e) {
            T b = T(0);
            if (e - e0 < n)
                for (int en = ent_off[row]; en < ent_off[row + 1]; ++en)
                    if (ent_soff[en] == rg_slot[e]) b = ent_beta[4 * int64_t(en) + (lane >> 4)];
            rg_beta[int64_t(e) * 64 + lane] = b;
        }
    }
}

// Row-group lists of the staged tile kernel (Hilbert layout, blocks of at most
// kMaxBlockAtoms atoms): per group the LDS offsets of the slots whose atoms
// touch it, and their weights, 256 (FP32) or 512 bytes an entry, kept as long as the
// handle.  Si clusters have 5.3 entries to a group that has any, 6.9 with the
// padding: 40 MB (FP32) and 80 MB (FP64) at 3 nm, 176 and 352 MB at 5 nm, 5.9 and
// 11.7 GB at 16 nm.  Built from the entry tables at ham_build.
void build_row_groups(chf_ham* H, hipStream_t s) {
    const HostProj& P = H->proj;
    if (H->grid.ordering != CHF_ORDER_HILBERT || P.n_proj == 0 || P.max_block_atoms > kMaxBlockAtoms) return;
    const int64_t n_rg = H->grid.n_blocks * kGroups;
    std::vector<int32_t> off, len, slot;
    // (block, x-line pair, plane): the planes of a pair are consecutive
    list_row_groups(P, n_rg, kRowGroup, kKbStep, kKbAhead, kSlotBytes, [](int64_t rg) {
        return rg / kGroups * kBlockPts + rg % 8 * 64 + rg / 8 % 4 * kRowGroup;
    }, off, len, slot);
    DevBuf dlen;
    upload(H->rg_off, off, s);
    upload(H->rg_slot, slot, s);
    upload(dlen, len, s);
    auto fill = [&](auto* beta, const auto* src) {
        using T = std::remove_pointer_t<decltype(beta)>;
        rg_beta_kernel<T><<<dim3(unsigned(std::min<int64_t>(n_rg, 1 << 16))), dim3(64), 0, s>>>(
            H->rg_off.as<int32_t>(), H->rg_slot.as<int32_t>(), dlen.as<int32_t>(), H->ent_off32.as<int32_t>(),
            H->ent_soff.as<int32_t>(), src, beta, n_rg);
        LAUNCH_CHECK();
    };
    const std::vector<TileRare<double>> rare64{{H->ent_off32.as<int32_t>(), H->ent_soff.as<int32_t>(),
        H->blk_atom_off.as<int32_t>(), H->blk_atoms.as<int32_t>(), H->ent_beta64.as<double>()}};
    const std::vector<TileRare<float>> rare32{{H->ent_off32.as<int32_t>(), H->ent_soff.as<int32_t>(),
        H->blk_atom_off.as<int32_t>(), H->blk_atoms.as<int32_t>(), H->ent_beta32.as<float>()}};
    if (H->dtypes & 2) {
        H->rg_beta64.alloc(slot.size() * 64 * sizeof(double));
        fill(H->rg_beta64.as<double>(), H->ent_beta64.as<double>());
        upload(H->rare64, rare64, s);
    }
    if (H->dtypes & 1) {
        H->rg_beta32.alloc(slot.size() * 64 * sizeof(float));
        fill(H->rg_beta32.as<float>(), H->ent_beta32.as<float>());
        upload(H->rare32, rare32, s);
    }
    HIP_CHECK(hipStreamSynchronize(s));   // the host lists and dlen go out of scope
}

template <class T, int PB, int SLOTS>
static void launch_tile(chf_ham* H, const T* X, int64_t ldx, T* Y, int64_t ldy, const T* Z, int64_t ldz, int nvec,
                        const T* C, const StepCoef<T>& coef, hipStream_t s) {
    const int n_chunks = (nvec + 8 * Wide<T>::N - 1) / (8 * Wide<T>::N);
    // Chunks at a time: 2 where rows are whole cache lines, all where chunks share
    // lines.  us per launch for 1, 2, 4, all: 5 nm 256 FP32 2358, 2360, 2454, 2494;
    // 5 nm 128 FP64 2682, 2561, 2619, 2632; 3 nm 256 FP64 1478, 1478, 1536, 1596;
    // 1.1 nm 128 FP64 102, 103, 108, 110; but 2 nm 97 FP64 449, 393, 374, 343.
    const int group = PB == 128 ? 2 : n_chunks;
    const int64_t nt = (H->grid.n_blocks + 7) / 8 * 8 * n_chunks;
    const T* rg_beta = std::is_same<T, double>::value ? H->rg_beta64.as<T>() : H->rg_beta32.as<T>();
    hx_tile_kernel<T, PB, SLOTS><<<dim3(unsigned(nt)), dim3(512), 0, s>>>(
        int(H->grid.n_blocks), n_chunks, group, H->block_nbr.as<int32_t>(), H->block_mask.as<uint64_t>(), veff_of<T>(H),
        H->rg_off.as<int32_t>(), H->rg_slot.as<int32_t>(), rg_beta, H->blk_atom_off.as<int32_t>(),
        H->blk_atoms.as<int32_t>(), C, nvec, X, ldx, Y, ldy, Z, ldz,
        std::is_same<T, double>::value ? H->rare64.as<TileRare<T>>() : H->rare32.as<TileRare<T>>(), coef);
    LAUNCH_CHECK();
}

template <class T>
void launch_hx_tiled(chf_ham* H, const T* X, int64_t ldx, T* Y, int64_t ldy, const T* Z, int64_t ldz, int nvec,
                     const T* C, double alpha, double shift, double beta, hipStream_t s) {
    const bool kb = H->proj.n_proj > 0;
    const StepCoef<T> coef = make_coef<T>(H, alpha, shift, beta);
    if (kb && H->proj.max_block_atoms <= kMaxBlockAtoms) {
        // rows of whole cache lines or of 16-byte pieces where widths, leading
        // dimensions and base addresses allow, else of 8-byte ones
        constexpr int N = Wide<T>::N;
        const bool a16 = nvec % N == 0 && ldx % N == 0 && ldy % N == 0 && (!Z || ldz % N == 0) &&
                         uintptr_t(X) % 16 == 0 && uintptr_t(Y) % 16 == 0 && uintptr_t(Z) % 16 == 0;
        const auto lines = [](const void* q, int64_t ld) { return uintptr_t(q) % 128 == 0 && ld * sizeof(T) % 128 == 0; };
        const bool whole = a16 && lines(X, ldx) && lines(Y, ldy) && (!Z || lines(Z, ldz));
        auto go = [&](auto slots) {
            constexpr int SLOTS = decltype(slots)::value;
            if (whole) launch_tile<T, 128, SLOTS>(H, X, ldx, Y, ldy, Z, ldz, nvec, C, coef, s);
            else if (a16) launch_tile<T, 16, SLOTS>(H, X, ldx, Y, ldy, Z, ldz, nvec, C, coef, s);
            else launch_tile<T, 8, SLOTS>(H, X, ldx, Y, ldy, Z, ldz, nvec, C, coef, s);
        };
        if (H->proj.max_block_atoms <= kFewSlots) go(std::integral_constant<int, kFewSlots>{});
        else go(std::integral_constant<int, kMaxBlockAtoms>{});
        return;
    }
    constexpr int CH = kLanes * Lane<T>::N;
    const int n_chunks = (nvec + CH - 1) / CH;
    const int64_t nt = H->grid.n_blocks * int64_t(n_chunks);
    const dim3 grid(unsigned(((nt + 7) / 8) * 8)), block(64 * kLanes);
    const int32_t* eo = kb ? H->ent_off32.as<int32_t>() : nullptr;
    hx_tiled_kernel<T><<<grid, block, 0, s>>>(H->grid.n_blocks, n_chunks, H->block_nbr.as<int32_t>(),
                                             H->block_mask.as<uint64_t>(), veff_of<T>(H), eo, H->ent_atom.as<int32_t>(),
                                             ent_beta_of<T>(H), C, nvec, X, ldx, Y, ldy, Z, ldz, coef);
    LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// Narrow H X: blocks of one row piece (1 or 2 FP64, 2 or 4 FP32 vectors: Lanczos,
// residual checks).  One workgroup per run of 8^3 blocks, one thread per point;
// the three arms of the stencil are staged in LDS as lines of 20, [z][y][20 x],
// [z][20 y][x], [20 z][y][x], the coefficients of the block's atoms beside them,
// and each thread walks its row's entries.  The vector tile kernel has 1 or 2
// of 16 lanes working on such blocks: 63 us per launch at 3 nm for 2 FP64
// vectors (1491 blocks, 12 MB of X), this one 38, and 23 for one FP64 vector.
// Bound by latency: one round of loads, two barriers and 36 LDS reads per block
// at 3 workgroups per CU or fewer.
// ---------------------------------------------------------------------------
// most workgroups of a launch, 2 per CU: each takes a run of blocks, and with
// `part` leaves one partial of x.y
constexpr int kNarrowGroups = 512;

template <class T, int N>
__global__ void __launch_bounds__(512) hx_narrow_kernel(int n_blocks, int per_group, const int32_t* __restrict__ bnb,
                                                        const uint64_t* __restrict__ bmask, const T* __restrict__ veff,
                                                        const int32_t* __restrict__ ent_off,
                                                        const int32_t* __restrict__ ent_soff,
                                                        const T* __restrict__ ent_beta,
                                                        const int32_t* __restrict__ blk_atom_off,
                                                        const int32_t* __restrict__ blk_atoms, const T* __restrict__ C,
                                                        const T* __restrict__ X, int64_t ldx, T* Y, int64_t ldy, const T* Z,
                                                        int64_t ldz, StepCoef<T> k, double* __restrict__ part) {
    using V = Piece<T, N>;
    using B4 = Piece<T, 4>;
    constexpr int XS = 21, YL = 64 * XS, ZL = YL + 8 * 20 * 8;
    __shared__ V lines[ZL + 20 * 64];
    __shared__ V cst[kMaxBlockAtoms * 4];
    __shared__ double sh[8];
    const int t = threadIdx.x, lane = t & 63, x = t & 7, y = (t >> 3) & 7;
    const int z = __builtin_amdgcn_readfirstlane(t >> 6);
    // XCD-aware: each XCD takes a contiguous run of blocks (grid = 8 * per_xcd)
    const int group = int(blockIdx.x % 8) * int(gridDim.x / 8) + int(blockIdx.x / 8);
    const int first = group * per_group, last = min(n_blocks, first + per_group);
    // halo values: 6 sides x 6 depths x 64, a wave takes whole (side, depth)
    // layers; along x, where a layer is 64 single values, 6 layers are dealt in
    // memory order instead
    int at[5], row[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        const int item = z + 8 * j, side = item / 6, c = item % 6, d = side & 1;
        if (side < 2) {
            const int i = c * 64 + lane, cc = i % 6, line = i / 6;      // line = y + 8 z
            row[j] = line * 8 + (d ? cc : 2 + cc);
            at[j] = line * XS + (d ? 14 + cc : cc);
        } else if (side < 4) {
            row[j] = (lane >> 3) * 64 + (d ? c : 2 + c) * 8 + x;
            at[j] = YL + ((lane >> 3) * 20 + (d ? 14 + c : c)) * 8 + x;
        } else {
            row[j] = (d ? c : 2 + c) * 64 + lane;
            at[j] = ZL + (d ? 14 + c : c) * 64 + lane;
        }
    }
    V zero;
#pragma unroll
    for (int e = 0; e < N; ++e) zero.e[e] = T(0);
    // (rows may start on any element)
    auto piece = [](const T* p) {
        V v;
        __builtin_memcpy(&v, p, sizeof(V));
        return v;
    };
    auto load = [&](int64_t r) { return piece(X + r * ldx); };
    double dot = 0.0;
    for (int blk = first; blk < last; ++blk) {
        const int64_t base = int64_t(blk) * kBlockPts;
        const V v = load(base + t);
        V hv[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            hv[j] = zero;
            const int item = z + 8 * j;
            if (item >= 36) continue;
            const int nb = bnb[6 * int64_t(blk) + item / 6];
            if (nb >= 0) hv[j] = load(int64_t(nb) * kBlockPts + row[j]);
        }
        const V zv = Z ? piece(Z + (base + t) * ldz) : zero;
        const T vr = veff[base + t];
        int e0 = 0, e1 = 0, na = 0, a0 = 0;
        V cv = zero;
        if (ent_off) {
            e0 = ent_off[base + t];
            e1 = ent_off[base + t + 1];
            a0 = blk_atom_off[blk];
            na = min(blk_atom_off[blk + 1] - a0, kMaxBlockAtoms);
            if (t < 4 * na)
                cv = *reinterpret_cast<const V*>(C + (int64_t(blk_atoms[a0 + (t >> 2)]) * 4 + (t & 3)) * N);
        }
        __syncthreads();             // the last block's lines have been read
        V* const cx = lines + (z * 8 + y) * XS + x + 6;
        V* const cy = lines + YL + (z * 20 + y + 6) * 8 + x;
        V* const cz = lines + ZL + (z + 6) * 64 + lane;
        *cx = *cy = *cz = v;
#pragma unroll
        for (int j = 0; j < 5; ++j)
            if (z + 8 * j < 36) lines[at[j]] = hv[j];
        if (t < 4 * na) cst[t] = cv;
        __syncthreads();
        // (an entry's weights and slot are loaded one entry ahead)
        V kb = zero;
        int so = 0;
        B4 bb{};
        if (e0 < e1) {
            so = ent_soff[e0];
            bb = *reinterpret_cast<const B4*>(ent_beta + 4 * int64_t(e0));
        }
        // unrolled by 2 the kernel takes fewer registers, so more waves share a CU:
        // 28 -> 23 us for one FP64 vector at 3 nm, 33 -> 26 for 4 FP32; 2 FP64
        // vectors do not fit 3 workgroups either way and lose (7.5 -> 16 us at
        // 1.1 nm)
        constexpr int U = sizeof(T) == 8 && N == 2 ? 6 : 2;
        V acc;
#pragma unroll
        for (int e = 0; e < N; ++e) acc.e[e] = T(0);
#pragma unroll U
        for (int s = 1; s <= 6; ++s) {
            const V zm = cz[-64 * s], zp = cz[64 * s], xm = cx[-s], xp = cx[s], ym = cy[-8 * s], yp = cy[8 * s];
#pragma unroll
            for (int e = 0; e < N; ++e) {
                T sum = zm.e[e] + zp.e[e];
                sum += xm.e[e];
                sum += xp.e[e];
                sum += ym.e[e];
                sum += yp.e[e];
                acc.e[e] = fma(k.ac[s], sum, acc.e[e]);
            }
        }
        for (int en = e0; en < e1; ++en) {
            const V* const c = cst + (so / kSlotBytes) * 4;
            const B4 b = bb;
            if (en + 1 < e1) {
                so = ent_soff[en + 1];
                bb = *reinterpret_cast<const B4*>(ent_beta + 4 * int64_t(en + 1));
            }
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int e = 0; e < N; ++e) kb.e[e] = fma(b.e[m], c[m].e[e], kb.e[e]);
        }
        const T dg = fma(k.alpha, vr, k.d0);
        const bool in = (bmask[8 * int64_t(blk) + z] >> lane) & 1;
        V out;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const T r = fma(-k.beta, zv.e[e], fma(dg, v.e[e], fma(k.alpha, kb.e[e], acc.e[e])));
            out.e[e] = in ? r : T(0);
        }
        __builtin_memcpy(Y + (base + t) * ldy, &out, sizeof(V));
        dot += double(v.e[0]) * double(out.e[0]);
    }
    if (part) {
        const double s = group_sum(dot, sh);
        if (t == 0) part[group] = s;
    }
}

// whether a block of nvec vectors is one row piece, on a handle with the tables
// that the kernel reads.  The rule is the width alone, so that a filter that goes
// through its columns one by one has the arithmetic of one that takes them at once.
template <class T>
static bool narrow_ok(const chf_ham* H, int nvec) {
    const int64_t bytes = int64_t(nvec) * int64_t(sizeof(T));
    return H->grid.ordering == CHF_ORDER_HILBERT && H->proj.max_block_atoms <= kMaxBlockAtoms && (bytes == 8 || bytes == 16);
}

// launches it and returns the number of workgroups (= partials)
template <class T>
static int launch_narrow(chf_ham* H, const T* X, int64_t ldx, T* Y, int64_t ldy, const T* Z, int64_t ldz, int nvec,
                         const T* C, double alpha, double shift, double beta, double* part, hipStream_t s) {
    const int nblk = int(H->grid.n_blocks);
    const int per = (nblk + kNarrowGroups - 1) / kNarrowGroups;
    const unsigned grid = unsigned(((nblk + per - 1) / per + 7) / 8 * 8);
    const bool kb = H->proj.n_proj > 0;
    auto go = [&](auto n) {
        hx_narrow_kernel<T, decltype(n)::value><<<grid, 512, 0, s>>>(
            nblk, per, H->block_nbr.as<int32_t>(), H->block_mask.as<uint64_t>(), veff_of<T>(H),
            kb ? H->ent_off32.as<int32_t>() : nullptr, H->ent_soff.as<int32_t>(), ent_beta_of<T>(H),
            H->blk_atom_off.as<int32_t>(), H->blk_atoms.as<int32_t>(), C, X, ldx, Y, ldy, Z, ldz,
            make_coef<T>(H, alpha, shift, beta), part);
    };
    constexpr int N8 = 8 / int(sizeof(T));
    if (nvec == N8) go(std::integral_constant<int, N8>{});
    else go(std::integral_constant<int, 2 * N8>{});
    LAUNCH_CHECK();
    return int(grid);
}

bool hx_dot_ok(const chf_ham* H) {
    return H->grid.ordering == CHF_ORDER_HILBERT && H->proj.max_block_atoms <= kMaxBlockAtoms;
}

// ---------------------------------------------------------------------------
// optional per-kernel timing: HIP events recorded on the launch stream
// around every H X and KB-gather launch while enabled
// ---------------------------------------------------------------------------
struct KernelTimer {
    std::atomic<bool> on{false};
    std::vector<std::pair<hipEvent_t, hipEvent_t>> spans[2];   // 0: H X, 1: KB gather
    std::vector<hipEvent_t> pool;
    hipEvent_t get() {
        if (!pool.empty()) {
            hipEvent_t e = pool.back();
            pool.pop_back();
            return e;
        }
        hipEvent_t e;
        HIP_CHECK(hipEventCreate(&e));
        return e;
    }
    void recycle() {
        for (auto& v : spans) {
            for (auto& p : v) {
                pool.push_back(p.first);
                pool.push_back(p.second);
            }
            v.clear();
        }
    }
};
static KernelTimer g_timer;
static std::mutex g_timer_mu;   // guards the event pool and the spans

template <class F>
static void timed(int which, hipStream_t s, F&& launch) {
    if (!g_timer.on.load(std::memory_order_relaxed)) {
        launch();
        return;
    }
    hipEvent_t a, b;
    {
        std::lock_guard<std::mutex> lk(g_timer_mu);
        a = g_timer.get();
        b = g_timer.get();
    }
    HIP_CHECK(hipEventRecord(a, s));
    launch();
    HIP_CHECK(hipEventRecord(b, s));
    std::lock_guard<std::mutex> lk(g_timer_mu);
    g_timer.spans[which].emplace_back(a, b);
}

void timed_hx(hipStream_t s, const std::function<void()>& launch) { timed(0, s, launch); }

int hx_dot(chf_ham* H, const double* x, double* y, double* part, hipStream_t s) {
    H->kb_coef.ensure(kb_coef_bytes(H, 1, sizeof(double)));
    double* C = H->kb_coef.as<double>();
    if (H->proj.n_proj > 0) timed(1, s, [&] { launch_kb_gather<double>(H, x, 1, 1, C, s); });
    int n = 0;
    timed(0, s, [&] { n = launch_narrow<double>(H, x, 1, y, 1, nullptr, 0, 1, C, 1.0, 0.0, 0.0, part, s); });
    return n;
}

// ---------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------
template <class T>
bool tiled_ok(const chf_ham* H, const void* X, int64_t ldx, const void* Y, int64_t ldy, const void* Z, int64_t ldz,
              int nvec) {
    constexpr int LN = Lane<T>::N;
    if (H->grid.ordering != CHF_ORDER_HILBERT) return false;
    if (nvec % LN || ldx % LN || ldy % LN || (Z && ldz % LN)) return false;
    if (int64_t(kBlockPts) * std::max(ldx, std::max(ldy, ldz)) * int64_t(sizeof(T)) >= (int64_t(1) << 30)) return false;
    const uintptr_t al = 8;
    if (uintptr_t(X) % al || uintptr_t(Y) % al || (Z && uintptr_t(Z) % al)) return false;
    return true;
}

// bytes of the KB coefficient scratch C [4 n_proj][nvec] of an H X launch
size_t kb_coef_bytes(const chf_ham* H, int nvec, size_t elem_bytes) {
    return size_t(std::max<int64_t>(1, H->proj.n_proj)) * 4 * size_t(nvec) * elem_bytes;
}

template <class T>
void hx_step(chf_ham* H, const T* X, int64_t ldx, T* Y, int64_t ldy, const T* Z, int64_t ldz, int nvec, double alpha,
             double shift, double beta, hipStream_t s, int force_kernel, bool lap_only, T* C_ext, bool narrow) {
    // the KB coefficients go to the handle's scratch (grown on demand), or to
    // the caller's C_ext (no allocation, no kernel timing)
    T* C = C_ext;
    if (!C) {
        H->kb_coef.ensure(kb_coef_bytes(H, nvec, sizeof(T)));
        C = H->kb_coef.as<T>();
    }
    auto run = [&](int which, auto&& launch) {
        if (C_ext) launch();
        else timed(which, s, launch);
    };
    if (H->proj.n_proj > 0 && !lap_only) run(1, [&] { launch_kb_gather<T>(H, X, ldx, nvec, C, s); });
    const bool tiled = force_kernel != 1 && !lap_only && tiled_ok<T>(H, X, ldx, Y, ldy, Z, ldz, nvec);
    if (tiled && narrow && narrow_ok<T>(H, nvec)) {
        run(0, [&] { launch_narrow<T>(H, X, ldx, Y, ldy, Z, ldz, nvec, C, alpha, shift, beta, nullptr, s); });
    } else if (tiled) {
        run(0, [&] { launch_hx_tiled<T>(H, X, ldx, Y, ldy, Z, ldz, nvec, C, alpha, shift, beta, s); });
    } else {
        if (!H->has_nbr) fail(CHF_EUNSUPPORTED, "generic H X needs the neighbour table (keep_nbr) for this layout");
        run(0, [&] { launch_hx_generic<T>(H, X, ldx, Y, ldy, Z, ldz, nvec, C, alpha, shift, beta, s, lap_only); });
    }
}

// Degree-m scaled filter (CheFSI paragraph; the Zhou-Saad form).  With
// e = (b - a) / 2, c = (b + a) / 2 and sigma_k = T_{k-1}(t0) / T_k(t0),
// t0 = (a0 - c) / e, the normalised iterates Y_k = T_k((H - c) / e) X / T_k(t0)
// obey
//   Y_1 = (sigma_1 / e) (H - c) X,
//   Y_k = (2 sigma_k / e) (H - c) Y_{k-1} - sigma_{k-1} sigma_k Y_{k-2},
//   sigma_1 = e / (a0 - c), sigma_k = 1 / (2 / sigma_1 - sigma_{k-1}).
// Y_k overwrites Y_{k-2} in place (X for even k, the work block for odd k).
// The vectors are independent, so a work block narrower than the block is
// used column block by column block: min(nvec, ldw, max_cols) columns at a
// time (a multiple of 64, else of 4, when fewer than nvec, so that every
// block keeps the kernels' 16-byte alignment).  C_ext: KB-coefficient
// scratch of the caller for max_cols vectors (NULL: the handle's own).
template <class T>
void filter_run(chf_ham* H, T* X, int64_t ldx, T* W, int64_t ldw, int nvec, int m, double a, double b, double a0,
                hipStream_t s, int force_kernel, int64_t max_cols, T* C_ext) {
    const double e = (b - a) / 2, c = (b + a) / 2;
    const double sigma1 = e / (a0 - c);
    int64_t nb = std::min<int64_t>(nvec, std::min<int64_t>(ldw, max_cols));
    if (nb < nvec && nb >= 64) nb -= nb % 64;
    else if (nb < nvec && nb >= 4) nb -= nb % 4;
    // (by the whole call's width, so that a column block of a wider call has
    // the arithmetic of its neighbours)
    const bool narrow = nvec * int(sizeof(T)) <= 16;
    for (int c0 = 0; c0 < nvec; c0 += int(nb)) {
        const int w = int(std::min<int64_t>(nb, nvec - c0));
        T* Xc = X + c0;
        double sigma = sigma1;
        hx_step<T>(H, Xc, ldx, W, ldw, nullptr, 0, w, sigma1 / e, c, 0.0, s, force_kernel, false, C_ext, narrow);
        for (int k = 2; k <= m; ++k) {
            const double sigma_next = 1.0 / (2.0 / sigma1 - sigma);
            const double alpha = 2.0 * sigma_next / e, beta = sigma * sigma_next;
            if (k % 2 == 0)
                hx_step<T>(H, W, ldw, Xc, ldx, Xc, ldx, w, alpha, c, beta, s, force_kernel, false, C_ext, narrow);
            else
                hx_step<T>(H, Xc, ldx, W, ldw, W, ldw, w, alpha, c, beta, s, force_kernel, false, C_ext, narrow);
            sigma = sigma_next;
        }
        if (m % 2 == 1)
            HIP_CHECK(hipMemcpy2DAsync(Xc, size_t(ldx) * sizeof(T), W, size_t(ldw) * sizeof(T), size_t(w) * sizeof(T),
                                       size_t(H->grid.n_rows), hipMemcpyDeviceToDevice, s));
    }
}

template void filter_run<float>(chf_ham*, float*, int64_t, float*, int64_t, int, int, double, double, double,
                                hipStream_t, int, int64_t, float*);
template void filter_run<double>(chf_ham*, double*, int64_t, double*, int64_t, int, int, double, double, double,
                                 hipStream_t, int, int64_t, double*);

// ---------------------------------------------------------------------------
// Allocation-free filter (chebyshev_filter_noalloc): the KB coefficients live
// in this fixed device array instead of the handle's scratch.  Each device
// the library runs on holds its own copy until the process ends; its address
// on a device is looked up once, with that device current, when the first
// Hamiltonian is built there (ham_build), and only that address is passed to
// kernels.  Calls that overlap on one device share the array and race.
// ---------------------------------------------------------------------------
constexpr size_t kNoallocScratchBytes = size_t(64) << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

void noalloc_scratch_init(int device) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    CHF_REQUIRE(device >= 0 && device < kMaxDevices, "device index %d beyond %d", device, kMaxDevices);
    if (g_scratch_ptr[device]) return;
    void* p = nullptr;
    HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    CHF_REQUIRE(p != nullptr, "no device address for the filter scratch");
    g_scratch_ptr[device] = p;
}

template <class T>
void filter_run_noalloc(chf_ham* H, T* X, int64_t ldx, T* W, int64_t ldw, int nvec, int m, double a, double b,
                        double a0, hipStream_t s) {
    void* p = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_scratch_mu);
        if (H->device >= 0 && H->device < kMaxDevices) p = g_scratch_ptr[H->device];
    }
    if (!p) fail(CHF_EINVAL, "chebyshev_filter_noalloc: no scratch on device %d (no Hamiltonian built there)", H->device);
    // KB coefficients of one vector: 4 channels per projector atom
    const size_t per_vec = kb_coef_bytes(H, 1, sizeof(T));
    const int64_t max_cols = int64_t(kNoallocScratchBytes / per_vec);
    if (max_cols < 1)
        fail(CHF_EINVAL, "chebyshev_filter_noalloc: the KB coefficients of one vector (%zu bytes for %lld projector "
             "atoms) exceed the %zu-byte scratch", per_vec, (long long)H->proj.n_proj, kNoallocScratchBytes);
    filter_run<T>(H, X, ldx, W, ldw, nvec, m, a, b, a0, s, 0, max_cols, static_cast<T*>(p));
}

template void filter_run_noalloc<float>(chf_ham*, float*, int64_t, float*, int64_t, int, int, double, double, double,
                                        hipStream_t);
template void filter_run_noalloc<double>(chf_ham*, double*, int64_t, double*, int64_t, int, int, double, double,
                                         double, hipStream_t);

void timer_enable(int on) {
    std::lock_guard<std::mutex> lk(g_timer_mu);
    g_timer.recycle();
    g_timer.on.store(on != 0, std::memory_order_relaxed);
}

void timer_read(double* ms, int64_t* launches) {
    HIP_CHECK(hipDeviceSynchronize());
    std::lock_guard<std::mutex> lk(g_timer_mu);
    for (int w = 0; w < 2; ++w) {
        double t = 0;
        for (auto& p : g_timer.spans[w]) {
            float f = 0;
            HIP_CHECK(hipEventElapsedTime(&f, p.first, p.second));
            t += f;
        }
        ms[w] = t;
        launches[w] = int64_t(g_timer.spans[w].size());
    }
}

template void hx_step<float>(chf_ham*, const float*, int64_t, float*, int64_t, const float*, int64_t, int, double,
                             double, double, hipStream_t, int, bool, float*, bool);
template void hx_step<double>(chf_ham*, const double*, int64_t, double*, int64_t, const double*, int64_t, int,
                              double, double, double, hipStream_t, int, bool, double*, bool);
template void launch_kb_gather<float>(chf_ham*, const float*, int64_t, int, float*, hipStream_t);
template void launch_kb_gather<double>(chf_ham*, const double*, int64_t, int, double*, hipStream_t);

}  // namespace chf
