// Gram products S = A^T B of row-major blocks on gfx950's matrix cores.
//
// A wave owns a 64 x 64 piece of S (32 x 32 or 16 x 16 for narrow blocks) and
// walks the rows of its slice 4 at a time: A^T and B have the rows as the
// contraction index, so a row-major block is already in operand order and the
// rows go from memory straight to the operand registers, 16 bytes per lane and
// load, without LDS.  A load's P consecutive columns belong to P different
// 16 x 16 products, which only permutes the columns a product stands for.
//
// Bound by the matrix cores: 16 products (512 cycles FP32, 1024 FP64) per 2 (4)
// loads of 1 KB per wave, 16 B per cycle and CU from the L1.  S = X^T X takes
// the pieces with i <= j only, which a general matrix product cannot skip.
// Measured against batched library products of 8192-row slices (us):
//   440,000 x 1024 FP32   X^T X 6940 -> 3960 (131 TFLOP/s done), A^T B 6850 -> 6460
//   440,000 x 600  FP64   X^T X 6015 -> 3160, A^T B 6100 -> 5050
//   120,000 x 128  FP64   X^T X 231 -> 81;   x 24: 227 -> 18.5
//   440,000 x 12   FP32   X^T X 125 -> 24
#include <algorithm>
#include <vector>

#include "internal.hpp"
#include "kernels.hpp"

namespace chf {

// rows per slice: an FP32 sum never runs over more than kGramSliceRows rows
// (the slices' partials are added in FP64); below that, enough slices for
// kGramTargetGroups workgroups, of at least kGramMinRows rows each, since a
// slice costs a partial of m x n values written and read once
constexpr int64_t kGramSliceRows = 8192;
constexpr int64_t kGramMinRows = 256;
constexpr int64_t kGramTargetGroups = 4096;
constexpr size_t kGramPartBytes = size_t(1) << 30;   // partials at once, a group of slices
constexpr int64_t kGramUnroll = 4;                   // 4-row steps per loop turn
constexpr int64_t kMaxGroups = int64_t(1) << 24;     // of 256 threads: a launch has less than 2^32

static int64_t gram_ldp(int n) { return (int64_t(n) + 3) / 4 * 4; }

// columns of a wave's piece, and whether 2 x 2 waves share a workgroup's piece
// of 128 x 128 (else one piece per workgroup, its 4 waves on 4 slices)
static int gram_width(int m, int n) {
    const int w = std::max(m, n);
    return w <= 16 ? 16 : w <= 32 ? 32 : 64;
}

GramSlices gram_slices(int64_t n_rows, int m, int n, size_t acc_bytes, size_t in_bytes, int64_t ld, bool symmetric) {
    const int W = gram_width(m, n);
    const bool quad = std::max(m, n) > 64;
    const int64_t side = quad ? 128 : W;
    const int64_t tm = (m + side - 1) / side, tn = (n + side - 1) / side;
    GramSlices g;
    g.tiles = symmetric ? tm * (tm + 1) / 2 : tm * tn;
    const int64_t per_group = quad ? 1 : 4;            // slices per workgroup
    const int64_t want = std::max<int64_t>(1, kGramTargetGroups * per_group / g.tiles);
    int64_t rows = std::max<int64_t>(1, (n_rows + want - 1) / want);
    rows = std::min(kGramSliceRows, std::max(kGramMinRows, rows));
    g.part_stride = int64_t(m) * gram_ldp(n);
    const size_t per = size_t(g.part_stride) * acc_bytes;
    const int64_t total = std::max<int64_t>(1, (n_rows + rows - 1) / rows);
    g.most = std::max((n_rows + kGramSliceRows - 1) / kGramSliceRows,
                      std::min(want, (n_rows + kGramMinRows - 1) / kGramMinRows));
    rows = std::max<int64_t>(1, (n_rows + total - 1) / total);             // balanced
    g.group = std::max<int64_t>(1, std::min<int64_t>(total, int64_t(kGramPartBytes / per)));
    g.part_bytes = size_t(g.group) * per;
    const int64_t fit = ((int64_t(1) << 32) - 1) / (ld * int64_t(in_bytes));   // 32-bit sizes of a slice
    g.rows = std::max<int64_t>(1, std::min(rows, fit));
    return g;
}

// Most bytes of partials over all products of at most n_rows rows, m x n columns:
// narrower ones have fewer pieces, so more slices, and may hold more in all.  With
// the number of pieces the slices are given, and the widest of that number holds
// most.
size_t gram_part_bound(int64_t n_rows, int m, int n, size_t acc_bytes, bool symmetric) {
    size_t most = 0;
    const auto widths = [](int w) {
        std::vector<int> v;
        for (int c : {16, 32, 64})
            if (c < w) v.push_back(c);
        for (int c = 128; c < w; c += 128) v.push_back(c);
        v.push_back(w);
        return v;
    };
    for (int a : widths(m))
        for (int b : widths(n)) {
            if (symmetric && a != b) continue;
            const GramSlices g = gram_slices(n_rows, a, b, acc_bytes, acc_bytes, 1, symmetric);
            const size_t per = size_t(g.part_stride) * acc_bytes;
            most = std::max(most, std::min(size_t(g.most) * per, std::max(kGramPartBytes, per)));
        }
    return most;
}

namespace {

using u32x4 = __attribute__((ext_vector_type(4))) unsigned;
using u32x2 = __attribute__((ext_vector_type(2))) unsigned;

template <class T>
using Acc = T __attribute__((ext_vector_type(4)));

__device__ inline Acc<float> mfma(float a, float b, Acc<float> c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ inline Acc<double> mfma(double a, double b, Acc<double> c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// row of the 16 x 16 result held by (register, lane); the column is lane % 16
template <class TA>
__device__ inline int result_row(int reg, int lane) {
    return sizeof(TA) == 4 ? 4 * (lane >> 4) + reg : 4 * reg + (lane >> 4);
}

template <class T, int P>
struct alignas(sizeof(T) * P) Cols {
    T e[P];
};
template <class T, int P>
__device__ inline Cols<T, P> load_cols(__amdgpu_buffer_rsrc_t r, unsigned off) {
    constexpr int bytes = int(sizeof(T)) * P;
    if constexpr (bytes == 16) return __builtin_bit_cast(Cols<T, P>, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    else if constexpr (bytes == 8) return __builtin_bit_cast(Cols<T, P>, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    else return __builtin_bit_cast(Cols<T, P>, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

}  // namespace

// part[slice][i][j] (row stride ldp) = sum over the slice's rows of A[r][i] B[r][j].
// An XCD takes a contiguous run of (slice, tile), so that the tiles of a slice
// share its rows in one L2.
template <class TI, class TA, int P, int G, bool QUAD>
__global__ void __launch_bounds__(256) gram_kernel(const TI* __restrict__ A, int64_t lda, const TI* __restrict__ B,
                                                   int64_t ldb, int64_t n_rows, int m, int n, int rows, int n_slices,
                                                   int tiles, int total, int symmetric, TA* __restrict__ part,
                                                   int64_t ldp) {
    constexpr int W = 16 * P * G, TC = P * G, U = G > 1 ? int(kGramUnroll) / 2 : int(kGramUnroll);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int id = int(blockIdx.x % 8) * int(gridDim.x / 8) + int(blockIdx.x / 8);
    if (id >= total) return;
    int tile = id % tiles, slice = id / tiles;
    constexpr int side = QUAD ? 2 * W : W;
    const int tn = (n + side - 1) / side;
    int ti = 0, tj;
    if (symmetric) {
        while (tile >= tn - ti) tile -= tn - ti, ++ti;
        tj = ti + tile;
    } else {
        ti = tile / tn;
        tj = tile % tn;
    }
    int i0 = ti * side, j0 = tj * side;
    if (QUAD) {
        i0 += (wave >> 1) * W;
        j0 += (wave & 1) * W;
    } else {
        slice = slice * 4 + wave;
    }
    if (slice >= n_slices || i0 >= m || j0 >= n || (symmetric && j0 < i0)) return;
    const int64_t r0 = int64_t(slice) * rows;
    const int nr = int(min(int64_t(rows), n_rows - r0));
    // rows past the slice and columns past the block read zero or values of
    // columns that are not stored
    const unsigned za = unsigned((int64_t(nr - 1) * lda + m) * int64_t(sizeof(TI)));
    const unsigned zb = unsigned((int64_t(nr - 1) * ldb + n) * int64_t(sizeof(TI)));
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<TI*>(A + r0 * lda), 0, int(za), 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<TI*>(B + r0 * ldb), 0, int(zb), 0x00020000);
    // offsets stay at the end of the slice once they have passed it
    auto clip = [](int64_t v, unsigned z) { return unsigned(min(v, int64_t(z))); };
    auto step = [](unsigned o, unsigned d, unsigned z) { return min(__builtin_elementwise_add_sat(o, d), z); };
    const unsigned sa = clip(4 * lda * int64_t(sizeof(TI)), za), sb = clip(4 * ldb * int64_t(sizeof(TI)), zb);
    unsigned oa = clip(((lane >> 4) * lda + i0 + P * (lane & 15)) * int64_t(sizeof(TI)), za);
    unsigned ob = clip(((lane >> 4) * ldb + j0 + P * (lane & 15)) * int64_t(sizeof(TI)), zb);
    using C = Cols<TI, P>;
    C a[2][U][G], b[2][U][G];
    auto fetch = [&](auto buf) {
        constexpr int k = decltype(buf)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                a[k][u][g] = load_cols<TI, P>(ra, step(oa, g * 16 * P * unsigned(sizeof(TI)), za));
                b[k][u][g] = load_cols<TI, P>(rb, step(ob, g * 16 * P * unsigned(sizeof(TI)), zb));
            }
            oa = step(oa, sa, za);
            ob = step(ob, sb, zb);
        }
    };
    Acc<TA> acc[TC][TC];
#pragma unroll
    for (int p = 0; p < TC; ++p)
#pragma unroll
        for (int q = 0; q < TC; ++q) acc[p][q] = Acc<TA>{0, 0, 0, 0};
    auto multiply = [&](auto buf) {
        constexpr int k = decltype(buf)::value;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int p = 0; p < TC; ++p)
#pragma unroll
                for (int q = 0; q < TC; ++q)
                    acc[p][q] = mfma(TA(a[k][u][p / P].e[p % P]), TA(b[k][u][q / P].e[q % P]), acc[p][q]);
    };
    using K0 = std::integral_constant<int, 0>;
    using K1 = std::integral_constant<int, 1>;
    fetch(K0{});
    for (int r = 0; r < nr; r += 8 * U) {
        fetch(K1{});
        multiply(K0{});
        fetch(K0{});
        multiply(K1{});
    }
    TA* const out = part + int64_t(slice) * m * ldp;
#pragma unroll
    for (int p = 0; p < TC; ++p)
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int i = i0 + p / P * 16 * P + P * result_row<TA>(reg, lane) + p % P;
            if (i >= m) continue;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int j = j0 + g * 16 * P + P * (lane & 15);
                if (j >= ldp) continue;
                Cols<TA, P> v;
#pragma unroll
                for (int q = 0; q < P; ++q) v.e[q] = acc[p][g * P + q][reg];
                *reinterpret_cast<Cols<TA, P>*>(out + int64_t(i) * ldp + j) = v;
            }
        }
}

// S[i][j] (+)= sum over slices of part[s][i][j], in FP64 and in a fixed order
// (accumulate: add to S, for the slice groups after the first); with a symmetric
// product only i <= j is summed and mirrored, so S is exactly symmetric.  A
// workgroup takes 32 columns of a row and 8 runs of slices, and goes on to the next
// of its pieces: a launch holds fewer than 2^24 workgroups of 256 threads, and more
// would be dropped without an error (from 23,171 x 23,171 on).
template <class TA>
__global__ void __launch_bounds__(256) gram_reduce_kernel(int m, int n, int n_slices, const TA* __restrict__ part,
                                                          int64_t ldp, double* __restrict__ S, int64_t lds, int symmetric,
                                                          int accumulate) {
    __shared__ double sh[8][33];
    const int chunks = (n + 31) / 32, q = threadIdx.x / 32;
    for (int64_t piece = blockIdx.x; piece < int64_t(m) * chunks; piece += gridDim.x) {
        const int i = int(piece / chunks), jb = int(piece % chunks) * 32, j = jb + int(threadIdx.x % 32);
        if (symmetric && jb + 31 < i) continue;
        const bool in = j < n && !(symmetric && i > j);
        double acc = 0.0;
        if (in) {
            const TA* const p = part + int64_t(i) * ldp + j;
            const int64_t stride = int64_t(m) * ldp;
#pragma unroll 8
            for (int k = q; k < n_slices; k += 8) acc += double(p[k * stride]);
        }
        __syncthreads();             // the last piece's sums have been read
        sh[q][threadIdx.x % 32] = acc;
        __syncthreads();
        if (q > 0 || !in) continue;
        double s = accumulate ? S[int64_t(i) * lds + j] : 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k) s += sh[k][threadIdx.x];
        S[int64_t(i) * lds + j] = s;
        if (symmetric && i < j) S[int64_t(j) * lds + i] = s;
    }
}

template <class TI, class TA>
void gram_product(chf_ctx* ctx, const TI* A, int64_t lda, const TI* B, int64_t ldb, int64_t n_rows, int m, int n,
                  double* S, int64_t lds, hipStream_t s) {
    const bool symmetric = (A == B) && (m == n) && (lda == ldb);
    const GramSlices g = gram_slices(n_rows, m, n, sizeof(TA), sizeof(TI), std::max(lda, ldb), symmetric);
    CHF_REQUIRE(lda <= INT32_MAX && ldb <= INT32_MAX, "gram: leading dimension beyond 32 bits");
    ctx->scratch2.ensure(g.part_bytes);
    TA* part = ctx->scratch2.as<TA>();
    const int64_t ldp = gram_ldp(n);
    const int64_t n_slices = (n_rows + g.rows - 1) / g.rows;
    const int W = gram_width(m, n);
    const bool quad = std::max(m, n) > 64;
    for (int64_t s0 = 0; s0 < n_slices; s0 += g.group) {
        const int cnt = int(std::min<int64_t>(g.group, n_slices - s0));
        const int64_t at = s0 * g.rows;
        const int64_t slots = (quad ? cnt : (cnt + 3) / 4);
        const int64_t total = slots * g.tiles, groups = (total + 7) / 8 * 8;
        CHF_REQUIRE(groups < kMaxGroups, "gram: grid too large");
        auto go = [&](auto p, auto gg, auto qd) {
            gram_kernel<TI, TA, decltype(p)::value, decltype(gg)::value, decltype(qd)::value>
                <<<unsigned(groups), 256, 0, s>>>(A + at * lda, lda, B + at * ldb, ldb, n_rows - at, m, n, int(g.rows),
                                                  cnt, int(g.tiles), int(total), symmetric ? 1 : 0,
                                                  part, ldp);
        };
        constexpr int PW = 16 / int(sizeof(TI));        // columns of a 16-byte load
        using One = std::integral_constant<int, 1>;
        using Two = std::integral_constant<int, 2>;
        if (quad) go(std::integral_constant<int, PW>{}, std::integral_constant<int, 4 / PW>{}, std::true_type{});
        else if (W == 64) go(std::integral_constant<int, PW>{}, std::integral_constant<int, 4 / PW>{}, std::false_type{});
        else if (W == 32) go(Two{}, One{}, std::false_type{});
        else go(One{}, One{}, std::false_type{});
        LAUNCH_CHECK();
        gram_reduce_kernel<TA><<<unsigned(std::min(kMaxGroups / 2, int64_t(m) * ((n + 31) / 32))), 256, 0, s>>>(
            m, n, cnt, part, ldp, S, lds, symmetric ? 1 : 0, s0 > 0 ? 1 : 0);
        LAUNCH_CHECK();
    }
}

template void gram_product<float, float>(chf_ctx*, const float*, int64_t, const float*, int64_t, int64_t, int, int,
                                         double*, int64_t, hipStream_t);
template void gram_product<double, double>(chf_ctx*, const double*, int64_t, const double*, int64_t, int64_t, int, int,
                                           double*, int64_t, hipStream_t);
template void gram_product<float, double>(chf_ctx*, const float*, int64_t, const float*, int64_t, int64_t, int, int,
                                          double*, int64_t, hipStream_t);

}  // namespace chf
