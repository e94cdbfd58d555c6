// Learned correction of the initial SCF density on gfx950: a 3-D U-Net
// (4 levels, 32 channels) trained and evaluated by hand-written kernels.
//
// The paper starts each SCF from a superposition of atomic densities; this
// network maps that superposition (on cubic patches of the real-space grid)
// to a correction towards the converged density, learned from densities the
// method itself produces.  Convolutions are implicit GEMMs on the BF16 MFMA
// (v_mfma_f32_16x16x16bf16_1k) with FP32 accumulation: BF16 weights and
// activations, FP32 master weights, pre-activations and gradients.
//
// Layout: activations channels-last [D][H][W][C]; weights [C_out][tap][C_in]
// with tap = (dz * 3 + dy) * 3 + dx (a single tap for the 1^3 output layer).
// Channel counts are padded to multiples of 4 (inputs) and 16 (outputs).
// Networks of 32 channels (the trained configuration) take the tiled kernels
// (conv3_kernel and the ones after it), other widths the direct ones.
//
// Architecture (f = SiLU, up = nearest x2, [.,.] = channel concat):
//   e1 = f(c1b(f(c1a(x))))                      S^3
//   e2 = f(c2b(f(c2a(f(d1(e1))))))              (S/2)^3, d* stride 2
//   e3 = f(c3b(f(c3a(f(d2(e2))))))              (S/4)^3
//   b  = f(c4b(f(c4a(f(d3(e3))))))              (S/8)^3
//   g3 = f(c5b(f(c5a([f(u3(up(b))), e3]))))
//   g2 = f(c6b(f(c6a([f(u2(up(g3))), e2]))))
//   g1 = f(c7b(f(c7a([f(u1(up(g2))), e1]))))
//   y  = out(g1)                                 1^3 conv, no activation
#include <cmath>
#include <cstring>
#include <memory>
#include <vector>

#include "internal.hpp"
#include "kernels.hpp"

namespace chf {
namespace dn {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned short bf16;

__device__ __host__ inline bf16 to_bf16(float f) {
    // round to nearest even
    const uint32_t u = __builtin_bit_cast(uint32_t, f);
    if ((u & 0x7f800000u) == 0x7f800000u) return bf16(u >> 16);   // inf / nan
    const uint32_t r = u + 0x7fffu + ((u >> 16) & 1u);
    return bf16(r >> 16);
}
__device__ __host__ inline float from_bf16(bf16 b) {
    return __builtin_bit_cast(float, uint32_t(b) << 16);
}

__device__ inline float silu(float z) { return z / (1.0f + expf(-z)); }
__device__ inline float silu_grad(float z) {
    const float s = 1.0f / (1.0f + expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

struct Layer {
    int cin, cout;          // real channel counts
    int cin_p, cout_p;      // padded: multiple of 4 / 16
    int k, stride;          // kernel edge (3 or 1), stride (1 or 2)
    int64_t w_off, b_off;   // offsets into the master parameter vector (padded layout)
    bool act;
};

// ---------------------------------------------------------------------------
// forward: out[p][co] = b[co] + sum_{tap, ci} W[co][tap][ci] in[stride p + t - pad][ci]
// M = co (padded to 16 per block, 2 blocks max), N = output positions (16 per
// wave, 64 per workgroup), K = tap x ci in chunks of 16.  Input channels come
// from one or two tensors (channel concat).
// MFMA 16x16x16 bf16 operands: A(i, k) at lane i + 16 (k / 4), element k % 4;
// B(k, j) at lane j + 16 (k / 4), element k % 4; D(i, j): lane j + 16 (i / 4),
// register i % 4.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) conv_fwd_kernel(int Di, int Do, int cin0, int cin1, int cin_p, int cout, int cout_p,
                                                       int k, int stride, const bf16* __restrict__ in0,
                                                       const bf16* __restrict__ in1, const bf16* __restrict__ Wb,
                                                       const float* __restrict__ bias, float* __restrict__ zout,
                                                       bf16* __restrict__ yout, int act) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t npos = int64_t(Do) * Do * Do;
    const int64_t p0 = (int64_t(blockIdx.x) * 4 + wave) * 16;
    const int j = lane & 15, kq = lane >> 4;
    const int64_t p = p0 + j;
    const bool pok = p < npos;
    const int pz = pok ? int(p / (int64_t(Do) * Do)) : 0, py = pok ? int((p / Do) % Do) : 0, px = pok ? int(p % Do) : 0;
    const int pad = k / 2, ntap = k * k * k;
    const int K = ntap * cin_p;
    const int nrb = cout_p / 16;
    f4 acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    for (int kc = 0; kc < K; kc += 16) {
        const int kk = kc + 4 * kq;           // first of this lane's 4 k values
        s4 b = {0, 0, 0, 0};
        if (kk < K && pok) {
            const int tap = kk / cin_p, ci = kk % cin_p;
            const int dz = tap / (k * k), dy = (tap / k) % k, dx = tap % k;
            const int z = stride * pz + dz - pad, y = stride * py + dy - pad, x = stride * px + dx - pad;
            if (z >= 0 && z < Di && y >= 0 && y < Di && x >= 0 && x < Di) {
                const int64_t q = (int64_t(z) * Di + y) * Di + x;
                const bf16* src = ci < cin0 ? in0 + q * cin0 + ci : in1 + q * cin1 + (ci - cin0);
                if (ci < cin0 + cin1) b = *reinterpret_cast<const s4*>(src);
            }
        }
        for (int rb = 0; rb < nrb; ++rb) {
            s4 a = {0, 0, 0, 0};
            const int co = rb * 16 + j;
            if (kk < K) a = *reinterpret_cast<const s4*>(Wb + (int64_t(co) * ntap) * cin_p + kk);
            acc[rb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[rb], 0, 0, 0);
        }
    }
    if (!pok) return;
    for (int rb = 0; rb < nrb; ++rb)
        for (int v = 0; v < 4; ++v) {
            const int co = rb * 16 + 4 * kq + v;
            if (co >= cout) continue;
            const float z = acc[rb][v] + bias[co];
            zout[p * cout + co] = z;
            yout[p * cout + co] = to_bf16(act ? silu(z) : z);
        }
}

// ---------------------------------------------------------------------------
// Tiled 3^3 convolutions of 32-channel networks.
//
// A workgroup of 4 waves computes a tile of 8 x TY x TZ positions and all
// result channels.  The input cells of the tile and its rim are staged in LDS
// once and used by all 27 taps; a wave takes NT groups of 16 positions (8 x 2)
// and keeps their NT x MB accumulators in registers, so a weight operand read
// (packed in operand order, 16 bytes per lane and tap) feeds 2 NT MFMAs.  The
// operand values and the order of the MFMAs of a result (taps, then channels
// in steps of 16) are those of conv_fwd_kernel and conv_bwd_data_kernel, so
// the results are the same bits.
//
// The direct kernels gathered each operand from memory, tap by tap, with the
// index arithmetic in every step, and were bound by that chain.  us per layer,
// before -> now: 32 -> 32 channels at 96^3 (49 GFLOP, 226 MB) 1267 -> 103, 64 ->
// 32 there 2508 -> 239, 32 -> 32 at 48^3 191 -> 27, at 24^3 and below 65 -> 13;
// input gradient at 64^3 287 -> 37 with the activation's derivative.  Now the
// large layers sit between the matrix cores (476 TFLOP/s) and memory (2.2
// TB/s), the small ones on the latency of staging and 27 dependent taps.
//
// LDS layout [half of 32 channels][kq][cell][8]: the 8 values that lane group
// kq of an operand holds for the half's two 16-channel steps (channels
// 16 c + 4 kq + e), so one 16-byte read serves both and the 8 cells of an x line
// are 128 consecutive bytes.
// ---------------------------------------------------------------------------
enum { kPlain, kUpsample, kDilate };        // where an input cell comes from
enum { kForward, kGradAct, kGradRaw };      // what becomes of a result

typedef short s8 __attribute__((ext_vector_type(8)));

struct Conv3 {
    int Din;                 // edge of the input as the convolution sees it
    int Dsrc;                // edge of the stored input (upsampled: Din / 2; dilated: (Din + 1) / 2)
    int Dout;
    const bf16* in0;         // channels 0..31 (dZ for gradients)
    const bf16* in1;         // channels 32..63, or null
    const s8* w;             // packed weights [tap][half][row block][lane]
    // forward
    const float* bias;
    float* z;
    bf16* y;
    // gradients
    const float* add;        // added to the result before the activation's derivative, or null
    const float* zprev;      // pre-activations of the layer that produced the input
    bf16* dzb;               // its dZ
    float* raw;              // kGradRaw: result; kGradAct with 64 channels: the second half
    float* bias_part;        // [workgroup][32] sums of dZ
};

// Packed weights of all layers in one launch (blockIdx.y = layer): value i of
// the 8 of (tap, half, row block, lane).  Forward: rows = output channels;
// transposed: rows = input channels, columns = output channels.  The first
// layer (1 input channel, stored as [cell][4] with three zeros) has 4 taps to an
// MFMA step and 4 values to a lane instead.
constexpr int kPackHalf = 27 * 2 * 64;      // s8 of 32 input channels
struct PackTable {
    int64_t w_off[20];
    int halves[20];          // 0: the first layer
};

__global__ void pack_kernel(PackTable tab, int transposed, const float* __restrict__ params, s8* __restrict__ packed) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x, layer = blockIdx.y;
    const int n_half = tab.halves[layer];
    const float* W = params + tab.w_off[layer];
    s8* out = packed + int64_t(layer) * 2 * kPackHalf;
    const int lane = idx & 63, j = lane & 15, kq = lane >> 4;
    if (n_half == 0) {
        if (transposed || idx >= 7 * 2 * 64) return;
        const int rb = (idx >> 6) & 1, tap = (idx >> 7) * 4 + kq;
        s4 v = {0, 0, 0, 0};
        if (tap < 27)
            for (int e = 0; e < 4; ++e) v[e] = short(to_bf16(W[(int64_t(rb * 16 + j) * 27 + tap) * 4 + e]));
        reinterpret_cast<s4*>(out)[idx] = v;
        return;
    }
    if (idx >= n_half * kPackHalf) return;
    const int cin = 32 * n_half;
    s8 v;
    if (!transposed) {
        const int rb = (idx >> 6) & 1, h = (idx >> 7) % n_half, tap = (idx >> 7) / n_half;
        for (int i = 0; i < 8; ++i)
            v[i] = short(to_bf16(W[(int64_t(rb * 16 + j) * 27 + tap) * cin + h * 32 + (i >> 2) * 16 + 4 * kq + (i & 3)]));
    } else {
        const int rb = (idx >> 6) % (2 * n_half), tap = (idx >> 6) / (2 * n_half);
        for (int i = 0; i < 8; ++i)
            v[i] = short(to_bf16(W[(int64_t((i >> 2) * 16 + 4 * kq + (i & 3)) * 27 + tap) * cin + rb * 16 + j]));
    }
    out[idx] = v;
}

// 32 channel sums of a workgroup of NW waves: lane (j, kq) holds the sums of
// channels rb 16 + 4 kq + v over its positions
template <int NW>
__device__ inline void channel_sums(f4 s0, f4 s1, float* sh, float* out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int m = 1; m < 16; m *= 2) {
            s0[v] += __shfl_xor(s0[v], m, 64);
            s1[v] += __shfl_xor(s1[v], m, 64);
        }
    if ((lane & 15) == 0)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            sh[wave * 32 + 4 * (lane >> 4) + v] = s0[v];
            sh[wave * 32 + 16 + 4 * (lane >> 4) + v] = s1[v];
        }
    __syncthreads();
    if (threadIdx.x < 32) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += sh[w * 32 + threadIdx.x];
        out[threadIdx.x] = t;
    }
}

template <int H, int STRIDE, int TY, int TZ, int LOAD, int MB, int EPI>
__global__ void __launch_bounds__(256) conv3_kernel(Conv3 a) {
    constexpr int IX = 7 * STRIDE + 3, IY = (TY - 1) * STRIDE + 3, IZ = (TZ - 1) * STRIDE + 3;
    constexpr int CELLS = IX * IY * IZ;
    constexpr int NT = TY * TZ / 8;               // groups of 16 positions per wave
    constexpr bool back = EPI != kForward;
    __shared__ s8 tile[H * 4 * CELLS];
    __shared__ float sums[4 * 32];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int j = lane & 15, kq = lane >> 4;
    const int nx = (a.Dout + 7) / 8, ny = (a.Dout + TY - 1) / TY;
    const int bx = int(blockIdx.x) % nx, by = int(blockIdx.x) / nx % ny, bz = int(blockIdx.x) / (nx * ny);
    const int ox0 = bx * 8, oy0 = by * TY, oz0 = bz * TZ;

    for (int i = t; i < CELLS * 4 * H; i += 256) {
        const int cell = i / (4 * H), part = i % (4 * H), h = part >> 2, q = part & 3;
        int x = ox0 * STRIDE - 1 + cell % IX, y = oy0 * STRIDE - 1 + cell / IX % IY, z = oz0 * STRIDE - 1 + cell / (IX * IY);
        bool ok = x >= 0 && y >= 0 && z >= 0 && x < a.Din && y < a.Din && z < a.Din;
        if (LOAD == kDilate) ok = ok && !((x | y | z) & 1);
        if (LOAD != kPlain) x >>= 1, y >>= 1, z >>= 1;
        s8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (ok) v = *reinterpret_cast<const s8*>((h ? a.in1 : a.in0) + ((int64_t(z) * a.Dsrc + y) * a.Dsrc + x) * 32 + q * 8);
        // channels 8 q .. 8 q + 7: step q / 2, lane groups 2 (q % 2) and the next
        s4* const d = reinterpret_cast<s4*>(tile + (h * 4 + 2 * (q & 1)) * CELLS + cell) + (q >> 1);
        d[0] = s4{v[0], v[1], v[2], v[3]};
        d[2 * CELLS] = s4{v[4], v[5], v[6], v[7]};
    }
    __syncthreads();

    int at[NT];                                   // cell of this lane's position for tap offset 0
    int ox[NT], oy[NT], oz[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int g = wave * NT + n, lx = j & 7, ly = (g % (TY / 2)) * 2 + (j >> 3), lz = g / (TY / 2);
        ox[n] = ox0 + lx, oy[n] = oy0 + ly, oz[n] = oz0 + lz;
        at[n] = kq * CELLS + (lz * STRIDE * IY + ly * STRIDE) * IX + lx * STRIDE;
    }
    f4 acc[NT][MB];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) acc[n][rb] = f4{0, 0, 0, 0};
#pragma unroll 3
    for (int tap = 0; tap < 27; ++tap) {
        const int dz = tap / 9, dy = tap / 3 % 3, dx = tap % 3;
        const int off = back ? ((2 - dz) * IY + (2 - dy)) * IX + (2 - dx) : (dz * IY + dy) * IX + dx;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            s8 w[MB];
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) w[rb] = a.w[((tap * H + h) * MB + rb) * 64 + lane];
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const s8 b = tile[h * 4 * CELLS + at[n] + off];
                const s4 b0 = {b[0], b[1], b[2], b[3]}, b1 = {b[4], b[5], b[6], b[7]};
#pragma unroll
                for (int rb = 0; rb < MB; ++rb) {
                    const s4 w0 = {w[rb][0], w[rb][1], w[rb][2], w[rb][3]}, w1 = {w[rb][4], w[rb][5], w[rb][6], w[rb][7]};
                    acc[n][rb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w0, b0, acc[n][rb], 0, 0, 0);
                    acc[n][rb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w1, b1, acc[n][rb], 0, 0, 0);
                }
            }
        }
    }
    f4 bs[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        if (ox[n] >= a.Dout || oy[n] >= a.Dout || oz[n] >= a.Dout) continue;
        const int64_t at0 = ((int64_t(oz[n]) * a.Dout + oy[n]) * a.Dout + ox[n]) * 32 + 4 * kq;
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) {
            const int64_t o = at0 + (rb & 1) * 16;
            f4 g = acc[n][rb];
            if constexpr (EPI == kForward) {
                s4 yb;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    g[v] += a.bias[rb * 16 + 4 * kq + v];
                    yb[v] = short(to_bf16(silu(g[v])));
                }
                *reinterpret_cast<f4*>(a.z + o) = g;
                *reinterpret_cast<s4*>(a.y + o) = yb;
            } else if (EPI == kGradRaw || rb >= 2) {
                *reinterpret_cast<f4*>(a.raw + o) = g;
            } else {
                if (a.add) {
                    const f4 e = *reinterpret_cast<const f4*>(a.add + o);
#pragma unroll
                    for (int v = 0; v < 4; ++v) g[v] += e[v];
                }
                const f4 zp = *reinterpret_cast<const f4*>(a.zprev + o);
                s4 yb;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    g[v] *= silu_grad(zp[v]);
                    bs[rb][v] += g[v];
                    yb[v] = short(to_bf16(g[v]));
                }
                *reinterpret_cast<s4*>(a.dzb + o) = yb;
            }
        }
    }
    if constexpr (EPI == kGradAct) channel_sums<4>(bs[0], bs[1], sums, a.bias_part + int64_t(blockIdx.x) * 32);
}

// First layer: K runs over (tap, 4 channels), 4 taps to an MFMA step.
__global__ void __launch_bounds__(256) conv_in_kernel(int D, const s4* __restrict__ in, const s4* __restrict__ w,
                                                      const float* __restrict__ bias, float* __restrict__ z,
                                                      bf16* __restrict__ y) {
    constexpr int IX = 10, IY = 10, IZ = 6, CELLS = IX * IY * IZ;
    __shared__ s4 tile[CELLS];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, j = lane & 15, kq = lane >> 4;
    const int nx = (D + 7) / 8;
    const int ox0 = int(blockIdx.x) % nx * 8, oy0 = int(blockIdx.x) / nx % nx * 8, oz0 = int(blockIdx.x) / (nx * nx) * 4;
    for (int i = t; i < CELLS; i += 256) {
        const int x1 = ox0 - 1 + i % IX, y1 = oy0 - 1 + i / IX % IY, z1 = oz0 - 1 + i / (IX * IY);
        const bool ok = x1 >= 0 && y1 >= 0 && z1 >= 0 && x1 < D && y1 < D && z1 < D;
        tile[i] = ok ? in[(int64_t(z1) * D + y1) * D + x1] : s4{0, 0, 0, 0};
    }
    __syncthreads();
    f4 acc[4][2];
#pragma unroll
    for (int n = 0; n < 4; ++n) acc[n][0] = acc[n][1] = f4{0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        const int tap = 4 * c + kq;
        const int ta = min(tap, 26), off = (ta / 9 * IY + ta / 3 % 3) * IX + ta % 3;
        const s4 w0 = w[c * 128 + lane], w1 = w[c * 128 + 64 + lane];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int cell = (wave * IY + 2 * n + (j >> 3)) * IX + (j & 7);
            const s4 b = tap < 27 ? tile[cell + off] : s4{0, 0, 0, 0};
            acc[n][0] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w0, b, acc[n][0], 0, 0, 0);
            acc[n][1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w1, b, acc[n][1], 0, 0, 0);
        }
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int ox = ox0 + (j & 7), oy = oy0 + 2 * n + (j >> 3), oz = oz0 + wave;
        if (ox >= D || oy >= D || oz >= D) continue;
        const int64_t at0 = ((int64_t(oz) * D + oy) * D + ox) * 32 + 4 * kq;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
            f4 g = acc[n][rb];
            s4 yb;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                g[v] += bias[rb * 16 + 4 * kq + v];
                yb[v] = short(to_bf16(silu(g[v])));
            }
            *reinterpret_cast<f4*>(z + at0 + rb * 16) = g;
            *reinterpret_cast<s4*>(y + at0 + rb * 16) = yb;
        }
    }
}

// output layer (1^3, 32 -> 1, no activation): 64 positions per wave
__global__ void __launch_bounds__(256) conv_out_kernel(int64_t n, const bf16* __restrict__ in, const float* __restrict__ W,
                                                       const float* __restrict__ bias, float* __restrict__ y) {
    const int lane = threadIdx.x & 63, j = lane & 15, kq = lane >> 4;
    const int64_t p0 = (int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6)) * 64;
    s4 w[2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) w[c][e] = short(to_bf16(W[j * 32 + c * 16 + 4 * kq + e]));
    s4 b[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int64_t p = p0 + i * 16 + j;
            b[i][c] = p < n ? *reinterpret_cast<const s4*>(in + p * 32 + c * 16 + 4 * kq) : s4{0, 0, 0, 0};
        }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f4 acc = {0, 0, 0, 0};
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[0], b[i][0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[1], b[i][1], acc, 0, 0, 0);
        if (kq == 0 && p0 + i * 16 + j < n) y[p0 + i * 16 + j] = acc[0] + bias[0];
    }
}

// ---------------------------------------------------------------------------
// Weight gradients of the tiled kernels: dW[co][tap][ci] = sum_p dZ[p][co]
// X[stride p + tap - 1][ci].  M = co, N = (tap, ci), K = positions.
//
// A workgroup stages the input cells and dZ of a tile in LDS, [cell][32] and
// [position][32] as they lie in memory, and reads both operands (4 consecutive
// positions of one channel per lane) with transposing LDS reads.  Wave w takes
// taps w, w + 4, ...: up to 7 taps x 2 channel blocks x 2 row blocks of
// accumulators, 28 MFMAs per 16 positions for 16 operand reads.  A workgroup
// walks its share of the tiles and writes one partial; the partials are added
// in order.  The direct kernel gathered both operands 2 bytes at a time: 1560 ->
// 57 us at 64^3 with 32 channels (18 GFLOP), 300 -> 16 at 16^3; the bias sums,
// one workgroup per channel, took 340 us and now ride with the kernel that
// forms dZ.
// ---------------------------------------------------------------------------
__device__ inline s4 tr_read(const bf16* p) {
    typedef __attribute__((address_space(3))) s4 lds_s4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p));
}

struct WGrad {
    int Din, Dsrc, Dout;
    const bf16* in0;         // blockIdx.y = 0: channels 0..31
    const bf16* in1;         // blockIdx.y = 1: channels 32..63
    const bf16* dzb;
    f4* part;                // [half][workgroup][27 taps][2 channel blocks][2 row blocks][lane]
};
constexpr int kWgradPart = 27 * 2 * 2 * 64;      // f4 of one workgroup

template <int STRIDE, int TY, int TZ, int LOAD>
__global__ void __launch_bounds__(256) wgrad3_kernel(WGrad a) {
    constexpr int IX = 7 * STRIDE + 3, IY = (TY - 1) * STRIDE + 3, IZ = (TZ - 1) * STRIDE + 3;
    constexpr int CELLS = IX * IY * IZ, POS = 8 * TY * TZ;
    __shared__ __align__(16) bf16 xt[CELLS * 32];
    __shared__ __align__(16) bf16 zt[POS * 32];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const bf16* in = blockIdx.y ? a.in1 : a.in0;
    const int nx = (a.Dout + 7) / 8, ny = (a.Dout + TY - 1) / TY, nz = (a.Dout + TZ - 1) / TZ;
    const int tiles = nx * ny * nz;
    // transposing reads: lane 4 r + q of a group of 16 addresses channels 4 q.. of
    // the group's row r; the group holds positions 4 (lane / 16) + r of the step
    const int r = (lane & 15) >> 2, q = lane & 3, pos = 4 * (lane >> 4) + r;
    const int px = pos & 7, py = pos >> 3;        // within the step's 8 x 2 positions
    f4 acc[7][2][2];
#pragma unroll
    for (int i = 0; i < 7; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[i][c][0] = acc[i][c][1] = f4{0, 0, 0, 0};
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int ox0 = tile % nx * 8, oy0 = tile / nx % ny * TY, oz0 = tile / (nx * ny) * TZ;
        __syncthreads();
        for (int i = t; i < CELLS * 4; i += 256) {
            const int cell = i >> 2;
            int x = ox0 * STRIDE - 1 + cell % IX, y = oy0 * STRIDE - 1 + cell / IX % IY, z = oz0 * STRIDE - 1 + cell / (IX * IY);
            const bool ok = x >= 0 && y >= 0 && z >= 0 && x < a.Din && y < a.Din && z < a.Din;
            if (LOAD == kUpsample) x >>= 1, y >>= 1, z >>= 1;
            s8 v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (ok) v = *reinterpret_cast<const s8*>(in + ((int64_t(z) * a.Dsrc + y) * a.Dsrc + x) * 32 + (i & 3) * 8);
            *reinterpret_cast<s8*>(xt + i * 8) = v;
        }
        for (int i = t; i < POS * 4; i += 256) {
            const int p = i >> 2, x = ox0 + (p & 7), y = oy0 + (p >> 3) % TY, z = oz0 + (p >> 3) / TY;
            s8 v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (x < a.Dout && y < a.Dout && z < a.Dout)
                v = *reinterpret_cast<const s8*>(a.dzb + ((int64_t(z) * a.Dout + y) * a.Dout + x) * 32 + (i & 3) * 8);
            *reinterpret_cast<s8*>(zt + i * 8) = v;
        }
        __syncthreads();
#pragma unroll 2
        for (int k = 0; k < POS / 16; ++k) {
            const int ly = (k % (TY / 2)) * 2 + py, lz = k / (TY / 2);
            const bf16* zp = zt + (k * 16 + pos) * 32 + q * 4;
            const s4 w0 = tr_read(zp), w1 = tr_read(zp + 16);
            const bf16* xp = xt + ((lz * STRIDE * IY + ly * STRIDE) * IX + px * STRIDE) * 32 + q * 4;
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                const int tap = wave + 4 * i;
                if (tap >= 27) continue;
                const int off = ((tap / 9) * IY + tap / 3 % 3) * IX + tap % 3;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const s4 b = tr_read(xp + off * 32 + c * 16);
                    acc[i][c][0] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w0, b, acc[i][c][0], 0, 0, 0);
                    acc[i][c][1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w1, b, acc[i][c][1], 0, 0, 0);
                }
            }
        }
    }
    f4* part = a.part + (int64_t(blockIdx.y) * gridDim.x + blockIdx.x) * kWgradPart;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const int tap = wave + 4 * i;
        if (tap >= 27) continue;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) part[((tap * 2 + c) * 2 + rb) * 64 + lane] = acc[i][c][rb];
    }
}

// gw[co][tap][ci] += sum of the partials, gb[co] += sum of the bias partials.
// 64 f4 elements x 4 slices of the partials per workgroup; the last workgroup
// of a launch does the bias.
__global__ void __launch_bounds__(256) wgrad3_reduce_kernel(int n_half, int n_part, const f4* __restrict__ part,
                                                            float* __restrict__ gw, int n_bias,
                                                            const float* __restrict__ bias_part, float* __restrict__ gb) {
    __shared__ f4 sh[256];
    const int t = threadIdx.x, e = t & 63, sl = t >> 6;
    const int groups = n_half * (kWgradPart / 64);
    if (int(blockIdx.x) == groups) {
        float* shf = reinterpret_cast<float*>(sh);
        float s = 0.0f;
#pragma unroll 16
        for (int p = t >> 5; p < n_bias; p += 8) s += bias_part[int64_t(p) * 32 + (t & 31)];
        shf[t] = s;
        __syncthreads();
        if (t >= 32) return;
        for (int w = 1; w < 8; ++w) s += shf[w * 32 + t];
        gb[t] += s;
        return;
    }
    const int h = int(blockIdx.x) / (kWgradPart / 64), blk = int(blockIdx.x) % (kWgradPart / 64);
    const f4* src = part + int64_t(h) * n_part * kWgradPart + blk * 64 + e;
    f4 s = {0, 0, 0, 0};
#pragma unroll 8
    for (int p = sl; p < n_part; p += 4) {
        const f4 v = src[int64_t(p) * kWgradPart];
        for (int i = 0; i < 4; ++i) s[i] += v[i];
    }
    sh[t] = s;
    __syncthreads();
    if (sl) return;
    for (int w = 1; w < 4; ++w)
        for (int i = 0; i < 4; ++i) s[i] += sh[w * 64 + e][i];
    const int rb = blk & 1, c = (blk >> 1) & 1, tap = blk >> 2;
    const int ci = h * 32 + c * 16 + (e & 15);
    for (int i = 0; i < 4; ++i) gw[(int64_t(rb * 16 + 4 * (e >> 4) + i) * 27 + tap) * (32 * n_half) + ci] += s[i];
}

// weight gradient of the first layer: dW[co][tap] = sum_p dZ[p][co] x[p + tap - 1],
// N = 27 taps, one 16-position step per wave at a time; partials [workgroup][2 tap
// blocks][2 row blocks][lane]
__global__ void __launch_bounds__(256) wgrad_in_kernel(int D, const bf16* __restrict__ in, const bf16* __restrict__ dzb,
                                                       f4* __restrict__ part) {
    constexpr int IX = 10, IY = 10, IZ = 6, CELLS = IX * IY * IZ;
    __shared__ bf16 xt[CELLS];
    __shared__ __align__(16) bf16 zt[256 * 32];
    __shared__ f4 sh[4][4][64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int j = lane & 15, r = j >> 2, q = lane & 3, kq = lane >> 4;
    const int nx = (D + 7) / 8, nz = (D + 3) / 4, tiles = nx * nx * nz;
    int off[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int tap = min(26, c * 16 + j);
        off[c] = (tap / 9 * IY + tap / 3 % 3) * IX + tap % 3;
    }
    f4 acc[2][2];
    acc[0][0] = acc[0][1] = acc[1][0] = acc[1][1] = f4{0, 0, 0, 0};
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int ox0 = tile % nx * 8, oy0 = tile / nx % nx * 8, oz0 = tile / (nx * nx) * 4;
        __syncthreads();
        for (int i = t; i < CELLS; i += 256) {
            const int x = ox0 - 1 + i % IX, y = oy0 - 1 + i / IX % IY, z = oz0 - 1 + i / (IX * IY);
            const bool ok = x >= 0 && y >= 0 && z >= 0 && x < D && y < D && z < D;
            xt[i] = ok ? in[((int64_t(z) * D + y) * D + x) * 4] : bf16(0);
        }
        for (int i = t; i < 1024; i += 256) {
            const int p = i >> 2, x = ox0 + (p & 7), y = oy0 + ((p >> 3) & 7), z = oz0 + (p >> 6);
            s8 v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (x < D && y < D && z < D)
                v = *reinterpret_cast<const s8*>(dzb + ((int64_t(z) * D + y) * D + x) * 32 + (i & 3) * 8);
            *reinterpret_cast<s8*>(zt + i * 8) = v;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {            // 8 x 2 positions: z line `wave`, y pair k
            const bf16* zp = zt + ((wave * 4 + k) * 16 + 4 * kq + r) * 32 + q * 4;
            const s4 w0 = tr_read(zp), w1 = tr_read(zp + 16);
            const int cell = (wave * IY + 2 * k + (kq >> 1)) * IX + 4 * (kq & 1);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                s4 b;
#pragma unroll
                for (int e = 0; e < 4; ++e) b[e] = short(xt[cell + e + off[c]]);
                acc[c][0] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w0, b, acc[c][0], 0, 0, 0);
                acc[c][1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w1, b, acc[c][1], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) sh[wave][i][lane] = acc[i >> 1][i & 1];
    __syncthreads();
    f4 s = sh[0][wave][lane];
    for (int w = 1; w < 4; ++w)
        for (int v = 0; v < 4; ++v) s[v] += sh[w][wave][lane][v];
    part[(int64_t(blockIdx.x) * 4 + wave) * 64 + lane] = s;
}

// first layer: gw[co][tap][0] and gb from the partials; one workgroup per 64 f4, one more for the bias
__global__ void __launch_bounds__(256) wgrad_in_reduce_kernel(int n_part, const f4* __restrict__ part, float* __restrict__ gw,
                                                              int n_bias, const float* __restrict__ bias_part,
                                                              float* __restrict__ gb) {
    __shared__ f4 sh[256];
    const int t = threadIdx.x, e = t & 63, sl = t >> 6;
    f4 s = {0, 0, 0, 0};
    if (blockIdx.x == 4) {
        float* shf = reinterpret_cast<float*>(sh);
        float b = 0.0f;
#pragma unroll 16
        for (int p = t >> 5; p < n_bias; p += 8) b += bias_part[int64_t(p) * 32 + (t & 31)];
        shf[t] = b;
        __syncthreads();
        if (t >= 32) return;
        for (int w = 1; w < 8; ++w) b += shf[w * 32 + t];
        gb[t] += b;
        return;
    }
    const int c = int(blockIdx.x) >> 1, rb = int(blockIdx.x) & 1;
#pragma unroll 8
    for (int p = sl; p < n_part; p += 4) {
        const f4 v = part[(int64_t(p) * 4 + blockIdx.x) * 64 + e];
        for (int i = 0; i < 4; ++i) s[i] += v[i];
    }
    sh[t] = s;
    __syncthreads();
    if (sl) return;
    for (int w = 1; w < 4; ++w)
        for (int i = 0; i < 4; ++i) s[i] += sh[w * 64 + e][i];
    const int tap = c * 16 + (e & 15);
    if (tap < 27)
        for (int i = 0; i < 4; ++i) gw[(int64_t(rb * 16 + 4 * (e >> 4) + i) * 27 + tap) * 4] += s[i];
}

// Backward of the output layer and the activation before it: dZ of the layer
// that made x (z: its pre-activations), and per workgroup 32 sums of that dZ, 32
// of dW_out[ci] = sum_p dy[p] x[p][ci] (both rounded to BF16) and the sum of dy.
constexpr int kOutSums = 65;
__global__ void __launch_bounds__(256) out_back_kernel(int64_t n, const float* __restrict__ dy, const float* __restrict__ W,
                                                       const bf16* __restrict__ x, const float* __restrict__ z,
                                                       bf16* __restrict__ dzb, float* __restrict__ bias_part,
                                                       float* __restrict__ out_part) {
    __shared__ float sh[256][9];
    const int t = threadIdx.x, c0 = (t & 7) * 4;          // this thread's 4 channels
    float w[4], sb[4] = {0, 0, 0, 0}, sw[4] = {0, 0, 0, 0}, sy = 0.0f;
    for (int v = 0; v < 4; ++v) w[v] = from_bf16(to_bf16(W[c0 + v]));
    for (int64_t p = int64_t(blockIdx.x) * 32 + (t >> 3); p < n; p += int64_t(gridDim.x) * 32) {
        const float d = dy[p], db = from_bf16(to_bf16(d));
        const s4 xv = *reinterpret_cast<const s4*>(x + p * 32 + c0);
        const f4 zv = *reinterpret_cast<const f4*>(z + p * 32 + c0);
        s4 o;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float g = db * w[v] * silu_grad(zv[v]);
            o[v] = short(to_bf16(g));
            sb[v] += g;
            sw[v] = fmaf(db, from_bf16(bf16(xv[v])), sw[v]);
        }
        *reinterpret_cast<s4*>(dzb + p * 32 + c0) = o;
        sy += d;
    }
    for (int v = 0; v < 4; ++v) sh[t][v] = sb[v], sh[t][4 + v] = sw[v];
    sh[t][8] = sy;
    __syncthreads();
    if (t >= 65) return;
    // channel c of the first 64 sums: threads (c / 4) + 8 k
    float s = 0.0f;
    const int c = t & 31, col = t < 64 ? (t >> 5) * 4 + (c & 3) : 8, first = t < 64 ? c >> 2 : 0;
    for (int k = 0; k < 32; ++k) s += sh[first + 8 * k][col];
    if (t < 32) bias_part[int64_t(blockIdx.x) * 32 + t] = s;
    else out_part[int64_t(blockIdx.x) * 33 + t - 32] = s;
}

__global__ void __launch_bounds__(256) out_reduce_kernel(int n_part, const float* __restrict__ part, float* __restrict__ gw,
                                                         float* __restrict__ gb) {
    __shared__ float sh[256];
    const int t = threadIdx.x, e = blockIdx.x;
    float s = 0.0f;
    for (int p = t; p < n_part; p += 256) s += part[int64_t(p) * 33 + e];
    sh[t] = s;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (t < st) sh[t] += sh[t + st];
        __syncthreads();
    }
    if (t == 0) (e < 32 ? gw[e] : gb[0]) += sh[0];
}

// gradient of an upsampled input summed over its 8 cells, times the derivative
// of the activation that made it; per workgroup 32 sums of the result
__global__ void __launch_bounds__(256) up_back_kernel(int Ds, const float* __restrict__ gd, const float* __restrict__ z,
                                                      bf16* __restrict__ dzb, float* __restrict__ bias_part) {
    __shared__ float sh[256][5];
    const int t = threadIdx.x, c0 = (t & 7) * 4, Dd = 2 * Ds;
    const int64_t n = int64_t(Ds) * Ds * Ds;
    f4 sb = {0, 0, 0, 0};
    for (int64_t p = int64_t(blockIdx.x) * 32 + (t >> 3); p < n; p += int64_t(gridDim.x) * 32) {
        const int pz = int(p / (int64_t(Ds) * Ds)), py = int((p / Ds) % Ds), px = int(p % Ds);
        f4 g = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const f4 e = *reinterpret_cast<const f4*>(
                gd + ((int64_t(2 * pz + (i >> 2)) * Dd + 2 * py + ((i >> 1) & 1)) * Dd + 2 * px + (i & 1)) * 32 + c0);
            for (int v = 0; v < 4; ++v) g[v] += e[v];
        }
        const f4 zv = *reinterpret_cast<const f4*>(z + p * 32 + c0);
        s4 o;
        for (int v = 0; v < 4; ++v) {
            g[v] *= silu_grad(zv[v]);
            sb[v] += g[v];
            o[v] = short(to_bf16(g[v]));
        }
        *reinterpret_cast<s4*>(dzb + p * 32 + c0) = o;
    }
    for (int v = 0; v < 4; ++v) sh[t][v] = sb[v];
    __syncthreads();
    if (t >= 32) return;
    float s = 0.0f;
    for (int k = 0; k < 32; ++k) s += sh[(t >> 2) + 8 * k][t & 3];
    bias_part[int64_t(blockIdx.x) * 32 + t] = s;
}

// dZ = dY * f'(Z) (or dY when no activation), kept in FP32 and BF16
__global__ void act_back_kernel(int64_t n, const float* __restrict__ dy, const float* __restrict__ z, int act,
                                float* __restrict__ dz, bf16* __restrict__ dzb) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = act ? dy[i] * silu_grad(z[i]) : dy[i];
    dz[i] = g;
    dzb[i] = to_bf16(g);
}

// transposed copy of the weights for the data gradient: WT[ci][tap][co] (co padded to 4)
__global__ void weight_t_kernel(int cout, int cout_p4, int ntap, int cin_p, const float* __restrict__ W, bf16* __restrict__ WT) {
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t total = int64_t(cin_p) * ntap * cout_p4;
    if (idx >= total) return;
    const int co = int(idx % cout_p4);
    const int tap = int((idx / cout_p4) % ntap);
    const int ci = int(idx / (int64_t(cout_p4) * ntap));
    WT[idx] = co < cout ? to_bf16(W[(int64_t(co) * ntap + tap) * cin_p + ci]) : bf16(0);
}

// data gradient: dX[q][ci] = sum_{tap, co} dZ[p][co] W[co][tap][ci] with
// stride p + tap - pad = q.  M = ci, N = input positions, K = tap x co.
__global__ void __launch_bounds__(256) conv_bwd_data_kernel(int Di, int Do, int cin, int cin_rows, int cout, int cout_p4, int k,
                                                            int stride, const bf16* __restrict__ dzb,
                                                            const bf16* __restrict__ WT, float* __restrict__ dx) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t npos = int64_t(Di) * Di * Di;
    const int64_t q0 = (int64_t(blockIdx.x) * 4 + wave) * 16;
    const int j = lane & 15, kq = lane >> 4;
    const int64_t q = q0 + j;
    const bool qok = q < npos;
    const int qz = qok ? int(q / (int64_t(Di) * Di)) : 0, qy = qok ? int((q / Di) % Di) : 0, qx = qok ? int(q % Di) : 0;
    const int pad = k / 2, ntap = k * k * k;
    const int K = ntap * cout_p4;
    const int nrb = (cin_rows + 15) / 16;
    f4 acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
    for (int kc = 0; kc < K; kc += 16) {
        const int kk = kc + 4 * kq;
        s4 b = {0, 0, 0, 0};
        int tap = 0;
        if (kk < K) tap = kk / cout_p4;
        const int co = kk % cout_p4;
        if (kk < K && qok) {
            const int dz = tap / (k * k), dy = (tap / k) % k, dx = tap % k;
            // output position p with stride p + d - pad = q
            const int nz = qz - dz + pad, ny = qy - dy + pad, nx = qx - dx + pad;
            if (nz >= 0 && ny >= 0 && nx >= 0 && nz % stride == 0 && ny % stride == 0 && nx % stride == 0) {
                const int z = nz / stride, y = ny / stride, x = nx / stride;
                if (z < Do && y < Do && x < Do) {
                    const int64_t p = (int64_t(z) * Do + y) * Do + x;
                    if (co + 3 < cout) {
                        b = *reinterpret_cast<const s4*>(dzb + p * cout + co);
                    } else {
                        for (int e = 0; e < 4; ++e) b[e] = co + e < cout ? short(dzb[p * cout + co + e]) : short(0);
                    }
                }
            }
        }
        for (int rb = 0; rb < nrb; ++rb) {
            s4 a = {0, 0, 0, 0};
            const int ci = rb * 16 + j;
            if (kk < K && ci < cin_rows) a = *reinterpret_cast<const s4*>(WT + (int64_t(ci) * ntap + tap) * cout_p4 + co);
            acc[rb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[rb], 0, 0, 0);
        }
    }
    if (!qok) return;
    for (int rb = 0; rb < nrb; ++rb)
        for (int v = 0; v < 4; ++v) {
            const int ci = rb * 16 + 4 * kq + v;
            if (ci < cin) dx[q * cin + ci] = acc[rb][v];
        }
}

// weight gradient partials: dW[co][tap][ci] = sum_p dZ[p][co] X[stride p + t - pad][ci]
// M = co, N = (tap, ci) columns (16 per wave), K = output positions (this
// workgroup's slice, 16 per step).
__global__ void __launch_bounds__(256) conv_bwd_weight_kernel(int Di, int Do, int cin0, int cin1, int cin_p, int cout,
                                                              int k, int stride, const bf16* __restrict__ dzb,
                                                              const bf16* __restrict__ in0, const bf16* __restrict__ in1,
                                                              int64_t pos_per_split, float* __restrict__ part) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, kq = lane >> 4;
    const int ntap = k * k * k, pad = k / 2;
    const int ncol = ntap * cin_p;
    const int col = (blockIdx.x * 4 + wave) * 16 + j;
    const bool cok = col < ncol;
    const int tap = cok ? col / cin_p : 0, ci = cok ? col % cin_p : 0;
    const int dz = tap / (k * k), dy = (tap / k) % k, dx = tap % k;
    const int64_t npos = int64_t(Do) * Do * Do;
    const int64_t pb = int64_t(blockIdx.y) * pos_per_split, pe = min(npos, pb + pos_per_split);
    const int nrb = (cout + 15) / 16;
    f4 acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    for (int64_t pc = pb; pc < pe; pc += 16) {
        s4 b = {0, 0, 0, 0};
        s4 a[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
        for (int e = 0; e < 4; ++e) {
            const int64_t p = pc + 4 * kq + e;
            if (p >= pe) continue;
            const int pz = int(p / (int64_t(Do) * Do)), py = int((p / Do) % Do), px = int(p % Do);
            if (cok && ci < cin0 + cin1) {
                const int z = stride * pz + dz - pad, y = stride * py + dy - pad, x = stride * px + dx - pad;
                if (z >= 0 && z < Di && y >= 0 && y < Di && x >= 0 && x < Di) {
                    const int64_t q = (int64_t(z) * Di + y) * Di + x;
                    b[e] = short(ci < cin0 ? in0[q * cin0 + ci] : in1[q * cin1 + ci - cin0]);
                }
            }
            for (int rb = 0; rb < nrb; ++rb) {
                const int co = rb * 16 + j;
                if (co < cout) a[rb][e] = short(dzb[p * cout + co]);
            }
        }
        for (int rb = 0; rb < nrb; ++rb) acc[rb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[rb], b, acc[rb], 0, 0, 0);
    }
    float* P = part + int64_t(blockIdx.y) * 32 * ncol;
    for (int rb = 0; rb < nrb; ++rb)
        for (int v = 0; v < 4; ++v) {
            const int co = rb * 16 + 4 * kq + v;
            if (co < cout && cok) P[int64_t(co) * ncol + col] = acc[rb][v];
        }
}

// grad[co][tap][ci] += sum over splits (fixed order); db[co] += sum_p dZ[p][co]
__global__ void wgrad_reduce_kernel(int cout, int ncol, int nsplit, const float* __restrict__ part, float* __restrict__ gw) {
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= int64_t(cout) * ncol) return;
    float s = 0.0f;
    for (int sp = 0; sp < nsplit; ++sp) s += part[int64_t(sp) * 32 * ncol + idx];
    gw[idx] += s;
}

__global__ void __launch_bounds__(256) bgrad_kernel(int64_t npos, int cout, const float* __restrict__ dz, float* __restrict__ gb) {
    const int co = blockIdx.x;
    __shared__ float sh[256];
    float s = 0.0f;
    for (int64_t p = threadIdx.x; p < npos; p += 256) s += dz[p * cout + co];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) gb[co] += sh[0];
}

__global__ void upsample_kernel(int Ds, int c, const bf16* __restrict__ src, bf16* __restrict__ dst) {
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int Dd = 2 * Ds;
    if (idx >= int64_t(Dd) * Dd * Dd * c) return;
    const int ch = int(idx % c);
    const int64_t q = idx / c;
    const int z = int(q / (int64_t(Dd) * Dd)), y = int((q / Dd) % Dd), x = int(q % Dd);
    dst[idx] = src[((int64_t(z / 2) * Ds + y / 2) * Ds + x / 2) * c + ch];
}

__global__ void upsample_back_kernel(int Ds, int c, const float* __restrict__ gd, float* __restrict__ gs) {
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= int64_t(Ds) * Ds * Ds * c) return;
    const int ch = int(idx % c);
    const int64_t q = idx / c;
    const int z = int(q / (int64_t(Ds) * Ds)), y = int((q / Ds) % Ds), x = int(q % Ds);
    const int Dd = 2 * Ds;
    float s = 0.0f;
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b)
            for (int e = 0; e < 2; ++e) s += gd[((int64_t(2 * z + a) * Dd + 2 * y + b) * Dd + 2 * x + e) * c + ch];
    gs[idx] = s;
}

// out = a (+ b) with channel split: take channels [c0, c0 + cn) of a [n][ca]
__global__ void slice_add_kernel(int64_t n, int ca, int c0, int cn, const float* __restrict__ a, const float* __restrict__ b,
                                 float* __restrict__ out) {
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= n * cn) return;
    const int64_t p = idx / cn;
    const int ch = int(idx % cn);
    out[idx] = a[p * ca + c0 + ch] + (b ? b[idx] : 0.0f);
}

__global__ void input_kernel(int64_t n, const float* __restrict__ x, bf16* __restrict__ xb) {
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= n) return;
    xb[4 * p] = to_bf16(x[p]);
    xb[4 * p + 1] = 0;
    xb[4 * p + 2] = 0;
    xb[4 * p + 3] = 0;
}

__global__ void output_kernel(int64_t n, const float* __restrict__ z, float* __restrict__ y) {
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p < n) y[p] = z[p];
}

__global__ void cast_params_kernel(int64_t n, const float* __restrict__ w, bf16* __restrict__ wb) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) wb[i] = to_bf16(w[i]);
}

__global__ void adam_kernel(int64_t n, float* __restrict__ w, float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    g[i] = 0.0f;
}

// MSE loss partials and gradient dy = 2 (y - t) / n
__global__ void __launch_bounds__(256) mse_kernel(int64_t n, const float* __restrict__ y, const float* __restrict__ t,
                                                  float* __restrict__ dy, double* __restrict__ part) {
    __shared__ double sh[256];
    double acc = 0.0;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
        const float d = y[i] - t[i];
        acc += double(d) * d;
        if (dy) dy[i] = 2.0f * d / float(n);
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// patch of edge S from a box of edge D at offset (ox, oy, oz) under one of
// the 48 cubic symmetries: sym = perm * 8 + flips, perm indexes the 6 axis
// permutations, bit a of flips mirrors output axis a.  Out-of-box cells read 0.
__global__ void crop_kernel(int D, int S, int ox, int oy, int oz, int sym, const float* __restrict__ box,
                            float* __restrict__ patch) {
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= int64_t(S) * S * S) return;
    int c[3] = {int(idx % S), int((idx / S) % S), int(idx / (int64_t(S) * S))};   // x, y, z of the patch
    const int perms[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
    const int pm = (sym >> 3) % 6, fl = sym & 7;
    for (int a = 0; a < 3; ++a)
        if (fl & (1 << a)) c[a] = S - 1 - c[a];
    int s[3];
    for (int a = 0; a < 3; ++a) s[perms[pm][a]] = c[a];
    const int x = ox + s[0], y = oy + s[1], z = oz + s[2];
    float v = 0.0f;
    if (x >= 0 && y >= 0 && z >= 0 && x < D && y < D && z < D) v = box[(int64_t(z) * D + y) * D + x];
    patch[idx] = v;
}

__global__ void rows_to_box_kernel(int64_t n_rows, const int32_t* __restrict__ ijk4, const double* __restrict__ rows,
                                   const double* __restrict__ base, double scale, float* __restrict__ box, int D,
                                   int off) {
    const int64_t r = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (r >= n_rows || !ijk4[4 * r + 3]) return;
    const int x = ijk4[4 * r] + off, y = ijk4[4 * r + 1] + off, z = ijk4[4 * r + 2] + off;
    if (x < 0 || y < 0 || z < 0 || x >= D || y >= D || z >= D) return;
    const double v = base ? rows[r] - base[r] : rows[r];
    box[(int64_t(z) * D + y) * D + x] = float(scale * v);
}

__global__ void box_to_rows_kernel(int64_t n_rows, const int32_t* __restrict__ ijk4, const float* __restrict__ box, int D,
                                   int off, double inv_scale, const double* __restrict__ base, double* __restrict__ out) {
    const int64_t r = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (r >= n_rows) return;
    if (!ijk4[4 * r + 3]) {
        out[r] = 0.0;
        return;
    }
    const int x = ijk4[4 * r] + off, y = ijk4[4 * r + 1] + off, z = ijk4[4 * r + 2] + off;
    double v = base ? base[r] : 0.0;
    if (x >= 0 && y >= 0 && z >= 0 && x < D && y < D && z < D) v += inv_scale * double(box[(int64_t(z) * D + y) * D + x]);
    out[r] = v;
}

// One pass of a separable, truncated, normalised Gaussian along one axis of a
// cubic box (x fastest), zero outside: blur[i] = sum_k g[k + r] in[i + k e], k
// ascending; with `box` the pass writes box - blur instead.
//
// A workgroup takes 32 lines x 64 cells along the axis, staged with their rims
// in LDS; a thread forms 8 consecutive cells from a run of 8 + 2 r values, so a
// staged value is read once for 8 results.  One thread per cell with all
// 2 r + 1 values from memory took 27 to 34 us per pass at 96^3, r = 24; now 14.
constexpr int kMaxBlur = 192;                 // r of the widest Gaussian (sigma 64)
struct BlurWeights {
    float g[2 * kMaxBlur + 1];
};

__global__ void __launch_bounds__(256) blur_pass_kernel(int D, int axis, int r, BlurWeights w, const float* __restrict__ in,
                                                        const float* __restrict__ box, float* __restrict__ out) {
    extern __shared__ float line[];
    const int t = threadIdx.x, len = 64 + 2 * r;
    // lines run along x for axis y and z (neighbours are coalesced), along y for axis x
    const int pitch = axis == 0 ? len + 1 - (len & 1) : 33;
    const int64_t sa = axis == 0 ? 1 : axis == 1 ? D : int64_t(D) * D;      // step along the axis
    const int64_t sl = axis == 0 ? D : 1;                                    // between lines
    const int64_t so = axis == 2 ? D : int64_t(D) * D;                       // between slabs of lines
    const int l0 = blockIdx.x * 32, c0 = blockIdx.y * 64;
    const int64_t base = int64_t(blockIdx.z) * so;
    for (int i = t; i < 32 * len; i += 256) {
        const int l = axis == 0 ? i / len : i & 31, c = axis == 0 ? i % len : i >> 5;
        const int gl = l0 + l, gc = c0 - r + c;
        const float v = gl < D && gc >= 0 && gc < D ? in[base + gl * sl + gc * sa] : 0.0f;
        line[axis == 0 ? l * pitch + c : c * pitch + l] = v;
    }
    __syncthreads();
    const int l = t & 31, s0 = (t >> 5) * 8;
    const float* src = axis == 0 ? line + l * pitch + s0 : line + s0 * pitch + l;
    const int step = axis == 0 ? 1 : pitch;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int i = 0; i < 2 * r + 8; ++i) {
        const float v = src[i * step];
        if (i >= 7 && i <= 2 * r) {
#pragma unroll
            for (int o = 0; o < 8; ++o) acc[o] = fmaf(w.g[i - o], v, acc[o]);
        } else {                              // the run's ends: not all 8 results take the value
#pragma unroll
            for (int o = 0; o < 8; ++o)
                if (i - o >= 0 && i - o <= 2 * r) acc[o] = fmaf(w.g[i - o], v, acc[o]);
        }
    }
    if (l0 + l >= D) return;
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        if (c0 + s0 + o >= D) break;
        const int64_t at = base + (l0 + l) * sl + (c0 + s0 + o) * sa;
        out[at] = box ? box[at] - acc[o] : acc[o];
    }
}

static uint64_t splitmix(uint64_t& s) {
    uint64_t z = (s += 0x9e3779b97f4a7c15ull);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

}  // namespace dn
}  // namespace chf

using namespace chf;
using namespace chf::dn;

struct dnet {
    int C = 32;
    std::vector<Layer> L;
    int64_t n_params = 0;
    DevBuf w, g, m, v;            // FP32 master params, grads, Adam moments
    DevBuf wb;                    // BF16 copy of the weights (widths other than 32)
    DevBuf wp;                    // BF16 weights in MFMA operand order (32 channels)
    DevBuf wt;                    // BF16 transposed weights (scratch, one layer)
    DevBuf part;                  // weight-gradient partials / loss partials
    int S = 0;                    // patch edge the activation buffers are sized for
    // activation tape: for each layer the input pointer(s) and Z / Y buffers
    struct Act {
        DevBuf z, y;
        int D = 0;                // output edge
    };
    std::vector<std::unique_ptr<Act>> act;
    DevBuf xin;                   // BF16 input [S^3][4]
    DevBuf up[3];                 // upsampled inputs of u3, u2, u1 (widths other than 32)
    DevBuf gA, gB, gC, gD;        // FP32 gradient scratch (32 channels: gA)
    DevBuf dzb;                   // BF16 dZ
    DevBuf dzb2;                  // BF16 dZ of the next layer down (32 channels)
    DevBuf skip[3];               // gradients of the skip connections (32 channels)
    DevBuf bias_part;             // [workgroup][32] sums of dZ (32 channels)
    hipStream_t stream = nullptr;
};

namespace {

enum {
    C1A, C1B, D1, C2A, C2B, D2, C3A, C3B, D3, C4A, C4B, U3, C5A, C5B, U2, C6A, C6B, U1, C7A, C7B, OUT, NLAYER
};

void make_layers(dnet* N) {
    const int C = N->C;
    struct Spec {
        int cin, cout, k, stride;
        bool act;
    };
    const Spec sp[NLAYER] = {{1, C, 3, 1, true},     {C, C, 3, 1, true},     {C, C, 3, 2, true}, {C, C, 3, 1, true},
                             {C, C, 3, 1, true},     {C, C, 3, 2, true},     {C, C, 3, 1, true}, {C, C, 3, 1, true},
                             {C, C, 3, 2, true},     {C, C, 3, 1, true},     {C, C, 3, 1, true}, {C, C, 3, 1, true},
                             {2 * C, C, 3, 1, true}, {C, C, 3, 1, true},     {C, C, 3, 1, true}, {2 * C, C, 3, 1, true},
                             {C, C, 3, 1, true},     {C, C, 3, 1, true},     {2 * C, C, 3, 1, true},
                             {C, C, 3, 1, true},     {C, 1, 1, 1, false}};
    int64_t off = 0;
    for (int i = 0; i < NLAYER; ++i) {
        Layer l;
        l.cin = sp[i].cin;
        l.cout = sp[i].cout;
        l.cin_p = ((l.cin + 3) / 4) * 4;
        l.cout_p = ((l.cout + 15) / 16) * 16;
        l.k = sp[i].k;
        l.stride = sp[i].stride;
        l.act = sp[i].act;
        l.w_off = off;
        off += int64_t(l.cout_p) * l.k * l.k * l.k * l.cin_p;
        l.b_off = off;
        off += l.cout_p;
        N->L.push_back(l);
    }
    N->n_params = off;
}

unsigned nb(int64_t n) { return unsigned((n + 255) / 256); }

// edge of the output of layer i for patch edge S: encoder levels S, S/2, S/4,
// S/8 (the stride-2 layer opens its level), decoder levels S/4, S/2, S (the
// upsampling conv opens its level), and the 1^3 output layer at S
int out_edge(int i, int S) {
    static const int div[NLAYER] = {1, 1,          // c1a c1b
                                    2, 2, 2,       // d1 c2a c2b
                                    4, 4, 4,       // d2 c3a c3b
                                    8, 8, 8,       // d3 c4a c4b
                                    4, 4, 4,       // u3 c5a c5b
                                    2, 2, 2,       // u2 c6a c6b
                                    1, 1, 1,       // u1 c7a c7b
                                    1};            // out
    return S / div[i];
}

void ensure_buffers(dnet* N, int S) {
    if (N->S == S) return;
    const int C = N->C;
    N->act.clear();
    for (int i = 0; i < NLAYER; ++i) {
        const int D = out_edge(i, S);
        const int64_t n = int64_t(D) * D * D * N->L[i].cout;
        N->act.emplace_back(new dnet::Act);
        N->act[i]->D = D;
        N->act[i]->z.alloc(size_t(n) * sizeof(float));
        N->act[i]->y.alloc(size_t(n) * sizeof(bf16));
    }
    N->xin.alloc(size_t(S) * S * S * 4 * sizeof(bf16));
    N->dzb.alloc(size_t(S) * S * S * C * sizeof(bf16));
    const size_t big = size_t(S) * S * S * 2 * C * sizeof(float);
    if (C == 32) {
        N->gA.alloc(big / 2);
    } else {
        N->up[0].alloc(size_t(S / 4) * (S / 4) * (S / 4) * C * sizeof(bf16));
        N->up[1].alloc(size_t(S / 2) * (S / 2) * (S / 2) * C * sizeof(bf16));
        N->up[2].alloc(size_t(S) * S * S * C * sizeof(bf16));
        N->gA.alloc(big);
        N->gB.alloc(big);
        N->gC.alloc(big);
        N->gD.alloc(big);
    }
    N->S = S;
}

// ---------------------------------------------------------------------------
// 32 channels: packed weights and the tiled kernels
// ---------------------------------------------------------------------------
int64_t pack_at(int i) { return int64_t(i) * 2 * kPackHalf; }

void pack_weights(dnet* N, bool transposed, hipStream_t s) {
    N->wp.ensure(size_t(pack_at(OUT)) * sizeof(s8));
    PackTable tab;
    for (int i = 0; i < OUT; ++i) {
        tab.w_off[i] = N->L[i].w_off;
        tab.halves[i] = N->L[i].cin / 32;
    }
    pack_kernel<<<dim3(nb(2 * kPackHalf), OUT), 256, 0, s>>>(tab, transposed ? 1 : 0, N->w.as<float>(), N->wp.as<s8>());
    LAUNCH_CHECK();
}

// Tile rule: 8 x 8 x 4 positions (4 groups per wave) where that still gives a
// workgroup to each CU, else 8 x 4 x 2.
bool big_tiles(int D) { return int64_t((D + 7) / 8) * ((D + 7) / 8) * ((D + 3) / 4) >= 256; }
unsigned n_tiles(int D, int ty, int tz) { return unsigned((D + 7) / 8) * ((D + ty - 1) / ty) * ((D + tz - 1) / tz); }

void conv3_forward(dnet* N, int i, int Di, const bf16* in0, const bf16* in1, bool upsampled, hipStream_t s) {
    const Layer& l = N->L[i];
    Conv3 a{};
    a.Din = Di;
    a.Dsrc = upsampled ? Di / 2 : Di;
    a.Dout = N->act[i]->D;
    a.in0 = in0;
    a.in1 = in1;
    a.w = N->wp.as<s8>() + pack_at(i);
    a.bias = N->w.as<float>() + l.b_off;
    a.z = N->act[i]->z.as<float>();
    a.y = N->act[i]->y.as<bf16>();
    const int D = a.Dout;
    const bool big = big_tiles(D);
    if (l.stride == 2) conv3_kernel<1, 2, 4, 2, kPlain, 2, kForward><<<n_tiles(D, 4, 2), 256, 0, s>>>(a);
    else if (in1 && big) conv3_kernel<2, 1, 8, 4, kPlain, 2, kForward><<<n_tiles(D, 8, 4), 256, 0, s>>>(a);
    else if (in1) conv3_kernel<2, 1, 4, 2, kPlain, 2, kForward><<<n_tiles(D, 4, 2), 256, 0, s>>>(a);
    else if (upsampled && big) conv3_kernel<1, 1, 8, 4, kUpsample, 2, kForward><<<n_tiles(D, 8, 4), 256, 0, s>>>(a);
    else if (upsampled) conv3_kernel<1, 1, 4, 2, kUpsample, 2, kForward><<<n_tiles(D, 4, 2), 256, 0, s>>>(a);
    else if (big) conv3_kernel<1, 1, 8, 4, kPlain, 2, kForward><<<n_tiles(D, 8, 4), 256, 0, s>>>(a);
    else conv3_kernel<1, 1, 4, 2, kPlain, 2, kForward><<<n_tiles(D, 4, 2), 256, 0, s>>>(a);
    LAUNCH_CHECK();
}

// one partial per workgroup, at most kWgradGroups of them (and halves) per layer
constexpr int kWgradGroups = 256;

// parameter gradients of layer i from its dZ and its input; n_bias partial sums of dZ
void conv3_weight_grad(dnet* N, int i, int Di, const bf16* in0, const bf16* in1, bool upsampled, const bf16* dzb, int n_bias,
                       hipStream_t s) {
    const Layer& l = N->L[i];
    const int D = N->act[i]->D;
    float* gw = N->g.as<float>() + l.w_off;
    float* gb = N->g.as<float>() + l.b_off;
    const float* bp = N->bias_part.as<float>();
    if (i == C1A) {
        const int np = int(std::min<unsigned>(kWgradGroups, n_tiles(D, 8, 4)));
        N->part.ensure(size_t(np) * 256 * sizeof(f4));
        wgrad_in_kernel<<<np, 256, 0, s>>>(D, in0, dzb, N->part.as<f4>());
        wgrad_in_reduce_kernel<<<5, 256, 0, s>>>(np, N->part.as<f4>(), gw, n_bias, bp, gb);
        LAUNCH_CHECK();
        return;
    }
    const int ty = l.stride == 2 ? 4 : 8, tz = l.stride == 2 ? 2 : 4, halves = in1 ? 2 : 1;
    const int np = int(std::min<unsigned>(kWgradGroups, n_tiles(D, ty, tz)));
    N->part.ensure(size_t(np) * halves * kWgradPart * sizeof(f4));
    const WGrad a{Di, upsampled ? Di / 2 : Di, D, in0, in1, dzb, N->part.as<f4>()};
    const dim3 grid(np, halves);
    if (l.stride == 2) wgrad3_kernel<2, 4, 2, kPlain><<<grid, 256, 0, s>>>(a);
    else if (upsampled) wgrad3_kernel<1, 8, 4, kUpsample><<<grid, 256, 0, s>>>(a);
    else wgrad3_kernel<1, 8, 4, kPlain><<<grid, 256, 0, s>>>(a);
    LAUNCH_CHECK();
    wgrad3_reduce_kernel<<<halves * (kWgradPart / 64) + 1, 256, 0, s>>>(halves, np, N->part.as<f4>(), gw, n_bias, bp, gb);
    LAUNCH_CHECK();
}

// Input gradient of layer i.  into >= 0: times the derivative of layer `into`'s
// activation (after `add`, the gradient that reached that layer through a skip)
// as its dZ in dz_out, with its bias sums; `raw` then takes the gradient of the
// second 32 channels.  into < 0: as it is into raw.  Returns the bias partials.
int conv3_input_grad(dnet* N, int i, int into, const bf16* dzb, const float* add, bf16* dz_out, float* raw, hipStream_t s) {
    const Layer& l = N->L[i];
    Conv3 a{};
    a.Dsrc = N->act[i]->D;
    a.Dout = a.Din = a.Dsrc * l.stride;
    a.in0 = dzb;
    a.w = N->wp.as<s8>() + pack_at(i);
    a.add = add;
    a.zprev = into >= 0 ? N->act[into]->z.as<float>() : nullptr;
    a.dzb = dz_out;
    a.raw = raw;
    a.bias_part = N->bias_part.as<float>();
    const int D = a.Dout;
    const bool big = big_tiles(D);
    const unsigned n = big ? n_tiles(D, 8, 4) : n_tiles(D, 4, 2);
    N->bias_part.ensure(size_t(n) * 32 * sizeof(float));
    a.bias_part = N->bias_part.as<float>();
    auto go = [&](auto load, auto mb, auto epi) {
        constexpr int L = decltype(load)::value, MB = decltype(mb)::value, E = decltype(epi)::value;
        if (big) conv3_kernel<1, 1, 8, 4, L, MB, E><<<n, 256, 0, s>>>(a);
        else conv3_kernel<1, 1, 4, 2, L, MB, E><<<n, 256, 0, s>>>(a);
    };
    using std::integral_constant;
    const integral_constant<int, kPlain> plain;
    const integral_constant<int, 2> two;
    if (into < 0) go(plain, two, integral_constant<int, kGradRaw>{});
    else if (l.cin == 64) go(plain, integral_constant<int, 4>{}, integral_constant<int, kGradAct>{});
    else if (l.stride == 2) go(integral_constant<int, kDilate>{}, two, integral_constant<int, kGradAct>{});
    else go(plain, two, integral_constant<int, kGradAct>{});
    LAUNCH_CHECK();
    return int(n);
}

// Backward of a 32-channel network, layer by layer: a layer's dZ alternates
// between two buffers, since its input gradient becomes the next dZ.
void backward32(dnet* N, const float* dy, hipStream_t s) {
    const int S = N->S;
    const int64_t n = int64_t(S) * S * S;
    const size_t bytes = size_t(n) * 32 * sizeof(bf16);
    N->dzb2.ensure(bytes);
    const int enc[3] = {C3B, C2B, C1B};
    for (int lvl = 0; lvl < 3; ++lvl) {
        const int64_t d = N->act[enc[lvl]]->D;
        N->skip[lvl].ensure(size_t(d * d * d) * 32 * sizeof(float));
    }
    pack_weights(N, true, s);
    auto Y = [&](int i) { return N->act[i]->y.as<bf16>(); };
    bf16* cur = N->dzb.as<bf16>();
    bf16* nxt = N->dzb2.as<bf16>();
    float* raw = N->gA.as<float>();
    const int blocks = int(std::min<int64_t>(1024, (n + 31) / 32));
    N->bias_part.ensure(size_t(blocks) * 32 * sizeof(float));
    N->part.ensure(size_t(blocks) * 33 * sizeof(float));
    out_back_kernel<<<blocks, 256, 0, s>>>(n, dy, N->w.as<float>() + N->L[OUT].w_off, Y(C7B), N->act[C7B]->z.as<float>(), cur,
                                           N->bias_part.as<float>(), N->part.as<float>());
    out_reduce_kernel<<<33, 256, 0, s>>>(blocks, N->part.as<float>(), N->g.as<float>() + N->L[OUT].w_off,
                                         N->g.as<float>() + N->L[OUT].b_off);
    LAUNCH_CHECK();
    int nbias = blocks;
    // layer i with plain input in0 = Y(into)
    auto step = [&](int i, int into, const float* add) {
        conv3_weight_grad(N, i, N->act[into]->D, Y(into), nullptr, false, cur, nbias, s);
        nbias = conv3_input_grad(N, i, into, cur, add, nxt, nullptr, s);
        std::swap(cur, nxt);
    };
    for (int lvl = 2; lvl >= 0; --lvl) {
        const int up = U3 + 3 * lvl, D = N->act[up]->D, Ds = D / 2;
        step(up + 2, up + 1, nullptr);
        conv3_weight_grad(N, up + 1, D, Y(up), Y(enc[lvl]), false, cur, nbias, s);
        nbias = conv3_input_grad(N, up + 1, up, cur, nullptr, nxt, N->skip[lvl].as<float>(), s);
        std::swap(cur, nxt);
        conv3_weight_grad(N, up, D, Y(up - 1), nullptr, true, cur, nbias, s);
        conv3_input_grad(N, up, -1, cur, nullptr, nullptr, raw, s);
        nbias = int(std::min<int64_t>(1024, (int64_t(Ds) * Ds * Ds + 31) / 32));
        N->bias_part.ensure(size_t(nbias) * 32 * sizeof(float));
        up_back_kernel<<<nbias, 256, 0, s>>>(Ds, raw, N->act[up - 1]->z.as<float>(), nxt, N->bias_part.as<float>());
        LAUNCH_CHECK();
        std::swap(cur, nxt);
    }
    for (int i = C4B; i >= C1B; --i) {
        // the input of a stride-2 layer also feeds the skip connection of its level
        const int lvl = i == D3 ? 0 : i == D2 ? 1 : i == D1 ? 2 : -1;
        step(i, i - 1, lvl >= 0 ? N->skip[lvl].as<float>() : nullptr);
    }
    conv3_weight_grad(N, C1A, S, N->xin.as<bf16>(), nullptr, false, cur, nbias, s);
}

void conv_forward(dnet* N, int i, int Di, const bf16* in0, int c0, const bf16* in1, int c1, hipStream_t s) {
    const Layer& l = N->L[i];
    const int Do = N->act[i]->D;
    const int64_t npos = int64_t(Do) * Do * Do;
    conv_fwd_kernel<<<unsigned((npos + 63) / 64), 256, 0, s>>>(
        Di, Do, c0, c1, l.cin_p, l.cout, l.cout_p, l.k, l.stride, in0, in1, N->wb.as<bf16>() + l.w_off,
        N->w.as<float>() + l.b_off, N->act[i]->z.as<float>(), N->act[i]->y.as<bf16>(), l.act ? 1 : 0);
    LAUNCH_CHECK();
}

// backward through layer i: dy (FP32, [Do^3][cout]) -> parameter grads and
// (optionally) dx (FP32, [Di^3][cin])
void conv_backward(dnet* N, int i, int Di, const bf16* in0, int c0, const bf16* in1, int c1, const float* dy, float* dx,
                   hipStream_t s) {
    const Layer& l = N->L[i];
    const int Do = N->act[i]->D;
    const int64_t npos = int64_t(Do) * Do * Do;
    const int ntap = l.k * l.k * l.k;
    float* dz = N->gD.as<float>();
    act_back_kernel<<<nb(npos * l.cout), 256, 0, s>>>(npos * l.cout, dy, N->act[i]->z.as<float>(), l.act ? 1 : 0, dz,
                                                      N->dzb.as<bf16>());
    LAUNCH_CHECK();
    // weight gradient: split-K over output positions
    const int ncol = ntap * l.cin_p;
    const int ncb = (ncol + 63) / 64;
    int nsplit = int(std::min<int64_t>(256, std::max<int64_t>(1, npos / 1024)));
    const int64_t per = ((npos + nsplit - 1) / nsplit + 15) / 16 * 16;
    nsplit = int((npos + per - 1) / per);
    N->part.ensure(size_t(nsplit) * 32 * ncol * sizeof(float));
    conv_bwd_weight_kernel<<<dim3(ncb, nsplit), 256, 0, s>>>(Di, Do, c0, c1, l.cin_p, l.cout, l.k, l.stride,
                                                             N->dzb.as<bf16>(), in0, in1, per, N->part.as<float>());
    LAUNCH_CHECK();
    wgrad_reduce_kernel<<<nb(int64_t(l.cout) * ncol), 256, 0, s>>>(l.cout, ncol, nsplit, N->part.as<float>(),
                                                                  N->g.as<float>() + l.w_off);
    LAUNCH_CHECK();
    bgrad_kernel<<<l.cout, 256, 0, s>>>(npos, l.cout, dz, N->g.as<float>() + l.b_off);
    LAUNCH_CHECK();
    if (!dx) return;
    const int cout_p4 = ((l.cout + 3) / 4) * 4;
    const int64_t nwt = int64_t(l.cin_p) * ntap * cout_p4;
    N->wt.ensure(size_t(nwt) * sizeof(bf16));
    weight_t_kernel<<<nb(nwt), 256, 0, s>>>(l.cout, cout_p4, ntap, l.cin_p, N->w.as<float>() + l.w_off, N->wt.as<bf16>());
    LAUNCH_CHECK();
    const int64_t nin = int64_t(Di) * Di * Di;
    conv_bwd_data_kernel<<<unsigned((nin + 63) / 64), 256, 0, s>>>(Di, Do, l.cin, l.cin_p, l.cout, cout_p4, l.k, l.stride,
                                                                   N->dzb.as<bf16>(), N->wt.as<bf16>(), dx);
    LAUNCH_CHECK();
}

template <class F>
int dguard(F&& f) {
    try {
        f();
        return CHF_OK;
    } catch (const Error& e) {
        set_last_error(e.what());
        return e.code;
    } catch (const std::bad_alloc&) {
        set_last_error("host allocation failed");
        return CHF_ENOMEM;
    } catch (const std::exception& e) {
        set_last_error(e.what());
        return CHF_EHIP;
    }
}

}  // namespace

extern "C" {

int dnet_create(int channels, uint64_t seed, dnet** out) {
    return dguard([&] {
        if (!out) fail(CHF_EINVAL, "dnet_create: null out");
        *out = nullptr;
        if (channels < 4 || channels > 32 || channels % 4) fail(CHF_EINVAL, "dnet_create: channels must be 4..32, multiple of 4");
        auto N = std::make_unique<dnet>();
        N->C = channels;
        make_layers(N.get());
        // He-normal weights (Box-Muller over splitmix64), zero biases, zero
        // output layer so the untrained network predicts no correction
        std::vector<float> h(size_t(N->n_params), 0.0f);
        uint64_t st = seed;
        for (int i = 0; i < NLAYER; ++i) {
            const Layer& l = N->L[i];
            if (i == OUT) continue;
            const int ntap = l.k * l.k * l.k;
            const double sd = std::sqrt(2.0 / (double(l.cin) * ntap));
            for (int co = 0; co < l.cout; ++co)
                for (int t = 0; t < ntap; ++t)
                    for (int ci = 0; ci < l.cin; ++ci) {
                        const double u1 = (double(splitmix(st) >> 11) + 0.5) / 9007199254740992.0;
                        const double u2 = double(splitmix(st) >> 11) / 9007199254740992.0;
                        const double z = std::sqrt(-2.0 * std::log(u1)) * std::cos(2.0 * 3.14159265358979323846 * u2);
                        h[size_t(l.w_off + (int64_t(co) * ntap + t) * l.cin_p + ci)] = float(sd * z);
                    }
        }
        N->w.alloc(size_t(N->n_params) * sizeof(float));
        N->g.alloc(size_t(N->n_params) * sizeof(float));
        N->m.alloc(size_t(N->n_params) * sizeof(float));
        N->v.alloc(size_t(N->n_params) * sizeof(float));
        N->wb.alloc(size_t(N->n_params) * sizeof(bf16));
        HIP_CHECK(hipMemcpy(N->w.p, h.data(), h.size() * sizeof(float), hipMemcpyHostToDevice));
        HIP_CHECK(hipMemset(N->g.p, 0, size_t(N->n_params) * sizeof(float)));
        HIP_CHECK(hipMemset(N->m.p, 0, size_t(N->n_params) * sizeof(float)));
        HIP_CHECK(hipMemset(N->v.p, 0, size_t(N->n_params) * sizeof(float)));
        *out = N.release();
    });
}

int dnet_destroy(dnet* N) {
    if (N) {
        (void)hipDeviceSynchronize();
        delete N;
    }
    return CHF_OK;
}

int dnet_param_count(const dnet* N, int64_t* n) {
    return dguard([&] {
        if (!N || !n) fail(CHF_EINVAL, "dnet_param_count: null argument");
        *n = N->n_params;
    });
}

int dnet_layer_info(const dnet* N, int layer, int* info6, int64_t* offsets2) {
    return dguard([&] {
        if (!N || !info6 || !offsets2 || layer < 0 || layer >= NLAYER) fail(CHF_EINVAL, "dnet_layer_info: bad argument");
        const Layer& l = N->L[size_t(layer)];
        info6[0] = l.cin;
        info6[1] = l.cout;
        info6[2] = l.cin_p;
        info6[3] = l.cout_p;
        info6[4] = l.k;
        info6[5] = l.stride;
        offsets2[0] = l.w_off;
        offsets2[1] = l.b_off;
    });
}

int dnet_plan(int S, int* edges) {
    return dguard([&] {
        if (!edges || S < 8 || S % 8) fail(CHF_EINVAL, "dnet_plan: S must be a positive multiple of 8");
        for (int i = 0; i < NLAYER; ++i) edges[i] = out_edge(i, S);
    });
}

int dnet_get_params(const dnet* N, float* host) {
    return dguard([&] {
        if (!N || !host) fail(CHF_EINVAL, "dnet_get_params: null argument");
        HIP_CHECK(hipDeviceSynchronize());
        HIP_CHECK(hipMemcpy(host, N->w.p, size_t(N->n_params) * sizeof(float), hipMemcpyDeviceToHost));
    });
}

int dnet_set_params(dnet* N, const float* host) {
    return dguard([&] {
        if (!N || !host) fail(CHF_EINVAL, "dnet_set_params: null argument");
        HIP_CHECK(hipDeviceSynchronize());
        HIP_CHECK(hipMemcpy(N->w.p, host, size_t(N->n_params) * sizeof(float), hipMemcpyHostToDevice));
    });
}

int dnet_forward(dnet* N, const float* x, int S, float* y, void* stream) {
    return dguard([&] {
        if (!N || !x || !y) fail(CHF_EINVAL, "dnet_forward: null argument");
        if (S < 8 || S % 8 || S > 512) fail(CHF_EINVAL, "dnet_forward: patch edge must be a multiple of 8 in [8, 512]");
        hipStream_t s = static_cast<hipStream_t>(stream);
        N->stream = s;
        ensure_buffers(N, S);
        const int C = N->C;
        const int64_t n = int64_t(S) * S * S;
        input_kernel<<<nb(n), 256, 0, s>>>(n, x, N->xin.as<bf16>());
        LAUNCH_CHECK();
        auto Y = [&](int i) { return N->act[i]->y.as<bf16>(); };
        if (C == 32) {
            pack_weights(N, false, s);
            const float* w = N->w.as<float>();
            conv_in_kernel<<<n_tiles(S, 8, 4), 256, 0, s>>>(S, N->xin.as<s4>(), N->wp.as<s4>() + 2 * pack_at(C1A),
                                                            w + N->L[C1A].b_off, N->act[C1A]->z.as<float>(), Y(C1A));
            LAUNCH_CHECK();
            for (int i = C1B; i <= C4B; ++i)
                conv3_forward(N, i, N->act[i - 1]->D, Y(i - 1), nullptr, false, s);
            const int enc[3] = {C3B, C2B, C1B};
            for (int lvl = 0; lvl < 3; ++lvl) {
                const int up = U3 + 3 * lvl, D = N->act[up]->D;
                conv3_forward(N, up, D, Y(up - 1), nullptr, true, s);
                conv3_forward(N, up + 1, D, Y(up), Y(enc[lvl]), false, s);
                conv3_forward(N, up + 2, D, Y(up + 1), nullptr, false, s);
            }
            conv_out_kernel<<<unsigned((n + 255) / 256), 256, 0, s>>>(n, Y(C7B), w + N->L[OUT].w_off, w + N->L[OUT].b_off, y);
            LAUNCH_CHECK();
            return;
        }
        cast_params_kernel<<<nb(N->n_params), 256, 0, s>>>(N->n_params, N->w.as<float>(), N->wb.as<bf16>());
        LAUNCH_CHECK();
        conv_forward(N, C1A, S, N->xin.as<bf16>(), 4, nullptr, 0, s);
        conv_forward(N, C1B, S, Y(C1A), C, nullptr, 0, s);
        conv_forward(N, D1, S, Y(C1B), C, nullptr, 0, s);
        conv_forward(N, C2A, S / 2, Y(D1), C, nullptr, 0, s);
        conv_forward(N, C2B, S / 2, Y(C2A), C, nullptr, 0, s);
        conv_forward(N, D2, S / 2, Y(C2B), C, nullptr, 0, s);
        conv_forward(N, C3A, S / 4, Y(D2), C, nullptr, 0, s);
        conv_forward(N, C3B, S / 4, Y(C3A), C, nullptr, 0, s);
        conv_forward(N, D3, S / 4, Y(C3B), C, nullptr, 0, s);
        conv_forward(N, C4A, S / 8, Y(D3), C, nullptr, 0, s);
        conv_forward(N, C4B, S / 8, Y(C4A), C, nullptr, 0, s);
        const int enc[3] = {C3B, C2B, C1B}, upl[3] = {U3, U2, U1}, ca[3] = {C5A, C6A, C7A}, cb[3] = {C5B, C6B, C7B};
        int prev = C4B;
        for (int lvl = 0; lvl < 3; ++lvl) {
            const int Ds = N->act[prev]->D, Dd = 2 * Ds;
            upsample_kernel<<<nb(int64_t(Dd) * Dd * Dd * C), 256, 0, s>>>(Ds, C, Y(prev), N->up[lvl].as<bf16>());
            LAUNCH_CHECK();
            conv_forward(N, upl[lvl], Dd, N->up[lvl].as<bf16>(), C, nullptr, 0, s);
            conv_forward(N, ca[lvl], Dd, Y(upl[lvl]), C, Y(enc[lvl]), C, s);
            conv_forward(N, cb[lvl], Dd, Y(ca[lvl]), C, nullptr, 0, s);
            prev = cb[lvl];
        }
        conv_forward(N, OUT, S, Y(C7B), C, nullptr, 0, s);
        output_kernel<<<nb(n), 256, 0, s>>>(n, N->act[OUT]->z.as<float>(), y);
        LAUNCH_CHECK();
    });
}

int dnet_backward(dnet* N, const float* dy, void* stream) {
    return dguard([&] {
        if (!N || !dy) fail(CHF_EINVAL, "dnet_backward: null argument");
        if (N->S == 0) fail(CHF_EINVAL, "dnet_backward: call dnet_forward first");
        hipStream_t s = static_cast<hipStream_t>(stream);
        if (N->C == 32) {
            backward32(N, dy, s);
            HIP_CHECK(hipStreamSynchronize(s));
            return;
        }
        const int S = N->S, C = N->C;
        auto Y = [&](int i) { return N->act[i]->y.as<bf16>(); };
        float* a = N->gA.as<float>();
        float* b = N->gB.as<float>();
        float* c = N->gC.as<float>();
        // out layer: input g1 = Y(C7B)
        conv_backward(N, OUT, S, Y(C7B), C, nullptr, 0, dy, a, s);   // a = dL/d g1
        // decoder levels (innermost last): keep the skip gradients
        float* skip[3] = {nullptr, nullptr, nullptr};
        const int enc[3] = {C3B, C2B, C1B}, upl[3] = {U3, U2, U1}, ca[3] = {C5A, C6A, C7A}, cb[3] = {C5B, C6B, C7B};
        const int prevl[3] = {C4B, C5B, C6B};
        std::vector<std::unique_ptr<DevBuf>> keep;
        for (int lvl = 2; lvl >= 0; --lvl) {
            const int Dd = N->act[cb[lvl]]->D, Ds = Dd / 2;
            const int64_t nd = int64_t(Dd) * Dd * Dd;
            conv_backward(N, cb[lvl], Dd, Y(ca[lvl]), C, nullptr, 0, a, b, s);             // b = dL/d Y(ca)
            conv_backward(N, ca[lvl], Dd, Y(upl[lvl]), C, Y(enc[lvl]), C, b, c, s);         // c = dL/d concat [nd][2C]
            keep.emplace_back(new DevBuf);
            keep.back()->alloc(size_t(nd) * C * sizeof(float));
            skip[lvl] = keep.back()->as<float>();
            slice_add_kernel<<<nb(nd * C), 256, 0, s>>>(nd, 2 * C, C, C, c, nullptr, skip[lvl]);  // encoder part
            LAUNCH_CHECK();
            slice_add_kernel<<<nb(nd * C), 256, 0, s>>>(nd, 2 * C, 0, C, c, nullptr, b);          // upsampled part
            LAUNCH_CHECK();
            conv_backward(N, upl[lvl], Dd, N->up[lvl].as<bf16>(), C, nullptr, 0, b, c, s);  // c = dL/d up(prev)
            upsample_back_kernel<<<nb(int64_t(Ds) * Ds * Ds * C), 256, 0, s>>>(Ds, C, c, a);  // a = dL/d Y(prev)
            LAUNCH_CHECK();
            (void)prevl;
        }
        // encoder: a = dL/d Y(C4B)
        conv_backward(N, C4B, S / 8, Y(C4A), C, nullptr, 0, a, b, s);
        conv_backward(N, C4A, S / 8, Y(D3), C, nullptr, 0, b, a, s);
        conv_backward(N, D3, S / 4, Y(C3B), C, nullptr, 0, a, b, s);                      // b = dL/d e3 (down path)
        int64_t n3 = int64_t(S / 4) * (S / 4) * (S / 4);
        slice_add_kernel<<<nb(n3 * C), 256, 0, s>>>(n3, C, 0, C, b, skip[0], a);
        LAUNCH_CHECK();
        conv_backward(N, C3B, S / 4, Y(C3A), C, nullptr, 0, a, b, s);
        conv_backward(N, C3A, S / 4, Y(D2), C, nullptr, 0, b, a, s);
        conv_backward(N, D2, S / 2, Y(C2B), C, nullptr, 0, a, b, s);
        int64_t n2 = int64_t(S / 2) * (S / 2) * (S / 2);
        slice_add_kernel<<<nb(n2 * C), 256, 0, s>>>(n2, C, 0, C, b, skip[1], a);
        LAUNCH_CHECK();
        conv_backward(N, C2B, S / 2, Y(C2A), C, nullptr, 0, a, b, s);
        conv_backward(N, C2A, S / 2, Y(D1), C, nullptr, 0, b, a, s);
        conv_backward(N, D1, S, Y(C1B), C, nullptr, 0, a, b, s);
        int64_t n1 = int64_t(S) * S * S;
        slice_add_kernel<<<nb(n1 * C), 256, 0, s>>>(n1, C, 0, C, b, skip[2], a);
        LAUNCH_CHECK();
        conv_backward(N, C1B, S, Y(C1A), C, nullptr, 0, a, b, s);
        conv_backward(N, C1A, S, N->xin.as<bf16>(), 4, nullptr, 0, b, nullptr, s);
        HIP_CHECK(hipStreamSynchronize(s));   // scratch buffers in `keep` are released below
    });
}

int dnet_get_grads(const dnet* N, float* host) {
    return dguard([&] {
        if (!N || !host) fail(CHF_EINVAL, "dnet_get_grads: null argument");
        HIP_CHECK(hipDeviceSynchronize());
        HIP_CHECK(hipMemcpy(host, N->g.p, size_t(N->n_params) * sizeof(float), hipMemcpyDeviceToHost));
    });
}

int dnet_adam(dnet* N, float lr, int step, void* stream) {
    return dguard([&] {
        if (!N || step < 1 || !(lr > 0)) fail(CHF_EINVAL, "dnet_adam: bad argument");
        const float b1 = 0.9f, b2 = 0.999f;
        const float c1 = 1.0f - std::pow(b1, float(step)), c2 = 1.0f - std::pow(b2, float(step));
        adam_kernel<<<nb(N->n_params), 256, 0, static_cast<hipStream_t>(stream)>>>(
            N->n_params, N->w.as<float>(), N->g.as<float>(), N->m.as<float>(), N->v.as<float>(), lr, b1, b2, 1e-8f, c1, c2);
        LAUNCH_CHECK();
    });
}

int dnet_mse(dnet* N, const float* y, const float* t, int64_t n, double* loss_host, float* dy, void* stream) {
    return dguard([&] {
        if (!N || !y || !t || !loss_host || n < 1) fail(CHF_EINVAL, "dnet_mse: bad argument");
        hipStream_t s = static_cast<hipStream_t>(stream);
        const int blocks = int(std::min<int64_t>(1024, (n + 255) / 256));
        N->part.ensure(size_t(blocks + 1) * sizeof(double));
        double* part = reinterpret_cast<double*>(N->part.p);
        mse_kernel<<<blocks, 256, 0, s>>>(n, y, t, dy, part);
        LAUNCH_CHECK();
        std::vector<double> h(static_cast<size_t>(blocks));
        HIP_CHECK(hipMemcpyAsync(h.data(), part, size_t(blocks) * sizeof(double), hipMemcpyDeviceToHost, s));
        HIP_CHECK(hipStreamSynchronize(s));
        double tot = 0;
        for (double v : h) tot += v;
        *loss_host = tot / double(n);
    });
}

int chf_rows_to_box(chf_ham* H, const double* rows, const double* base, double scale, float* box, int D, int off,
                    void* stream) {
    return dguard([&] {
        if (!H || !rows || !box || D < 1) fail(CHF_EINVAL, "chf_rows_to_box: bad argument");
        hipStream_t s = static_cast<hipStream_t>(stream);
        HIP_CHECK(hipMemsetAsync(box, 0, size_t(D) * D * D * sizeof(float), s));
        rows_to_box_kernel<<<nb(H->grid.n_rows), 256, 0, s>>>(H->grid.n_rows, H->row_ijk4.as<int32_t>(), rows, base,
                                                              scale, box, D, off);
        LAUNCH_CHECK();
    });
}

int chf_box_to_rows(chf_ham* H, const float* box, int D, int off, double scale, const double* base, double* out,
                    void* stream) {
    return dguard([&] {
        if (!H || !box || !out || D < 1 || !(scale != 0)) fail(CHF_EINVAL, "chf_box_to_rows: bad argument");
        box_to_rows_kernel<<<nb(H->grid.n_rows), 256, 0, static_cast<hipStream_t>(stream)>>>(
            H->grid.n_rows, H->row_ijk4.as<int32_t>(), box, D, off, 1.0 / scale, base, out);
        LAUNCH_CHECK();
    });
}

int dnet_highpass(const float* box, int D, double sigma, float* out, float* work, void* stream) {
    return dguard([&] {
        if (!box || !out || !work || D < 1 || !(sigma > 0) || sigma > 64) fail(CHF_EINVAL, "dnet_highpass: bad argument");
        const int r = int(std::ceil(3.0 * sigma));
        BlurWeights w{};
        double tot = 0;
        for (int k = -r; k <= r; ++k) tot += std::exp(-double(k) * k / (2.0 * sigma * sigma));
        for (int k = -r; k <= r; ++k) w.g[k + r] = float(std::exp(-double(k) * k / (2.0 * sigma * sigma)) / tot);
        hipStream_t s = static_cast<hipStream_t>(stream);
        const int64_t n = int64_t(D) * D * D;
        float* t1 = work;
        float* t2 = work + n;
        const dim3 grid((D + 31) / 32, (D + 63) / 64, D);
        const int len = 64 + 2 * r;
        const size_t lds_x = size_t(32) * (len + 1 - (len & 1)) * sizeof(float), lds = size_t(len) * 33 * sizeof(float);
        blur_pass_kernel<<<grid, 256, lds_x, s>>>(D, 0, r, w, box, nullptr, t1);
        blur_pass_kernel<<<grid, 256, lds, s>>>(D, 1, r, w, t1, nullptr, t2);
        blur_pass_kernel<<<grid, 256, lds, s>>>(D, 2, r, w, t2, box, out);
        LAUNCH_CHECK();
        HIP_CHECK(hipStreamSynchronize(s));
    });
}

int dnet_crop(const float* box, int D, int S, int ox, int oy, int oz, int sym, float* patch, void* stream) {
    return dguard([&] {
        if (!box || !patch || D < 1 || S < 1 || sym < 0 || sym >= 48) fail(CHF_EINVAL, "dnet_crop: bad argument");
        crop_kernel<<<nb(int64_t(S) * S * S), 256, 0, static_cast<hipStream_t>(stream)>>>(D, S, ox, oy, oz, sym, box, patch);
        LAUNCH_CHECK();
    });
}

}  // extern "C"
