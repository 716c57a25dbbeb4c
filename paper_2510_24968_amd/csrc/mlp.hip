// BF16 matrix-core kernels of the learned initial-guess network: a GEMM on
// v_mfma_f32_16x16x16bf16_1k with FP32 accumulation (optional transposes,
// split-K with FP32 atomics, fused bias + ReLU epilogue), and the elementwise
// pieces of training (ReLU backward, bias gradient, MSE loss and gradient,
// Adam with FP32 master weights, FP32 -> BF16 rounding).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "../../include/fsim.h"

namespace fsim {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// round-to-nearest-even FP32 -> BF16 (NaN kept quiet)
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Two 16x16x16 products, K steps s and s + 1: lane l holds k = 4 (l / 16) + j,
// j < 4, of each.  (The 16x16x32 instruction of gfx950 sums its 32 products in
// another order, which flips BF16 roundings of the hidden activations.)
struct Frag {
    uint2 lo, hi;
};
__device__ __forceinline__ f32x4 mma32(const Frag &a, const Frag &b, f32x4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, a.lo),
                                                  __builtin_bit_cast(bf16x4, b.lo), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, a.hi),
                                                     __builtin_bit_cast(bf16x4, b.hi), c, 0, 0, 0);
}

constexpr int GT = 64;    // block tile (M and N)
constexpr int GK = 64;    // K per stage (four MFMA steps)
constexpr int GP = 76;    // LDS row pitch: 8-byte rows, at most two-way bank conflicts

// A 64 x 64 slice of one operand, held by the block's 256 threads as two
// 16-byte vectors each, then kept in LDS as [row][k].  KC: k is contiguous in
// memory (thread: one row, 16 k); otherwise the row index is (thread: two
// neighbouring k, 8 rows, transposed on the way to LDS).  x0: first row, R:
// rows in all, vec: 16-byte loads are allowed (base and pitch aligned).
template <bool KC>
__device__ __forceinline__ void slice_load(uint4 (&v)[2], const uint16_t *__restrict__ M, int ld,
                                           int x0, int R, int k0, int kend, bool vec) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int x = KC ? x0 + (tid >> 2) : x0 + (tid & 7) * 8;
        const int k = KC ? k0 + (tid & 3) * 16 + 8 * h : k0 + (tid >> 3) * 2 + h;
        const size_t at = KC ? (size_t)x * ld + k : (size_t)k * ld + x;
        const bool whole = KC ? (x < R && k + 8 <= kend) : (k < kend && x + 8 <= R);
        if (vec && whole) {
            v[h] = *(const uint4 *)(M + at);
        } else {
            uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool in = KC ? (x < R && k + e < kend) : (k < kend && x + e < R);
                if (in) w[e >> 1] |= (uint32_t)M[at + e] << (16 * (e & 1));
            }
            v[h] = uint4{w[0], w[1], w[2], w[3]};
        }
    }
}
template <bool KC>
__device__ __forceinline__ void slice_store(uint16_t *S, const uint4 (&v)[2]) {
    const int tid = threadIdx.x;
    if constexpr (KC) {
        uint2 *d = (uint2 *)(S + (tid >> 2) * GP + (tid & 3) * 16);
        d[0] = uint2{v[0].x, v[0].y};
        d[1] = uint2{v[0].z, v[0].w};
        d[2] = uint2{v[1].x, v[1].y};
        d[3] = uint2{v[1].z, v[1].w};
    } else {
        const uint32_t a[4] = {v[0].x, v[0].y, v[0].z, v[0].w};
        const uint32_t b[4] = {v[1].x, v[1].y, v[1].z, v[1].w};
        uint16_t *d = S + (tid & 7) * 8 * GP + (tid >> 3) * 2;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t lo = (a[e >> 1] >> (16 * (e & 1))) & 0xffffu;
            const uint32_t hi = (b[e >> 1] >> (16 * (e & 1))) & 0xffffu;
            *(uint32_t *)(d + e * GP) = lo | (hi << 16);
        }
    }
}

// C[M x N] (+)= op(A)[M x K] op(B)[K x N]; A, B BF16 row-major with leading
// dimensions lda, ldb (op = transpose when TA / TB).  256 threads = 4 waves,
// each wave owns a 32 x 32 quarter of the 64 x 64 tile (2 x 2 MFMA tiles).
// grid.z splits K, kper a multiple of GK per block; with splits > 1 the
// partial sums are added atomically into C (which the caller zeroes) and the
// epilogue must be plain.  At the network's sizes (K 64 or 256, N up to 256)
// it is bound by its loads and launches: 16-byte loads of the next stage run
// under the products of this one.  8192 x 256 x 256: 37 -> 8 us, its weight
// gradient over 32 splits 48 -> 14 us.
template <bool TA, bool TB>
__global__ __launch_bounds__(256) void k_gemm_bf16(int M, int N, int K, const uint16_t *__restrict__ A,
                                                   int lda, bool va, const uint16_t *__restrict__ B,
                                                   int ldb, bool vb, float *C, int ldc,
                                                   uint16_t *Cb, const float *__restrict__ bias,
                                                   int relu, int kper, int atomic) {
    __shared__ __align__(16) uint16_t As[GT * GP], Bs[GT * GP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m0 = blockIdx.y * GT, n0 = blockIdx.x * GT;
    const int kbeg = blockIdx.z * kper, kend = min(K, kbeg + kper);
    if (kbeg >= kend) return;   // the whole block: nothing to add
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int r16 = lane & 15, kq = (lane >> 4) * 4;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint4 ra[2], rb[2];
    slice_load<!TA>(ra, A, lda, m0, M, kbeg, kend, va);
    slice_load<TB>(rb, B, ldb, n0, N, kbeg, kend, vb);
    for (int k0 = kbeg; k0 < kend; k0 += GK) {
        slice_store<!TA>(As, ra);
        slice_store<TB>(Bs, rb);
        __syncthreads();
        if (k0 + GK < kend) {
            slice_load<!TA>(ra, A, lda, m0, M, k0 + GK, kend, va);
            slice_load<TB>(rb, B, ldb, n0, N, k0 + GK, kend, vb);
        }
#pragma unroll
        for (int ks = 0; ks < GK; ks += 32) {
            Frag a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint16_t *pa = As + (wm + 16 * i + r16) * GP + ks + kq;
                const uint16_t *pb = Bs + (wn + 16 * i + r16) * GP + ks + kq;
                a[i] = Frag{*(const uint2 *)pa, *(const uint2 *)(pa + 16)};
                b[i] = Frag{*(const uint2 *)pb, *(const uint2 *)(pb + 16)};
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = mma32(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
    // result layout: column = lane % 16, rows 4 (lane / 16) + q
    const int c16 = lane & 15, rq = (lane >> 4) * 4;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int gm = m0 + wm + 16 * i + rq + q, gn = n0 + wn + 16 * j + c16;
                if (gm >= M || gn >= N) continue;
                float v = acc[i][j][q];
                if (atomic) {
                    atomicAdd(&C[(size_t)gm * ldc + gn], v);
                    continue;
                }
                if (bias) v += bias[gn];
                if (relu) v = v > 0.f ? v : 0.f;
                if (C) C[(size_t)gm * ldc + gn] = v;
                if (Cb) Cb[(size_t)gm * ldc + gn] = f2bf(v);
            }
}

__global__ void k_f2bf(size_t n, const float *__restrict__ x, uint16_t *y) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        y[i] = f2bf(x[i]);
}

// dH <- dH * (H > 0) (FP32), and its BF16 copy
__global__ void k_relu_bwd(size_t n, const float *__restrict__ H, float *dH, uint16_t *dHb) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        const float g = H[i] > 0.f ? dH[i] : 0.f;
        dH[i] = g;
        if (dHb) dHb[i] = f2bf(g);
    }
}

// out[y][j] = sum of column j over the rows [y split, (y + 1) split) of dY, y =
// blockIdx.y, in an order that depends on the rows alone, so that equal inputs
// give equal bits: 256 partial sums of the rows r, r + 256, ..., then a tree.  A
// thread holds the partial sums of K lanes of one column; a wave reads 64 / COLS
// rows of COLS columns at a time, 16 or 8 loads in flight per thread.  Bound by
// the loads of the few CUs it runs on.
constexpr int CS_THREADS = 1024, CS_LANES = 256;
template <int COLS>
__global__ __launch_bounds__(CS_THREADS) void k_column_sums(int n, int m, int split,
                                                            const float *__restrict__ dY,
                                                            float *__restrict__ out) {
    constexpr int RG = CS_THREADS / COLS, K = CS_LANES / RG, U = COLS == 16 ? 4 : 1;
    const int c = threadIdx.x % COLS, r = threadIdx.x / COLS;
    const int j = blockIdx.x * COLS + c;
    const long long i0 = (long long)blockIdx.y * split;
    const unsigned rows = n - i0 < split ? (unsigned)(n - i0) : (unsigned)split;
    const float *__restrict__ p = dY + i0 * m + j;
    float s[K];
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] = 0.f;
    if (j < m) {
        unsigned i = r;
        for (; i + (U * K - 1) * RG < rows; i += U * CS_LANES) {
            float v[U][K];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < K; ++k) v[u][k] = p[(size_t)(i + (u * K + k) * RG) * m];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < K; ++k) s[k] += v[u][k];
        }
        for (; i < rows; i += CS_LANES)
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (i + k * RG < rows) s[k] += p[(size_t)(i + k * RG) * m];
    }
#pragma unroll
    for (int o = K / 2; o > 0; o >>= 1)
#pragma unroll
        for (int k = 0; k < o; ++k) s[k] += s[k + o];
    __shared__ float red[RG][COLS];
    red[r][c] = s[0];
    __syncthreads();
    for (int o = RG / 2; o > 0; o >>= 1) {
        if (r < o) red[r][c] += red[r + o][c];
        __syncthreads();
    }
    if (r == 0 && j < m) out[(long long)blockIdx.y * m + j] = red[0][c];
}

// masked MSE: loss += sum mask (Y - T)^2 / count;  dY = 2 mask (Y - T) / count
__global__ void k_mse(size_t n, const float *__restrict__ Y, const float *__restrict__ T,
                      const float *__restrict__ mask, float inv_count, float *dY, float *loss) {
    __shared__ float red[256];
    float s = 0.f;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        const float d = (Y[i] - T[i]) * mask[i];
        s += d * d;
        dY[i] = 2.f * d * inv_count;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicAdd(loss, red[0] * inv_count);
}

// Adam on FP32 master weights, then the BF16 copy
__global__ void k_adam(size_t n, float *w, const float *__restrict__ g, float *m1, float *m2,
                       float lr, float b1, float b2, float eps, float c1, float c2, uint16_t *wb) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float a = b1 * m1[i] + (1.f - b1) * gi, b = b2 * m2[i] + (1.f - b2) * gi * gi;
        m1[i] = a;
        m2[i] = b;
        const float v = w[i] - lr * (a * c1) / (sqrtf(b * c2) + eps);
        w[i] = v;
        if (wb) wb[i] = f2bf(v);
    }
}

// ---------------------------------------------------------------------------
// Fused inference of the three-layer guess network.  A block of 8 waves keeps
// the weights in registers (wave w the columns [32 w, 32 w + 32) of both
// hidden layers, waves 0-2 one column tile of the output layer) and takes
// row tiles of 32 through all three layers in turn; the BF16 hidden
// activations stay in LDS, rounded where the layered GEMMs round them, and
// the K loop runs in the same MFMA steps in the same order, so the output
// equals the layered forward pass bit for bit.  Reading the 200 KB of weights
// from L2 for every 32 rows was what bound the kernel (51,360 rows: 28.5 us;
// with one block per CU that reads them once: 21.9 us).
// ---------------------------------------------------------------------------
constexpr int FR = 32;                          // rows per tile
constexpr int FW = 8;                           // waves per block
constexpr int FIN = 64, FH = 256, FOUT = 36;
constexpr int FXP = FIN + 12, FHP = FH + 12;    // LDS row pitches (BF16): 8-byte rows, skewed banks

// Packed fragment layout of a K x N BF16 matrix (row-major, ld = N): for K
// step s (16 rows) and column tile t (16 columns), lane l holds rows
// 16 s + 4 (l / 16) + j, j < 4, of column 16 t + l % 16 (zero past N):
// Wp[((s * ntile + t) * 64 + l) * 4 + j].
__global__ void k_pack_frag(int K, int N, const uint16_t *__restrict__ W, uint16_t *Wp) {
    const int ntile = (N + 15) / 16;
    const size_t total = (size_t)(K / 16) * ntile * 256;
    for (size_t x = blockIdx.x * (size_t)blockDim.x + threadIdx.x; x < total;
         x += (size_t)gridDim.x * blockDim.x) {
        const int j = x & 3, l = (x >> 2) & 63;
        const size_t st = x >> 8;
        const int t = (int)(st % ntile), sk = (int)(st / ntile);
        const int k = 16 * sk + 4 * (l >> 4) + j, n = 16 * t + (l & 15);
        Wp[x] = n < N ? W[(size_t)k * N + n] : (uint16_t)0;
    }
}

// B fragments of column tile t of a packed K x N matrix, K in steps of 32
template <int K>
__device__ __forceinline__ void frag_load(Frag (&w)[K / 32], const uint16_t *__restrict__ Wp,
                                          int ntile, int t) {
    const uint2 *__restrict__ p = (const uint2 *)Wp + (size_t)t * 64 + (threadIdx.x & 63);
#pragma unroll
    for (int s = 0; s < K / 32; ++s)
        w[s] = Frag{p[(size_t)(2 * s) * ntile * 64], p[(size_t)(2 * s + 1) * ntile * 64]};
}
// A fragment of rows row0 .. row0 + 15, k step s, from LDS
__device__ __forceinline__ Frag frag_a(const uint16_t *S, int pitch, int row0, int s) {
    const int lane = threadIdx.x & 63;
    const uint16_t *p = S + (row0 + (lane & 15)) * pitch + 32 * s + 4 * (lane >> 4);
    return Frag{*(const uint2 *)p, *(const uint2 *)(p + 16)};
}

__global__ __launch_bounds__(64 * FW) void k_mlp_forward(int n, const uint16_t *__restrict__ X,
                                                         const uint16_t *__restrict__ W1p,
                                                         const float *__restrict__ b1,
                                                         const uint16_t *__restrict__ W2p,
                                                         const float *__restrict__ b2,
                                                         const uint16_t *__restrict__ W3p,
                                                         const float *__restrict__ b3, float *Y) {
    __shared__ __align__(16) uint16_t xs[FR * FXP];
    __shared__ __align__(16) uint16_t h1[FR * FHP];
    __shared__ __align__(16) uint16_t h2[FR * FHP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, rq = (lane >> 4) * 4;
    const int ntile = (n + FR - 1) / FR;
    // this thread's 8 bytes of an input tile; rows past n are zero
    const int xr = tid / (FIN / 4), xc = tid % (FIN / 4) * 4;
    static_assert(64 * FW == FR * (FIN / 4), "one 8-byte vector per thread and input tile");
    auto xload = [&](int t) {
        uint2 v = {0u, 0u};
        const int r = t * FR + xr;
        if (t < ntile && r < n) v = *(const uint2 *)(X + (size_t)r * FIN + xc);
        return v;
    };
    uint2 xv = xload(blockIdx.x);
    Frag w1[2][FIN / 32], w2[2][FH / 32], w3[FH / 32];
    float bb1[2], bb2[2], bb3 = 0.f;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        frag_load<FIN>(w1[c], W1p, FH / 16, 2 * wave + c);
        frag_load<FH>(w2[c], W2p, FH / 16, 2 * wave + c);
        bb1[c] = b1[32 * wave + 16 * c + c16];
        bb2[c] = b2[32 * wave + 16 * c + c16];
    }
    // output layer: 2 row tiles x 3 column tiles on waves 0..5
    const int orow = 16 * (wave & 1), ocol = 16 * (wave >> 1) + c16;
    if (wave < 6) {
        frag_load<FH>(w3, W3p, 3, wave >> 1);
        if (ocol < FOUT) bb3 = b3[ocol];
    }
    for (int t = blockIdx.x; t < ntile; t += gridDim.x) {
        *(uint2 *)(xs + xr * FXP + xc) = xv;
        __syncthreads();
        xv = xload(t + gridDim.x);   // the next tile's rows, under this tile's layers
        auto hidden = [&](const uint16_t *in, int pitch, auto &w, const float (&bias)[2],
                          uint16_t *out, auto ksteps) {
            constexpr int KS = decltype(ksteps)::value;
            f32x4 acc[2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[i][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const Frag a = frag_a(in, pitch, 16 * i, s);
#pragma unroll
                    for (int c = 0; c < 2; ++c) acc[i][c] = mma32(a, w[c][s], acc[i][c]);
                }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float v = acc[i][c][q] + bias[c];
                        v = v > 0.f ? v : 0.f;
                        out[(16 * i + rq + q) * FHP + 32 * wave + 16 * c + c16] = f2bf(v);
                    }
        };
        hidden(xs, FXP, w1, bb1, h1, std::integral_constant<int, FIN / 32>{});
        __syncthreads();
        hidden(h1, FHP, w2, bb2, h2, std::integral_constant<int, FH / 32>{});
        __syncthreads();
        // the next tile's xs and h1 are written after this barrier, and its h2
        // after two more, so no barrier follows the output layer
        if (wave < 6) {
            f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < FH / 32; ++s) acc = mma32(frag_a(h2, FHP, orow, s), w3[s], acc);
            if (ocol < FOUT)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = t * FR + orow + rq + q;
                    if (row < n) Y[(size_t)row * FOUT + ocol] = acc[q] + bb3;
                }
        }
    }
}

// Resident blocks of the fused forward pass: one per CU.
static int mlp_blocks(int ntile) {
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        ncu < 1)
        ncu = 256;
    return ntile < ncu ? ntile : ncu;
}

static inline dim3 grid1(size_t n) {
    size_t b = (n + 255) / 256;
    if (b > 4096) b = 4096;
    if (b < 1) b = 1;
    return dim3((unsigned)b);
}

}  // namespace fsim

using namespace fsim;

extern "C" fsim_status fsim_gemm_bf16(int32_t M, int32_t N, int32_t K, const uint16_t *A,
                                      int32_t lda, int32_t ta, const uint16_t *B, int32_t ldb,
                                      int32_t tb, float *C, int32_t ldc, uint16_t *Cb,
                                      const float *bias, int32_t relu, int32_t ksplit,
                                      void *stream) {
    if (M <= 0 || N <= 0 || K <= 0 || !A || !B || (!C && !Cb)) return FSIM_EINVAL;
    if (ksplit < 1) ksplit = 1;
    if (ksplit > 1 && (!C || Cb || bias || relu)) return FSIM_EINVAL;
    dim3 g((N + GT - 1) / GT, (M + GT - 1) / GT, ksplit);
    // whole stages per split, so that every split starts on a vector boundary
    const long long per = ((long long)K + ksplit - 1) / ksplit;
    const int kper = ksplit > 1 ? (int)((per + GK - 1) / GK * GK) : K;
    // 16-byte loads need an aligned base and a row pitch of whole vectors
    const bool va = ((uintptr_t)A & 15) == 0 && lda % 8 == 0;
    const bool vb = ((uintptr_t)B & 15) == 0 && ldb % 8 == 0;
    auto kernel = ta ? (tb ? k_gemm_bf16<true, true> : k_gemm_bf16<true, false>)
                     : (tb ? k_gemm_bf16<false, true> : k_gemm_bf16<false, false>);
    hipLaunchKernelGGL(kernel, g, dim3(256), 0, (hipStream_t)stream, M, N, K, A, lda, va, B, ldb,
                       vb, C, ldc, Cb, bias, relu, kper, ksplit > 1 ? 1 : 0);
    return hipGetLastError() == hipSuccess ? FSIM_OK : FSIM_EHIP;
}

extern "C" fsim_status fsim_f32_to_bf16(int64_t n, const float *x, uint16_t *y, void *stream) {
    if (n < 0 || (n > 0 && (!x || !y))) return FSIM_EINVAL;
    if (n == 0) return FSIM_OK;
    hipLaunchKernelGGL(k_f2bf, grid1(n), dim3(256), 0, (hipStream_t)stream, (size_t)n, x, y);
    return hipGetLastError() == hipSuccess ? FSIM_OK : FSIM_EHIP;
}

extern "C" fsim_status fsim_relu_backward(int64_t n, const float *H, float *dH, uint16_t *dHb,
                                          void *stream) {
    if (n <= 0 || !H || !dH) return FSIM_EINVAL;
    hipLaunchKernelGGL(k_relu_bwd, grid1(n), dim3(256), 0, (hipStream_t)stream, (size_t)n, H, dH, dHb);
    return hipGetLastError() == hipSuccess ? FSIM_OK : FSIM_EHIP;
}

// Up to CS_ONE_PASS rows in one launch over blocks of 16 columns, which reads a
// matrix on few CUs (from memory, 2048 x 256: 5.7 us, 7.4 in two launches).  More
// rows in runs of CS_SPLIT whose sums, in ws, a second launch sums (4096 x 256:
// 7.5 us against 9.5, 8192 x 256: 7.6 against 17, 32768 x 36: 7.6 against 44),
// with 32 columns to a block, whole cache lines (32768 x 256: 9.8 us, 14.6 with
// 16 columns).  Without ws in one launch all the same.
constexpr int CS_ONE_PASS = 2048, CS_SPLIT = 1024, CS_SPLITS_MAX = 32768;
extern "C" fsim_status fsim_bias_grad_ws(int32_t n, int32_t m, const float *dY, float *db,
                                         float *ws, void *stream) {
    if (n <= 0 || m <= 0 || !dY || !db) return FSIM_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    auto sums = [&](auto cols, int rows, int split, const float *x, float *out) {
        constexpr int C = decltype(cols)::value;
        hipLaunchKernelGGL((k_column_sums<C>), dim3((m - 1) / C + 1, (rows - 1) / split + 1),
                           dim3(CS_THREADS), 0, s, rows, m, split, x, out);
    };
    const std::integral_constant<int, 16> narrow;
    const std::integral_constant<int, 32> wide;
    if (n <= CS_ONE_PASS || !ws) {
        sums(narrow, n, n, dY, db);
    } else {
        int split = CS_SPLIT;
        while ((n - 1) / split + 1 > CS_SPLITS_MAX) split *= 2;
        const int ns = (n - 1) / split + 1;
        sums(wide, n, split, dY, ws);
        sums(wide, ns, ns, ws, db);
    }
    return hipGetLastError() == hipSuccess ? FSIM_OK : FSIM_EHIP;
}
extern "C" fsim_status fsim_bias_grad(int32_t n, int32_t m, const float *dY, float *db,
                                      void *stream) {
    return fsim_bias_grad_ws(n, m, dY, db, nullptr, stream);
}

constexpr int64_t MSE_SHARE = 256 * 36;
extern "C" fsim_status fsim_mse(int64_t n, const float *Y, const float *T, const float *mask,
                                float inv_count, float *dY, float *loss, void *stream) {
    if (n <= 0 || !Y || !T || !mask || !dY || !loss) return FSIM_EINVAL;
    // every block ends in an add to the one loss word, and these queue up at 13 ns
    // each, while a block streams 8 GB/s: 128 blocks to start with, then one for
    // every MSE_SHARE values up to six to a CU.  8192 x 36 values take 5.2 us
    // (15.5 in 1024 blocks), 131072 x 36 20.5 (44.9 in 128, 58.9 in 4096),
    // 1048576 x 36 116 (560 in 128, 126 in 4096).
    const int64_t most = n / MSE_SHARE < 128 ? 128 : (n / MSE_SHARE > 1536 ? 1536 : n / MSE_SHARE);
    dim3 g = grid1(n);
    if (g.x > most) g.x = (unsigned)most;
    hipLaunchKernelGGL(k_mse, g, dim3(256), 0, (hipStream_t)stream, (size_t)n, Y, T, mask,
                       inv_count, dY, loss);
    return hipGetLastError() == hipSuccess ? FSIM_OK : FSIM_EHIP;
}

extern "C" fsim_status fsim_adam(int64_t n, float *w, const float *g, float *m1, float *m2,
                                 float lr, float b1, float b2, float eps, int32_t step,
                                 uint16_t *wb, void *stream) {
    if (n <= 0 || !w || !g || !m1 || !m2 || step < 1) return FSIM_EINVAL;
    float pb1 = 1.f, pb2 = 1.f;
    for (int i = 0; i < step; ++i) {
        pb1 *= b1;
        pb2 *= b2;
    }
    const float c1 = 1.f / (1.f - pb1), c2 = 1.f / (1.f - pb2);
    hipLaunchKernelGGL(k_adam, grid1(n), dim3(256), 0, (hipStream_t)stream, (size_t)n, w, g, m1,
                       m2, lr, b1, b2, eps, c1, c2, wb);
    return hipGetLastError() == hipSuccess ? FSIM_OK : FSIM_EHIP;
}

extern "C" fsim_status fsim_mlp_pack(int32_t K, int32_t N, const uint16_t *W, uint16_t *Wp,
                                     void *stream) {
    if (K <= 0 || K % 16 || N <= 0 || !W || !Wp) return FSIM_EINVAL;
    if ((uintptr_t)Wp & 7) return FSIM_EINVAL;      // read back as 8-byte fragments
    const size_t total = (size_t)(K / 16) * ((N + 15) / 16) * 256;
    hipLaunchKernelGGL(k_pack_frag, grid1(total), dim3(256), 0, (hipStream_t)stream, K, N, W, Wp);
    return hipGetLastError() == hipSuccess ? FSIM_OK : FSIM_EHIP;
}

extern "C" fsim_status fsim_mlp_forward(int32_t n, const uint16_t *X, const uint16_t *W1p,
                                        const float *b1, const uint16_t *W2p, const float *b2,
                                        const uint16_t *W3p, const float *b3, float *Y,
                                        void *stream) {
    if (n < 0) return FSIM_EINVAL;
    if (n == 0) return FSIM_OK;
    if (!X || !W1p || !b1 || !W2p || !b2 || !W3p || !b3 || !Y) return FSIM_EINVAL;
    // the kernel reads X rows and weight fragments 8 bytes at a time
    for (const void *q : {(const void *)X, (const void *)W1p, (const void *)W2p, (const void *)W3p})
        if ((uintptr_t)q & 7) return FSIM_EINVAL;
    hipLaunchKernelGGL(k_mlp_forward, dim3(mlp_blocks((n + FR - 1) / FR)), dim3(64 * FW), 0,
                       (hipStream_t)stream, n, X, W1p, b1, W2p, b2, W3p, b3, Y);
    return hipGetLastError() == hipSuccess ? FSIM_OK : FSIM_EHIP;
}
