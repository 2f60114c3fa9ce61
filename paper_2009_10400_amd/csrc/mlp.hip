// Learned surrogate: a bfloat16 multilayer perceptron trained and evaluated on
// the matrix cores of gfx950 (v_mfma_f32_16x16x32_bf16, FP32 accumulation).
// C-ABI in include/tled_surrogate.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/tled_surrogate.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

constexpr int kThreads = 256;
constexpr int BM = 64, BN = 64, BK = 64, BKP = BK + 8;   // LDS rows padded against bank conflicts

__device__ inline float bf2f(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }
// float -> bfloat16 bits by the hardware convert (v_cvt_pk_bf16_f32 on gfx950,
// round to nearest even).
__device__ inline uint16_t bf16_bits(float x) {
    const __bf16 h = static_cast<__bf16>(x);
    uint16_t u;
    __builtin_memcpy(&u, &h, 2);
    return u;
}

// Two floats to bfloat16 bits in one word (one v_cvt_pk_bf16_f32; a convert per value and
// the shifts to join them took five instructions).
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// Logistic function from the hardware base-2 exponential and reciprocal
// (v_exp_f32, v_rcp_f32; each within about 1 ulp, far below the bfloat16
// rounding the activations then take).  Every SiLU of the forward passes and its
// derivative in the backward pass use this one function.
__device__ __forceinline__ float sigmoidf_hw(float z) {
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}

// sin(2 pi t) or cos(2 pi t) for t in revolutions: reduced to [-1/2, 1/2] (exact
// for |t| < 2^22), then the hardware sine/cosine, which take revolutions.
__device__ __forceinline__ float fourier_feature(float t, bool sine) {
    const float r = t - rintf(t);
    return sine ? __builtin_amdgcn_sinf(r) : __builtin_amdgcn_cosf(r);
}

// Revolutions of Fourier feature f at x: frequency (3 floats) times position.
__device__ __forceinline__ float feature_turns(const float *__restrict__ Bf, float x0, float x1, float x2) {
    return Bf[0] * x0 + Bf[1] * x1 + Bf[2] * x2;
}

enum { EPI_F32 = 0, EPI_BIAS_SILU = 1, EPI_BIAS_F32 = 2, EPI_SILU_BACK = 3 };
// How an operand tile is read from global memory: element by element (any
// strides), 16-byte vectors along k (k contiguous), or 16-byte vectors along
// the tile's rows (rows contiguous).  Chosen on the host from strides and alignment.
enum { LD_SCALAR = 0, LD_KVEC = 1, LD_RVEC = 2 };

// One thread's share (8 values) of half h (k in [k0 + 32h, k0 + 32h + 32)) of a
// 64 x 64 operand tile X(r, k) = X[r*sr + k*sk], rows r0.., zero outside r < R, k < ke,
// packed two bfloat16 per 32-bit word (value i in the low half of word i/2 when even).
struct TileRegs {
    uint4 w;
};

__device__ inline uint4 pack8(const uint16_t (&e)[8]) {
    return make_uint4(uint32_t(e[0]) | (uint32_t(e[1]) << 16), uint32_t(e[2]) | (uint32_t(e[3]) << 16),
                      uint32_t(e[4]) | (uint32_t(e[5]) << 16), uint32_t(e[6]) | (uint32_t(e[7]) << 16));
}

// Value i of a thread's share, as a float.
__device__ inline float tile_value(const TileRegs &q, int i) {
    const uint32_t u = i < 2 ? q.w.x : i < 4 ? q.w.y : i < 6 ? q.w.z : q.w.w;
    return bf2f(uint16_t((i & 1) ? (u >> 16) : (u & 0xffffu)));
}

template <int MODE>
__device__ inline void tile_load(TileRegs &q, const uint16_t *__restrict__ X, long sr, long sk, int r0, int R,
                                 int k0, int ke, int t, int h) {
    uint16_t e[8];
    if (MODE == LD_KVEC) {
        const int r = r0 + (t >> 2), k = k0 + 32 * h + (t & 3) * 8;
        if (r < R && k + 8 <= ke) {
            q.w = *reinterpret_cast<const uint4 *>(X + r * sr + k);
            return;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = (r < R && k + i < ke) ? X[r * sr + k + i] : uint16_t(0);
    } else if (MODE == LD_RVEC) {
        const int k = k0 + 32 * h + (t >> 3), r = r0 + (t & 7) * 8;
        if (k < ke && r + 8 <= R) {
            q.w = *reinterpret_cast<const uint4 *>(X + k * sk + r);
            return;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = (k < ke && r + i < R) ? X[k * sk + r + i] : uint16_t(0);
    } else {
        const int r = r0 + (t >> 2), k = k0 + 32 * h + (t & 3) * 8;
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = (r < R && k + i < ke) ? X[r * sr + (k + i) * sk] : uint16_t(0);
    }
    q.w = pack8(e);
}

// Stores a thread's share of half h of the 64-deep tile at k offset koff into an
// LDS operand of row pitch P: S[r P + k], or, for tiles read with rows contiguous,
// S[k P + r] as loaded (one 16-byte store either way; the MFMA fragments of a
// k-major operand are then fetched with the transpose read, see frag()).
template <int MODE>
__device__ inline void tile_store(const TileRegs &q, uint16_t *S, int P, int koff, int t, int h) {
    if (MODE == LD_RVEC) {
        const int k = koff + 32 * h + (t >> 3), r = (t & 7) * 8;
        *reinterpret_cast<uint4 *>(&S[k * P + r]) = q.w;
    } else {
        const int r = t >> 2, k = koff + 32 * h + (t & 3) * 8;
        *reinterpret_cast<uint4 *>(&S[r * P + k]) = q.w;
    }
}

// The 16 x 32 MFMA operand fragment of rows r0..r0+15, k in [k0, k0 + 32), of an
// LDS operand of row pitch P: lane l gets X(r0 + l%16, k0 + 8(l/16) + 0..7).  From
// an r-major operand (S[r P + k]) that is one 16-byte read.  From a k-major one
// (S[k P + r]) it takes two ds_read_b64_tr_b16: each lane of a 16-lane group reads
// 4 consecutive values of one k row, and the instruction hands lane i of the group
// value i%4 of lane 4j + i/4's read as its value j; lane 4j + q therefore reads row
// k + j at columns r0 + 4q.., which gives lane i the 4 k values of column r0 + i.
template <int MODE>
__device__ inline bf16x8 frag(const uint16_t *S, int P, int r0, int k0, int l) {
    if (MODE == LD_RVEC) {
        const int k = k0 + 8 * (l >> 4) + ((l & 15) >> 2), r = r0 + 4 * (l & 3);
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(&S[k * P + r]));
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(&S[(k + 4) * P + r]));
        const i16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, v);
    } else {
        return *reinterpret_cast<const bf16x8 *>(&S[(r0 + (l & 15)) * P + k0 + 8 * (l >> 4)]);
    }
}

// The epilogue of a wavefront's 32 x 32 output block (see gemm_kernel).
template <int EPI>
__device__ inline void gemm_epilogue(const f32x4 (&acc)[2][2], int m0, int n0, int wm, int wn, int l, int M, int N,
                                     float *__restrict__ C, long scm, long scn, uint16_t *__restrict__ Act,
                                     const float *__restrict__ bias) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm + 16 * i + 4 * (l >> 4) + r;
                const int n = n0 + wn + 16 * j + (l & 15);
                if (m >= M || n >= N) continue;
                float v = acc[i][j][r];
                if (EPI == EPI_F32) {
                    if (gridDim.z > 1) C[size_t(m) * N + n] = v;
                    else C[m * scm + n * scn] = v;
                } else if (EPI == EPI_BIAS_F32) {
                    C[m * scm + n * scn] = v + bias[n];
                } else if (EPI == EPI_SILU_BACK) {
                    const float z = bias[size_t(m) * N + n], sg = sigmoidf_hw(z);
                    Act[size_t(m) * N + n] = bf16_bits(v * sg * (1.0f + z * (1.0f - sg)));
                } else {
                    const float z = v + bias[n];
                    C[m * scm + n * scn] = z;
                    Act[size_t(m) * N + n] = bf16_bits(z * sigmoidf_hw(z));
                }
            }
}

// EPI_SILU_BACK through LDS: the workgroup's 64 x 64 FP32 products go to LDS, then
// each thread takes 16 consecutive columns of one row, so the pre-activations are read
// and dZ written in 16-byte vectors (the arithmetic of gemm_epilogue, element by
// element).  tile: at least 64 x 68 floats of LDS that the k loop no longer reads.
// (Split-K partials written the same way measured slower than gemm_epilogue's.)
__device__ inline void silu_back_epilogue(const f32x4 (&acc)[2][2], float *tile, int m0, int n0, int wm, int wn,
                                          int l, int t, int M, int N, uint16_t *__restrict__ Act,
                                          const float *__restrict__ Z) {
    constexpr int TP = BN + 4;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) tile[(wm + 16 * i + 4 * (l >> 4) + r) * TP + wn + 16 * j + (l & 15)] = acc[i][j][r];
    __syncthreads();
    const int row = t >> 2, c0 = 16 * (t & 3), m = m0 + row;
    if (m >= M) return;
#pragma unroll
    for (int q = 0; q < 16; q += 8) {
        const int n = n0 + c0 + q;
        const float *v = tile + row * TP + c0 + q;
        if (N % 8 == 0 && n + 8 <= N) {
            const float4 za = *reinterpret_cast<const float4 *>(Z + size_t(m) * N + n);
            const float4 zb = *reinterpret_cast<const float4 *>(Z + size_t(m) * N + n + 4);
            const float zz[8] = {za.x, za.y, za.z, za.w, zb.x, zb.y, zb.z, zb.w};
            uint16_t h[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float z = zz[c], sg = sigmoidf_hw(z);
                h[c] = bf16_bits(v[c] * sg * (1.0f + z * (1.0f - sg)));
            }
            *reinterpret_cast<uint4 *>(Act + size_t(m) * N + n) = pack8(h);
        } else {
            for (int c = 0; c < 8 && n + c < N; ++c) {
                const float z = Z[size_t(m) * N + n + c], sg = sigmoidf_hw(z);
                Act[size_t(m) * N + n + c] = bf16_bits(v[c] * sg * (1.0f + z * (1.0f - sg)));
            }
        }
    }
}

// XCD-aware tile order.  The hardware hands workgroup H (x fastest, then y, then z)
// to XCD H mod 8; with the tile count a multiple of 8, each XCD takes one contiguous
// range of the tiles in that order instead, so the workgroups that share operand rows
// (the column tiles of one row block; all tiles of one k chunk) run on the same XCD
// and read them through its L2 once.  Only which workgroup computes a tile changes.
constexpr int kNumXcd = 8;
__device__ inline void tile_of_block(int &bx, int &by, int &bz) {
    const int nx = int(gridDim.x), ny = int(gridDim.y), T = nx * ny * int(gridDim.z);
    int H = int(blockIdx.x) + nx * (int(blockIdx.y) + ny * int(blockIdx.z));
    if (T % kNumXcd == 0) H = (H % kNumXcd) * (T / kNumXcd) + H / kNumXcd;
    bx = H % nx;
    by = (H / nx) % ny;
    bz = H / (nx * ny);
}

// C = A B with A(m,k) = A[m*lda + k], B(k,n) = B[k*sbk + n*sbn] (bfloat16 bits).
// 64x64 output tile per workgroup of four wavefronts, each wavefront 32x32 as
// 2x2 MFMA 16x16x32 tiles.  Lane l of a 16x16x32 MFMA supplies A[l%16][8(l/16)..+7]
// and B[8(l/16)..+7][l%16] and receives D[4(l/16)+r][l%16], r = 0..3.  k runs in
// 64-deep LDS tiles (two 32-deep MFMA steps each, in increasing k).
// Epilogues: EPI_F32 C(m,n) = acc; EPI_BIAS_F32 C = acc + bias[n];
// EPI_BIAS_SILU Z = acc + bias[n] (FP32 into C) and Act[m*N+n] = bf16(Z sigmoid(Z));
// EPI_SILU_BACK (backward through a SiLU; `bias` then points at the layer's FP32
// pre-activations z, row-major M x N): Act[m*N+n] = bf16(acc s (1 + z (1 - s))),
// s = sigmoid(z).
// Split-K: workgroup z covers k in [z*kchunk, (z+1)*kchunk) and (EPI_F32 only)
// writes its partial tile to C + z*M*N (row-major M x N); a reduction follows.
// Four wavefronts per SIMD (four workgroups per CU, which is also what the 36.9 KB of
// LDS allows): the k loop waits on global memory, so occupancy is what hides the
// latency (64-68 VGPRs with the staged values packed two per register).
template <int EPI, int AM, int BMODE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void gemm_kernel(
    int M, int N, int K, const uint16_t *__restrict__ A, long lda, const uint16_t *__restrict__ B, long sbk,
    long sbn, float *__restrict__ C, long scm, long scn, uint16_t *__restrict__ Act, const float *__restrict__ bias,
    int kchunk) {
    static_assert(AM != LD_RVEC, "A has its rows along k");
    static_assert(BN == BK, "a k-major tile of B reuses the r-major tile's array");
    __shared__ __attribute__((aligned(16))) uint16_t As[2][BM][BKP];
    __shared__ __attribute__((aligned(16))) uint16_t Bt[2][BN][BKP];
    int bx, by, bz;
    tile_of_block(bx, by, bz);
    const int m0 = by * BM, n0 = bx * BN;
    const int t = threadIdx.x, w = t >> 6, l = t & 63;
    const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int kb = bz * kchunk, ke = min(K, kb + kchunk);
    if (gridDim.z > 1) C += size_t(bz) * M * N;
    const int ntiles = ke > kb ? (ke - kb + BK - 1) / BK : 0;
    TileRegs qa[2], qb[2];
    // double-buffered 64-deep k tiles: tile t + 1 is read from global memory into
    // registers while tile t is multiplied out of LDS; one barrier per tile
    if (ntiles > 0) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            tile_load<AM>(qa[h], A, lda, 1, m0, M, kb, ke, t, h);
            tile_load<BMODE>(qb[h], B, sbn, sbk, n0, N, kb, ke, t, h);
            tile_store<AM>(qa[h], &As[0][0][0], BKP, 0, t, h);
            tile_store<BMODE>(qb[h], &Bt[0][0][0], BKP, 0, t, h);
        }
    }
    __syncthreads();
    for (int tk = 0; tk < ntiles; ++tk) {
        const int k0 = kb + tk * BK, cur = tk & 1;
        const bool more = tk + 1 < ntiles;
        if (more) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                tile_load<AM>(qa[h], A, lda, 1, m0, M, k0 + BK, ke, t, h);
                tile_load<BMODE>(qb[h], B, sbn, sbk, n0, N, k0 + BK, ke, t, h);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (k0 + 32 * h >= ke) break;        // the same 32-deep MFMA steps as a 32-deep loop
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const bf16x8 a = frag<AM>(&As[cur][0][0], BKP, wm + 16 * i, 32 * h, l);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const bf16x8 b = frag<BMODE>(&Bt[cur][0][0], BKP, wn + 16 * j, 32 * h, l);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[i][j], 0, 0, 0);
                }
            }
        }
        if (more) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                tile_store<AM>(qa[h], &As[cur ^ 1][0][0], BKP, 0, t, h);
                tile_store<BMODE>(qb[h], &Bt[cur ^ 1][0][0], BKP, 0, t, h);
            }
        }
        __syncthreads();
    }
    if constexpr (EPI == EPI_SILU_BACK) {
        static_assert(sizeof(As) >= sizeof(float) * BM * (BN + 4), "the FP32 tile fits in the A tiles' LDS");
        silu_back_epilogue(acc, reinterpret_cast<float *>(&As[0][0][0]), m0, n0, wm, wn, l, t, M, N, Act, bias);
    } else {
        gemm_epilogue<EPI>(acc, m0, n0, wm, wn, l, M, N, C, scm, scn, Act, bias);
    }
}

// Fixed-order sum of split-K partials (nz x M x N, row-major) into C(m, n).  A block
// takes 64 elements; wavefront w adds partials w, w + 4, ... in order (64 consecutive
// elements per load), and the four sums are combined as (s0 + s1) + (s2 + s3).
__global__ __launch_bounds__(kThreads) void splitk_reduce_kernel(int nz, int M, int N, const float *__restrict__ part,
                                                                 float *__restrict__ C, long scm, long scn) {
    __shared__ float sh[4][64];
    const long MN = long(M) * N;
    const int w = threadIdx.x >> 6, c = threadIdx.x & 63;
    const long i = long(blockIdx.x) * 64 + c;
    float s = 0.f;
    if (i < MN) {
#pragma unroll 8
        for (int z = w; z < nz; z += 4) s += part[size_t(z) * MN + i];   // loads in flight, additions in order
    }
    sh[w][c] = s;
    __syncthreads();
    if (w == 0 && i < MN) {
        const long m = i / N, n = i % N;
        C[m * scm + n * scn] = (sh[0][c] + sh[1][c]) + (sh[2][c] + sh[3][c]);
    }
}

// Where the tiled forward kernel's copy of the hidden layers' weights lies.  Weight (unit o,
// input k) is in MFMA fragment (o / 16, k / 32) of 16 units x 32 inputs, as value k % 8 of
// lane o % 16 + 16 ((k % 32) / 8), so that a wavefront loads a fragment as 1 KB in a row.
// The tiled backward kernel's copy holds the transposes in the same order, of the layers
// after the first (the output layer's with its units padded to a multiple of 32).
struct PackedWeights {
    uint16_t *w, *t;              // null where those kernels do not apply
    int K0, W, depth, nko;        // nko: output units / 32, rounded up
    long biases;                  // where the output layer's biases begin
};
__device__ __forceinline__ unsigned packed_index(unsigned o, unsigned k, unsigned ksteps) {
    return ((o / 16 * ksteps + k / 32) * 64 + o % 16 + 16 * (k % 32 / 8)) * 8 + k % 8;
}

// The bfloat16 copies of parameter i: row-major and, of a hidden layer's weights, packed.
__device__ __forceinline__ void put_bf16(float v, long i, uint16_t *__restrict__ wb, const PackedWeights &pw) {
    const uint16_t h = bf16_bits(v);
    wb[i] = h;
    if (!pw.w) return;
    const unsigned W = pw.W, first = W * (pw.K0 + 1), other = W * (W + 1);   // a layer's weights and biases
    const bool in0 = unsigned(i) < first;
    const unsigned layer = in0 ? 0 : 1 + (unsigned(i) - first) / other, K = in0 ? pw.K0 : W;
    const unsigned e = in0 ? unsigned(i) : (unsigned(i) - first) % other;
    const unsigned o = e / K, k = e % K;
    if (layer == unsigned(pw.depth)) {
        if (i < pw.biases) pw.t[(layer - 1) * W * W + packed_index(k, o, pw.nko)] = h;
        return;
    }
    if (o >= W) return;                                   // a bias
    pw.w[(in0 ? 0 : W * pw.K0 + (layer - 1) * W * W) + packed_index(o, k, K / 32)] = h;
    if (!in0) pw.t[(layer - 1) * W * W + packed_index(k, o, W / 32)] = h;
}

// ---------------------------------------------------------------- weight gradients
//
// All layers' weight and bias gradients in one launch: job j is dW = A^T B with A the
// layer's dZ (n x M; the output layer's dY) and B its inputs (n x N), both row-major, and
// the bias gradient is the column sums of A.  A workgroup computes a 128 x 128 tile over
// one chunk of rows, four wavefronts of 64 x 64 each, and writes its FP32 partials where
// the gradient's elements lie in chunk z's partial vector.  grad_finish_kernel adds the
// chunks in order.  Bound by the latency of the operands' reads (two workgroups per CU, as
// their LDS and registers allow, and one 64-deep step ahead; a second step ahead gave
// nothing) and by the partials that leave the L2 at the end: matrix cores busy 4 us of 28.
// Five layers of 256, 16384 rows: 28 us and 8 us for the sums with the optimizer, where a
// GEMM and a reduction per layer (64 x 64 tiles, 64 chunks, so 75 MB of partials written
// and read), the output layer's own two kernels, its dZ and the optimizer took 103 us in 14
// launches.  2500 rows: 12.4 us, and 14.9 with loads under a branch per row, which the
// compiler waits for one by one before the first step.
struct GradJob {
    const uint16_t *A, *B;
    int lda, ldb, M, N;           // lda, ldb: multiples of 8, rows 16-byte aligned
    int first, nx;                // first tile, tiles along N
    long w_off, b_off;            // of the weights (M x N) and biases (M) in the gradient
};
constexpr int kGradJobs = 12;     // per launch
struct GradJobs {
    GradJob j[kGradJobs];
    int count, tiles;
};
// GP: an LDS row pitch of 8 banks past a multiple of 64, so that the 8 k rows of 16 columns
// that half a wavefront fetches with one transpose read lie in different banks
constexpr int GT = 128, GK = 64, GP = GT + 16;

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void weight_grad_kernel(
    GradJobs jobs, long n, int nz, long kchunk, float *__restrict__ part, long stride) {
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // [2][A, B][GK][GP]
    // the tiles of one chunk of rows on one XCD: they share their operands through its L2
    const int T = jobs.tiles, b = int(blockIdx.x);
    const int q = b / kNumXcd, z = nz % kNumXcd ? b / T : b % kNumXcd + kNumXcd * (q / T);
    const int tile = nz % kNumXcd ? b % T : q % T;
    int ji = 0;
    while (ji + 1 < jobs.count && tile >= jobs.j[ji + 1].first) ++ji;
    const GradJob &J = jobs.j[ji];
    const int lda = J.lda, ldb = J.ldb, nx = J.nx, tx = (tile - J.first) % nx, ty = (tile - J.first) / nx;
    const int m0 = GT * ty, n0 = GT * tx, t = threadIdx.x, w = t >> 6, l = t & 63;
    const int wm = 64 * (w >> 1), wn = 64 * (w & 1);
    const long kb = z * kchunk, ke = min(n, kb + kchunk);
    if (kb >= ke) return;
    const int lk = t >> 4, lr = 8 * (t & 15);          // staging: rows lk + 16 h, columns lr..lr+7
    const bool cols = tx == 0;
    const bool on = m0 + wm < J.M && n0 + wn < J.N;    // this wavefront has outputs
    // columns past a row are read as column 0: they reach no output
    const uint16_t *pa = J.A + kb * lda + (m0 + lr < lda ? m0 + lr : 0);
    const uint16_t *pb = J.B + kb * ldb + (n0 + lr < ldb ? n0 + lr : 0);
    const int nrow = int(ke - kb);
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    TileRegs qa[4], qb[4];
    // rows past the chunk are read as its last one (loads without branches stay in flight
    // together), then cleared
    auto load = [&](int k0) {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const long k = min(k0 + lk + 16 * h, nrow - 1);
            qa[h].w = *reinterpret_cast<const uint4 *>(pa + k * lda);
            qb[h].w = *reinterpret_cast<const uint4 *>(pb + k * ldb);
        }
    };
    auto store = [&](int buf, int k0) {
        uint16_t *S = lds + buf * (2 * GK * GP);
        if (k0 + GK > nrow)
#pragma unroll
            for (int h = 0; h < 4; ++h)
                if (k0 + lk + 16 * h >= nrow) qa[h].w = qb[h].w = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            *reinterpret_cast<uint4 *>(&S[(lk + 16 * h) * GP + lr]) = qa[h].w;
            *reinterpret_cast<uint4 *>(&S[(GK + lk + 16 * h) * GP + lr]) = qb[h].w;
        }
        if (cols)
#pragma unroll
            for (int h = 0; h < 4; ++h)
#pragma unroll
                for (int i = 0; i < 8; ++i) cs[i] += tile_value(qa[h], i);
    };
    // as frag<LD_RVEC>, with k in the order 4 (l / 16) + 0..3, 16 + 4 (l / 16) + 0..3 in both operands
    auto fragment = [&](const uint16_t *S, int r0, int k0) {
        const int k = k0 + 4 * (l >> 4) + ((l & 15) >> 2), r = r0 + 4 * (l & 3);
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(&S[k * GP + r]));
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(&S[(k + 16) * GP + r]));
        return __builtin_bit_cast(bf16x8, i16x8(__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)));
    };
    const int nk = (nrow + GK - 1) / GK;
    load(0);
    store(0, 0);
    __syncthreads();
    for (int tk = 0; tk < nk; ++tk) {
        const uint16_t *SA = lds + (tk & 1) * (2 * GK * GP), *SB = SA + GK * GP;
        const bool more = tk + 1 < nk;
        if (more) load((tk + 1) * GK);
        if (on)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                bf16x8 fa[4], fb[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) fa[i] = fragment(SA, wm + 16 * i, 32 * h);
#pragma unroll
                for (int j = 0; j < 4; ++j) fb[j] = fragment(SB, wn + 16 * j, 32 * h);
                // the inputs are the MFMA A operand: a lane ends with 4 consecutive columns of dW
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
            }
        if (more) store((tk + 1) & 1, (tk + 1) * GK);
        __syncthreads();
    }
    float *out = part + z * stride;
    if (on)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = m0 + wm + 16 * i + (l & 15);
            if (m >= J.M) continue;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = n0 + wn + 16 * j + 4 * (l >> 4);       // N is a multiple of 32
                if (c < J.N)
                    *reinterpret_cast<float4 *>(out + J.w_off + long(m) * J.N + c) =
                        make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            }
        }
    if (cols) {                                        // the 16 row phases, combined in order
        float *red = reinterpret_cast<float *>(lds);
#pragma unroll
        for (int i = 0; i < 8; ++i) red[lk * GT + lr + i] = cs[i];
        __syncthreads();
        if (t < GT && m0 + t < J.M) {
            float a = 0.f;
            for (int g = 0; g < 16; ++g) a += red[g * GT + t];
            out[J.b_off + m0 + t] = a;
        }
    }
}

// Adam's state and constants; w null: gradients only.
struct AdamArgs {
    float *w, *m, *v;
    float lr, c1, c2;
    uint16_t *wb;
    PackedWeights pw;
};

// The chunks' partial gradients added in a fixed order (wavefront w adds chunks w, w + 4,
// ..., the four sums are combined as (s0 + s1) + (s2 + s3)), then the gradient stored or,
// in a training step, Adam on the FP32 master parameters and their bfloat16 copies.  The
// last block adds the loss partials in order.  A block takes 256 elements.
template <bool ADAM>
__global__ __launch_bounds__(kThreads) void grad_finish_kernel(long P, int nz, long stride,
                                                               const float *__restrict__ part, float *__restrict__ g,
                                                               AdamArgs ad, int nloss, const float *__restrict__ lpart,
                                                               float scale, float *__restrict__ loss) {
    __shared__ float sh[4][kThreads];
    const int t = threadIdx.x, w = t >> 6;
    if (blockIdx.x == gridDim.x - 1) {
        float a = 0.f;
#pragma unroll 8
        for (int i = t; i < nloss; i += kThreads) a += lpart[i];     // loads in flight, additions in order
        sh[0][t] = a;
        __syncthreads();
        for (int k = kThreads / 2; k > 0; k >>= 1) {
            if (t < k) sh[0][t] += sh[0][t + k];
            __syncthreads();
        }
        if (t == 0) loss[0] = sh[0][0] * scale;
        return;
    }
    const long e0 = long(blockIdx.x) * kThreads + 4 * (t & 63);      // stride is a multiple of 4
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (e0 < stride) {
#pragma unroll 4
        for (int z = w; z < nz; z += 4) {
            const float4 v = *reinterpret_cast<const float4 *>(part + z * stride + e0);
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
        }
    }
    *reinterpret_cast<float4 *>(&sh[w][4 * (t & 63)]) = s;
    __syncthreads();
    const long i = long(blockIdx.x) * kThreads + t;
    if (i >= P) return;
    const float gi = (sh[0][t] + sh[1][t]) + (sh[2][t] + sh[3][t]);
    if (!ADAM) {
        g[i] = gi;
        return;
    }
    const float mi = 0.9f * ad.m[i] + 0.1f * gi;
    const float vi = 0.999f * ad.v[i] + 0.001f * gi * gi;
    ad.m[i] = mi;
    ad.v[i] = vi;
    const float wi = ad.w[i] - ad.lr * (mi * ad.c1) / (sqrtf(vi * ad.c2) + 1e-8f);
    ad.w[i] = wi;
    put_bf16(wi, i, ad.wb, ad.pw);
}

// Features of sample i: [sin(2 pi B x_i), cos(2 pi B x_i), p_i, 0 ...] as bfloat16 (row of K0).
__global__ void features_kernel(long n, const float *__restrict__ x, const float *__restrict__ p,
                                const float *__restrict__ Bf, int nf, int np, int K0, uint16_t *__restrict__ out) {
    const long idx = long(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= n * K0) return;
    const long i = idx / K0;
    const int j = int(idx % K0);
    float v = 0.f;
    if (j < 2 * nf) {
        const int f = j < nf ? j : j - nf;
        v = fourier_feature(feature_turns(Bf + 3 * f, x[3 * i], x[3 * i + 1], x[3 * i + 2]), j < nf);
    } else if (j < 2 * nf + np) {
        v = p[i * np + (j - 2 * nf)];
    }
    out[idx] = bf16_bits(v);
}

// Element i of dY = 2 (Y - T) / (n n_out) (bfloat16, n rows of nop >= n_out padded with
// zeros), and (Y - T)^2 summed over the wavefront's 64 elements, in its first lane.
__device__ __forceinline__ uint16_t loss_gradient(long i, long n, int nout, int nop, const float *__restrict__ Y,
                                                  const float *__restrict__ T, float &e2) {
    uint16_t h = 0;
    e2 = 0.f;
    if (i < n * nop) {
        const long r = i / nop;
        const int o = int(i - r * nop);
        if (o < nout) {
            const float d = Y[r * nout + o] - T[r * nout + o];
            e2 = d * d;
            h = bf16_bits(2.0f * d / float(n * nout));
        }
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) e2 += __shfl_down(e2, s);
    return h;
}

__global__ void loss_grad_kernel(long n, int nout, int nop, const float *__restrict__ Y, const float *__restrict__ T,
                                 uint16_t *__restrict__ dY, float *__restrict__ part) {
    const long i = long(blockIdx.x) * blockDim.x + threadIdx.x;
    float e2;
    const uint16_t h = loss_gradient(i, n, nout, nop, Y, T, e2);
    if (i >= n * nop) return;
    dY[i] = h;
    if (i % 64 == 0) part[i / 64] = e2;
}

__global__ void to_bf16_kernel(long n, const float *__restrict__ x, uint16_t *__restrict__ wb,
                               PackedWeights pw) {
    const long i = long(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) put_bf16(x[i], i, wb, pw);
}

// Whole-network inference, 64 samples per workgroup of four wavefronts; the
// activations never leave LDS.  Features are formed in LDS as in
// features_kernel.  Each hidden layer computes its output transposed,
// Z^T = W A^T + b, with W (bfloat16, row-major out x in) streamed from global
// memory straight into the MFMA A operand (8 consecutive k of one unit per lane)
// and A (64 x K) read from LDS as the B operand; wavefront w owns units
// [w W/4, (w+1) W/4), and each lane ends with 4 consecutive units of one sample,
// written back as one 8-byte store of bf16(SiLU(z)).  All waves finish reading A
// before any writes over it.  The output layer gives wavefront w samples
// [16w, 16w + 16).  Every output is the same k-ordered sum of the same products
// as in gemm_kernel, with the same epilogue arithmetic, so the result equals the
// layer-by-layer forward pass bit for bit (tested).  Registers are capped for
// three waves per SIMD (152 VGPRs for width 256, no spills): at millions of
// samples the extra wave hides more of the weight-load latency.
constexpr int kFusedRows = 64;
constexpr int kFusedMaxDepth = 8;
struct NetOffsets {
    long w[kFusedMaxDepth + 1];
    long b[kFusedMaxDepth + 1];
    long p[kFusedMaxDepth];            // hidden layers in the packed copy
};
// The training forward keeps what the backward pass reads: the features (bf16,
// n x K0) and every hidden layer's FP32 pre-activation and bf16 activation
// (n x W, row-major), the same arrays the layer-by-layer GEMMs write.
struct TrainStore {
    uint16_t *x0;
    float *z[kFusedMaxDepth];
    uint16_t *a[kFusedMaxDepth];
};

// Z^T (16 NT units x 64 samples per wavefront) = W A^T with A (64 x K, LDS), K
// in steps of 32: the weights are the MFMA A operand and the activations the B
// operand, so each lane ends with 4 consecutive units of one sample.  The
// weight fragments of step k + 32 are requested before the MFMAs of step k.
template <int NT>
__device__ __forceinline__ void fused_k_step(f32x4 (&acc)[4][NT], const uint16_t *act, int P, const uint16_t *wrow,
                                             int K, int ldw, int k0, bf16x8 (&bn)[NT], int l) {
    bf16x8 b[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) b[j] = bn[j];
    if (k0 + 32 < K) {
#pragma unroll
        for (int j = 0; j < NT; ++j) bn[j] = *reinterpret_cast<const bf16x8 *>(wrow + long(16 * j) * ldw + k0 + 32);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&act[(16 * i + (l & 15)) * P + k0 + 8 * (l >> 4)]);
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a, acc[i][j], 0, 0, 0);
    }
}

// Z^T (16 NT units x 64 samples per wavefront) = W A^T with A (64 x K, LDS), K
// in steps of 32: the weights are the MFMA A operand and the activations the B
// operand, so each lane ends with 4 consecutive units of one sample.  The
// weight fragments of step k + 32 are requested before the MFMAs of step k.
// KFIX > 0: K = KFIX known at compile time (the loop unrolls fully).
template <int NT, int KFIX>
__device__ __forceinline__ void fused_layer_k(f32x4 (&acc)[4][NT], const uint16_t *act, int P, const uint16_t *Wl,
                                              int K, int nb, int l) {
    const int ldw = KFIX > 0 ? KFIX : K;
    const uint16_t *wrow = Wl + long(nb + (l & 15)) * ldw + 8 * (l >> 4);
    bf16x8 bn[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) bn[j] = *reinterpret_cast<const bf16x8 *>(wrow + long(16 * j) * ldw);
    if constexpr (KFIX > 0) {
#pragma unroll
        for (int k0 = 0; k0 < KFIX; k0 += 32) fused_k_step<NT>(acc, act, P, wrow, KFIX, KFIX, k0, bn, l);
    } else {
        for (int k0 = 0; k0 < K; k0 += 32) fused_k_step<NT>(acc, act, P, wrow, K, K, k0, bn, l);
    }
}

// TRAIN: also stores the features, pre-activations and activations (TrainStore)
// for the backward pass.
template <int W, bool TRAIN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void fused_forward_kernel(long n, const float *__restrict__ x,
                                                                 const float *__restrict__ p,
                                                                 const float *__restrict__ Bf, int nf, int np,
                                                                 int K0, int depth, int nout,
                                                                 const uint16_t *__restrict__ wb,
                                                                 const float *__restrict__ wf, NetOffsets off,
                                                                 float *__restrict__ out, TrainStore ts) {
    extern __shared__ __attribute__((aligned(16))) uint16_t act[];
    const int P = (K0 > W ? K0 : W) + 8;          // LDS row pitch (elements)
    const long r0 = long(blockIdx.x) * kFusedRows;
    constexpr int NW = 4;
    const int t = threadIdx.x, w = t >> 6, l = t & 63;
    for (int idx = t; idx < kFusedRows * K0; idx += 64 * NW) {
        const int row = idx / K0, j = idx % K0;
        const long i = r0 + row;
        float v = 0.f;
        if (i < n) {
            if (j < 2 * nf) {
                const int f = j < nf ? j : j - nf;
                v = fourier_feature(feature_turns(Bf + 3 * f, x[3 * i], x[3 * i + 1], x[3 * i + 2]), j < nf);
            } else if (j < 2 * nf + np) {
                v = p[i * np + (j - 2 * nf)];
            }
        }
        const uint16_t bits = bf16_bits(v);
        act[row * P + j] = bits;
        if (TRAIN && i < n) ts.x0[i * K0 + j] = bits;
    }
    __syncthreads();
    constexpr int NT = W / (16 * NW);              // 16-column tiles per wavefront
    static_assert(NT >= 1, "at least one 16-unit tile per wavefront");
    const int nb = w * (W / NW);
    for (int layer = 0; layer < depth; ++layer) {
        const uint16_t *Wl = wb + off.w[layer];
        f32x4 acc[4][NT];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (layer == 0) {
            fused_layer_k<NT, 0>(acc, act, P, Wl, K0, nb, l);
        } else {
            fused_layer_k<NT, W>(acc, act, P, Wl, W, nb, l);
        }
        __syncthreads();
        const float *bias = wf + off.b[layer];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int u0 = nb + 16 * j + 4 * (l >> 4);              // 4 consecutive units
            const float4 bc = *reinterpret_cast<const float4 *>(bias + u0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 16 * i + (l & 15);                  // sample
                const float z0 = acc[i][j][0] + bc.x, z1 = acc[i][j][1] + bc.y;
                const float z2 = acc[i][j][2] + bc.z, z3 = acc[i][j][3] + bc.w;
                uint2 q;
                q.x = uint32_t(bf16_bits(z0 * sigmoidf_hw(z0))) | (uint32_t(bf16_bits(z1 * sigmoidf_hw(z1))) << 16);
                q.y = uint32_t(bf16_bits(z2 * sigmoidf_hw(z2))) | (uint32_t(bf16_bits(z3 * sigmoidf_hw(z3))) << 16);
                *reinterpret_cast<uint2 *>(&act[row * P + u0]) = q;
                if (TRAIN && r0 + row < n) {
                    const size_t o = size_t(r0 + row) * W + u0;
                    *reinterpret_cast<float4 *>(ts.z[layer] + o) = make_float4(z0, z1, z2, z3);
                    *reinterpret_cast<uint2 *>(ts.a[layer] + o) = q;
                }
            }
        }
        __syncthreads();
    }
    // output layer: rows [16w, 16w + 16), up to four 16-column tiles
    const uint16_t *Wo = wb + off.w[depth];
    const float *bo = wf + off.b[depth];
    f32x4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int ntile = (nout + 15) / 16;
    for (int k0 = 0; k0 < W; k0 += 32) {
        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&act[(16 * w + (l & 15)) * P + k0 + 8 * (l >> 4)]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j >= ntile) break;
            const int col = 16 * j + (l & 15);
            bf16x8 b;
            if (col < nout) {
                b = *reinterpret_cast<const bf16x8 *>(Wo + long(col) * W + k0 + 8 * (l >> 4));
            } else {
#pragma unroll
                for (int q = 0; q < 8; ++q) b[q] = __bf16(0.0f);
            }
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (j >= ntile) break;
        const int col = 16 * j + (l & 15);
        if (col >= nout) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const long row = r0 + 16 * w + 4 * (l >> 4) + r;
            if (row < n) out[row * nout + col] = acc[j][r] + bo[col];
        }
    }
}

// ---------------------------------------------------------------- tiled fused forward
//
// Whole-network inference with the weights of a layer in registers.  fused_forward_kernel
// streams every weight for each 64 samples (11 GB through the L2s for a million samples,
// 1.4 ms, 18 % of the matrix cores' time); here a workgroup holds ROWS samples in LDS and
// wavefront w keeps the weights of its units [w W/NW, (w+1) W/NW) for the whole layer,
// the next layer's arriving meanwhile, and walks the ROWS / 16 sample tiles.  Activations
// alternate between two LDS buffers, so the wavefronts meet once per layer and in between
// drift apart as they like: one's SiLU (half of the work) runs under another's products.
// A tile's SiLU is done after the next tile's LDS reads have gone out.  The weights come
// from a copy in the order of the matrix cores' fragments, 1 KB in a row per load: read
// from the row-major matrix, every load touches 16 rows 512 bytes apart, and each layer
// begins with a wait for its weights.  Measured, 5 layers of 256, 75 features: 1 M
// samples 1.43 ms -> 0.78 to 0.82 ms (from the row-major weights 1.08; with one buffer, a
// barrier per tile and two workgroups per CU 0.98), 1331 samples 33 -> 13 us.  What bounds
// it: counted over the kernel, matrix cores are busy 33 % of the time, vector instructions
// issue in 54 % and LDS works in 43 %, half of it bank conflicts, so the three overlap
// little; the features, the output layer and the first tile of each layer have no products
// to run under.
// Products, their order and the epilogue arithmetic are those of the layer-by-layer
// GEMMs, so the outputs have the same bits.
constexpr int kTiledK = 8;            // 32-deep k steps of a layer held in registers: inputs up to 256
// Features of the workgroup's ROWS samples in LDS as in features_kernel.  Frequencies in
// eights: a lane computes the phases of its sample once for sine and cosine and stores
// 16 bytes of each (an element at a time, with the divisions that takes and every phase
// twice, this was half of fused_forward_kernel's vector instructions).
template <int NW, int ROWS>
__device__ __forceinline__ void tiled_features(uint16_t *act, int P, long n, long r0, const float *__restrict__ x,
                                               const float *__restrict__ p, const float *__restrict__ Bf, int nf, int np,
                                               int K0, int w, int l) {
    if (nf % 8 == 0) {
        constexpr int RL = ROWS < 64 ? ROWS : 64, RG = ROWS / RL, SUB = 64 / RL;   // rows per wavefront, row groups, sub-units
        static_assert(NW % RG == 0, "a wavefront keeps its row group");
        // the parameters of the workgroup's rows lie in a row: a few independent loads per thread
        const int total = ROWS * np, tid = 64 * w + l;
        constexpr int PB = 4;
        for (int i0 = tid; i0 < total; i0 += PB * 64 * NW) {
            float v[PB];
#pragma unroll
            for (int c = 0; c < PB; ++c) {
                const int i = i0 + c * 64 * NW;
                v[c] = (i < total && r0 * np + i < n * np) ? p[r0 * np + i] : 0.f;
            }
#pragma unroll
            for (int c = 0; c < PB; ++c) {
                const int i = i0 + c * 64 * NW;
                if (i < total) act[(i / np) * P + 2 * nf + i % np] = bf16_bits(v[c]);
            }
        }
        for (int row = tid; row < ROWS; row += 64 * NW)
            for (int j = 2 * nf + np; j < K0; ++j) act[row * P + j] = 0;
        const int row = (w % RG) * RL + l % RL, sub = l / RL;
        const long i = r0 + row;
        const float x0 = i < n ? x[3 * i] : 0.f, x1 = i < n ? x[3 * i + 1] : 0.f, x2 = i < n ? x[3 * i + 2] : 0.f;
        for (int f0 = 8 * ((w / RG) * SUB + sub); f0 < nf; f0 += 8 * (NW / RG) * SUB) {
            uint16_t sn[8], cs[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float turns = feature_turns(Bf + 3 * (f0 + q), x0, x1, x2);
                sn[q] = i < n ? bf16_bits(fourier_feature(turns, true)) : uint16_t(0);
                cs[q] = i < n ? bf16_bits(fourier_feature(turns, false)) : uint16_t(0);
            }
            *reinterpret_cast<uint4 *>(&act[row * P + f0]) = pack8(sn);
            *reinterpret_cast<uint4 *>(&act[row * P + nf + f0]) = pack8(cs);
        }
    } else {
        for (int idx = 64 * w + l; idx < ROWS * K0; idx += 64 * NW) {
            const int row = idx / K0, j = idx % K0;
            const long i = r0 + row;
            float v = 0.f;
            if (i < n) {
                if (j < 2 * nf) {
                    const int f = j < nf ? j : j - nf;
                    v = fourier_feature(feature_turns(Bf + 3 * f, x[3 * i], x[3 * i + 1], x[3 * i + 2]), j < nf);
                } else if (j < 2 * nf + np) {
                    v = p[i * np + (j - 2 * nf)];
                }
            }
            act[row * P + j] = bf16_bits(v);
        }
    }
}

template <int W, bool TRAIN, int ROWS, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void tiled_forward_kernel(
    long n, const float *__restrict__ x, const float *__restrict__ p, const float *__restrict__ Bf, int nf, int np, int K0,
    int depth, int nout, const uint16_t *__restrict__ wb, const uint16_t *__restrict__ wp, const float *__restrict__ wf,
    NetOffsets off, float *__restrict__ out, TrainStore ts) {
    constexpr int NT = W / (16 * NW), T = ROWS / 16, KW = W / 32;
    static_assert(NT >= 1 && KW <= kTiledK && T >= 2, "tiles");
    extern __shared__ __attribute__((aligned(16))) uint16_t act[];
    const int P = (K0 > W ? K0 : W) + 8;          // LDS row pitch (elements)
    uint16_t *cur = act, *nxt = act + ROWS * P;   // a layer's inputs and outputs
    const long r0 = long(blockIdx.x) * ROWS;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63;
    const int nb = w * (W / NW), lr = l & 15, lk = 8 * (l >> 4);
    const int nk0 = K0 / 32;
    // this lane's part of the fragments of units nb + 16 j, k step ks: units + lr, k + lk + 0..7
    auto load_weights = [&](bf16x8 (&wt)[NT][kTiledK], int layer) {
        const int K = layer == 0 ? nk0 : KW;
        const bf16x8 *frag0 = reinterpret_cast<const bf16x8 *>(wp + off.p[layer]) + long(nb / 16) * K * 64 + l;
#pragma unroll
        for (int ks = 0; ks < kTiledK; ++ks)
            if (layer == 0 ? ks < nk0 : ks < KW) {
#pragma unroll
                for (int j = 0; j < NT; ++j) wt[j][ks] = frag0[(j * K + ks) * 64];
            }
    };
    // the output layer's weights of column col (zero past n_out); those of the first sixteen
    // columns are fetched while the last hidden layer runs
    auto output_weights = [&](int col, int ks) {
        bf16x8 v = *reinterpret_cast<const bf16x8 *>(wb + off.w[depth] + long(min(col, nout - 1)) * W + 32 * ks + lk);
        if (col >= nout)
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = __bf16(0.0f);
        return v;
    };
    bf16x8 wa[NT][kTiledK], wc[NT][kTiledK], wo[KW];
    load_weights(wa, 0);
    tiled_features<NW, ROWS>(act, P, n, r0, x, p, Bf, nf, np, K0, w, l);
    __syncthreads();
    if (TRAIN)
        for (int row = w; row < ROWS; row += NW)
            if (r0 + row < n)
                for (int c = 8 * l; c < K0; c += 512)
                    *reinterpret_cast<uint4 *>(ts.x0 + (r0 + row) * K0 + c) = *reinterpret_cast<const uint4 *>(&act[row * P + c]);
    f32x4 pacc[NT];                               // products of the last tile, to be finished
    auto silu = [&](const float4 (&bias)[NT], uint2 (&q)[NT], f32x4 (&z)[NT]) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            z[j][0] = pacc[j][0] + bias[j].x; z[j][1] = pacc[j][1] + bias[j].y;
            z[j][2] = pacc[j][2] + bias[j].z; z[j][3] = pacc[j][3] + bias[j].w;
            q[j].x = bf16_pair(z[j][0] * sigmoidf_hw(z[j][0]), z[j][1] * sigmoidf_hw(z[j][1]));
            q[j].y = bf16_pair(z[j][2] * sigmoidf_hw(z[j][2]), z[j][3] * sigmoidf_hw(z[j][3]));
        }
    };
    auto finish = [&](int tile, int layer, const uint2 (&q)[NT], const f32x4 (&z)[NT]) {
        const int row = 16 * tile + lr;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int u0 = nb + 16 * j + 4 * (l >> 4);              // 4 consecutive units of one sample
            *reinterpret_cast<uint2 *>(&nxt[row * P + u0]) = q[j];
            if (TRAIN && r0 + row < n) {
                const size_t o = size_t(r0 + row) * W + u0;
                *reinterpret_cast<float4 *>(ts.z[layer] + o) = make_float4(z[j][0], z[j][1], z[j][2], z[j][3]);
                *reinterpret_cast<uint2 *>(ts.a[layer] + o) = q[j];
            }
        }
    };
    // NK: k steps of the layer's inputs
    auto run_layer = [&](bf16x8 (&wt)[NT][kTiledK], bf16x8 (&wnext)[NT][kTiledK], int layer, auto nk) {
        constexpr int NK = decltype(nk)::value;
        float4 bias[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j)
            bias[j] = *reinterpret_cast<const float4 *>(wf + off.b[layer] + nb + 16 * j + 4 * (l >> 4));
        if (layer + 1 < depth) load_weights(wnext, layer + 1);
        else
#pragma unroll
            for (int ks = 0; ks < KW; ++ks) wo[ks] = output_weights(lr, ks);
        auto step = [&](int tile, auto some) {    // products of a tile, SiLU of the one before
            constexpr bool SOME = decltype(some)::value;
            const uint16_t *arow = &cur[(16 * tile + lr) * P + lk];
            bf16x8 a[NK];
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) a[ks] = *reinterpret_cast<const bf16x8 *>(arow + 32 * ks);
            uint2 q[NT];
            f32x4 z[NT], acc[NT];
            if constexpr (SOME) silu(bias, q, z);
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < NK; ++ks)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[j][ks], a[ks], acc[j], 0, 0, 0);
            if constexpr (SOME) finish(tile - 1, layer, q, z);
#pragma unroll
            for (int j = 0; j < NT; ++j) pacc[j] = acc[j];
        };
        step(0, std::false_type{});
#pragma unroll 1
        for (int tile = 1; tile < T; ++tile) step(tile, std::true_type{});
        uint2 q[NT];
        f32x4 z[NT];
        silu(bias, q, z);
        finish(T - 1, layer, q, z);
        __syncthreads();
        uint16_t *swap = cur;
        cur = nxt;
        nxt = swap;
    };
    switch (nk0) {
        case 1: run_layer(wa, wc, 0, std::integral_constant<int, 1>{}); break;
        case 2: run_layer(wa, wc, 0, std::integral_constant<int, 2>{}); break;
        case 3: run_layer(wa, wc, 0, std::integral_constant<int, 3>{}); break;
        case 4: run_layer(wa, wc, 0, std::integral_constant<int, 4>{}); break;
        case 5: run_layer(wa, wc, 0, std::integral_constant<int, 5>{}); break;
        case 6: run_layer(wa, wc, 0, std::integral_constant<int, 6>{}); break;
        case 7: run_layer(wa, wc, 0, std::integral_constant<int, 7>{}); break;
        default: run_layer(wa, wc, 0, std::integral_constant<int, 8>{}); break;
    }
    for (int layer = 1; layer < depth; layer += 2) {
        run_layer(wc, wa, layer, std::integral_constant<int, KW>{});
        if (layer + 1 < depth) run_layer(wa, wc, layer + 1, std::integral_constant<int, KW>{});
    }
    // output layer: wavefront w takes sample tiles w, w + NW, ...
    const float *bo = wf + off.b[depth];
    const int ntile = (nout + 15) / 16;
    for (int tile = w; tile < T; tile += NW) {
        bf16x8 a[KW];
#pragma unroll
        for (int ks = 0; ks < KW; ++ks)
            a[ks] = *reinterpret_cast<const bf16x8 *>(&cur[(16 * tile + lr) * P + 32 * ks + lk]);
        for (int j = 0; j < ntile; ++j) {
            f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
            const int col = 16 * j + lr;
            if (j > 0 || (ntile > 1 && tile > w))
#pragma unroll
                for (int ks = 0; ks < KW; ++ks) wo[ks] = output_weights(col, ks);
#pragma unroll
            for (int ks = 0; ks < KW; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks], wo[ks], acc, 0, 0, 0);
            if (col >= nout) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const long row = r0 + 16 * tile + 4 * (l >> 4) + r;
                if (row < n) out[row * nout + col] = acc[r] + bo[col];
            }
        }
    }
}

// ---------------------------------------------------------------- tiled backward
//
// dY and the loss partials, then every hidden layer's dZ = (dZ of the next layer times its
// weights) through the SiLU at z, in one launch for a workgroup's ROWS samples: the split,
// the buffers and the weights' way are tiled_forward_kernel's, with the transposed weights.
// dZ stays in LDS from layer to layer and is written once for the weight gradients.  The
// arithmetic is that of the GEMMs with the EPI_SILU_BACK epilogue, bit for bit.  Bound by
// the memory side (z read and dZ written, 126 MB for five layers of 256 and 16384 samples)
// and the latency of products and SiLUs: 32 us there and 18 us for 2500 samples, where a
// kernel for dY, a GEMM per layer and one for the output took 55 and 38.
struct BackStore {
    const float *z[kFusedMaxDepth];
    uint16_t *dz[kFusedMaxDepth];
};

template <int W, int ROWS, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void tiled_backward_kernel(
    long n, const float *__restrict__ y, const float *__restrict__ target, int nout, int nop, int nko, int depth,
    const uint16_t *__restrict__ wt, uint16_t *__restrict__ dY, float *__restrict__ lpart, BackStore bs) {
    constexpr int NT = W / (16 * NW), T = ROWS / 16, KW = W / 32, P = W + 8;
    extern __shared__ __attribute__((aligned(16))) uint16_t act[];
    uint16_t *cur = act, *nxt = act + ROWS * P;
    const long r0 = long(blockIdx.x) * ROWS;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63;
    const int nb = w * (W / NW), lr = l & 15, lk = 8 * (l >> 4);
    // the fragments of the layer after hidden layer `layer` (the output layer's have nko k steps)
    auto load_weights = [&](bf16x8 (&q)[NT][KW], int layer) {
        const int K = layer == depth - 1 ? nko : KW;
        const bf16x8 *frag0 = reinterpret_cast<const bf16x8 *>(wt + long(layer) * W * W) + long(nb / 16) * K * 64 + l;
#pragma unroll
        for (int ks = 0; ks < KW; ++ks)
            if (ks < K) {
#pragma unroll
                for (int j = 0; j < NT; ++j) q[j][ks] = frag0[(j * K + ks) * 64];
            }
    };
    bf16x8 wa[NT][KW], wc[NT][KW];
    load_weights(wa, depth - 1);
    for (int e = t; e < ROWS * nop; e += 64 * NW) {      // ROWS nop is a multiple of 64
        const long i = r0 * nop + e;
        float e2;
        const uint16_t h = loss_gradient(i, n, nout, nop, y, target, e2);
        cur[e / nop * P + e % nop] = h;
        if (i < n * nop) {
            dY[i] = h;
            if (l == 0) lpart[i / 64] = e2;
        }
    }
    const int pad = 32 * nko - nop;                      // 0 or 16 columns
    for (int e = t; e < ROWS * pad; e += 64 * NW) cur[e / 16 * P + nop + e % 16] = 0;
    __syncthreads();
    f32x4 pacc[NT];                                      // products of the last tile, to be finished
    float4 zp[NT];                                       // and its pre-activations
    auto silu_back = [](float v, float z) {
        const float sg = sigmoidf_hw(z);
        return v * sg * (1.0f + z * (1.0f - sg));
    };
    auto finish = [&](int tile, int layer) {
        const int row = 16 * tile + lr;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            uint2 q;
            q.x = bf16_pair(silu_back(pacc[j][0], zp[j].x), silu_back(pacc[j][1], zp[j].y));
            q.y = bf16_pair(silu_back(pacc[j][2], zp[j].z), silu_back(pacc[j][3], zp[j].w));
            const int u0 = nb + 16 * j + 4 * (l >> 4);
            *reinterpret_cast<uint2 *>(&nxt[row * P + u0]) = q;
            if (r0 + row < n) *reinterpret_cast<uint2 *>(bs.dz[layer] + size_t(r0 + row) * W + u0) = q;
        }
    };
    // NK: k steps of the next layer's units
    auto run_layer = [&](bf16x8 (&wt_)[NT][KW], bf16x8 (&wnext)[NT][KW], int layer, auto nk) {
        constexpr int NK = decltype(nk)::value;
        if (layer > 0) load_weights(wnext, layer - 1);
        auto step = [&](int tile, auto some) {
            constexpr bool SOME = decltype(some)::value;
            const uint16_t *arow = &cur[(16 * tile + lr) * P + lk];
            bf16x8 a[NK];
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) a[ks] = *reinterpret_cast<const bf16x8 *>(arow + 32 * ks);
            float4 z[NT];
            const long row = r0 + 16 * tile + lr;
#pragma unroll
            for (int j = 0; j < NT; ++j)
                z[j] = row < n ? *reinterpret_cast<const float4 *>(bs.z[layer] + size_t(row) * W + nb + 16 * j + 4 * (l >> 4))
                               : make_float4(0.f, 0.f, 0.f, 0.f);
            f32x4 acc[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < NK; ++ks)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt_[j][ks], a[ks], acc[j], 0, 0, 0);
            if constexpr (SOME) finish(tile - 1, layer);
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                pacc[j] = acc[j];
                zp[j] = z[j];
            }
        };
        step(0, std::false_type{});
#pragma unroll 1
        for (int tile = 1; tile < T; ++tile) step(tile, std::true_type{});
        finish(T - 1, layer);
        __syncthreads();
        uint16_t *swap = cur;
        cur = nxt;
        nxt = swap;
    };
    if (nko == 1) run_layer(wa, wc, depth - 1, std::integral_constant<int, 1>{});
    else run_layer(wa, wc, depth - 1, std::integral_constant<int, 2>{});
    for (int layer = depth - 2; layer >= 0; layer -= 2) {
        run_layer(wc, wa, layer, std::integral_constant<int, KW>{});
        if (layer > 0) run_layer(wa, wc, layer - 1, std::integral_constant<int, KW>{});
    }
}

// Ensemble statistics over K members' outputs (K x n x n_out, member-major):
// mean[i][o] = scale[o] (sum_k out[k][i][o]) / K and
// spread[i] = scale[0] (max_k out[k][i][0] - min_k out[k][i][0]); members summed in order.
__global__ void ensemble_stats_kernel(long n, int K, int nout, const float *__restrict__ outs,
                                      const float *__restrict__ scale, float *__restrict__ mean,
                                      float *__restrict__ spread) {
    const long i = long(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float invK = 1.0f / float(K);
    for (int o = 0; o < nout; ++o) {
        float s = 0.f, lo = INFINITY, hi = -INFINITY;
        for (int k = 0; k < K; ++k) {
            const float v = outs[(size_t(k) * n + i) * nout + o];
            s += v;
            lo = fminf(lo, v);
            hi = fmaxf(hi, v);
        }
        mean[i * nout + o] = scale[o] * s * invK;
        if (o == 0) spread[i] = scale[0] * (hi - lo);
    }
}

// Scenario of row r: the s with row_begin[s] <= r < row_begin[s + 1] (binary
// search over the n_scen + 1 offsets; rows of empty scenarios never occur).
__device__ inline int scenario_of(const int64_t *__restrict__ row_begin, int n_scen, int64_t r) {
    int lo = 0, hi = n_scen - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (row_begin[mid] <= r) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Network inputs of many scenarios in one pass over their nodes: coordinates
// relative to the scenario's probe in units of its coordinate scale, and the
// parameter row (coordinates times p_scale, then the scenario's constants).
// The coordinate arithmetic is FP64, rounded once to FP32.
__global__ void scenario_inputs_kernel(int n_scen, int n_prm, const int64_t *__restrict__ row_begin,
                                       const double *__restrict__ X, const double *__restrict__ probe,
                                       const double *__restrict__ xi, double p_scale, const float *__restrict__ prm,
                                       float *__restrict__ x_out, float *__restrict__ p_out) {
#pragma clang fp contract(off)
    const int64_t r = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (r >= row_begin[n_scen]) return;
    const int sc = scenario_of(row_begin, n_scen, r);
    const int w = 3 + n_prm;
    for (int i = 0; i < 3; ++i) {
        const double x = X[3 * r + i];
        const double rel = x - probe[3 * sc + i];
        x_out[3 * r + i] = float(rel * xi[sc]);
        p_out[w * r + i] = float(x * p_scale);
    }
    for (int k = 0; k < n_prm; ++k) p_out[w * r + 3 + k] = prm[size_t(n_prm) * sc + k];
}

// Ensemble mean and spread (scaled targets) to physical fields of each row's
// scenario, in FP32 with one rounding per operation (no fused multiply-add):
// T = T0 + sT * m0, u = su * m1..3, spread_K = sT * spread.
__global__ void scenario_outputs_kernel(int n_scen, const int64_t *__restrict__ row_begin,
                                        const float *__restrict__ mean, const float *__restrict__ spread,
                                        const float *__restrict__ T0, const float *__restrict__ sT,
                                        const float *__restrict__ su, float *__restrict__ T_out,
                                        float *__restrict__ u_out, float *__restrict__ spread_out) {
    // plain operators under contract(off): hipcc would otherwise form an FMA
    // (its rounding intrinsics are header functions the pragma does not reach)
#pragma clang fp contract(off)
    const int64_t r = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (r >= row_begin[n_scen]) return;
    const int sc = scenario_of(row_begin, n_scen, r);
    const float rise = sT[sc] * mean[4 * r];
    T_out[r] = T0[sc] + rise;
    for (int i = 0; i < 3; ++i) u_out[3 * r + i] = su[sc] * mean[4 * r + 1 + i];
    spread_out[r] = sT[sc] * spread[r];
}

inline unsigned blocks(long n) { return unsigned((n + kThreads - 1) / kThreads); }

struct Layer {
    int in, out;      // in: padded input width
    long w_off, b_off;
};

}  // namespace

// Split-K partials of tled_mlp_gemm_static: a static device array (each GPU the
// library runs on holds its own copy for the life of the process).  Host code
// never passes `scratch` itself (on the host it names a stand-in, not a device
// address): its per-device address comes from hipGetSymbolAddress, taken once
// per device with that device current, when a handle is created there.  With
// the split rule of gemm() (nz x output tiles <= 512, 64 x 64 tiles) the
// partials never exceed 512 x 4096 floats, which is this array's size.
constexpr size_t kStaticSplitFloats = size_t(512) * 64 * 64;
static __device__ __align__(256) float scratch[kStaticSplitFloats];

namespace {
std::mutex g_scratch_mu;
std::vector<float *> g_scratch_addr;   // device ordinal -> address of `scratch` on that device

// Call with `device` current.
tled_status resolve_scratch(int device) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (size_t(device) >= g_scratch_addr.size()) g_scratch_addr.resize(size_t(device) + 1, nullptr);
    if (g_scratch_addr[device]) return TLED_OK;
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return TLED_E_HIP;
    g_scratch_addr[device] = static_cast<float *>(p);
    return TLED_OK;
}
}  // namespace

struct tled_mlp {
    int device = 0;
    int cus = 256;                     // compute units of the device
    float *d_static_split = nullptr;   // this device's `scratch` (resolved at creation)
    hipStream_t stream = nullptr;
    bool own_stream = false;
    tled_mlp_config cfg{};
    int K0 = 0;
    std::vector<Layer> layers;
    long P = 0;
    std::vector<float> freq;
    float *d_w = nullptr, *d_g = nullptr, *d_m = nullptr, *d_v = nullptr, *d_freq = nullptr;
    uint16_t *d_wb = nullptr;
    uint16_t *d_wp = nullptr, *d_wt = nullptr;   // weights packed for the tiled kernels (behind d_wb;
                                                 // null where those do not apply)
    long adam_t = 0;
    // workspace for up to cap samples
    long cap = 0;
    uint16_t *d_x0 = nullptr;
    std::vector<float *> d_z;        // per hidden layer, cap x width
    std::vector<uint16_t *> d_a;     // per hidden layer, cap x width
    float *d_y = nullptr, *d_part = nullptr, *d_loss = nullptr, *d_gpart = nullptr;
    int nop = 0;                     // columns of d_dy: n_out padded to a multiple of 16
    uint16_t *d_dy = nullptr;
    std::vector<uint16_t *> d_dz;    // per hidden layer, cap x width
    long grad_kchunk = 0, grad_tiles = 0, grad_stride = 0;   // of all layers' weight gradients; floats of a partial vector
    std::vector<void *> ws;
    std::string err;
    float *d_split = nullptr;        // split-K partials
    size_t split_cap = 0;
    // calls on their caller's stream (tled_mlp_begin): the thread between begin and end, the
    // handle's own stream meanwhile, and what the last of them left behind
    std::mutex in_call;
    std::atomic<std::thread::id> caller{};
    hipStream_t kept_stream = nullptr;
    hipEvent_t done = nullptr;
    bool done_valid = false;
    // timing
    bool timing = false;
    double gemm_ms = 0.0, fused_ms = 0.0, gemm_flops = 0.0, fused_flops = 0.0;
};

namespace {

tled_status mfail(tled_mlp *s, tled_status st, const std::string &m) {
    if (s) s->err = m;
    return st;
}

#define MCHK(s, expr)                                                                                  \
    do {                                                                                               \
        hipError_t e_ = (expr);                                                                        \
        if (e_ != hipSuccess) return mfail(s, TLED_E_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

#define MTRY(expr)                        \
    do {                                  \
        tled_status st_ = (expr);         \
        if (st_ != TLED_OK) return st_;   \
    } while (0)

uint64_t splitmix(uint64_t &s) {
    uint64_t z = (s += 0x9e3779b97f4a7c15ULL);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
    return z ^ (z >> 31);
}
double uniform01(uint64_t &s) { return double(splitmix(s) >> 11) * (1.0 / 9007199254740992.0); }

void free_ws(tled_mlp *s) {
    for (void *p : s->ws) (void)hipFree(p);
    s->ws.clear();
    s->d_z.clear();
    s->d_a.clear();
    s->d_dz.clear();
    s->cap = 0;
}

template <typename T>
tled_status walloc(tled_mlp *s, T **p, size_t n) {
    void *q = nullptr;
    if (hipMalloc(&q, std::max<size_t>(n, 1) * sizeof(T)) != hipSuccess) return mfail(s, TLED_E_OOM, "hipMalloc failed");
    s->ws.push_back(q);
    *p = static_cast<T *>(q);
    return TLED_OK;
}

// Chunks of rows of the weight-gradient launch: about two workgroups per CU in all, in
// eights (one chunk's tiles share an XCD) where there are that many.  Five layers of 256,
// 16384 rows: one / two / three / four workgroups per CU 38.7 / 30.2 / 32.1 / 34.1 us, and
// the sums after them 5.5 / 7.0 / 9.8 / 11.1.
int grad_chunks(const tled_mlp *s) {
    const long c = std::min<long>(64, std::max<long>(1, 2L * s->cus / s->grad_tiles));
    return int(c >= kNumXcd ? c / kNumXcd * kNumXcd : c);
}

tled_status ensure_workspace(tled_mlp *s, long n) {
    if (n <= s->cap) return TLED_OK;
    MCHK(s, hipStreamSynchronize(s->stream));
    free_ws(s);
    const long W = s->cfg.width, no = s->cfg.n_out;
    const long cap = std::max<long>(n, 1024);
    MTRY(walloc(s, &s->d_x0, size_t(cap) * s->K0));
    for (int l = 0; l < s->cfg.depth; ++l) {
        float *z;
        uint16_t *a, *dz;
        MTRY(walloc(s, &z, size_t(cap) * W));
        MTRY(walloc(s, &a, size_t(cap) * W));
        MTRY(walloc(s, &dz, size_t(cap) * W));
        s->d_dz.push_back(dz);
        s->d_z.push_back(z);
        s->d_a.push_back(a);
    }
    MTRY(walloc(s, &s->d_y, size_t(cap) * no));
    MTRY(walloc(s, &s->d_dy, size_t(cap) * s->nop));
    MTRY(walloc(s, &s->d_part, size_t((cap * s->nop + 63) / 64)));
    MTRY(walloc(s, &s->d_loss, 1));
    MTRY(walloc(s, &s->d_gpart, size_t(grad_chunks(s)) * s->grad_stride));
    s->cap = cap;
    return TLED_OK;
}

// Vector loads need 16-byte aligned vectors: base aligned and the strided axis a multiple of 8.
int load_mode(const uint16_t *X, long sr, long sk) {
    if (reinterpret_cast<uintptr_t>(X) % 16 != 0) return LD_SCALAR;
    if (sk == 1 && sr % 8 == 0) return LD_KVEC;
    if (sr == 1 && sk % 8 == 0) return LD_RVEC;
    return LD_SCALAR;
}

// split_ext: split-K partials in a caller-held buffer of split_ext_cap floats
// (nothing is allocated and no timing events are created); else the handle's
// buffer, grown on demand.  Split-K (EPI_F32, fewer than 256 output tiles): about 512
// workgroups (nz x tiles), at most 64 k chunks.
template <int EPI>
tled_status gemm(tled_mlp *s, int M, int N, int K, const uint16_t *A, long lda, const uint16_t *B,
                 long sbk, long sbn, float *C, long scm, long scn, uint16_t *Act, const float *bias,
                 float *split_ext = nullptr, size_t split_ext_cap = 0) {
    const long tiles = long((M + BM - 1) / BM) * ((N + BN - 1) / BN);
    int nz = 1;
    if (EPI == EPI_F32 && tiles < 256 && K >= 4 * BK)
        nz = int(std::min<long>(64, std::max<long>(1, 512 / tiles)));
    int kchunk = ((K + nz - 1) / nz + BK - 1) / BK * BK;
    nz = (K + kchunk - 1) / kchunk;
    const int am = load_mode(A, lda, 1), bmode = load_mode(B, sbn, sbk);
    float *split = s->d_split;
    if (nz > 1 && split_ext) {
        const size_t need = size_t(nz) * M * N;
        if (need > split_ext_cap)
            return mfail(s, TLED_E_ARG, "split-K partials of " + std::to_string(need) + " floats exceed the " +
                                            std::to_string(split_ext_cap) + " of the static scratch array");
        split = split_ext;
    } else if (nz > 1) {
        const size_t need = size_t(nz) * M * N;
        if (need > s->split_cap) {
            MCHK(s, hipStreamSynchronize(s->stream));   // earlier launches may still use the old buffer
            if (s->d_split) (void)hipFree(s->d_split);
            s->d_split = nullptr;
            s->split_cap = 0;
            void *p = nullptr;
            if (hipMalloc(&p, need * sizeof(float)) != hipSuccess) return mfail(s, TLED_E_OOM, "hipMalloc failed");
            s->d_split = static_cast<float *>(p);
            s->split_cap = need;
        }
        split = s->d_split;
    }
    dim3 grid((N + BN - 1) / BN, (M + BM - 1) / BM, nz);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    const bool timed = s->timing && !split_ext;
    if (timed) {
        MCHK(s, hipEventCreate(&e0));
        MCHK(s, hipEventCreate(&e1));
        MCHK(s, hipEventRecord(e0, s->stream));
    }
    float *Cout = nz > 1 ? split : C;
#define TLED_GEMM_LAUNCH(AMODE, BMODE_)                                                                       \
    hipLaunchKernelGGL((gemm_kernel<EPI, AMODE, BMODE_>), grid, dim3(kThreads), 0, s->stream, M, N, K, A, lda, B, \
                       sbk, sbn, Cout, scm, scn, Act, bias, kchunk)
    if (am == LD_KVEC && bmode == LD_KVEC) TLED_GEMM_LAUNCH(LD_KVEC, LD_KVEC);
    else if (am == LD_KVEC && bmode == LD_RVEC) TLED_GEMM_LAUNCH(LD_KVEC, LD_RVEC);
    else TLED_GEMM_LAUNCH(LD_SCALAR, LD_SCALAR);
#undef TLED_GEMM_LAUNCH
    if (nz > 1)
        hipLaunchKernelGGL(splitk_reduce_kernel, dim3(unsigned((long(M) * N + 63) / 64)), dim3(kThreads), 0,
                           s->stream, nz, M, N, split, C, scm, scn);
    MCHK(s, hipGetLastError());
    if (timed) {
        MCHK(s, hipEventRecord(e1, s->stream));
        MCHK(s, hipEventSynchronize(e1));
        float ms = 0.f;
        MCHK(s, hipEventElapsedTime(&ms, e0, e1));
        s->gemm_ms += ms;
        s->gemm_flops += 2.0 * double(M) * N * K;
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    return TLED_OK;
}

// Fused inference applies to widths 64/128/256, depth <= 8, and LDS rows that fit.
size_t fused_lds_bytes(const tled_mlp *s) {
    return size_t(kFusedRows) * (std::max(s->K0, s->cfg.width) + 8) * sizeof(uint16_t);
}

bool fused_ok(const tled_mlp *s) {
    const int W = s->cfg.width;
    return !s->cfg.layerwise && (W == 64 || W == 128 || W == 256) && s->cfg.depth <= kFusedMaxDepth &&
           fused_lds_bytes(s) <= 64 * 1024;
}

// The tiled kernel applies where the fused one does and the inputs fit its registers.
bool tiled_ok(const tled_mlp *s) { return fused_ok(s) && s->K0 <= 32 * kTiledK; }

size_t tiled_lds_bytes(const tled_mlp *s, int rows) {
    return 2 * size_t(rows) * (std::max(s->K0, s->cfg.width) + 8) * sizeof(uint16_t);
}

PackedWeights packed_weights(const tled_mlp *s) {
    return PackedWeights{s->d_wp, s->d_wt, s->K0, s->cfg.width, s->cfg.depth, (s->cfg.n_out + 31) / 32, s->layers.back().b_off};
}

// Samples per workgroup of the tiled kernel, 0 where it does not apply.  At width 256 a
// workgroup's registers and LDS fill a CU, so a workgroup takes the fewest samples that
// need one round of workgroups (5 layers, 8192 / 16384 / 32768 samples: 32 rows 14.5 /
// 25.3 / 47.1 us, 64 rows 18.6 / 19.7 / 35.0, 128 rows 27.2 / 27.4 / 29.4).  Two or more
// workgroups of a narrower network share a CU and fill each other's waits: 128 rows never
// lead by more than 4 % (width 128, 3 layers, 16384 / 24576 / 65536: 32 rows 8.6 / 13.0 /
// 26.5 us, 64 rows 8.5 / 11.5 / 20.5, 128 rows 12.2 / 12.4 / 22.5).
int tiled_rows(const tled_mlp *s, long n) {
    if (!s->d_wp) return 0;
    if (s->cfg.width < 256) return n <= 64L * s->cus ? 32 : 64;
    if (n <= 32L * s->cus) return 32;
    if (n <= 64L * s->cus) return 64;
    return 128;
}

// ts: the training forward (stores for the backward pass); null for inference.
tled_status fused_forward(tled_mlp *s, long n, const float *coords, const float *params, float *out,
                          const TrainStore *ts = nullptr) {
    NetOffsets off{};
    for (int l = 0; l <= s->cfg.depth; ++l) {
        off.w[l] = s->layers[l].w_off;
        off.b[l] = s->layers[l].b_off;
        if (l < s->cfg.depth) off.p[l] = l ? long(s->cfg.width) * (s->K0 + (l - 1) * s->cfg.width) : 0;
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (s->timing) {
        MCHK(s, hipEventCreate(&e0));
        MCHK(s, hipEventCreate(&e1));
        MCHK(s, hipEventRecord(e0, s->stream));
    }
#define TLED_FUSED(WIDTH, TR)                                                                                \
    hipLaunchKernelGGL((fused_forward_kernel<WIDTH, TR>), dim3(unsigned((n + kFusedRows - 1) / kFusedRows)),   \
                       dim3(256), fused_lds_bytes(s), s->stream, n, coords, params, s->d_freq, s->cfg.n_freq,  \
                       s->cfg.n_param, s->K0, s->cfg.depth, s->cfg.n_out, s->d_wb, s->d_w, off, out,            \
                       ts ? *ts : TrainStore{})
#define TLED_TILED(WIDTH, TR, ROWS, NW)                                                                      \
    hipLaunchKernelGGL((tiled_forward_kernel<WIDTH, TR, ROWS, NW>), dim3(unsigned((n + ROWS - 1) / ROWS)),     \
                       dim3(64 * NW), tiled_lds_bytes(s, ROWS), s->stream, n, coords, params, s->d_freq,       \
                       s->cfg.n_freq, s->cfg.n_param, s->K0, s->cfg.depth, s->cfg.n_out, s->d_wb, s->d_wp,     \
                       s->d_w, off, out, ts ? *ts : TrainStore{})
#define TLED_TILED_ROWS(WIDTH, TR, NW)                      \
    switch (rows) {                                         \
        case 32: TLED_TILED(WIDTH, TR, 32, NW); break;      \
        case 64: TLED_TILED(WIDTH, TR, 64, NW); break;      \
        case 128: TLED_TILED(256, TR, 128, 8); break;       \
        default: TLED_FUSED(WIDTH, TR); break;              \
    }
    const int rows = tiled_rows(s, n);
    if (ts) {
        if (s->cfg.width == 64) { TLED_TILED_ROWS(64, true, 4) }
        else if (s->cfg.width == 128) { TLED_TILED_ROWS(128, true, 8) }
        else { TLED_TILED_ROWS(256, true, 8) }
    } else {
        if (s->cfg.width == 64) { TLED_TILED_ROWS(64, false, 4) }
        else if (s->cfg.width == 128) { TLED_TILED_ROWS(128, false, 8) }
        else { TLED_TILED_ROWS(256, false, 8) }
    }
#undef TLED_TILED_ROWS
#undef TLED_TILED
#undef TLED_FUSED
    MCHK(s, hipGetLastError());
    if (s->timing) {
        MCHK(s, hipEventRecord(e1, s->stream));
        MCHK(s, hipEventSynchronize(e1));
        float ms = 0.f;
        MCHK(s, hipEventElapsedTime(&ms, e0, e1));
        const double W = s->cfg.width;
        const double fl = 2.0 * double(n) * (double(s->K0) * W + (s->cfg.depth - 1) * W * W + W * s->cfg.n_out);
        if (ts) {   // the training forward: counted with the step's GEMMs
            s->gemm_ms += ms;
            s->gemm_flops += fl;
        } else {
            s->fused_ms += ms;
            s->fused_flops += fl;
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    return TLED_OK;
}

// Forward pass for n samples: features, hidden layers (Z, activations kept), output into d_y.
// With the fused kernel available, one launch writes all of them (the same bits as the
// layer-by-layer GEMMs, whose epilogue arithmetic it repeats).
tled_status forward(tled_mlp *s, long n, const float *coords, const float *params) {
    MTRY(ensure_workspace(s, n));
    const int W = s->cfg.width;
    if (fused_ok(s)) {
        TrainStore ts{};
        ts.x0 = s->d_x0;
        for (int l = 0; l < s->cfg.depth; ++l) {
            ts.z[l] = s->d_z[l];
            ts.a[l] = s->d_a[l];
        }
        return fused_forward(s, n, coords, params, s->d_y, &ts);
    }
    hipLaunchKernelGGL(features_kernel, dim3(blocks(n * s->K0)), dim3(kThreads), 0, s->stream, n, coords, params,
                       s->d_freq, s->cfg.n_freq, s->cfg.n_param, s->K0, s->d_x0);
    MCHK(s, hipGetLastError());
    const uint16_t *a = s->d_x0;
    int in = s->K0;
    for (int l = 0; l < s->cfg.depth; ++l) {
        const Layer &L = s->layers[l];
        MTRY(gemm<EPI_BIAS_SILU>(s, int(n), W, in, a, in, s->d_wb + L.w_off, 1, in, s->d_z[l], W, 1, s->d_a[l],
                                 s->d_w + L.b_off));
        a = s->d_a[l];
        in = W;
    }
    const Layer &O = s->layers.back();
    MTRY(gemm<EPI_BIAS_F32>(s, int(n), s->cfg.n_out, W, a, W, s->d_wb + O.w_off, 1, W, s->d_y, s->cfg.n_out, 1,
                            nullptr, s->d_w + O.b_off));
    return TLED_OK;
}

// Runs work between two events where the handle times its kernels, adding to its GEMMs.
template <typename F>
tled_status timed_gemm(tled_mlp *s, double flops, F work) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (s->timing) {
        MCHK(s, hipEventCreate(&e0));
        MCHK(s, hipEventCreate(&e1));
        MCHK(s, hipEventRecord(e0, s->stream));
    }
    work();
    MCHK(s, hipGetLastError());
    if (s->timing) {
        MCHK(s, hipEventRecord(e1, s->stream));
        MCHK(s, hipEventSynchronize(e1));
        float ms = 0.f;
        MCHK(s, hipEventElapsedTime(&ms, e0, e1));
        s->gemm_ms += ms;
        s->gemm_flops += flops;
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    return TLED_OK;
}

// dY, the loss partials and every hidden layer's dZ (see tiled_backward_kernel).
tled_status tiled_backward(tled_mlp *s, long n, const float *target) {
    const int W = s->cfg.width, D = s->cfg.depth, nko = (s->cfg.n_out + 31) / 32;
    BackStore bs{};
    for (int l = 0; l < D; ++l) {
        bs.z[l] = s->d_z[l];
        bs.dz[l] = s->d_dz[l];
    }
#define TLED_BACK(WIDTH, ROWS, NW)                                                                              \
    hipLaunchKernelGGL((tiled_backward_kernel<WIDTH, ROWS, NW>), dim3(unsigned((n + ROWS - 1) / ROWS)),           \
                       dim3(64 * NW), 2 * size_t(ROWS) * (WIDTH + 8) * sizeof(uint16_t), s->stream, n, s->d_y,    \
                       target, s->cfg.n_out, s->nop, nko, D, s->d_wt, s->d_dy, s->d_part, bs)
    const int rows = tiled_rows(s, n);
    return timed_gemm(s, 2.0 * double(n) * W * (s->cfg.n_out + double(D - 1) * W), [&] {
        if (W == 64) {
            if (rows == 32) TLED_BACK(64, 32, 4);
            else TLED_BACK(64, 64, 4);
        } else if (W == 128) {
            if (rows == 32) TLED_BACK(128, 32, 8);
            else TLED_BACK(128, 64, 8);
        } else {
            if (rows == 32) TLED_BACK(256, 32, 8);
            else if (rows == 64) TLED_BACK(256, 64, 8);
            else TLED_BACK(256, 128, 8);
        }
    });
#undef TLED_BACK
}

// Every layer's weight and bias gradient, as grad_chunks partials (see weight_grad_kernel).
tled_status weight_gradients(tled_mlp *s, long n) {
    const int nz = grad_chunks(s);
    s->grad_kchunk = ((n + nz - 1) / nz + 31) / 32 * 32;
    constexpr size_t lds = 4 * size_t(GK) * GP * sizeof(uint16_t);
    const int D = s->cfg.depth;
    double flops = 0.0;
    for (const Layer &L : s->layers) flops += 2.0 * double(n) * L.out * L.in;
    return timed_gemm(s, flops, [&] {
        for (int l0 = 0; l0 <= D; l0 += kGradJobs) {
            GradJobs jobs{};
            for (int l = l0; l <= D && l < l0 + kGradJobs; ++l) {
                const Layer &L = s->layers[l];
                const int nx = (L.in + GT - 1) / GT;
                jobs.j[jobs.count++] = GradJob{l < D ? s->d_dz[l] : s->d_dy, l > 0 ? s->d_a[l - 1] : s->d_x0,
                                               l < D ? L.out : s->nop, L.in, L.out, L.in, jobs.tiles, nx, L.w_off, L.b_off};
                jobs.tiles += nx * ((L.out + GT - 1) / GT);
            }
            hipLaunchKernelGGL(weight_grad_kernel, dim3(unsigned(jobs.tiles * nz)), dim3(kThreads), lds, s->stream, jobs, n,
                               nz, s->grad_kchunk, s->d_gpart, s->grad_stride);
        }
    });
}

// Loss and gradient, into d_g or, with adam, into a step of the optimizer (and *loss on the
// host if requested).
tled_status backward(tled_mlp *s, long n, const float *target, float *loss, const AdamArgs *adam) {
    const int W = s->cfg.width, no = s->cfg.n_out, D = s->cfg.depth;
    const Layer &O = s->layers.back();
    if (s->d_wt) {
        MTRY(tiled_backward(s, n, target));
    } else {
        hipLaunchKernelGGL(loss_grad_kernel, dim3(blocks(n * s->nop)), dim3(kThreads), 0, s->stream, n, no, s->nop, s->d_y,
                           target, s->d_dy, s->d_part);
        MCHK(s, hipGetLastError());
        // dZ of a hidden layer: the next layer's times its weights, through the SiLU, in the GEMM's epilogue
        MTRY(gemm<EPI_SILU_BACK>(s, int(n), W, no, s->d_dy, s->nop, s->d_wb + O.w_off, W, 1, nullptr, W, 1,
                                 s->d_dz[D - 1], s->d_z[D - 1]));
        for (int l = D - 1; l > 0; --l)
            MTRY(gemm<EPI_SILU_BACK>(s, int(n), W, W, s->d_dz[l], W, s->d_wb + s->layers[l].w_off, W, 1, nullptr, W, 1,
                                     s->d_dz[l - 1], s->d_z[l - 1]));
    }
    MTRY(weight_gradients(s, n));
    const AdamArgs none{};
    const long nfin = (s->P + kThreads - 1) / kThreads + 1;
    const int nz = int((n + s->grad_kchunk - 1) / s->grad_kchunk);
    const float scale = 1.0f / float(n * no);
    const int nl = int((n * s->nop + 63) / 64);
    if (adam)
        hipLaunchKernelGGL((grad_finish_kernel<true>), dim3(unsigned(nfin)), dim3(kThreads), 0, s->stream, s->P, nz,
                           s->grad_stride, s->d_gpart, s->d_g, *adam, nl, s->d_part, scale, s->d_loss);
    else
        hipLaunchKernelGGL((grad_finish_kernel<false>), dim3(unsigned(nfin)), dim3(kThreads), 0, s->stream, s->P, nz,
                           s->grad_stride, s->d_gpart, s->d_g, none, nl, s->d_part, scale, s->d_loss);
    MCHK(s, hipGetLastError());
    if (loss) {
        MCHK(s, hipMemcpyAsync(loss, s->d_loss, sizeof(float), hipMemcpyDeviceToHost, s->stream));
        MCHK(s, hipStreamSynchronize(s->stream));
    }
    return TLED_OK;
}

}  // namespace

extern "C" {

const char *tled_mlp_last_error(const tled_mlp *mlp) { return mlp ? mlp->err.c_str() : "null handle"; }

tled_status tled_mlp_create(tled_mlp **out, int device, const tled_mlp_config *cfg) {
    if (!out || !cfg) return TLED_E_ARG;
    *out = nullptr;
    if (cfg->n_param < 0 || cfg->n_freq < 1 || cfg->width < 64 || cfg->width % 64 || cfg->depth < 1 ||
        cfg->n_out < 1 || cfg->n_out > 64 || !(cfg->sigma > 0))
        return TLED_E_ARG;
    int nd = 0;
    if (hipGetDeviceCount(&nd) != hipSuccess || device < 0 || device >= nd) return TLED_E_HIP;
    if (hipSetDevice(device) != hipSuccess) return TLED_E_HIP;
    if (resolve_scratch(device) != TLED_OK) return TLED_E_HIP;
    tled_mlp *s = new (std::nothrow) tled_mlp();
    if (!s) return TLED_E_OOM;
    s->device = device;
    if (hipDeviceGetAttribute(&s->cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) {
        delete s;
        return TLED_E_HIP;
    }
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        s->d_static_split = g_scratch_addr[device];
    }
    s->cfg = *cfg;
    s->K0 = ((2 * cfg->n_freq + cfg->n_param + 31) / 32) * 32;
    long off = 0;
    int in = s->K0;
    for (int l = 0; l <= cfg->depth; ++l) {
        const int o = l < cfg->depth ? cfg->width : cfg->n_out;
        Layer L{in, o, off, off + long(o) * in};
        off += long(o) * in + o;
        s->layers.push_back(L);
        in = cfg->width;
    }
    s->P = off;
    s->nop = (cfg->n_out + 15) / 16 * 16;
    s->grad_stride = (off + 3) / 4 * 4;
    for (const Layer &L : s->layers) s->grad_tiles += long((L.out + GT - 1) / GT) * ((L.in + GT - 1) / GT);
    // frequencies ~ N(0, sigma^2) (Box-Muller) and uniform Glorot initial weights
    uint64_t rs = cfg->seed ^ 0x5eedf00dULL;
    s->freq.resize(3 * size_t(cfg->n_freq));
    for (auto &f : s->freq) {
        const double u1 = std::max(uniform01(rs), 1e-300), u2 = uniform01(rs);
        f = float(cfg->sigma * std::sqrt(-2.0 * std::log(u1)) * std::cos(6.283185307179586 * u2));
    }
    std::vector<float> w(s->P, 0.f);
    const double scale = cfg->init_scale > 0 ? cfg->init_scale : 1.0;
    for (int l = 0; l <= cfg->depth; ++l) {
        const Layer &L = s->layers[l];
        const int fan_in = l == 0 ? 2 * cfg->n_freq + cfg->n_param : L.in;
        const double lim = scale * std::sqrt(6.0 / double(fan_in + L.out));
        for (int o = 0; o < L.out; ++o)
            for (int i = 0; i < L.in; ++i)
                w[L.w_off + long(o) * L.in + i] = (l == 0 && i >= fan_in) ? 0.f : float(lim * (2.0 * uniform01(rs) - 1.0));
    }
    auto fail_free = [&](tled_status st) {
        tled_mlp_destroy(s);
        return st;
    };
    if (hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking) != hipSuccess) return fail_free(TLED_E_HIP);
    s->own_stream = true;
    if (hipEventCreateWithFlags(&s->done, hipEventDisableTiming) != hipSuccess) return fail_free(TLED_E_HIP);
    void *p;
    if (hipMalloc(&p, sizeof(float) * s->P) != hipSuccess) return fail_free(TLED_E_OOM);
    s->d_w = static_cast<float *>(p);
    if (hipMalloc(&p, sizeof(float) * s->P) != hipSuccess) return fail_free(TLED_E_OOM);
    s->d_g = static_cast<float *>(p);
    if (hipMalloc(&p, sizeof(float) * s->P) != hipSuccess) return fail_free(TLED_E_OOM);
    s->d_m = static_cast<float *>(p);
    if (hipMalloc(&p, sizeof(float) * s->P) != hipSuccess) return fail_free(TLED_E_OOM);
    s->d_v = static_cast<float *>(p);
    const long packed0 = (s->P + 7) / 8 * 8, later = long(cfg->depth - 1) * cfg->width * cfg->width;
    const long packed = tiled_ok(s) ? long(cfg->width) * s->K0 + later : 0;
    const long packed_t = tiled_ok(s) ? later + long(cfg->width) * 32 * ((cfg->n_out + 31) / 32) : 0;
    if (hipMalloc(&p, sizeof(uint16_t) * (packed0 + packed + packed_t)) != hipSuccess) return fail_free(TLED_E_OOM);
    s->d_wb = static_cast<uint16_t *>(p);
    if (packed) {
        s->d_wp = s->d_wb + packed0;
        s->d_wt = s->d_wp + packed;
        if (hipMemset(s->d_wt, 0, sizeof(uint16_t) * packed_t) != hipSuccess) return fail_free(TLED_E_HIP);   // padded units
    }
    if (hipMalloc(&p, sizeof(float) * s->freq.size()) != hipSuccess) return fail_free(TLED_E_OOM);
    s->d_freq = static_cast<float *>(p);
    if (hipMemcpy(s->d_freq, s->freq.data(), sizeof(float) * s->freq.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemset(s->d_m, 0, sizeof(float) * s->P) != hipSuccess ||
        hipMemset(s->d_v, 0, sizeof(float) * s->P) != hipSuccess)
        return fail_free(TLED_E_HIP);
    *out = s;
    if (tled_mlp_set_params(s, w.data()) != TLED_OK) {
        *out = nullptr;
        return fail_free(TLED_E_HIP);
    }
    return TLED_OK;
}

void tled_mlp_destroy(tled_mlp *s) {
    if (!s) return;
    (void)hipSetDevice(s->device);
    if (s->stream) (void)hipStreamSynchronize(s->stream);
    if (s->done_valid) (void)hipEventSynchronize(s->done);
    if (s->done) (void)hipEventDestroy(s->done);
    free_ws(s);
    if (s->d_split) (void)hipFree(s->d_split);
    for (void *p : {static_cast<void *>(s->d_w), static_cast<void *>(s->d_g), static_cast<void *>(s->d_m),
                    static_cast<void *>(s->d_v), static_cast<void *>(s->d_wb), static_cast<void *>(s->d_freq)})
        if (p) (void)hipFree(p);
    if (s->own_stream && s->stream) (void)hipStreamDestroy(s->stream);
    delete s;
}

// Work on stream from here on comes after what earlier calls have enqueued, whatever their
// streams: a handle's value does not tell one stream from another (hipStreamPerThread is
// one value for a stream per thread, and a destroyed stream's address is used again).  A
// stream under capture is left alone: an event from outside must not enter its graph.
static tled_status order_after_calls(tled_mlp *s, hipStream_t stream) {
    if (!s->done_valid) return TLED_OK;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    MCHK(s, hipStreamIsCapturing(stream, &capture));
    if (capture == hipStreamCaptureStatusNone) MCHK(s, hipStreamWaitEvent(stream, s->done, 0));
    return TLED_OK;
}

// Whether this thread is between begin and end (it then holds in_call).
static bool in_own_call(const tled_mlp *s) { return s->caller.load() == std::this_thread::get_id(); }

// Holds in_call over a call that may also be made between begin and end.
static std::unique_lock<std::mutex> call_lock(tled_mlp *s) {
    return in_own_call(s) ? std::unique_lock<std::mutex>() : std::unique_lock<std::mutex>(s->in_call);
}

tled_status tled_mlp_begin(tled_mlp *s, void *hip_stream) {
    if (!s) return TLED_E_ARG;
    if (in_own_call(s)) return mfail(s, TLED_E_STATE, "begin without the end of the one before");
    s->in_call.lock();
    const hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    tled_status st = TLED_OK;
    if (hipSetDevice(s->device) != hipSuccess) st = mfail(s, TLED_E_HIP, "hipSetDevice failed");
    if (st == TLED_OK) st = order_after_calls(s, stream);
    if (st != TLED_OK) {
        s->in_call.unlock();
        return st;
    }
    s->kept_stream = s->stream;
    s->stream = stream;
    s->caller = std::this_thread::get_id();
    return TLED_OK;
}

tled_status tled_mlp_end(tled_mlp *s) {
    if (!s) return TLED_E_ARG;
    if (!in_own_call(s)) return TLED_E_STATE;     // nothing is written: another thread may be in its calls
    const hipStream_t stream = s->stream;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(stream, &capture);
    if (e == hipSuccess && capture == hipStreamCaptureStatusNone) {
        e = hipEventRecord(s->done, stream);
        s->done_valid = s->done_valid || e == hipSuccess;
    }
    s->stream = s->kept_stream;
    s->caller = std::thread::id();
    const tled_status st = e == hipSuccess ? TLED_OK : mfail(s, TLED_E_HIP, hipGetErrorString(e));
    s->in_call.unlock();
    return st;
}

tled_status tled_mlp_set_stream(tled_mlp *s, void *hip_stream) {
    if (!s) return TLED_E_ARG;
    if (in_own_call(s)) return mfail(s, TLED_E_STATE, "set_stream between begin and end");
    std::lock_guard<std::mutex> lock(s->in_call);
    MCHK(s, hipStreamSynchronize(s->stream));
    if (s->done_valid) MCHK(s, hipEventSynchronize(s->done));
    if (s->own_stream && s->stream) (void)hipStreamDestroy(s->stream);
    s->own_stream = false;
    s->stream = static_cast<hipStream_t>(hip_stream);
    if (!s->stream) {
        MCHK(s, hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking));
        s->own_stream = true;
    }
    return TLED_OK;
}

tled_status tled_mlp_param_count(const tled_mlp *s, int64_t *n) {
    if (!s || !n) return TLED_E_ARG;
    *n = s->P;
    return TLED_OK;
}

tled_status tled_mlp_get_params(tled_mlp *s, float *host) {
    if (!s || !host) return TLED_E_ARG;
    const std::unique_lock<std::mutex> lock = call_lock(s);
    MCHK(s, hipSetDevice(s->device));
    MTRY(order_after_calls(s, s->stream));
    MCHK(s, hipMemcpyAsync(host, s->d_w, sizeof(float) * s->P, hipMemcpyDeviceToHost, s->stream));
    MCHK(s, hipStreamSynchronize(s->stream));
    return TLED_OK;
}

tled_status tled_mlp_set_params(tled_mlp *s, const float *host) {
    if (!s || !host) return TLED_E_ARG;
    const std::unique_lock<std::mutex> lock = call_lock(s);
    MCHK(s, hipSetDevice(s->device));
    MTRY(order_after_calls(s, s->stream));
    MCHK(s, hipMemcpyAsync(s->d_w, host, sizeof(float) * s->P, hipMemcpyHostToDevice, s->stream));
    hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks(s->P)), dim3(kThreads), 0, s->stream, s->P, s->d_w, s->d_wb,
                       packed_weights(s));
    MCHK(s, hipGetLastError());
    MCHK(s, hipStreamSynchronize(s->stream));
    return TLED_OK;
}

tled_status tled_mlp_get_frequencies(tled_mlp *s, float *host) {
    if (!s || !host) return TLED_E_ARG;
    std::memcpy(host, s->freq.data(), sizeof(float) * s->freq.size());
    return TLED_OK;
}

tled_status tled_mlp_forward(tled_mlp *s, int64_t n, const float *coords, const float *params, float *out) {
    if (!s || n < 0 || (n > 0 && (!coords || !out || (s->cfg.n_param > 0 && !params)))) return TLED_E_ARG;
    if (n == 0) return TLED_OK;
    MCHK(s, hipSetDevice(s->device));
    if (fused_ok(s)) return fused_forward(s, long(n), coords, params, out);
    MTRY(forward(s, long(n), coords, params));
    MCHK(s, hipMemcpyAsync(out, s->d_y, sizeof(float) * size_t(n) * s->cfg.n_out, hipMemcpyDeviceToDevice, s->stream));
    return TLED_OK;
}

tled_status tled_mlp_gradient(tled_mlp *s, int64_t n, const float *coords, const float *params, const float *target,
                              float *grad_host, float *loss) {
    if (!s || n <= 0 || !coords || !target || (s->cfg.n_param > 0 && !params)) return TLED_E_ARG;
    MCHK(s, hipSetDevice(s->device));
    MTRY(forward(s, long(n), coords, params));
    MTRY(backward(s, long(n), target, loss, nullptr));
    if (grad_host) {
        MCHK(s, hipMemcpyAsync(grad_host, s->d_g, sizeof(float) * s->P, hipMemcpyDeviceToHost, s->stream));
        MCHK(s, hipStreamSynchronize(s->stream));
    }
    return TLED_OK;
}

tled_status tled_mlp_train_step(tled_mlp *s, int64_t n, const float *coords, const float *params,
                                const float *target, float lr, float *loss) {
    if (!s || n <= 0 || !coords || !target || (s->cfg.n_param > 0 && !params) || !(lr > 0)) return TLED_E_ARG;
    MCHK(s, hipSetDevice(s->device));
    MTRY(forward(s, long(n), coords, params));
    // the step counts once its launches are through
    const float c1 = float(1.0 / (1.0 - std::pow(0.9, double(s->adam_t + 1))));
    const float c2 = float(1.0 / (1.0 - std::pow(0.999, double(s->adam_t + 1))));
    const AdamArgs adam{s->d_w, s->d_m, s->d_v, lr, c1, c2, s->d_wb,
                        packed_weights(s)};
    MTRY(backward(s, long(n), target, loss, &adam));
    s->adam_t += 1;
    MCHK(s, hipGetLastError());
    return TLED_OK;
}

tled_status tled_mlp_gemm(tled_mlp *s, int32_t m, int32_t n, int32_t k, const uint16_t *A, const uint16_t *B,
                          float *C) {
    if (!s || m <= 0 || n <= 0 || k <= 0 || !A || !B || !C) return TLED_E_ARG;
    MCHK(s, hipSetDevice(s->device));
    s->gemm_ms = s->fused_ms = s->gemm_flops = s->fused_flops = 0.0;
    MTRY(gemm<EPI_F32>(s, m, n, k, A, k, B, n, 1, C, n, 1, nullptr, nullptr));
    return TLED_OK;
}

tled_status tled_mlp_gemm_static(tled_mlp *s, int32_t m, int32_t n, int32_t k, const uint16_t *A,
                                 const uint16_t *B, float *C) {
    if (!s || m <= 0 || n <= 0 || k <= 0 || !A || !B || !C) return TLED_E_ARG;
    if (!s->d_static_split) return mfail(s, TLED_E_STATE, "static scratch not resolved for this device");
    MCHK(s, hipSetDevice(s->device));
    return gemm<EPI_F32>(s, m, n, k, A, k, B, n, 1, C, n, 1, nullptr, nullptr, s->d_static_split,
                         kStaticSplitFloats);
}

tled_status tled_mlp_ensemble_stats(int64_t n, int32_t members, int32_t n_out, const float *outs,
                                    const float *scale, float *mean, float *spread, void *hip_stream) {
    if (n < 0 || members < 1 || n_out < 1 || n_out > 64 || (n > 0 && (!outs || !scale || !mean || !spread)))
        return TLED_E_ARG;
    if (n == 0) return TLED_OK;
    hipLaunchKernelGGL(ensemble_stats_kernel, dim3(blocks(n)), dim3(kThreads), 0,
                       static_cast<hipStream_t>(hip_stream), long(n), int(members), int(n_out), outs, scale, mean,
                       spread);
    return hipGetLastError() == hipSuccess ? TLED_OK : TLED_E_HIP;
}

tled_status tled_mlp_scenario_inputs(int32_t n_scen, int32_t n_prm, int64_t n_rows, const int64_t *row_begin,
                                     const double *X, const double *probe, const double *xi, double p_scale,
                                     const float *prm, float *x_out, float *p_out, void *hip_stream) {
    if (n_scen < 1 || n_prm < 0 || n_prm > 64 || n_rows < 0 ||
        (n_rows > 0 && (!row_begin || !X || !probe || !xi || (n_prm > 0 && !prm) || !x_out || !p_out)))
        return TLED_E_ARG;
    if (n_rows == 0) return TLED_OK;
    hipLaunchKernelGGL(scenario_inputs_kernel, dim3(blocks(n_rows)), dim3(kThreads), 0,
                       static_cast<hipStream_t>(hip_stream), int(n_scen), int(n_prm), row_begin, X, probe, xi,
                       p_scale, prm, x_out, p_out);
    return hipGetLastError() == hipSuccess ? TLED_OK : TLED_E_HIP;
}

tled_status tled_mlp_scenario_outputs(int32_t n_scen, int64_t n_rows, const int64_t *row_begin, const float *mean,
                                      const float *spread, const float *T0, const float *sT, const float *su,
                                      float *T_out, float *u_out, float *spread_out, void *hip_stream) {
    if (n_scen < 1 || n_rows < 0 ||
        (n_rows > 0 && (!row_begin || !mean || !spread || !T0 || !sT || !su || !T_out || !u_out || !spread_out)))
        return TLED_E_ARG;
    if (n_rows == 0) return TLED_OK;
    hipLaunchKernelGGL(scenario_outputs_kernel, dim3(blocks(n_rows)), dim3(kThreads), 0,
                       static_cast<hipStream_t>(hip_stream), int(n_scen), row_begin, mean, spread, T0, sT, su, T_out,
                       u_out, spread_out);
    return hipGetLastError() == hipSuccess ? TLED_OK : TLED_E_HIP;
}

tled_status tled_mlp_set_timing(tled_mlp *s, int on) {
    if (!s) return TLED_E_ARG;
    s->timing = on != 0;
    s->gemm_ms = s->fused_ms = s->gemm_flops = s->fused_flops = 0.0;
    return TLED_OK;
}

tled_status tled_mlp_last_timing(tled_mlp *s, double ms[2], double flops[2]) {
    if (!s || !ms || !flops) return TLED_E_ARG;
    ms[0] = s->gemm_ms;
    ms[1] = s->fused_ms;
    flops[0] = s->gemm_flops;
    flops[1] = s->fused_flops;
    return TLED_OK;
}

}  // extern "C"
