// Kernels of the warm-start network (a small BF16 MLP, FP32 accumulation) for
// gfx950: a tiled GEMM on the matrix cores (v_mfma_f32_16x16x32_bf16), masked
// softmax cross-entropy, column sums for bias gradients, row gathers and
// Adam.  Each is a C-ABI call on caller-owned device buffers, asynchronous
// on the given stream; the network itself is orchestrated by the caller.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "pmx.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));

void pmx_set_error(const char* m);   // shared with the game library (pmx_last_error)

static int mfail(int code, const char* m) {
  pmx_set_error(m);
  return code;
}

#define MLP_TRY(expr)                                   \
  do {                                                  \
    hipError_t e_ = (expr);                             \
    if (e_ != hipSuccess) return mfail(PMX_EDEVICE, hipGetErrorString(e_)); \
  } while (0)

// Round to nearest even (one conversion instruction on gfx950; a NaN stays one).
__device__ inline uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ inline float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// ---------------------------------------------------------------------------
// C[M x N] = op(A)[M x K] * op(B)[K x N], FP32 accumulation on the gfx950
// matrix cores (v_mfma_f32_16x16x32_bf16: a 16 x 16 tile over 32 k per
// instruction, eight BF16 values of A and of B per lane).
// op(A)(m, k) = transA ? A[k * lda + m] : A[m * lda + k]
// op(B)(k, n) = transB ? B[n * ldb + k] : B[k * ldb + n]
// Epilogue per element: + bias[n]; ReLU; zero where mask[m * ldm + n] <= 0;
// store FP32 (C) and / or BF16 (Cb).
//
// Workgroup: 4 wavefronts, 64 x 64 output tile; each wavefront owns a 32 x 32
// quadrant (2 x 2 MFMA tiles).  K advances 64 per stage; both operands sit in
// LDS as [row][k] (k contiguous, rows padded by 16 bytes), so that a lane's
// eight k values of a fragment are one 16-byte LDS read.  Global loads are
// 16 bytes per lane where the operand's layout and alignment allow: eight
// consecutive k of one row (no transpose), or eight consecutive rows of one
// k, scattered into the [row][k] layout (transpose).  Two LDS buffers: the
// next stage's global loads are in flight while the current stage's MFMAs
// run, and one barrier per stage separates them.
//
// Split K (weight gradients: K = rows of the batch, M x N small): blockIdx.y
// takes one range of K and writes its raw FP32 tile to a workspace; a second
// kernel adds the ranges in a fixed order and applies the epilogue.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr int GT = 64, GK = 64, GKP = GK + 8;   // tile, K stage, padded LDS row (bf16)

struct GemmArgs {
  int M, N, K, kchunk;          // kchunk: K range per blockIdx.y (a multiple of GK)
  const uint16_t* A;
  int lda;
  const uint16_t* B;
  int ldb;
  const float* bias;
  int relu;
  const float* mask;
  int ldm;
  float* C;
  int ldc;
  uint16_t* Cb;
  int ldcb;
  float* work;                  // split K: [gridDim.y][M][N] partial sums
};

// One operand's share of a stage: two 16-byte pieces per thread (64 rows x
// 64 k = 512 pieces).  Rows count along M (for A) or N (for B); TR: the
// operand is stored row-contiguous (X[k * ld + r]), else k-contiguous
// (X[r * ld + k]); VEC: 16-byte loads are aligned.
template <bool TR, bool VEC>
struct StageLoad {
  uint4 v[2];
  __device__ inline void load(const uint16_t* __restrict__ X, int ld, int rows, int r0, int k0, int kend,
                              int tid) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = tid + 256 * j;
      uint16_t e[8];
      if (!TR) {   // X[r * ld + k]: eight consecutive k of row r
        const int r = r0 + c / 8, k = k0 + 8 * (c % 8);
        if (VEC && r < rows && k + 8 <= kend) {
          v[j] = *(const uint4*)(X + (int64_t)r * ld + k);
          continue;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = (r < rows && k + i < kend) ? X[(int64_t)r * ld + k + i] : (uint16_t)0;
      } else {     // X[k * ld + r]: eight consecutive rows at one k
        const int k = k0 + c / 8, r = r0 + 8 * (c % 8);
        if (VEC && k < kend && r + 8 <= rows) {
          v[j] = *(const uint4*)(X + (int64_t)k * ld + r);
          continue;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = (k < kend && r + i < rows) ? X[(int64_t)k * ld + r + i] : (uint16_t)0;
      }
      v[j] = make_uint4(e[0] | (uint32_t)e[1] << 16, e[2] | (uint32_t)e[3] << 16, e[4] | (uint32_t)e[5] << 16,
                        e[6] | (uint32_t)e[7] << 16);
    }
  }
  __device__ inline void store(uint16_t (*S)[GKP], int tid) const {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = tid + 256 * j;
      if (!TR) {
        *(uint4*)&S[c / 8][8 * (c % 8)] = v[j];
      } else {
        const int k = c / 8, r = 8 * (c % 8);
        const uint32_t w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          S[r + 2 * i][k] = (uint16_t)(w[i] & 0xffffu);
          S[r + 2 * i + 1][k] = (uint16_t)(w[i] >> 16);
        }
      }
    }
  }
};

__device__ inline void gemm_epilogue(const GemmArgs& P, int m, int n, float v) {
  if (P.bias) v += P.bias[n];
  if (P.relu) v = v > 0.f ? v : 0.f;
  if (P.mask && !(P.mask[(int64_t)m * P.ldm + n] > 0.f)) v = 0.f;
  if (P.C) P.C[(int64_t)m * P.ldc + n] = v;
  if (P.Cb) P.Cb[(int64_t)m * P.ldcb + n] = f2bf(v);
}

template <bool TRA, bool TRB, bool VA, bool VB>
__global__ __launch_bounds__(256) void k_gemm_bf16(GemmArgs P) {
  __shared__ __attribute__((aligned(16))) uint16_t As[2][GT][GKP];   // [m][k]
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][GT][GKP];   // [n][k]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int nbn = (P.N + GT - 1) / GT;
  const int m0 = (int)(blockIdx.x / nbn) * GT, n0 = (int)(blockIdx.x % nbn) * GT;
  const int kb = (int)blockIdx.y * P.kchunk, ke = min(P.K, kb + P.kchunk);
  const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  StageLoad<TRA, VA> la;
  StageLoad<TRB, VB> lb;
  const int nst = (ke - kb + GK - 1) / GK;
  if (nst > 0) {
    la.load(P.A, P.lda, P.M, m0, kb, ke, tid);
    lb.load(P.B, P.ldb, P.N, n0, kb, ke, tid);
    la.store(As[0], tid);
    lb.store(Bs[0], tid);
  }
  __syncthreads();
  for (int s = 0; s < nst; ++s) {
    const int buf = s & 1;
    if (s + 1 < nst) {   // the next stage's loads in flight during this stage's MFMAs
      la.load(P.A, P.lda, P.M, m0, kb + (s + 1) * GK, ke, tid);
      lb.load(P.B, P.ldb, P.N, n0, kb + (s + 1) * GK, ke, tid);
    }
#pragma unroll
    for (int kk = 0; kk < GK; kk += 32) {
      const int kq = kk + 8 * (lane >> 4);
      bf16x8 a[2], b[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        a[t] = *(const bf16x8*)&As[buf][wm + 16 * t + (lane & 15)][kq];
        b[t] = *(const bf16x8*)&Bs[buf][wn + 16 * t + (lane & 15)][kq];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (s + 1 < nst) {
      la.store(As[buf ^ 1], tid);
      lb.store(Bs[buf ^ 1], tid);
    }
    __syncthreads();
  }
  // lane holds D[4 * (lane / 16) + r][lane % 16] of each 16 x 16 tile
  float* wk = P.work ? P.work + (int64_t)blockIdx.y * P.M * P.N : nullptr;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
        const int n = n0 + wn + 16 * j + (lane & 15);
        if (m >= P.M || n >= P.N) continue;
        if (wk) wk[(int64_t)m * P.N + n] = acc[i][j][r];
        else gemm_epilogue(P, m, n, acc[i][j][r]);
      }
}

// Split K: the ranges' partial tiles added in range order, then the epilogue.
__global__ __launch_bounds__(256) void k_gemm_reduce(GemmArgs P, int splits) {
  const int64_t mn = (int64_t)P.M * P.N;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < mn; i += (int64_t)gridDim.x * blockDim.x) {
    float v = 0.f;
    for (int z = 0; z < splits; ++z) v += P.work[z * mn + i];
    gemm_epilogue(P, (int)(i / P.N), (int)(i % P.N), v);
  }
}

// ---------------------------------------------------------------------------
// Inference of the whole network (64 -> 512 -> 512 -> 8, ReLU) in one kernel:
// the activations of a tile of rows never leave the CU.  Everything runs
// transposed, features x rows, so that a lane of an MFMA result holds four
// consecutive features of one row: the hidden layer goes to LDS as [row][k]
// by 8-byte writes and comes back as 16-byte B fragments (rows padded by 16
// bytes: the 16 rows of a fragment fall on different banks), and the second
// hidden layer feeds the output layer's 16x16x16 MFMA straight from
// registers.
//
// Eight wavefronts, each 64 features of a hidden layer for every row of the
// tile; the second layer's weights stream from L2, the next k step in
// flight during the current one's MFMAs.  A tile of 128 rows (152 KB of LDS)
// asks 31 bytes per cycle and CU of L2 at the MFMA rate, a quarter of what 32
// rows would.  PACKED: those weights in fragment order, 1 KB contiguous per
// load; as stored, a k step would use half of each 128-byte line and find
// the other half evicted.  Workgroups take tiles in turn, the next tile's
// inputs in flight during the second layer.
//
// 1.5 M rows: 6.12 ms layer by layer with the activations through HBM in FP32
// and BF16 (148 TFLOP/s), 0.75 ms here (1,210 TFLOP/s; an 8192^3 library
// product reaches 1,190).  Up to 8,192 rows: 20 us, the latency of one tile.
// ---------------------------------------------------------------------------
constexpr int NetIn = 64, NetW = 512, NetOut = 8;
constexpr int NetPitch = NetW + 8;
constexpr int NetWaves = 8;                      // 64 features of a hidden layer each
typedef short s16x4 __attribute__((ext_vector_type(4)));

struct NetArgs {
  int64_t M;
  const uint16_t *X, *W1, *W2, *W3;
  const float *b1, *b2, *b3;
  float* Z;
};

// W2 in fragment order: [feature tile of 16][k step of 32][lane][8]
__global__ __launch_bounds__(256) void k_net_pack(const uint16_t* __restrict__ W, uint16_t* __restrict__ Wp) {
  const int i = blockIdx.x * 256 + threadIdx.x;   // one 16-byte piece
  const int lane = i & 63, ks = (i >> 6) % (NetW / 32), ft = (i >> 6) / (NetW / 32);
  ((uint4*)Wp)[i] = *(const uint4*)(W + (int64_t)(16 * ft + (lane & 15)) * NetW + 32 * ks + 8 * (lane >> 4));
}

__device__ inline s16x4 net_hidden(f32x4 v, const float* __restrict__ bias) {
  const float4 b = *(const float4*)bias;
  const float t[4] = {v[0] + b.x, v[1] + b.y, v[2] + b.z, v[3] + b.w};
  s16x4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = (short)f2bf(t[i] > 0.f ? t[i] : 0.f);
  return o;
}

template <int RT, bool PACKED>
__global__ __launch_bounds__(64 * NetWaves) __attribute__((amdgpu_waves_per_eu(RT == 8 ? 2 : 4)))
void k_net(NetArgs P, const uint16_t* __restrict__ W2p) {
  extern __shared__ __attribute__((aligned(16))) char net_smem[];
  constexpr int ROWS = 16 * RT;
  constexpr int XP = NetIn + 8;
  uint16_t* H = (uint16_t*)net_smem;             // [ROWS][NetPitch], then the waves' partial outputs
  uint16_t* Xs = H + ROWS * NetPitch;            // [ROWS][XP] inputs of the tile
  float* part = (float*)net_smem;                // [NetWaves][ROWS][NetOut]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l16 = lane & 15, lq = lane >> 4, f0 = 64 * w;
  // a tile's inputs as 16-byte pieces, at most two per thread (one for half
  // of the threads in a 32-row tile)
  constexpr int PIECES = ROWS * NetIn / 8, NT = 64 * NetWaves;
  static_assert(PIECES <= 2 * NT && (PIECES <= NT || PIECES == 2 * NT), "one or two input pieces per thread");
  const int xc0 = min(tid, PIECES - 1), xr0 = xc0 / (NetIn / 8), xk = 8 * (xc0 % (NetIn / 8));
  constexpr int xrd = NT / (NetIn / 8);          // rows between a thread's two pieces
  const int64_t tiles = (P.M + ROWS - 1) / ROWS;
  int64_t tile = blockIdx.x;
  uint4 xa = *(const uint4*)(P.X + min(tile * ROWS + xr0, P.M - 1) * NetIn + xk), xb = xa;
  if (PIECES > NT) xb = *(const uint4*)(P.X + min(tile * ROWS + xr0 + xrd, P.M - 1) * NetIn + xk);
  // this lane's second-layer fragments: feature tile i, k step ks at w2 + i * w2t + ks * w2k
  const uint16_t* w2 = PACKED ? W2p + (int64_t)(4 * w) * (NetW / 32) * 512 + 8 * lane
                              : P.W2 + (int64_t)(f0 + l16) * NetW + 8 * lq;
  constexpr int w2t = 16 * NetW, w2k = PACKED ? 512 : 32;
  for (; tile < tiles; tile += gridDim.x) {
    if (PIECES >= NT || tid < PIECES) *(uint4*)&Xs[xr0 * XP + xk] = xa;
    if (PIECES > NT) *(uint4*)&Xs[(xr0 + xrd) * XP + xk] = xb;
    f32x4 acc[4][RT];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < RT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();   // the inputs are in place; the last tile's partial outputs are read
    // layer 1
#pragma unroll
    for (int ks = 0; ks < NetIn / 32; ++ks) {
      bf16x8 a[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        a[i] = *(const bf16x8*)(P.W1 + (int64_t)(f0 + 16 * i + l16) * NetIn + 32 * ks + 8 * lq);
#pragma unroll
      for (int j = 0; j < RT; ++j) {
        const bf16x8 b = *(const bf16x8*)&Xs[(16 * j + l16) * XP + 32 * ks + 8 * lq];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b, acc[i][j], 0, 0, 0);
      }
    }
    bf16x8 an[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) an[i] = *(const bf16x8*)(w2 + i * w2t);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < RT; ++j) {
        *(s16x4*)&H[(16 * j + l16) * NetPitch + f0 + 16 * i + 4 * lq] = net_hidden(acc[i][j], P.b1 + f0 + 16 * i + 4 * lq);
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    __syncthreads();
    // layer 2, the next tile's inputs on their way
    if (tile + gridDim.x < tiles) {
      const int64_t r = (tile + gridDim.x) * ROWS + xr0;
      xa = *(const uint4*)(P.X + min(r, P.M - 1) * NetIn + xk);
      if (PIECES > NT) xb = *(const uint4*)(P.X + min(r + xrd, P.M - 1) * NetIn + xk);
    }
#pragma unroll 2
    for (int ks = 0; ks < NetW / 32; ++ks) {
      const int kn = min(ks + 1, NetW / 32 - 1);
      bf16x8 a[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = an[i];
#pragma unroll
      for (int i = 0; i < 4; ++i) an[i] = *(const bf16x8*)(w2 + i * w2t + kn * w2k);
#pragma unroll
      for (int j = 0; j < RT; ++j) {
        const bf16x8 b = *(const bf16x8*)&H[(16 * j + l16) * NetPitch + 32 * ks + 8 * lq];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b, acc[i][j], 0, 0, 0);
      }
    }
    // layer 3: this wavefront's 64 features, outputs 8 to 15 of the MFMA unused
    f32x4 z[RT];
#pragma unroll
    for (int j = 0; j < RT; ++j) z[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s16x4 a3 = {0, 0, 0, 0};
      if (l16 < NetOut) a3 = *(const s16x4*)(P.W3 + (int64_t)l16 * NetW + f0 + 16 * i + 4 * lq);
#pragma unroll
      for (int j = 0; j < RT; ++j)
        z[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a3, net_hidden(acc[i][j], P.b2 + f0 + 16 * i + 4 * lq), z[j], 0, 0, 0);
    }
    __syncthreads();   // the hidden layer is read
    if (lq < NetOut / 4)
#pragma unroll
      for (int j = 0; j < RT; ++j)
        *(f32x4*)&part[((w * ROWS) + 16 * j + l16) * NetOut + 4 * lq] = z[j];
    __syncthreads();
    for (int i = tid; i < ROWS * NetOut; i += 64 * NetWaves) {
      float v = 0.f;
#pragma unroll
      for (int k = 0; k < NetWaves; ++k) v += part[k * ROWS * NetOut + i];
      const int64_t r = tile * ROWS + i / NetOut;
      if (r < P.M) P.Z[r * NetOut + i % NetOut] = v + P.b3[i % NetOut];
    }
  }
}

// ---------------------------------------------------------------------------
// One training step's loss and gradients in three kernels after a repacking
// of the second layer's weights.
//
// k_net_rows: forward and backward of 32 rows per workgroup (256 workgroups at
// 8,192 rows), rows x features: a lane of an MFMA result holds four rows of
// one feature, so the eight rows that a lane holds over the tile's two row
// blocks are one 16-byte fragment of the weight gradients' products, whose
// contraction runs over rows.  Activations and their gradients go to LDS as
// [row][k] for the next layer and to HBM as such fragments (BF16, 1 KB
// contiguous per wavefront); ReLU masks stay in registers.
// k_net_wgrad: the three weight gradients as one launch of 64 x 64 wavefront
// tiles straight from the fragments (no LDS), K split over the grid.
// k_net_grads: the ranges' partial products, the workgroups' bias sums and the
// losses, each added in a fixed order.
//
// Layer by layer through HBM it was 16 launches, 300 us at 8,192 rows, of
// which column sums took 113 us (one thread per column adding 128 partials)
// and the GEMMs, at 64 x 64 tiles with 2-byte transposes through LDS, 160 us.
// Now 52 us with Adam's; in a kernel trace, where they add up to 56:
// k_net_rows 27 (every CU reads the second layer's weights twice, 512 KB in
// 6.3 us each time), k_net_wgrad 18 (its fragments' loads, 512 KB per
// workgroup), k_net_grads 5, Adam 4, packing 2.4.
// ---------------------------------------------------------------------------
constexpr int NetRows = 32;                      // rows per workgroup of k_net_rows
constexpr int NetBias = 2 * NetW + NetOut;       // bias gradients: b1, b2, b3
constexpr int NetGrads = NetW * NetW + NetW * NetIn + 16 * NetW;   // W2, W1, W3 (padded to 16 outputs)
// Ranges that the weight gradients' sums over rows are cut into: of eight row
// blocks while that fills the chip, up to 16; of 32 (1,024 rows) from 16 such
// on, up to 64 of any length, so that FP32 sums are no longer than the
// layer-by-layer products' (MFMA steps and partial sums in a row: 48 and 48 at
// 16,384 rows, 50 and 64 at 32,768, 52 and 96 at 65,536).  More ranges cost
// partial sums: 32,768 rows 156 us with 64, 151 us with 16.
__host__ __device__ constexpr int64_t net_splits(int64_t nb) {
  const int64_t s = nb / 8 < 16 ? nb / 8 : nb / 32 < 16 ? 16 : nb / 32;
  return s < 1 ? 1 : s > 64 ? 64 : s;
}

struct NetTrain {
  int64_t M, nb;                                 // rows; blocks of 32 rows
  const uint16_t* X;
  const float *T, *Wt;
  const uint16_t *W1, *W3;
  const float *b1, *b2, *b3;
  const uint16_t *W2f, *W2t;                     // W2 and its transpose in fragment order
  uint16_t *Xf, *H1f, *H2f, *D1f, *D2f, *D3f;    // row fragments [feature tile][row block][lane][8]
  float* bias;                                   // [nb][NetBias]
  float* loss;                                   // [nb]
};

// Fragment order of a 512 x 512 operand: [tile of 16 rows][k step of 32][lane][8];
// blockIdx.y = 1: of its transpose.
__global__ __launch_bounds__(256) void k_net_pack2(const uint16_t* __restrict__ W, uint16_t* __restrict__ Wf,
                                                   uint16_t* __restrict__ Wt) {
  const int i = blockIdx.x * 256 + threadIdx.x;   // one 16-byte piece
  const int lane = i & 63, ks = (i >> 6) % (NetW / 32), ft = (i >> 6) / (NetW / 32);
  const int r = 16 * ft + (lane & 15), k = 32 * ks + 8 * (lane >> 4);
  if (blockIdx.y == 0) {
    ((uint4*)Wf)[i] = *(const uint4*)(W + (int64_t)r * NetW + k);
  } else {
    uint32_t e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = W[(int64_t)(k + j) * NetW + r];
    ((uint4*)Wt)[i] = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
  }
}

// acc += A B^T over 512 k: A the rows in LDS, B this wavefront's 64 features
// in fragment order, PF k steps of it in flight.
__device__ inline void net_layer(f32x4 (&acc)[4][2], const uint16_t* __restrict__ S, const uint16_t* __restrict__ Wf,
                                 int w, int lane) {
  constexpr int PF = 4, KS = NetW / 32;
  const int l16 = lane & 15, lq = lane >> 4;
  const uint16_t* p = Wf + (int64_t)(4 * w) * KS * 512 + 8 * lane;
  bf16x8 bn[PF][4];
#pragma unroll
  for (int d = 0; d < PF; ++d)
#pragma unroll
    for (int i = 0; i < 4; ++i) bn[d][i] = *(const bf16x8*)(p + (i * KS + d) * 512);
#pragma unroll 1
  for (int k0 = 0; k0 < KS; k0 += PF) {
#pragma unroll
    for (int d = 0; d < PF; ++d) {
      bf16x8 b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) b[i] = bn[d][i];
      const int kn = min(k0 + d + PF, KS - 1);
#pragma unroll
      for (int i = 0; i < 4; ++i) bn[d][i] = *(const bf16x8*)(p + (i * KS + kn) * 512);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 a = *(const bf16x8*)&S[(16 * j + l16) * NetPitch + 32 * (k0 + d) + 8 * lq];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[i], acc[i][j], 0, 0, 0);
      }
    }
  }
}

typedef short s16x8 __attribute__((ext_vector_type(8)));

__global__ __launch_bounds__(64 * NetWaves) __attribute__((amdgpu_waves_per_eu(2))) void k_net_rows(NetTrain P) {
  extern __shared__ __attribute__((aligned(16))) char net_smem[];
  constexpr int R = NetRows, XP = NetIn + 8;
  uint16_t* H1 = (uint16_t*)net_smem;            // [R][NetPitch]
  uint16_t* H2 = H1 + R * NetPitch;              // [R][NetPitch], later the second layer's gradient
  uint16_t* Xs = H2 + R * NetPitch;              // [R][XP]
  uint16_t* W3 = Xs + R * XP;                    // [NetOut][NetPitch]
  uint16_t* Ds = W3 + NetOut * NetPitch;         // [R][16] output gradients, BF16 (8 unused)
  float* zs = (float*)(Ds + R * 16);             // [R][NetOut + 1] logits
  float* dz = zs + R * (NetOut + 1);             // [R][NetOut + 1] output gradients
  float* ls = dz + R * (NetOut + 1);             // [R] losses
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l16 = lane & 15, lq = lane >> 4, f0 = 64 * w;
  const int64_t rb = blockIdx.x, r0 = rb * R;
  // everything that does not depend on a previous layer is asked for at once
  if (tid < R * NetIn / 8) {
    const int r = tid / (NetIn / 8), k = 8 * (tid % (NetIn / 8));
    *(uint4*)&Xs[r * XP + k] = *(const uint4*)(P.X + min(r0 + r, P.M - 1) * NetIn + k);
  }
  *(uint4*)&W3[(tid / 64) * NetPitch + 8 * (tid % 64)] = *(const uint4*)(P.W3 + 8 * tid);
  static_assert(NetOut * NetW == 8 * 64 * NetWaves, "one 16-byte piece of W3 per thread");
  bf16x8 w1[2][4];
  float b1[4], b2[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int f = f0 + 16 * i + l16;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) w1[ks][i] = *(const bf16x8*)(P.W1 + (int64_t)f * NetIn + 32 * ks + 8 * lq);
    b1[i] = P.b1[f];
    b2[i] = P.b2[f];
  }
  __syncthreads();
  f32x4 acc[4][2];
  uint32_t on1 = 0, on2 = 0;                     // ReLU masks, bit 8 i + 4 j + r
  // layer 1
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16x8 a = *(const bf16x8*)&Xs[(16 * j + l16) * XP + 32 * ks + 8 * lq];
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w1[ks][i], acc[i][j], 0, 0, 0);
    }
  auto hidden = [&](uint16_t* __restrict__ S, uint16_t* __restrict__ F, const float (&bias)[4], uint32_t& on) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s16x8 o;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = acc[i][j][r] + bias[i];
          const bool pos = v > 0.f;
          on |= pos ? 1u << (8 * i + 4 * j + r) : 0u;
          const uint16_t h = f2bf(pos ? v : 0.f);
          o[4 * j + r] = (short)h;
          S[(16 * j + 4 * lq + r) * NetPitch + f0 + 16 * i + l16] = h;
          acc[i][j][r] = 0.f;
        }
      *(s16x8*)(F + ((int64_t)(4 * w + i) * P.nb + rb) * 512 + 8 * lane) = o;
    }
  };
  hidden(H1, P.H1f, b1, on1);
  if (w < NetIn / 16) {   // the inputs' row fragments, one feature tile per wavefront
    s16x8 o;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[4 * j + r] = (short)Xs[(16 * j + 4 * lq + r) * XP + 16 * w + l16];
    *(s16x8*)(P.Xf + ((int64_t)w * P.nb + rb) * 512 + 8 * lane) = o;
  }
  __syncthreads();
  // layer 2
  net_layer(acc, H1, P.W2f, w, lane);
  hidden(H2, P.H2f, b2, on2);
  __syncthreads();
  // logits: wavefronts 0 and 1, one row block each, over all features in the
  // order of the layer-by-layer product (another order would round a few
  // output gradients, and with them whole rows behind them, the other way)
  if (w < 2) {
    f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int ks = 0; ks < NetW / 32; ++ks) {
      const int k = 32 * ks + 8 * lq;
      const bf16x8 b = *(const bf16x8*)&W3[(l16 & (NetOut - 1)) * NetPitch + k];   // outputs 8 to 15 unused
      z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8*)&H2[(16 * w + l16) * NetPitch + k], b, z, 0, 0, 0);
    }
    if (l16 < NetOut)
#pragma unroll
      for (int r = 0; r < 4; ++r) zs[(16 * w + 4 * lq + r) * (NetOut + 1) + l16] = z[r] + P.b3[l16];
  }
  __syncthreads();
  if (tid < R) {
    // masked softmax cross-entropy, one row per thread (targets < 0: invalid)
    const bool live = r0 + tid < P.M;
    const int64_t row = live ? r0 + tid : P.M - 1;
    const float* zr = zs + tid * (NetOut + 1);
    float tr[NetOut];
    *(float4*)&tr[0] = make_float4(P.T[row * NetOut], P.T[row * NetOut + 1], P.T[row * NetOut + 2], P.T[row * NetOut + 3]);
    *(float4*)&tr[4] = make_float4(P.T[row * NetOut + 4], P.T[row * NetOut + 5], P.T[row * NetOut + 6], P.T[row * NetOut + 7]);
    const float wt = P.Wt ? P.Wt[row] : 1.f;
    float mx = -INFINITY;
#pragma unroll
    for (int a = 0; a < NetOut; ++a)
      if (tr[a] >= 0.f) mx = fmaxf(mx, zr[a]);
    float se = 0.f;
#pragma unroll
    for (int a = 0; a < NetOut; ++a)
      if (tr[a] >= 0.f) se += __expf(zr[a] - mx);
    const float lse = mx + __logf(se);
    float loss = 0.f;
#pragma unroll
    for (int a = 0; a < NetOut; ++a) {
      float g = 0.f;
      if (tr[a] >= 0.f) {
        const float lp = zr[a] - lse;
        loss -= tr[a] * lp;
        g = wt * (__expf(lp) - tr[a]);
      }
      g = live ? g : 0.f;
      dz[tid * (NetOut + 1) + a] = g;
      Ds[tid * 16 + a] = f2bf(g);
      Ds[tid * 16 + 8 + a] = 0;
    }
    ls[tid] = live ? loss * wt : 0.f;
  }
  __syncthreads();
  if (tid < NetOut) {
    float v = 0.f;
    for (int r = 0; r < R; ++r) v += dz[r * (NetOut + 1) + tid];
    P.bias[rb * NetBias + 2 * NetW + tid] = v;
  } else if (w == 1) {
    float v = ls[lane & (R - 1)];
#pragma unroll
    for (int m = R / 2; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
    if (lane == 0) P.loss[rb] = v;
  } else if (w == 2) {   // the output gradients' row fragment
    s16x8 o;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[4 * j + r] = (short)Ds[(16 * j + 4 * lq + r) * 16 + l16];
    *(s16x8*)(P.D3f + rb * 512 + 8 * lane) = o;
  }
  // masked gradient of a hidden layer: BF16 to LDS (if S) and as row
  // fragments, FP32 column sums (over lanes 16 apart) to the bias sums
  auto backward = [&](uint16_t* __restrict__ S, uint16_t* __restrict__ F, uint32_t on, int boff) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s16x8 o;
      float cs = 0.f;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = (on >> (8 * i + 4 * j + r)) & 1u ? acc[i][j][r] : 0.f;
          cs += v;
          const uint16_t h = f2bf(v);
          o[4 * j + r] = (short)h;
          if (S) S[(16 * j + 4 * lq + r) * NetPitch + f0 + 16 * i + l16] = h;
          acc[i][j][r] = 0.f;
        }
      *(s16x8*)(F + ((int64_t)(4 * w + i) * P.nb + rb) * 512 + 8 * lane) = o;
      cs += __shfl_xor(cs, 16, 64);
      cs += __shfl_xor(cs, 32, 64);
      if (lq == 0) P.bias[rb * NetBias + boff + f0 + 16 * i + l16] = cs;
    }
  };
  // second layer's gradient: dz W3 over the 8 outputs (k 8 to 31 of the MFMA zero)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    s16x8 b = {0, 0, 0, 0, 0, 0, 0, 0};
    if (lq == 0)
#pragma unroll
      for (int k = 0; k < NetOut; ++k) b[k] = (short)W3[k * NetPitch + f0 + 16 * i + l16];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      s16x8 a = {0, 0, 0, 0, 0, 0, 0, 0};
      if (lq == 0) a = *(const s16x8*)&Ds[(16 * j + l16) * 16];
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                          f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
  }
  backward(H2, P.D2f, on2, NetW);   // every wavefront has read H2 (the barriers above)
  __syncthreads();
  // first layer's gradient
  net_layer(acc, H2, P.W2t, w, lane);
  backward(nullptr, P.D1f, on1, 0);
}

// Weight gradients: wavefront tiles of 64 x 64 (16 x 64 for W3's, 8 of the 16
// outputs valid) over a range of row blocks: 64 tiles of dW2 = D2^T H1, 8 of
// dW1 = D1^T X, 8 of dW3 = D3^T H2, four per workgroup.
struct NetWgrad {
  const uint16_t *Xf, *H1f, *H2f, *D1f, *D2f, *D3f;
  float* part;                                   // [splits][NetGrads]
  int nb, per, splits;                           // row blocks; per split
};
constexpr int NetWgradTiles = 20;                // workgroups per split
template <int MT>
__device__ inline void net_wgrad(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, int nb, int k0, int k1,
                                 float* __restrict__ C, int ldc, int lane) {
  f32x4 acc[MT][4];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // PF row blocks of fragments in flight
  constexpr int PF = 4;
  bf16x8 an[PF][MT], bn[PF][4];
  const int64_t ts = (int64_t)nb * 512;          // next feature tile
#pragma unroll
  for (int d = 0; d < PF; ++d) {
    const int64_t kd = (int64_t)min(k0 + d, k1 - 1) * 512 + 8 * lane;
#pragma unroll
    for (int i = 0; i < MT; ++i) an[d][i] = *(const bf16x8*)(A + i * ts + kd);
#pragma unroll
    for (int j = 0; j < 4; ++j) bn[d][j] = *(const bf16x8*)(B + j * ts + kd);
  }
#pragma unroll 1
  for (int kb = k0; kb < k1; kb += PF) {
#pragma unroll
    for (int d = 0; d < PF; ++d) {
      if (kb + d >= k1) break;
      bf16x8 a[MT], b[4];
      const int64_t kn = (int64_t)min(kb + d + PF, k1 - 1) * 512 + 8 * lane;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        a[i] = an[d][i];
        an[d][i] = *(const bf16x8*)(A + i * ts + kn);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        b[j] = bn[d][j];
        bn[d][j] = *(const bf16x8*)(B + j * ts + kn);
      }
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) C[(int64_t)(16 * i + 4 * (lane >> 4) + r) * ldc + 16 * j + (lane & 15)] = acc[i][j][r];
}
__global__ __launch_bounds__(256) void k_net_wgrad(NetWgrad P) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // workgroups go to the eight XCDs in turn: the tiles of one split, which
  // read the same rows, share an XCD and its L2
  const int q = (int)blockIdx.x >> 3, split = ((int)blockIdx.x & 7) + 8 * (q / NetWgradTiles);
  if (split >= P.splits) return;
  const int k0 = split * P.per, k1 = min(P.nb, k0 + P.per);
  float* part = P.part + (int64_t)split * NetGrads;
  const int64_t ts = (int64_t)P.nb * 512;
  const int b = q % NetWgradTiles;
  if (b < 16) {
    const int mt = 2 * (b >> 2) + (w >> 1), nt = 2 * (b & 3) + (w & 1);   // 128 x 128 per workgroup
    net_wgrad<4>(P.D2f + 4 * mt * ts, P.H1f + 4 * nt * ts, P.nb, k0, k1, part + (int64_t)64 * mt * NetW + 64 * nt, NetW,
                 lane);
  } else if (b < 18) {
    const int mt = 4 * (b - 16) + w;
    net_wgrad<4>(P.D1f + 4 * mt * ts, P.Xf, P.nb, k0, k1, part + NetW * NetW + (int64_t)64 * mt * NetIn, NetIn, lane);
  } else {
    const int nt = 4 * (b - 18) + w;
    net_wgrad<1>(P.D3f, P.H2f + 4 * nt * ts, P.nb, k0, k1, part + NetW * NetW + NetW * NetIn + 64 * nt, NetW, lane);
  }
}

struct NetOutGrads {
  float *W1, *b1, *W2, *b2, *W3, *b3, *loss;
};
constexpr int NetGradBlocks = (NetGrads - 8 * NetW) / 1024;        // 1,024 weights per workgroup
constexpr int NetBiasBlocks = (NetBias + 15) / 16;                 // 16 bias gradients per workgroup
__global__ __launch_bounds__(256) void k_net_grads(const float* __restrict__ part, int splits,
                                                   const float* __restrict__ bias, const float* __restrict__ loss,
                                                   int nb, int n_loss, NetOutGrads O) {
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < NetGradBlocks) {
    const int i = (int)blockIdx.x * 1024 + 4 * tid;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    // 16 ranges in order, then the next 16
    for (int z0 = 0; z0 < splits; z0 += 16) {
      float4 u = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
      for (int z = z0; z < min(splits, z0 + 16); ++z) {
        const float4 p = *(const float4*)(part + (int64_t)z * NetGrads + i);
        u.x += p.x, u.y += p.y, u.z += p.z, u.w += p.w;
      }
      v.x += u.x, v.y += u.y, v.z += u.z, v.w += u.w;
    }
    float* dst = i < NetW * NetW ? O.W2 + i
               : i < NetW * NetW + NetW * NetIn ? O.W1 + (i - NetW * NetW) : O.W3 + (i - NetW * NetW - NetW * NetIn);
    *(float4*)dst = v;
    return;
  }
  const int b = (int)blockIdx.x - NetGradBlocks;
  if (b < NetBiasBlocks) {
    // 16 gradients, 16 ranges of row blocks each, the ranges added in order
    __shared__ float red[16][17];
    const int f = 16 * b + (tid & 15), sg = tid >> 4, per = (nb + 15) / 16;
    float v = 0.f;
    if (f < NetBias)
#pragma unroll 8
      for (int k = sg * per; k < min(nb, (sg + 1) * per); ++k) v += bias[(int64_t)k * NetBias + f];
    red[sg][tid & 15] = v;
    __syncthreads();
    if (tid < 16 && f < NetBias) {
      v = 0.f;
      for (int k = 0; k < 16; ++k) v += red[k][tid];
      (f < NetW ? O.b1 + f : f < 2 * NetW ? O.b2 + (f - NetW) : O.b3 + (f - 2 * NetW))[0] = v;
    }
    return;
  }
  const int i = (b - NetBiasBlocks) * 256 + tid;   // losses per 256 rows
  if (i < n_loss) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = 8 * i + k < nb ? loss[8 * i + k] : 0.f;
    O.loss[i] = ((v[0] + v[4]) + (v[2] + v[6])) + ((v[1] + v[5]) + (v[3] + v[7]));
  }
}

// Masked softmax cross-entropy per row: targets < 0 mark invalid actions.
// loss_r = w_r * sum_a -t_a log p_a ; dlogits = w_r * (p - t) on valid actions.
__global__ __launch_bounds__(256) void k_softmax_xent(int rows, int K, const float* __restrict__ z, int ldz,
                                                      const float* __restrict__ t, const float* __restrict__ wt,
                                                      float* __restrict__ dz, uint16_t* __restrict__ dzb,
                                                      float* __restrict__ partial) {
  __shared__ float red[256];
  const int r = blockIdx.x * 256 + threadIdx.x;
  float loss = 0.f;
  if (r < rows) {
    const float* zr = z + (int64_t)r * ldz;
    const float* tr = t + (int64_t)r * K;
    float mx = -INFINITY;
    for (int a = 0; a < K; ++a)
      if (tr[a] >= 0.f) mx = fmaxf(mx, zr[a]);
    float se = 0.f;
    for (int a = 0; a < K; ++a)
      if (tr[a] >= 0.f) se += __expf(zr[a] - mx);
    const float lse = mx + __logf(se);
    const float w = wt ? wt[r] : 1.f;
    for (int a = 0; a < K; ++a) {
      float g = 0.f;
      if (tr[a] >= 0.f) {
        const float lp = zr[a] - lse;
        loss -= tr[a] * lp;
        g = w * (__expf(lp) - tr[a]);
      }
      if (dz) dz[(int64_t)r * K + a] = g;
      if (dzb) dzb[(int64_t)r * K + a] = f2bf(g);
    }
    loss *= w;
  }
  red[threadIdx.x] = loss;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0 && partial) partial[blockIdx.x] = red[0];
}

// db[n] = sum over rows of dZ[m][n] (fixed order).  Without a workspace one
// thread per column walks every row; with one, blockIdx.y sums a range of
// kColRows rows into the workspace and k_colsum_reduce adds the ranges in
// order.
constexpr int kColRows = 64;
__global__ __launch_bounds__(256) void k_colsum(int rows, int cols, const float* __restrict__ dz,
                                                float* __restrict__ db, float* __restrict__ work) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  if (n >= cols) return;
  const int r0 = work ? (int)blockIdx.y * kColRows : 0, r1 = work ? min(rows, r0 + kColRows) : rows;
  float s = 0.f;
  for (int m = r0; m < r1; ++m) s += dz[(int64_t)m * cols + n];
  if (work) work[(int64_t)blockIdx.y * cols + n] = s;
  else db[n] = s;
}
__global__ __launch_bounds__(256) void k_colsum_reduce(int parts, int cols, const float* __restrict__ work,
                                                       float* __restrict__ db) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  if (n >= cols) return;
  float s = 0.f;
  for (int z = 0; z < parts; ++z) s += work[(int64_t)z * cols + n];
  db[n] = s;
}

// Adam over up to kAdamMax tensors in one launch (blockIdx.y: tensor).
constexpr int kAdamMax = 8;
struct AdamSet {
  int64_t n[kAdamMax];
  float *w[kAdamMax], *m[kAdamMax], *v[kAdamMax];
  const float* g[kAdamMax];
  uint16_t* wb[kAdamMax];
};
__global__ void k_adam(AdamSet S, float lr, float b1, float b2, float eps, float wd, float c1, float c2) {
  const int t = blockIdx.y;
  const int64_t n = S.n[t];
  float* __restrict__ w = S.w[t];
  const float* __restrict__ g = S.g[t];
  float* __restrict__ m = S.m[t];
  float* __restrict__ v = S.v[t];
  uint16_t* __restrict__ wb = S.wb[t];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i] + wd * w[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    if (wb) wb[i] = f2bf(wi);
  }
}

__global__ void k_gather_bf16(int64_t n, int width, const int64_t* __restrict__ idx,
                              const uint16_t* __restrict__ src, uint16_t* __restrict__ dst) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n * width;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / width, c = i % width;
    dst[i] = src[idx[r] * width + c];
  }
}

__global__ void k_gather_f32(int64_t n, int width, const int64_t* __restrict__ idx,
                             const float* __restrict__ src, float* __restrict__ dst) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n * width;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / width, c = i % width;
    dst[i] = src[idx[r] * width + c];
  }
}

__global__ void k_cast_bf16(int64_t n, const float* __restrict__ src, uint16_t* __restrict__ dst) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = f2bf(src[i]);
}

static int grid_for(int64_t n) { return (int)std::min<int64_t>((n + 255) / 256, 8192); }

extern "C" {

int mlp_gemm_bf16(int32_t M, int32_t N, int32_t K, const uint16_t* A, int32_t lda, int32_t transA,
                  const uint16_t* B, int32_t ldb, int32_t transB, const float* bias, int32_t relu,
                  const float* mask, int32_t ldm, float* C, int32_t ldc, uint16_t* Cb, int32_t ldcb,
                  float* work, int64_t work_elems, void* stream) {
  if (M < 0 || N < 0 || K < 0 || !A || !B || (!C && !Cb) || work_elems < 0)
    return mfail(PMX_EINVAL, "bad GEMM arguments");
  if ((transA ? lda < M : lda < K) || (transB ? ldb < K : ldb < N) || (C && ldc < N) ||
      (Cb && ldcb < N) || (mask && ldm < N))
    return mfail(PMX_EINVAL, "GEMM leading dimension too small");
  if (M == 0 || N == 0) return PMX_OK;
  const int64_t tiles = (int64_t)((N + GT - 1) / GT) * ((M + GT - 1) / GT);
  if (tiles > 0x7fffffff) return mfail(PMX_EINVAL, "GEMM too large");
  // split K when the tiles alone leave the chip idle and K is long: about
  // 2048 workgroups, at least 256 of K each, as the workspace allows
  int splits = 1;
  if (work && tiles < 512 && K >= 2 * 256) {
    const int64_t want = std::min<int64_t>(K / 256, (2048 + tiles - 1) / tiles);
    const int64_t room = work_elems / ((int64_t)M * N);
    splits = (int)std::max<int64_t>(1, std::min<int64_t>({want, room, 64}));
  }
  int kchunk = (int)((((int64_t)K + splits - 1) / splits + GK - 1) / GK * GK);
  if (kchunk == 0) kchunk = GK;
  splits = (int)(((int64_t)K + kchunk - 1) / kchunk);
  if (splits < 1) splits = 1;
  GemmArgs P{M, N, K, kchunk, A, lda, B, ldb, bias, relu, mask, ldm, C, ldc, Cb, ldcb, splits > 1 ? work : nullptr};
  // 16-byte loads need 16-byte aligned rows: base and leading dimension
  const bool va = ((uintptr_t)A % 16 == 0) && (lda % 8 == 0);
  const bool vb = ((uintptr_t)B % 16 == 0) && (ldb % 8 == 0);
  const dim3 grid((unsigned)tiles, (unsigned)splits);
  hipStream_t s = (hipStream_t)stream;
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, P); };
  // op(A) row-contiguous when transposed; op(B) when not (B[k * ldb + n])
  const int sel = (transA ? 8 : 0) | (transB ? 0 : 4) | (va ? 2 : 0) | (vb ? 1 : 0);
  switch (sel) {
    case 0: go(k_gemm_bf16<false, false, false, false>); break;
    case 1: go(k_gemm_bf16<false, false, false, true>); break;
    case 2: go(k_gemm_bf16<false, false, true, false>); break;
    case 3: go(k_gemm_bf16<false, false, true, true>); break;
    case 4: go(k_gemm_bf16<false, true, false, false>); break;
    case 5: go(k_gemm_bf16<false, true, false, true>); break;
    case 6: go(k_gemm_bf16<false, true, true, false>); break;
    case 7: go(k_gemm_bf16<false, true, true, true>); break;
    case 8: go(k_gemm_bf16<true, false, false, false>); break;
    case 9: go(k_gemm_bf16<true, false, false, true>); break;
    case 10: go(k_gemm_bf16<true, false, true, false>); break;
    case 11: go(k_gemm_bf16<true, false, true, true>); break;
    case 12: go(k_gemm_bf16<true, true, false, false>); break;
    case 13: go(k_gemm_bf16<true, true, false, true>); break;
    case 14: go(k_gemm_bf16<true, true, true, false>); break;
    default: go(k_gemm_bf16<true, true, true, true>); break;
  }
  if (splits > 1) {
    const int64_t mn = (int64_t)M * N;
    hipLaunchKernelGGL(k_gemm_reduce, dim3((unsigned)std::min<int64_t>((mn + 255) / 256, 4096)), dim3(256), 0, s,
                       P, splits);
  }
  MLP_TRY(hipGetLastError());
  return PMX_OK;
}

// Rows up to which the 32-row tiles are used, one workgroup per CU: they read
// the second layer's weights four times as often as 128-row tiles but give a
// small call four times the workgroups and need no packed weights (8,192 rows:
// 20.1 us, 21.4 us with 128-row tiles; beyond 256 workgroups they would run in
// rounds).
static constexpr int64_t kNetSmallRows = 32 * 256;

int mlp_forward_bf16(int64_t M, const uint16_t* X, const uint16_t* W1, const float* b1, const uint16_t* W2,
                     const float* b2, const uint16_t* W3, const float* b3, float* Z, uint16_t* work, void* stream) {
  if (M == 0) return PMX_OK;   // buffers of no rows may have no address
  if (M < 0 || !X || !W1 || !b1 || !W2 || !b2 || !W3 || !b3 || !Z || !work)
    return mfail(PMX_EINVAL, "bad network arguments");
  const uintptr_t all = (uintptr_t)X | (uintptr_t)W1 | (uintptr_t)b1 | (uintptr_t)W2 | (uintptr_t)b2 | (uintptr_t)W3 |
                        (uintptr_t)work;
  if (all % 16) return mfail(PMX_EINVAL, "network buffers must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const NetArgs P{M, X, W1, W2, W3, b1, b2, b3, Z};
  auto lds = [](int rows) { return sizeof(uint16_t) * (size_t)rows * (NetPitch + NetIn + 8); };
  if (M > kNetSmallRows) {
    hipLaunchKernelGGL(k_net_pack, dim3(NetW * NetW / 8 / 256), dim3(256), 0, s, W2, work);
    const int64_t tiles = (M + 127) / 128;
    hipLaunchKernelGGL((k_net<8, true>), dim3((unsigned)std::min<int64_t>(tiles, 256)), dim3(64 * NetWaves), lds(128),
                       s, P, work);
  } else {
    hipLaunchKernelGGL((k_net<2, false>), dim3((unsigned)((M + 31) / 32)), dim3(64 * NetWaves), lds(32), s, P, work);
  }
  MLP_TRY(hipGetLastError());
  return PMX_OK;
}

// Scratch of mlp_loss_and_grad_bf16: W2 twice in fragment order, the row
// fragments (M rounded up to 32 rows), split-K partial products, bias sums and
// losses per 32 rows; every part on a 256-byte boundary.
static int64_t net_train_layout(int64_t M, int64_t off[11]) {
  const int64_t nb = (M + NetRows - 1) / NetRows;
  const int64_t frag = nb * 512 * (int64_t)sizeof(uint16_t);   // one feature tile
  const int64_t bytes[10] = {2 * NetW * NetW, 2 * NetW * NetW, frag * (NetIn / 16), frag * (NetW / 16),
                             frag * (NetW / 16), frag * (NetW / 16), frag * (NetW / 16), frag,
                             (int64_t)sizeof(float) * net_splits(nb) * NetGrads,
                             (int64_t)sizeof(float) * nb * NetBias};
  off[0] = 0;
  for (int i = 0; i < 10; ++i) off[i + 1] = off[i] + (bytes[i] + 255) / 256 * 256;
  return off[10] + (int64_t)sizeof(float) * nb;
}

int64_t mlp_loss_and_grad_work(int64_t M) {
  int64_t off[11];
  return M < 0 ? 0 : net_train_layout(M, off);
}

int mlp_loss_and_grad_bf16(int64_t M, const uint16_t* X, const float* target, const float* weight, const uint16_t* W1,
                           const float* b1, const uint16_t* W2, const float* b2, const uint16_t* W3, const float* b3,
                           float* loss, float* gW1, float* gb1, float* gW2, float* gb2, float* gW3, float* gb3,
                           void* work, int64_t work_bytes, void* stream) {
  if (M < 1 || M > ((int64_t)1 << 34) || !X || !target || !W1 || !b1 || !W2 || !b2 || !W3 || !b3 || !loss || !gW1 ||
      !gb1 || !gW2 || !gb2 || !gW3 || !gb3 || !work)
    return mfail(PMX_EINVAL, "bad network arguments");
  const uintptr_t all = (uintptr_t)X | (uintptr_t)W1 | (uintptr_t)W2 | (uintptr_t)W3 | (uintptr_t)gW1 |
                        (uintptr_t)gW2 | (uintptr_t)gW3 | (uintptr_t)work;
  if (all % 16) return mfail(PMX_EINVAL, "network buffers must be 16-byte aligned");
  int64_t off[11];
  if (work_bytes < net_train_layout(M, off)) return mfail(PMX_EINVAL, "network workspace too small");
  char* wk = (char*)work;
  hipStream_t s = (hipStream_t)stream;
  NetTrain P;
  P.M = M;
  P.nb = (M + NetRows - 1) / NetRows;
  P.X = X;
  P.T = target;
  P.Wt = weight;
  P.W1 = W1;
  P.W3 = W3;
  P.b1 = b1;
  P.b2 = b2;
  P.b3 = b3;
  P.W2f = (uint16_t*)(wk + off[0]);
  P.W2t = (uint16_t*)(wk + off[1]);
  P.Xf = (uint16_t*)(wk + off[2]);
  P.H1f = (uint16_t*)(wk + off[3]);
  P.H2f = (uint16_t*)(wk + off[4]);
  P.D1f = (uint16_t*)(wk + off[5]);
  P.D2f = (uint16_t*)(wk + off[6]);
  P.D3f = (uint16_t*)(wk + off[7]);
  float* part = (float*)(wk + off[8]);
  P.bias = (float*)(wk + off[9]);
  P.loss = (float*)(wk + off[10]);
  hipLaunchKernelGGL(k_net_pack2, dim3(NetW * NetW / 8 / 256, 2), dim3(256), 0, s, W2, (uint16_t*)P.W2f,
                     (uint16_t*)P.W2t);
  const size_t lds = sizeof(uint16_t) * (NetRows * (2 * NetPitch + NetIn + 8 + 16) + NetOut * NetPitch) +
                     sizeof(float) * NetRows * (2 * (NetOut + 1) + 1);
  hipLaunchKernelGGL(k_net_rows, dim3((unsigned)P.nb), dim3(64 * NetWaves), lds, s, P);
  const int64_t splits0 = net_splits(P.nb);
  const int per = (int)((P.nb + splits0 - 1) / splits0), splits = (int)((P.nb + per - 1) / per);
  const NetWgrad Q{P.Xf, P.H1f, P.H2f, P.D1f, P.D2f, P.D3f, part, (int)P.nb, per, splits};
  hipLaunchKernelGGL(k_net_wgrad, dim3(8 * ((splits + 7) / 8) * NetWgradTiles), dim3(256), 0, s, Q);
  const int n_loss = (int)((M + 255) / 256);
  hipLaunchKernelGGL(k_net_grads, dim3(NetGradBlocks + NetBiasBlocks + (n_loss + 255) / 256), dim3(256), 0, s, part,
                     splits, P.bias, P.loss, (int)P.nb, n_loss, NetOutGrads{gW1, gb1, gW2, gb2, gW3, gb3, loss});
  MLP_TRY(hipGetLastError());
  return PMX_OK;
}

int mlp_softmax_xent(int32_t rows, int32_t K, const float* logits, int32_t ldl, const float* target,
                     const float* weight, float* dlogits, uint16_t* dlogits_bf16, float* loss_partial,
                     void* stream) {
  if (rows < 0 || K < 1 || K > 64 || !logits || !target || ldl < K) return mfail(PMX_EINVAL, "bad xent arguments");
  if (rows == 0) return PMX_OK;
  hipLaunchKernelGGL(k_softmax_xent, dim3((rows + 255) / 256), dim3(256), 0, (hipStream_t)stream, rows, K,
                     logits, ldl, target, weight, dlogits, dlogits_bf16, loss_partial);
  MLP_TRY(hipGetLastError());
  return PMX_OK;
}

int mlp_colsum(int32_t rows, int32_t cols, const float* dz, float* db, float* work, int64_t work_elems,
               void* stream) {
  if (rows < 0 || cols < 1 || !dz || !db || work_elems < 0) return mfail(PMX_EINVAL, "bad colsum arguments");
  hipStream_t s = (hipStream_t)stream;
  const int parts = (rows + kColRows - 1) / kColRows;
  if (work && parts > 1 && (int64_t)parts * cols <= work_elems) {
    hipLaunchKernelGGL(k_colsum, dim3((cols + 255) / 256, parts), dim3(256), 0, s, rows, cols, dz, db, work);
    hipLaunchKernelGGL(k_colsum_reduce, dim3((cols + 255) / 256), dim3(256), 0, s, parts, cols, work, db);
  } else {
    hipLaunchKernelGGL(k_colsum, dim3((cols + 255) / 256), dim3(256), 0, s, rows, cols, dz, db, nullptr);
  }
  MLP_TRY(hipGetLastError());
  return PMX_OK;
}

int mlp_adam_multi(int32_t n_tensors, const int64_t* n, float* const* w, const float* const* g, float* const* m,
                   float* const* v, uint16_t* const* w_bf16, float lr, float beta1, float beta2, float eps,
                   float weight_decay, int32_t step, void* stream) {
  if (n_tensors < 0 || n_tensors > kAdamMax || (n_tensors > 0 && (!n || !w || !g || !m || !v)) || step < 1)
    return mfail(PMX_EINVAL, "bad Adam arguments");
  AdamSet S{};
  int64_t most = 0;
  for (int t = 0; t < n_tensors; ++t) {
    if (n[t] < 0 || !w[t] || !g[t] || !m[t] || !v[t]) return mfail(PMX_EINVAL, "bad Adam arguments");
    S.n[t] = n[t];
    S.w[t] = w[t];
    S.g[t] = g[t];
    S.m[t] = m[t];
    S.v[t] = v[t];
    S.wb[t] = w_bf16 ? w_bf16[t] : nullptr;
    most = std::max(most, n[t]);
  }
  if (most == 0) return PMX_OK;
  const float c1 = 1.f - std::pow(beta1, (float)step), c2 = 1.f - std::pow(beta2, (float)step);
  hipLaunchKernelGGL(k_adam, dim3(grid_for(most), n_tensors), dim3(256), 0, (hipStream_t)stream, S, lr, beta1, beta2,
                     eps, weight_decay, c1, c2);
  MLP_TRY(hipGetLastError());
  return PMX_OK;
}

int mlp_adam(int64_t n, float* w, const float* g, float* m, float* v, uint16_t* w_bf16, float lr, float beta1,
             float beta2, float eps, float weight_decay, int32_t step, void* stream) {
  return mlp_adam_multi(1, &n, &w, &g, &m, &v, &w_bf16, lr, beta1, beta2, eps, weight_decay, step, stream);
}

int mlp_gather_bf16(int64_t n, int32_t width, const int64_t* idx, const uint16_t* src, uint16_t* dst,
                    void* stream) {
  if (n < 0 || width < 1 || !idx || !src || !dst) return mfail(PMX_EINVAL, "bad gather arguments");
  if (n == 0) return PMX_OK;
  hipLaunchKernelGGL(k_gather_bf16, dim3(grid_for(n * width)), dim3(256), 0, (hipStream_t)stream, n, width, idx,
                     src, dst);
  MLP_TRY(hipGetLastError());
  return PMX_OK;
}

int mlp_gather_f32(int64_t n, int32_t width, const int64_t* idx, const float* src, float* dst, void* stream) {
  if (n < 0 || width < 1 || !idx || !src || !dst) return mfail(PMX_EINVAL, "bad gather arguments");
  if (n == 0) return PMX_OK;
  hipLaunchKernelGGL(k_gather_f32, dim3(grid_for(n * width)), dim3(256), 0, (hipStream_t)stream, n, width, idx,
                     src, dst);
  MLP_TRY(hipGetLastError());
  return PMX_OK;
}

int mlp_cast_bf16(int64_t n, const float* src, uint16_t* dst, void* stream) {
  if (n < 0 || !src || !dst) return mfail(PMX_EINVAL, "bad cast arguments");
  if (n == 0) return PMX_OK;
  hipLaunchKernelGGL(k_cast_bf16, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, n, src, dst);
  MLP_TRY(hipGetLastError());
  return PMX_OK;
}

}  // extern "C"
