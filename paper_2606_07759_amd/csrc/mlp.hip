// Small multilayer perceptron for misregistration estimation: forward,
// backward (MSE loss) and Adam, hand-written for gfx950 in FP32.
//
// Net: x (n_in) -> h1 -> h2 -> n_out, y = x W^T + b per layer, ReLU after the
// two hidden layers.  Parameters are one packed buffer:
//   W1 [h1][n_in], b1 [h1], W2 [h2][h1], b2 [h2], W3 [n_out][h2], b3 [n_out].
// Inputs arrive compact: the input layer's non-zero inputs lie in two column
// segments of the full input (the rest is identically zero), so x is
// [B][len0 + len1] and compact column c feeds W1 column seg0 + c (c < len0) or
// seg1 + c - len0; the zero inputs contribute nothing and are skipped exactly.
#include <algorithm>
#include <climits>
#include <cmath>

#include "common.hpp"

namespace synim {
namespace {

// ------------------------------------------------------------ FP32 GEMM
// C[m][n] = alpha sum_k X(k, m) Y(k, n) (+ beta C[m][n]) (+ bias[n]) (then
// ReLU), X(k, m) = X[k sxk + m sxm], Y(k, n) = Y[k syk + n syn], C row-major.
// On the matrix cores: one 256-thread workgroup per 64x64 tile of C, each wave
// a 32x32 quarter as 2x2 blocks of v_mfma_f32_16x16x4f32 (lane l feeds
// A[l%16][l/16] and B[l/16][l%16] and holds D[4(l/16) + r][l%16], r = 0..3,
// checked on the device).  K advances in chunks of 32 through two LDS buffers,
// the next chunk's global loads in flight while the current one is multiplied.
// Split K: workgroup z of a split launch sums k in [z kc, (z+1) kc) and writes
// its partial tile to part[z][M][N]; gemm_reduce_kernel adds the partials in z
// order (a fixed order: the result does not depend on scheduling) and applies
// alpha, beta, bias and ReLU.
constexpr int MT = 64, MK = 32, MPAD = 1;
constexpr int MLOADS = MT * MK / 256;   // elements of one operand chunk per thread

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct MGemm {
  int M, N, K;
  const float* X;
  long sxk, sxm;
  const float* Y;
  long syk, syn;
  float* C;
  long ldc;
  float alpha, beta;
  const float* bias;
  int relu;
  float* part;   // split launches: [splits][M][N]
  int kc;        // K per split (a multiple of MK)
  int splits;
};

// (kk, mm) of element q of this thread in an MK x MT chunk, consecutive
// threads along the operand's unit stride
__device__ __forceinline__ void mg_elem(long sk, int tid, int q, int& kk, int& mm) {
  const int e = tid + 256 * q;
  if (sk == 1) {
    kk = e % MK;
    mm = e / MK;
  } else {
    kk = e / MT;
    mm = e % MT;
  }
}

__device__ __forceinline__ void mg_fetch(const float* P, long sk, long sm, int k0, int k1, int m0,
                                         int M, int tid, float (&r)[MLOADS]) {
#pragma unroll
  for (int q = 0; q < MLOADS; ++q) {
    int kk, mm;
    mg_elem(sk, tid, q, kk, mm);
    const int k = k0 + kk, m = m0 + mm;
    r[q] = (k < k1 && m < M) ? P[(long)k * sk + (long)m * sm] : 0.f;
  }
}

__device__ __forceinline__ void mg_put(long sk, int tid, const float (&r)[MLOADS],
                                       float (*S)[MT + MPAD]) {
#pragma unroll
  for (int q = 0; q < MLOADS; ++q) {
    int kk, mm;
    mg_elem(sk, tid, q, kk, mm);
    S[kk][mm] = r[q];
  }
}

__device__ __forceinline__ float mg_epilogue(const MGemm& g, float acc, int m, int n) {
  float v = g.alpha * acc;
  if (g.beta != 0.f) v += g.beta * g.C[(long)m * g.ldc + n];
  if (g.bias) v += g.bias[n];
  if (g.relu) v = fmaxf(v, 0.f);
  return v;
}

__global__ __launch_bounds__(256) void gemm_mfma_kernel(MGemm g) {
  const int m0 = blockIdx.y * MT, n0 = blockIdx.x * MT;
  const int kb = blockIdx.z * g.kc, ke = min(g.K, kb + g.kc);
  __shared__ float Xs[2][MK][MT + MPAD], Ys[2][MK][MT + MPAD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float rx[MLOADS], ry[MLOADS];
  mg_fetch(g.X, g.sxk, g.sxm, kb, ke, m0, g.M, tid, rx);
  mg_fetch(g.Y, g.syk, g.syn, kb, ke, n0, g.N, tid, ry);
  mg_put(g.sxk, tid, rx, Xs[0]);
  mg_put(g.syk, tid, ry, Ys[0]);
  __syncthreads();
  const int nk = ke > kb ? (ke - kb + MK - 1) / MK : 0;
  for (int c = 0; c < nk; ++c) {
    const int buf = c & 1;
    const bool more = c + 1 < nk;
    if (more) {
      mg_fetch(g.X, g.sxk, g.sxm, kb + (c + 1) * MK, ke, m0, g.M, tid, rx);
      mg_fetch(g.Y, g.syk, g.syn, kb + (c + 1) * MK, ke, n0, g.N, tid, ry);
    }
#pragma unroll
    for (int s = 0; s < MK / 4; ++s) {
      const int kr = 4 * s + (lane >> 4);
      float a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = Xs[buf][kr][wm + 16 * i + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = Ys[buf][kr][wn + 16 * j + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (more) {
      // the other buffer was last read in iteration c - 1, before its closing barrier
      mg_put(g.sxk, tid, rx, Xs[buf ^ 1]);
      mg_put(g.syk, tid, ry, Ys[buf ^ 1]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
        const int n = n0 + wn + 16 * j + (lane & 15);
        if (m >= g.M || n >= g.N) continue;
        if (g.splits > 1)
          g.part[((long)blockIdx.z * g.M + m) * g.N + n] = acc[i][j][r];
        else
          g.C[(long)m * g.ldc + n] = mg_epilogue(g, acc[i][j][r], m, n);
      }
}

__global__ __launch_bounds__(256) void gemm_reduce_kernel(MGemm g) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)g.M * g.N) return;
  const int m = (int)(i / g.N), n = (int)(i - (long)m * g.N);
  float s = 0.f;
  for (int z = 0; z < g.splits; ++z) s += g.part[(long)z * g.M * g.N + i];
  g.C[(long)m * g.ldc + n] = mg_epilogue(g, s, m, n);
}

// K splits of an M x N x K product: enough workgroups to cover the CUs when
// the tile grid alone is small, each split at least 4 chunks of K.
int gemm_splits(int M, int N, int K) {
  const long tiles = (long)((M + MT - 1) / MT) * ((N + MT - 1) / MT);
  long s = (256 + tiles - 1) / tiles;
  s = std::min<long>(s, std::max(1, K / (4 * MK)));
  return (int)std::max<long>(1, std::min<long>(s, 16));
}

long gemm_part_floats(int M, int N, int K) {
  const int s = gemm_splits(M, N, K);
  return s > 1 ? (long)s * M * N : 0;
}

// op(A) is M x K (A stored [M][lda] or, transposed, [K][lda]); op(B) is K x N
// (B stored [K][ldb] or, transposed, [N][ldb]).  part: gemm_part_floats floats.
template <bool TA, bool TB>
int gemm(int M, int N, int K, float alpha, const float* A, int lda, const float* B, int ldb,
         float beta, float* C, int ldc, const float* bias, int relu, float* part,
         hipStream_t st) {
  if (M <= 0 || N <= 0 || K <= 0) return SYNIM_OK;
  MGemm g{};
  g.M = M;
  g.N = N;
  g.K = K;
  g.X = A;
  g.sxk = TA ? lda : 1;
  g.sxm = TA ? 1 : lda;
  g.Y = B;
  g.syk = TB ? 1 : ldb;
  g.syn = TB ? ldb : 1;
  g.C = C;
  g.ldc = ldc;
  g.alpha = alpha;
  g.beta = beta;
  g.bias = bias;
  g.relu = relu;
  g.splits = gemm_splits(M, N, K);
  g.kc = (K + g.splits - 1) / g.splits;
  g.kc = (g.kc + MK - 1) / MK * MK;
  g.splits = (K + g.kc - 1) / g.kc;
  g.part = part;
  if (g.splits > 1 && !part) return SYNIM_E_WORKSPACE;
  dim3 grid((N + MT - 1) / MT, (M + MT - 1) / MT, g.splits);
  if (grid.y > 65535) return SYNIM_E_SHAPE;
  hipLaunchKernelGGL(gemm_mfma_kernel, grid, dim3(256), 0, st, g);
  SYNIM_HIP_TRY(hipGetLastError());
  if (g.splits > 1) {
    const long n = (long)M * N;
    hipLaunchKernelGGL(gemm_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g);
    SYNIM_HIP_TRY(hipGetLastError());
  }
  return SYNIM_OK;
}

// ------------------------------------------------- direct FP32 products
// C = X Y of small products whose operands allow 16-byte loads, without a
// workgroup-wide staging pipeline.  What bounds such a product is latency (the
// input layer, [256 x 2080] x [2080 x 512], is 0.55 GFLOP), so the W waves of a
// workgroup split K over one 16 BM x 16 BN tile of C, each keeps several 32-deep
// steps of loads in flight, and their partial tiles are added once, in wave
// order, through LDS; no step of the product waits at a barrier.
//   v_mfma_f32_16x16x4f32: lane l feeds A[l%16][l/16] and B[l/16][l%16] and holds
// D[4(l/16) + r][l%16].  A 32-deep step is eight of them; a lane's k in the e-th is
// 8(l/16) + e.  An operand contiguous across k (not AK, BK) is loaded as the lane
// needs it, a BM- (BN-) wide vector per e, whose element i belongs to block i (row
// BM r + i of the tile).  One contiguous in k is loaded in whole 128-byte row
// segments, eight lanes each, and turned through LDS of the wave's own (loaded
// as needed, no two neighbouring lanes would read one row: 62 cache accesses
// per load, and the input layer took 16 us in place of 13).
// Measured on the training step of the estimator (B = 256): input layer 28 us
// before (column gather, staged product, split-K reduction), 13 now; a step
// 162 us and 24 launches before, 70 us and 7 now, of which 18 are Adam's.
struct DGemm {
  int M, N, K;
  const float* X;    // AK: X[m][k] (ldx), else X[k][m]
  const float* Y;    // BK: Y[n][k] (ldy), else Y[k][n]
  long ldx, ldy;
  float* C;
  long ldc;
  const float* bias;   // [N], added (nullable)
  const float* mask;   // [M][ldc]: C = 0 where it is not positive (nullable)
  int relu;
  // column maps (input layer): k of Y (BK), or column n of C, from len0 on
  // lies at shift + itself
  int len0, shift;     // len0 = INT_MAX: none
  float* rowsum;       // [M]: sum over k of X(k, m) (nullable; !AK)
  // zero fill of C's columns outside the map by the workgroups past the tiles
  int zero_cols;       // full width of C (0: none)
  int col0;            // first mapped column
};

template <int V>
__device__ __forceinline__ void load_vec(const float* p, float (&r)[V]) {
  if constexpr (V == 4) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    r[0] = t.x; r[1] = t.y; r[2] = t.z; r[3] = t.w;
  } else if constexpr (V == 2) {
    const float2 t = *reinterpret_cast<const float2*>(p);
    r[0] = t.x; r[1] = t.y;
  } else {
    r[0] = *p;
  }
}

constexpr int DIRECT_PITCH = 36;   // floats from row to row of a turned step

// Registers one operand of a 32-deep step takes per lane: 8 NB floats.
// Contiguous in k: float4 j is row 8 j + l/8, k = 4(l%8); else element e NB + i.
// Rows (or vectors) past the operand's extent repeat its last; k past ke reads
// zero (ke is a multiple of 4 where the operand is contiguous in k).
template <int NB, bool KC>
__device__ __forceinline__ void direct_load(const float* P, long ld, int m0, int M, int k0, int ke,
                                            int len0, int shift, int lane, float (&r)[8 * NB]) {
  if constexpr (KC) {
    const int k = k0 + 4 * (lane & 7);
    const float* base = P + (k < len0 ? k : k + shift);
#pragma unroll
    for (int j = 0; j < 2 * NB; ++j) {
      const int m = min(m0 + 8 * j + (lane >> 3), M - 1);
      float t[4] = {0.f, 0.f, 0.f, 0.f};
      if (k < ke) load_vec<4>(base + (long)m * ld, t);
#pragma unroll
      for (int u = 0; u < 4; ++u) r[4 * j + u] = t[u];
    }
  } else {
    const int m = min(m0 + NB * (lane & 15), M - NB);
    const int k = k0 + 8 * (lane >> 4);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float t[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) t[i] = 0.f;
      if (k + e < ke) load_vec<NB>(P + (long)(k + e) * ld + m, t);
#pragma unroll
      for (int i = 0; i < NB; ++i) r[e * NB + i] = t[i];
    }
  }
}

// Orders a wave's own LDS writes before its lanes' reads of each other's (and
// the other way round); the LDS serves a wave's operations in order.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int NB>
__device__ __forceinline__ void direct_put(const float (&r)[8 * NB], float* lds, int lane) {
#pragma unroll
  for (int j = 0; j < 2 * NB; ++j)
    *reinterpret_cast<float4*>(lds + (8 * j + (lane >> 3)) * DIRECT_PITCH + 4 * (lane & 7)) =
        make_float4(r[4 * j], r[4 * j + 1], r[4 * j + 2], r[4 * j + 3]);
}
// block i's values for the four e of half h
template <int NB>
__device__ __forceinline__ void direct_get(const float* lds, int h, int lane, float (&v)[4][NB]) {
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    float t[4];
    load_vec<4>(lds + (16 * i + (lane & 15)) * DIRECT_PITCH + 8 * (lane >> 4) + 4 * h, t);
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s][i] = t[s];
  }
}

// LDS floats a wave turns its operands in
constexpr int direct_turn(int bm, int bn, bool ak, bool bk) {
  return ((ak ? bm : 0) + (bk ? bn : 0)) * 16 * DIRECT_PITCH;
}

template <int BM, int BN, bool AK, bool BK>
__device__ __forceinline__ void direct_tile(const DGemm& g, int tile, float* lds) {
  constexpr int TM = 16 * BM, TN = 16 * BN;
  constexpr int DEPTH = BM * BN >= 4 ? 2 : 4;   // steps of loads in flight
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, W = blockDim.x >> 6;
  // Consecutive workgroups go to the 8 XCDs in turn.  Where the column tiles
  // divide by 8, an XCD takes an eighth of them with every row tile, so that
  // its L2 reads its own eighth of Y (the weights) and X once; otherwise row by
  // row of tiles.
  const int tn = (g.N + TN - 1) / TN;
  int tm_i = tile / tn, tn_i = tile % tn;
  if (tn % 8 == 0) {
    const int per = tn / 8, q = tile >> 3;
    tn_i = (tile & 7) * per + q % per;
    tm_i = q / per;
  }
  const int m0 = tm_i * TM, n0 = tn_i * TN;
  const int steps = (g.K + 31) / 32;
  const int s0 = (int)((long)steps * wave / W), s1 = (int)((long)steps * (wave + 1) / W);
  f32x4 acc[BM][BN];
#pragma unroll
  for (int i = 0; i < BM; ++i)
#pragma unroll
    for (int j = 0; j < BN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float rs[BM];
#pragma unroll
  for (int i = 0; i < BM; ++i) rs[i] = 0.f;
  float* const turn_a = lds + (size_t)wave * direct_turn(BM, BN, AK, BK);
  float* const turn_b = turn_a + (AK ? BM * 16 * DIRECT_PITCH : 0);
  float a[DEPTH][8 * BM], b[DEPTH][8 * BN];
  auto load = [&](int d, int st) {
    direct_load<BM, AK>(g.X, g.ldx, m0, g.M, 32 * st, g.K, INT_MAX, 0, lane, a[d]);
    direct_load<BN, BK>(g.Y, g.ldy, n0, g.N, 32 * st, g.K, BK ? g.len0 : INT_MAX, g.shift, lane,
                        b[d]);
  };
#pragma unroll
  for (int d = 0; d < DEPTH; ++d)
    if (s0 + d < s1) load(d, s0 + d);
  for (int st = s0; st < s1; st += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      if (st + d >= s1) break;
      if constexpr (AK || BK) {
        wave_sync();
        if constexpr (AK) direct_put<BM>(a[d], turn_a, lane);
        if constexpr (BK) direct_put<BN>(b[d], turn_b, lane);
        wave_sync();
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float va[4][BM], vb[4][BN];
        if constexpr (AK) direct_get<BM>(turn_a, h, lane, va);
        if constexpr (BK) direct_get<BN>(turn_b, h, lane, vb);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          if constexpr (!AK)
#pragma unroll
            for (int i = 0; i < BM; ++i) {
              va[s][i] = a[d][(4 * h + s) * BM + i];
              rs[i] += va[s][i];
            }
          if constexpr (!BK)
#pragma unroll
            for (int j = 0; j < BN; ++j) vb[s][j] = b[d][(4 * h + s) * BN + j];
#pragma unroll
          for (int i = 0; i < BM; ++i)
#pragma unroll
            for (int j = 0; j < BN; ++j)
              acc[i][j] =
                  __builtin_amdgcn_mfma_f32_16x16x4f32(va[s][i], vb[s][j], acc[i][j], 0, 0, 0);
        }
      }
      if (st + d + DEPTH < s1) load(d, st + d + DEPTH);
    }
  }
  if constexpr (AK || BK) __syncthreads();   // the turning space is the partial tiles' now
  // The waves' partial tiles, row-major (+1 float per row against conflicts):
  // the upper half of the waves hands its tiles to the lower half, whose sums
  // then lie side by side (half the LDS of all tiles at once).
  constexpr int LD = TN + 1;
  const int H = W >> 1;
  float* mine = lds + (size_t)(wave >= H ? wave - H : wave) * TM * LD;
  auto each = [&](auto f) {
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int rr = 4 * (lane >> 4) + r;
          const int row = AK ? 16 * i + rr : BM * rr + i;
          const int col = BK ? 16 * j + (lane & 15) : BN * (lane & 15) + j;
          f(acc[i][j][r], mine[row * LD + col]);
        }
  };
  if (wave >= H) each([](float v, float& slot) { slot = v; });
  __syncthreads();
  if (wave < H) each([](float v, float& slot) { slot = v + slot; });
  const bool sums = !AK && g.rowsum != nullptr && n0 == 0;
  float* rsl = lds + (size_t)H * TM * LD;   // [W][4][TM]
  if (sums) {
#pragma unroll
    for (int i = 0; i < BM; ++i)
      rsl[(wave * 4 + (lane >> 4)) * TM + BM * (lane & 15) + i] = rs[i];
  }
  __syncthreads();
  for (int e = tid; e < TM * TN; e += blockDim.x) {
    const int row = e / TN, col = e % TN;
    float v = 0.f;
    for (int w = 0; w < H; ++w) v += lds[((size_t)w * TM + row) * LD + col];
    const int m = m0 + row, n = n0 + col;
    if (m >= g.M || n >= g.N) continue;
    if (g.bias) v += g.bias[n];
    if (g.relu) v = fmaxf(v, 0.f);
    if (g.mask && !(g.mask[(long)m * g.ldc + n] > 0.f)) v = 0.f;
    g.C[(long)m * g.ldc + (BK ? n : (n < g.len0 ? n : n + g.shift))] = v;
  }
  if (sums)
    for (int row = tid; row < TM; row += blockDim.x) {
      float v = 0.f;
      for (int w = 0; w < 4 * W; ++w) v += rsl[w * TM + row];
      if (m0 + row < g.M) g.rowsum[m0 + row] = v;
    }
}

// Tiles of one product (t1 = 0), or of two that share a launch; before them
// (they only store, and overlap the tiles' loads) the nz workgroups that zero
// C's unmapped columns, ZERO_ROWS rows each, rounded up to a multiple of 8.
constexpr int ZERO_ROWS = 1;
template <int BM, int BN, bool AK, bool BK, int BM1, int BN1, bool AK1, bool BK1>
__global__ __launch_bounds__(512) void direct_kernel(int nz, DGemm g, int t0, DGemm h, int t1) {
  extern __shared__ __align__(16) float dyn_lds[];
  const int t = (int)blockIdx.x - nz;
  if (t >= 0 && t < t0) {
    direct_tile<BM, BN, AK, BK>(g, t, dyn_lds);
  } else if (t >= t0) {
    direct_tile<BM1, BN1, AK1, BK1>(h, t - t0, dyn_lds);
  } else {
    // columns [0, col0), the gap between the segments, and what follows them
    const int m0 = (int)blockIdx.x * ZERO_ROWS;
    const int end0 = g.col0 + g.len0;                       // end of the first segment
    const int beg1 = g.col0 + g.len0 + g.shift;             // start of the second
    const int end1 = g.col0 + g.shift + g.N;
    float* C0 = g.C - g.col0;
    for (int r = 0; r < ZERO_ROWS && m0 + r < g.M; ++r) {
      float* row = C0 + (long)(m0 + r) * g.ldc;
      for (int c = 4 * threadIdx.x; c < g.zero_cols; c += 4 * blockDim.x) {
        const bool used = (c >= g.col0 && c < end0) || (c >= beg1 && c < end1);
        if (!used) *reinterpret_cast<float4*>(row + c) = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  }
}

constexpr int direct_lds(int W, int bm, int bn, bool ak, bool bk) {
  return std::max(W / 2 * 16 * bm * (16 * bn + 1) + W * 4 * 16 * bm,
                  W * direct_turn(bm, bn, ak, bk)) * (int)sizeof(float);
}
inline int direct_tiles(int M, int N, int bm, int bn) {
  return ((M + 16 * bm - 1) / (16 * bm)) * ((N + 16 * bn - 1) / (16 * bn));
}
// Waves per workgroup: as many as leave each at least two 32-deep steps, while
// the tiles alone do not give every SIMD a few waves.
inline int direct_waves(int tiles, int K, int most) {
  int W = 4;
  while (W < most && (long)tiles * W < 256 * 8 && (K + 31) / 32 >= 4 * W) W *= 2;
  return W;
}

// Small batches (B <= 16): one workgroup per output unit, lanes split K, so the
// weight rows stream once at full bandwidth.  x [B][ldx], W rows of length ldw
// with the compact-to-full column map (seg0, len0, seg1) for the input layer.
template <int MB>
__global__ __launch_bounds__(256) void linear_small_kernel(int B, int N, int K,
                                                           const float* __restrict__ x, int ldx,
                                                           const float* __restrict__ W, int ldw,
                                                           int seg0, int len0, int seg1,
                                                           const float* __restrict__ bias,
                                                           int relu, float* __restrict__ y,
                                                           int ldy) {
  const int n = blockIdx.x;
  const float* w = W + (size_t)n * ldw;
  float acc[MB] = {};
  for (int k = threadIdx.x; k < K; k += 256) {
    const int col = k < len0 ? seg0 + k : seg1 + (k - len0);
    const float wk = w[col];
#pragma unroll
    for (int b = 0; b < MB; ++b)
      if (b < B) acc[b] = __fmaf_rn(wk, x[(size_t)b * ldx + k], acc[b]);
  }
  __shared__ float red[MB][256];
#pragma unroll
  for (int b = 0; b < MB; ++b) red[b][threadIdx.x] = acc[b];
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s)
#pragma unroll
      for (int b = 0; b < MB; ++b) red[b][threadIdx.x] += red[b][threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x < MB && threadIdx.x < B) {
    float v = red[threadIdx.x][0] + (bias ? bias[n] : 0.f);
    if (relu) v = fmaxf(v, 0.f);
    y[(size_t)threadIdx.x * ldy + n] = v;
  }
}

__global__ void relu_mask_kernel(float* __restrict__ g, const float* __restrict__ h, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && !(h[i] > 0.f)) g[i] = 0.f;
}

// Column sums of g [B][N] (bias gradients) in a fixed order: 64 columns per
// 256-thread workgroup, each column's rows split over 4 thread groups with 4
// independent accumulators each (16 loads in flight per column instead of one
// long dependent chain), then combined in a fixed order.
constexpr int CS_COLS = 64, CS_PARTS = 4, CS_ACC = 4;
__global__ __launch_bounds__(256) void colsum_kernel(const float* __restrict__ g, int B, int N,
                                                     float* __restrict__ out) {
  __shared__ float red[CS_PARTS][CS_COLS];
  const int c = threadIdx.x % CS_COLS, part = threadIdx.x / CS_COLS;
  const int n = blockIdx.x * CS_COLS + c;
  float acc[CS_ACC] = {};
  if (n < N) {
    int b = part;
    for (; b + (CS_ACC - 1) * CS_PARTS < B; b += CS_ACC * CS_PARTS)
#pragma unroll
      for (int u = 0; u < CS_ACC; ++u) acc[u] += g[(size_t)(b + u * CS_PARTS) * N + n];
    for (int u = 0; b < B; b += CS_PARTS, ++u) acc[u] += g[(size_t)b * N + n];
  }
  red[part][c] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (part == 0 && n < N) out[n] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
}

// dY = 2 (Y - T) / (B * n_out) and the MSE loss (one workgroup).
__global__ void mse_grad_kernel(const float* __restrict__ y, const float* __restrict__ t, int n,
                                float scale, float* __restrict__ dy, float* __restrict__ loss) {
  __shared__ float red[256];
  float s = 0.f;
  for (int i = threadIdx.x; i < n; i += 256) {
    const float d = y[i] - t[i];
    dy[i] = 2.f * d * scale;
    s += d * d;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0 && loss) *loss = red[0] * scale;
}

// One Adam step.  The coefficients come from the host, formed in double from
// the double hyperparameters (1 - beta2 in float would lose five digits).
__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g,
                            float* __restrict__ m, float* __restrict__ v, long n, float lr,
                            float b1, float omb1, float b2, float omb2, float eps, float inv_c1,
                            float inv_c2) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + omb1 * gi;
  const float vi = b2 * v[i] + omb2 * (gi * gi);
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * inv_c1) / (sqrtf(vi * inv_c2) + eps);
}

__global__ void scatter_cols_kernel(const float* __restrict__ src, int N, int K, int seg0,
                                    int len0, int seg1, float* __restrict__ dst, int ldd) {
  // dst[n][col(k)] = src[n][k] for the compact-to-full column map
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)N * K) return;
  const int n = (int)(i / K), k = (int)(i - (long)n * K);
  const int col = k < len0 ? seg0 + k : seg1 + (k - len0);
  dst[(size_t)n * ldd + col] = src[i];
}

__global__ void gather_cols_kernel(const float* __restrict__ W, int N, int K, int seg0, int len0,
                                   int seg1, int ldw, float* __restrict__ dst) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)N * K) return;
  const int n = (int)(i / K), k = (int)(i - (long)n * K);
  const int col = k < len0 ? seg0 + k : seg1 + (k - len0);
  dst[i] = W[(size_t)n * ldw + col];
}

struct Layout {
  size_t w1, b1, w2, b2, w3, b3, total;
};

Layout params_layout(const synim_mlp& net) {
  Layout L{};
  L.w1 = 0;
  L.b1 = L.w1 + (size_t)net.h1 * net.n_in;
  L.w2 = L.b1 + net.h1;
  L.b2 = L.w2 + (size_t)net.h2 * net.h1;
  L.w3 = L.b2 + net.h2;
  L.b3 = L.w3 + (size_t)net.n_out * net.h2;
  L.total = L.b3 + net.n_out;
  return L;
}

int check_net(const synim_mlp* net) {
  if (!net) return SYNIM_E_NULL;
  if (net->n_in < 1 || net->h1 < 1 || net->h2 < 1 || net->n_out < 1) return SYNIM_E_SHAPE;
  if (net->len0 < 0 || net->len1 < 0 || net->len0 + net->len1 < 1) return SYNIM_E_SHAPE;
  if (net->seg0 < 0 || net->seg0 + net->len0 > net->n_in || net->seg1 < 0 ||
      net->seg1 + net->len1 > net->n_in)
    return SYNIM_E_SHAPE;
  if (net->len0 > 0 && net->len1 > 0 && net->seg0 + net->len0 > net->seg1 &&
      net->seg1 + net->len1 > net->seg0)
    return SYNIM_E_SHAPE;   // overlapping segments
  return SYNIM_OK;
}

// Caller's scratch (floats): h1 [B][h1], h2 [B][h2] kept from the forward pass
// for the backward pass, then dy [B][n_out], dh2 [B][h2], dh1 [B][h1], the
// used W1 columns (forward) or their gradient (backward) [h1][K], and the
// split-K partial products of the largest product of either pass.
struct Scratch {
  float *h1, *h2, *dy, *dh2, *dh1, *w1c, *part;
  size_t total;
};

long part_floats(const synim_mlp& net, int B) {
  const int K = net.len0 + net.len1;
  const int shapes[8][3] = {{B, net.h1, K},         {B, net.h2, net.h1},    {B, net.n_out, net.h2},
                            {net.n_out, net.h2, B}, {B, net.h2, net.n_out}, {net.h2, net.h1, B},
                            {B, net.h1, net.h2},    {net.h1, K, B}};
  long m = 0;
  for (const auto& sh : shapes) m = std::max(m, gemm_part_floats(sh[0], sh[1], sh[2]));
  return m;
}

Scratch scratch_layout(const synim_mlp& net, int B, float* base) {
  const size_t K = (size_t)net.len0 + net.len1;
  Scratch S{};
  size_t off = 0;
  auto take = [&](size_t n) {
    float* p = base ? base + off : nullptr;
    off += n;
    return p;
  };
  S.h1 = take((size_t)B * net.h1);
  S.h2 = take((size_t)B * net.h2);
  S.dy = take((size_t)B * net.n_out);
  S.dh2 = take((size_t)B * net.h2);
  S.dh1 = take((size_t)B * net.h1);
  S.w1c = take((size_t)net.h1 * K);
  S.part = take((size_t)part_floats(net, B));
  S.total = off;
  return S;
}

// y [B][N] = h W^T + bias for the few outputs of the last layer: one wave per row.
constexpr int OUT_MAX = 8;
__global__ __launch_bounds__(256) void out_layer_kernel(const float* __restrict__ h, int B, int K,
                                                        const float* __restrict__ W, int N,
                                                        const float* __restrict__ bias,
                                                        float* __restrict__ y) {
  const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (b >= B) return;
  float acc[OUT_MAX];
#pragma unroll
  for (int j = 0; j < OUT_MAX; ++j) acc[j] = 0.f;
  for (int k = 4 * lane; k < K; k += 256) {   // K % 4 == 0
    const float4 v = *reinterpret_cast<const float4*>(h + (size_t)b * K + k);
#pragma unroll
    for (int j = 0; j < OUT_MAX; ++j)
      if (j < N) {
        const float4 w = *reinterpret_cast<const float4*>(W + (size_t)j * K + k);
        acc[j] = __fmaf_rn(v.x, w.x, acc[j]);
        acc[j] = __fmaf_rn(v.y, w.y, acc[j]);
        acc[j] = __fmaf_rn(v.z, w.z, acc[j]);
        acc[j] = __fmaf_rn(v.w, w.w, acc[j]);
      }
  }
#pragma unroll
  for (int j = 0; j < OUT_MAX; ++j) {
    if (j >= N) break;
    float v = acc[j];
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane == 0) y[(size_t)b * N + j] = v + bias[j];
  }
}

// Everything of the last layer's backward pass and the loss in one launch (its
// products are too small for a launch each): dY = 2 (Y - T) / (B n_out),
//   workgroups [0, n_w):  dW3 [N][K] = dY^T h for OUT_COLS columns of h each, the
//                         rows split over OUT_PARTS thread groups added in order;
//   workgroup n_w:        db3 = sum dY and the loss;
//   the others:           dh [B][K] = dY W3 where h > 0, a row each.
constexpr int OUT_COLS = 16, OUT_PARTS = 256 / OUT_COLS, OUT_CHUNK = 512;
__global__ __launch_bounds__(256) void out_backward_kernel(
    const float* __restrict__ y, const float* __restrict__ t, const float* __restrict__ h, int B,
    int K, const float* __restrict__ W, int N, float scale, int n_w, float* __restrict__ dW,
    float* __restrict__ db, float* __restrict__ dh, float* __restrict__ loss) {
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < n_w) {
    __shared__ float dy[OUT_CHUNK * OUT_MAX];
    __shared__ float red[OUT_PARTS][OUT_COLS][OUT_MAX];
    const int c = tid % OUT_COLS, part = tid / OUT_COLS;
    const int k = min((int)blockIdx.x * OUT_COLS + c, K - 1);
    float acc[OUT_MAX];
#pragma unroll
    for (int j = 0; j < OUT_MAX; ++j) acc[j] = 0.f;
    for (int b0 = 0; b0 < B; b0 += OUT_CHUNK) {
      const int nb = min(OUT_CHUNK, B - b0);
      __syncthreads();
      for (int e = tid; e < nb * N; e += 256)
        dy[e] = 2.f * (y[(size_t)b0 * N + e] - t[(size_t)b0 * N + e]) * scale;
      __syncthreads();
      // eight rows' loads in flight per thread
      for (int r0 = part; r0 < nb; r0 += 8 * OUT_PARTS) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          v[u] = r0 + OUT_PARTS * u < nb ? h[(size_t)(b0 + r0 + OUT_PARTS * u) * K + k] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (r0 + OUT_PARTS * u >= nb) break;
#pragma unroll
          for (int j = 0; j < OUT_MAX; ++j)
            if (j < N) acc[j] = __fmaf_rn(dy[(r0 + OUT_PARTS * u) * N + j], v[u], acc[j]);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < OUT_MAX; ++j) red[part][c][j] = acc[j];
    __syncthreads();
    if (part < N && (int)blockIdx.x * OUT_COLS + c < K) {
      float v = 0.f;
      for (int q = 0; q < OUT_PARTS; ++q) v += red[q][c][part];
      dW[(size_t)part * K + k] = v;
    }
    return;
  }
  if ((int)blockIdx.x == n_w) {
    // thread (row group, output): rows in order, groups in a fixed tree
    __shared__ float rd[256], rq[256];
    const int ng = 256 / N, j = tid % N, q = tid / N;
    float sd = 0.f, sq = 0.f;
    if (q < ng)
      for (int b = q; b < B; b += ng) {
        const float d = y[(size_t)b * N + j] - t[(size_t)b * N + j];
        sd += 2.f * d * scale;
        sq += d * d;
      }
    rd[tid] = sd;
    rq[tid] = sq;
    __syncthreads();
    for (int half = 1; half < ng; half *= 2) {
      if (q < ng && q % (2 * half) == 0 && q + half < ng) {
        rd[tid] += rd[tid + half * N];
        rq[tid] += rq[tid + half * N];
      }
      __syncthreads();
    }
    if (tid < N) db[tid] = rd[tid];
    if (tid == 0 && loss) {
      float v = 0.f;
      for (int o = 0; o < N; ++o) v += rq[o];
      *loss = v * scale;
    }
    return;
  }
  const size_t b = blockIdx.x - n_w - 1;
  float d[OUT_MAX];
#pragma unroll
  for (int j = 0; j < OUT_MAX; ++j)
    d[j] = j < N ? 2.f * (y[b * N + j] - t[b * N + j]) * scale : 0.f;
  for (int k = tid; k < K; k += 256) {
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < OUT_MAX; ++j)
      if (j < N) v = __fmaf_rn(d[j], W[(size_t)j * K + k], v);
    dh[b * K + k] = h[b * K + k] > 0.f ? v : 0.f;
  }
}

// The direct products need 16-byte loads of every operand: layer widths and
// segments in whole float4, aligned arrays, few outputs.  (Other shapes take
// the staged products, with the input layer's columns gathered.)
bool direct_ok(const synim_mlp& net, const float* params, const float* x, const Scratch& S) {
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  return net.n_out <= OUT_MAX && net.h1 % 4 == 0 && net.h2 % 4 == 0 && net.n_in % 4 == 0 &&
         net.len0 % 4 == 0 && net.len1 % 4 == 0 && net.seg0 % 4 == 0 && net.seg1 % 4 == 0 &&
         net.seg1 >= net.seg0 + net.len0 && net.h1 >= 4 && net.h2 >= 4 && al(params) && al(x) &&
         al(S.h1) && al(S.h2) && al(S.dh1) && al(S.dh2);
}

template <int BM, int BN, bool AK, bool BK>
int direct_launch(const DGemm& g, hipStream_t st) {
  const int tiles = direct_tiles(g.M, g.N, BM, BN);
  const int zero = g.zero_cols > 0 ? ((g.M + ZERO_ROWS - 1) / ZERO_ROWS + 7) / 8 * 8 : 0;
  const int W = direct_waves(tiles, g.K, BM * BN >= 4 ? 4 : 8);   // at most 64 KB of LDS
  hipLaunchKernelGGL((direct_kernel<BM, BN, AK, BK, BM, BN, AK, BK>), dim3(tiles + zero),
                     dim3(64 * W), direct_lds(W, BM, BN, AK, BK), st, zero, g, tiles, g, 0);
  SYNIM_HIP_TRY(hipGetLastError());
  return SYNIM_OK;
}

// 32 x 32 tiles once they alone give every CU one, else 16 x 32.  (64 x 64 tiles
// halve the loads, but dW1 of the estimator, 264 of them, took 19 us against 16:
// with one workgroup per CU nothing hides their latency.)
template <bool AK, bool BK>
int direct_product(const DGemm& g, hipStream_t st) {
  if (direct_tiles(g.M, g.N, 2, 2) >= 256) return direct_launch<2, 2, AK, BK>(g, st);
  return direct_launch<1, 2, AK, BK>(g, st);
}

DGemm dgemm(int M, int N, int K, const float* X, long ldx, const float* Y, long ldy, float* C,
            long ldc) {
  DGemm g{};
  g.M = M;
  g.N = N;
  g.K = K;
  g.X = X;
  g.ldx = ldx;
  g.Y = Y;
  g.ldy = ldy;
  g.C = C;
  g.ldc = ldc;
  g.len0 = INT_MAX;
  return g;
}

int forward_direct(const synim_mlp& net, const Layout& L, const float* P, const float* x, int B,
                   const Scratch& S, float* y, hipStream_t st) {
  const int K = net.len0 + net.len1;
  // input layer on W1's own columns: compact k feeds column seg0 + k, from
  // len0 on column seg1 + k - len0
  DGemm g = dgemm(B, net.h1, K, x, K, P + L.w1 + net.seg0, net.n_in, S.h1, net.h1);
  g.len0 = net.len0;
  g.shift = net.seg1 - net.seg0 - net.len0;
  g.bias = P + L.b1;
  g.relu = 1;
  int rc = direct_product<true, true>(g, st);
  if (rc != SYNIM_OK) return rc;
  DGemm h = dgemm(B, net.h2, net.h1, S.h1, net.h1, P + L.w2, net.h1, S.h2, net.h2);
  h.bias = P + L.b2;
  h.relu = 1;
  if ((rc = direct_product<true, true>(h, st)) != SYNIM_OK) return rc;
  hipLaunchKernelGGL(out_layer_kernel, dim3((B + 3) / 4), dim3(256), 0, st, S.h2, B, net.h2,
                     P + L.w3, net.n_out, P + L.b3, y);
  SYNIM_HIP_TRY(hipGetLastError());
  return SYNIM_OK;
}

int backward_direct(const synim_mlp& net, const Layout& L, const float* P, const float* x, int B,
                    const Scratch& S, const float* y, const float* t, float* G, float* loss,
                    hipStream_t st) {
  const int K = net.len0 + net.len1;
  const int n_w = (net.h2 + OUT_COLS - 1) / OUT_COLS;
  hipLaunchKernelGGL(out_backward_kernel, dim3(n_w + 1 + B), dim3(256), 0,
                     st, y, t, S.h2, B, net.h2, P + L.w3, net.n_out, 1.f / (B * net.n_out), n_w,
                     G + L.w3, G + L.b3, S.dh2, loss);
  SYNIM_HIP_TRY(hipGetLastError());
  // layer 2: dW2 = dh2^T h1 with db2, and dh1 = dh2 W2 where h1 > 0, in one launch
  DGemm w2 = dgemm(net.h2, net.h1, B, S.dh2, net.h2, S.h1, net.h1, G + L.w2, net.h1);
  w2.rowsum = G + L.b2;
  DGemm d1 = dgemm(B, net.h1, net.h2, S.dh2, net.h2, P + L.w2, net.h1, S.dh1, net.h1);
  d1.mask = S.h1;
  const int tw = direct_tiles(w2.M, w2.N, 2, 2), td = direct_tiles(d1.M, d1.N, 2, 2);
  const int W = direct_waves(tw + td, std::min(B, net.h2), 8);
  hipLaunchKernelGGL((direct_kernel<2, 2, false, false, 2, 2, true, false>), dim3(tw + td),
                     dim3(64 * W),
                     std::max(direct_lds(W, 2, 2, false, false), direct_lds(W, 2, 2, true, false)),
                     st, 0, w2, tw, d1, td);
  SYNIM_HIP_TRY(hipGetLastError());
  // layer 1: dW1 = dh1^T x into the used columns, zero elsewhere, db1
  DGemm w1 = dgemm(net.h1, K, B, S.dh1, net.h1, x, K, G + L.w1 + net.seg0, net.n_in);
  w1.rowsum = G + L.b1;
  w1.len0 = net.len0;
  w1.shift = net.seg1 - net.seg0 - net.len0;
  w1.zero_cols = net.n_in;
  w1.col0 = net.seg0;
  return direct_product<false, false>(w1, st);
}

__global__ void fill_zero_kernel(float* __restrict__ p, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

}  // namespace
}  // namespace synim

using namespace synim;

extern "C" size_t synim_mlp_param_count(const synim_mlp* net) {
  if (check_net(net) != SYNIM_OK) return 0;
  return params_layout(*net).total;
}

extern "C" size_t synim_mlp_scratch_floats(const synim_mlp* net, int B) {
  if (check_net(net) != SYNIM_OK || B < 1) return 0;
  return scratch_layout(*net, B, nullptr).total;
}

// Forward pass.  scratch: synim_mlp_scratch_floats floats; y: [B][n_out].
extern "C" int synim_mlp_forward(const synim_mlp* net, const float* params, const float* x, int B,
                                 float* scratch, float* y, void* stream) {
  int rc = check_net(net);
  if (rc != SYNIM_OK) return rc;
  if (!params || !x || !scratch || !y) return SYNIM_E_NULL;
  if (B < 1) return SYNIM_E_SHAPE;
  hipStream_t st = (hipStream_t)stream;
  const Layout L = params_layout(*net);
  const int K = net->len0 + net->len1;
  const Scratch S = scratch_layout(*net, B, scratch);
  float* h1 = S.h1;
  float* h2 = S.h2;
  const float* P = params;
  if (B <= 16) {
    hipLaunchKernelGGL(linear_small_kernel<16>, dim3(net->h1), dim3(256), 0, st, B, net->h1, K,
                       x, K, P + L.w1, net->n_in, net->seg0, net->len0, net->seg1, P + L.b1, 1,
                       h1, net->h1);
    SYNIM_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(linear_small_kernel<16>, dim3(net->h2), dim3(256), 0, st, B, net->h2,
                       net->h1, h1, net->h1, P + L.w2, net->h1, 0, net->h1, 0, P + L.b2, 1, h2,
                       net->h2);
    SYNIM_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(linear_small_kernel<16>, dim3(net->n_out), dim3(256), 0, st, B,
                       net->n_out, net->h2, h2, net->h2, P + L.w3, net->h2, 0, net->h2, 0,
                       P + L.b3, 0, y, net->n_out);
    SYNIM_HIP_TRY(hipGetLastError());
    return SYNIM_OK;
  }
  if (direct_ok(*net, params, x, S)) return forward_direct(*net, L, P, x, B, S, y, st);
  // input layer: gather the used W1 columns once, then a dense GEMM
  float* w1c = S.w1c;
  const long nk = (long)net->h1 * K;
  hipLaunchKernelGGL(gather_cols_kernel, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, st,
                     P + L.w1, net->h1, K, net->seg0, net->len0, net->seg1, net->n_in, w1c);
  SYNIM_HIP_TRY(hipGetLastError());
  rc = gemm<false, true>(B, net->h1, K, 1.f, x, K, w1c, K, 0.f, h1, net->h1, P + L.b1, 1, S.part, st);
  if (rc != SYNIM_OK) return rc;
  rc = gemm<false, true>(B, net->h2, net->h1, 1.f, h1, net->h1, P + L.w2, net->h1, 0.f, h2,
                         net->h2, P + L.b2, 1, S.part, st);
  if (rc != SYNIM_OK) return rc;
  return gemm<false, true>(B, net->n_out, net->h2, 1.f, h2, net->h2, P + L.w3, net->h2, 0.f, y,
                           net->n_out, P + L.b3, 0, S.part, st);
}

// Backward pass of the MSE loss after synim_mlp_forward on the same x and
// scratch: grads (packed like params, fully overwritten; W1 columns outside
// the segments get 0), loss (device float, nullable) = mean((y - t)^2).
extern "C" int synim_mlp_backward(const synim_mlp* net, const float* params, const float* x,
                                  int B, float* scratch, const float* y, const float* t,
                                  float* grads, float* loss, void* stream) {
  int rc = check_net(net);
  if (rc != SYNIM_OK) return rc;
  if (!params || !x || !scratch || !y || !t || !grads) return SYNIM_E_NULL;
  if (B < 1) return SYNIM_E_SHAPE;
  hipStream_t st = (hipStream_t)stream;
  const Layout L = params_layout(*net);
  const int K = net->len0 + net->len1;
  const Scratch S = scratch_layout(*net, B, scratch);
  float* h1 = S.h1;
  float* h2 = S.h2;
  float* dy = S.dy;
  float* dh2 = S.dh2;
  float* dh1 = S.dh1;
  float* dw1c = S.w1c;   // [h1][K] before scattering into W1's columns
  const float* P = params;
  float* G = grads;
  if (B > 16 && direct_ok(*net, params, x, S) && (reinterpret_cast<uintptr_t>(grads) & 15) == 0)
    return backward_direct(*net, L, P, x, B, S, y, t, G, loss, st);
  const int ny = B * net->n_out;
  hipLaunchKernelGGL(mse_grad_kernel, dim3(1), dim3(256), 0, st, y, t, ny, 1.f / ny, dy, loss);
  SYNIM_HIP_TRY(hipGetLastError());
  // layer 3: dW3 = dy^T h2, db3 = sum dy, dh2 = dy W3 (masked by h2 > 0)
  rc = gemm<true, false>(net->n_out, net->h2, B, 1.f, dy, net->n_out, h2, net->h2, 0.f, G + L.w3,
                         net->h2, nullptr, 0, S.part, st);
  if (rc != SYNIM_OK) return rc;
  hipLaunchKernelGGL(colsum_kernel, dim3((net->n_out + CS_COLS - 1) / CS_COLS), dim3(256), 0, st, dy, B,
                     net->n_out, G + L.b3);
  SYNIM_HIP_TRY(hipGetLastError());
  rc = gemm<false, false>(B, net->h2, net->n_out, 1.f, dy, net->n_out, P + L.w3, net->h2, 0.f,
                          dh2, net->h2, nullptr, 0, S.part, st);
  if (rc != SYNIM_OK) return rc;
  const long n2 = (long)B * net->h2;
  hipLaunchKernelGGL(relu_mask_kernel, dim3((unsigned)((n2 + 255) / 256)), dim3(256), 0, st, dh2,
                     h2, n2);
  SYNIM_HIP_TRY(hipGetLastError());
  // layer 2
  rc = gemm<true, false>(net->h2, net->h1, B, 1.f, dh2, net->h2, h1, net->h1, 0.f, G + L.w2,
                         net->h1, nullptr, 0, S.part, st);
  if (rc != SYNIM_OK) return rc;
  hipLaunchKernelGGL(colsum_kernel, dim3((net->h2 + CS_COLS - 1) / CS_COLS), dim3(256), 0, st, dh2, B,
                     net->h2, G + L.b2);
  SYNIM_HIP_TRY(hipGetLastError());
  rc = gemm<false, false>(B, net->h1, net->h2, 1.f, dh2, net->h2, P + L.w2, net->h1, 0.f, dh1,
                          net->h1, nullptr, 0, S.part, st);
  if (rc != SYNIM_OK) return rc;
  const long n1 = (long)B * net->h1;
  hipLaunchKernelGGL(relu_mask_kernel, dim3((unsigned)((n1 + 255) / 256)), dim3(256), 0, st, dh1,
                     h1, n1);
  SYNIM_HIP_TRY(hipGetLastError());
  // layer 1: only the used columns of W1 get gradient, the rest is zero
  rc = gemm<true, false>(net->h1, K, B, 1.f, dh1, net->h1, x, K, 0.f, dw1c, K, nullptr, 0, S.part, st);
  if (rc != SYNIM_OK) return rc;
  const long nw1 = (long)net->h1 * net->n_in;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((nw1 + 255) / 256)), dim3(256), 0, st,
                     G + L.w1, nw1);
  SYNIM_HIP_TRY(hipGetLastError());
  const long nk = (long)net->h1 * K;
  hipLaunchKernelGGL(scatter_cols_kernel, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, st,
                     dw1c, net->h1, K, net->seg0, net->len0, net->seg1, G + L.w1, net->n_in);
  SYNIM_HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(colsum_kernel, dim3((net->h1 + CS_COLS - 1) / CS_COLS), dim3(256), 0, st, dh1, B,
                     net->h1, G + L.b1);
  SYNIM_HIP_TRY(hipGetLastError());
  return SYNIM_OK;
}

extern "C" int synim_adam_step(float* params, const float* grads, float* m, float* v, size_t n,
                               int step, double lr, double beta1, double beta2, double eps,
                               void* stream) {
  if (!params || !grads || !m || !v) return SYNIM_E_NULL;
  if (step < 1 || !(lr > 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) ||
      !(eps >= 0))
    return SYNIM_E_PARAM;
  if (n == 0) return SYNIM_OK;
  const double c1 = 1.0 - std::pow(beta1, (double)step);
  const double c2 = 1.0 - std::pow(beta2, (double)step);
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, params, grads, m, v, (long)n, (float)lr, (float)beta1,
                     (float)(1.0 - beta1), (float)beta2, (float)(1.0 - beta2), (float)eps,
                     (float)(1.0 / c1), (float)(1.0 / c2));
  SYNIM_HIP_TRY(hipGetLastError());
  return SYNIM_OK;
}
