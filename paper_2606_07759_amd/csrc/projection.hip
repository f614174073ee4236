// Tomographic projection P_opt = (P_DM^T P_DM + lambda I)^-1 P_DM^T P_Layer
// (paper Sec. 2.5): the projection matrices sampled on the device, their Gram
// and cross products by an FP64 MFMA GEMM, a blocked Cholesky factorisation
// and two blocked triangular solves, all in FP64.
//
// Storage: a projection matrix P (rows = (direction, pupil block), columns =
// basis functions) is kept transposed, Pt[col][row], so that every basis
// function's samples are contiguous (the sampler writes them coalesced) and
// the products are  G = Pt_dm Pt_dm^T  and  B = Pt_dm Pt_layer^T.
#include <algorithm>
#include <cfloat>
#include <climits>
#include <cmath>
#include <vector>

#include "common.hpp"

namespace synim {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ sampling
// Row (direction, block) of basis function a: the mean over the block's fine
// pupil pixels of the bilinear sample of the function at c + (r + h theta) / s
// (zero outside the component grid).
constexpr int PT = 128;        // columns of a product's tile (and of an occupancy row)
constexpr int PK = 16;         // matrix rows of a product's step (and of an occupancy bit)

struct SampleArgs {
  const float* basis;          // [n][H][W]
  int n, H, W;
  double h, s;                 // altitude (m), pixel (m)
  const double2* dirs;         // [n_dir] (theta_x, theta_y) radians
  int n_dir;
  const int2* blocks;          // [n_blocks] (by, bx)
  int n_blocks, bin;
  const uint8_t* pupil;        // [Hp][Wp]
  int Hp, Wp;
  double sp;                   // pupil pixel (m)
  double* Pt;                  // column base: Pt + col0 * ld
  long ld;
  long col0;                   // this component's first column in its matrix
  // per tile of PT columns, a bit for each PK matrix rows that hold a non-zero
  // sample (null: not wanted), words 64-bit words a tile; *wild is set where a
  // sample is not finite
  unsigned long long* occ;
  int words;
  int* wild;
  int group;                   // functions of a workgroup's loop
};

// The sample by its definition, pixel by pixel.
__device__ double proj_sample(const SampleArgs& g, long row, int a) {
  const int d = (int)(row / g.n_blocks), blk = (int)(row - (long)d * g.n_blocks);
  const int2 bb = g.blocks[blk];
  const double2 th = g.dirs[d];
  const double cy = (g.H - 1) * 0.5, cx = (g.W - 1) * 0.5;
  const double cpy = (g.Hp - 1) * 0.5, cpx = (g.Wp - 1) * 0.5;
  const float* F = g.basis + (size_t)a * g.H * g.W;
  double acc = 0.0;
  int cnt = 0;
  for (int fy = 0; fy < g.bin; ++fy)
    for (int fx = 0; fx < g.bin; ++fx) {
      const int y = bb.x * g.bin + fy, x = bb.y * g.bin + fx;
      if (!g.pupil[(size_t)y * g.Wp + x]) continue;
      const double gx = cx + ((x - cpx) * g.sp + g.h * th.x) / g.s;
      const double gy = cy + ((y - cpy) * g.sp + g.h * th.y) / g.s;
      const double fi = floor(gx), fj = floor(gy);
      const int i = (int)fi, j = (int)fj;
      const double u = gx - fi, v = gy - fj;
      auto tap = [&](int ii, int jj) -> double {
        return (ii >= 0 && ii < g.W && jj >= 0 && jj < g.H) ? (double)F[(size_t)jj * g.W + ii]
                                                            : 0.0;
      };
      acc += (1.0 - u) * (1.0 - v) * tap(i, j) + u * (1.0 - v) * tap(i + 1, j) +
             (1.0 - u) * v * tap(i, j + 1) + u * v * tap(i + 1, j + 1);
      ++cnt;
    }
  return cnt > 0 ? acc / cnt : 0.0;
}

// Marks the steps of PK rows in which a lane of the wave, whose first lane holds
// matrix row `row`, a multiple of 64, has a non-zero sample of column col (nz: the
// lanes that do).  LOOK: a word that has the bits already is left alone, where the
// waves of many functions mark the same rows: atomics on one address are served one
// after another.  (Without need the look costs its latency at each wave's end.)
template <bool LOOK>
__device__ __forceinline__ void mark_rows(const SampleArgs& g, long col, long row,
                                          unsigned long long nz) {
  unsigned long long m = 0;
#pragma unroll
  for (int q = 0; q < 64 / PK; ++q)
    if ((nz >> (q * PK)) & ((1ull << PK) - 1)) m |= 1ull << q;
  m <<= row / PK % 64;
  unsigned long long* word = g.occ + col / PT * g.words + row / (64 * PK);
  if (!LOOK || (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & m) != m)
    atomicOr(word, m);
}

// One thread per (row, basis function), for blocks whose taps span more than the
// largest window below.  (One mark a wave: with one a thread, 700 dense functions
// on blocks of 8 x 8 pixels took P_opt 34 ms, now 3.2.)
__global__ __launch_bounds__(256) void proj_sample_kernel(SampleArgs g) {
  const long row = (long)blockIdx.x * 256 + threadIdx.x;
  const int a = blockIdx.y;
  if (row >= (long)g.n_dir * g.n_blocks) return;
  const double out = proj_sample(g, row, a);
  g.Pt[(size_t)a * g.ld + row] = out;
  if (g.occ == nullptr) return;
  const unsigned long long nz = __ballot(out != 0.0);
  if (!(fabs(out) <= DBL_MAX)) *g.wild = 1;
  if ((threadIdx.x & 63) == 0) mark_rows<true>(g, g.col0 + a, row, nz);
}

// A row's sample is linear in the function, with weights that depend on the row
// alone: a thread forms its row's weights over the NT x NT grid points its taps
// span once, keeps them in registers and takes one small dot product per
// function of its group.  Read pixel by pixel a binned row took 64 taps of one
// float and, per pixel, two FP64 divisions, for every function again: 72 ms for
// 12278 functions of 512^2 on 94104 rows (4 x 4 pixels each), now 19; reading
// the functions once and writing the matrix takes 5.  Consecutive lanes are
// neighbouring blocks, whose window rows lie next to each other in memory.  The
// rows' workgroups of one group of functions run on one XCD, whose L2 then holds
// the functions for all directions.  Grid points of the window that are no
// tap carry weight zero; where a sample comes out not finite it is formed again
// by its definition, so that such a point's value never enters one.
template <int NT>
struct __attribute__((packed, aligned(4))) Window {   // NT neighbouring points
  float v[NT];
};
template <int NT>
__global__ __launch_bounds__(256) void proj_window_kernel(SampleArgs g, int n_rb, int by_xcd) {
  const int sb = by_xcd ? blockIdx.x >> 3 : blockIdx.x;
  const long grp = by_xcd ? (long)(sb / n_rb) * 8 + (blockIdx.x & 7) : sb / n_rb;
  const long row = (long)(sb % n_rb) * 256 + threadIdx.x;
  // the functions of this group: a whole number of groups per tile of columns
  const long c0 = g.col0 / g.group * g.group + grp * g.group;
  const int a_begin = (int)max(0L, c0 - g.col0);
  const int a_end = (int)min((long)g.n, c0 + g.group - g.col0);
  if (a_begin >= a_end) return;   // the whole workgroup
  const bool on = row < (long)g.n_dir * g.n_blocks;
  double w[NT][NT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < NT; ++i) w[j][i] = 0.0;
  int i0 = 0, j0 = 0;
  double mean = 0.0;
  if (on) {
    const int d = (int)(row / g.n_blocks), blk = (int)(row - (long)d * g.n_blocks);
    const int2 bb = g.blocks[blk];
    const double2 th = g.dirs[d];
    const double cy = (g.H - 1) * 0.5, cx = (g.W - 1) * 0.5;
    const double cpy = (g.Hp - 1) * 0.5, cpx = (g.Wp - 1) * 0.5;
    auto at_x = [&](int fx) { return cx + ((bb.y * g.bin + fx - cpx) * g.sp + g.h * th.x) / g.s; };
    auto at_y = [&](int fy) { return cy + ((bb.x * g.bin + fy - cpy) * g.sp + g.h * th.y) / g.s; };
    // the window's corner, moved inside the grid; cells outside the grid are
    // brought next to it, where they have no tap on it either
    auto cell = [](double f, int n) { return (int)fmin(fmax(f, -2.0), (double)n); };
    i0 = min(max(cell(floor(at_x(0)), g.W), 0), g.W - NT);
    j0 = min(max(cell(floor(at_y(0)), g.H), 0), g.H - NT);
    int cnt = 0;
    for (int fy = 0; fy < g.bin; ++fy) {
      double wx[NT];
#pragma unroll
      for (int i = 0; i < NT; ++i) wx[i] = 0.0;
      for (int fx = 0; fx < g.bin; ++fx) {
        if (!g.pupil[(size_t)(bb.x * g.bin + fy) * g.Wp + bb.y * g.bin + fx]) continue;
        const double gx = at_x(fx), fi = floor(gx), u = gx - fi;
        const int i = cell(fi, g.W) - i0;
#pragma unroll
        for (int k = 0; k < NT; ++k) wx[k] += k == i ? 1.0 - u : k == i + 1 ? u : 0.0;
        ++cnt;
      }
      const double gy = at_y(fy), fj = floor(gy), v = gy - fj;
      const int j = cell(fj, g.H) - j0;
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        const double wy = k == j ? 1.0 - v : k == j + 1 ? v : 0.0;
#pragma unroll
        for (int i = 0; i < NT; ++i) w[k][i] = __fma_rn(wy, wx[i], w[k][i]);
      }
    }
    mean = cnt > 0 ? 1.0 / cnt : 0.0;
  }
  const size_t plane = (size_t)g.H * g.W;
  const float* F = g.basis + (size_t)j0 * g.W + i0;
  bool nz = false, wild = false;
  for (int a = a_begin; a < a_end; ++a) {
    Window<NT> f[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
      f[j] = *reinterpret_cast<const Window<NT>*>(F + a * plane + (size_t)j * g.W);
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      double s = w[j][0] * (double)f[j].v[0];
#pragma unroll
      for (int i = 1; i < NT; ++i) s = __fma_rn(w[j][i], (double)f[j].v[i], s);
      acc += s;
    }
    acc *= mean;
    if (on) g.Pt[(size_t)a * g.ld + row] = acc;
    nz = nz || (on && acc != 0.0);
    wild = wild || (on && !(fabs(acc) <= DBL_MAX));
  }
  if (wild) {   // by the definition: such a point need not be a tap
    wild = false;
    nz = true;
    for (int a = a_begin; a < a_end; ++a) {
      double* at = g.Pt + (size_t)a * g.ld + row;
      if (fabs(*at) <= DBL_MAX) continue;
      *at = proj_sample(g, row, a);
      wild = wild || !(fabs(*at) <= DBL_MAX);
    }
  }
  if (g.occ == nullptr) return;
  const unsigned long long bits = __ballot(nz);
  if (wild) *g.wild = 1;
  if ((threadIdx.x & 63) == 0 && bits != 0) mark_rows<false>(g, g.col0 + a_begin, row, bits);
}

// ---------------------------------------------------------------- FP64 GEMM
// C[m][n] = alpha sum_k X(k, m) Y(k, n) + beta C[m][n], X(k, m) = X[k sxk + m sxm],
// Y(k, n) = Y[k syk + n syn], C row-major with ldc.  One workgroup of 256
// threads per 128 x 128 tile of C; each wave owns a 64 x 64 quarter as 4 x 4
// blocks of v_mfma_f64_16x16x4f64 (lane l feeds A[l%16][l/16] and B[l/16][l%16]
// and holds D[4r + l/16][l%16], r = 0..3).  K advances in chunks of 16 through two
// LDS buffers: the next chunk's global loads are in flight while the current one
// feeds the matrix cores, and a second workgroup of the CU covers the barriers and
// the pass over C.  An operand is read along its unit stride from one pointer a
// thread; XCD x takes the tile rows x, x + 8, ..., so that a row's operand stays
// in its L2.  lower: only tiles with some m >= n (a symmetric result's lower
// triangle) are computed.  An update of 7915 x 4107 over 256 columns: 0.62 ms
// with 256 x 128 tiles of one workgroup a CU, 0.52 with these tiles, now 0.43 with
// the addresses out of the loop and C read ahead.
constexpr int GK = 16, GPAD = 2;

struct GemmArgs {
  int M, N, K;
  const double* X;
  long sxk, sxm;
  const double* Y;
  long syk, syn;
  double* C;
  long ldc;
  double alpha, beta;
  int lower;
};

constexpr int GT = 128;          // tile side
constexpr int GQ = GK * GT / 256;   // elements of an operand chunk a thread moves

// One thread's share of an operand's chunks: elements q = 0.. GQ - 1 at rows
// k = k0 + kk + q dk and columns mm + q dm of the tile, read along the operand's
// unit stride.
struct GOperand {
  const double* p;   // element 0 of the next chunk
  long step, chunk;  // to the next element, to the next chunk
  int kk, mm, dk, dm, left;   // left: columns of the operand from the tile's first
  __device__ __forceinline__ GOperand(const double* base, long sk, long sm, int m0, int M, int tid) {
    if (sk == 1) {
      kk = tid % GK;
      mm = tid / GK;
      dk = 0;
      dm = 256 / GK;
    } else {
      kk = tid / GT;
      mm = tid % GT;
      dk = 256 / GT;
      dm = 0;
    }
    p = base + (long)kk * sk + (long)(m0 + mm) * sm;
    step = dk * sk + dm * sm;
    chunk = GK * sk;
    left = M - m0;
  }
  // rows: of the chunk that exist
  __device__ __forceinline__ void fetch(int rows, double (&r)[GQ]) {
#pragma unroll
    for (int q = 0; q < GQ; ++q)
      r[q] = kk + q * dk < rows && mm + q * dm < left ? p[q * step] : 0.0;
    p += chunk;
  }
  __device__ __forceinline__ void put(const double (&r)[GQ], double (*S)[GT + GPAD]) const {
#pragma unroll
    for (int q = 0; q < GQ; ++q) S[kk + q * dk][mm + q * dm] = r[q];
  }
};

// BETA: C is read (beta is not 0).  Without, a test for each element's read took 5.3 of
// the 20.2 us of 64 x 64 x 64.
template <bool BETA>
__global__ __launch_bounds__(256, 2) void gemm_f64_kernel(GemmArgs g, int nt) {
  const int row = (int)(blockIdx.x >> 3) / nt * 8 + (int)(blockIdx.x & 7);
  const int m0 = row * GT, n0 = (int)(blockIdx.x >> 3) % nt * GT;
  if (m0 >= g.M || (g.lower && m0 + GT - 1 < n0)) return;   // tile wholly above the diagonal
  __shared__ double Xs[2][GK][GT + GPAD], Ys[2][GK][GT + GPAD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  d4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  GOperand X(g.X, g.sxk, g.sxm, m0, g.M, tid), Y(g.Y, g.syk, g.syn, n0, g.N, tid);
  double rx[GQ], ry[GQ];
  X.fetch(g.K, rx);
  Y.fetch(g.K, ry);
  X.put(rx, Xs[0]);
  Y.put(ry, Ys[0]);
  __syncthreads();
  const int nk = (g.K + GK - 1) / GK;
  for (int c = 0; c < nk; ++c) {
    const int buf = c & 1;
    const bool more = c + 1 < nk;
    if (more) {
      X.fetch(g.K - (c + 1) * GK, rx);
      Y.fetch(g.K - (c + 1) * GK, ry);
    }
#pragma unroll
    for (int s = 0; s < GK / 4; ++s) {
      const int kr = 4 * s + (lane >> 4);
      double a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = Xs[buf][kr][wm + 16 * i + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Ys[buf][kr][wn + 16 * j + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (more) {
      // the other buffer was last read in iteration c - 1, before its closing barrier
      X.put(rx, Xs[buf ^ 1]);
      Y.put(ry, Ys[buf ^ 1]);
    }
    __syncthreads();
  }
  // (a block row's elements of C are all read before the first is written: one
  // by one, each read would wait for the write before it, which may be the same
  // memory for all the compiler knows)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    double* at[4];
    bool on[4][4];
    double old[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm + 16 * i + 4 * r + (lane >> 4);
      at[r] = g.C + (long)m * g.ldc + n0 + wn + (lane & 15);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = n0 + wn + 16 * j + (lane & 15);
        on[r][j] = m < g.M && n < g.N && (!g.lower || m >= n);
        if constexpr (BETA) old[r][j] = on[r][j] ? at[r][16 * j] : 0.0;
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (on[r][j])
          at[r][16 * j] = g.alpha * acc[i][j][r] + (BETA ? g.beta * old[r][j] : 0.0);
  }
}

int gemm(const GemmArgs& a, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) return SYNIM_OK;
  const long nt = (a.N + GT - 1) / GT, mt = ((a.M + GT - 1) / GT + 7) / 8 * 8;
  if (nt * mt > INT_MAX) return SYNIM_E_SHAPE;
  const auto kernel = a.beta != 0.0 ? gemm_f64_kernel<true> : gemm_f64_kernel<false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(nt * mt)), dim3(256), 0, st, a, (int)nt);
  SYNIM_HIP_TRY(hipGetLastError());
  return SYNIM_OK;
}

// ------------------------------------------------- products of sampled columns
// C = Pt_x Pt_y^T over the steps of PK rows in which both tiles of PT columns hold
// a non-zero sample: an influence function reaches a small part of the pupil
// (FP32 Gaussians 14 widths around the actuator, measured ones less), so that of
// the steps of a system of three mirrors and three layers 8% (Gram) and 12%
// (cross) are left.  A step of zeros adds exact zeros, so the sums are the same
// bits; where a sample is not finite (0 x inf) every step is taken.
// 128 x 128 tiles, 4 x 4 matrix-core blocks per wave, two workgroups a CU so that
// one's steps cover the other's loads and barriers.  Tiles differ in their number
// of steps: those with the most come first.  Where the tiles alone leave the chip
// idle each is split into `parts` of equally many steps, added in order after.
// The two products of 8171 x 94104 (lower half) and 8171 x 4107 x 94104: 180 and
// 149 ms dense in 256 x 128 tiles, now 12 and 15.  Functions that are non-zero
// everywhere have no step to skip: the whole of P_opt on that system takes 282 ms
// (489 with the dense products and solves in blocks of 64).
struct SkipArgs {
  int M, N, K;
  const double *X, *Y;         // X(k, m) = X[m ld + k], Y(k, n) = Y[n ld + k]
  long ld;
  double* C;
  long ldc;
  int lower;
  const unsigned long long *ox, *oy;   // occupancy of X's and Y's column tiles
  int words;
  const int* wild;
  const int* order;            // [tiles] (m tile << 16) | n tile
  int tiles, parts;
  double* part;                // [tiles][parts][PT][PT] (parts > 1)
};

// Steps both tiles share, one wave per tile of the mt x nt grid (-1 above the
// diagonal of a lower product).
__global__ __launch_bounds__(256) void skip_count_kernel(SkipArgs g, int mt, int nt,
                                                         int* __restrict__ count) {
  const int t = (int)((blockIdx.x * 256 + threadIdx.x) >> 6), lane = threadIdx.x & 63;
  if (t >= mt * nt) return;
  const int m = t / nt, n = t % nt;
  int c = 0;
  for (int w = lane; w < g.words; w += 64)
    c += __popcll(g.ox[(size_t)m * g.words + w] & g.oy[(size_t)n * g.words + w]);
  for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, 64);
  if (lane == 0) count[t] = g.lower && n > m ? -1 : c;
}

// The tiles in descending order of their steps (by 1024ths of the most there are).
__global__ __launch_bounds__(1024) void skip_order_kernel(const int* __restrict__ count, int total,
                                                          int nt, int most, int* __restrict__ order) {
  __shared__ int s_at[1024], s_sum[1024];
  const int tid = threadIdx.x;
  auto bucket = [&](int c) { return 1023 - (int)((long)c * 1023 / max(1, most)); };
  s_at[tid] = 0;
  __syncthreads();
  for (int t = tid; t < total; t += 1024)
    if (count[t] >= 0) atomicAdd(&s_at[bucket(count[t])], 1);
  __syncthreads();
  const int own = s_at[tid];
  s_sum[tid] = own;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int add = tid >= o ? s_sum[tid - o] : 0;
    __syncthreads();
    s_sum[tid] += add;
    __syncthreads();
  }
  s_at[tid] = s_sum[tid] - own;
  __syncthreads();
  for (int t = tid; t < total; t += 1024)
    if (count[t] >= 0) order[atomicAdd(&s_at[bucket(count[t])], 1)] = (t / nt) << 16 | (t % nt);
}

struct __attribute__((packed, aligned(8))) Two {   // rows k, k + 1 of a column
  double a, b;
};

__global__ __launch_bounds__(256, 2) void skip_gemm_kernel(SkipArgs g) {
  constexpr int LDT = PT + GPAD;
  __shared__ double Xs[2][PK][LDT], Ys[2][PK][LDT];
  extern __shared__ unsigned long long s_occ[];
  __shared__ int s_steps;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int item = blockIdx.x / g.parts, q = blockIdx.x % g.parts;
  const int mn = g.order[item];
  const int m0 = (mn >> 16) * PT, n0 = (mn & 0xffff) * PT;
  const int nk = (g.K + PK - 1) / PK;
  if (tid == 0) s_steps = 0;
  __syncthreads();
  const bool all = *g.wild != 0;
  int c = 0;
  for (int w = tid; w < g.words; w += 256) {
    const int left = nk - 64 * w;
    const unsigned long long v =
        all ? (left >= 64 ? ~0ull : (1ull << left) - 1)
            : g.ox[(size_t)(mn >> 16) * g.words + w] & g.oy[(size_t)(mn & 0xffff) * g.words + w];
    s_occ[w] = v;
    c += __popcll(v);
  }
  if (c != 0) atomicAdd(&s_steps, c);
  __syncthreads();
  // this part's steps: numbers [first, first + left) of the tile's
  const int steps = s_steps;
  const int first = (int)((long)steps * q / g.parts);
  int left = (int)((long)steps * (q + 1) / g.parts) - first;
  int word = -1;
  unsigned long long bits = 0;
  for (int before = 0; left > 0;) {
    bits = s_occ[++word];
    const int n = __popcll(bits);
    if (before + n > first) {
      for (int k = first - before; k > 0; --k) bits &= bits - 1;
      break;
    }
    before += n;
  }
  // row of the next step (left > 0)
  auto next = [&]() {
    while (bits == 0) bits = s_occ[++word];
    const int k = (64 * word + __ffsll(bits) - 1) * PK;
    bits &= bits - 1;
    --left;
    return __builtin_amdgcn_readfirstlane(k);
  };
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  d4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  // this thread's eight pairs of rows: rows 2 (tid % 8) and the next of columns
  // tid / 8 + 32 u
  const int kk = 2 * (tid & 7), mm = tid >> 3;
  Two rx[4], ry[4];
  auto fetch = [&](const double* P, int c0, int M, int k0, Two (&r)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int col = c0 + mm + 32 * u, k = k0 + kk;
      r[u] = Two{0.0, 0.0};
      if (col < M) {
        const double* at = P + (long)col * g.ld + k;
        if (k + 1 < g.K) r[u] = *reinterpret_cast<const Two*>(at);
        else if (k < g.K) r[u].a = *at;
      }
    }
  };
  auto put = [&](const Two (&r)[4], double (*S)[LDT]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      S[kk][mm + 32 * u] = r[u].a;
      S[kk + 1][mm + 32 * u] = r[u].b;
    }
  };
  bool more = left > 0;
  if (more) {
    const int k0 = next();
    fetch(g.X, m0, g.M, k0, rx);
    fetch(g.Y, n0, g.N, k0, ry);
  }
  for (int buf = 0; more; buf ^= 1) {
    put(rx, Xs[buf]);
    put(ry, Ys[buf]);
    __syncthreads();   // the other buffer has been read by everyone, too
    more = left > 0;
    if (more) {
      const int k0 = next();
      fetch(g.X, m0, g.M, k0, rx);
      fetch(g.Y, n0, g.N, k0, ry);
    }
#pragma unroll
    for (int s = 0; s < PK / 4; ++s) {
      const int kr = 4 * s + (lane >> 4);
      double a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = Xs[buf][kr][wm + 16 * i + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Ys[buf][kr][wn + 16 * j + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
  double* part = g.parts > 1 ? g.part + (size_t)blockIdx.x * PT * PT : nullptr;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = wm + 16 * i + 4 * r + (lane >> 4), n = wn + 16 * j + (lane & 15);
        if (part != nullptr)
          part[m * PT + n] = acc[i][j][r];
        else if (m0 + m < g.M && n0 + n < g.N && (!g.lower || m0 + m >= n0 + n))
          g.C[(long)(m0 + m) * g.ldc + n0 + n] = acc[i][j][r];
      }
}

// The parts of each tile added in order.
__global__ __launch_bounds__(256) void skip_reduce_kernel(SkipArgs g) {
  const int item = blockIdx.y, e = blockIdx.x * 256 + threadIdx.x;
  const int mn = g.order[item];
  const int m = (mn >> 16) * PT + e / PT, n = (mn & 0xffff) * PT + e % PT;
  if (m >= g.M || n >= g.N || (g.lower && m < n)) return;
  double s = 0.0;
  for (int q = 0; q < g.parts; ++q) s += g.part[((size_t)item * g.parts + q) * PT * PT + e];
  g.C[(long)m * g.ldc + n] = s;
}

// Column tiles of an M x N product, and the parts each is split into: one round of
// two workgroups a CU, parts of 16 steps or more.
long skip_tiles(long M, long N, bool lower) {
  const long mt = (M + PT - 1) / PT, nt = (N + PT - 1) / PT;
  return lower ? mt * (mt + 1) / 2 : mt * nt;
}
int skip_parts(long tiles, long rows) {
  return (int)std::clamp(std::min(512 / tiles, rows / PK / 16), 1L, 64L);
}
// Occupancy words a workgroup keeps beside its tiles, two workgroups in a CU's LDS
// (1.6 million rows).
constexpr int SKIP_WORDS = 1600;

int skip_gemm(SkipArgs g, int* count, hipStream_t st) {
  const int mt = (g.M + PT - 1) / PT, nt = (g.N + PT - 1) / PT;
  g.tiles = (int)skip_tiles(g.M, g.N, g.lower);
  g.parts = skip_parts(g.tiles, g.K);
  int* order = count + (long)mt * nt;
  g.order = order;
  hipLaunchKernelGGL(skip_count_kernel, dim3((unsigned)((mt * nt + 3) / 4)), dim3(256), 0, st, g,
                     mt, nt, count);
  SYNIM_HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(skip_order_kernel, dim3(1), dim3(1024), 0, st, count, mt * nt, nt,
                     (g.K + PK - 1) / PK, order);
  SYNIM_HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(skip_gemm_kernel, dim3((unsigned)(g.tiles * g.parts)), dim3(256),
                     g.words * sizeof(unsigned long long), st, g);
  SYNIM_HIP_TRY(hipGetLastError());
  if (g.parts > 1) {
    hipLaunchKernelGGL(skip_reduce_kernel, dim3(PT * PT / 256, (unsigned)g.tiles), dim3(256), 0, st,
                       g);
    SYNIM_HIP_TRY(hipGetLastError());
  }
  return SYNIM_OK;
}

__global__ void zero_words_kernel(unsigned long long* __restrict__ p, long n) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

__global__ void zero_status_kernel(int* s) {
  if (threadIdx.x < 16) s[threadIdx.x] = 0;
}

__global__ void add_diag_kernel(double* A, int n, long ld, double lam) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) A[(long)i * ld + i] += lam;
}

// ------------------------------------------------------------------ Cholesky
// Lower Cholesky of a symmetric positive definite matrix held (lower triangle)
// row-major, blocked by CB: factor the diagonal block in LDS, solve the panel
// below it, update the trailing lower triangle with the GEMM.
constexpr int CB = 64;

// One workgroup: the nb x nb diagonal block at (k, k), unblocked, in LDS.  A
// pivot that is not positive sets *status (the matrix is not positive
// definite) and the block is left as it is.
__global__ __launch_bounds__(256) void potrf_diag_kernel(double* A, long ld, int k, int nb,
                                                         int* status) {
  __shared__ double L[CB][CB + 1];
  __shared__ int bad;
  const int tid = threadIdx.x;
  if (tid == 0) bad = 0;
  for (int e = tid; e < nb * nb; e += 256) {
    const int i = e / nb, j = e % nb;
    L[i][j] = j <= i ? A[(long)(k + i) * ld + k + j] : 0.0;
  }
  __syncthreads();
  for (int j = 0; j < nb; ++j) {
    if (tid == 0) {
      const double d = L[j][j];
      if (!(d > 0.0)) bad = 1;
      L[j][j] = d > 0.0 ? sqrt(d) : 1.0;
    }
    __syncthreads();
    const double djj = L[j][j];
    for (int i = j + 1 + tid; i < nb; i += 256) L[i][j] /= djj;
    __syncthreads();
    // trailing update of the block's lower triangle
    const int rem = nb - j - 1;
    for (int e = tid; e < rem * rem; e += 256) {
      const int i = j + 1 + e / rem, c = j + 1 + e % rem;
      if (c <= i) L[i][c] -= L[i][j] * L[c][j];
    }
    __syncthreads();
  }
  for (int e = tid; e < nb * nb; e += 256) {
    const int i = e / nb, j = e % nb;
    if (j <= i) A[(long)(k + i) * ld + k + j] = L[i][j];
  }
  if (tid == 0 && bad) atomicOr(status, 1);
}

// Panel rows i in [r0, n): row i of block column k becomes x with
// x L_kk^T = a (forward substitution along the row).  One thread per row.
__global__ __launch_bounds__(256) void potrf_panel_kernel(double* A, long ld, int k, int nb,
                                                          int r0, int n) {
  __shared__ double L[CB][CB + 1];
  const int tid = threadIdx.x;
  for (int e = tid; e < nb * nb; e += 256) {
    const int i = e / nb, j = e % nb;
    L[i][j] = j <= i ? A[(long)(k + i) * ld + k + j] : 0.0;
  }
  __syncthreads();
  const int i = r0 + blockIdx.x * 256 + tid;
  if (i >= n) return;
  double* row = A + (long)i * ld + k;
  double x[CB];
#pragma unroll
  for (int j = 0; j < CB; ++j) x[j] = j < nb ? row[j] : 0.0;
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    if (j >= nb) break;
    double v = x[j];
    for (int c = 0; c < j; ++c) v -= x[c] * L[j][c];
    x[j] = v / L[j][j];
  }
#pragma unroll
  for (int j = 0; j < CB; ++j)
    if (j < nb) row[j] = x[j];
}

int potrf(double* A, int n, long ld, int* status, hipStream_t st) {
  for (int k = 0; k < n; k += CB) {
    const int nb = std::min(CB, n - k);
    hipLaunchKernelGGL(potrf_diag_kernel, dim3(1), dim3(256), 0, st, A, ld, k, nb, status);
    SYNIM_HIP_TRY(hipGetLastError());
    const int r0 = k + nb;
    if (r0 >= n) break;
    hipLaunchKernelGGL(potrf_panel_kernel, dim3((unsigned)((n - r0 + 255) / 256)), dim3(256), 0,
                       st, A, ld, k, nb, r0, n);
    SYNIM_HIP_TRY(hipGetLastError());
    // trailing lower triangle: A[r0:, r0:] -= P P^T, P = A[r0:, k:k+nb]
    GemmArgs g{};
    g.M = g.N = n - r0;
    g.K = nb;
    g.X = g.Y = A + (long)r0 * ld + k;
    g.sxk = g.syk = 1;
    g.sxm = g.syn = ld;
    g.C = A + (long)r0 * ld + r0;
    g.ldc = ld;
    g.alpha = -1.0;
    g.beta = 1.0;
    g.lower = 1;
    int rc = gemm(g, st);
    if (rc != SYNIM_OK) return rc;
  }
  return SYNIM_OK;
}

// ------------------------------------------------------- triangular solves
// B [n][m] (row-major, ldb) <- L_kk^-1 B[k:k+nb] (forward) or L_kk^-T B[k:k+nb]
// (backward) for the diagonal block at k; one thread per right-hand-side
// column, the block's rows sequential.
__global__ __launch_bounds__(256) void trsm_block_kernel(const double* L, long ld, int k, int nb,
                                                         double* B, long ldb, int m,
                                                         int backward) {
  __shared__ double T[CB][CB + 1];
  const int tid = threadIdx.x;
  for (int e = tid; e < nb * nb; e += 256) {
    const int i = e / nb, j = e % nb;
    T[i][j] = j <= i ? L[(long)(k + i) * ld + k + j] : 0.0;
  }
  __syncthreads();
  const int col = blockIdx.x * 256 + tid;
  if (col >= m) return;
  double x[CB];
#pragma unroll
  for (int r = 0; r < CB; ++r) x[r] = r < nb ? B[(long)(k + r) * ldb + col] : 0.0;
  if (!backward) {
    for (int r = 0; r < nb; ++r) {
      double v = x[r];
      for (int c = 0; c < r; ++c) v -= T[r][c] * x[c];
      x[r] = v / T[r][r];
    }
  } else {
    for (int r = nb - 1; r >= 0; --r) {
      double v = x[r];
      for (int c = r + 1; c < nb; ++c) v -= T[c][r] * x[c];
      x[r] = v / T[r][r];
    }
  }
#pragma unroll
  for (int r = 0; r < CB; ++r)
    if (r < nb) B[(long)(k + r) * ldb + col] = x[r];
}

int potrs(const double* L, int n, long ld, double* B, int m, long ldb, hipStream_t st) {
  const dim3 tg((unsigned)((m + 255) / 256));
  // forward: L Y = B, right-looking
  for (int k = 0; k < n; k += CB) {
    const int nb = std::min(CB, n - k);
    hipLaunchKernelGGL(trsm_block_kernel, tg, dim3(256), 0, st, L, ld, k, nb, B, ldb, m, 0);
    SYNIM_HIP_TRY(hipGetLastError());
    if (k + nb >= n) break;
    // B[k+nb:] -= L[k+nb:, k:k+nb] Y_k
    GemmArgs g{};
    g.M = n - k - nb;
    g.N = m;
    g.K = nb;
    g.X = L + (long)(k + nb) * ld + k;
    g.sxk = 1;
    g.sxm = ld;
    g.Y = B + (long)k * ldb;
    g.syk = ldb;
    g.syn = 1;
    g.C = B + (long)(k + nb) * ldb;
    g.ldc = ldb;
    g.alpha = -1.0;
    g.beta = 1.0;
    int rc = gemm(g, st);
    if (rc != SYNIM_OK) return rc;
  }
  // backward: L^T X = Y, from the last block
  const int last = ((n - 1) / CB) * CB;
  for (int k = last; k >= 0; k -= CB) {
    const int nb = std::min(CB, n - k);
    hipLaunchKernelGGL(trsm_block_kernel, tg, dim3(256), 0, st, L, ld, k, nb, B, ldb, m, 1);
    SYNIM_HIP_TRY(hipGetLastError());
    if (k == 0) break;
    // B[0:k] -= L[k:k+nb, 0:k]^T X_k
    GemmArgs g{};
    g.M = k;
    g.N = m;
    g.K = nb;
    g.X = L + (long)k * ld;
    g.sxk = ld;
    g.sxm = 1;
    g.Y = B + (long)k * ldb;
    g.syk = ldb;
    g.syn = 1;
    g.C = B;
    g.ldc = ldb;
    g.alpha = -1.0;
    g.beta = 1.0;
    int rc = gemm(g, st);
    if (rc != SYNIM_OK) return rc;
  }
  return SYNIM_OK;
}

// ------------------------------------- factorisation and solves in two levels
// Blocked Cholesky and solves with the diagonal blocks inverted, for a matrix of
// thousands of columns: blocks of CB within panels of CW columns.  Within a panel
// two launches a block: its diagonal block is brought up to date, factored and
// inverted by one workgroup, then each workgroup brings 64 rows below it up to
// date and multiplies them by L_kk^-T, in place.  The rest of the matrix is
// updated once per panel, so that it is read and written n / CW times and not
// n / CB (both bound by that traffic and by launches: blocks of 64 alone took 87 ms
// for n = 8171 and 4107 right-hand sides, 16 of them in the diagonal blocks, now
// 29).  Linv: ceil(n / CB) blocks of CB x CB doubles.
constexpr int CW = 4 * CB;
constexpr int CPAD = 2;
typedef double CBlock[CB][CB + CPAD];

// 16 elements a thread of a 64 x 64 block: rows r0 + 0..63 below row end, columns
// c0 + 0..63 below column end (else 0), to registers and from there to LDS.
__device__ __forceinline__ void block_fetch(const double* A, long ld, int r0, int rend, int c0,
                                            int cend, int tid, double (&v)[16]) {
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int r = (tid >> 6) + 4 * u, c = tid & 63;
    v[u] = r0 + r < rend && c0 + c < cend ? A[(long)(r0 + r) * ld + c0 + c] : 0.0;
  }
}
__device__ __forceinline__ void block_put(const double (&v)[16], int tid, CBlock& S) {
#pragma unroll
  for (int u = 0; u < 16; ++u) S[(tid >> 6) + 4 * u][tid & 63] = v[u];
}

// acc (16 rows of a wave, 4 blocks of 16 columns) += a X Y^T over 64 terms, X's
// rows from x0, Y's all.
__device__ __forceinline__ void mul_nt(const CBlock& X, int x0, const CBlock& Y, double a, int lane,
                                       d4 (&acc)[4]) {
#pragma unroll 4
  for (int s = 0; s < CB / 4; ++s) {
    const int k = 4 * s + (lane >> 4);
    const double x = a * X[x0 + (lane & 15)][k];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, Y[16 * j + (lane & 15)][k], acc[j], 0, 0, 0);
  }
}

// One 16 x 16 block of X Y (16 terms): X at (xr, xc), Y at (yr, yc).
__device__ __forceinline__ d4 mul16(const CBlock& X, int xr, int xc, const CBlock& Y, int yr, int yc,
                                    int lane, d4 acc) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = 4 * s + (lane >> 4);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[xr + (lane & 15)][xc + k],
                                               Y[yr + k][yc + (lane & 15)], acc, 0, 0, 0);
  }
  return acc;
}
__device__ __forceinline__ void put16(CBlock& S, int r, int c, int lane, const d4& v, double a) {
#pragma unroll
  for (int e = 0; e < 4; ++e) S[r + 4 * e + (lane >> 4)][c + (lane & 15)] = a * v[e];
}

__device__ __forceinline__ double from_lane(double v, int lane) {
  const unsigned long long b = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, lane);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), lane);
  return __longlong_as_double((unsigned long long)hi << 32 | lo);
}

// Diagonal block k of the panel from column K: brought up to date with the panel's
// columns before it, factored (written back) and inverted (to Linv, CB x CB, zero
// above the diagonal and outside nb x nb).  A pivot that is not positive sets
// *status and counts as 1.  One workgroup: the chain of 64 pivots is all latency,
// so it runs in 16 columns of one wave, lane i holding row i in registers (no
// barrier and no LDS between pivots), with the rest by matrix products (64
// columns with two barriers each and an inverse of one thread per column: 125 us,
// now 29).
__global__ __launch_bounds__(256) void panel_diag_kernel(double* A, long ld, int K, int k, int nb,
                                                         int* status, double* Linv) {
  __shared__ CBlock L, P, X;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double v[16];
  block_fetch(A, ld, k, k + nb, k, k + nb, tid, v);
  d4 acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = d4{0.0, 0.0, 0.0, 0.0};
  for (int c = K; c < k; c += CB) {
    double w[16];
    block_fetch(A, ld, k, k + nb, c, k, tid, w);
    __syncthreads();
    block_put(w, tid, P);
    __syncthreads();
    mul_nt(P, 16 * wave, P, -1.0, lane, acc);
  }
  block_put(v, tid, L);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = 16 * wave + 4 * e + (lane >> 4), c = 16 * j + (lane & 15);
      // (above the diagonal the matrix holds nothing; past nb the identity)
      const double d = r < nb && c <= r ? L[r][c] + acc[j][e] : r == c ? 1.0 : 0.0;
      L[r][c] = d;
      X[r][c] = 0.0;
    }
  __syncthreads();
  bool bad = false;
#pragma unroll 1
  for (int s = 0; s < 4; ++s) {
    const int c0 = 16 * s;
    if (wave == 0) {
      double a[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) a[j] = L[lane][c0 + j];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        double d = from_lane(a[j], c0 + j);
        if (!(d > 0.0)) {
          bad = true;
          d = 1.0;
        }
        d = sqrt(d);
        a[j] = lane == c0 + j ? d : a[j] / d;
#pragma unroll
        for (int q = j + 1; q < 16; ++q) a[q] = __fma_rn(-a[j], from_lane(a[j], c0 + q), a[q]);
      }
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (lane >= c0 + j) L[lane][c0 + j] = a[j];
    }
    __syncthreads();
    // the block's remaining columns, 16 rows a wave
    if (wave > s)
      for (int j = s + 1; j <= wave; ++j) {
        d4 t{};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int kk = c0 + 4 * q + (lane >> 4);
          t = __builtin_amdgcn_mfma_f64_16x16x4f64(L[16 * wave + (lane & 15)][kk],
                                                   L[16 * j + (lane & 15)][kk], t, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 16 * wave + 4 * e + (lane >> 4), c = 16 * j + (lane & 15);
          if (c <= r) L[r][c] -= t[e];
        }
      }
    __syncthreads();
  }
  if (wave == 0 && lane == 0 && bad) atomicOr(status, 1);
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int r = wave + 4 * u, c = lane;
    if (r < nb && c <= r) A[(long)(k + r) * ld + k + c] = L[r][c];
  }
  // inverse: the four diagonal 16 x 16 blocks, a wave each, lane c its column c ...
  {
    const int d0 = 16 * wave, c = lane & 15;
    double x[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = r == c ? 1.0 : 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      x[q] = x[q] / L[d0 + q][d0 + q];
#pragma unroll
      for (int r = q + 1; r < 16; ++r) x[r] = __fma_rn(-L[d0 + r][d0 + q], x[q], x[r]);
    }
    if (lane < 16)
#pragma unroll
      for (int r = 0; r < 16; ++r) X[d0 + r][d0 + c] = x[r];
  }
  __syncthreads();
  // ... then the blocks below them, by distance: X_ij = -X_ii sum_k L_ik X_kj
#pragma unroll 1
  for (int dist = 1; dist < 4; ++dist) {
    const int i = wave, j = wave - dist;
    if (j >= 0) {
      d4 t{};
      for (int q = j; q < i; ++q) t = mul16(L, 16 * i, 16 * q, X, 16 * q, 16 * j, lane, t);
      put16(P, 16 * i, 0, lane, t, 1.0);
      // (a wave reads back only what it wrote)
      __builtin_amdgcn_wave_barrier();
      d4 r{};
      r = mul16(X, 16 * i, 16 * i, P, 16 * i, 0, lane, r);
      put16(X, 16 * i, 16 * j, lane, r, -1.0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int r = wave + 4 * u, c = lane;
    Linv[r * CB + c] = r < nb && c < nb ? X[r][c] : 0.0;
  }
}

// Rows [r0, n) of block column k: brought up to date with the panel's columns [K, k),
// then multiplied by L_kk^-T; 64 rows a workgroup, in place.
__global__ __launch_bounds__(256) void panel_rows_kernel(double* A, long ld, int K, int k, int r0,
                                                         int n, const double* __restrict__ Linv) {
  __shared__ CBlock T, R, D;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i0 = r0 + blockIdx.x * CB;
  double v[16], w[16];
  block_fetch(Linv, CB, 0, CB, 0, CB, tid, v);
  d4 acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = i0 + 16 * wave + 4 * e + (lane >> 4);
      acc[j][e] = r < n ? A[(long)r * ld + k + 16 * j + (lane & 15)] : 0.0;
    }
  block_put(v, tid, T);
  for (int c = K; c < k; c += CB) {
    block_fetch(A, ld, i0, n, c, k, tid, v);
    block_fetch(A, ld, k, k + CB, c, k, tid, w);
    __syncthreads();
    block_put(v, tid, R);
    block_put(w, tid, D);
    __syncthreads();
    mul_nt(R, 16 * wave, D, -1.0, lane, acc);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) put16(R, 16 * wave, 16 * j, lane, acc[j], 1.0);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = d4{0.0, 0.0, 0.0, 0.0};
  mul_nt(R, 16 * wave, T, 1.0, lane, acc);
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = i0 + 16 * wave + 4 * e + (lane >> 4);
      if (r < n) A[(long)r * ld + k + 16 * j + (lane & 15)] = acc[j][e];
    }
}

int potrf_inv(double* A, int n, long ld, int* status, double* Linv, hipStream_t st) {
  for (int K = 0; K < n; K += CW) {
    const int K1 = std::min(n, K + CW);
    for (int k = K; k < K1; k += CB) {
      const int nb = std::min(CB, n - k), r0 = k + nb;
      double* Li = Linv + (long)(k / CB) * CB * CB;
      hipLaunchKernelGGL(panel_diag_kernel, dim3(1), dim3(256), 0, st, A, ld, K, k, nb, status, Li);
      SYNIM_HIP_TRY(hipGetLastError());
      if (r0 >= n) break;
      hipLaunchKernelGGL(panel_rows_kernel, dim3((unsigned)((n - r0 + CB - 1) / CB)), dim3(256), 0,
                         st, A, ld, K, k, r0, n, Li);
      SYNIM_HIP_TRY(hipGetLastError());
    }
    if (K1 >= n) break;
    // trailing lower triangle: A[K1:, K1:] -= P P^T, P = A[K1:, K:K1]
    GemmArgs g{};
    g.M = g.N = n - K1;
    g.K = K1 - K;
    g.X = g.Y = A + (long)K1 * ld + K;
    g.sxk = g.syk = 1;
    g.sxm = g.syn = ld;
    g.C = A + (long)K1 * ld + K1;
    g.ldc = ld;
    g.alpha = -1.0;
    g.beta = 1.0;
    g.lower = 1;
    const int rc = gemm(g, st);
    if (rc != SYNIM_OK) return rc;
  }
  return SYNIM_OK;
}

// Rows [K, K1) of B: solved against the panel's diagonal triangle, forward (L) or
// backward (L^T), SCOLS right-hand sides a workgroup, which keeps them in LDS over
// the panel's blocks.  The next 64 x 64 block of L or of an inverse is fetched
// while the current one feeds the matrix cores.
constexpr int SCOLS = 32;
template <bool BACK>
__global__ __launch_bounds__(256) void panel_solve_kernel(const double* __restrict__ L, long ld,
                                                          int K, int K1,
                                                          const double* __restrict__ Linv,
                                                          double* B, long ldb, int m) {
  __shared__ double Y[CW][SCOLS + 2];
  __shared__ CBlock S;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c0 = blockIdx.x * SCOLS;
  const int nblk = (K1 - K + CB - 1) / CB;
  for (int e = tid; e < CW * SCOLS; e += 256) {
    const int r = e / SCOLS, c = e % SCOLS;
    Y[r][c] = K + r < K1 && c0 + c < m ? B[(long)(K + r) * ldb + c0 + c] : 0.0;
  }
  // block t of the products of block s: L of the blocks solved before it, then the
  // inverse of its own
  auto fetch = [&](int s, int t, double (&v)[16]) {
    const int a = BACK ? nblk - 1 - s : s, b = BACK ? nblk - 1 - t : t;   // block rows of B
    if (t == s)
      block_fetch(Linv + (long)(K / CB + a) * CB * CB, CB, 0, CB, 0, CB, tid, v);
    else if (BACK)
      block_fetch(L, ld, K + b * CB, K1, K + a * CB, K1, tid, v);   // used transposed
    else
      block_fetch(L, ld, K + a * CB, K1, K + b * CB, K1, tid, v);
  };
  double v[16];
  fetch(0, 0, v);
  for (int s = 0; s < nblk; ++s) {
    const int a = BACK ? nblk - 1 - s : s;
    d4 acc[2];
    for (int t = 0; t <= s; ++t) {
      __syncthreads();   // the block before has been read (and Y written)
      block_put(v, tid, S);
      __syncthreads();
      if (t < s) fetch(s, t + 1, v);
      else if (s + 1 < nblk) fetch(s + 1, 0, v);
      const int y0 = (BACK ? nblk - 1 - t : t) * CB, o0 = a * CB + 16 * wave;
      if (t == 0 && s > 0) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[j][e] = Y[o0 + 4 * e + (lane >> 4)][16 * j + (lane & 15)];
      }
      if (t == s) {
        // the block's right-hand sides, brought up to date, back to LDS for the
        // product with the inverse (block 0's are there)
        if (s > 0) {
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              Y[o0 + 4 * e + (lane >> 4)][16 * j + (lane & 15)] = acc[j][e];
          __syncthreads();
        }
        acc[0] = acc[1] = d4{0.0, 0.0, 0.0, 0.0};
      }
      const double sign = t == s ? 1.0 : -1.0;
#pragma unroll 4
      for (int q = 0; q < CB / 4; ++q) {
        const int kk = 4 * q + (lane >> 4), r = 16 * wave + (lane & 15);
        const double x = sign * (BACK ? S[kk][r] : S[r][kk]);
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, Y[y0 + kk][16 * j + (lane & 15)], acc[j],
                                                        0, 0, 0);
      }
      if (t == s) {
        __syncthreads();   // every wave has read the right-hand sides
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            Y[o0 + 4 * e + (lane >> 4)][16 * j + (lane & 15)] = acc[j][e];
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < CW * SCOLS; e += 256) {
    const int r = e / SCOLS, c = e % SCOLS;
    if (K + r < K1 && c0 + c < m) B[(long)(K + r) * ldb + c0 + c] = Y[r][c];
  }
}

int potrs_inv(const double* L, int n, long ld, double* B, int m, long ldb, const double* Linv,
              hipStream_t st) {
  const dim3 sg((unsigned)((m + SCOLS - 1) / SCOLS));
  // forward: L Y = B, right-looking
  for (int K = 0; K < n; K += CW) {
    const int K1 = std::min(n, K + CW);
    hipLaunchKernelGGL(panel_solve_kernel<false>, sg, dim3(256), 0, st, L, ld, K, K1, Linv, B, ldb,
                       m);
    SYNIM_HIP_TRY(hipGetLastError());
    if (K1 >= n) break;
    // B[K1:] -= L[K1:, K:K1] Y_K
    GemmArgs g{};
    g.M = n - K1;
    g.N = m;
    g.K = K1 - K;
    g.X = L + (long)K1 * ld + K;
    g.sxk = 1;
    g.sxm = ld;
    g.Y = B + (long)K * ldb;
    g.syk = ldb;
    g.syn = 1;
    g.C = B + (long)K1 * ldb;
    g.ldc = ldb;
    g.alpha = -1.0;
    g.beta = 1.0;
    const int rc = gemm(g, st);
    if (rc != SYNIM_OK) return rc;
  }
  // backward: L^T X = Y, from the last panel
  for (int K = (n - 1) / CW * CW; K >= 0; K -= CW) {
    const int K1 = std::min(n, K + CW);
    hipLaunchKernelGGL(panel_solve_kernel<true>, sg, dim3(256), 0, st, L, ld, K, K1, Linv, B, ldb,
                       m);
    SYNIM_HIP_TRY(hipGetLastError());
    if (K == 0) break;
    // B[0:K] -= L[K:K1, 0:K]^T X_K
    GemmArgs g{};
    g.M = K;
    g.N = m;
    g.K = K1 - K;
    g.X = L + (long)K * ld;
    g.sxk = ld;
    g.sxm = 1;
    g.Y = B + (long)K * ldb;
    g.syk = ldb;
    g.syn = 1;
    g.C = B;
    g.ldc = ldb;
    g.alpha = -1.0;
    g.beta = 1.0;
    const int rc = gemm(g, st);
    if (rc != SYNIM_OK) return rc;
  }
  return SYNIM_OK;
}

// Kept b x b blocks of the pupil mask, row-major.
std::vector<int2> pupil_blocks(const uint8_t* pupil, int Hp, int Wp, int bin) {
  std::vector<int2> out;
  for (int by = 0; by < Hp / bin; ++by)
    for (int bx = 0; bx < Wp / bin; ++bx) {
      bool any = false;
      for (int y = by * bin; y < by * bin + bin && !any; ++y)
        for (int x = bx * bin; x < bx * bin + bin; ++x)
          if (pupil[(size_t)y * Wp + x]) {
            any = true;
            break;
          }
      if (any) out.push_back(make_int2(by, bx));
    }
  return out;
}

struct ProjLayout {
  size_t dirs, blocks, pupil, status, pt_dm, pt_l, gram, occ_dm, occ_l, count, part, total;
  int words;       // occupancy words per column tile (0: the products take every step)
};

ProjLayout proj_layout(int n_dir, int n_blocks, int Hp, int Wp, long rows, long n_dm, long n_l,
                       bool with_skip = true) {
  ProjLayout L{};
  size_t off = 0;
  auto take = [&](size_t n) {
    size_t at = off;
    off = align_up(off + n, 256);
    return at;
  };
  L.dirs = take((size_t)n_dir * sizeof(double2));
  L.blocks = take((size_t)n_blocks * sizeof(int2));
  L.pupil = take((size_t)Hp * Wp);
  L.status = take(16 * sizeof(int));
  L.pt_dm = take((size_t)n_dm * rows * sizeof(double));
  L.pt_l = take((size_t)n_l * rows * sizeof(double));
  L.gram = take((size_t)n_dm * n_dm * sizeof(double));
  // the products' occupancy, tile lists and split sums (a single matrix has none)
  const long mt = (n_dm + PT - 1) / PT, nt = (n_l + PT - 1) / PT, w = (rows + 64 * PK - 1) / (64 * PK);
  const bool skip = with_skip && n_dm > 0 && n_l > 0 && w <= SKIP_WORDS && mt < 0x8000 && nt < 0x10000 &&
                    mt * std::max(mt, nt) < INT_MAX / 64;
  L.words = skip ? (int)w : 0;
  L.occ_dm = take(skip ? mt * w * sizeof(unsigned long long) : 0);
  L.occ_l = take(skip ? nt * w * sizeof(unsigned long long) : 0);
  L.count = take(skip ? 2 * mt * std::max(mt, nt) * sizeof(int) : 0);
  size_t part = 0;
  if (skip)
    for (const bool lower : {true, false}) {
      const long tiles = skip_tiles(n_dm, lower ? n_dm : n_l, lower);
      const int parts = skip_parts(tiles, rows);
      if (parts > 1) part = std::max(part, (size_t)tiles * parts * PT * PT * sizeof(double));
    }
  L.part = take(part);
  L.total = off;
  return L;
}

int check_comps(const synim_proj_component* c, int n) {
  if (!c || n < 1) return SYNIM_E_NULL;
  for (int i = 0; i < n; ++i) {
    if (!c[i].basis) return SYNIM_E_NULL;
    if (c[i].n < 1 || c[i].H < 2 || c[i].W < 2) return SYNIM_E_SHAPE;
    if (!(c[i].pixel_m > 0.0)) return SYNIM_E_PARAM;
  }
  return SYNIM_OK;
}

long total_cols(const synim_proj_component* c, int n) {
  long t = 0;
  for (int i = 0; i < n; ++i) t += c[i].n;
  return t;
}

// Whether the directions and the pupil pixel are plain numbers (the window sampler
// takes no others).
bool plain_numbers(const double* dirs, int n_dir, double sp) {
  bool ok = std::isfinite(sp);
  for (int i = 0; i < 2 * n_dir; ++i) ok = ok && std::isfinite(dirs[i]);
  return ok;
}

// Samples every component into Pt (columns in component order) from the
// device tables at ws.
int sample_all(const synim_proj_component* comps, int n_comp, const double2* dirs_dev, int n_dir,
               const int2* blocks_dev, int n_blocks, int bin, const uint8_t* pupil_dev, int Hp,
               int Wp, double sp, double* Pt, long ld, unsigned long long* occ, int words, int* wild,
               bool plain, hipStream_t st) {
  long col = 0;
  const long rows = (long)n_dir * n_blocks;
  for (int c = 0; c < n_comp; ++c) {
    SampleArgs g{};
    g.basis = comps[c].basis;
    g.n = comps[c].n;
    g.H = comps[c].H;
    g.W = comps[c].W;
    g.h = comps[c].altitude_m;
    g.s = comps[c].pixel_m;
    g.dirs = dirs_dev;
    g.n_dir = n_dir;
    g.blocks = blocks_dev;
    g.n_blocks = n_blocks;
    g.bin = bin;
    g.pupil = pupil_dev;
    g.Hp = Hp;
    g.Wp = Wp;
    g.sp = sp;
    g.Pt = Pt + col * ld;
    g.ld = ld;
    g.col0 = col;
    g.occ = occ;
    g.words = words;
    g.wild = wild;
    // grid points a block's taps can span along a side
    const double span = (bin - 1) * sp / g.s;
    const int need = bin == 1 ? 2 : span < 8.0 ? (int)(span * (1 + 1e-9) + 1e-9) + 3 : 99;
    const int NT = (need + 1) / 2 * 2;
    if (NT <= 8 && NT <= std::min(g.H, g.W) && plain && std::isfinite(g.h) && std::isfinite(g.s)) {
      const int n_rb = (int)((rows + 255) / 256);
      // functions per workgroup: 64 spread the weights' cost best, fewer where that
      // would leave less than eight workgroups a CU
      g.group = 64;
      while (g.group > 8 && (long)n_rb * ((g.n + g.group - 1) / g.group) < 2048) g.group /= 2;
      long groups = (col + g.n - 1) / g.group - col / g.group + 1;
      const bool by_xcd = groups >= 8;
      if (by_xcd) groups = (groups + 7) / 8 * 8;
      if (groups * n_rb > INT_MAX) return SYNIM_E_SHAPE;
      const auto kernel = NT == 2   ? proj_window_kernel<2>
                          : NT == 4 ? proj_window_kernel<4>
                          : NT == 6 ? proj_window_kernel<6>
                                    : proj_window_kernel<8>;
      hipLaunchKernelGGL(kernel, dim3((unsigned)(groups * n_rb)), dim3(256), 0, st, g, n_rb,
                         by_xcd ? 1 : 0);
      SYNIM_HIP_TRY(hipGetLastError());
    } else {
      for (int a0 = 0; a0 < g.n; a0 += 65535) {
        SampleArgs gg = g;
        gg.basis = g.basis + (size_t)a0 * g.H * g.W;
        gg.Pt = g.Pt + (long)a0 * ld;
        gg.col0 = col + a0;
        gg.n = std::min(65535, g.n - a0);
        hipLaunchKernelGGL(proj_sample_kernel,
                           dim3((unsigned)((rows + 255) / 256), (unsigned)gg.n), dim3(256), 0, st,
                           gg);
        SYNIM_HIP_TRY(hipGetLastError());
      }
    }
    col += g.n;
  }
  return SYNIM_OK;
}

int proj_common(const synim_proj_component* dms, int n_dm, const double* dirs, int n_dir,
                const uint8_t* pupil, int Hp, int Wp, double sp, int bin) {
  if (!dirs || !pupil) return SYNIM_E_NULL;
  int rc = check_comps(dms, n_dm);
  if (rc != SYNIM_OK) return rc;
  if (n_dir < 1 || Hp < 1 || Wp < 1 || bin < 1 || Hp % bin || Wp % bin) return SYNIM_E_SHAPE;
  if (!(sp > 0.0)) return SYNIM_E_PARAM;
  return SYNIM_OK;
}

}  // namespace
}  // namespace synim

using namespace synim;

extern "C" int synim_proj_rows(const uint8_t* pupil, int Hp, int Wp, int bin, int n_dir,
                               int* n_rows) {
  if (!pupil || !n_rows) return SYNIM_E_NULL;
  if (n_dir < 1 || Hp < 1 || Wp < 1 || bin < 1 || Hp % bin || Wp % bin) return SYNIM_E_SHAPE;
  *n_rows = (int)(pupil_blocks(pupil, Hp, Wp, bin).size() * (size_t)n_dir);
  return SYNIM_OK;
}

extern "C" int synim_proj_workspace(const synim_proj_component* dms, int n_dm,
                                    const synim_proj_component* layers, int n_layer, int n_dir,
                                    const uint8_t* pupil, int Hp, int Wp, int bin,
                                    size_t* bytes) {
  if (!bytes || !pupil) return SYNIM_E_NULL;
  int rc = check_comps(dms, n_dm);
  if (rc != SYNIM_OK) return rc;
  if (layers && n_layer > 0 && (rc = check_comps(layers, n_layer)) != SYNIM_OK) return rc;
  if (n_dir < 1 || Hp < 1 || Wp < 1 || bin < 1 || Hp % bin || Wp % bin) return SYNIM_E_SHAPE;
  const int nb = (int)pupil_blocks(pupil, Hp, Wp, bin).size();
  const long rows = (long)nb * n_dir;
  const long ndm = total_cols(dms, n_dm), nl = layers ? total_cols(layers, n_layer) : 0;
  *bytes = proj_layout(n_dir, nb, Hp, Wp, rows, ndm, nl).total;
  return SYNIM_OK;
}

extern "C" int synim_proj_matrix(const synim_proj_component* comps, int n_comp,
                                 const double* dirs, int n_dir, const uint8_t* pupil, int Hp,
                                 int Wp, double pupil_pixel_m, int bin, double* Pt, long ld,
                                 void* ws, size_t ws_bytes, void* stream) {
  int rc = proj_common(comps, n_comp, dirs, n_dir, pupil, Hp, Wp, pupil_pixel_m, bin);
  if (rc != SYNIM_OK) return rc;
  if (!Pt || !ws) return SYNIM_E_NULL;
  hipStream_t st = (hipStream_t)stream;
  const std::vector<int2> blocks = pupil_blocks(pupil, Hp, Wp, bin);
  const long rows = (long)blocks.size() * n_dir;
  if (ld < rows) return SYNIM_E_SHAPE;
  const ProjLayout L = proj_layout(n_dir, (int)blocks.size(), Hp, Wp, rows, 0, 0);
  if (ws_bytes < L.total) return SYNIM_E_WORKSPACE;
  char* w = static_cast<char*>(ws);
  SYNIM_HIP_TRY(hipMemcpyAsync(w + L.dirs, dirs, (size_t)n_dir * sizeof(double2),
                               hipMemcpyHostToDevice, st));
  SYNIM_HIP_TRY(hipMemcpyAsync(w + L.blocks, blocks.data(), blocks.size() * sizeof(int2),
                               hipMemcpyHostToDevice, st));
  SYNIM_HIP_TRY(hipMemcpyAsync(w + L.pupil, pupil, (size_t)Hp * Wp, hipMemcpyHostToDevice, st));
  rc = sample_all(comps, n_comp, reinterpret_cast<const double2*>(w + L.dirs), n_dir,
                  reinterpret_cast<const int2*>(w + L.blocks), (int)blocks.size(), bin,
                  reinterpret_cast<const uint8_t*>(w + L.pupil), Hp, Wp, pupil_pixel_m, Pt, ld,
                  nullptr, 0, nullptr, plain_numbers(dirs, n_dir, pupil_pixel_m), st);
  if (rc != SYNIM_OK) return rc;
  // the host vectors must outlive the copies
  SYNIM_HIP_TRY(hipStreamSynchronize(st));
  return SYNIM_OK;
}

extern "C" int synim_gemm_f64(int M, int N, int K, double alpha, const double* X, long sxk,
                              long sxm, const double* Y, long syk, long syn, double beta,
                              double* C, long ldc, void* stream) {
  if (!C || (K > 0 && (!X || !Y))) return SYNIM_E_NULL;
  if (M < 0 || N < 0 || K < 0 || ldc < N) return SYNIM_E_SHAPE;
  if (K == 0) {
    if (beta == 1.0) return SYNIM_OK;
    // C = beta C: run the GEMM over an empty K (its epilogue scales C)
  }
  GemmArgs g{M, N, K, X, sxk, sxm, Y, syk, syn, C, ldc, alpha, beta, 0};
  return gemm(g, (hipStream_t)stream);
}

extern "C" int synim_potrf_f64(double* A, int n, long ld, int* status, void* stream) {
  if (!A || !status) return SYNIM_E_NULL;
  if (n < 1 || ld < n) return SYNIM_E_SHAPE;
  return potrf(A, n, ld, status, (hipStream_t)stream);
}

extern "C" int synim_potrs_f64(const double* L, int n, long ld, double* B, int m, long ldb,
                               void* stream) {
  if (!L || !B) return SYNIM_E_NULL;
  if (n < 1 || m < 1 || ld < n || ldb < m) return SYNIM_E_SHAPE;
  return potrs(L, n, ld, B, m, ldb, (hipStream_t)stream);
}

extern "C" int synim_proj_opt(const synim_proj_component* dms, int n_dm,
                              const synim_proj_component* layers, int n_layer, const double* dirs,
                              int n_dir, const uint8_t* pupil, int Hp, int Wp,
                              double pupil_pixel_m, int bin, double lambda, double* popt,
                              void* ws, size_t ws_bytes, void* stream) {
  int rc = proj_common(dms, n_dm, dirs, n_dir, pupil, Hp, Wp, pupil_pixel_m, bin);
  if (rc != SYNIM_OK) return rc;
  if ((rc = check_comps(layers, n_layer)) != SYNIM_OK) return rc;
  if (!popt || !ws) return SYNIM_E_NULL;
  if (!(lambda >= 0.0)) return SYNIM_E_PARAM;
  hipStream_t st = (hipStream_t)stream;
  const std::vector<int2> blocks = pupil_blocks(pupil, Hp, Wp, bin);
  const long rows = (long)blocks.size() * n_dir;
  const long ndm = total_cols(dms, n_dm), nl = total_cols(layers, n_layer);
  if (ndm > INT_MAX || nl > INT_MAX || rows > INT_MAX) return SYNIM_E_SHAPE;
  ProjLayout L = proj_layout(n_dir, (int)blocks.size(), Hp, Wp, rows, ndm, nl);
  // a workspace that holds the matrices alone is enough for the dense products
  if (ws_bytes < L.total)
    L = proj_layout(n_dir, (int)blocks.size(), Hp, Wp, rows, ndm, nl, false);
  if (ws_bytes < L.total) return SYNIM_E_WORKSPACE;
  char* w = static_cast<char*>(ws);
  SYNIM_HIP_TRY(hipMemcpyAsync(w + L.dirs, dirs, (size_t)n_dir * sizeof(double2),
                               hipMemcpyHostToDevice, st));
  SYNIM_HIP_TRY(hipMemcpyAsync(w + L.blocks, blocks.data(), blocks.size() * sizeof(int2),
                               hipMemcpyHostToDevice, st));
  SYNIM_HIP_TRY(hipMemcpyAsync(w + L.pupil, pupil, (size_t)Hp * Wp, hipMemcpyHostToDevice, st));
  hipLaunchKernelGGL(zero_status_kernel, dim3(1), dim3(64), 0, st,
                     reinterpret_cast<int*>(w + L.status));
  SYNIM_HIP_TRY(hipGetLastError());
  double* pt_dm = reinterpret_cast<double*>(w + L.pt_dm);
  double* pt_l = reinterpret_cast<double*>(w + L.pt_l);
  double* G = reinterpret_cast<double*>(w + L.gram);
  const auto* dirs_dev = reinterpret_cast<const double2*>(w + L.dirs);
  const auto* blocks_dev = reinterpret_cast<const int2*>(w + L.blocks);
  const auto* pupil_dev = reinterpret_cast<const uint8_t*>(w + L.pupil);
  int* status = reinterpret_cast<int*>(w + L.status);
  auto* occ_dm = reinterpret_cast<unsigned long long*>(w + L.occ_dm);
  auto* occ_l = reinterpret_cast<unsigned long long*>(w + L.occ_l);
  if (L.words > 0) {
    const long n = (long)(L.count - L.occ_dm) / 8;   // both occupancies
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       occ_dm, n);
    SYNIM_HIP_TRY(hipGetLastError());
  } else {
    occ_dm = occ_l = nullptr;
  }
  const bool plain = plain_numbers(dirs, n_dir, pupil_pixel_m);
  rc = sample_all(dms, n_dm, dirs_dev, n_dir, blocks_dev, (int)blocks.size(), bin, pupil_dev, Hp,
                  Wp, pupil_pixel_m, pt_dm, rows, occ_dm, L.words, status + 1, plain, st);
  if (rc == SYNIM_OK)
    rc = sample_all(layers, n_layer, dirs_dev, n_dir, blocks_dev, (int)blocks.size(), bin,
                    pupil_dev, Hp, Wp, pupil_pixel_m, pt_l, rows, occ_l, L.words, status + 1,
                    plain, st);
  if (rc != SYNIM_OK) return rc;
  // G = Pt_dm Pt_dm^T (lower triangle) + lambda I;  B = Pt_dm Pt_l^T into popt
  auto product = [&](const double* Y, const unsigned long long* oy, long N, double* C, long ldc,
                     int lower) {
    if (L.words == 0) {
      return gemm(GemmArgs{(int)ndm, (int)N, (int)rows, pt_dm, 1, rows, Y, 1, rows, C, ldc, 1.0, 0.0,
                           lower}, st);
    }
    SkipArgs g{};
    g.M = (int)ndm;
    g.N = (int)N;
    g.K = (int)rows;
    g.X = pt_dm;
    g.Y = Y;
    g.ld = rows;
    g.C = C;
    g.ldc = ldc;
    g.lower = lower;
    g.ox = occ_dm;
    g.oy = oy;
    g.words = L.words;
    g.wild = status + 1;
    g.part = reinterpret_cast<double*>(w + L.part);
    return skip_gemm(g, reinterpret_cast<int*>(w + L.count), st);
  };
  if ((rc = product(pt_dm, occ_dm, ndm, G, ndm, 1)) != SYNIM_OK) return rc;
  hipLaunchKernelGGL(add_diag_kernel, dim3((unsigned)((ndm + 255) / 256)), dim3(256), 0, st, G,
                     (int)ndm, ndm, lambda);
  SYNIM_HIP_TRY(hipGetLastError());
  if ((rc = product(pt_l, occ_l, nl, popt, nl, 0)) != SYNIM_OK) return rc;
  // the sampled matrices are spent: their memory holds the inverted diagonal
  // blocks (where they are too small, the substitution forms need no memory)
  double* linv = pt_dm;
  if ((size_t)((ndm + CB - 1) / CB) * CB * CB <= (size_t)rows * (size_t)ndm) {
    if ((rc = potrf_inv(G, (int)ndm, ndm, status, linv, st)) != SYNIM_OK) return rc;
    if ((rc = potrs_inv(G, (int)ndm, ndm, popt, (int)nl, nl, linv, st)) != SYNIM_OK) return rc;
  } else {
    if ((rc = potrf(G, (int)ndm, ndm, status, st)) != SYNIM_OK) return rc;
    if ((rc = potrs(G, (int)ndm, ndm, popt, (int)nl, nl, st)) != SYNIM_OK) return rc;
  }
  // the host vectors must outlive the copies
  SYNIM_HIP_TRY(hipStreamSynchronize(st));
  int host_status = 0;
  SYNIM_HIP_TRY(hipMemcpy(&host_status, status, sizeof(int), hipMemcpyDeviceToHost));
  return host_status ? SYNIM_E_PARAM : SYNIM_OK;
}
