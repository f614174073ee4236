// Standalone slope step (paper Sec. 2.2): central differences at every pupil
// pixel of a haloed phase map, averaged over each valid subaperture.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace synim {
namespace {

constexpr int SBLOCK = 256;          // most threads of a workgroup, two pixel columns each
constexpr int SROWS = 4;             // most subaperture rows one workgroup walks in turn

// Two neighbouring samples (any float alignment: one 8-byte load).
struct __attribute__((packed, aligned(4))) Pair {
  float a, b;
};
// A thread's samples of a pixel row: columns x and x + 1, and the ones beside them.
struct Row {
  float c0, c1, left, right;
};
constexpr int DPP_WAVE_SHL1 = 0x130, DPP_WAVE_SHR1 = 0x138;   // lane i from i + 1, from i - 1
template <int DPP>
__device__ __forceinline__ float from_beside(float at_edge, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(at_edge), __float_as_int(v), DPP,
                                                    0xf, 0xf, false));
}

// One workgroup per (group of up to SROWS subaperture rows, run of whole subapertures
// across the block's pixel columns, run of phase maps).  Thread t owns pixel columns
// x = x0 + 2t and x + 1 and walks down the group's pixel rows with three of them in
// registers: one 8-byte load per row holds both columns' samples, the lanes
// beside it the samples left and right of them (one load more for the wave's two
// outer lanes), the rows before and after it the ones above and below.  What
// bounds it is the cache's accesses and the vector instructions, each about two
// thirds busy (four separate loads and a pupil byte per pixel: 0.40 ms for 1200
// maps of 482 x 482; a 16-byte load that overlaps its neighbours' took a cache
// access for nearly every lane, 0.33), at small stacks the chain of a wave's rows.
// U pixel rows' loads are in flight, a divisor of p where there is one (RAGGED: none,
// the last rows of a subaperture are loaded and left out), and the pupil comes as a
// word of bits for them: with a test, a branch and a count a row in one kernel for
// every p, one map of 2 x 2 subapertures of 32 pixels took 11.5 us, now 7.2 (8.2
// with a column a thread), of 16 x 16 of 24 11.0, now 7.5.
// A wave whose columns lie outside the pupil over a subaperture row reads nothing
// there, one wholly inside it tests no pupil bits.
// The pupil-masked differences and the pupil count are summed down each subaperture
// row; the per-subaperture sums then add those column sums in column order (a
// fixed order, so results are bit-reproducible).  The pupil of a thread's columns
// is kept as bits over the run of maps.
// Each XCD takes all blocks of a map before its next, so that shared rows and lines
// meet in its L2.  Now 0.25.
template <int U, bool RAGGED>
__global__ __launch_bounds__(SBLOCK) void slopes_kernel(const float* __restrict__ phase, int n,
                                                        const int32_t* __restrict__ valid,
                                                        const uint8_t* __restrict__ pupil,
                                                        int n_sub_x, int n_sub_y, int p, int nv,
                                                        int subs_per_block, int maps_per_run,
                                                        int longer,
                                                        int by_xcd, int srows,
                                                        float* __restrict__ slopes) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, T = blockDim.x;
  // column sums [gx, gy, pupil count][subaperture row][2 T], then the valid-list
  // index of the group's subapertures
  extern __shared__ __align__(16) float s_sum[];
  int* const s_kk = reinterpret_cast<int*>(s_sum + 12 * T);
  auto sum_at = [&](int what, int r, int c) -> float& { return s_sum[(2 * what + r) * 2 * T + c]; };
  const int n_runs = (n_sub_x + subs_per_block - 1) / subs_per_block;
  const int n_blk = (n_sub_y + srows - 1) / srows * n_runs;
  const int sb = by_xcd ? blockIdx.x >> 3 : blockIdx.x;
  const int blk = sb % n_blk;
  // the maps of this block's run: the first `longer` runs have one more
  const int run = by_xcd ? sb / n_blk * 8 + (blockIdx.x & 7) : sb / n_blk;
  const int i0 = run * maps_per_run + min(run, longer);
  const int i_end = min(n, i0 + maps_per_run + (run < longer ? 1 : 0));
  if (i0 >= i_end) return;
  const int grp = blk / n_runs;
  const int u0 = (blk - grp * n_runs) * subs_per_block;
  const int W = n_sub_x * p, H = n_sub_y * p;
  const int Wh = W + 2;
  const int nu = min(subs_per_block, n_sub_x - u0);
  const int x = u0 * p + 2 * t;
  const int v0 = grp * srows, v_end = min(n_sub_y, v0 + srows);
  // valid-list index of every subaperture of the group (-1: not valid)
  for (int e = t; e < (v_end - v0) * nu; e += T) s_kk[e] = -1;
  __syncthreads();
  for (int v = v0 + wave; v < v_end; v += T >> 6) {
    const int k0 = v * n_sub_x + u0;
    const int lo = first_at_least(valid, nv, k0, lane);
    for (int j = lo + lane; j < min(nv, lo + nu); j += 64) {
      const int u = valid[j] - k0;
      if (u < nu) s_kk[(v - v0) * nu + u] = j;
    }
  }
  // this thread's columns: on (the first lies in the block), two (the second too)
  const bool on = 2 * t < nu * p, two = 2 * t + 1 < nu * p;
  const int y_beg = v0 * p, y_end = v_end * p;
  // offsets in a haloed row: of column x (columns past W are read as W - 1, W), of
  // the column before the wave's first and after its last
  const int at = 1 + min(x, W - 1);
  const bool edge = lane == 0 || (lane == 63 && x + 2 <= W);
  const int at_outer = lane == 0 ? min(x, W) : min(x + 3, W + 1);
  // pupil bits of rows y_beg.. of the two columns (at most 64 rows: the host's rule)
  unsigned long long in0 = 0, in1 = 0;
  if (on) {
    const int second = two ? 1 : 0;
    for (int y = y_beg; y < y_end; y += 8) {
      uint8_t q[8][2];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint8_t* at = pupil + (size_t)min(y + k, y_end - 1) * W + x;
        q[k][0] = at[0];
        q[k][1] = at[second];
      }
      unsigned m0 = 0, m1 = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        m0 |= (q[k][0] != 0 ? 1u : 0u) << k;
        m1 |= (q[k][1] != 0 ? 1u : 0u) << k;
      }
      const unsigned there = (1u << min(8, y_end - y)) - 1;
      in0 |= (unsigned long long)(m0 & there) << (y - y_beg);
      in1 |= (unsigned long long)(two ? m1 & there : 0u) << (y - y_beg);
    }
  }
  for (int i = i0; i < i_end; ++i) {
    const float* ph = phase + (size_t)i * (size_t)(H + 2) * (size_t)Wh;
    float* out = slopes + (size_t)i * 2 * nv;
    // pixel row y (haloed row y + 1): its own two columns per lane, and one of the
    // wave's two outer columns for its first and last lane
    auto own = [&](int y) {
      return *reinterpret_cast<const Pair*>(ph + (size_t)(y + 1) * Wh + at);
    };
    auto outer = [&](int y) { return ph[(size_t)(y + 1) * Wh + at_outer]; };
    auto make = [&](const Pair& v, float e) {
      Row r;
      r.c0 = x < W ? v.a : v.b;   // (the pair of column W starts one before it)
      r.c1 = v.b;
      r.left = from_beside<DPP_WAVE_SHR1>(e, r.c1);
      r.right = from_beside<DPP_WAVE_SHL1>(e, r.c0);
      return r;
    };
    Row prev{}, cur{};
    bool have = false;   // prev and cur hold the pixel rows above and at the next row
    // two subaperture rows per step between barriers
    for (int v = v0; v < v_end; v += 2) {
      const int nr = min(2, v_end - v);
      float gx[2][2] = {}, gy[2][2] = {}, cnt[2][2] = {};   // [subaperture row][column]
      // subaperture row r; FULL: all of the wave's pixels are in the pupil
      auto walk = [&](int r, auto full) {
        constexpr bool FULL = decltype(full)::value;
        const int ya = (v + r) * p;
        if (!have) {
          const Pair pv = own(ya - 1), pc = own(ya);
          const float e = edge ? outer(ya) : 0.f;
          prev = make(pv, 0.f);
          cur = make(pc, e);
        }
        float sx0 = 0.f, sx1 = 0.f, sy0 = 0.f, sy1 = 0.f;
        int c0 = 0, c1 = 0;
        for (int d0 = 0; d0 < p; d0 += U) {
          Pair nx[U];
          float e[U];
#pragma unroll
          for (int u = 0; u < U; ++u) nx[u] = own(min(ya + d0 + u + 1, y_end));
#pragma unroll
          for (int u = 0; u < U; ++u) e[u] = 0.f;
          if (edge) {
#pragma unroll
            for (int u = 0; u < U; ++u) e[u] = outer(min(ya + d0 + u + 1, y_end));
          }
          unsigned m0 = ~0u, m1 = ~0u;
          if (!FULL) {
            m0 = (unsigned)(in0 >> (ya + d0 - y_beg));
            m1 = (unsigned)(in1 >> (ya + d0 - y_beg));
            const unsigned here = (1u << min(U, p - d0)) - 1;
            c0 += __popc(m0 & here);
            c1 += __popc(m1 & here);
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (RAGGED && d0 + u >= p) break;
            const Row next = make(nx[u], e[u]);
            const float ex0 = 0.5f * (cur.c1 - cur.left), ex1 = 0.5f * (cur.right - cur.c0);
            const float ey0 = 0.5f * (next.c0 - prev.c0), ey1 = 0.5f * (next.c1 - prev.c1);
            const bool a = FULL || (m0 >> u & 1), b = FULL || (m1 >> u & 1);
            sx0 += a ? ex0 : 0.f;
            sy0 += a ? ey0 : 0.f;
            sx1 += b ? ex1 : 0.f;
            sy1 += b ? ey1 : 0.f;
            prev = cur;
            cur = next;
          }
        }
        gx[r][0] = sx0;
        gx[r][1] = sx1;
        gy[r][0] = sy0;
        gy[r][1] = sy1;
        cnt[r][0] = FULL ? (float)p : (float)c0;
        cnt[r][1] = FULL ? (float)p : (float)c1;
      };
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        if (r >= nr) break;
        // how the wave's columns lie over this row's pixels: outside the pupil
        // nothing is read
        const unsigned long long px = (p < 64 ? (1ull << p) - 1 : ~0ull) << ((v + r) * p - y_beg);
        const bool some = __any(((in0 | in1) & px) != 0);
        const bool full = __all(!on || (two && (in0 & in1 & px) == px));
        if (some) {   // (the wave as a whole: its lanes read each other)
          if (full) walk(r, std::true_type{});
          else walk(r, std::false_type{});
        }
        have = some;
      }
      __syncthreads();   // the previous step's sums have been read (and s_kk written)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        *reinterpret_cast<float2*>(&sum_at(0, r, 2 * t)) = make_float2(gx[r][0], gx[r][1]);
        *reinterpret_cast<float2*>(&sum_at(1, r, 2 * t)) = make_float2(gy[r][0], gy[r][1]);
        *reinterpret_cast<float2*>(&sum_at(2, r, 2 * t)) = make_float2(cnt[r][0], cnt[r][1]);
      }
      __syncthreads();
      for (int e = t; e < nr * nu; e += T) {
        const int r = e / nu, u = e - r * nu;
        const int kk = s_kk[(v - v0 + r) * nu + u];
        if (kk < 0) continue;
        float sx = 0.f, sy = 0.f, cn = 0.f;
        const float* const sums = &sum_at(0, r, u * p);
#pragma unroll 4
        for (int c = 0; c < p; ++c) {
          sx += sums[c];
          sy += sums[4 * T + c];
          cn += sums[8 * T + c];
        }
        out[kk] = cn > 0.f ? sx / cn : 0.f;
        out[nv + kk] = cn > 0.f ? sy / cn : 0.f;
      }
    }
  }
}
}  // namespace
}  // namespace synim

extern "C" int synim_sa_slopes(const float* phase, int n, const synim_wfs* wfs, float* slopes,
                               void* stream) {
  using namespace synim;
  if (!phase || !slopes) return SYNIM_E_NULL;
  int st = validate_wfs(wfs);
  if (st != SYNIM_OK) return st;
  if (n < 1 || n > 65535) return SYNIM_E_SHAPE;
  if (wfs->p > SBLOCK) return SYNIM_E_SHAPE;
  // as many threads as half the grid's columns need, up to four waves (any of 64,
  // 128, 256 threads within 3% of each other on 480 columns)
  const int T = std::min(SBLOCK, ((wfs->n_sub_x * wfs->p + 1) / 2 + 63) / 64 * 64);
  const int spb = std::min(wfs->n_sub_x, 2 * T / wfs->p);
  // Workgroups that are resident together (20 waves a CU) in one round, each with
  // as many maps as that takes, up to 8, and two or four subaperture rows, which read
  // fewer rows twice, where one would take more than two rounds and the chain of pixel
  // rows is no longer than 20.  Maps of 80 x 80 subapertures of 6 pixels, 24 / 64 / 200
  // / 1200 of them: 8.8, 17, 35, 254 us; with rows and maps a workgroup chosen for 48 to
  // 64 waves a CU 13, 28, 50, 286, with one map and eight rows each 17, 24, 55, 394.
  // (Rooms of 12 to 28 waves, chains of 12 to 24 rows: 0.3 to 2% slower over maps of 23
  // sensors.)  Runs of even length; eight or more in whole eights, an equal number
  // for each XCD, fewer spread over all.
  const int p = wfs->p;
  const long cols = (wfs->n_sub_x + spb - 1) / spb, room = 256 * (20 / (T / 64));
  auto blocks = [&](int rows) { return (wfs->n_sub_y + rows - 1) / rows * cols; };
  int srows = 1;
  while (2 * srows <= std::min(SROWS, wfs->n_sub_y) && 2 * srows * p <= 20 &&
         n * blocks(srows) > 2 * room)
    srows *= 2;
  const long bx = blocks(srows), mpr = std::clamp((n * bx + room - 1) / room, 1L, 8L);
  long runs = (n + mpr - 1) / mpr;
  const bool by_xcd = runs >= 8;
  if (by_xcd) runs = (runs + 7) / 8 * 8;
  if (runs * bx > 0x7fffffffL) return SYNIM_E_SHAPE;
  const auto kernel = p % 6 == 0   ? slopes_kernel<6, false>
                      : p % 7 == 0 ? slopes_kernel<7, false>
                      : p % 5 == 0 ? slopes_kernel<5, false>
                      : p % 8 == 0 ? slopes_kernel<8, false>
                      : p % 4 == 0 ? slopes_kernel<4, false>
                      : p % 3 == 0 ? slopes_kernel<3, false>
                                   : slopes_kernel<4, true>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(runs * bx)),
                     dim3(T),
                     (12 * T + SROWS * spb) * sizeof(float),
                     (hipStream_t)stream, phase, n, wfs->valid_idx, wfs->pupil, wfs->n_sub_x,
                     wfs->n_sub_y, wfs->p, wfs->n_valid, spb, (int)(n / runs), (int)(n % runs), by_xcd ? 1 : 0, srows, slopes);
  SYNIM_HIP_TRY(hipGetLastError());
  return SYNIM_OK;
}
