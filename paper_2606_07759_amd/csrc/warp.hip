// Standalone single-step bilinear resampling of an IF stack onto the WFS grid
// (paper Sec. 2.1: the composite map is applied once, with one interpolation).
#include <algorithm>
#include <cmath>

#include "common.hpp"

namespace synim {
namespace {

constexpr int WX = 128, WY = 2;   // a workgroup's output pixels
constexpr int MOST = 8;           // IFs of a run at most, in one pass
// What bounds the step is memory: each source pixel under the window once, the
// window written.  A workgroup covers 128 x 2 output pixels of a run of IFs, its
// FP64 source coordinates formed once and the taps of up to 8 IFs in flight.  1200
// ELT IFs of 512^2 onto 482^2: runs of 4 IFs 0.95 ms, of 8 0.60, of 16 0.64, of 64
// 0.70 (256 x 4 pixels: 0.65 with 8; runs of two, four separate taps waited for in
// turn: 1.15).  Runs of up to 8 also where that makes few workgroups, as a
// workgroup's coordinates cost more than the IFs (8 IFs onto 482^2: 6.0 us in one run,
// 11.5 one by one; onto 82^2 no difference).
// Consecutive workgroups go to the 8 XCDs in turn; from six runs on their number is
// a multiple of 8, of even length, and each XCD takes every window block of one run
// before its next, so that the source rows neighbouring blocks share, and the
// output lines they share, meet in its L2 (64 IFs onto 482^2: 21 us, 31 spread over
// all; fewer than six would leave XCDs idle).  Runs of equal length with a short
// last one, one by one from 8 IFs on, took 16 us for 9 IFs onto 386^2 (two on the
// first XCD), now 6.7.

// Two neighbouring taps (any float alignment: one 8-byte load).
struct __attribute__((packed, aligned(4))) Pair {
  float x, y;
};

// UNR: IFs in flight, a power of two that holds the workgroup's run (a run of two
// with eight in flight reads its last IF six times over: 55 IFs onto 170 x 170
// pixels then took longer than the 10.9 us of one IF a workgroup, now 9.0).
template <int UNR>
__global__ __launch_bounds__(WX* WY) void warp_kernel(const float* __restrict__ ifs, int n,
                                                      int H_in, int W_in, MapD m, int H_out,
                                                      int W_out, int halo, int if_per_run,
                                                      int longer, int by_xcd,
                                                      float* __restrict__ out,
                                                      int32_t* __restrict__ oob) {
  const int Wh = W_out + 2 * halo, Hh = H_out + 2 * halo;
  const int bx = (Wh + WX - 1) / WX, by = (Hh + WY - 1) / WY, nxy = bx * by;
  const int s = by_xcd ? blockIdx.x >> 3 : blockIdx.x;
  const int run = by_xcd ? s / nxy * 8 + (blockIdx.x & 7) : s / nxy, xy = s % nxy;
  // the IFs of this block's run: the first `longer` runs have one more
  const int i_begin = run * if_per_run + min(run, longer);
  const int i_end = min(n, i_begin + if_per_run + (run < longer ? 1 : 0));
  if (i_begin >= i_end) return;
  const int ox = xy % bx * WX + (threadIdx.x % WX);
  const int oy = xy / bx * WY + (threadIdx.x / WX);
  const bool active = ox < Wh && oy < Hh;

  double xs, ys;
  src_xy(m, ox - halo, oy - halo, xs, ys);
  const double fi = floor(xs), fj = floor(ys);
  const double ad = xs - fi, cd = ys - fj;
  // tap validity in FP64 first, so huge coordinates never reach an int conversion
  const bool vi0 = fi >= 0.0 && fi <= W_in - 1.0;
  const bool vi1 = fi + 1.0 >= 0.0 && fi + 1.0 <= W_in - 1.0;
  const bool vj0 = fj >= 0.0 && fj <= H_in - 1.0;
  const bool vj1 = fj + 1.0 >= 0.0 && fj + 1.0 <= H_in - 1.0;
  const int i0 = (vi0 || vi1) ? (int)fi : 0;
  const int j0 = (vj0 || vj1) ? (int)fj : 0;
  const float w00 = (float)((1.0 - ad) * (1.0 - cd));
  const float w01 = (float)(ad * (1.0 - cd));
  const float w10 = (float)((1.0 - ad) * cd);
  const float w11 = (float)(ad * cd);
  const bool t00 = active && vj0 && vi0, t01 = active && vj0 && vi1;
  const bool t10 = active && vj1 && vi0, t11 = active && vj1 && vi1;
  const size_t r0 = (size_t)j0 * W_in + i0;
  const size_t r1 = r0 + W_in;

  if (oob != nullptr && run == 0) {
    const bool o = active && (xs < 0.0 || xs > W_in - 1.0 || ys < 0.0 || ys > H_in - 1.0);
    const int cnt = __syncthreads_count(o);
    if (threadIdx.x == 0 && cnt > 0) atomicAdd(oob, cnt);
  }
  if (!active) return;

  const size_t plane_in = (size_t)H_in * W_in;
  const size_t plane_out = (size_t)Hh * Wh;
  const size_t o0 = (size_t)oy * Wh + ox;
  // UNR IFs per pass (one pass): all taps are loaded before the first one is used, so a
  // thread keeps that many gathers in flight instead of one IF's.  (Past the
  // run's end the last IF is read again and not stored.)
  if (__all(t00 && t01 && t10 && t11)) {   // the wave's taps all lie on the grid
    for (int i = i_begin; i < i_end; i += UNR) {
      Pair a[UNR], b[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const float* F = ifs + (size_t)min(i + u, i_end - 1) * plane_in;
        a[u] = *reinterpret_cast<const Pair*>(F + r0);
        b[u] = *reinterpret_cast<const Pair*>(F + r1);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        float acc = __fmaf_rn(w00, a[u].x, 0.0f);
        acc = __fmaf_rn(w01, a[u].y, acc);
        acc = __fmaf_rn(w10, b[u].x, acc);
        acc = __fmaf_rn(w11, b[u].y, acc);
        if (i + u < i_end) out[(size_t)(i + u) * plane_out + o0] = acc;
      }
    }
    return;
  }
  for (int i = i_begin; i < i_end; i += UNR) {
    float v[UNR][4];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const float* F = ifs + (size_t)min(i + u, i_end - 1) * plane_in;
      v[u][0] = t00 ? F[r0] : 0.0f;
      v[u][1] = t01 ? F[r0 + 1] : 0.0f;
      v[u][2] = t10 ? F[r1] : 0.0f;
      v[u][3] = t11 ? F[r1 + 1] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      float acc = 0.0f;
      if (t00) acc = __fmaf_rn(w00, v[u][0], acc);
      if (t01) acc = __fmaf_rn(w01, v[u][1], acc);
      if (t10) acc = __fmaf_rn(w10, v[u][2], acc);
      if (t11) acc = __fmaf_rn(w11, v[u][3], acc);
      if (i + u < i_end) out[(size_t)(i + u) * plane_out + o0] = acc;
    }
  }
}

}  // namespace
}  // namespace synim

extern "C" int synim_affine_warp(const float* ifs, int n, int H_in, int W_in,
                                 const synim_affine* A, int H_out, int W_out, int halo, float* out,
                                 int32_t* oob_count, void* stream) {
  using namespace synim;
  if (!ifs || !A || !out) return SYNIM_E_NULL;
  if (n < 1 || H_in < 1 || W_in < 1 || H_out < 1 || W_out < 1 || halo < 0 || halo > 8)
    return SYNIM_E_SHAPE;
  if ((long)H_out + 2 * halo > 65536 || (long)W_out + 2 * halo > 65536) return SYNIM_E_SHAPE;
  const int Wh = W_out + 2 * halo, Hh = H_out + 2 * halo;
  const int bx = (Wh + WX - 1) / WX, by = (Hh + WY - 1) / WY;
  const long xy = (long)bx * by;
  long runs = ((long)n + MOST - 1) / MOST;
  const bool by_xcd = runs >= 6;
  if (by_xcd) runs = (runs + 7) / 8 * 8;   // an equal number for each XCD
  const long ipb = (n + runs - 1) / runs;
  const long blocks = runs * xy;
  if (blocks > 0x7fffffffL) return SYNIM_E_SHAPE;
  const auto kernel = ipb > 4   ? warp_kernel<8>
                      : ipb > 2 ? warp_kernel<4>
                      : ipb > 1 ? warp_kernel<2>
                                : warp_kernel<1>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(WX * WY), 0, (hipStream_t)stream, ifs,
                     n, H_in, W_in, to_map(*A), H_out, W_out, halo, (int)(n / runs),
                     (int)(n % runs), by_xcd ? 1 : 0, out, oob_count);
  SYNIM_HIP_TRY(hipGetLastError());
  return SYNIM_OK;
}
