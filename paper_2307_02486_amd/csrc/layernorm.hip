// LayerNorm of the LongNet attention layer (the input LayerNorm and Magneto's
// sub-LayerNorm around the dilated attention, Sec. 4.1), forward and
// backward, bf16 rows of E <= 2048 elements with float32 statistics.
//
// Forward: one wave per row; each lane holds J chunks of 8 elements
// (chunk c = lane + 64 j), the mean and then the variance of the deviations
// come from two wave sums, y = (x - mean) rstd g + b.
// Backward: one wave per row as well, 4-element chunks (E = 768 fills three
// per lane, where 8-element chunks left a quarter of the lanes idle), several
// rows per wave; with xhat = (x - mean) rstd recomputed from the saved
// statistics and dxhat = dy g,
//   dx = rstd (dxhat - mean(dxhat) - xhat mean(dxhat xhat)).
// The parameter gradients dg = sum_rows dy xhat and db = sum_rows dy are
// summed per lane over a wave's rows, over the workgroup's waves through LDS,
// and then over workgroups by a second kernel, all in a fixed order (the
// result does not depend on scheduling).
// The row loop was bound by its vector work and the latency of its two wave
// sums (LDS lane exchanges, 12 in a chain); with full lanes, sums by DPP, no
// lane masks in the sums (but in the last chunks) and one resident round of
// workgroups the 32768 x 768 backward takes 25.7 us instead of 34.0 (5.9 TB/s),
// 28 instead of 48 on data that no cache holds, and its reduction 4 us in one
// kernel instead of 8.5 in two.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.h"

namespace da {
namespace {

constexpr int kLnThreads = 256;

// Sum over the wave's 64 lanes, the same in every lane: within 16 lanes by DPP
// (lane exchanges on the vector ALU, no LDS round trips), then across the rows
// of 16 and the half-waves by lane swaps.
template <int kCtrl>
__device__ inline float dpp_add(float v) {
  const int u = __builtin_bit_cast(int, v);
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(u, u, kCtrl, 0xf, 0xf, true));
}
__device__ inline float wave_sum(float v) {
  v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
  v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
  v = dpp_add<0x141>(v);  // row_half_mirror: the other quad of eight lanes
  v = dpp_add<0x140>(v);  // row_mirror: the other eight of sixteen
  // the rows of 16 lanes in pairs, then the half-waves (adding the two results
  // of a swap of v with itself directly is not an option: the compiler takes
  // both for the same register)
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  v += __builtin_bit_cast(float, lane & 16 ? r[0] : r[1]);
  return v + other_half(v);
}

__device__ inline void unpack8(const u32x4 w, float* f) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __builtin_bit_cast(float, w[i] << 16);
    f[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xffff0000u);
  }
}

__device__ inline void load8f(const u16* p, float* f) { unpack8(*reinterpret_cast<const u32x4*>(p), f); }

__device__ inline void store8bf(u16* p, const float* f) {
  u32x4 w;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    w[i] = static_cast<unsigned>(__builtin_bit_cast(u16, (__bf16)f[2 * i])) |
           (static_cast<unsigned>(__builtin_bit_cast(u16, (__bf16)f[2 * i + 1])) << 16);
  *reinterpret_cast<u32x4*>(p) = w;
}

struct LnFwdArgs {
  const u16 *x, *g, *b;
  u16* y;
  float *mean, *rstd;
  int64_t rows;
  int32_t E;
  float eps;
};

template <int J>
__global__ __launch_bounds__(kLnThreads) void ln_fwd(LnFwdArgs a) {
  const int lane = __builtin_amdgcn_workitem_id_x() & 63;
  const int64_t row = static_cast<int64_t>(launch_index()) * (kLnThreads / 64) + (__builtin_amdgcn_workitem_id_x() >> 6);
  if (row >= a.rows) return;  // whole waves only; the kernel has no barrier
  const int nch = a.E >> 3;
  const u16* xr = a.x + row * a.E;
  float v[J][8];
  float s = 0.0f;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = lane + 64 * j;
    if (c < nch) {
      load8f(xr + 8 * c, v[j]);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[j][e];
    }
  }
  const float inv_e = 1.0f / static_cast<float>(a.E);
  const float mean = wave_sum(s) * inv_e;
  float q = 0.0f;
#pragma unroll
  for (int j = 0; j < J; ++j)
    if (lane + 64 * j < nch)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float d = v[j][e] - mean;
        q += d * d;
      }
  const float rstd = 1.0f / sqrtf(wave_sum(q) * inv_e + a.eps);
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = lane + 64 * j;
    if (c < nch) {
      float g[8], b[8], y[8];
      load8f(a.g + 8 * c, g);
      load8f(a.b + 8 * c, b);
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = (v[j][e] - mean) * rstd * g[e] + b[e];
      store8bf(a.y + row * a.E + 8 * c, y);
    }
  }
  if (lane == 0) {
    a.mean[row] = mean;
    a.rstd[row] = rstd;
  }
}

struct LnBwdArgs {
  const u16 *dy, *x, *g;
  const float *mean, *rstd;
  u16* dx;
  float* part;  // [workgroups][2E]: dg partials, then db partials
  int64_t rows;
  int32_t E, rpw;  // rows per wave
};

// Four bf16 elements of one 8-byte word pair as floats.
__device__ inline void unpack4(const u32x2 w, float* f) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    f[2 * i] = __builtin_bit_cast(float, w[i] << 16);
    f[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xffff0000u);
  }
}

template <int J>
__global__ __launch_bounds__(kLnThreads) void ln_bwd(LnBwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) float red[];  // [4 waves][2E]
  const int tid = __builtin_amdgcn_workitem_id_x();
  const int lane = tid & 63, wv = tid >> 6;
  const int nch = a.E >> 2;
  constexpr int kFull = J <= 4 ? J - 1 : J - 2;  // chunks that every lane has (see the launch)
  float g[J][4], pg[J][4], pb[J][4];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = lane + 64 * j;
#pragma unroll
    for (int e = 0; e < 4; ++e) g[j][e] = pg[j][e] = pb[j][e] = 0.0f;
    if (c < nch) unpack4(*reinterpret_cast<const u32x2*>(a.g + 4 * c), g[j]);
  }
  const float inv_e = 1.0f / static_cast<float>(a.E);
  const int64_t r0 =
      (static_cast<int64_t>(__builtin_amdgcn_workgroup_id_x()) * (kLnThreads / 64) + wv) * a.rpw;
  const int nrow = static_cast<int>(min(static_cast<int64_t>(a.rpw), a.rows - r0));  // may be <= 0
  // Row i + 1's x and dy are loaded (as raw bf16) while row i is processed.
  u32x2 nx[J], ndy[J];
  float nmean = 0.0f, nrstd = 0.0f;
#pragma unroll
  for (int j = 0; j < J; ++j) nx[j] = ndy[j] = u32x2{0u, 0u};  // lanes past the row's end hold zeros
  auto load_row = [&](int64_t row) {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = lane + 64 * j;
      if (c < nch) {
        nx[j] = *reinterpret_cast<const u32x2*>(a.x + row * a.E + 4 * c);
        ndy[j] = *reinterpret_cast<const u32x2*>(a.dy + row * a.E + 4 * c);
      }
    }
    nmean = a.mean[row];
    nrstd = a.rstd[row];
  };
  if (nrow > 0) load_row(r0);
  for (int i = 0; i < nrow; ++i) {
    const int64_t row = r0 + i;
    const float mean = nmean, rstd = nrstd;
    u32x2 xr[J], dyr[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      xr[j] = nx[j];
      dyr[j] = ndy[j];
    }
    if (i + 1 < nrow) load_row(row + 1);
    // Lanes past the row's end (in the last chunks only) have dy = g = 0 and,
    // with an rstd of zero, xhat = 0 where mean * rstd would overflow: they add
    // nothing.
    float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      float x[4], dy[4];
      unpack4(xr[j], x);
      unpack4(dyr[j], dy);
      const float rj = j < kFull || lane + 64 * j < nch ? rstd : 0.0f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float xh = (x[e] - mean) * rj, dxh = dy[e] * g[j][e];
        s1 += dxh;
        s2 += dxh * xh;
        pg[j][e] += dy[e] * xh;
        pb[j][e] += dy[e];
      }
    }
    const float m1 = wave_sum(s1) * inv_e, m2 = wave_sum(s2) * inv_e;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = lane + 64 * j;
      if (c < nch) {
        float x[4], dy[4], dx[4];
        unpack4(xr[j], x);
        unpack4(dyr[j], dy);
#pragma unroll
        for (int e = 0; e < 4; ++e) dx[e] = rstd * (dy[e] * g[j][e] - m1 - (x[e] - mean) * rstd * m2);
        u32x2 w;
#pragma unroll
        for (int k = 0; k < 2; ++k)
          w[k] = static_cast<unsigned>(__builtin_bit_cast(u16, (__bf16)dx[2 * k])) |
                 (static_cast<unsigned>(__builtin_bit_cast(u16, (__bf16)dx[2 * k + 1])) << 16);
        *reinterpret_cast<u32x2*>(a.dx + row * a.E + 4 * c) = w;
      }
    }
  }
  float* mine = red + wv * 2 * a.E;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = lane + 64 * j;
    if (c < nch) {
      *reinterpret_cast<f32x4*>(mine + 4 * c) = f32x4{pg[j][0], pg[j][1], pg[j][2], pg[j][3]};
      *reinterpret_cast<f32x4*>(mine + a.E + 4 * c) = f32x4{pb[j][0], pb[j][1], pb[j][2], pb[j][3]};
    }
  }
  __syncthreads();
  float* out = a.part + static_cast<int64_t>(__builtin_amdgcn_workgroup_id_x()) * 2 * a.E;
  for (int i = 4 * tid; i < 2 * a.E; i += 4 * kLnThreads) {
    auto at = [&](int w) { return *reinterpret_cast<const f32x4*>(red + w * 2 * a.E + i); };
    *reinterpret_cast<f32x4*>(out + i) = (at(0) + at(1)) + (at(2) + at(3));
  }
}

// part [nwg][2E] -> dg [E], db [E] in bf16: 16 columns per workgroup, four per
// thread, the partials over 64 threads: 16 of each wave by lane exchanges, the
// waves through LDS, in a fixed order.  No partials: zeros.
__global__ __launch_bounds__(kLnThreads) void ln_reduce(const float* part, u16* dg, u16* db, int nwg, int E) {
  __shared__ __attribute__((aligned(16))) float red[kLnThreads / 64][16];
  const int tid = __builtin_amdgcn_workitem_id_x();
  const int lane = tid & 63, wv = tid >> 6;
  const int col = __builtin_amdgcn_workgroup_id_x() * 16 + (lane & 3) * 4;  // 2E is a multiple of 16
  f32x4 s = f32x4{0, 0, 0, 0};
#pragma unroll 8
  for (int r = wv * 16 + (lane >> 2); r < nwg; r += 64)
    s += *reinterpret_cast<const f32x4*>(part + static_cast<int64_t>(r) * 2 * E + col);
#pragma unroll
  for (int m = 4; m < 64; m <<= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] += __shfl_xor(s[e], m, 64);
  if (lane < 4) *reinterpret_cast<f32x4*>(&red[wv][4 * lane]) = s;
  __syncthreads();
  if (tid >= 16) return;
  const float t = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
  const int c = __builtin_amdgcn_workgroup_id_x() * 16 + tid;
  u16* dst = c < E ? dg + c : db + (c - E);
  *dst = __builtin_bit_cast(u16, (__bf16)t);
}

}  // namespace

// Partials that the workspace holds: one per 32 rows and one more per 1024.
static int64_t ln_partials(int64_t rows) {
  const int64_t blocks = (rows + 31) / 32;
  return blocks + (blocks + 31) / 32;
}

// Rows per wave of the backward: at most as many workgroups as are resident at
// once, and no more than the workspace has partials for.  The rows a lane
// holds set the registers: up to four chunks (E <= 1024) 154, three waves per
// SIMD and so three workgroups per CU; six (E <= 1536) 208, two; eight 265, one.
// Backward, us, 768 workgroups at every width -> by this rule: 24000 x 1280
// 42 -> 37, 50000 x 1536 111 -> 102, 24000 x 1704 57 -> 47, 16384 x 2048 47 ->
// 42, 65536 x 2048 170 -> 173; 512 at E <= 1024: 65536 x 768 55 -> 62.
static int64_t ln_rows_per_wave(int64_t rows, int64_t E) {
  const int64_t resident = E <= 1024 ? 768 : E <= 1536 ? 512 : 256;
  const int64_t waves = std::min(resident, std::max<int64_t>(1, ln_partials(rows))) * (kLnThreads / 64);
  return std::max<int64_t>(1, (rows + waves - 1) / waves);
}

uint64_t layernorm_bwd_workspace(int64_t rows, int64_t E) {
  return static_cast<uint64_t>(ln_partials(rows)) * 2 * E * 4;
}

hipError_t launch_layernorm_fwd(const void* x, const void* g, const void* b, void* y, float* mean, float* rstd,
                                int64_t rows, int64_t E, float eps, hipStream_t stream) {
  LnFwdArgs a{static_cast<const u16*>(x), static_cast<const u16*>(g), static_cast<const u16*>(b),
              static_cast<u16*>(y), mean, rstd, rows, static_cast<int32_t>(E), eps};
  if (rows == 0) return hipSuccess;
  const dim3 grid = grid_of((rows + 3) / 4);
  const int J = static_cast<int>((E / 8 + 63) / 64);
  if (J == 1) hipLaunchKernelGGL(ln_fwd<1>, grid, dim3(kLnThreads), 0, stream, a);
  else if (J == 2) hipLaunchKernelGGL(ln_fwd<2>, grid, dim3(kLnThreads), 0, stream, a);
  else hipLaunchKernelGGL(ln_fwd<4>, grid, dim3(kLnThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_layernorm_bwd(const void* dy, const void* x, const void* g, const float* mean, const float* rstd,
                                void* dx, void* dg, void* db, int64_t rows, int64_t E, void* workspace,
                                hipStream_t stream) {
  const int64_t rpw = ln_rows_per_wave(rows, E);
  const int64_t per_wg = rpw * (kLnThreads / 64);
  const int64_t nwg = (rows + per_wg - 1) / per_wg;
  float* part = static_cast<float*>(workspace);
  LnBwdArgs a{static_cast<const u16*>(dy), static_cast<const u16*>(x), static_cast<const u16*>(g), mean, rstd,
              static_cast<u16*>(dx), part, rows, static_cast<int32_t>(E),
              static_cast<int32_t>(rpw)};
  const dim3 grid(static_cast<unsigned>(nwg));
  const size_t smem = static_cast<size_t>(kLnThreads / 64) * 2 * E * sizeof(float);
  if (nwg > 0) {  // no rows: only the reduction, which then writes zeros
    switch ((E + 255) / 256) {
      case 1: hipLaunchKernelGGL(ln_bwd<1>, grid, dim3(kLnThreads), smem, stream, a); break;
      case 2: hipLaunchKernelGGL(ln_bwd<2>, grid, dim3(kLnThreads), smem, stream, a); break;
      case 3: hipLaunchKernelGGL(ln_bwd<3>, grid, dim3(kLnThreads), smem, stream, a); break;
      case 4: hipLaunchKernelGGL(ln_bwd<4>, grid, dim3(kLnThreads), smem, stream, a); break;
      case 5: case 6: hipLaunchKernelGGL(ln_bwd<6>, grid, dim3(kLnThreads), smem, stream, a); break;
      default: hipLaunchKernelGGL(ln_bwd<8>, grid, dim3(kLnThreads), smem, stream, a); break;
    }
  }
  hipLaunchKernelGGL(ln_reduce, dim3(static_cast<unsigned>(E / 8)), dim3(kLnThreads), 0, stream,
                     static_cast<const float*>(part), static_cast<u16*>(dg), static_cast<u16*>(db),
                     static_cast<int>(nwg), static_cast<int>(E));
  return hipGetLastError();
}

}  // namespace da
