// Weight gradient of the LongNet attention layer's projections (the layer
// around the dilated attention, Sec. 4.1): dW[m][n] = sum_k dY[k][m] X[k][n]
// for dY [K, M] and X [K, N] bf16 row-major, K = the layer's B * N rows.
// The reduction is long (tens of thousands of rows) and the output small
// (E x E), so the work is split along k: workgroup (tile, split) computes a
// 128 x 128 output tile over one k-chunk into a float32 partial, and a second
// kernel sums the partials into bf16.  The bias gradient (dY's column sums)
// comes from the dY tiles already in LDS, as products with a column of ones:
// dY is not read a second time and no launches are added (K = 32768, M = N =
// 768 with the bias gradient: 50 us, and 59 us when two more kernels formed it).
//
// Both operands go from HBM straight to LDS as row-major 64 x 128 tiles
// (double buffered) and reach the MFMA (v_mfma_f32_32x32x16_bf16) through
// transposed LDS reads, which give each lane eight consecutive k of one
// column, the operand layout both A = dY^T and B = X need.  Four waves, each a
// 64 x 64 quarter of the tile.  Bound by the tiles' way from L2 into LDS (590
// MB at the shape above, 14-20 TB/s: with the products taken out the loads
// alone take 32 of the kernel's 46 us) and the partials.  Measured and not
// kept: five 32-row stages instead of two of 64 rows (48-50 us for the kernel
// against 43), eight waves sharing a tile with half the partials (50 us),
// that with fragments read one step ahead (slower), 256 x 256 tiles (slower).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.h"

namespace da {
namespace {

constexpr int kWgThreads = 256;
constexpr int kTileK = 64;    // k rows per LDS tile
constexpr int kTileMN = 128;  // output tile edge
using TLw = TileLayout<kTileMN>;
constexpr int kWgLoads = kTileK * TLw::kSlots / 64 / (kWgThreads / 64);  // 16-byte loads per lane and operand

struct WgradArgs {
  const u16* dy;
  const u16* x;
  float* part;     // [splits][M][N]
  float* db_part;  // [splits][db_share][M] column sums of dy
  int64_t K;
  int32_t M, N, chunk, tiles_n, tiles;
  int32_t db_share;        // column tiles that share out a block row's column sums
  int32_t items, per_xcd;  // tiles * splits, and items per XCD (rounded up)
};

struct SmemWgrad {
  __attribute__((aligned(16))) u16 a[2][kTileK * kTileMN];
  __attribute__((aligned(16))) u16 b[2][kTileK * kTileMN];
};

template <bool kBias>
__global__ __launch_bounds__(kWgThreads) void wgrad_partial(WgradArgs a) {
  __shared__ SmemWgrad sm;
  const int tid = __builtin_amdgcn_workitem_id_x();
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hi = lane >> 5;
  // Workgroup i runs on XCD i % 8.  Item (split, tile) = split * tiles + tile
  // goes to workgroup (item % per) * 8 + item / per, so that XCD x takes items
  // [x per, (x + 1) per): the tiles of one or two neighbouring k-chunks, whose
  // rows its own L2 then serves to every tile after the first fetch.
  const int blk = __builtin_amdgcn_workgroup_id_x();
  const int item = (blk & 7) * a.per_xcd + (blk >> 3);
  if (item >= a.items) return;
  const int tile = item % a.tiles, split = item / a.tiles;
  const int tile_n = tile % a.tiles_n;
  const int m0 = (tile / a.tiles_n) * kTileMN, n0 = tile_n * kTileMN;
  const int64_t k0 = static_cast<int64_t>(split) * a.chunk;
  const int64_t k1 = k0 + a.chunk < a.K ? k0 + a.chunk : a.K;
  const int ntk = static_cast<int>((k1 - k0 + kTileK - 1) / kTileK);

  // HBM -> LDS loads: load i of this wave fills 64 consecutive 16-byte slots.
  int lrow[kWgLoads], lslot[kWgLoads];
#pragma unroll
  for (int i = 0; i < kWgLoads; ++i) {
    const int s = 64 * (wv * kWgLoads + i) + lane;
    lrow[i] = s / TLw::kSlots;
    lslot[i] = (s % TLw::kSlots) ^ TLw::swz(lrow[i]);
  }
  auto load_tile = [&](int kt, int buf) {
    const int64_t r0 = k0 + static_cast<int64_t>(kt) * kTileK;
    const int valid = static_cast<int>(k1 - r0 < kTileK ? k1 - r0 : kTileK);  // rows past k1 read as 0
    const __amdgpu_buffer_rsrc_t sa = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<u16*>(a.dy + r0 * a.M + m0), 0, valid * a.M * 2, kBufferFlags);
    const __amdgpu_buffer_rsrc_t sb = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<u16*>(a.x + r0 * a.N + n0), 0, valid * a.N * 2, kBufferFlags);
    char* la = reinterpret_cast<char*>(&sm.a[buf][0]);
    char* lb = reinterpret_cast<char*>(&sm.b[buf][0]);
#pragma unroll
    for (int i = 0; i < kWgLoads; ++i) {
      const int lds_off = 1024 * (wv * kWgLoads + i);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(sa, (lds_void*)(la + lds_off), 16, lrow[i] * a.M * 2 + lslot[i] * 16,
                                               0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(sb, (lds_void*)(lb + lds_off), 16, lrow[i] * a.N * 2 + lslot[i] * 16,
                                               0, 0, 0);
    }
  };

  // Transposed-read addresses: lane's column (m or n) within its wave's 64,
  // rows 8t + 4hi + 0..3 of each 16-row k-step.
  const int wm = wv & 1, wn = wv >> 1;
  const int tr_r = (lane & 15) >> 2;
  const int tr_c = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
  int aoff[2][2], boff[2][2];
#pragma unroll
  for (int blk2 = 0; blk2 < 2; ++blk2)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int cm = wm * 64 + blk2 * 32 + tr_c, cn = wn * 64 + blk2 * 32 + tr_c;
      aoff[blk2][t] = TLw::offset(8 * t + 4 * hi + tr_r, cm >> 3) + (cm & 7) * 2;
      boff[blk2][t] = TLw::offset(8 * t + 4 * hi + tr_r, cn >> 3) + (cn & 7) * 2;
    }

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};

  // The column sums of dy are dY^T times a column of ones, formed by one of
  // the two waves that hold the same rows.  The first db_share tiles of a block
  // row share its k tiles out: each takes every db_share-th.
  f32x16 acc_db[2] = {f32x16{}, f32x16{}};
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
  const bool has_db = kBias && wn == 0 && tile_n < a.db_share;
  int db_next = has_db ? tile_n : ntk;

  if (ntk > 0) load_tile(0, 0);
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  __syncthreads();
  for (int kt = 0; kt < ntk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < ntk) load_tile(kt + 1, cur ^ 1);
    const uint32_t la = lds_addr(&sm.a[cur][0]), lb = lds_addr(&sm.b[cur][0]);
    const bool do_db = kt == db_next;
    static_for<0, kTileK / 16>([&](auto KK) {
      constexpr int row = 16 * decltype(KK)::value;  // multiple of 16: the swizzle of rows 0..15
      u32x2 fa[2][2], fb[2][2];
      static_for<0, 2>([&](auto B2) {
        static_for<0, 2>([&](auto T) {
          constexpr int bb = decltype(B2)::value, t = decltype(T)::value;
          fa[bb][t] = lds_read_tr16<row * TLw::kRowBytes>(la + aoff[bb][t]);
          fb[bb][t] = lds_read_tr16<row * TLw::kRowBytes>(lb + boff[bb][t]);
        });
      });
      lds_wait<0>();
      bf16x8 av[2], bv[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        lds_bind(fa[i][0]);
        lds_bind(fa[i][1]);
        lds_bind(fb[i][0]);
        lds_bind(fb[i][1]);
        av[i] = __builtin_bit_cast(bf16x8, u32x4{fa[i][0][0], fa[i][0][1], fa[i][1][0], fa[i][1][1]});
        bv[i] = __builtin_bit_cast(bf16x8, u32x4{fb[i][0][0], fb[i][0][1], fb[i][1][0], fb[i][1][1]});
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
      if constexpr (kBias)
        if (do_db)
#pragma unroll
          for (int i = 0; i < 2; ++i) acc_db[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], ones, acc_db[i], 0, 0, 0);
    });
    if (do_db) db_next += a.db_share;
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
  }

  // C layout: lane holds column n = lane % 32 and rows 8 jj + 4 hi + e.
  float* part = a.part + static_cast<int64_t>(split) * a.M * a.N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = m0 + wm * 64 + i * 32 + 8 * jj + 4 * hi + e;
          const int n = n0 + wn * 64 + j * 32 + (lane & 31);
          part[static_cast<int64_t>(m) * a.N + n] = acc[i][j][4 * jj + e];
        }
  if (has_db && (lane & 31) == 0) {
    // every column of the product with ones is the same: lanes 0 and 32 store theirs
    float* db = a.db_part + static_cast<int64_t>(split * a.db_share + tile_n) * a.M + m0 + wm * 64 + 4 * hi;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        *reinterpret_cast<f32x4*>(db + i * 32 + 8 * jj) =
            f32x4{acc_db[i][4 * jj], acc_db[i][4 * jj + 1], acc_db[i][4 * jj + 2], acc_db[i][4 * jj + 3]};
  }
}

// dst[i] = the sum over the rows of src [rows][width], rounded to bf16: four
// columns per thread, the rows over kLanes threads combined through LDS in a
// fixed order.
template <int kLanes>
__device__ inline void sum_rows(const float* src, u16* dst, int64_t width, int rows, int blk, float* red) {
  constexpr int kCols = kWgThreads / kLanes;
  const int tid = __builtin_amdgcn_workitem_id_x();
  const int cl = tid % kCols, rl = tid / kCols;
  const int64_t i = (static_cast<int64_t>(blk) * kCols + cl) * 4;
  f32x4 s = f32x4{0, 0, 0, 0};
  // Rows by eights keep their loads in flight; of fewer than 16 rows steps of two
  // measured faster (the call without bias, by eights -> by twos: 1024 x 1024, K =
  // 4096, 8 rows, 24.7 -> 24.4 us, 2048 x 512, K = 8192 33.9 -> 33.0; 512 x 512, K =
  // 16384, 32 rows, 21.7 -> 22.2).
  if (i < width) {
    if (kLanes == 1 && rows < 16) {
#pragma unroll 2
      for (int p = 0; p < rows; ++p) s += *reinterpret_cast<const f32x4*>(src + p * width + i);
    } else {
#pragma unroll 8
      for (int p = rl; p < rows; p += kLanes) s += *reinterpret_cast<const f32x4*>(src + p * width + i);
    }
  }
  if constexpr (kLanes > 1) {
    if (rl > 0) *reinterpret_cast<f32x4*>(red + 4 * ((rl - 1) * kCols + cl)) = s;
    __syncthreads();
    if (rl > 0) return;
#pragma unroll
    for (int l = 0; l < kLanes - 1; ++l) s += *reinterpret_cast<const f32x4*>(red + 4 * (l * kCols + cl));
  }
  if (i >= width) return;
  u16 o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = __builtin_bit_cast(u16, (__bf16)s[e]);
  *reinterpret_cast<u32x2*>(dst + i) = u32x2{o[0] | (static_cast<unsigned>(o[1]) << 16),
                                             o[2] | (static_cast<unsigned>(o[3]) << 16)};
}

// dw from the partials; the workgroups from dw_blocks on make db from its rows.
constexpr int kDbLanes = 8;
template <int kLanes>
__global__ __launch_bounds__(kWgThreads) void wgrad_sum(const float* part, u16* dw, int64_t mn, int splits,
                                                        const float* db_part, u16* db, int M, int R, int dw_blocks) {
  __shared__ __attribute__((aligned(16))) float red[kWgThreads * 4];
  const int blk = __builtin_amdgcn_workgroup_id_x();
  if (blk < dw_blocks) sum_rows<kLanes>(part, dw, mn, splits, blk, red);
  else sum_rows<kDbLanes>(db_part, db, M, R, blk - dw_blocks, red);
}

}  // namespace

// Rows of M floats kept for the column sums: one per 256 rows of dy, at most 1024.
static int64_t db_rows(int64_t K) {
  if (K <= 0) return 0;
  const int64_t R = std::min<int64_t>(1024, (K + 255) / 256);
  const int64_t rows = (K + R - 1) / R;
  return (K + rows - 1) / rows;
}

// Splits of the reduction: at most 512 workgroups in all (two per compute
// unit, as 64 KiB of LDS per workgroup allows) unless the output alone has
// more tiles, each split a whole number of k tiles and `least` rows if there
// are that many; no split for K = 0 (dW is then zero).
static int64_t splits_of(int64_t K, int64_t M, int64_t N, int64_t least, int64_t* chunk) {
  *chunk = 0;
  if (K <= 0) return 0;
  const int64_t tiles = (M / kTileMN) * (N / kTileMN);
  const int64_t ktiles = (K + kTileK - 1) / kTileK;
  const int64_t s = std::max<int64_t>(1, std::min<int64_t>(512 / tiles, ktiles * kTileK / least));
  *chunk = (ktiles + s - 1) / s * kTileK;
  return (K + *chunk - 1) / *chunk;
}

// 256 rows per split at least: a split costs a partial output, written and
// read, and for small outputs the sum over many of them is a long chain (K =
// 32768, M = N = 128: 144 us for a call with its 512 splits of 64 rows, 17 us with 128).
int64_t wgrad_splits(int64_t K, int64_t M, int64_t N, int64_t* chunk) { return splits_of(K, M, N, 256, chunk); }

// Room for splits of a single k tile, of which wgrad_splits never has more.
uint64_t wgrad_workspace(int64_t K, int64_t M, int64_t N) {
  int64_t chunk = 0;
  return static_cast<uint64_t>(splits_of(K, M, N, kTileK, &chunk) * N + db_rows(K)) * M * 4;
}

hipError_t launch_wgrad(const void* dy, const void* x, void* dw, void* db, int64_t K, int64_t M, int64_t N,
                        void* workspace, hipStream_t stream) {
  int64_t chunk = 0;
  const int64_t splits = wgrad_splits(K, M, N, &chunk);
  WgradArgs a;
  a.dy = static_cast<const u16*>(dy);
  a.x = static_cast<const u16*>(x);
  a.part = static_cast<float*>(workspace);
  a.K = K;
  a.M = static_cast<int32_t>(M);
  a.N = static_cast<int32_t>(N);
  a.chunk = static_cast<int32_t>(chunk);
  a.tiles_n = static_cast<int32_t>(N / kTileMN);
  a.tiles = static_cast<int32_t>((M / kTileMN) * (N / kTileMN));
  a.items = static_cast<int32_t>(a.tiles * splits);
  a.per_xcd = (a.items + 7) / 8;
  // every split has a row of its own for the column sums at least (the splits
  // are at most K / 256, or one)
  a.db_part = a.part + splits * M * N;
  a.db_share = splits > 0 ? static_cast<int32_t>(std::min<int64_t>(a.tiles_n, db_rows(K) / splits)) : 0;
  const dim3 grid(static_cast<unsigned>(8 * a.per_xcd));
  if (splits > 0) {
    if (db) hipLaunchKernelGGL(wgrad_partial<true>, grid, dim3(kWgThreads), 0, stream, a);
    else hipLaunchKernelGGL(wgrad_partial<false>, grid, dim3(kWgThreads), 0, stream, a);
  }
  // K = 0: no partials, the sums below write zeros
  const int64_t mn = M * N;
  // One thread sums all splits of its columns where that makes 256 workgroups
  // (768 x 768, 14 splits: 6.3 us, 8.3 with four), four threads below that.
  const int lanes = mn >= 256 * 4 * kWgThreads ? 1 : 4;
  const int dw_blocks = static_cast<int>((mn * lanes + 4 * kWgThreads - 1) / (4 * kWgThreads));
  const int db_blocks = db ? static_cast<int>((M * kDbLanes + 4 * kWgThreads - 1) / (4 * kWgThreads)) : 0;
  hipLaunchKernelGGL(lanes == 1 ? wgrad_sum<1> : wgrad_sum<4>, dim3(static_cast<unsigned>(dw_blocks + db_blocks)),
                     dim3(kWgThreads), 0, stream, static_cast<const float*>(a.part), static_cast<u16*>(dw), mn,
                     static_cast<int>(splits), static_cast<const float*>(a.db_part), static_cast<u16*>(db),
                     static_cast<int>(M), static_cast<int>(splits * a.db_share), dw_blocks);
  return hipGetLastError();
}

}  // namespace da
