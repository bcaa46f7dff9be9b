// Wavelet analysis behind the method (Sections 3.2-3.3): how much of the information gathered by attention,
// s[n] = a[n] * v[n], sits in each Haar frequency band, position by position.
//
// For the Haar pair the reconstruction from one level's detail coefficients alone has a closed form: over a block
// of 2^l positions Rec(D_l) is +-2^-l * (sum of the block's first half - sum of its second half), so its magnitude
// is one number per block and column.  The multi-level decomposition is therefore a tree of pairwise sums over 32
// consecutive rows (five levels), and the kernel is one streaming read of V: a wave takes 32 rows, a lane 16 bytes
// of a few consecutive rows (the low levels stay inside the lane, the top ones cross lanes by shuffles), the
// magnitudes are averaged over the d columns (lane-local, then across the lanes that share a row) and leave
// through a small LDS tile as whole rows of the output.
//
//   wavelet_components_kernel   grid (ceil(t / 128), heads) x 256 threads -> per_head [heads][levels][t]
//   wavelet_mean_kernel         a workgroup per 16 (32) outputs x 512 (1024) threads -> mean [levels][t], heads added in a fixed order

#include "treekv_internal.h"

namespace tkv {
namespace {

constexpr int WV_THREADS = 256;
constexpr int WV_WAVES = WV_THREADS / 64;
constexpr int WV_BLOCK = 32;          // rows per wave pass = 2^5, the deepest level
constexpr int WV_LEVELS = 5;

template <int N> struct IntTag { static constexpr int value = N; };

// The value of this lane and of the lane STRIDE away (index xor STRIDE), without LDS where the chip can swap lane rows.
template <int STRIDE>
__device__ inline float2 lane_pair(float v) {
  if constexpr (STRIDE == 16 || STRIDE == 32) {
    const unsigned x = __float_as_uint(v);
    const auto r = STRIDE == 16 ? __builtin_amdgcn_permlane16_swap(x, x, false, false)
                                : __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1]));
  } else {
    return make_float2(v, __shfl_xor(v, STRIDE, 64));
  }
}

constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x / 2); }

// Bound by the read of V.  What hides its latency is waves, not requests ahead within one: a wave takes one 32-row block,
// registers are capped for 6 waves per SIMD (2 for 512-byte rows, whose lanes hold 16 rows each), V is read with the
// non-temporal hint, and lanes exchange through DPP and row swaps instead of LDS.  8192 heads x 512 x 128 bf16, 5 levels:
// 188 us = 6.2 TB/s; with four blocks per wave and the next one requested ahead, 3 waves per SIMD, 230 us (212 at 4 waves,
// 201 with the hint and without LDS exchanges, 196 with two blocks per wave).
template <typename T, int D>
__global__ __launch_bounds__(WV_THREADS, sizeof(T) * D > 256 ? 2 : 6) void wavelet_components_kernel(const float* __restrict__ a,
                                                                        const T* __restrict__ V, int t, int levels,
                                                                        float* __restrict__ per_head) {
  constexpr int EPL = Storage<T>::EPL;
  constexpr int LPR = D / EPL;            // lanes that share a row
  constexpr int RG = 64 / LPR;            // row groups of a wave
  constexpr int RPLN = WV_BLOCK / RG;     // consecutive rows of one lane
  constexpr int IN = ilog2(RPLN);         // levels that stay inside a lane
  static_assert(RG * RPLN == WV_BLOCK && (1 << IN) == RPLN && IN >= 1 && IN < WV_LEVELS, "shape");
  __shared__ float tile[WV_WAVES][WV_LEVELS][WV_BLOCK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane % LPR, ri = lane / LPR;
  const int head = blockIdx.y;
  const T* Vh = V + (size_t)head * t * D;
  const float* ah = a + (size_t)head * t;
  const int base = (blockIdx.x * WV_WAVES + wave) * WV_BLOCK;      // wave uniform
  if (base >= t) return;

  // 16 bytes of V and the weight of each of the lane's rows, all requested at once
  uint4 raw[RPLN];
  float w[RPLN];
#pragma unroll
  for (int j = 0; j < RPLN; ++j) {
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    const int row = base + ri * RPLN + j, rc = min(row, t - 1);
    const v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(Vh + (size_t)rc * D + li * EPL));
    raw[j] = make_uint4(v.x, v.y, v.z, v.w);
    w[j] = row < t ? ah[rc] : 0.f;                               // rows past the end count as zero
  }
  // s = a o V for this lane's rows and columns
  float x[RPLN][EPL];
#pragma unroll
  for (int j = 0; j < RPLN; ++j) {
    float vf[EPL];
    Storage<T>::widen(raw[j], vf);
#pragma unroll
    for (int e = 0; e < EPL; ++e) x[j][e] = w[j] * vf[e];
  }
  // levels inside the lane: pairwise differences and sums; |difference| added over the lane's columns
  float mag_in[RPLN];                 // RPLN >> l entries per level l = 1.., one level after the other
#pragma unroll
  for (int i = 0; i < RPLN; ++i) mag_in[i] = 0.f;
  float top[EPL];                     // sum of the lane's rows, per column
#pragma unroll
  for (int e = 0; e < EPL; ++e) {
    float s[RPLN];
#pragma unroll
    for (int j = 0; j < RPLN; ++j) s[j] = x[j][e];
    int off = 0;
#pragma unroll
    for (int l = 1; l <= IN; ++l) {
      const int n = RPLN >> l;
#pragma unroll
      for (int m = 0; m < n; ++m) {
        const float lo = s[2 * m], hi = s[2 * m + 1];
        mag_in[off + m] += fabsf(lo - hi);
        s[m] = lo + hi;
      }
      off += n;
    }
    top[e] = s[0];
  }
  // levels across row groups
  float mag_x[WV_LEVELS - IN];
  auto cross = [&](auto level) {
    constexpr int l = decltype(level)::value;
    if constexpr (l < WV_LEVELS - IN) {
      float acc = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const float2 h = lane_pair<(LPR << l)>(top[e]);
        acc += fabsf(h.x - h.y);
        top[e] = h.x + h.y;
      }
      mag_x[l] = acc;
    }
  };
  cross(IntTag<0>{}); cross(IntTag<1>{}); cross(IntTag<2>{}); cross(IntTag<3>{});
  // add over the lanes that share the rows
#pragma unroll
  for (int i = 0; i < RPLN - 1; ++i) mag_in[i] = group_sum<LPR>(mag_in[i]);
#pragma unroll
  for (int l = 0; l < WV_LEVELS - IN; ++l) mag_x[l] = group_sum<LPR>(mag_x[l]);
  // |Rec(D_l)| = 2^-l |first half - second half|, the same for all 2^l rows of the block; mean over the D columns
  if (li == 0) {
    int off = 0;
#pragma unroll
    for (int l = 1; l <= IN; ++l) {
      const int n = RPLN >> l;
      const float f = 1.0f / (float)((1 << l) * D);
#pragma unroll
      for (int m = 0; m < n; ++m)
#pragma unroll
        for (int r = 0; r < (1 << l); ++r) tile[wave][l - 1][ri * RPLN + (m << l) + r] = mag_in[off + m] * f;
      off += n;
    }
#pragma unroll
    for (int l = 0; l < WV_LEVELS - IN; ++l) {
      const float f = 1.0f / (float)((1 << (IN + 1 + l)) * D);
#pragma unroll
      for (int r = 0; r < RPLN; ++r) tile[wave][IN + l][ri * RPLN + r] = mag_x[l] * f;
    }
  }
  // the tile is this wave's own: written and read by the same wave, in program order
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (int i = lane; i < levels * WV_BLOCK; i += 64) {
    const int l = i / WV_BLOCK, r = i % WV_BLOCK;
    if (base + r < t) per_head[((size_t)head * levels + l) * t + base + r] = tile[wave][l][r];
  }
}

// Mean over the heads: a workgroup owns 16 or 32 adjacent outputs and adds up the heads of every output in
// an order that depends on nothing but `heads`: 128 head lanes take every 128th head each, eight lanes' sums go up a tree,
// the 16 results are added one after the other.
//   QUADS   a thread is one head lane of four outputs (16-byte loads), the tree is lane exchanges.
//   else    (per_head not 16-byte aligned, or rows that are no whole groups of four outputs) a thread is four head lanes of
//           one output, the tree goes through LDS.
// Bound by the bytes in flight and by what still is in the memory-side cache (the components kernel reads V past it): with
// 16-byte loads, 16 of them per thread, and half a 128-byte line per workgroup, so that 5 levels of 512 give 160 of them, the
// two halves of a line on one XCD.  A whole call at 8192 heads x 512: 207-210 us (209-213 with whole lines), 64 wide 115.8
// (118.0), 64 heads x 96 5.4 (5.4); quarters of a line were slower than whole ones (215.5 and 210.6, 64 wide 126.4 and 120.0).
// The kernel alone took 35 us with 4-byte loads, 22 with whole lines, 20 now.
constexpr int MEAN_LANES = 128;
template <bool QUADS>
struct Mean {
  static constexpr int COLS = QUADS ? 16 : 32, THREADS = MEAN_LANES * COLS / 4;
  static constexpr int SHARE = 32 / COLS;            // workgroups that read the same 128-byte lines
};
template <bool QUADS>
__global__ __launch_bounds__(Mean<QUADS>::THREADS) void wavelet_mean_kernel(const float* __restrict__ per_head, int heads, int n,
                                                                    float* __restrict__ mean) {
  constexpr int GROUPS = MEAN_LANES / 8, MEAN_COLS = Mean<QUADS>::COLS, MEAN_THREADS = Mean<QUADS>::THREADS;
  constexpr int SHARE = Mean<QUADS>::SHARE;
  __shared__ float red[GROUPS][MEAN_COLS];
  // workgroups are dealt to the 8 XCDs in turn: those that share lines get ids 8 apart, so one of them brings the line in
  const int w = blockIdx.x, line = w / (8 * SHARE) * 8 + w % 8;
  const int tid = threadIdx.x, first = line * 32 + w / 8 % SHARE * MEAN_COLS;
  if constexpr (QUADS) {
    constexpr int TX = MEAN_COLS / 4;
    const int tx = tid % TX, lane = tid / TX, i = first + tx * 4;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    if (i < n) {
#pragma unroll 16
      for (int h = lane; h < heads; h += MEAN_LANES) {
        const float4 v = *reinterpret_cast<const float4*>(per_head + (size_t)h * n + i);
        acc[0] += v.x; acc[1] += v.y; acc[2] += v.z; acc[3] += v.w;
      }
    }
#pragma unroll
    for (int o = TX; o < 8 * TX; o <<= 1)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
    if (tid % (8 * TX) < TX) {
#pragma unroll
      for (int e = 0; e < 4; ++e) red[tid / (8 * TX)][tx * 4 + e] = acc[e];
    }
  } else {
    constexpr int STEP = MEAN_THREADS / MEAN_COLS;
    __shared__ float sums[MEAN_LANES][MEAN_COLS];
    const int tx = tid % MEAN_COLS, ty = tid / MEAN_COLS;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};                 // head lanes ty, ty + 32, ty + 64, ty + 96
    if (first + tx < n) {
      const float* src = per_head + first + tx;
      int h = ty;
#pragma unroll 4
      for (; h + 3 * STEP < heads; h += MEAN_LANES)
#pragma unroll
        for (int y = 0; y < 4; ++y) acc[y] += src[(size_t)(h + y * STEP) * n];
#pragma unroll
      for (int y = 0; y < 3; ++y)
        if (h + y * STEP < heads) acc[y] += src[(size_t)(h + y * STEP) * n];
    }
#pragma unroll
    for (int y = 0; y < 4; ++y) sums[ty + y * STEP][tx] = acc[y];
    __syncthreads();
    if (tid < GROUPS * MEAN_COLS) {
      float s[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) s[k] = sums[ty * 8 + k][tx];
      red[ty][tx] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    }
  }
  __syncthreads();
  if (tid < MEAN_COLS && first + tid < n) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < GROUPS; ++w) sum += red[w][tid];
    mean[first + tid] = sum / (float)heads;
  }
}

template <typename T, int D>
void launch_components(const float* a, const void* V, int heads, int t, int levels, float* per_head, hipStream_t s) {
  const int rows = WV_BLOCK * WV_WAVES;
  const int blocks = (t + rows - 1) / rows;
  hipLaunchKernelGGL((wavelet_components_kernel<T, D>), dim3(blocks, heads), dim3(WV_THREADS), 0, s, a, (const T*)V, t,
                     levels, per_head);
}

}  // namespace

int launch_wavelet(const float* a, const void* V, int dtype, int heads, int t, int d, int levels, float* per_head,
                   float* mean, hipStream_t s) {
  if (dtype == TREEKV_BF16 && d == 128) launch_components<uint16_t, 128>(a, V, heads, t, levels, per_head, s);
  else if (dtype == TREEKV_BF16 && d == 64) launch_components<uint16_t, 64>(a, V, heads, t, levels, per_head, s);
  else if (dtype == TREEKV_F32 && d == 128) launch_components<float, 128>(a, V, heads, t, levels, per_head, s);
  else if (dtype == TREEKV_F32 && d == 64) launch_components<float, 64>(a, V, heads, t, levels, per_head, s);
  else return TREEKV_EUNSUPPORTED;
  if (mean) {
    const int n = levels * t;
    // 16-byte loads need whole groups of four outputs in every head's row
    const int lines = (n + 31) / 32;
    if (n % 4 == 0 && (reinterpret_cast<uintptr_t>(per_head) & 15) == 0)
      hipLaunchKernelGGL(wavelet_mean_kernel<true>, dim3((lines + 7) / 8 * 8 * Mean<true>::SHARE), dim3(Mean<true>::THREADS), 0, s,
                         per_head, heads, n, mean);
    else
      hipLaunchKernelGGL(wavelet_mean_kernel<false>, dim3((lines + 7) / 8 * 8), dim3(Mean<false>::THREADS), 0, s, per_head, heads, n, mean);
  }
  return finish_launch();
}

}  // namespace tkv
