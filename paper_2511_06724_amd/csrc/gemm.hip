// MFMA GEMM with an implicit-convolution A loader (gfx950).
//
// One kernel template covers every dense contraction of the UNet: the 3x3
// convolutions (implicit GEMM over NHWC activations, with stride-2 downsample,
// nearest-x2 upsample addressing and two-source channel concatenation), the
// 1x1 skip convolutions and every linear layer of the transformer blocks
// (fused QKV, attention outputs, GEGLU feed-forward, projections).
//
// Tiling: 256 threads = 4 waves in a 2x2 grid; block tile BM x BN in
// {128x128, 64x64}, wave tile (BM/2) x (BN/2) built from 32x32x16 MFMA blocks; K
// step BK = 128 bytes of each row (64 bf16 / 32 fp32), staged through
// double-buffered LDS (one barrier per K step; the next tile's global loads are
// issued a full K step ahead). The MFMA is issued as C^T = B A^T so that each
// lane holds four consecutive output columns of one row: the epilogue stores
// 8 (bf16) or 16 (fp32) contiguous bytes per lane and reads bias / residual as
// vectors. Rows of A and B beyond M / N are clamped on load and masked on store.
//
// Work distribution: tiles are numbered so that each XCD (consecutive
// workgroup ids go round-robin over the 8 XCDs) works through a contiguous band
// of output columns with all row tiles, keeping that band of B in its L2.
#include <algorithm>
#include <cmath>

#include "gemm_epilogue.h"

namespace dn {
namespace {

constexpr int kThreads = 256;
constexpr int kXcds = 8;

template <typename T, int BM, int BN, bool CONV>
__global__ __launch_bounds__(kThreads) void gemm_kernel(GemmParams p, int mt, int nt) {
  using MM = Mma<T>;
  constexpr int VEC = 16 / sizeof(T);
  constexpr int BK = gemm_bk<T>();
  constexpr int VPR = BK / VEC;          // 16-byte vectors per tile row (8)
  constexpr int SA = BK + VEC;           // LDS row stride in elements (16-byte pad)
  constexpr int RPP = kThreads / VPR;    // tile rows covered by one pass of the block (32)
  constexpr int AV = BM / RPP;
  constexpr int BV = BN / RPP;
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int FM = WM / 32, FN = WN / 32;
  constexpr int STAGE = (BM + BN) * SA;

  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* lds = reinterpret_cast<T*>(smem_raw);

  // ---- tile assignment (XCD-aware: each XCD walks a contiguous band of columns)
  const int total = mt * nt;
  const int wg = blockIdx.x;
  const int xcd = wg % kXcds, idx = wg / kXcds;
  const int base = total / kXcds, rem = total % kXcds;
  const int logical = xcd * base + min(xcd, rem) + idx;
  const int n_tile = logical / mt;
  const int m_tile = logical - n_tile * mt;
  const int n0 = n_tile * BN;
  const int m0 = m_tile * BM;
  const int kt_begin = 0;
  const int kt_end = p.K / BK;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int vc = tid % VPR;
  const int rr = tid / VPR;

  // Per-thread A row descriptors.
  int a_row[AV];
  int a_sy[AV], a_oy[AV], a_ox[AV];
  const int opix = p.out_h * p.out_w;
#pragma unroll
  for (int i = 0; i < AV; ++i) {
    const int m = min(m0 + rr + i * RPP, p.M - 1);
    a_row[i] = m;
    if (CONV) {
      const int s = m / opix;
      const int rem2 = m - s * opix;
      const int oy = rem2 / p.out_w;
      const int ox = rem2 - oy * p.out_w;
      a_sy[i] = s * p.in_h;
      a_oy[i] = oy * p.stride - 1;
      a_ox[i] = ox * p.stride - 1;
    }
  }
  const T* b_ptr[BV];
#pragma unroll
  for (int i = 0; i < BV; ++i) {
    const int n = min(n0 + rr + i * RPP, p.N - 1);
    b_ptr[i] = static_cast<const T*>(p.b) + (long long)n * p.ldb + vc * VEC;
  }

  uint4 ra[AV], rb[BV];
  const int ct = p.c0 + p.c1;
  const int hl = p.in_h << p.up, wl = p.in_w << p.up;

  auto load_tile = [&](int k0) {
    int tap = 0, c = k0;
    if (CONV) {
      tap = k0 / ct;
      c = k0 - tap * ct;
    }
    const T* src;
    int ld;
    if (c < p.c0) {
      src = static_cast<const T*>(p.a0);
      ld = p.lda0;
    } else {
      src = static_cast<const T*>(p.a1);
      ld = p.lda1;
      c -= p.c0;
    }
    c += vc * VEC;
    if (CONV) {
      const int ky = tap / 3, kx = tap - 3 * (tap / 3);
#pragma unroll
      for (int i = 0; i < AV; ++i) {
        const int iy = a_oy[i] + ky, ix = a_ox[i] + kx;
        if (iy >= 0 && iy < hl && ix >= 0 && ix < wl) {
          const long long pix = (long long)(a_sy[i] + (iy >> p.up)) * p.in_w + (ix >> p.up);
          ra[i] = ld16(src + pix * ld + c);
        } else {
          ra[i] = make_uint4(0u, 0u, 0u, 0u);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < AV; ++i) ra[i] = ld16(src + (long long)a_row[i] * ld + c);
    }
#pragma unroll
    for (int i = 0; i < BV; ++i) rb[i] = ld16(b_ptr[i] + k0);
  };
  auto store_tile = [&](int buf) {
    T* As = lds + buf * STAGE;
    T* Bs = As + BM * SA;
#pragma unroll
    for (int i = 0; i < AV; ++i) st16(As + (rr + i * RPP) * SA + vc * VEC, ra[i]);
#pragma unroll
    for (int i = 0; i < BV; ++i) st16(Bs + (rr + i * RPP) * SA + vc * VEC, rb[i]);
  };

  // acc[i][j]: rows = output columns n0 + wn*WN + 32 j + acc_row(r),
  //            column = output row m0 + wm*WM + 32 i + (lane % 32).
  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int frag_off = (lane & 31) * SA + (lane >> 5) * MM::KPL;
  if (kt_begin < kt_end) {
    load_tile(kt_begin * BK);
    store_tile(0);
    if (kt_begin + 1 < kt_end) load_tile((kt_begin + 1) * BK);
    __syncthreads();
    for (int kt = kt_begin; kt < kt_end; ++kt) {
      const int cur = (kt - kt_begin) & 1;
      const T* As = lds + cur * STAGE + wm * WM * SA + frag_off;
      const T* Bs = lds + cur * STAGE + BM * SA + wn * WN * SA + frag_off;
#pragma unroll
      for (int ks = 0; ks < BK / MM::KS; ++ks) {
        typename MM::frag a[FM], b[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i) a[i] = MM::load(As + i * 32 * SA + ks * MM::KS);
#pragma unroll
        for (int j = 0; j < FN; ++j) b[j] = MM::load(Bs + j * 32 * SA + ks * MM::KS);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) acc[i][j] = MM::mma(b[j], a[i], acc[i][j]);
      }
      if (kt + 1 < kt_end) {
        store_tile(cur ^ 1);
        if (kt + 2 < kt_end) load_tile((kt + 2) * BK);
      }
      __syncthreads();
    }
  }

  const int col = lane & 31;
  const int h4 = 4 * (lane >> 5);

  // ---- epilogue
  if (!p.geglu) {
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int m = m0 + wm * WM + i * 32 + col;
      if (m >= p.M) continue;
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int n = n0 + wn * WN + j * 32 + 8 * g + h4;
          float v[4] = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
          epilogue_group<T>(p, m, n, v);
        }
    }
  } else {
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int m = m0 + wm * WM + i * 32 + col;
      if (m >= p.M) continue;
#pragma unroll
      for (int j = 0; j < FN / 2; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int nv = n0 + wn * WN + 2 * j * 32 + 8 * g + h4;   // value column (gate = nv + 32)
          const int o = (n0 + wn * WN) / 2 + j * 32 + 8 * g + h4;  // output column
          if (o >= p.n_store) continue;
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float a = acc[i][2 * j][4 * g + e] + (p.bias ? p.bias[nv + e] : 0.f);
            const float gg = acc[i][2 * j + 1][4 * g + e] + (p.bias ? p.bias[nv + 32 + e] : 0.f);
            v[e] = a * gelu_erf(gg);
          }
          store4<T>(p, m, o, v, p.n_store);
        }
    }
  }
}

template <typename T, int BM, int BN, bool CONV>
void launch(const GemmParams& p, hipStream_t s) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int SA = gemm_bk<T>() + VEC;
  const size_t lds = size_t(2) * (BM + BN) * SA * sizeof(T);
  static bool attr_set = false;
  if (!attr_set) {
    DN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_kernel<T, BM, BN, CONV>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    attr_set = true;
  }
  const int mt = ceil_div(p.M, BM), nt = ceil_div(p.N, BN);
  hipLaunchKernelGGL((gemm_kernel<T, BM, BN, CONV>), dim3(mt * nt), dim3(kThreads), lds, s, p, mt, nt);
  DN_HIP(hipGetLastError());
}

// fp32 GEMM for grids too small to fill the chip: a workgroup owns one 32 x 32 tile (with
// GEGLU, 32 value and the matching 32 gate columns) and its eight waves split K. Bound by
// latency, not by rate: 512 x 64 x 576 (a 3x3 convolution of the 16 x 16 denoiser) is 8 tiles
// of 64 x 64, whose four waves walk K alone (21.4 us per launch); 32 tiles of eight waves each
// run an eighth of K (10.2 us; GEGLU 512 x 2 x 256 x 64 13.0 -> 9.1 us).
// Operands come straight from global memory: lane l takes four consecutive k (16 bytes) at
// 4 (l / 32) of an 8-deep step for row l % 32 of A and of B, and MFMA e of the step contracts
// component e of both (any k order common to both operands gives the same sum). Two sets of
// kWsSteps steps, the next loaded while the current one is multiplied. The partial tiles meet
// in LDS in wave order (deterministic).
constexpr int kWsWaves = 8, kWsSteps = 3;

template <bool CONV, int NB>
__global__ __launch_bounds__(64 * kWsWaves) void gemm_wavesplit_kernel(GemmParams p, int mt) {
  using MM = Mma<float>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float* red = reinterpret_cast<float*>(smem_raw);  // [wave][NB][16][64]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_tile = blockIdx.x / mt, m_tile = blockIdx.x - n_tile * mt;
  const int m0 = m_tile * 32, n0 = n_tile * 32 * NB;
  const int k4 = 4 * (lane >> 5);
  const int m = min(m0 + (lane & 31), p.M - 1);
  const float* bp[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
    bp[j] = static_cast<const float*>(p.b) + (long long)min(n0 + 32 * j + (lane & 31), p.N - 1) * p.ldb + k4;
  const int ct = p.c0 + p.c1;
  int smp = 0, iy0 = 0, ix0 = 0;
  const int hl = p.in_h << p.up, wl = p.in_w << p.up;
  if (CONV) {
    const int opix = p.out_h * p.out_w;
    smp = m / opix;
    const int r2 = m - smp * opix, oy = r2 / p.out_w;
    iy0 = oy * p.stride - 1;
    ix0 = (r2 - oy * p.out_w) * p.stride - 1;
  }
  const int ns = p.K / 8;
  const int s0 = ns * wave / kWsWaves, s1 = ns * (wave + 1) / kWsWaves;
  // the wave's steps past s1 read its last step again and are not multiplied
  auto load = [&](int st, f32x4& a, f32x4 (&b)[NB]) {
    const int k = 8 * min(st, s1 - 1);
    int tap = 0, c = k;
    if (CONV) {
      tap = k / ct;
      c = k - tap * ct;
    }
    const bool first = c < p.c0;
    const float* src = static_cast<const float*>(first ? p.a0 : p.a1);
    const int ld = first ? p.lda0 : p.lda1, cc = (first ? c : c - p.c0) + k4;
    if (CONV) {
      const int ky = tap / 3, iy = iy0 + ky, ix = ix0 + tap - 3 * ky;
      const bool in = iy >= 0 && iy < hl && ix >= 0 && ix < wl;
      const long long pix = in ? (long long)(smp * p.in_h + (iy >> p.up)) * p.in_w + (ix >> p.up) : 0;
      const f32x4 v = *reinterpret_cast<const f32x4*>(src + pix * ld + cc);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = in ? v[e] : 0.f;
    } else {
      a = *reinterpret_cast<const f32x4*>(src + (long long)m * ld + cc);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) b[j] = *reinterpret_cast<const f32x4*>(bp[j] + k);
  };
  f32x16 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  if (s0 < s1) {
    f32x4 a[2][kWsSteps], b[2][kWsSteps][NB];
    auto load_set = [&](int st, int u) {
#pragma unroll
      for (int t = 0; t < kWsSteps; ++t) load(st + t, a[u][t], b[u][t]);
    };
    auto mma_set = [&](int st, int u) {
#pragma unroll
      for (int t = 0; t < kWsSteps; ++t)
        if (st + t < s1) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[j] = MM::mma(b[u][t][j][e], a[u][t][e], acc[j]);
        }
    };
    load_set(s0, 0);
    for (int st = s0; st < s1; st += 2 * kWsSteps) {
      load_set(st + kWsSteps, 1);
      mma_set(st, 0);
      load_set(st + 2 * kWsSteps, 0);
      mma_set(st + kWsSteps, 1);
    }
  }
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) red[((wave * NB + j) * 16 + r) * 64 + lane] = acc[j][r];
  __syncthreads();
  // thread: four columns 8 g + 4 (l / 32) .. of row l % 32
  if (threadIdx.x >= 256) return;
  const int g = threadIdx.x >> 6, h4 = 4 * (lane >> 5);
  float v[NB][4];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = red[(j * 16 + 4 * g + e) * 64 + lane];
#pragma unroll
      for (int w = 1; w < kWsWaves; ++w) x += red[((w * NB + j) * 16 + 4 * g + e) * 64 + lane];
      v[j][e] = x;
    }
  const int row = m0 + (lane & 31);
  if (row >= p.M) return;
  if constexpr (NB == 2) {
    const int nv = n0 + 8 * g + h4, o = n0 / 2 + 8 * g + h4;  // value column (gate 32 further), output column
    if (o >= p.n_store) return;
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      y[e] = (v[0][e] + (p.bias ? p.bias[nv + e] : 0.f)) * gelu_erf(v[NB - 1][e] + (p.bias ? p.bias[nv + 32 + e] : 0.f));
    store4<float>(p, row, o, y, p.n_store);
  } else {
    epilogue_group<float>(p, row, n0 + 8 * g + h4, v[0]);
  }
}

template <bool CONV, int NB> void launch_wavesplit(const GemmParams& p, hipStream_t s) {
  const int mt = ceil_div(p.M, 32), nt = ceil_div(p.N, 32 * NB);
  const size_t lds = sizeof(float) * kWsWaves * NB * 16 * 64;
  static bool attr_set = false;
  if (!attr_set) {
    DN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_wavesplit_kernel<CONV, NB>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    attr_set = true;
  }
  hipLaunchKernelGGL((gemm_wavesplit_kernel<CONV, NB>), dim3(mt * nt), dim3(64 * kWsWaves), lds, s, p, mt);
  DN_HIP(hipGetLastError());
}

template <typename T, bool CONV> void dispatch(const GemmParams& p, const GemmPlan& g, hipStream_t s) {
  if constexpr (sizeof(T) == 4) {
    if (g.bm == 32) {
      if (p.geglu)
        launch_wavesplit<CONV, 2>(p, s);
      else
        launch_wavesplit<CONV, 1>(p, s);
      return;
    }
  }
  if (g.bm == 64 && g.bn == 64)
    launch<T, 64, 64, CONV>(p, s);
  else
    launch<T, 128, 128, CONV>(p, s);
}

}  // namespace

// Fragment-B kernels: tile, split and tail bands by a cost model fitted to launches measured
// on MI355X (every tile and split of some 800 shapes; weights from HBM, activations as the launch
// before leaves them). A tile variant runs up to `wg` workgroups per CU; with c of them on the
// busiest CU a K stage (64 bf16 or 128 fp8 values) takes stage[c - 1] us, so a round of units
// costs fixed + wgcost c + stages x stage[c - 1], a grid is its full rounds plus the
// remainder's round, and the outputs cost per_mb us per MB written (an fp32 output also reads
// its residual). In bf16 a stage's time nearly doubles with a second workgroup on the CU (a
// 128 x 256 linear tile 0.68 -> 1.41 us), so that filling a round's second half costs about as
// much as its first; in fp8 it hardly grows (0.78 -> 1.06). Splitting K adds the reduction
// launch (reduce us) and its slab traffic (at reduce_mb MB / us), or, when a LayerNorm sums the
// slabs, that kernel's extra reads. The chosen plan against the best one: 0.4 to 0.5 % in the
// mean for linear layers (332 shapes), V^T (122), convolutions (215) and fp8 (135).
struct TileCost {
  int bm, bn, x5, wg;
  double fixed, wgcost, stage[4], per_mb;
};
static const TileCost kLinCost[] = {{128, 256, 0, 2, 5.2, 0.0, {0.684, 1.408}, 0.068},
                                    {128, 128, 0, 2, 2.9, 0.0, {0.468, 0.953}, 0.114},
                                    {64, 128, 0, 4, 1.6, 0.14, {0.310, 0.610, 0.877, 1.172}, 0.145},
                                    {128, 160, 1, 2, 4.5, 0.0, {0.536, 1.083}, 0.094},
                                    {64, 160, 0, 1, 2.3, 0.0, {0.380}, 0.081},
                                    {128, 160, 0, 1, 3.1, 0.0, {0.636}, 0.097}};
// Linear layers with a V^T output (attention input projections): unsplit, not on the four-wave
// 128 x 160 tile, and with V^T's short stores, dearer in the wide tiles. 122 shapes of 128 to
// 16384 rows: 0.4 % from the best plan in the mean; priced as plain linear layers 1.8 %, and
// more where the four-wave tile was chosen and the five-wave one ran
// (12348 x 1536 x 320 54.5 us with V^T as it was then, 37.0 as it is, 27.2 on 64 x 128).
static const TileCost kVtCost[] = {{128, 256, 0, 2, 6.24, 0.0, {0.703, 1.512}, 0.273},
                                   {128, 128, 0, 2, 4.34, 0.0, {0.476, 0.904}, 0.239},
                                   {64, 128, 0, 4, 3.73, 0.0, {0.285, 0.542, 0.869, 1.240}, 0.164},
                                   {64, 160, 0, 1, 4.09, 0.0, {0.378}, 0.0},
                                   {128, 160, 0, 1, 5.02, 0.0, {0.714}, 0.110}};
// Convolutions, upsampling and strided ones among them. A 128 x 256 workgroup alone on a CU takes
// 0.94 us a stage and two together 1.55, so the 2048-row convolutions run as two workgroups per
// CU (six parts, or four of 128 x 160), not as three parts with one: 512 pixels x 1280 x 11520
// upsampled 98.8 -> 82.9 us, 2048 x 1280 x 23040 142 -> 133.
static const TileCost kConvCost[] = {{128, 256, 0, 2, 1.957, 0.0, {0.941, 1.549}, 0.296},
                                     {128, 128, 0, 2, 2.370, 0.0, {0.647, 1.019}, 0.278},
                                     {64, 128, 0, 4, 1.522, 0.034, {0.402, 0.600, 0.962, 1.171}, 0.278},
                                     {128, 160, 1, 2, 3.905, 0.0, {0.662, 1.110}, 0.315}};
// fp8: 16384 x 320 x 1280 as 128 x 128 tiles (20.5 us; 24.0 as 128 x 256), 1152 x 320 x 1280
// in three parts (11.1; 11.9 whole), 2048 rows whole (12.0; 13.0 in two parts).
static const TileCost kFp8Cost[] = {{128, 256, 0, 2, 7.559, 0.0, {0.928, 1.185}, 0.144},
                                    {128, 128, 0, 2, 2.976, 0.0, {0.675, 0.765}, 0.267}};

// by PlanKind; reduce in us, reduce_mb in us per MB (slabs read, outputs written)
struct PlanCost {
  const TileCost* tiles;
  int n;
  double reduce, reduce_mb;
};
static const PlanCost kPlanCost[] = {{kLinCost, 6, 3.5, 1 / 6.0},
                                     {kVtCost, 5, 0.0, 0.0},  // never split
                                     {kConvCost, 4, 5.745, 0.011},
                                     {kFp8Cost, 2, 2.019, 0.206}};

GemmPlan frag_plan(int M, int N, int K, int geglu, int cus, bool fused_reduce, PlanKind kind, bool out_f32) {
  const PlanCost& cost = kPlanCost[kind];
  const int nk = K / (kind == kPlanFp8 ? 128 : 64);
  const int min_stages = kind == kPlanFp8 ? 2 : 4;  // K stages a split part must have
  const double mn = (double)M * N / 1e6;
  GemmPlan best{128, 256};
  best.frag = 1;
  double best_t = 1e300;
  for (int vi = 0; vi < cost.n; ++vi) {
    const TileCost& v = cost.tiles[vi];
    if (geglu && v.bn != 256) continue;  // GEGLU needs 64-column value / gate pairs per wave
    const long long tiles = (long long)ceil_div(M, v.bm) * ceil_div(N, v.bn);
    const long long slots = (long long)cus * v.wg;
    for (int sp = 1; sp <= kMaxSplit; ++sp) {
      if (sp > 1 && (geglu || kind == kPlanVt || nk / sp < min_stages)) break;
      const long long units = tiles * sp, full = units / slots, rem = units % slots;
      const double st = (double)nk / sp;
      double t = full * (v.fixed + v.wgcost * v.wg + st * v.stage[v.wg - 1]);
      if (rem) {
        const int c = static_cast<int>((rem + cus - 1) / cus);
        t += v.fixed + v.wgcost * c + st * v.stage[c - 1];
      }
      if (sp == 1) {
        t += v.per_mb * mn * (geglu ? 1 : out_f32 ? 8 : 2);
      } else {
        t += v.per_mb * mn * 4 * sp;
        t += fused_reduce ? 1.5 + mn * 4 * (sp + 1) / 7.0 : cost.reduce + mn * (4 * sp + (out_f32 ? 8 : 2)) * cost.reduce_mb;
      }
      if (t < best_t) {
        best_t = t;
        best.bm = v.bm;
        best.bn = v.bn;
        best.x5 = v.x5;
        best.split = sp;
      }
    }
  }
  // 128 x 256 linear tiles (two workgroups per CU) with a last round of at most half a tile
  // per CU: its whole column bands run as 64-row tiles, one per CU (FF-in 2048 x 10240 x 1280
  // 54.2 -> 51.2 us, fp8 33.3 -> 29.3). With a tile per CU left over, 64-row tiles only add
  // prologues (4096 x 10240 x 1280 97 -> 112 us).
  if (kind != kPlanConv && best.bm == 128 && best.bn == 256 && best.split == 1) {
    const long long mt = ceil_div(M, 128), nt = ceil_div(N, 256), slots = 2LL * cus;
    const long long tiles = mt * nt, rem = tiles % slots;
    if (rem > 0 && 2 * rem <= cus && rem % mt == 0) {
      const long long bands = rem / mt, tail = (long long)ceil_div(M, 64) * bands;
      if ((tiles - rem) % 8 == 0 && tail % 8 == 0 && bands < nt) best.tail_bands = static_cast<int>(bands);
    }
  }
  return best;
}

// Which fp32 launches take the 32-column tiles whose waves split K. Their operands come straight
// from global memory, so the form pays while a CU gets one workgroup; with more, the other
// workgroups' re-reads cost what the shorter walk gains. Measured (us, 64 x 64 or, with GEGLU,
// 128 x 128 tiles -> these), units being 32-row tiles:
//  - linear, up to one per CU: 512 x 256 x 576 18.4 -> 10.3, 512 x 512 x 5120 124.8 -> 51.1; at
//    K = 64, one step per wave, 5.7 -> 6.2, so from 96 on. Two per CU only for long K and where
//    an operand value meets enough others: 1024 x 512 x 2560 65.3 -> 50.0, but x 64 6.6 -> 11.2,
//    8192 x 64 x 1280 36.6 -> 39.6. Four per CU: 1024 x 960 x 1280 36.1 -> 57.0.
//  - GEGLU, up to one: 512 x 2 x 512 x 64 11.5 -> 8.2; two: x 128 16.0 -> 15.2, x 64 11.6 -> 14.7.
//  - convolutions (whose 64-row tiles wait on their gathers), up to two: 8192 x 64 x 576 21.6 ->
//    17.4; three: 4096 x 192 x 1152 38.2 -> 34.0, x 288 12.9 -> 15.3; 2048 x 448 x 2880 87.8 -> 102.
bool wavesplit(int M, int N, int K, int geglu, bool conv, int cus) {
  const long long units = (long long)ceil_div(M, 32) * ceil_div(N, geglu ? 64 : 32);
  if (conv) return units <= 2ll * cus || (units <= 3ll * cus && K >= 1152);
  if (geglu) return units <= cus || (units <= 2ll * cus && K >= 256);
  if (units <= cus) return K > 64;
  return units <= 2ll * cus && K >= 1024 && (long long)M * N >= 120ll * ((long long)M + N);
}

// Tile choice of the register-staged kernel (fp32, the check mode, and bf16 shapes the
// fragment layout does not take: N % 32 != 0 or K % 64 != 0, e.g. conv_in and the
// output head): 64 x 64 tiles when there are fewer 128 x 128 tiles than CUs (GEGLU
// needs 64-column value/gate pairs per wave, i.e. a block width of at least 128), else
// 128 x 128 tiles with two resident workgroups per CU.
template <typename T>
GemmPlan gemm_plan(int M, int N, int K, int geglu, int cus, bool vt, bool fused_reduce, bool conv,
                   bool out_f32) {
  if (sizeof(T) == 2 && gemm_frag_layout(N, K))
    return frag_plan(M, N, K, geglu, cus, fused_reduce, conv ? kPlanConv : vt ? kPlanVt : kPlanLinear, out_f32);
  if (sizeof(T) == 4 && wavesplit(M, N, K, geglu, conv, cus)) return GemmPlan{32, geglu ? 64 : 32};
  const long long t128 = (long long)ceil_div(M, 128) * ceil_div(N, 128);
  if (!geglu && t128 < cus) return GemmPlan{64, 64};
  return GemmPlan{128, 128};
}

template <typename T> void gemm(const GemmParams& p, const GemmPlan& g, hipStream_t s) {
  constexpr int BK = gemm_bk<T>();
  DN_CHECK(p.M >= 1 && p.N >= 1 && p.K >= BK, "gemm: empty or too small problem");
  DN_CHECK(p.K % BK == 0, "gemm: K must be a multiple of the K tile");
  DN_CHECK(p.taps == 1 || p.taps == 9, "gemm: taps must be 1 or 9");
  DN_CHECK(p.K == p.taps * (p.c0 + p.c1), "gemm: K != taps * channels");
  DN_CHECK(p.c1 == 0 || p.c0 % BK == 0, "gemm: concatenation split must be a multiple of the K tile");
  DN_CHECK(p.taps == 1 || (p.c0 + p.c1) % BK == 0, "gemm: conv channels must be a multiple of the K tile");
  DN_CHECK(p.a0 && p.b && p.out && (p.c1 == 0 || p.a1), "gemm: null operand");
  DN_CHECK(!p.geglu || (p.N % 64 == 0), "gemm: GEGLU needs N % 64 == 0");
  DN_CHECK(!p.geglu || g.bm == 32 || (g.bn / 2) % 64 == 0,
           "gemm: GEGLU needs 64-column value/gate pairs per wave");
  DN_CHECK(p.ldb % (16 / (int)sizeof(T)) == 0 && p.lda0 % (16 / (int)sizeof(T)) == 0 &&
               (p.c1 == 0 || p.lda1 % (16 / (int)sizeof(T)) == 0),
           "gemm: leading dimensions must be multiples of 16 bytes");
  if (g.frag) {
    DN_CHECK(sizeof(T) == 2, "gemm: the fragment-B kernel is bf16 only");
    gemm_bf16_frag(p, g, s);
    return;
  }
  if (p.taps == 9)
    dispatch<T, true>(p, g, s);
  else
    dispatch<T, false>(p, g, s);
}

template GemmPlan gemm_plan<float>(int, int, int, int, int, bool, bool, bool, bool);
template GemmPlan gemm_plan<bf16>(int, int, int, int, int, bool, bool, bool, bool);
template void gemm<float>(const GemmParams&, const GemmPlan&, hipStream_t);
template void gemm<bf16>(const GemmParams&, const GemmPlan&, hipStream_t);

}  // namespace dn
