// bf16 GEMM / implicit-GEMM conv with fragment-ordered weights (gfx950).
//
// Same contraction and epilogue as gemm.hip (see kernels.h), organised for the
// dense bf16 hot path:
//  - B, the packed weight matrix, is stored in MFMA fragment order (to_frag, below):
//    for each block of 32 output columns and each k-step of 16, the 64 lanes' 16-byte
//    operands lie in 1 KB of contiguous memory. Each wave loads its own B fragments
//    with one coalesced 16-byte load per lane straight into registers, one to three LDS
//    stages ahead, so B costs no LDS bandwidth (as far ahead as the A stages where the
//    registers allow: the compiler, which does not see the A loads, waits for a B
//    register by counting B loads only, so each such wait also retires the oldest A
//    loads issued after that B load);
//  - A (the activations, or the implicit-convolution gather) goes global -> LDS with
//    global_load_lds_dwordx4 into S stages of BK = 64 (128-byte rows, chunk c of row r
//    at position c ^ f(r), f(r) = (r & 7) ^ ((r >> 3) & 1)), shared by the waves (four
//    issue the loads);
//  - block tile BM x NW * 32 FN: the NW (4 or 5) waves split the columns, each computes
//    BM x 32 FN with 32x32x16 MFMAs issued as C^T = B A^T (four consecutive output
//    columns per lane). The 160-column tiles take four waves (X5): wave w owns column
//    block w and computes column block 4 over k-step w of every stage, so the four SIMDs
//    carry equal work; the four partial sums of block 4 meet in LDS in wave order;
//  - every k-step interleaves one MFMA, one LDS fragment read for the next k-step and
//    its share of B loads (scheduling groups); the stage hand-over (wait + barrier)
//    sits before the last k-step, whose MFMAs cover the first reads of the next stage;
//  - split-K: the units (tile, split) cover contiguous K ranges and write fp32 partial
//    tiles; a second kernel sums the slabs in split order (deterministic) and applies
//    the epilogue;
//  - epilogue from registers (wave_epilogue); the split-K slabs go through LDS as whole rows;
//  - tiles go to XCDs in contiguous ranges (workgroup ids are dealt round-robin over the
//    8 XCDs), ordered by column band, split, then row tile, so that the units sharing a
//    band of B run on one XCD and share its L2;
//  - a 128 x 256 grid whose last round would be at most half full runs its last column
//    bands as 64-row tiles in the same launch (a wrapper decodes full and tail units), so
//    that the fraction of a round spreads over every CU.
#include <algorithm>
#include <type_traits>

#include "gemm_epilogue.h"

namespace dn {
namespace {

constexpr int kXcds = 8;
constexpr int kBK = 64;
constexpr int kRowBytes = 128;

// Scheduling-group pattern of one k-step: NM MFMAs, each followed by one LDS read
// (while the NR reads last) and by its share of the NV B loads.
template <int I, int NM, int NR, int NV> struct KSched {
  __device__ static __forceinline__ void apply() {
    if constexpr (I < NM) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
      if constexpr (I < NR) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
      constexpr int v = NV * (I + 1) / NM - NV * I / NM;
      if constexpr (v > 0) __builtin_amdgcn_sched_group_barrier(0x020, v, 0);  // VM load
      KSched<I + 1, NM, NR, NV>::apply();
    }
  }
};

__device__ __forceinline__ bool aligned16(const void* q) {
  return (reinterpret_cast<__UINTPTR_TYPE__>(q) & 15) == 0;
}

// ---------------------------------------------------------------- epilogue
//
// A wave's accumulators leave straight from registers. Lane l of a 32 x 32 block holds row
// l % 32 and, in registers 4 g .. 4 g + 3, the four columns 8 g + 4 (l / 32) ... For bf16 one
// v_permlane32_swap per dword exchanges the halves' pieces of two g, after which a lane holds
// 8 consecutive columns (16 bytes); then, for both types, v_permlane16_swap trades 16-lane
// rows between two such pieces, so that a store (and a residual load) covers 64 bytes of each
// of 16 rows. The next block's residual is loaded before the current one is finished.
//
// What bounds it: every workgroup of a launch reaches its epilogue together and runs every
// instruction of it once, so its time is instruction fetch and the store burst. Hence one
// short path per kind of output (the kernels hold every kind, chosen at run time; a launch
// fetches one). The previous form, one long path through LDS with run-time cases and
// element-wise tails in it, took 5.1 us of a 128 x 128 tile's launch
// and 13 us of a lone 128 x 256 tile's; measured whole launches, before -> after: QKV
// 2048 x 3840 x 1280 32.3 -> 28.2 us, projection 2048 x 1280 x 1280 with an fp32 residual
// 20.1 -> 17.8 us, FF-in 66.6 -> 63.1 us, 32768-row convolution 320 -> 320 77.9 -> 72.7 us.
// Layouts the vector forms do not take (bases or leading dimensions that are not 16-byte
// aligned) go through LDS in a rolled loop.

// kinds of the vector path
enum EpiKind { kEpiGeneric = 0, kEpiBf16, kEpiF32, kEpiGeglu };

__device__ __forceinline__ bool bias_vec(const GemmParams& p) { return !p.bias || aligned16(p.bias); }

// Uniform over the launch. Column blocks are whole (n_store is a multiple of 32, or of 4 and
// equal to N for the slabs), so only row tails are masked.
__device__ __forceinline__ int epi_kind(const GemmParams& p) {
  if (p.n_store % 32 != 0 || !bias_vec(p) || !aligned16(p.out) || (p.wscale && !aligned16(p.wscale))) return kEpiGeneric;
  if (p.geglu) return !p.out_f32 && p.ldo % 16 == 0 ? kEpiGeglu : kEpiGeneric;
  if (p.out_fp8) return kEpiGeneric;
  if (p.rowvec && (p.rowvec_ld % 4 != 0 || !aligned16(p.rowvec))) return kEpiGeneric;
  if (p.resid && (!aligned16(p.resid) || p.ldr % 8 != 0)) return kEpiGeneric;
  if (p.vt && (p.out_f32 || p.rowvec || p.resid)) return kEpiGeneric;
  if (p.out_f32) return p.ldo % 4 == 0 ? kEpiF32 : kEpiGeneric;
  return p.ldo % 8 == 0 ? kEpiBf16 : kEpiGeneric;
}

// V^T columns of the kEpiBf16 kind as 4-byte token pairs: every sample starts at an even row
// and an even, 4-byte aligned address. Otherwise (odd token counts: 77 text tokens, 25 x 21
// grids) those blocks, and only those, store 2-byte tokens: 25.4 us at 1922 x 3840 x 1280 (961
// tokens a sample), where the whole launch through LDS took 35.8; the 77-token context
// 308 x 1280 x 768 7.4 against 9.5.
__device__ __forceinline__ bool vt_pairs(const GemmParams& p) {
  return p.vt_col0 % 32 == 0 && p.vt_seq % 2 == 0 && p.vt_ld % 2 == 0 && (reinterpret_cast<__UINTPTR_TYPE__>(p.vt) & 3) == 0;
}

__device__ __forceinline__ f32x4 ld_f4(const float* q) { return *reinterpret_cast<const f32x4*>(q); }

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  const bf16x2 v = {static_cast<bf16>(a), static_cast<bf16>(b)};
  return __builtin_bit_cast(unsigned, v);
}

// v_permlane32_swap: lanes 32 - 63 of a and lanes 0 - 31 of b trade places.
struct Pair {
  unsigned a, b;
};
__device__ __forceinline__ Pair swap32(unsigned a, unsigned b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  return Pair{r[0], r[1]};
}

// v_permlane16_swap: the odd 16-lane rows of a and the even ones of b trade places.
__device__ __forceinline__ Pair swap16(unsigned a, unsigned b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  return Pair{r[0], r[1]};
}

// Register layout (lane: row l % 32) <-> store layout (lane: row l % 16, a later column group
// in the odd 16-lane rows): a, b hold two column groups of 32 rows on one side, 16-row
// halves of both groups on the other. Self-inverse.
__device__ __forceinline__ void rows16(uint4& a, uint4& b) {
  const Pair x = swap16(a.x, b.x), y = swap16(a.y, b.y), z = swap16(a.z, b.z), w = swap16(a.w, b.w);
  a = make_uint4(x.a, y.a, z.a, w.a);
  b = make_uint4(x.b, y.b, z.b, w.b);
}
__device__ __forceinline__ void rows16(f32x4& a, f32x4& b) {
  uint4 u = __builtin_bit_cast(uint4, a), v = __builtin_bit_cast(uint4, b);
  rows16(u, v);
  a = __builtin_bit_cast(f32x4, u);
  b = __builtin_bit_cast(f32x4, v);
}

// Two groups of four columns, v0 of g and v1 of g + 1 (g even) -> 8 consecutive columns of the
// row in 16 bytes: columns 8 g .. in lanes 0 - 31, 8 g + 8 .. in lanes 32 - 63.
__device__ __forceinline__ uint4 bf16_row8(const float* v0, const float* v1) {
  const Pair x = swap32(pack_bf16(v0[0], v0[1]), pack_bf16(v1[0], v1[1]));
  const Pair y = swap32(pack_bf16(v0[2], v0[3]), pack_bf16(v1[2], v1[3]));
  return make_uint4(x.a, y.a, x.b, y.b);
}

__device__ __forceinline__ void add_bf16x4(float* v, unsigned lo, unsigned hi) {
  v[0] += __uint_as_float(lo << 16);
  v[1] += __uint_as_float(lo & 0xffff0000u);
  v[2] += __uint_as_float(hi << 16);
  v[3] += __uint_as_float(hi & 0xffff0000u);
}

// x * Phi(x) with Phi from the erf of Abramowitz & Stegun 7.1.26, as gelu_erf, arranged as
// max(x, 0) - |x| q with q = (1 - erf(|x| / sqrt 2)) / 2 (halved coefficients): four VALU
// operations fewer, and no cancellation for negative x.
__device__ __forceinline__ float gelu_q(float x) {
  const float ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(ax, 0.3275911f * 0.70710678118654752f, 1.0f));
  const float poly = t * (0.127414796f + t * (-0.142248368f + t * (0.7107068705f + t * (-0.7265760135f + t * 0.5307027145f))));
  const float e = __builtin_amdgcn_exp2f(x * (x * -0.72134752044448170f));
  return fmaf(-fminf(ax, 3.4e38f), poly * e, fmaxf(x, 0.0f));  // finite |x| times zero at x = +-inf
}

// Accumulators scaled by the column's weight scale (fp8) or as they are.
template <bool SCALE> __device__ __forceinline__ f32x4 epi_scale(const GemmParams& p, int n) {
  if constexpr (SCALE) return ld_f4(p.wscale + n);
  return f32x4{1.f, 1.f, 1.f, 1.f};
}

// Four output columns [n, n + 4) of row m in the output type, masked past n_store.
template <bool SCALE> __device__ __forceinline__ void store_out4(const GemmParams& p, int m, int n, const float* v) {
  if (SCALE && p.out_fp8) {
    uint8_t* o = static_cast<uint8_t*>(p.out) + (long long)m * p.ldo + n;
    const unsigned w = fp8x4(v[0], v[1], v[2], v[3]);
    for (int e = 0; e < 4; ++e)
      if (n + e < p.n_store) o[e] = static_cast<uint8_t>(w >> (8 * e));
  } else {
    store4<bf16>(p, m, n, v, p.n_store);
  }
}

// One wave's 32 rows x 32 FN accumulator columns in LDS -> outputs, any layout.
template <int FN, bool SCALE>
__device__ __forceinline__ void generic_rows(const GemmParams& p, const float* ep, int mb, int nw0) {
  constexpr int WN = 32 * FN, EPL = WN + 4;
  const int lane = threadIdx.x & 63;
  const int cols = p.geglu ? WN / 2 : WN;  // output columns of the wave
#pragma unroll 1
  for (int t = lane; t < 32 * (cols / 4); t += 64) {
    const int rr = t / (cols / 4), c = (t - rr * (cols / 4)) * 4;
    const int m = mb + rr;
    if (m >= p.M) continue;
    float v[4];
    if (p.geglu) {
      const int lc = c / 32 * 64 + c % 32;  // value column; its gate is 32 further
      const int o = nw0 / 2 + c, nv = nw0 + lc;
      if (o >= p.n_store) continue;
      for (int e = 0; e < 4; ++e) {
        float a = ep[rr * EPL + lc + e], g = ep[rr * EPL + lc + 32 + e];
        if constexpr (SCALE) a *= p.wscale[nv + e], g *= p.wscale[nv + 32 + e];
        if (p.bias) a += p.bias[nv + e], g += p.bias[nv + 32 + e];
        v[e] = a * gelu_q(g);
      }
      store_out4<SCALE>(p, m, o, v);
    } else {
      const int n = nw0 + c;
      for (int e = 0; e < 4; ++e) {
        v[e] = ep[rr * EPL + c + e];
        if constexpr (SCALE) v[e] *= n + e < p.n_store ? p.wscale[n + e] : 0.f;
      }
      if (SCALE && p.out_fp8) {
        for (int e = 0; e < 4; ++e) {
          if (n + e >= p.n_store) continue;
          if (p.bias) v[e] += p.bias[n + e];
          const long long ro = (long long)m * p.ldr + n + e;
          if (p.resid)
            v[e] += p.resid_f32 ? static_cast<const float*>(p.resid)[ro]
                                : static_cast<float>(static_cast<const bf16*>(p.resid)[ro]);
        }
        store_out4<SCALE>(p, m, n, v);
      } else {
        epilogue_group<bf16>(p, m, n, v);
      }
    }
  }
}

// The wave's blocks acc[i][j] (rows m0 + 32 i .., columns nw0 + 32 j ..), i < FM, j < FN.
// pin: with use_pin, the fp32 residual of the kEpiF32 kind already in registers.
// ep: 32 x (32 FN + 4) floats of LDS of this wave (generic path).
// VT: the launch may have a V^T output (else its code stays out of the kernel).
template <int FM, int FN, bool SPLIT, bool SCALE, bool PIN, bool VT>
__device__ __forceinline__ void wave_epilogue(const GemmParams& p, const f32x16 (*acc)[FN], const int m0, const int nw0,
                                              const int split, const int kind, const f32x4 (*pin)[FN][4], const bool use_pin,
                                              float* ep) {
  const int lane = threadIdx.x & 63;
  const int row = lane & 31, hh = lane >> 5, h4 = 4 * hh;
  // store layout: row and, for fp32 (a pair of g) and bf16 (a 32-column block), first column
  const int r16 = lane & 15, c8 = 8 * ((lane >> 4) & 1) + h4, c16 = 16 * ((lane >> 4) & 1) + 8 * hh;
  if constexpr (SPLIT) {
    // whole rows of the wave's columns through LDS (128 or 256 bytes per row and store): the
    // slabs are the largest output here, and 64-byte pieces straight from registers took
    // 49.5 us instead of 45.3 (2048 x 1280 x 5120, four slabs)
    constexpr int WN = 32 * FN, EPL = WN + 4, LPR = WN / 4, RPI = 64 / LPR;
    float* slab = p.part + (long long)split * p.M * p.n_store;
    const int c4 = (lane % LPR) * 4, n = nw0 + c4;
    f32x4 sc = {1.f, 1.f, 1.f, 1.f};
    if constexpr (SCALE) {
#pragma unroll
      for (int e = 0; e < 4; ++e) sc[e] = n + e < p.n_store ? p.wscale[n + e] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<f32x4*>(ep + row * EPL + j * 32 + 8 * g + h4) =
              f32x4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
#pragma unroll
      for (int t = 0; t < 32 / RPI; ++t) {
        const int rr = t * RPI + lane / LPR, m = m0 + 32 * i + rr;
        f32x4 v = *reinterpret_cast<const f32x4*>(ep + rr * EPL + c4);
        if (m >= p.M || n >= p.n_store) continue;
        if constexpr (SCALE) v *= sc;
        *reinterpret_cast<f32x4*>(slab + (long long)m * p.n_store + n) = v;
      }
    }
    return;
  }
  // value of register 4 g + e with the column scale and the bias
  auto biased = [&](const f32x16& a, int n, int g, const f32x4& bias, float* v) {
    const f32x4 sc = epi_scale<SCALE>(p, n + 8 * g + h4);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (SCALE ? a[4 * g + e] * sc[e] : a[4 * g + e]) + bias[e];
  };
  // a bf16 block of 32 rows and columns [n, n + 32), as bf16_row8 gives it
  auto store_rows = [&](int mb, int n, uint4 w0, uint4 w1) {
    rows16(w0, w1);
    bf16* d = static_cast<bf16*>(p.out) + (long long)(mb + r16) * p.ldo + n + c16;
    if (mb + r16 < p.M) *reinterpret_cast<uint4*>(d) = w0;
    if (mb + r16 + 16 < p.M) *reinterpret_cast<uint4*>(d + 16ll * p.ldo) = w1;
  };
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  if (kind == kEpiGeglu) {
    if constexpr (FN % 2 == 0) {
#pragma unroll
      for (int j = 0; j < FN; j += 2) {
        const int n = nw0 + 32 * j, o = n / 2;  // value columns n .. n + 31, gates n + 32 ..
        if (o >= p.n_store) break;
        f32x4 ba[4], bg[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          ba[g] = p.bias ? ld_f4(p.bias + n + 8 * g + h4) : zero;
          bg[g] = p.bias ? ld_f4(p.bias + n + 32 + 8 * g + h4) : zero;
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const int m = m0 + 32 * i + row;
          float v[4][4];
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            float va[4], vg[4];
            biased(acc[i][j], n, g, ba[g], va);
            biased(acc[i][j + 1], n + 32, g, bg[g], vg);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[g][e] = va[e] * gelu_q(vg[e]);
          }
          if (SCALE && p.out_fp8) {
            // 4 codes per g; two swaps give a lane 16 consecutive codes of 32
            const Pair x = swap32(fp8x4(v[0][0], v[0][1], v[0][2], v[0][3]), fp8x4(v[2][0], v[2][1], v[2][2], v[2][3]));
            const Pair y = swap32(fp8x4(v[1][0], v[1][1], v[1][2], v[1][3]), fp8x4(v[3][0], v[3][1], v[3][2], v[3][3]));
            if (m < p.M)
              *reinterpret_cast<uint4*>(static_cast<uint8_t*>(p.out) + (long long)m * p.ldo + o + 16 * hh) = make_uint4(x.a, x.b, y.a, y.b);
          } else {
            store_rows(m0 + 32 * i, o, bf16_row8(v[0], v[1]), bf16_row8(v[2], v[3]));
          }
        }
      }
    }
    return;
  }
  if (SCALE && kind == kEpiF32) {
    // fp8 (no row vector): whole rows of the wave's columns through LDS, a block's residual loaded
    // before the block is. The short main loop leaves nothing to hide the residual behind, and
    // whole rows (128 or 256 bytes) are what its reads and the output's writes want: 8192 x 640 x
    // 2560 32.1 -> 27.9 us, 3000 x 320 x 1280 14.2 -> 12.2. In bf16 it is slower as often as faster
    // (9216 x 640 x 640 21.6 -> 22.9, 4096 x 1280 x 5120 63.3 -> 66.7).
    constexpr int WN = 32 * FN, EPL = WN + 4, LPR = WN / 4, RPI = 64 / LPR, NP = 32 / RPI;
    const int c4 = (lane % LPR) * 4, n = nw0 + c4;
    const bool in = n < p.n_store;
    const int nn = in ? n : 0;
    const f32x4 sc = epi_scale<SCALE>(p, nn), bias = p.bias ? ld_f4(p.bias + nn) : zero;
    const bool rf32 = p.resid && p.resid_f32, rb16 = p.resid && !p.resid_f32;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      f32x4 r[NP];
      if (rf32) {
#pragma unroll
        for (int t = 0; t < NP; ++t)
          r[t] = ld_f4(static_cast<const float*>(p.resid) + (long long)min(m0 + 32 * i + t * RPI + lane / LPR, p.M - 1) * p.ldr + nn);
      }
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<f32x4*>(ep + row * EPL + j * 32 + 8 * g + h4) =
              f32x4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
#pragma unroll
      for (int t = 0; t < NP; ++t) {
        const int rr = t * RPI + lane / LPR, m = m0 + 32 * i + rr;
        f32x4 v = *reinterpret_cast<const f32x4*>(ep + rr * EPL + c4) * sc + bias;
        if (m >= p.M || !in) continue;
        if (rb16) {
          const bf16x4 b = *reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(p.resid) + (long long)m * p.ldr + n);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += static_cast<float>(b[e]);
        }
        if (rf32) v += r[t];
        *reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + (long long)m * p.ldo + n) = v;
      }
    }
    return;
  }
  if (!SCALE && kind == kEpiF32) {
    // residual of block t = i FN + j (fp32, or bf16 widened when it is used), one block ahead
    f32x4 rf[2][4];
    bf16x4 rb[2][4];
    const bool rf32 = p.resid && p.resid_f32 && !(PIN && use_pin), rb16 = p.resid && !p.resid_f32;
    auto load_resid = [&](int t) {
      const int n = min(nw0 + 32 * (t % FN), p.n_store - 32), mb = m0 + 32 * (t / FN);
      if (rf32) {  // store layout: rf[g], rf[g + 1] the two 16-row halves of the pair
        const float* r0 = static_cast<const float*>(p.resid) + (long long)min(mb + r16, p.M - 1) * p.ldr + n + c8;
        const float* r1 = static_cast<const float*>(p.resid) + (long long)min(mb + r16 + 16, p.M - 1) * p.ldr + n + c8;
#pragma unroll
        for (int g = 0; g < 4; g += 2) {
          rf[t & 1][g] = ld_f4(r0 + 8 * g);
          rf[t & 1][g + 1] = ld_f4(r1 + 8 * g);
        }
      }
      if (rb16) {
        const bf16* r = static_cast<const bf16*>(p.resid) + (long long)min(mb + row, p.M - 1) * p.ldr + n + h4;
#pragma unroll
        for (int g = 0; g < 4; ++g) rb[t & 1][g] = *reinterpret_cast<const bf16x4*>(r + 8 * g);
      }
    };
    load_resid(0);
    f32x4 bias[FN][4];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        bias[j][g] = p.bias ? ld_f4(p.bias + min(nw0 + 32 * j, p.n_store - 32) + 8 * g + h4) : zero;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int m = m0 + 32 * i + row;
      const float* rv = p.rowvec ? p.rowvec + (long long)(min(m, p.M - 1) / p.rows_per_sample) * p.rowvec_ld + h4 : nullptr;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int n = nw0 + 32 * j, t = i * FN + j;
        if (t + 1 < FM * FN) load_resid(t + 1);
        if (n >= p.n_store) continue;
        f32x4 w[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float v[4];
          biased(acc[i][j], n, g, bias[j][g], v);
          w[g] = f32x4{v[0], v[1], v[2], v[3]};
          if (rv) w[g] += ld_f4(rv + n + 8 * g);
          if (rb16)
#pragma unroll
            for (int e = 0; e < 4; ++e) w[g][e] += static_cast<float>(rb[t & 1][g][e]);
        }
#pragma unroll
        for (int g = 0; g < 4; g += 2) {
          rows16(w[g], w[g + 1]);
          if constexpr (PIN) {
            if (use_pin) {
              w[g] += pin[i][j][g];
              w[g + 1] += pin[i][j][g + 1];
            }
          }
          if (rf32) {
            w[g] += rf[t & 1][g];
            w[g + 1] += rf[t & 1][g + 1];
          }
          float* d = static_cast<float*>(p.out) + (long long)(m0 + 32 * i + r16) * p.ldo + n + 8 * g + c8;
          if (m0 + 32 * i + r16 < p.M) *reinterpret_cast<f32x4*>(d) = w[g];
          if (m0 + 32 * i + r16 + 16 < p.M) *reinterpret_cast<f32x4*>(d + 16ll * p.ldo) = w[g + 1];
        }
      }
    }
    return;
  }
  if (kind == kEpiBf16) {
    // residual: bf16 as whole 16-byte rows, one block t = i FN + j ahead (swapped into the
    // register layout when used), or fp32
    uint4 rb[2][2];
    const bool pairs = VT && p.vt && vt_pairs(p);
    const bool rb16 = p.resid && !p.resid_f32, rf32 = p.resid && p.resid_f32;
    auto load_resid = [&](int t) {
      if (!rb16) return;
      const int mb = m0 + 32 * (t / FN);
      const bf16* r = static_cast<const bf16*>(p.resid) + min(nw0 + 32 * (t % FN), p.n_store - 32) + c16;
      rb[t & 1][0] = *reinterpret_cast<const uint4*>(r + (long long)min(mb + r16, p.M - 1) * p.ldr);
      rb[t & 1][1] = *reinterpret_cast<const uint4*>(r + (long long)min(mb + r16 + 16, p.M - 1) * p.ldr);
    };
    load_resid(0);
    f32x4 bias[FN][4];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        bias[j][g] = p.bias ? ld_f4(p.bias + min(nw0 + 32 * j, p.n_store - 32) + 8 * g + h4) : zero;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int m = m0 + 32 * i + row;
      const float* rv = p.rowvec ? p.rowvec + (long long)(min(m, p.M - 1) / p.rows_per_sample) * p.rowvec_ld + h4 : nullptr;
      const float* rf =
          rf32 ? static_cast<const float*>(p.resid) + (long long)min(m, p.M - 1) * p.ldr + h4 : nullptr;
      // V^T output: sample and token of the row
      int vb = 0, vs = 0;
      if (VT && p.vt && nw0 + 32 * FN > p.vt_col0) {
        vb = m / p.vt_seq;
        vs = m - vb * p.vt_seq;
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int n = nw0 + 32 * j, tb = i * FN + j;
        if (tb + 1 < FM * FN) load_resid(tb + 1);
        if (n >= p.n_store) continue;
        float v[4][4];
#pragma unroll
        for (int g = 0; g < 4; ++g) biased(acc[i][j], n, g, bias[j][g], v[g]);
        if (VT && p.vt && n + 32 > p.vt_col0) {
          // rows are tokens; column nn of V^T is row nn of the sample's heads x dp
          bf16* dst = static_cast<bf16*>(p.vt) +
                      ((long long)vb * p.vt_heads * p.vt_dp + n - p.vt_col0 + h4) * p.vt_ld + vs;
          if (__builtin_expect(pairs, true)) {
            // neighbouring lanes exchange one of two columns, so a lane stores two
            // consecutive tokens of a column (4 bytes; 64-byte segments)
            const bool odd = lane & 1;
            if (odd) dst += p.vt_ld - 1;
            const unsigned sel = odd ? 0x03020706u : 0x05040100u;
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
              for (int e = 0; e < 4; e += 2) {
                const unsigned x = pack_bf16(v[g][e], v[g][e + 1]);
                const unsigned y = __builtin_amdgcn_update_dpp(0u, x, 0xb1, 0xf, 0xf, true);  // lane ^ 1
                const unsigned w = __builtin_amdgcn_perm(y, x, sel);
                if (m < p.M) *reinterpret_cast<unsigned*>(dst + (long long)(8 * g + e) * p.vt_ld) = w;
              }
          } else if (m < p.M) {
            // one token per lane: lanes 0 - 31 and 32 - 63 store 32 consecutive tokens of a
            // column each; in a block that straddles the split, columns before it to out
            bf16* out = static_cast<bf16*>(p.out) + (long long)m * p.ldo + n + h4;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              if (n + 8 * g + h4 >= p.vt_col0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[(long long)(8 * g + e) * p.vt_ld] = static_cast<bf16>(v[g][e]);
              } else {
                OutVec<bf16>::store(out + 8 * g, v[g]);
              }
            }
          }
          continue;
        }
        if (rv)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 r = ld_f4(rv + n + 8 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[g][e] += r[e];
          }
        if (rf)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 r = ld_f4(rf + n + 8 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[g][e] += r[e];
          }
        if (rb16) {
          rows16(rb[tb & 1][0], rb[tb & 1][1]);
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const uint4 r = rb[tb & 1][t];
            const Pair x = swap32(r.x, r.z), y = swap32(r.y, r.w);
            add_bf16x4(v[2 * t], x.a, y.a);
            add_bf16x4(v[2 * t + 1], x.b, y.b);
          }
        }
        store_rows(m0 + 32 * i, n, bf16_row8(v[0], v[1]), bf16_row8(v[2], v[3]));
      }
    }
    return;
  }
  // generic: 32 rows at a time through LDS, one group of four columns per lane and step
  constexpr int WN = 32 * FN, EPL = WN + 4;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4*>(ep + row * EPL + j * 32 + 8 * g + h4) =
            f32x4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
    generic_rows<FN, SCALE>(p, ep, m0 + 32 * i, nw0);
  }
}

template <int BM, int FN, int S, int NW, bool X5 = false> constexpr size_t frag_lds_bytes() {
  constexpr size_t stages = size_t(S) * BM * kRowBytes;
  constexpr size_t epi = size_t(NW) * 32 * (32 * FN + 4) * 4;
  constexpr size_t part5 = X5 ? size_t(4) * (BM / 32) * 16 * 64 * 4 : 0;  // block-4 partial sums
  constexpr size_t m1 = stages > epi ? stages : epi;
  return m1 > part5 ? m1 : part5;
}

// MODE: 0 linear layer (one A source), 1 linear layer over two concatenated A sources,
// 2 implicit 3x3 convolution (one source). SPLIT: write fp32 partial tiles.
// D: B register buffers (B is loaded D stages ahead). WPE: waves per SIMD the register
// allocation must allow (2: two workgroups share a CU, so one's prologue, barriers and
// epilogue overlap the other's MFMAs). NW: waves per workgroup, each owning
// 32 FN columns; with five (a 160-column tile) the first four issue the A DMA. X5: the
// 160-column tile on four waves (see the file comment).
// One unit: the BM x BN tile at (m0, n0) over the K stages [kt0, kt1) (split-K part
// `split` when SPLIT).
template <int BM, int FN, int S, int D, int WPE, int MODE, bool SPLIT, int NW, bool X5>
__device__ __forceinline__ void frag_tile(const GemmParams& p, const int m0, const int n0, const int split,
                                          const int kt0, const int kt1) {
  constexpr int FM = BM / 32;
  constexpr int WN = 32 * FN;
  static_assert(!X5 || (NW == 4 && FN == 1), "X5: four waves of one column block each");
  constexpr int NB = 4 * FN + (X5 ? 1 : 0);  // B loads per wave and stage
  constexpr int STAGE = BM * kRowBytes;
  constexpr int PW = BM / 32;  // DMA instructions (8 rows of 128 B) per DMA wave per stage
  static_assert(NW == 4 || NW == 5, "four or five waves");
  constexpr int NM = FM * FN;
  static_assert(D >= 1 && D <= 3, "one to three B buffers");
  static_assert(S >= 2 && S <= 6, "2 to 6 LDS stages");
  static_assert(BM % 32 == 0 && BM <= 256, "BM");

  extern __shared__ __align__(16) unsigned char smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // ---- A rows: instruction j of this wave loads tile rows [8 q, 8 q + 8), q = wave * PW + j;
  // the lane fetches logical chunk (lane & 7) ^ f(row) of row 8 q + (lane >> 3). Each row
  // keeps a 32-bit element offset at k = 0 (linear: row * lda; conv: the input pixel of tap
  // (0, 0), possibly outside the image, times lda) and, for conv, a tap mask (bit 3 ky + kx:
  // tap inside the input; bits 9 / 10: output row / column parity, which picks the source
  // pixel of the taps of a nearest-x2 upsampled input); MODE 1 keeps the second source's
  // offset instead.
  const int lrow = lane >> 3;
  const int lc_even = ((lane & 7) ^ lrow) * 8, lc_odd = ((lane & 7) ^ lrow ^ 1) * 8;
  int off0[PW];
  int off1[PW];
  const int hl = p.in_h << p.up, wl = p.in_w << p.up;
#pragma unroll
  for (int j = 0; j < PW; ++j) {
    const int q = wave * PW + j;
    const int lc = (q & 1) ? lc_odd : lc_even;
    const int m = min(m0 + 8 * q + lrow, p.M - 1);
    off1[j] = 0;
    if (MODE == 2) {
      const int opix = p.out_h * p.out_w;
      const int smp = m / opix;
      const int r2 = m - smp * opix;
      const int oy = r2 / p.out_w, ox = r2 - (r2 / p.out_w) * p.out_w;
      const int iy0 = oy * p.stride - 1, ix0 = ox * p.stride - 1;
      int mk = 0;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int iy = iy0 + t / 3, ix = ix0 + t % 3;
        mk |= (iy >= 0 && iy < hl && ix >= 0 && ix < wl) ? (1 << t) : 0;
      }
      mk |= (oy & 1) << 9 | (ox & 1) << 10;
      const int pix = (smp * p.in_h + (iy0 >> p.up)) * p.in_w + (ix0 >> p.up);
      off0[j] = pix * p.lda0 + lc;
      off1[j] = mk;
    } else {
      off0[j] = m * p.lda0 + lc;
      if (MODE == 1) off1[j] = m * p.lda1 + lc;
    }
  }
  const int ct = p.c0 + p.c1;
  const bf16* const gA0 = static_cast<const bf16*>(p.a0);
  const bf16* const gA1 = static_cast<const bf16*>(p.a1);

  // DMA of A stage kt into LDS slot `slot`: PW global_load_lds per DMA wave, no branches
  // (a fifth wave issues none).
  // Stages past this unit's range read the 16-byte zero block instead, so every
  // hand-over issues the same number of loads.
  auto issue_a = [&](int kt_in, int slot) {
    const bool real = kt_in < kt1;
    const int kt = real ? kt_in : kt1 - 1;
    const int k0 = kt * kBK;
    unsigned char* stage = smem + slot * STAGE;
    int tap = 0, c = k0;
    if (MODE == 2) {
      tap = k0 / ct;
      c = k0 - tap * ct;
    }
    const int ky = tap / 3, kx = tap - 3 * (tap / 3);
    const bool second = MODE == 1 && c >= p.c0;
    const bf16* a_src = second ? gA1 : gA0;
    const int a_c = second ? c - p.c0 : c;
    const int tap_off = (MODE == 2 && !p.up) ? (ky * p.in_w + kx) * p.lda0 : 0;
    if (NW > 4 && wave >= 4) return;
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int q = wave * PW + j;
      const bf16* g;
      if (MODE == 2) {
        int off = off0[j] + a_c + tap_off;
        if (p.up) {
          const int dy = ky == 2 || (ky == 1 && !(off1[j] & (1 << 9)));
          const int dx = kx == 2 || (kx == 1 && !(off1[j] & (1 << 10)));
          off += (dy ? p.in_w * p.lda0 : 0) + (dx ? p.lda0 : 0);
        }
        const bool inb = (off1[j] >> tap) & 1;
        g = inb ? a_src + off : static_cast<const bf16*>(p.zero16);
      } else {
        g = a_src + ((MODE == 1 && second) ? off1[j] : off0[j]) + a_c;
      }
      if (!real) g = static_cast<const bf16*>(p.zero16);
      dma16(g, (lds_void*)(stage + q * 1024));
    }
  };

  // ---- B fragments of this wave: column blocks nb = (n0 + wave * WN) / 32 + j, clamped
  // to the packed rows (columns past N are computed and dropped by the epilogue).
  const int kbs = p.K / 16;
  const int nb_last = (p.N + 31) / 32 - 1;
  const bf16* bptr[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int nb = min((n0 + wave * WN) / 32 + j, nb_last);
    bptr[j] = static_cast<const bf16*>(p.b) + (long long)nb * kbs * 512 + lane * 8;
  }
  typedef bf16x8 BReg[4][FN];
  auto load_b_step = [&](int kt_in, int s, BReg& dst) {
    const int kt = kt_in < kt1 ? kt_in : kt1 - 1;
#pragma unroll
    for (int j = 0; j < FN; ++j) dst[s][j] = *reinterpret_cast<const bf16x8*>(bptr[j] + (kt * 4 + s) * 512);
  };
  // X5: the fragment of column block 4 for k-step `wave` of a stage
  const bf16* const bptr5 =
      static_cast<const bf16*>(p.b) + (long long)min(n0 / 32 + 4, nb_last) * kbs * 512 + lane * 8 + wave * 512;
  auto load_b5 = [&](int kt_in, bf16x8& dst) {
    const int kt = kt_in < kt1 ? kt_in : kt1 - 1;
    dst = *reinterpret_cast<const bf16x8*>(bptr5 + kt * 4 * 512);
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  f32x16 acc5[X5 ? FM : 1];
#pragma unroll
  for (int i = 0; i < (X5 ? FM : 1); ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc5[i][r] = 0.f;

  // fp32 residual of an fp32 output for small wave tiles of the linear modes (where the
  // registers are free): loaded right after the prologue's A and B loads, so the first wait
  // (in-order vector-memory counter) does not include it and the main loop hides it.
  const int kind = SPLIT ? 0 : epi_kind(p);
  constexpr bool kPreIn = !SPLIT && !X5 && MODE != 2 && FM * FN <= 2 && WPE <= 2;
  const int nw0 = n0 + wave * WN;
  const bool pre_in = kPreIn && kind == kEpiF32 && p.resid && p.resid_f32;
  f32x4 pin[kPreIn ? FM : 1][FN][4];
  auto load_pre_in = [&]() {
    if constexpr (kPreIn) {
      if (pre_in) {
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          // store layout of wave_epilogue: 16-row halves of each pair of g
          const float* r = static_cast<const float*>(p.resid) + 8 * ((lane >> 4) & 1) + 4 * (lane >> 5);
          const float* r0 = r + (long long)min(m0 + i * 32 + (lane & 15), p.M - 1) * p.ldr;
          const float* r1 = r + (long long)min(m0 + i * 32 + 16 + (lane & 15), p.M - 1) * p.ldr;
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int g = 0; g < 4; g += 2) {
              const int n = min(nw0 + 32 * j, p.n_store - 32) + 8 * g;
              pin[i][j][g] = ld_f4(r0 + n);
              pin[i][j][g + 1] = ld_f4(r1 + n);
            }
        }
      }
    }
  };

  // A fragment of k-step s: row (lane % 32) of each 32-row block, logical chunk
  // 2 s + (lane / 32) at its swizzled position.
  const int frow = lane & 31;
  const int fs = (lane & 7) ^ ((lane >> 3) & 1);
  const int hh = lane >> 5;
  bf16x8 fa[2][FM];
  auto read_a = [&](int slot, int s, bf16x8* a) {
    const unsigned char* st = smem + slot * STAGE + frow * kRowBytes + (((2 * s + hh) ^ fs) * 16);
#pragma unroll
    for (int i = 0; i < FM; ++i) a[i] = *reinterpret_cast<const bf16x8*>(st + i * 32 * kRowBytes);
  };
  auto mfmas = [&](const bf16x8* a, const bf16x8* b) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
  };
  bf16x8 a5[X5 ? FM : 1];
  auto mfmas5 = [&](const bf16x8& b) {
#pragma unroll
    for (int i = 0; i < FM; ++i) acc5[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a5[i], acc5[i], 0, 0, 0);
  };

  {
    BReg bq[D];
    bf16x8 b5q[X5 ? D : 1];
    // One k-step: [the DMA of a later A stage first, when `dma`], the next k-step's A
    // fragments from LDS, this k-step's MFMAs and the B loads of stage kt + D for this
    // k-step, interleaved one MFMA / one LDS read / a share of the VM loads. X5 (part):
    // k-step 0 also reads the A fragments of k-step `wave` of the stage, k-step 1 runs
    // the column-block-4 MFMAs on them, k-step 2 loads the block-4 fragment of stage
    // kt + D (after its use).
    auto kstep = [&](auto dma, auto part, int dma_kt, int dma_slot, int rd_slot, int rd_s, bf16x8* a_use,
                     bf16x8* a_next, bf16x8* b_use, int bkt, int s, BReg& bb, bf16x8& b5) {
      constexpr int X = X5 ? decltype(part)::value : 0;
      if constexpr (decltype(dma)::value) issue_a(dma_kt, dma_slot);
      read_a(rd_slot, rd_s, a_next);
      if constexpr (X == 1) read_a(rd_slot, wave, a5);
      mfmas(a_use, b_use);
      if constexpr (X == 2) mfmas5(b5);
      load_b_step(bkt, s, bb);
      if constexpr (X == 3) load_b5(bkt, b5);
      KSched<0, NM + (X == 2 ? FM : 0), FM, FN + (X == 3 ? 1 : 0)>::apply();
      __builtin_amdgcn_sched_barrier(0);
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using P2 = std::integral_constant<int, 2>;
    using P3 = std::integral_constant<int, 3>;

    // prologue: A stages kt0 .. kt0 + S - 1 (every slot), B stages kt0 .. kt0 + D - 1; the
    // wait covers A stages kt0 .. kt0 + Q (see the hand-over below)
    constexpr int Q = (S - 1 - D) > 1 ? (S - 1 - D) : 1;
  #pragma unroll
    for (int s = 0; s < S; ++s) issue_a(kt0 + s, s);
  #pragma unroll
    for (int d = 0; d < D; ++d) {
  #pragma unroll
      for (int s = 0; s < 4; ++s) load_b_step(kt0 + d, s, bq[d]);
      if constexpr (X5) load_b5(kt0 + d, b5q[d]);
    }
    // the epilogue inputs come after every prologue load: the waits below count only
    // loads issued after their target, so more of them (these) keep the waits exact or
    // conservative
    load_pre_in();
    __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0((S - 1 - Q) * PW + D * NB));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_a(0, 0, fa[0]);

    // Stage kt (slot (kt - kt0) % S, B buffer bb): k-steps 0..2; the hand-over: this wave's
    // DMA of stage kt + 1 has landed once at most VM_END later VM loads are pending, and
    // after the barrier every wave's has, and every wave is done reading slot kt; then
    // k-step 3 issues stage kt + S into that slot and reads stage kt + 1's first fragments.
    // VM loads issued after the DMA of stage kt + 1 (made in k-step 3 of stage kt + 1 - S):
    // B(3) of that stage, S - 2 whole stages (NB B loads + PW DMA each), the B loads of
    // k-steps 0..2 of stage kt (NB - FN). When stage kt + 1 (kt = kt0 + r) came from the
    // prologue, the loads after its DMA are (S - 2 - r) PW + D NB + r (NB + PW) + NB - FN,
    // at least VM_END once D + r >= S - 1; the prologue itself waited for stages up to
    // kt0 + Q, Q = max(1, S - 1 - D).
    constexpr int VM_END = NB + (S - 2) * (NB + PW);
    static_assert(VM_END < 64 && (S - 1 - Q) * PW + D * NB < 64, "vmcnt range");
    auto stage = [&](int kt, BReg& bb, bf16x8& b5) {
      const int rel = kt - kt0;
      const int slot = rel % S;
      const int nslot = (rel + 1) % S;
      kstep(std::false_type{}, P1{}, 0, 0, slot, 1, fa[0], fa[1], bb[0], kt + D, 0, bb, b5);
      kstep(std::false_type{}, P2{}, 0, 0, slot, 2, fa[1], fa[0], bb[1], kt + D, 1, bb, b5);
      kstep(std::false_type{}, P3{}, 0, 0, slot, 3, fa[0], fa[1], bb[2], kt + D, 2, bb, b5);
      __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(VM_END));
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      kstep(std::true_type{}, P0{}, kt + S, slot, nslot, 0, fa[1], fa[0], bb[3], kt + D, 3, bb, b5);
    };

    if constexpr (D == 3) {
      // Triples of stages, then the rest (as for pairs below)
      int kt = kt0;
      for (; kt + 2 < kt1; kt += 3) {
        stage(kt, bq[0], b5q[0]);
        stage(kt + 1, bq[1], b5q[X5 ? 1 : 0]);
        stage(kt + 2, bq[2], b5q[X5 ? 2 : 0]);
      }
      if (kt < kt1) stage(kt, bq[0], b5q[0]);
      if (kt + 1 < kt1) stage(kt + 1, bq[1], b5q[X5 ? 1 : 0]);
    } else if constexpr (D == 2) {
      // Pairs of stages, then the odd one: no stage of the loop body is conditional, so
      // the compiler's wait for a B register counts both stages' loads issued after it.
      int kt = kt0;
      for (; kt + 1 < kt1; kt += 2) {
        stage(kt, bq[0], b5q[0]);
        stage(kt + 1, bq[1], b5q[X5 ? 1 : 0]);
      }
      if (kt < kt1) stage(kt, bq[0], b5q[0]);
    } else {
      for (int kt = kt0; kt < kt1; ++kt) stage(kt, bq[0], b5q[0]);
    }
  }
  // The loads past the range (zero block, clamped B) must land before LDS is reused.
  __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
  __syncthreads();

  // ---- epilogue (one wave-private LDS block for the generic path)
  float* ep = reinterpret_cast<float*>(smem) + wave * (32 * (WN + 4));
  if constexpr (X5) {
    // the partial sums of column block 4 go to LDS in the register layout; wave w < FM then
    // sums row block w of it over the four waves in wave order
    float* part5 = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) part5[((wave * FM + i) * 16 + r) * 64 + lane] = acc5[i][r];
    __syncthreads();
    f32x16 blk5[1][1];
    if (wave < FM) {
#pragma unroll
      for (int r = 0; r < 16; ++r) blk5[0][0][r] = part5[((0 * FM + wave) * 16 + r) * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; ++w)
#pragma unroll
        for (int r = 0; r < 16; ++r) blk5[0][0][r] += part5[((w * FM + wave) * 16 + r) * 64 + lane];
    }
    __syncthreads();
    wave_epilogue<FM, FN, SPLIT, false, false, false>(p, acc, m0, nw0, split, kind, nullptr, false, ep);
    if (wave < FM && n0 + 128 < p.N)
      wave_epilogue<1, 1, SPLIT, false, false, false>(p, blk5, m0 + wave * 32, n0 + 128, split, kind, nullptr, false, ep);
  } else if constexpr (kPreIn) {
    wave_epilogue<FM, FN, SPLIT, false, true, MODE == 0>(p, acc, m0, nw0, split, kind, pin, pre_in, ep);
  } else {
    wave_epilogue<FM, FN, SPLIT, false, false, MODE == 0>(p, acc, m0, nw0, split, kind, nullptr, false, ep);
  }
}

// The kernel: unit assignment (see the file comment), then the unit's tile. TBM > 0 with
// tail_bands > 0 (no split): the first tail_full units are BM-row tiles of the column
// bands before the last tail_bands, the rest TBM-row tiles of those last bands; each
// XCD takes its share of both kinds, full tiles first (tail_full and the tail count
// are multiples of the XCD count). A grid of BM-row tiles that fills a whole number of
// rounds plus a fraction of one leaves that fraction to half the CUs; TBM-row tiles
// spread it over all of them.
template <int BM, int FN, int S, int D, int WPE, int MODE, bool SPLIT, int NW = 4, bool X5 = false,
          int TBM = 0>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void gemm_frag_kernel(
    GemmParams p, int mt, int nt, int nsplit, int tail_full, int tail_bands) {
  constexpr int BN = X5 ? 160 : NW * 32 * FN;
  const int wg = blockIdx.x;
  const int xcd = wg % kXcds, idx = wg / kXcds;
  const int nk = p.K / kBK;
  if constexpr (TBM > 0) {
    static_assert(!SPLIT, "tail tiles take no split");
    if (tail_bands > 0) {
      const int fx = tail_full / kXcds;
      const int tm = (p.M + TBM - 1) / TBM;
      const int tx = tm * tail_bands / kXcds;
      if (idx < fx) {
        const int f = xcd * fx + idx;
        frag_tile<BM, FN, S, D, WPE, MODE, SPLIT, NW, X5>(p, (f % mt) * BM, (f / mt) * BN, 0, 0, nk);
      } else {
        const int t = xcd * tx + (idx - fx);
        frag_tile<TBM, FN, S, 1, WPE, MODE, SPLIT, NW, X5>(p, (t % tm) * TBM,
                                                                (nt - tail_bands + t / tm) * BN, 0, 0, nk);
      }
      return;
    }
  }
  const int units = mt * nt * nsplit;
  const int base = units / kXcds, rem = units % kXcds;
  const int logical = xcd * base + min(xcd, rem) + idx;
  const int m_tile = logical % mt;
  const int ns = logical / mt;
  const int split = ns % nsplit;
  const int n_tile = ns / nsplit;
  const int kt0 = (int)((long long)split * nk / nsplit);
  const int kt1 = (int)((long long)(split + 1) * nk / nsplit);
  frag_tile<BM, FN, S, D, WPE, MODE, SPLIT, NW, X5>(p, m_tile * BM, n_tile * BN, split, kt0, kt1);
}

// Sum of the split-K partial slabs [NS][M][n_store] in split order, then the epilogue;
// one thread per 4 consecutive columns of a row, all slab loads issued before the sum.
template <int NS> __global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmParams p) {
  const int q = p.n_store / 4;
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= (long long)p.M * q) return;
  const int m = (int)(i / q);
  const int n = (int)(i - (long long)m * q) * 4;
  const long long slab = (long long)p.M * p.n_store;
  const float* src = p.part + (long long)m * p.n_store + n;
  f32x4 t[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) t[k] = *reinterpret_cast<const f32x4*>(src + k * slab);
  f32x4 s = t[0];
#pragma unroll
  for (int k = 1; k < NS; ++k) {
    s[0] += t[k][0];
    s[1] += t[k][1];
    s[2] += t[k][2];
    s[3] += t[k][3];
  }
  float v[4] = {s[0], s[1], s[2], s[3]};
  epilogue_group<bf16>(p, m, n, v);
}

void splitk_reduce(const GemmParams& p, int nsplit, hipStream_t s) {
  const long long nq = (long long)p.M * (p.n_store / 4);
  const dim3 grid(static_cast<unsigned>((nq + 255) / 256));
  switch (nsplit) {
    case 2: hipLaunchKernelGGL(splitk_reduce_kernel<2>, grid, dim3(256), 0, s, p); break;
    case 3: hipLaunchKernelGGL(splitk_reduce_kernel<3>, grid, dim3(256), 0, s, p); break;
    case 4: hipLaunchKernelGGL(splitk_reduce_kernel<4>, grid, dim3(256), 0, s, p); break;
    case 5: hipLaunchKernelGGL(splitk_reduce_kernel<5>, grid, dim3(256), 0, s, p); break;
    case 6: hipLaunchKernelGGL(splitk_reduce_kernel<6>, grid, dim3(256), 0, s, p); break;
    case 7: hipLaunchKernelGGL(splitk_reduce_kernel<7>, grid, dim3(256), 0, s, p); break;
    case 8: hipLaunchKernelGGL(splitk_reduce_kernel<8>, grid, dim3(256), 0, s, p); break;
    default: throw Error(-1, "gemm: split-K reduction takes 2 to 8 slabs");
  }
  DN_HIP(hipGetLastError());
}

template <int BM, int FN, int S, int D, int WPE, int MODE, bool SPLIT, int NW, bool X5, int TBM = 0>
void launch_frag(const GemmParams& p, int nsplit, hipStream_t s, int tail_bands = 0) {
  constexpr size_t lds_full = frag_lds_bytes<BM, FN, S, NW, X5>();
  constexpr size_t lds_tail = TBM > 0 ? frag_lds_bytes<(TBM > 0 ? TBM : BM), FN, S, NW, X5>() : 0;
  constexpr size_t lds = lds_full > lds_tail ? lds_full : lds_tail;
  static bool attr_set = false;
  if (!attr_set) {
    DN_HIP(hipFuncSetAttribute(
        reinterpret_cast<const void*>(&gemm_frag_kernel<BM, FN, S, D, WPE, MODE, SPLIT, NW, X5, TBM>),
        hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    attr_set = true;
  }
  const int mt = ceil_div(p.M, BM), nt = ceil_div(p.N, X5 ? 160 : 32 * FN * NW);
  int grid = mt * nt * nsplit, tail_full = 0;
  if (TBM > 0 && tail_bands > 0) {
    tail_full = mt * (nt - tail_bands);
    const int tail = ceil_div(p.M, TBM > 0 ? TBM : BM) * tail_bands;
    DN_CHECK(nsplit == 1 && tail_bands < nt && tail_full % kXcds == 0 && tail % kXcds == 0,
             "gemm: tail tiles need no split and tile counts divisible by the XCD count");
    grid = tail_full + tail;
  }
  hipLaunchKernelGGL((gemm_frag_kernel<BM, FN, S, D, WPE, MODE, SPLIT, NW, X5, TBM>), dim3(grid), dim3(64 * NW),
                     lds, s, p, mt, nt, nsplit, tail_full, TBM > 0 ? tail_bands : 0);
  DN_HIP(hipGetLastError());
}

template <int BM, int FN, int S, int D, int WPE, int MODE, int NW = 4, bool X5 = false>
void run_frag(const GemmParams& p, int nsplit, hipStream_t s) {
  if (p.raw_partial) {
    launch_frag<BM, FN, S, D, WPE, MODE, true, NW, X5>(p, nsplit, s);
  } else if (nsplit > 1) {
    launch_frag<BM, FN, S, D, WPE, MODE, true, NW, X5>(p, nsplit, s);
    splitk_reduce(p, nsplit, s);
  } else {
    launch_frag<BM, FN, S, D, WPE, MODE, false, NW, X5>(p, 1, s);
  }
}

// Tile plans (three LDS stages): 128 x 256 (FN = 2) with two B buffers (one for the
// convolution), two workgroups per CU; 128 x 128 (FN = 1) and 64 x 128 with two B buffers,
// two / four workgroups per CU; for linear layers 64 x 160 and 128 x 160 on five waves with
// three B buffers, one workgroup per CU; 128 x 160 on four waves (x5) with two B buffers, two
// workgroups per CU.
template <int MODE> void dispatch_frag(const GemmParams& p, const GemmPlan& g, hipStream_t s) {
  if (g.bm == 128 && g.bn == 256) {
    // B two stages ahead where the registers allow it (the implicit convolution's
    // address registers do not leave room)
    if constexpr (MODE == 2) {
      return run_frag<128, 2, 3, 1, 2, MODE>(p, g.split, s);
    } else {
      // the last column bands of a grid with a partial last round as 64-row tiles
      if (g.tail_bands > 0 && g.split == 1 && !p.raw_partial) {
        launch_frag<128, 2, 3, 2, 2, MODE, false, 4, false, 64>(p, 1, s, g.tail_bands);
        return;
      }
      return run_frag<128, 2, 3, 2, 2, MODE>(p, g.split, s);
    }
  }
  if (g.bm == 128 && g.bn == 128) return run_frag<128, 1, 3, 2, 2, MODE>(p, g.split, s);
  if (g.bm == 64 && g.bn == 128) return run_frag<64, 1, 3, 2, 4, MODE>(p, g.split, s);
  if constexpr (MODE != 2) {
    if (g.bm == 64 && g.bn == 160) return run_frag<64, 1, 3, 3, 2, MODE, 5>(p, g.split, s);
    if (g.bm == 128 && g.bn == 160 && !g.x5) return run_frag<128, 1, 3, 3, 2, MODE, 5>(p, g.split, s);
  }
  if (g.bm == 128 && g.bn == 160 && g.x5) return run_frag<128, 1, 3, 2, 2, MODE, 4, true>(p, g.split, s);
  throw Error(-1, "gemm: no fragment-B kernel for this tile plan");
}

// ---------------------------------------------------------------- fp8 (E4M3) kernel
//
// The same organisation as gemm_frag_kernel for E4M3 operands on the 32x32x64 fp8
// matrix-core step (v_mfma_scale_f32_32x32x64_f8f6f4 with unit block scales): an LDS
// stage still holds 128-byte rows, now 128 k-values, i.e. two matrix-core steps; lane l
// supplies row (l % 32) and the 32 consecutive k-values 32 (l / 32) .. + 32 of a step
// (two 16-byte LDS reads; any k order common to both operands gives the same sum).
// B is packed by pack_fp8: per 32 output rows and 64-deep step, the lanes' 32-byte
// operands in 2 KB. The epilogue multiplies each column by its row scale of B.
typedef int v8i __attribute__((ext_vector_type(8)));

__device__ __forceinline__ v8i v8i_of(const uint4& a, const uint4& b) {
  v8i r;
  r[0] = (int)a.x, r[1] = (int)a.y, r[2] = (int)a.z, r[3] = (int)a.w;
  r[4] = (int)b.x, r[5] = (int)b.y, r[6] = (int)b.z, r[7] = (int)b.w;
  return r;
}

template <int BM, int FN, int S, int WPE, bool SPLIT>
__device__ __forceinline__ void fp8_tile(const GemmParams& p, const int m0, const int n0, const int split,
                                         const int kt0, const int kt1) {
  constexpr int NW = 4;
  constexpr int FM = BM / 32;
  constexpr int WN = 32 * FN;
  constexpr int STAGE = BM * kRowBytes;
  constexpr int PW = BM / 32;  // DMA instructions (8 rows of 128 B) per wave per stage
  constexpr int NM = FM * FN;
  static_assert(S >= 3 && S <= 4, "three or four LDS stages");

  extern __shared__ __align__(16) unsigned char smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // A rows: DMA instruction j of this wave fills tile rows [8 q, 8 q + 8), q = wave PW + j
  const int lrow = lane >> 3;
  const int lc_even = ((lane & 7) ^ lrow) * 16, lc_odd = ((lane & 7) ^ lrow ^ 1) * 16;
  int off0[PW];
#pragma unroll
  for (int j = 0; j < PW; ++j) {
    const int q = wave * PW + j;
    const int m = min(m0 + 8 * q + lrow, p.M - 1);
    off0[j] = m * p.lda0 + ((q & 1) ? lc_odd : lc_even);
  }
  const uint8_t* const gA = static_cast<const uint8_t*>(p.a0);
  auto issue_a = [&](int kt_in, int slot) {
    const bool real = kt_in < kt1;
    unsigned char* stage = smem + slot * STAGE;
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int q = wave * PW + j;
      const uint8_t* g = real ? gA + off0[j] + kt_in * 128 : static_cast<const uint8_t*>(p.zero16);
      dma16(g, (lds_void*)(stage + q * 1024));
    }
  };

  // B operands of this wave: column blocks nb = (n0 + wave WN) / 32 + j (clamped)
  const int ksteps = p.K / 64;
  const int nb_last = (p.N + 31) / 32 - 1;
  const uint8_t* bptr[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int nb = min((n0 + wave * WN) / 32 + j, nb_last);
    bptr[j] = static_cast<const uint8_t*>(p.b) + (long long)nb * ksteps * 2048 + lane * 32;
  }
  typedef uint4 BStep[FN][2];  // one 64-deep step: FN column blocks, 32 bytes per lane
  auto load_b = [&](int step_in, BStep& dst) {
    const int st = step_in < 2 * kt1 ? step_in : 2 * kt1 - 1;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const uint8_t* src = bptr[j] + (long long)st * 2048;
      dst[j][0] = *reinterpret_cast<const uint4*>(src);
      dst[j][1] = *reinterpret_cast<const uint4*>(src + 16);
    }
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int frow = lane & 31;
  const int fs = (lane & 7) ^ ((lane >> 3) & 1);
  const int hh = lane >> 5;
  auto read_a = [&](int slot, int s2, v8i* a) {
    const unsigned char* st = smem + slot * STAGE + frow * kRowBytes;
    const int c0 = 4 * s2 + 2 * hh;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const uint4 lo = *reinterpret_cast<const uint4*>(st + i * 32 * kRowBytes + ((c0 ^ fs) * 16));
      const uint4 hi = *reinterpret_cast<const uint4*>(st + i * 32 * kRowBytes + (((c0 + 1) ^ fs) * 16));
      a[i] = v8i_of(lo, hi);
    }
  };
  auto mfmas = [&](const v8i* a, const BStep& b) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(v8i_of(b[j][0], b[j][1]), a[i], acc[i][j], 0, 0,
                                                                    0, 127, 0, 127);
  };

  // B is loaded two 64-deep steps ahead into two register sets. Stage kt (r = kt - kt0):
  // wait until this wave's DMA of stage kt landed, barrier; step 2 kt, then B of step
  // 2 kt + 2 into its set; step 2 kt + 1, then B of step 2 kt + 3; last, the DMA of stage
  // kt + 2 into the slot of stage kt - 1. The compiler waits for a B set counting only the
  // B loads issued after it, so each of its waits also retires the oldest DMA issued
  // after that B load: with this order that is at most the DMA of stage kt + 1, in the
  // second half of stage kt, just before it is needed (with FN = 1 the first wait of a
  // stage retires half of it). Loads issued after the DMA of stage kt: PW + 4 FN
  // (r = 0: the prologue's second DMA and B sets; steady state: stage kt - 1's B loads
  // and DMA), 8 FN + PW (r = 1: the prologue's B sets and stage kt0's loads).
  static_assert(S == 3, "three LDS stages");
  constexpr int WS = PW + 4 * FN;
  constexpr int W1 = 8 * FN + PW;
  static_assert(W1 < 64, "vmcnt range");
  issue_a(kt0, 0);
  issue_a(kt0 + 1, 1);
  BStep b0, b1;
  load_b(2 * kt0, b0);
  load_b(2 * kt0 + 1, b1);
  for (int kt = kt0; kt < kt1; ++kt) {
    const int r = kt - kt0;
    if (r == 1)
      __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(W1));
    else
      __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(WS));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const int slot = r % 3;
    v8i a[FM];
    read_a(slot, 0, a);
    mfmas(a, b0);
    KSched<0, NM, 0, 0>::apply();
    __builtin_amdgcn_sched_barrier(0);
    load_b(2 * kt + 2, b0);
    read_a(slot, 1, a);
    mfmas(a, b1);
    KSched<0, NM, 0, 0>::apply();
    __builtin_amdgcn_sched_barrier(0);
    load_b(2 * kt + 3, b1);
    issue_a(kt + 2, (r + 2) % 3);
  }
  __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
  __syncthreads();

  float* ep = reinterpret_cast<float*>(smem) + wave * (32 * (WN + 4));
  wave_epilogue<FM, FN, SPLIT, true, false, false>(p, acc, m0, n0 + wave * WN, split, SPLIT ? 0 : epi_kind(p), nullptr, false, ep);
}

// The fp8 kernel: unit assignment as gemm_frag_kernel (XCD-contiguous; with TBM > 0 and
// tail_bands > 0 the last column bands as TBM-row tiles, full tiles first on every XCD).
template <int BM, int FN, int S, int WPE, bool SPLIT, int TBM = 0>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void gemm_fp8_kernel(
    GemmParams p, int mt, int nt, int nsplit, int tail_full, int tail_bands) {
  constexpr int BN = 4 * 32 * FN;
  const int wg = blockIdx.x;
  const int xcd = wg % kXcds, idx = wg / kXcds;
  const int nk = p.K / 128;
  if constexpr (TBM > 0) {
    static_assert(!SPLIT, "tail tiles take no split");
    if (tail_bands > 0) {
      const int fx = tail_full / kXcds;
      const int tm = (p.M + TBM - 1) / TBM;
      const int tx = tm * tail_bands / kXcds;
      if (idx < fx) {
        const int f = xcd * fx + idx;
        fp8_tile<BM, FN, S, WPE, SPLIT>(p, (f % mt) * BM, (f / mt) * BN, 0, 0, nk);
      } else {
        const int t = xcd * tx + (idx - fx);
        fp8_tile<TBM, FN, S, WPE, SPLIT>(p, (t % tm) * TBM, (nt - tail_bands + t / tm) * BN, 0, 0, nk);
      }
      return;
    }
  }
  const int units = mt * nt * nsplit;
  const int base = units / kXcds, rem = units % kXcds;
  const int logical = xcd * base + min(xcd, rem) + idx;
  const int m_tile = logical % mt;
  const int ns = logical / mt;
  const int split = ns % nsplit;
  const int n_tile = ns / nsplit;
  const int kt0 = (int)((long long)split * nk / nsplit);
  const int kt1 = (int)((long long)(split + 1) * nk / nsplit);
  fp8_tile<BM, FN, S, WPE, SPLIT>(p, m_tile * BM, n_tile * BN, split, kt0, kt1);
}

template <int BM, int FN, int S, int WPE, bool SPLIT, int TBM = 0>
void launch_fp8(const GemmParams& p, int nsplit, hipStream_t s, int tail_bands = 0) {
  constexpr size_t lds_full = frag_lds_bytes<BM, FN, S, 4>();
  constexpr size_t lds_tail = TBM > 0 ? frag_lds_bytes<(TBM > 0 ? TBM : BM), FN, S, 4>() : 0;
  constexpr size_t lds = lds_full > lds_tail ? lds_full : lds_tail;
  static bool attr_set = false;
  if (!attr_set) {
    DN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_fp8_kernel<BM, FN, S, WPE, SPLIT, TBM>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    attr_set = true;
  }
  const int mt = ceil_div(p.M, BM), nt = ceil_div(p.N, 32 * FN * 4);
  int grid = mt * nt * nsplit, tail_full = 0;
  if (TBM > 0 && tail_bands > 0) {
    tail_full = mt * (nt - tail_bands);
    const int tail = ceil_div(p.M, TBM > 0 ? TBM : BM) * tail_bands;
    DN_CHECK(nsplit == 1 && tail_bands < nt && tail_full % kXcds == 0 && tail % kXcds == 0,
             "gemm_fp8: tail tiles need no split and tile counts divisible by the XCD count");
    grid = tail_full + tail;
  }
  hipLaunchKernelGGL((gemm_fp8_kernel<BM, FN, S, WPE, SPLIT, TBM>), dim3(grid), dim3(256), lds, s, p, mt, nt, nsplit,
                     tail_full, TBM > 0 ? tail_bands : 0);
  DN_HIP(hipGetLastError());
}

template <int BM, int FN, int S, int WPE> void run_fp8(const GemmParams& p, int nsplit, hipStream_t s) {
  if (p.raw_partial) {
    launch_fp8<BM, FN, S, WPE, true>(p, nsplit, s);
  } else if (nsplit > 1) {
    launch_fp8<BM, FN, S, WPE, true>(p, nsplit, s);
    // the slabs hold scaled sums; the reduction applies bias / residual (unit scales)
    GemmParams q = p;
    splitk_reduce(q, nsplit, s);
  } else {
    launch_fp8<BM, FN, S, WPE, false>(p, 1, s);
  }
}

// Fragment order of a packed [N][K] weight matrix (N rounded up to 32, K % 16 == 0):
// element (n, k) lives at ((n / 32) * (K / 16) + k / 16) * 512 + lane * 8 + k % 8 with
// lane = n % 32 + 32 * ((k % 16) / 8).
__global__ void to_frag_kernel(const bf16* src, int N, int K, int lds, bf16* dst, int Npad) {
  const long long nv = (long long)Npad * K / 8;
  const int kbs = K / 16;
  for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < nv; v += (long long)gridDim.x * blockDim.x) {
    const int lane = (int)(v % 64);
    const long long t = v / 64;
    const int kb = (int)(t % kbs);
    const int nb = (int)(t / kbs);
    const int n = nb * 32 + (lane & 31);
    const int k = kb * 16 + (lane >> 5) * 8;
    uint4 val = make_uint4(0u, 0u, 0u, 0u);
    if (n < N) val = *reinterpret_cast<const uint4*>(src + (long long)n * lds + k);
    *reinterpret_cast<uint4*>(dst + v * 8) = val;
  }
}

}  // namespace

bool gemm_frag_layout(int N, int K) { return N >= 32 && N % 32 == 0 && K >= kBK && K % kBK == 0; }

size_t gemm_frag_elems(int N, int K) { return (size_t)((N + 31) / 32 * 32) * K; }

void to_frag(const bf16* src, int N, int K, int ld_src, bf16* dst, hipStream_t s) {
  DN_CHECK(K % 16 == 0 && ld_src % 8 == 0 && ld_src >= K, "to_frag: K and the source pitch must suit 16-byte rows");
  const int Npad = (N + 31) / 32 * 32;
  const long long nv = (long long)Npad * K / 8;
  const int blocks = static_cast<int>(std::min<long long>((nv + 255) / 256, 16384));
  hipLaunchKernelGGL(to_frag_kernel, dim3(std::max(blocks, 1)), dim3(256), 0, s, src, N, K, ld_src, dst, Npad);
  DN_HIP(hipGetLastError());
}

bool gemm_fp8_layout(int N, int K) { return N >= 32 && N % 32 == 0 && K >= 128 && K % 128 == 0; }

size_t gemm_fp8_code_bytes(int N, int K) { return (size_t)((N + 31) / 32 * 32) * K; }

GemmPlan gemm_plan_fp8(int M, int N, int K, int geglu, int cus, bool fused_reduce, bool out_f32) {
  return frag_plan(M, N, K, geglu, cus, fused_reduce, kPlanFp8, out_f32);
}

void gemm_fp8(const GemmParams& p, const GemmPlan& g, hipStream_t s) {
  DN_CHECK(gemm_fp8_layout(p.N, p.K), "gemm_fp8: N % 32 == 0 and K % 128 == 0 needed");
  DN_CHECK(p.taps == 1 && p.c1 == 0 && p.c0 == p.K, "gemm_fp8: one linear A source");
  DN_CHECK(p.a0 && p.b && p.out && p.wscale && p.zero16, "gemm_fp8: null operand");
  DN_CHECK(p.lda0 % 16 == 0, "gemm_fp8: A rows must be 16-byte aligned");
  DN_CHECK(!p.vt && !p.rowvec, "gemm_fp8: no V^T output, no row vector");
  DN_CHECK(g.split >= 1 && g.split <= kMaxSplit && p.K / 128 >= g.split, "gemm_fp8: bad split");
  DN_CHECK(!p.geglu || g.bn == 256, "gemm_fp8: GEGLU needs 64-column value/gate pairs per wave");
  if (g.split > 1 || p.raw_partial) {
    DN_CHECK(!p.geglu && !p.out_fp8, "gemm_fp8: split-K takes neither GEGLU nor fp8 output");
    DN_CHECK(p.n_store % 4 == 0 && p.n_store == p.N, "gemm_fp8: split-K needs n_store == N, a multiple of 4");
    DN_CHECK(p.part && p.part_floats >= (size_t)g.split * p.M * p.n_store, "gemm_fp8: split-K workspace too small");
  }
  if (g.bn == 256 && g.split == 1 && g.tail_bands > 0 && !p.raw_partial)
    launch_fp8<128, 2, 3, 2, false, 64>(p, 1, s, g.tail_bands);
  else if (g.bn == 256)
    run_fp8<128, 2, 3, 2>(p, g.split, s);
  else
    run_fp8<128, 1, 3, 2>(p, g.split, s);
}

void gemm_bf16_frag(const GemmParams& p, const GemmPlan& g, hipStream_t s) {
  DN_CHECK(gemm_frag_layout(p.N, p.K), "gemm: fragment-B kernel needs N % 32 == 0 and K % 64 == 0");
  DN_CHECK(p.taps == 1 || (p.c0 + p.c1) % kBK == 0, "gemm: conv channels must be a multiple of 64");
  DN_CHECK(p.c1 == 0 || p.c0 % kBK == 0, "gemm: concatenation split must be a multiple of 64");
  DN_CHECK(p.taps == 1 || p.zero16, "gemm: implicit conv needs the zero block");
  DN_CHECK(p.taps == 1 || p.c1 == 0, "gemm: the fragment-B conv takes one input source");
  DN_CHECK(g.split >= 1 && g.split <= kMaxSplit && p.K / kBK >= g.split, "gemm: bad split");
  DN_CHECK(!p.geglu || (g.bn / 4) % 64 == 0, "gemm: GEGLU needs 64-column value/gate pairs per wave");
  DN_CHECK(!p.vt || (p.taps == 1 && p.c1 == 0 && !g.x5),
           "gemm: the V^T output takes a plain linear layer, and not the four-wave 128 x 160 tile");
  if (g.split > 1 || p.raw_partial) {
    DN_CHECK(!p.geglu && !p.vt, "gemm: split-K takes neither GEGLU nor the V^T output");
    DN_CHECK(p.n_store % 4 == 0 && p.n_store == p.N, "gemm: split-K needs n_store == N, a multiple of 4");
    DN_CHECK(p.part && p.part_floats >= (size_t)g.split * p.M * p.n_store, "gemm: split-K workspace too small");
  }
  if (p.taps == 9)
    dispatch_frag<2>(p, g, s);
  else if (p.c1)
    dispatch_frag<1>(p, g, s);
  else
    dispatch_frag<0>(p, g, s);
}

}  // namespace dn
