// Flash-style multi-head attention for the UNet transformer blocks (gfx950).
//
// O = softmax(Q K^T * scale) V per (sample, head), never materialising the
// score matrix. A workgroup holds 32 queries per wave; key tiles of 64 rows of K
// and the matching 64 columns of V^T (V stored transposed per head by the
// projection GEMM, so both tiles are row-contiguous) are double-buffered in LDS:
// the next tile's global loads are in flight while the current one is used.
//
// Each wave computes S^T = K Q^T with 32x32 MFMA so that a lane owns one query
// column: the softmax row statistics are a per-lane reduction plus one exchange
// with the partner lane (lane ^ 32), and the probabilities already sit in the
// B-operand layout of O^T = V^T P^T; the V^T operand is read with the key
// permutation of the accumulator layout (two 8-byte reads per fragment).
//
// Lazy rescaling: the reference maximum m of a row is only moved (and O, l
// rescaled by exp2(m_old - m_new)) when a tile's maximum exceeds it by more than
// 2^8 in the exponent; otherwise probabilities up to 2^8 are accumulated against
// the old reference. softmax(x) = exp(x - m) / sum exp(x - m) holds for any m, so
// this changes rounding only, and saves the O rescale on most tiles.
#include <algorithm>

#include "kernels.h"

namespace dn {
namespace {

constexpr int kKT = 64;          // keys per LDS tile
typedef __attribute__((address_space(1))) void gbl_void_t;
constexpr float kLazy = 8.0f;    // log2 headroom before the reference max moves

// 2^x with the hardware exponential (v_exp_f32): arguments here are <= kLazy, and
// results below 2^-126 (flushed to zero) are far below bf16 / fp32 resolution of the
// row sums they join.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

template <typename T> struct PvFrag;
template <> struct PvFrag<bf16> {
  // P registers [8c, 8c + 8) of a 32-key block, lane half h, hold keys
  // 16c + 4h + {0..3} and 16c + 8 + 4h + {0..3}.
  __device__ static __forceinline__ bf16x8 v(const bf16* vt_row, int kb, int c, int h) {
    const bf16* base = vt_row + kb * 32 + 16 * c + 4 * h;
    const bf16x4 lo = *reinterpret_cast<const bf16x4*>(base);
    const bf16x4 hi = *reinterpret_cast<const bf16x4*>(base + 8);
    bf16x8 r;
    r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
    r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
    return r;
  }
  __device__ static __forceinline__ bf16x8 p(const f32x16& s, int c) {
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = static_cast<bf16>(s[8 * c + e]);
    return r;
  }
};
template <> struct PvFrag<float> {
  // Register c of a 32-key block belongs to key 8 (c / 4) + 4h + (c % 4).
  __device__ static __forceinline__ float v(const float* vt_row, int kb, int c, int h) {
    return vt_row[kb * 32 + 8 * (c >> 2) + 4 * h + (c & 3)];
  }
  __device__ static __forceinline__ float p(const f32x16& s, int c) { return s[c]; }
};

template <typename T, int D, int NW>
__global__ __launch_bounds__(64 * NW) void attn_kernel(AttnParams p) {
  using MM = Mma<T>;
  constexpr int NT = 64 * NW;
  constexpr int VEC = 16 / sizeof(T);
  constexpr int SK = D + VEC;                      // K tile row stride (elements)
  constexpr int SV = kKT + VEC;                    // V^T tile row stride (keys)
  constexpr int NS = D / MM::KS;                   // MFMA steps over the head dim
  constexpr int DB = D / 32;                       // 32-row blocks of O^T
  constexpr int PCH = 16 / MM::KPL;                // MFMAs per 32-key block (P side)
  constexpr int KV_VEC = kKT * D / VEC;            // 16-byte vectors per K tile (= per V^T tile)
  constexpr int PER_T = (2 * KV_VEC + NT - 1) / NT;
  constexpr int STAGE = kKT * SK + D * SV;

  extern __shared__ __align__(16) unsigned char attn_smem[];
  T* lds = reinterpret_cast<T*>(attn_smem);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int half = lane >> 5;
  const int b = blockIdx.z, h = blockIdx.y;
  const int q0 = blockIdx.x * (32 * NW) + wave * 32;

  const T* qp = static_cast<const T*>(p.q) + b * p.q_bs + h * D;
  const T* kp = static_cast<const T*>(p.k) + b * p.k_bs + h * D;
  const T* vtp = static_cast<const T*>(p.vt) + ((long long)b * p.heads + h) * D * p.vt_ld;

  const int qrow = min(q0 + (lane & 31), p.Sq - 1);
  typename MM::frag qf[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) qf[s] = MM::load(qp + (long long)qrow * p.ldq + s * MM::KS + half * MM::KPL);

  f32x16 o[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;

  uint4 reg[PER_T];
  auto load = [&](int t) {
    const int k0 = t * kKT;
#pragma unroll
    for (int i = 0; i < PER_T; ++i) {
      const int v = tid + i * NT;
      if (v < KV_VEC) {  // K row (key) kr, vector kc
        const int kr = v / (D / VEC), kc = v - (v / (D / VEC)) * (D / VEC);
        const long long key = min(k0 + kr, p.Skv - 1);
        reg[i] = ld16(kp + key * p.ldk + kc * VEC);
      } else if (v < 2 * KV_VEC) {  // V^T row d, keys [k0 + kc*VEC, +VEC)
        const int w = v - KV_VEC;
        const int d = w / (kKT / VEC), kc = w - (w / (kKT / VEC)) * (kKT / VEC);
        reg[i] = ld16(vtp + (long long)d * p.vt_ld + k0 + kc * VEC);
      }
    }
  };
  auto store = [&](int buf) {
    T* Ks = lds + buf * STAGE;
    T* Vt = Ks + kKT * SK;
#pragma unroll
    for (int i = 0; i < PER_T; ++i) {
      const int v = tid + i * NT;
      if (v < KV_VEC) {
        const int kr = v / (D / VEC), kc = v - (v / (D / VEC)) * (D / VEC);
        st16(Ks + kr * SK + kc * VEC, reg[i]);
      } else if (v < 2 * KV_VEC) {
        const int w = v - KV_VEC;
        const int d = w / (kKT / VEC), kc = w - (w / (kKT / VEC)) * (kKT / VEC);
        st16(Vt + d * SV + kc * VEC, reg[i]);
      }
    }
  };

  const int ntiles = (p.Skv + kKT - 1) / kKT;
  load(0);
  store(0);
  if (ntiles > 1) load(1);
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    const int k0 = t * kKT;
    const T* Ks = lds + (t & 1) * STAGE;
    const T* Vt = Ks + kKT * SK;

    f32x16 sacc[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[kb][r] = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        sacc[kb] = MM::mma(MM::load(&Ks[(kb * 32 + (lane & 31)) * SK + s * MM::KS + half * MM::KPL]), qf[s],
                           sacc[kb]);

    if (k0 + kKT > p.Skv) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (k0 + kb * 32 + acc_row(r, lane) >= p.Skv) sacc[kb][r] = -INFINITY;
    }

    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[kb][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * p.scale_log2;
    if (__any(mx > m_ref + kLazy)) {
      const float m_new = fmaxf(m_ref, mx);
      const float alpha = fast_exp2(m_ref - m_new);
      l_run *= alpha;
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
      m_ref = m_new;
    }
    float rs = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float e = fast_exp2(sacc[kb][r] * p.scale_log2 - m_ref);
        sacc[kb][r] = e;
        rs += e;
      }
    l_run += rs + __shfl_xor(rs, 32, 64);

#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int c = 0; c < PCH; ++c) {
        const typename MM::frag pf = PvFrag<T>::p(sacc[kb], c);
#pragma unroll
        for (int d = 0; d < DB; ++d)
          o[d] = MM::mma(PvFrag<T>::v(&Vt[(d * 32 + (lane & 31)) * SV], kb, c, half), pf, o[d]);
      }

    if (t + 1 < ntiles) {
      store((t + 1) & 1);
      if (t + 2 < ntiles) load(t + 2);
    }
    __syncthreads();
  }

  const int qi = q0 + (lane & 31);
  if (qi < p.Sq) {
    const float inv = 1.f / l_run;
    T* op = static_cast<T*>(p.o) + b * p.o_bs + (long long)qi * p.ldo + h * D;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = o[d][4 * g + e] * inv;
        T* dst = op + d * 32 + 8 * g + 4 * half;
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[e] = from_f32<T>(v[e]);
      }
  }
}

// ---------------------------------------------------------------------------
// Few queries: eight waves split the keys of 32 queries. A workgroup of attn_kernel walks all
// key tiles alone (2 x 4 heads, 256 x 256, head dim 32, fp32: 32 workgroups, 12.0 us); here
// each wave takes every eighth 32-key tile straight from global memory, keeps its own
// reference maximum, and the partial (m, l, O) meet in LDS in wave order (deterministic;
// 4.7 us). fp32 operands are read as in the wave-split GEMM: four consecutive head dims (K, Q)
// or keys (V^T) per lane, the same k order for both operands of an MFMA.
constexpr int kKsWaves = 8;

template <typename T, int D>
__global__ __launch_bounds__(64 * kKsWaves) void attn_keysplit_kernel(AttnParams p) {
  using MM = Mma<T>;
  constexpr int DB = D / 32;
  constexpr int NV = D / (sizeof(T) == 4 ? 8 : 16);  // 16-byte operands of a K or Q row per lane
  __shared__ float sm[kKsWaves][32], sl[kKsWaves][32];
  extern __shared__ __align__(16) unsigned char attn_smem[];
  float* so = reinterpret_cast<float*>(attn_smem);  // [wave][DB][16][64]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, r32 = lane & 31;
  const int b = blockIdx.z, h = blockIdx.y, q0 = blockIdx.x * 32;
  constexpr int VEC = 16 / sizeof(T);
  const T* qp = static_cast<const T*>(p.q) + b * p.q_bs + h * D + half * VEC;
  const T* kp = static_cast<const T*>(p.k) + b * p.k_bs + h * D + half * VEC;
  const T* vtp = static_cast<const T*>(p.vt) + ((long long)b * p.heads + h) * D * p.vt_ld;
  uint4 qv[NV];
#pragma unroll
  for (int s = 0; s < NV; ++s) qv[s] = ld16(qp + (long long)min(q0 + r32, p.Sq - 1) * p.ldq + s * 2 * VEC);
  f32x16 o[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;
  for (int k0 = wave * 32; k0 < p.Skv; k0 += 32 * kKsWaves) {
    uint4 kv[NV];
    const T* kr = kp + (long long)min(k0 + r32, p.Skv - 1) * p.ldk;
#pragma unroll
    for (int s = 0; s < NV; ++s) kv[s] = ld16(kr + s * 2 * VEC);
    f32x16 sa;
#pragma unroll
    for (int r = 0; r < 16; ++r) sa[r] = 0.f;
#pragma unroll
    for (int s = 0; s < NV; ++s) {
      if constexpr (sizeof(T) == 4) {
        const f32x4 ka = __builtin_bit_cast(f32x4, kv[s]), qa = __builtin_bit_cast(f32x4, qv[s]);
#pragma unroll
        for (int e = 0; e < 4; ++e) sa = MM::mma(ka[e], qa[e], sa);
      } else {
        sa = MM::mma(__builtin_bit_cast(bf16x8, kv[s]), __builtin_bit_cast(bf16x8, qv[s]), sa);
      }
    }
    if (k0 + 32 > p.Skv) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (k0 + acc_row(r, lane) >= p.Skv) sa[r] = -INFINITY;
    }
    float mx = sa[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sa[r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * p.scale_log2;
    const float m_new = fmaxf(m_ref, mx);
    const float alpha = fast_exp2(m_ref - m_new);
    float rs = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sa[r] = fast_exp2(sa[r] * p.scale_log2 - m_new);
      rs += sa[r];
    }
    l_run = l_run * alpha + rs + __shfl_xor(rs, 32, 64);
    m_ref = m_new;
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      const T* vr = vtp + (long long)(d * 32 + r32) * p.vt_ld + k0;
#pragma unroll
      for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
      if constexpr (sizeof(T) == 4) {
        // register 4 g + e: key 8 g + 4 half + e
        f32x4 vv[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) vv[g] = *reinterpret_cast<const f32x4*>(vr + 8 * g + 4 * half);
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[d] = MM::mma(vv[g][e], sa[4 * g + e], o[d]);
      } else {
#pragma unroll
        for (int c = 0; c < 2; ++c) o[d] = MM::mma(PvFrag<T>::v(vr, 0, c, half), PvFrag<T>::p(sa, c), o[d]);
      }
    }
  }
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) so[((wave * DB + d) * 16 + r) * 64 + lane] = o[d][r];
  if (half == 0) {
    sm[wave][r32] = m_ref;
    sl[wave][r32] = l_run;
  }
  __syncthreads();
  // thread: head dims 32 d + 8 g + 4 half .. + 3 of query r32; waves that had no keys hold
  // m = -inf and weigh nothing
  const int qi = q0 + r32;
  for (int u = threadIdx.x >> 6; u < 4 * DB; u += kKsWaves) {
    const int d = u >> 2, g = u & 3;
    float m = sm[0][r32];
#pragma unroll
    for (int w = 1; w < kKsWaves; ++w) m = fmaxf(m, sm[w][r32]);
    float l = 0.f, v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kKsWaves; ++w) {
      const float f = fast_exp2(sm[w][r32] - m);
      l += f * sl[w][r32];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += f * so[((w * DB + d) * 16 + 4 * g + e) * 64 + lane];
    }
    if (qi >= p.Sq) continue;
    const float inv = 1.f / l;
    T* dst = static_cast<T*>(p.o) + b * p.o_bs + (long long)qi * p.ldo + h * D + d * 32 + 8 * g + 4 * half;
#pragma unroll
    for (int e = 0; e < 4; ++e) dst[e] = from_f32<T>(v[e] * inv);
  }
}

// ---------------------------------------------------------------------------
// bf16, head dim 64: software-pipelined kernel for long key ranges.
//
// Same math as attn_kernel. A workgroup covers NQ x 32 queries of one (sample,
// head); workgroup ids are dealt so that each XCD (ids congruent mod 8) holds a
// contiguous range of heads, whose K and V^T then stay in that XCD's L2. Key tiles of
// 64 (K rows and the V^T rows of those keys, 16 KB) go global -> LDS with
// global_load_lds_dwordx4 into a ring of R tiles. Per key tile g every wave
//  - passes a hand-over (its loads of the tile it needs next landed, then a barrier:
//    everyone's have, and everyone is done with tile g - 1's slot) and issues tile
//    g + R - 1 into that slot;
//  - with score read-ahead (PIPE): reads K of tile g + 1 and V^T of tile g from LDS,
//    takes tile g's row maximum, then issues the S^T = K Q^T MFMAs of tile g + 1
//    interleaved with the exponentials of tile g, and O^T += V^T P^T for tile g;
//    without: scores and softmax of tile g in turn.
// Q enters the MFMAs multiplied by scale * log2(e) (rounded to bf16), and the score
// accumulators start from minus the reference maximum of the lane's query, so the
// MFMAs produce the base-2 exponent directly (the first tile starts from zero; a move
// of the reference shifts the current tile's scores by the difference).
// Within each 16-key group the K tile holds its keys in the order of bit 2 and bit 3
// of the key index swapped: score register 8c + e of a 32-key block then belongs to
// key 16c + 8h + e (h = lane half), so the V^T operand of a P fragment is 8
// consecutive keys, one 16-byte LDS read. The row sum is taken on the bf16
// probabilities that enter the P V product (dot products with (1, 1)); the partner
// lane's statistics come over v_permlane32_swap. The score and output accumulators
// stay in VGPRs (WPE waves per SIMD); only the last tile can hold key padding
// (masked). Row maxima need no NaN quieting (this file is built without NaN
// semantics: every input is finite and key padding is -inf, never NaN).
template <int NQ, int R, int WPE, bool PIPE>
__global__ __launch_bounds__(64 * NQ) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void attn_pipe_kernel(
    AttnParams p, int qtiles) {
  constexpr int D = 64;
  constexpr int ROWB = 128;                  // bytes per LDS row (64 bf16)
  constexpr int TILE = 2 * kKT * ROWB;       // K tile then V^T tile (16 KB)
  constexpr int TI = 2 * kKT / 8;            // DMA instructions per tile (8 rows each)
  constexpr int PW = TI / NQ;                // per wave per tile
  constexpr int U = R % 2 == 0 ? R : 2 * R;  // unroll: ring slot and score buffer fixed
  static_assert(TI % NQ == 0, "DMA instructions must divide over the waves");
  static_assert((kKT / 8) % PW == 0, "a wave's DMA rows must be all K rows or all V^T rows (two or more waves)");
  static_assert(R >= (PIPE ? 3 : 2) && R <= 5, "ring of 3 (2 without score read-ahead) to 5 tiles");

  extern __shared__ __align__(16) unsigned char smem[];

  const int total = qtiles * p.heads * p.B;
  const int wg = blockIdx.x;
  const int xcd = wg % 8, idx = wg / 8;
  const int base = total / 8, rem = total % 8;
  const int logical = xcd * base + min(xcd, rem) + idx;
  const int qt = logical % qtiles;
  const int bh = logical / qtiles;
  const int h = bh % p.heads, b = bh / p.heads;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5;
  const int q0 = qt * (32 * NQ) + wave * 32;

  const bf16* qp = static_cast<const bf16*>(p.q) + b * p.q_bs + h * D;
  const bf16* kp = static_cast<const bf16*>(p.k) + b * p.k_bs + h * D;
  const bf16* vtp = static_cast<const bf16*>(p.vt) + ((long long)b * p.heads + h) * D * p.vt_ld;

  // Q times scale * log2(e), rounded to bf16: the MFMAs then produce base-2 logits
  bf16x8 qf[4];
  {
    const int qrow = min(q0 + (lane & 31), p.Sq - 1);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bf16x8 raw = *reinterpret_cast<const bf16x8*>(qp + (long long)qrow * p.ldq + s * 16 + half * 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[s][e] = static_cast<bf16>(static_cast<float>(raw[e]) * p.scale_log2);
    }
  }

  // DMA: instruction i = wave * PW + j of a tile fills rows [8 i, 8 i + 8) of its ring
  // slot (rows 0..63: K, the key of row r being k0 + swap23(r); rows 64..127: V^T
  // head dims); the lane fetches logical chunk (lane & 7) ^ f(row). A wave's rows are
  // all K or all V^T (8 DMA rows per wave group), so its source is a wave-uniform
  // base, advanced by one tile per issue, plus fixed 32-bit lane offsets; only the
  // last tile (key rows clamped to Skv - 1) sets its offsets again. Issues past the
  // last tile load the last one again (the same count of loads per hand-over; nothing
  // reads them).
  const int lrow = lane >> 3;
  const int ntiles = (p.Skv + kKT - 1) / kKT;
  auto swap23 = [](int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); };
  const bool k_rows = wave * PW < kKT / 8;
  const char* gbase = k_rows ? reinterpret_cast<const char*>(kp) : reinterpret_cast<const char*>(vtp);
  const long long gstep = k_rows ? (long long)kKT * p.ldk * 2 : kKT * 2;
  unsigned goff[PW];
  auto set_offsets = [&](int t) {
    const int k0 = t * kKT;
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int i = wave * PW + j;
      const int row = 8 * i + lrow;
      const int lc = ((lane & 7) ^ lrow ^ (i & 1)) * 8;
      if (k_rows)
        goff[j] = 2u * (unsigned)(min(k0 + swap23(row), p.Skv - 1) - k0) * (unsigned)p.ldk + 2u * lc;
      else
        goff[j] = 2u * (unsigned)((row - kKT) * p.vt_ld + lc);
    }
  };
  set_offsets(0);
  int next_issue = 0;
  auto issue = [&](int slot) {
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int i = wave * PW + j;
      __builtin_amdgcn_global_load_lds((gbl_void_t*)(gbase + goff[j]), (lds_void*)(smem + slot * TILE + i * 1024), 16,
                                       0, 0);
    }
    if (next_issue < ntiles - 1) {
      ++next_issue;
      gbase += gstep;
      if (next_issue == ntiles - 1) set_offsets(next_issue);
    }
  };

  const int frow = lane & 31;
  const int fs = (lane & 7) ^ ((lane >> 3) & 1);
  // lane byte offsets: K fragment of k-step s (key block kb adds 32 rows), V^T
  // fragment of key chunk 4 kb + 2 c + h (head-dim block d adds 32 rows)
  int koff[4], voff[2][2];
#pragma unroll
  for (int s2 = 0; s2 < 4; ++s2) koff[s2] = frow * ROWB + ((2 * s2 + half) ^ fs) * 16;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int c = 0; c < 2; ++c) voff[kb][c] = kKT * ROWB + frow * ROWB + ((4 * kb + 2 * c + half) ^ fs) * 16;

  auto load_k = [&](const unsigned char* T, bf16x8 (&kf)[2][4]) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) kf[kb][s2] = *reinterpret_cast<const bf16x8*>(T + kb * 32 * ROWB + koff[s2]);
  };
  auto load_v = [&](const unsigned char* T, bf16x8 (&vf)[2][2][2]) {
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int c = 0; c < 2; ++c) vf[d][kb][c] = *reinterpret_cast<const bf16x8*>(T + d * 32 * ROWB + voff[kb][c]);
  };
  // S^T = K Q^T - m for the 64 keys of a tile (two 32-key blocks): the accumulators
  // start from c0, the negated reference maximum of the lane's query (or zero)
  auto mfma_scores = [&](const bf16x8 (&kf)[2][4], f32x16* sa, const f32x16& c0) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) sa[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb][0], qf[0], c0, 0, 0, 0);
#pragma unroll
    for (int s2 = 1; s2 < 4; ++s2)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        sa[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb][s2], qf[s2], sa[kb], 0, 0, 0);
  };

  f32x16 o[2];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;
  f32x16 sacc[2][2];
  // -m_ref in all 16 registers: the start value of the next tile's score accumulators,
  // which then hold base-2 logits minus the reference maximum
  f32x16 negm;
#pragma unroll
  for (int r = 0; r < 16; ++r) negm[r] = 0.f;

  // value of x in lane l ^ 32 (lanes l and l ^ 32 hold one query's two key halves)
  auto partner = [](float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x),
                                                    false, false);
    return __builtin_bit_cast(float, (threadIdx.x & 32) ? r[0] : r[1]);
  };

  // softmax, first part: key padding of the last tile, the tile's row maximum, and a
  // move of the reference maximum (rescaling O and l) when it grew by more than kLazy.
  // The tile's scores hold logit - m_fold (m_fold = m_ref when they were computed, 0 for
  // the first tile); on a move they are shifted to the new reference.
  auto softmax_max = [&](int k0, f32x16* sa, float m_fold) {
    if (k0 + kKT > p.Skv) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (k0 + kb * 32 + 16 * (r >> 3) + 8 * half + (r & 7) >= p.Skv) sa[kb][r] = -INFINITY;
    }
    float mc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float m = fmaxf(fmaxf(sa[0][4 * j], sa[0][4 * j + 1]), sa[0][4 * j + 2]);
      m = fmaxf(fmaxf(m, sa[0][4 * j + 3]), sa[1][4 * j]);
      m = fmaxf(fmaxf(m, sa[1][4 * j + 1]), sa[1][4 * j + 2]);
      mc[j] = fmaxf(m, sa[1][4 * j + 3]);
    }
    float mx = fmaxf(fmaxf(mc[0], mc[1]), fmaxf(mc[2], mc[3]));
    mx += m_fold;
    if (__any(mx > m_ref + kLazy)) {  // either half of a query's keys: they exchange maxima only here
      const float m_new = fmaxf(m_ref, fmaxf(mx, partner(mx)));
      const float alpha = fast_exp2(m_ref - m_new);
      l_run *= alpha;
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
      const float shift = m_new - m_fold;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) sa[kb][r] -= shift;
      m_ref = m_new;
#pragma unroll
      for (int r = 0; r < 16; ++r) negm[r] = -m_new;
    }
  };
  // softmax, second part: P = 2^(s scale - m) in bf16, its row sum, O^T += V^T P^T
  auto softmax_pv = [&](const f32x16* sa, const bf16x8 (&vf)[2][2][2]) {
    bf16x8 pf[2][2];
    float sp[2] = {0.f, 0.f};
    const bf16x2 ones = {static_cast<bf16>(1.f), static_cast<bf16>(1.f)};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        bf16x8 pv;
#pragma unroll
        for (int e = 0; e < 8; ++e) pv[e] = static_cast<bf16>(fast_exp2(sa[kb][8 * c + e]));
        pf[kb][c] = pv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bf16x2 pair = {pv[2 * e], pv[2 * e + 1]};
          sp[e & 1] = __builtin_amdgcn_fdot2_f32_bf16(pair, ones, sp[e & 1], false);
        }
      }
    l_run += sp[0] + sp[1];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int d = 0; d < 2; ++d)
          o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[d][kb][c], pf[kb][c], o[d], 0, 0, 0);
  };

  // prologue: tiles 0 .. R - 2 in flight (with score read-ahead: tile 0 landed
  // everywhere, its scores taken)
#pragma unroll
  for (int t = 0; t < R - 1; ++t) issue(t);
  if (PIPE) {
    __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0((R - 2) * PW));
    __builtin_amdgcn_s_barrier();
    bf16x8 kf[2][4];
    load_k(smem, kf);
    mfma_scores(kf, sacc[0], negm);
  }

  // Key tile g: the tile needed now (g + 1 with read-ahead, else g) was issued in an
  // earlier iteration or the prologue, and the DMAs of R - 3 (R - 2) later tiles follow
  // it, hence the vmcnt. After the barrier every wave is done with tile g - 1, whose
  // slot takes tile g + R - 1. With read-ahead, the scores of tile g + 1 are taken in
  // every iteration (after the last tile its slot holds a valid reload of the last
  // tile; those scores go unused), and their MFMAs are interleaved with the
  // exponentials of tile g.
  for (int g0 = 0; g0 < ntiles; g0 += U) {
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int g = g0 + j;
      if (g < ntiles) {
        __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0((PIPE ? R - 3 : R - 2) * PW));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        issue((j + R - 1) % R);
        const unsigned char* Tg = smem + (j % R) * TILE;
        bf16x8 kf[2][4], vf[2][2][2];
        if (PIPE) {
          load_k(smem + ((j + 1) % R) * TILE, kf);
          load_v(Tg, vf);
          softmax_max(g * kKT, sacc[j & 1], g == 0 ? 0.f : m_ref);
          mfma_scores(kf, sacc[(j + 1) & 1], negm);
          softmax_pv(sacc[j & 1], vf);
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);  // six VALU
          }
        } else {
          load_k(Tg, kf);
          const float m_fold = g == 0 ? 0.f : m_ref;
          mfma_scores(kf, sacc[0], negm);
          softmax_max(g * kKT, sacc[0], m_fold);
          load_v(Tg, vf);
          softmax_pv(sacc[0], vf);
        }
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));

  l_run += partner(l_run);  // each half has summed its own keys
  const int qi = q0 + (lane & 31);
  if (qi < p.Sq) {
    const float inv = 1.f / l_run;
    bf16* op = static_cast<bf16*>(p.o) + b * p.o_bs + (long long)qi * p.ldo + h * D;
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = static_cast<bf16>(o[d][4 * g + e] * inv);
        *reinterpret_cast<bf16x4*>(op + d * 32 + 8 * g + 4 * half) = v;
      }
  }
}

template <int NQ, int R, int WPE, bool PIPE> void launch_pipe(const AttnParams& p, hipStream_t s) {
  constexpr size_t lds = size_t(R) * 2 * kKT * 128;
  static bool attr_set = false;
  if (!attr_set) {
    DN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_pipe_kernel<NQ, R, WPE, PIPE>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    attr_set = true;
  }
  const int qtiles = (p.Sq + 32 * NQ - 1) / (32 * NQ);
  hipLaunchKernelGGL((attn_pipe_kernel<NQ, R, WPE, PIPE>), dim3(qtiles * p.heads * p.B), dim3(64 * NQ), lds, s, p,
                     qtiles);
}

template <typename T, int D> void launch_keysplit(const AttnParams& p, hipStream_t s) {
  constexpr size_t lds = sizeof(float) * kKsWaves * (D / 32) * 16 * 64;
  static bool attr_set = false;
  if (!attr_set) {
    DN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_keysplit_kernel<T, D>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    attr_set = true;
  }
  hipLaunchKernelGGL((attn_keysplit_kernel<T, D>), dim3((p.Sq + 31) / 32, p.heads, p.B), dim3(64 * kKsWaves), lds, s, p);
}

template <typename T, int D, int NW> void launch(dim3 grid, const AttnParams& p, hipStream_t s) {
  constexpr int VEC = 16 / sizeof(T);
  const size_t lds = size_t(2) * (kKT * (D + VEC) + D * (kKT + VEC)) * sizeof(T);
  static bool attr_set = false;
  if (!attr_set) {
    DN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_kernel<T, D, NW>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    attr_set = true;
  }
  hipLaunchKernelGGL((attn_kernel<T, D, NW>), grid, dim3(64 * NW), lds, s, p);
}

}  // namespace

template <typename T> void attention(const AttnParams& p, int D, int cus, hipStream_t s) {
  DN_CHECK(p.B >= 1 && p.heads >= 1 && p.Sq >= 1 && p.Skv >= 1, "attention: empty problem");
  DN_CHECK(D == 32 || D == 64, "attention: padded head dim must be 32 or 64");
  DN_CHECK(p.q && p.k && p.vt && p.o, "attention: null operand");
  constexpr int VEC = 16 / sizeof(T);
  DN_CHECK(p.ldq % VEC == 0 && p.ldk % VEC == 0 && p.vt_ld % VEC == 0, "attention: strides must be 16-byte multiples");
  DN_CHECK(p.vt_ld >= (p.Skv + kKT - 1) / kKT * kKT, "attention: V^T rows must cover whole 64-key tiles");
  // bf16, head dim 64: the software-pipelined kernel. Four waves (128 queries) per workgroup
  // share a key tile; the variant follows from how many such workgroups a CU gets, since the
  // CU with one more sets the time (measured, us, in the order below):
  //  - up to half of one: two-wave workgroups with score read-ahead, one per CU and twice as many
  //    (2 x 8 heads, 1024 keys 13.3, four waves 14.4; 2 x 20, 256 queries, 4096 keys 43.0, 45.7);
  //  - up to one: two waves per SIMD's registers (2 x 20 heads, 576 keys 10.1, three waves per
  //    SIMD 10.2, two-wave workgroups with score read-ahead 12.0; 2 x 10, 1024: 14.5, 15.0, 17.7);
  //  - up to 1.6: two-wave workgroups with read-ahead halve the uneven part (2 x 10, 1600: 28.2,
  //    29.2, 25.5; 2 x 20, 1024: 20.5, 21.1, 19.3);
  //  - up to two: as up to one (2 x 8, 4096: 74.2, 76.3, 105.9);
  //  - more: three waves per SIMD (2 x 10, 4096: 110.2, 102.1, 148.3; 4 x 20, 1024: 33.5, 30.7, 38.3).
  // Rings of three key tiles instead of two were no faster without read-ahead (107.9, 32.1).
  // Short key ranges (the 77 text tokens) take three waves per SIMD (2 x 10, 4096 queries: 11.9,
  // 10.1, 13.1).
  if (sizeof(T) == 2 && D == 64) {
    const long long heads = (long long)p.heads * p.B;
    const long long wgs = (p.Sq + 127) / 128 * heads, half_wgs = (p.Sq + 63) / 64 * heads;
    if (p.Skv < 256 || wgs > 2ll * cus)
      launch_pipe<4, 2, 3, false>(p, s);
    else if (half_wgs <= cus || (wgs > cus && 10 * wgs <= 16ll * cus))
      launch_pipe<2, 3, 2, true>(p, s);
    else
      launch_pipe<4, 2, 2, false>(p, s);
    DN_HIP(hipGetLastError());
    return;
  }
  // fp32 and head dim 32 with fewer 64-query workgroups than CUs: the keys split over waves,
  // from the shortest key ranges to long ones (fp32, head dim 64, against the kernel below, us:
  // 2 x 8 heads, 960 queries and 77 keys 15.7 -> 10.0; 2 x 2, 4032 and as many 315 -> 179; one
  // head, 16320 and as many 1260 -> 694)
  if ((long long)((p.Sq + 63) / 64) * p.heads * p.B < cus) {
    if (D == 32)
      launch_keysplit<T, 32>(p, s);
    else if constexpr (sizeof(T) == 4)  // (bf16 with head dim 64 has returned)
      launch_keysplit<T, 64>(p, s);
    DN_HIP(hipGetLastError());
    return;
  }
  // The register-staged kernel: fewer, wider workgroups when there are many queries; two waves
  // per workgroup otherwise, so that short sequences still spread over every CU.
  const long long wg4 = (long long)((p.Sq + 127) / 128) * p.heads * p.B;
  if (wg4 >= 512) {
    dim3 grid((p.Sq + 127) / 128, p.heads, p.B);
    if (D == 64)
      launch<T, 64, 4>(grid, p, s);
    else
      launch<T, 32, 4>(grid, p, s);
  } else {
    dim3 grid((p.Sq + 63) / 64, p.heads, p.B);
    if (D == 64)
      launch<T, 64, 2>(grid, p, s);
    else
      launch<T, 32, 2>(grid, p, s);
  }
  DN_HIP(hipGetLastError());
}

template void attention<float>(const AttnParams&, int, int, hipStream_t);
template void attention<bf16>(const AttnParams&, int, int, hipStream_t);

}  // namespace dn
