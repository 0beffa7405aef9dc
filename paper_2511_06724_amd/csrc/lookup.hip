// Top-1 cosine search over the prompt-embedding cache (HBM-bound; gfx950).
//
// Pass 1: every half-wave (32 lanes) scores two cache rows per iteration — all
// 16-byte coalesced fp16 loads of both rows issued before any arithmetic, packed
// fp16 dot products accumulating in fp32 (v_dot2_f32_f16: the fp16 x fp16 products
// are exact in fp32) for q.c and c.c, then 5-step butterflies — and keeps its best
// (score, index); each workgroup writes the best of its 8 half-waves. Pass 2: one
// workgroup reduces the per-workgroup winners. Ties go to the lowest index at every
// stage, so the result is the first maximum, independent of the launch shape.
//
// Batched search (up to 64 queries per pass): the scores of 32-row tiles against all queries
// are [32 x dim] x [dim x 64] contractions on the matrix cores (v_mfma_f32_32x32x16_f16: fp16
// operands, exact products, fp32 sums), so the table is read from HBM once per 64 queries
// instead of once per query. The queries stay in registers, the rows stream through LDS. Row
// norms come from the same operands (packed fp16 dot products), and the top-1 per query is
// kept in registers while a wave walks its tiles.
#include "kernels.h"

namespace dn {
namespace {

constexpr int kScanBlocks = 2048;  // a multiple of 256 (the reduction's per-thread share)
constexpr int kQMaxVec = 4;  // fast path: dim <= 32 lanes * 4 vectors * 8 = 1024

struct Cand {
  float s;
  long long i;
};

__device__ __forceinline__ bool better(float s, long long i, float bs, long long bi) {
  return s > bs || (s == bs && i < bi);
}

__device__ __forceinline__ float h2f(uint16_t h) { return static_cast<float>(__builtin_bit_cast(_Float16, h)); }

__device__ __forceinline__ float half_sum(float v) {
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Score of one row (cosine up to the positive factor 1/|q|); -inf for a zero row.
__device__ __forceinline__ float row_score(float dot, float cc) { return cc > 0.f ? dot * rsqrtf(cc) : -INFINITY; }

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ h2 as_h2(unsigned u) { return __builtin_bit_cast(h2, u); }

// q . x and x . x over one 16-byte vector (8 fp16 values), accumulated in fp32.
__device__ __forceinline__ void dot8(const h2 (&qv)[4], const uint4 x, float& dot, float& cc) {
  const unsigned w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const h2 v = as_h2(w[k]);
    dot = __builtin_amdgcn_fdot2(qv[k], v, dot, false);
    cc = __builtin_amdgcn_fdot2(v, v, cc, false);
  }
}

template <int NQ>
__global__ __launch_bounds__(256) void scan_vec_kernel(const uint16_t* q, const uint16_t* cache, long long n, int dim,
                                                       Cand* part) {
  const int lane = threadIdx.x & 63;
  const int li = lane & 31;
  const int hw = threadIdx.x >> 5;  // half-wave in block, 0..7
  const int V = dim / 8;
  h2 qv[NQ][4];
  bool act[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    const int v = li + 32 * j;
    act[j] = v < V;
    const uint4 raw = act[j] ? ld16(q + v * 8) : make_uint4(0u, 0u, 0u, 0u);
    qv[j][0] = as_h2(raw.x);
    qv[j][1] = as_h2(raw.y);
    qv[j][2] = as_h2(raw.z);
    qv[j][3] = as_h2(raw.w);
  }
  float best_s = -INFINITY;
  long long best_i = n;
  const long long stride = (long long)gridDim.x * 16;
  // rows r and r + 1 per half-wave; past the end the second row re-reads row r and is not scored
  for (long long r = (long long)blockIdx.x * 16 + 2 * hw; r < n; r += stride) {
    const bool two = r + 1 < n;
    const uint16_t* c0 = cache + r * dim;
    const uint16_t* c1 = two ? c0 + dim : c0;
    uint4 x0[NQ], x1[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      const int v = act[j] ? li + 32 * j : 0;
      x0[j] = ld16(c0 + v * 8);
      x1[j] = ld16(c1 + v * 8);
    }
    float d0 = 0.f, s0 = 0.f, d1 = 0.f, s1 = 0.f;
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      if (!act[j]) continue;
      dot8(qv[j], x0[j], d0, s0);
      dot8(qv[j], x1[j], d1, s1);
    }
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) {
      d0 += __shfl_xor(d0, o, 64);
      s0 += __shfl_xor(s0, o, 64);
      d1 += __shfl_xor(d1, o, 64);
      s1 += __shfl_xor(s1, o, 64);
    }
    const float sc0 = row_score(d0, s0);
    if (better(sc0, r, best_s, best_i)) {
      best_s = sc0;
      best_i = r;
    }
    const float sc1 = row_score(d1, s1);
    if (two && better(sc1, r + 1, best_s, best_i)) {
      best_s = sc1;
      best_i = r + 1;
    }
  }
  __shared__ Cand red[8];
  if (li == 0) red[hw] = Cand{best_s, best_i};
  __syncthreads();
  if (threadIdx.x == 0) {
    Cand b = red[0];
    for (int k = 1; k < 8; ++k)
      if (better(red[k].s, red[k].i, b.s, b.i)) b = red[k];
    part[blockIdx.x] = b;
  }
}

// Any dim / alignment: element-wise loads, q staged in LDS.
__global__ __launch_bounds__(256) void scan_scalar_kernel(const uint16_t* q, const uint16_t* cache, long long n,
                                                          int dim, Cand* part) {
  extern __shared__ float qs[];
  for (int e = threadIdx.x; e < dim; e += 256) qs[e] = h2f(q[e]);
  __syncthreads();
  const int li = threadIdx.x & 31;
  const int hw = threadIdx.x >> 5;
  float best_s = -INFINITY;
  long long best_i = n;
  const long long stride = (long long)gridDim.x * 8;
  for (long long row = (long long)blockIdx.x * 8 + hw; row < n; row += stride) {
    const uint16_t* c = cache + row * dim;
    float dot = 0.f, cc = 0.f;
    for (int e = li; e < dim; e += 32) {
      const float x = h2f(c[e]);
      dot += qs[e] * x;
      cc += x * x;
    }
    dot = half_sum(dot);
    cc = half_sum(cc);
    const float s = row_score(dot, cc);
    if (better(s, row, best_s, best_i)) {
      best_s = s;
      best_i = row;
    }
  }
  __shared__ Cand red[8];
  if (li == 0) red[hw] = Cand{best_s, best_i};
  __syncthreads();
  if (threadIdx.x == 0) {
    Cand b = red[0];
    for (int k = 1; k < 8; ++k)
      if (better(red[k].s, red[k].i, b.s, b.i)) b = red[k];
    part[blockIdx.x] = b;
  }
}

// Level of the table for a result (index -1: nothing retrieved, level 0).
__device__ __forceinline__ int select_level(const KTable& kt, long long idx, float score) {
  if (idx < 0) return 0;
  int j = 0;
  for (int i = 0; i < kt.n; ++i)
    if (score >= kt.thr[i]) j = i + 1;
  return kt.level[j];
}

// Pass 2, one workgroup: every thread loads its (up to kScanBlocks / 256) winners
// before comparing them; waves reduce with shuffles, then the 4 wave winners in order.
// The squared norm of q (for the reported cosine) is summed alongside. The result may
// be written to pinned host memory.
__global__ __launch_bounds__(256) void reduce_kernel(const Cand* part, int nb, const uint16_t* q, int dim,
                                                     long long* idx, float* score, KTable kt, int* kout) {
  constexpr int kPer = kScanBlocks / 256;
  __shared__ float ws_s[4], ws_q[4];
  __shared__ long long ws_i[4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  Cand c[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int j = t + 256 * k;
    c[k] = j < nb ? part[j] : Cand{-INFINITY, 0x7fffffffffffffffll};
  }
  float qq = 0.f;
  for (int e = t; e < dim; e += 256) {
    const float x = h2f(q[e]);
    qq += x * x;
  }
  float bs = c[0].s;
  long long bi = c[0].i;
#pragma unroll
  for (int k = 1; k < kPer; ++k)
    if (better(c[k].s, c[k].i, bs, bi)) {
      bs = c[k].s;
      bi = c[k].i;
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float s2 = __shfl_xor(bs, o, 64);
    const long long i2 = __shfl_xor(bi, o, 64);
    if (better(s2, i2, bs, bi)) {
      bs = s2;
      bi = i2;
    }
    qq += __shfl_xor(qq, o, 64);
  }
  if (lane == 0) {
    ws_s[w] = bs;
    ws_i[w] = bi;
    ws_q[w] = qq;
  }
  __syncthreads();
  if (t == 0) {
    float qn = ws_q[0];
    for (int k = 1; k < 4; ++k) {
      if (better(ws_s[k], ws_i[k], bs, bi)) {
        bs = ws_s[k];
        bi = ws_i[k];
      }
      qn += ws_q[k];
    }
    // A zero query (or a cache of zero rows) has no defined cosine: report no row.
    const long long r = (qn > 0.f && bs > -INFINITY) ? bi : -1;
    const float sc = bs * rsqrtf(qn);
    *idx = r;
    *score = sc;
    if (kout) *kout = select_level(kt, r, sc);
  }
}


// ---------------------------------------------------------------- batched search

constexpr int kBatchQ = 64;        // queries per pass: two 32-query halves
constexpr int kBatchBlocks = 256;  // at most one workgroup per CU
// dims per LDS stage; a tile takes at least two stages
constexpr int stage_k(int dim) { return dim >= 512 ? 256 : 128; }
// 256 dims: tables from this many rows on split a tile's rows over the waves, not its dims.
constexpr int kRowSplitMin = 50000;

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// dim = 16 KS. Two row groups of four waves share a workgroup. Wave (qh, kh) of a group holds
// queries [32 qh, 32 qh + 32) over half kh of every stage's dims in registers (2 KS VGPRs: B
// operands of the 32x32x16 f16 matrix-core step, lane l query l % 32, dims 16 s + 8 (l / 32)
// ..), and the four waves score the group's 32-row tiles together: the kh = 1 halves of the
// sums and norms reach the kh = 0 wave through LDS, which scores a tile one stage later. ROWS: a
// wave holds its queries over all dims and scores half kh of a 64-row tile. At 256 dims the
// exchange and a barrier per 8 KB of rows cost long scans more than the longer query loads
// (64 queries, dims split -> rows split: 300,000 rows 42.0 -> 39.1 us, 100,000 21.6 -> 20.3,
// 30,000 12.4 -> 12.9, 2,000 8.7 -> 10.9). The rows go global -> LDS in 512-byte (256 dims: 256-byte) pieces into a ring
// of R stages per group, swizzled (16-byte chunk c of row r at position c ^ (r % 16)), so that
// the A operands are conflict-free 16-byte LDS reads. A group's rows are contiguous; rows past
// its range read its last row and are not scored.
// Bound by HBM (the table once per 64 queries). The previous form loaded the A operands
// straight from the table (64-byte pieces of 16 rows per load, half a line each) and re-read
// every query operand from LDS per 16-row tile, which its loads did not hide: 48.0 us for
// 100,000 x 768 against 39.2 us here; the table's own bound at the rate of a large copy
// (5.0 TB/s) is 30 us.
constexpr int kBatchGroups = 2, kBatchWaves = 4 * kBatchGroups;
constexpr int kRingBytes = 64 * 1024;  // per group

template <int KS, bool ROWS>
__global__ __launch_bounds__(kBatchWaves * 64) void scan_mfma_kernel(const uint16_t* q, int nq, const uint16_t* cache,
                                                                     int n, Cand* part) {
  constexpr int NG = kBatchGroups;
  constexpr int dim = 16 * KS, SK = stage_k(dim), ST = dim / SK;  // stages per tile
  constexpr int RB = 2 * SK;                                      // bytes of a row per stage
  constexpr int TR = ROWS ? 64 : 32;                              // rows per tile
  constexpr int SB = TR * RB, R = kRingBytes / SB;                // bytes per stage, ring depth
  constexpr int HS = ROWS ? SK / 16 : SK / 32;                   // k-steps per wave and stage
  constexpr int CPR = RB / 16, RPI = 64 / CPR;                    // 16-byte chunks per row, rows per DMA
  constexpr int DR = TR / 4, NI = DR / RPI;                       // rows, DMA instructions per wave and stage
  static_assert(ST >= 2, "the partial sums of a tile are read before the next tile's are written");
  constexpr int NR = ROWS ? 2 * NG : NG;                // winners per query to merge
  extern __shared__ __align__(16) unsigned char ring[];  // [group][R][TR rows][RB]
  __shared__ float half_acc[ROWS ? 1 : NG][2][16][64];
  __shared__ float half_cc[NG][2][32];
  __shared__ float inv[NG][4][32];
  __shared__ Cand red[NR][kBatchQ];
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int grp = w >> 2, qh = w & 1, kh = (w >> 1) & 1;
  const int r32 = lane & 31, h = lane >> 5;
  const int rb = ROWS ? 32 * kh : 0;         // the wave's first row of a tile
  const int dk = ROWS ? 0 : HS * kh;         // and its first k-step of a stage
  const bool scores = ROWS || kh == 0;
  // this group's rows [row0, row1): equal contiguous shares
  const int shares = (int)gridDim.x * NG, per = n / shares + (n % shares != 0);
  const long long begin = (long long)(blockIdx.x * NG + grp) * per;
  const int row0 = (int)(begin < n ? begin : n), row1 = (int)(begin + per < n ? begin + per : n);
  const int tiles = (per + TR - 1) / TR;  // the same for every group: barriers match
  const int total = tiles * ST;

  // DMA of stage g (tile g / ST, dims [SK (g % ST), + SK)): wave j of the group loads rows
  // [DR j, DR j + DR), RPI per instruction; stages past the end repeat the last one
  unsigned char* const gring = ring + grp * kRingBytes;
  const int drow = DR * (w & 3) + lane / CPR;
  const int last_row = row1 > 0 ? row1 - 1 : 0;
  int dg = 0, dbase = row0 < last_row ? row0 : last_row, dst = 0;  // next stage, its tile's first row, its dims
  auto issue = [&]() {
    unsigned char* slot = gring + (dg % R) * SB;
    const uint16_t* src = cache + (long long)dbase * dim + dst * SK;  // wave-uniform
    const int lim = last_row - dbase;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int row = drow + RPI * j;
      const unsigned off = (unsigned)min(row, lim) * (2 * dim) + (unsigned)(((lane % CPR) ^ (row & 15)) * 16);
      dma16_base(src, off, (lds_void*)(slot + (DR * (w & 3) + RPI * j) * RB));
    }
    ++dg;
    const bool more = dg < total, wrap = dst + 1 == ST;
    dbase = more && wrap ? min(dbase + TR, last_row) : dbase;
    dst = more ? (wrap ? 0 : dst + 1) : dst;
  };
#pragma unroll
  for (int s = 0; s < R - 1; ++s) issue();

  f16x8 qf[ST * HS];
  {
    const int qi = 32 * qh + r32;
    const uint16_t* qp = q + (long long)(qi < nq ? qi : 0) * dim + 16 * dk + 8 * h;
#pragma unroll
    for (int s = 0; s < ST * HS; ++s)
      qf[s] = *reinterpret_cast<const f16x8*>(qp + (s / HS) * SK + 16 * (s % HS));
    // landed before the loop: waits for them inside it would drain the ring's DMA every tile
#pragma unroll
    for (int s = 0; s < ST * HS; ++s) asm volatile("" : "+v"(qf[s]));
  }

  float best_s = -INFINITY;
  int best_i = n;
  // even and odd k-steps apart: half the length of the dependent chains
  f32x16 acc[2], prev;
  float cc[2] = {0.f, 0.f}, prev_cc = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = prev[r] = 0.f;
  // scores the wave's rows of tile `tile` from prev (dims split: plus the other half, in LDS)
  auto finish = [&](int tile) {
    const float c2 = ROWS ? prev_cc : prev_cc + half_cc[grp][qh][r32];
    inv[grp][w & 3][r32] = c2 > 0.f ? rsqrtf(c2) : -1.f;  // 1 / |c| of row r32, -1 for a zero row
    const int base = tile * TR + rb;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      // c_row . q_(32 qh + r32), row = 8 (r / 4) + 4 h + r % 4: rows ascend with r
      const int rr = 8 * (r >> 2) + 4 * h + (r & 3);
      const float iv = inv[grp][w & 3][rr];
      const float dot = ROWS ? prev[r] : prev[r] + half_acc[grp][qh][r][lane];
      const float sc = iv > 0.f ? dot * iv : -INFINITY;
      if (base + rr < row1 - row0 && sc > best_s) {
        best_s = sc;
        best_i = row0 + base + rr;
      }
    }
  };
  int g = 0;
  for (int tile = 0; tile < tiles; ++tile) {
#pragma unroll
    for (int st = 0; st < ST; ++st, ++g) {
      // this wave's DMA of stage g has landed (R - 2 later stages of NI loads follow it);
      // after the barrier every wave's has, and every wave is done with stage g - 1, whose
      // slot takes stage g + R - 1
      __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0((R - 2) * NI));
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      issue();
      const unsigned char* slot = gring + (g % R) * SB + (rb + r32) * RB;
#pragma unroll
      for (int s = 0; s < HS; ++s) {
        const f16x8 a = *reinterpret_cast<const f16x8*>(slot + (((2 * (dk + s) + h) ^ (r32 & 15)) * 16));
        acc[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, qf[st * HS + s], acc[s & 1], 0, 0, 0);
        const uint4 u = __builtin_bit_cast(uint4, a);
        const unsigned wd[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) cc[k & 1] = __builtin_amdgcn_fdot2(as_h2(wd[k]), as_h2(wd[k]), cc[k & 1], false);
      }
      // the norm's terms are taken here (the compiler would sink them to the tile's end and
      // keep every operand until then)
      asm volatile("" : "+v"(cc[0]), "+v"(cc[1]));
      if (st == 0 && scores && tile > 0) finish(tile - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    prev = acc[0] + acc[1];
    prev_cc = cc[0] + cc[1];
    prev_cc += __shfl_xor(prev_cc, 32, 64);
    if (!scores) {
#pragma unroll
      for (int r = 0; r < 16; ++r) half_acc[grp][qh][r][lane] = prev[r];
      half_cc[grp][qh][r32] = prev_cc;
    }
    cc[0] = cc[1] = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.f;
  }
  __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
  __syncthreads();
  if (scores) {
    finish(tiles - 1);
    // the two lane halves of a query
    const float s2 = __shfl_xor(best_s, 32, 64);
    const int i2 = __shfl_xor(best_i, 32, 64);
    if (better(s2, i2, best_s, best_i)) {
      best_s = s2;
      best_i = i2;
    }
    if (h == 0) red[ROWS ? 2 * grp + kh : grp][32 * qh + r32] = Cand{best_s, best_i};
  }
  __syncthreads();
  if (t < kBatchQ) {
    Cand b = red[0][t];
    for (int k = 1; k < NR; ++k)
      if (better(red[k][t].s, red[k][t].i, b.s, b.i)) b = red[k][t];
    part[(long long)blockIdx.x * kBatchQ + t] = b;
  }
}

// One workgroup per query: the nb workgroup winners of its column, and |q|^2 for the
// reported cosine. Writes idx[j] = -1 where the query has no defined cosine.
__global__ __launch_bounds__(256) void reduce_batch_kernel(const Cand* part, int nb, const uint16_t* q, int dim,
                                                           long long* idx, float* score, KTable kt, int* kout) {
  __shared__ float ws_s[4], ws_q[4];
  __shared__ long long ws_i[4];
  const int j = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  Cand c = t < nb ? part[(long long)t * kBatchQ + j] : Cand{-INFINITY, 0x7fffffffffffffffll};
  float qq = 0.f;
  for (int e = t; e < dim; e += 256) {
    const float x = h2f(q[(long long)j * dim + e]);
    qq += x * x;
  }
  float bs = c.s;
  long long bi = c.i;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float s2 = __shfl_xor(bs, o, 64);
    const long long i2 = __shfl_xor(bi, o, 64);
    if (better(s2, i2, bs, bi)) {
      bs = s2;
      bi = i2;
    }
    qq += __shfl_xor(qq, o, 64);
  }
  if (lane == 0) {
    ws_s[w] = bs;
    ws_i[w] = bi;
    ws_q[w] = qq;
  }
  __syncthreads();
  if (t == 0) {
    float qn = ws_q[0];
    for (int k = 1; k < 4; ++k) {
      if (better(ws_s[k], ws_i[k], bs, bi)) {
        bs = ws_s[k];
        bi = ws_i[k];
      }
      qn += ws_q[k];
    }
    const long long r = (qn > 0.f && bs > -INFINITY) ? bi : -1;
    const float sc = bs * rsqrtf(qn);
    idx[j] = r;
    score[j] = sc;
    if (kout) kout[j] = select_level(kt, r, sc);
  }
}

// Launches the scan over at most 256 workgroups, each group with at least a tile's rows where
// the table has them; returns that count.
template <int KS, bool ROWS = false>
int launch_batch(const uint16_t* q, int nq, const uint16_t* cache, int n, Cand* part, hipStream_t s) {
  const int rows = (ROWS ? 64 : 32) * kBatchGroups;
  const int want = n / rows + (n % rows != 0);
  const int nb = want < kBatchBlocks ? want : kBatchBlocks;
  const size_t lds = (size_t)kBatchGroups * kRingBytes;
  static bool attr = false;  // per process: the attribute belongs to the code object
  if (!attr) {
    DN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&(scan_mfma_kernel<KS, ROWS>)),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    attr = true;
  }
  hipLaunchKernelGGL((scan_mfma_kernel<KS, ROWS>), dim3(nb), dim3(kBatchWaves * 64), lds, s, q, nq, cache, n, part);
  return nb;
}

}  // namespace

size_t lookup_workspace_bytes() { return sizeof(Cand) * kScanBlocks; }

void lookup(const uint16_t* q, const uint16_t* cache, long long n, int dim, void* ws, long long* idx_out,
            float* score_out, hipStream_t s, const KTable* kt, int* k_out) {
  DN_CHECK(n >= 1 && dim >= 1, "lookup: empty cache");
  Cand* part = static_cast<Cand*>(ws);
  const long long want = (n + 15) / 16;
  const int nb = static_cast<int>(want < kScanBlocks ? want : kScanBlocks);
  const bool aligned = (reinterpret_cast<uintptr_t>(cache) % 16 == 0) && (reinterpret_cast<uintptr_t>(q) % 16 == 0);
  const int V = dim / 8;
  if (aligned && dim % 8 == 0 && V <= 32 * kQMaxVec) {
    const int nq = (V + 31) / 32;
    if (nq == 1)
      hipLaunchKernelGGL(scan_vec_kernel<1>, dim3(nb), dim3(256), 0, s, q, cache, n, dim, part);
    else if (nq == 2)
      hipLaunchKernelGGL(scan_vec_kernel<2>, dim3(nb), dim3(256), 0, s, q, cache, n, dim, part);
    else if (nq == 3)
      hipLaunchKernelGGL(scan_vec_kernel<3>, dim3(nb), dim3(256), 0, s, q, cache, n, dim, part);
    else
      hipLaunchKernelGGL(scan_vec_kernel<4>, dim3(nb), dim3(256), 0, s, q, cache, n, dim, part);
  } else {
    DN_CHECK(dim <= 16384, "lookup: dim too large for the scalar path");
    hipLaunchKernelGGL(scan_scalar_kernel, dim3(nb), dim3(256), dim * sizeof(float), s, q, cache, n, dim, part);
  }
  const KTable tab = kt ? *kt : KTable();
  hipLaunchKernelGGL(reduce_kernel, dim3(1), dim3(256), 0, s, part, nb, q, dim, idx_out, score_out, tab,
                     kt ? k_out : nullptr);
  DN_HIP(hipGetLastError());
}

}  // namespace dn

namespace dn {

size_t lookup_batch_workspace_bytes() { return sizeof(Cand) * kBatchBlocks * kBatchQ; }

int lookup_batch_max_queries() { return kBatchQ; }

bool lookup_batch_supported(const uint16_t* q, const uint16_t* cache, long long n, int dim) {
  if (n > (1ll << 31) - 64) return false;  // 32-bit row indices in the scan
  const bool aligned = (reinterpret_cast<uintptr_t>(cache) % 16 == 0) && (reinterpret_cast<uintptr_t>(q) % 16 == 0);
  return aligned && (dim == 256 || dim == 512 || dim == 768 || dim == 1024);
}

void lookup_batch(const uint16_t* q, int nq, const uint16_t* cache, long long n, int dim, void* ws,
                  long long* idx_out, float* score_out, hipStream_t s, const KTable* kt, int* k_out) {
  DN_CHECK(n >= 1 && dim >= 1, "lookup_batch: empty cache");
  DN_CHECK(nq >= 1 && nq <= kBatchQ, "lookup_batch: 1 to 64 queries per pass");
  DN_CHECK(lookup_batch_supported(q, cache, n, dim),
           "lookup_batch: dim must be 256, 512, 768 or 1024, 16-byte aligned, n < 2^31 - 64");
  const int n32 = static_cast<int>(n);
  Cand* part = static_cast<Cand*>(ws);
  int nb = 0;
  switch (dim) {
    case 256:
      nb = n32 >= kRowSplitMin ? launch_batch<16, true>(q, nq, cache, n32, part, s)
                               : launch_batch<16>(q, nq, cache, n32, part, s);
      break;
    case 512: nb = launch_batch<32>(q, nq, cache, n32, part, s); break;
    case 768: nb = launch_batch<48>(q, nq, cache, n32, part, s); break;
    default: nb = launch_batch<64>(q, nq, cache, n32, part, s); break;
  }
  const KTable tab = kt ? *kt : KTable();
  hipLaunchKernelGGL(reduce_batch_kernel, dim3(nq), dim3(256), 0, s, part, nb, q, dim, idx_out, score_out, tab,
                     kt ? k_out : nullptr);
  DN_HIP(hipGetLastError());
}

}  // namespace dn
