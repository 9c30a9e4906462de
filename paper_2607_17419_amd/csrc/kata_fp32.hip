// kata_fp32.hip -- fp32 VALU kernels of libkata: the general-shape chunked
// forward (any d <= 64, dv <= 256, C <= 128, fp32 or bf16 inputs), the state
// prefill, the recurrent decode step, and the exclusive associative scan over
// chunk states that both forward paths use.
//
// Feature layout: packed row-major upper triangle, f(a, b) = a*d - a(a-1)/2 + b - a.
// With g > 1 feature blocks (KATA-Mg, section "From rank-one rays to low-rank
// PSD packing": one rank-one factor per block of m = d/g coordinates) the
// features of block i are the pairs of coordinates inside it, packed the same
// way over m, at offset i*m(m+1)/2; n = g*m(m+1)/2, and the score of a
// (query, key) pair is sum_i (q_i . k_i)^2.  g = 1 is KATA-M1.
// A chunk-state record is S[f][j] (n x dv) followed by z[f] (n), fp32.
#include <type_traits>

#include "kata_common.hpp"
#include "kata_internal.hpp"
#include "kata_scan.hpp"

namespace kata {

// Pair table for packed features: entry f holds (a, b) in the low/high byte.
__device__ __forceinline__ void build_pair_table(uint16_t* tab, int d, int g) {
  const int m = d / g, nm = m * (m + 1) / 2;
  for (int x = threadIdx.x; x < d; x += blockDim.x) {
    const int blk = x / m, a = x % m;
    for (int b = a; b < m; ++b)
      tab[blk * nm + packed_index(a, b, m)] =
          static_cast<uint16_t>((blk * m + a) | ((blk * m + b) << 8));
  }
}

// The pair (a, b) of feature f (one thread's lookup, no table).
__device__ __forceinline__ uint16_t pair_of(int f, int d, int g) {
  const int m = d / g, nm = m * (m + 1) / 2;
  const int blk = f / nm, fl = f % nm;
  int a = 0;
  while (a + 1 < m && packed_index(a + 1, a + 1, m) <= fl) ++a;
  const int b = a + (fl - packed_index(a, a, m));
  return static_cast<uint16_t>((blk * m + a) | ((blk * m + b) << 8));
}

// ---------------------------------------------------------------------------
// Chunk state (eq. chunk-SZ) on the matrix cores: for chunk c of head bh, over
// tokens [c*C, min(c*C + C, T)),  S[f][j] = sum_t k_a k_b v_j,
// z[f] = sum_t k_a k_b.  With C >= T and one chunk this is the prefill state.
//
// A tile is 32 features by all dv columns (NT tiles of 32).  Rows of k and v
// are staged transposed ([dim][token]) in blocks of kSTB tokens, so that a
// lane reads 8 (bf16) or 4 (fp32) consecutive tokens of its feature's two
// coordinates at once; the next block's rows are in registers meanwhile.
//   bf16 inputs: a feature k_a k_b has at most 16 significant bits, so it is
//     the sum of two bf16 values exactly (the fp32 product truncated to 8
//     bits, and the rest); two bf16 MFMAs per tile then add exact products in
//     fp32.  The vector products and splits, about 56 instructions for four
//     MFMAs, bound the loop.  A product that overflows fp32 has no such split
//     (inf - inf), nor has an infinite v against a zero rest: a tile whose sums
//     are not finite is formed again in fp32, on the matrix cores (B4 H16 T2000
//     with one NaN in v 0.42 ms, T8192 of one head 1.2 ms; one thread per output
//     took 5.9 and 1.6 ms, scalar sums per lane here 8 and 30 ms).
//   fp32 inputs: fp32 MFMAs (v_mfma_f32_32x32x2_f32), whose rate bounds it.
// B4 H16 T2000 d64 bf16: 5.90 ms with one thread per output and scalar fp32
// sums, 0.117 ms here.
// SPLIT 1: each of the workgroup's four waves owns a tile.  SPLIT 4: the waves
// share one tile, each taking every fourth K-step, and add their sums in LDS
// in wave order; four times the workgroups, for calls with few heads.
// 128-token blocks measured 143-152 us at that shape; three or five waves per
// SIMD instead of four 143 and 142 us.
// grid (ceil(tiles * SPLIT / 4), NC, BH), block 256.
// ---------------------------------------------------------------------------

constexpr int kSTB = 64;  // tokens staged per block

typedef float st_f32x4 __attribute__((ext_vector_type(4)));

// LDS element and row length (elements) of the transposed rows: an odd number
// of 16-byte pieces, so that 16-byte reads of 16 consecutive rows cover all
// banks.
template <typename Tin> struct StateLds;
template <> struct StateLds<bf16_t> { using T = uint16_t; static constexpr int S = kSTB + 8; };
template <> struct StateLds<float> { using T = float; static constexpr int S = kSTB + 4; };

__device__ __forceinline__ uint16_t state_raw(bf16_t x) { return x.bits; }
__device__ __forceinline__ float state_raw(float x) { return x; }

// Tokens past the chunk are zero in LDS, and so are columns past dv.
template <typename Tin, int NT, int SPLIT>
__global__ __launch_bounds__(256, NT <= 2 ? (std::is_same<Tin, bf16_t>::value ? 4 : 3) : 1) void chunk_state_mf(
    const Tin* __restrict__ k, const Tin* __restrict__ v, float* __restrict__ S_out,
    float* __restrict__ z_out, int T, int d, int dv, int C, int g, long long S_bh_stride,
    long long S_chunk_stride, long long z_bh_stride, long long z_chunk_stride) {
  using LT = typename StateLds<Tin>::T;
  constexpr int LS = StateLds<Tin>::S;
  constexpr bool BF = std::is_same<Tin, bf16_t>::value;
  constexpr int DVP = 32 * NT;
  constexpr int kRed = SPLIT > 1 ? (4 / SPLIT) * 64 * (16 * NT + 1) * 4 : 0;  // bytes of one wave's sums
  constexpr int kStage = (64 + DVP) * LS * static_cast<int>(sizeof(LT));
  __shared__ __attribute__((aligned(16))) char lds[kStage > kRed ? kStage : kRed];
  LT* kT = reinterpret_cast<LT*>(lds);  // [64][LS]
  LT* vT = kT + 64 * LS;                // [DVP][LS]
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, h = lane >> 5;
  const int n = g * ((d / g) * (d / g + 1) / 2);
  const int tile = blockIdx.x * (4 / SPLIT) + w / SPLIT;
  const int ws = w % SPLIT;  // this wave's share of the K-steps
  const int bh = blockIdx.z;
  const long long t_begin = static_cast<long long>(blockIdx.y) * C;
  const long long t_end = min(static_cast<long long>(T), t_begin + C);
  const Tin* kh = k + static_cast<long long>(bh) * T * d;
  const Tin* vh = v + static_cast<long long>(bh) * T * dv;
  const int f = 32 * tile + c;
  const uint16_t pr = pair_of(f < n ? f : 0, d, g);  // features past n: computed, not stored
  const int fa = pr & 0xFF, fb = pr >> 8;

  // Staging.  Rows of whole 16-byte pieces (d and dv multiples of 8 in bf16,
  // of 4 in fp32): a task is 8 columns of a token pair (bf16) or 4 columns of
  // a token (fp32), the lanes of a wave on consecutive tokens, whose LDS words
  // are neighbours.  Other widths go one element at a time.
  constexpr int CPP = BF ? 8 : 4;              // columns per piece
  constexpr int TOK = BF ? kSTB / 2 : kSTB;    // tasks per column group
  constexpr int MAXT = (TOK * (64 + DVP) / CPP + 255) / 256;
  const bool vec = d % CPP == 0 && dv % CPP == 0;
  uint4 pc[MAXT][BF ? 2 : 1];
  const int kg = d / CPP, ngrp = kg + dv / CPP;
  auto fetch = [&](long long t0) {
#pragma unroll
    for (int i = 0; i < MAXT; ++i) {
      const int task = tid + 256 * i, cg = task / TOK, p = task % TOK;
#pragma unroll
      for (int e = 0; e < (BF ? 2 : 1); ++e) {
        pc[i][e] = make_uint4(0u, 0u, 0u, 0u);
        const long long t = t0 + (BF ? 2 * p + e : p);
        if (cg >= ngrp || t >= t_end) continue;
        const Tin* row = cg < kg ? kh + t * d + CPP * cg : vh + t * dv + CPP * (cg - kg);
        pc[i][e] = *reinterpret_cast<const uint4*>(row);
      }
    }
  };
  auto commit = [&]() {
#pragma unroll
    for (int i = 0; i < MAXT; ++i) {
      const int task = tid + 256 * i, cg = task / TOK, p = task % TOK;
      if (cg >= ngrp) continue;
      LT* row = cg < kg ? kT + CPP * cg * LS : vT + CPP * (cg - kg) * LS;
      uint32_t* dst = reinterpret_cast<uint32_t*>(row) + p;
      const uint32_t a[4] = {pc[i][0].x, pc[i][0].y, pc[i][0].z, pc[i][0].w};
      if constexpr (BF) {
        const uint32_t b[4] = {pc[i][1].x, pc[i][1].y, pc[i][1].z, pc[i][1].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          dst[(2 * e) * (LS / 2)] = __builtin_amdgcn_perm(b[e], a[e], 0x05040100u);
          dst[(2 * e + 1) * (LS / 2)] = __builtin_amdgcn_perm(b[e], a[e], 0x07060302u);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[e * LS] = a[e];
      }
    }
  };
  auto stage_elems = [&](long long t0) {
    for (int i = tid; i < kSTB * d; i += 256) {
      const int t = i / d, a = i % d;
      kT[a * LS + t] = t0 + t < t_end ? state_raw(kh[(t0 + t) * d + a]) : LT(0);
    }
    for (int i = tid; i < kSTB * dv; i += 256) {
      const int t = i / dv, j = i % dv;
      vT[j * LS + t] = t0 + t < t_end ? state_raw(vh[(t0 + t) * dv + j]) : LT(0);
    }
  };
  // columns past dv stay zero throughout
  for (int i = tid; i < (DVP - dv) * LS; i += 256) vT[dv * LS + i] = LT(0);

  f32x16 acc[NT];
#pragma unroll
  for (int m = 0; m < NT; ++m) acc[m] = f32x16{};
  float zacc = 0.f;
  const LT* ra = kT + fa * LS;
  const LT* rb = kT + fb * LS;
  const LT* rv = vT + c * LS;

  if (vec) fetch(t_begin);
  for (long long t0 = t_begin; t0 < t_end; t0 += kSTB) {
    __syncthreads();  // the previous block's readers are done
    if (vec) commit();
    else stage_elems(t0);
    __syncthreads();
    if (vec) fetch(t0 + kSTB);  // zeros past the chunk, no loads
    if constexpr (BF) {
#pragma unroll
      for (int kk = 0; kk < kSTB / 16 / SPLIT; ++kk) {
        const int o = 16 * (kk * SPLIT + ws) + 8 * h;
        const uint4 xa4 = *reinterpret_cast<const uint4*>(ra + o);
        const uint4 xb4 = *reinterpret_cast<const uint4*>(rb + o);
        const uint32_t xa[4] = {xa4.x, xa4.y, xa4.z, xa4.w}, xb[4] = {xb4.x, xb4.y, xb4.z, xb4.w};
        uint32_t ph[4], pl[4];
        float zs = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p0 = bf16lo_f32(xa[e]) * bf16lo_f32(xb[e]);
          const float p1 = bf16hi_f32(xa[e]) * bf16hi_f32(xb[e]);
          zs += p0 + p1;
          const uint32_t u0 = __float_as_uint(p0), u1 = __float_as_uint(p1);
          ph[e] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
          const float r0 = p0 - __uint_as_float(u0 & 0xFFFF0000u);
          const float r1 = p1 - __uint_as_float(u1 & 0xFFFF0000u);
          pl[e] = __builtin_amdgcn_perm(__float_as_uint(r1), __float_as_uint(r0), 0x07060302u);
        }
        zacc += zs;
        const bf16x8 ah = __builtin_bit_cast(bf16x8, make_uint4(ph[0], ph[1], ph[2], ph[3]));
        const bf16x8 al = __builtin_bit_cast(bf16x8, make_uint4(pl[0], pl[1], pl[2], pl[3]));
#pragma unroll
        for (int m = 0; m < NT; ++m) {
          const bf16x8 b = *reinterpret_cast<const bf16x8*>(rv + 32 * m * LS + o);
          acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, b, acc[m], 0, 0, 0);
          acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, b, acc[m], 0, 0, 0);
        }
      }
    } else {
      // 8 tokens per step: lane group h holds tokens 4h .. 4h+3, one per MFMA
      // (the order of the tokens inside a sum is free)
#pragma unroll 2
      for (int kk = 0; kk < kSTB / 8 / SPLIT; ++kk) {
        const int o = 8 * (kk * SPLIT + ws) + 4 * h;
        const st_f32x4 p = *reinterpret_cast<const st_f32x4*>(ra + o) *
                           *reinterpret_cast<const st_f32x4*>(rb + o);
        zacc += (p[0] + p[1]) + (p[2] + p[3]);
#pragma unroll
        for (int m = 0; m < NT; ++m) {
          const st_f32x4 b = *reinterpret_cast<const st_f32x4*>(rv + 32 * m * LS + o);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(p[e], b[e], acc[m], 0, 0, 0);
        }
      }
    }
  }
  if constexpr (SPLIT > 1) {
    // the tile's first wave collects the other waves' sums, one at a time
    float* red = reinterpret_cast<float*>(lds) + (w / SPLIT) * (16 * NT + 1) * 64;
    for (int s = 1; s < SPLIT; ++s) {
      __syncthreads();
      if (ws == s) {
#pragma unroll
        for (int m = 0; m < NT; ++m)
#pragma unroll
          for (int r = 0; r < 16; ++r) red[(16 * m + r) * 64 + lane] = acc[m][r];
        red[16 * NT * 64 + lane] = zacc;
      }
      __syncthreads();
      if (ws == 0) {
#pragma unroll
        for (int m = 0; m < NT; ++m)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[m][r] += red[(16 * m + r) * 64 + lane];
        zacc += red[16 * NT * 64 + lane];
      }
    }
    if (ws != 0) return;
  }
  zacc += __shfl_xor(zacc, 32);
  float* So = S_out + bh * S_bh_stride + blockIdx.y * S_chunk_stride;
  float* zo = z_out + bh * z_bh_stride + blockIdx.y * z_chunk_stride;
  if constexpr (BF) {
    float worst = 0.f;
#pragma unroll
    for (int m = 0; m < NT; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) worst += acc[m][r] - acc[m][r];  // 0, or NaN
    if (__builtin_expect(__any(!(worst == 0.f)), 0)) {
      // the tile again from the inputs, with fp32 products and sums on the fp32
      // matrix cores, one token per lane half (z is such a sum already)
      constexpr int U = NT <= 2 ? 8 : 4;
#pragma unroll
      for (int m = 0; m < NT; ++m) acc[m] = f32x16{};
#pragma unroll 1
      for (long long t0 = t_begin; t0 < t_end; t0 += 2 * U) {
        const Tin* kr = kh + t0 * d;
        const Tin* vr = vh + t0 * dv;
        const int left = static_cast<int>(min(t_end - t0, static_cast<long long>(2 * U)));
        float p[U], x[U][NT];
#pragma unroll
        for (int e = 0; e < U; ++e) {
          const bool in = 2 * e + h < left;
          const int t = in ? 2 * e + h : 0;
          p[e] = to_f32(kr[t * d + fa]) * to_f32(kr[t * d + fb]);
          if (!in) p[e] = 0.f;
#pragma unroll
          for (int m = 0; m < NT; ++m) {
            const float y = to_f32(vr[t * dv + min(32 * m + c, dv - 1)]);
            x[e][m] = in ? y : 0.f;  // columns past dv are not stored
          }
        }
#pragma unroll
        for (int e = 0; e < U; ++e)
#pragma unroll
          for (int m = 0; m < NT; ++m)
            acc[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(p[e], x[e][m], acc[m], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int m = 0; m < NT; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int fr = 32 * tile + 8 * (r >> 2) + 4 * h + (r & 3), j = 32 * m + c;
      if (fr < n && j < dv) So[static_cast<long long>(fr) * dv + j] = acc[m][r];
    }
  if (h == 0 && f < n) zo[f] = zacc;
}

// Launches chunk_state_mf over NC chunks of BH heads.  SPLIT 4 below 400 tiles
// in all (one wave each on 1024 SIMDs): 65 tiles over 8192 tokens take 0.10 ms
// split; at 520 tiles of 2000 tokens 47 us whole against 52 us split, at 1040
// 58 against 95 us.
constexpr int kSplitTiles = 400;

template <typename Tin>
void launch_chunk_state(const void* k, const void* v, float* S, float* z, int BH, int T, int d,
                        int dv, int C, int NC, int g, long long S_bh, long long S_c,
                        long long z_bh, long long z_c, hipStream_t st) {
  const int n = g * ((d / g) * (d / g + 1) / 2);
  const int tiles = (n + 31) / 32;
  const bool split = static_cast<long long>(tiles) * NC * BH < kSplitTiles;
  auto go = [&](auto nt_c) {
    constexpr int NT = decltype(nt_c)::value;
    const Tin* kp = static_cast<const Tin*>(k);
    const Tin* vp = static_cast<const Tin*>(v);
    if (split)
      chunk_state_mf<Tin, NT, 4><<<dim3(tiles, NC, BH), 256, 0, st>>>(
          kp, vp, S, z, T, d, dv, C, g, S_bh, S_c, z_bh, z_c);
    else
      chunk_state_mf<Tin, NT, 1><<<dim3((tiles + 3) / 4, NC, BH), 256, 0, st>>>(
          kp, vp, S, z, T, d, dv, C, g, S_bh, S_c, z_bh, z_c);
  };
  if (dv <= 32) go(std::integral_constant<int, 1>{});
  else if (dv <= 64) go(std::integral_constant<int, 2>{});
  else if (dv <= 128) go(std::integral_constant<int, 4>{});
  else go(std::integral_constant<int, 8>{});
}

// ---------------------------------------------------------------------------
// Chunk output (eq. chunk-out): for chunk c of head bh,
//   P[r][s] = sum_i (q_{r,i} . k_{s,i})^2 over the g blocks, for s <= r
//   (lower-triangular mask incl. diagonal),
//   N = Phi_w(Q_c) S_pre + P V_c,  D = Phi_w(Q_c) z_pre + P 1,  O = N / D (0 if D = 0),
// Phi_w the query-side packed feature (weight 2 off the diagonal).
// grid (NC, BH), block 256; C <= 128, d <= 64.
// ---------------------------------------------------------------------------
template <typename Tin>
__global__ __launch_bounds__(256) void chunk_out_f32(
    const Tin* __restrict__ q, const Tin* __restrict__ k, const Tin* __restrict__ v,
    const float* __restrict__ pre, float* __restrict__ out, int T, int d, int dv, int C, int g,
    long long bh_stride, long long chunk_stride) {
  extern __shared__ float smem[];
  const int m = d / g;
  const int n = g * (m * (m + 1) / 2);
  float* qs = smem;                 // [C][d]
  float* ks = qs + C * d;           // [C][d]
  float* P = ks + C * d;            // [C][C]
  float* Dn = P + C * C;            // [C]
  uint16_t* pairs = reinterpret_cast<uint16_t*>(Dn + C);  // [n]
  const int c = blockIdx.x;
  const int bh = blockIdx.y;
  const int tid = threadIdx.x;
  const long long t0 = static_cast<long long>(c) * C;
  const int nt = static_cast<int>(min(static_cast<long long>(C), T - t0));
  const Tin* qh = q + static_cast<long long>(bh) * T * d;
  const Tin* kh = k + static_cast<long long>(bh) * T * d;
  const Tin* vh = v + static_cast<long long>(bh) * T * dv;
  build_pair_table(pairs, d, g);
  for (int i = tid; i < C * d; i += 256) {
    int r = i / d, a = i % d;
    qs[i] = (r < nt) ? load_f32(qh, (t0 + r) * d + a) : 0.f;
    ks[i] = (r < nt) ? load_f32(kh, (t0 + r) * d + a) : 0.f;
  }
  __syncthreads();
  for (int i = tid; i < C * C; i += 256) {
    int r = i / C, s = i % C;
    float p = 0.f;
    if (s <= r)
      for (int blk = 0; blk < g; ++blk) {
        float a = 0.f;
        for (int x = blk * m; x < blk * m + m; ++x) a += qs[r * d + x] * ks[s * d + x];
        p += a * a;
      }
    P[i] = p;
  }
  __syncthreads();
  const float* Sp = pre + bh * bh_stride + c * chunk_stride;
  const float* zp = Sp + static_cast<long long>(n) * dv;
  for (int r = tid; r < C; r += 256) {
    float D = 0.f;
    for (int f = 0; f < n; ++f) {
      int a = pairs[f] & 0xFF, b = pairs[f] >> 8;
      float w = (a == b) ? 1.f : 2.f;
      D += (w * qs[r * d + a] * qs[r * d + b]) * zp[f];
    }
    for (int s = 0; s < C; ++s) D += P[r * C + s];
    Dn[r] = D;
  }
  __syncthreads();
  for (int o = tid; o < nt * dv; o += 256) {
    int r = o / dv, j = o % dv;
    float acc = 0.f;
    for (int f = 0; f < n; ++f) {
      int a = pairs[f] & 0xFF, b = pairs[f] >> 8;
      float w = (a == b) ? 1.f : 2.f;
      acc += (w * qs[r * d + a] * qs[r * d + b]) * Sp[static_cast<long long>(f) * dv + j];
    }
    for (int s = 0; s <= r; ++s) acc += P[r * C + s] * load_f32(vh, (t0 + s) * dv + j);
    float D = Dn[r];
    out[(static_cast<long long>(bh) * T + t0 + r) * dv + j] = (D > 0.f) ? acc / D : 0.f;
  }
}

// ---------------------------------------------------------------------------
// Decode step (eq. linatt's recurrence + normalised readout with the updated
// state).  One workgroup per head; S is streamed once (read-modify-write).
// grid BH, block 256; d <= 64, dv <= 256.
// ---------------------------------------------------------------------------
// S rows per thread whose loads are in flight together.  26 divides the 130
// rows each thread walks at n = 2080, dv = 64 and still fits 256 VGPRs
// (measured against 8, 16, 32, 40 and 48).
constexpr int kDecodeUnroll = 26;

// The state is touched once per step: stream it past the caches (non-temporal
// loads and stores; together they raise the step from 5.1 to 5.85 TB/s).
typedef float decode_f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 stream_load4(const float* p) {
  const decode_f4 t = __builtin_nontemporal_load(reinterpret_cast<const decode_f4*>(p));
  return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void stream_store4(float* p, float4 s) {
  const decode_f4 t = {s.x, s.y, s.z, s.w};
  __builtin_nontemporal_store(t, reinterpret_cast<decode_f4*>(p));
}

template <typename Tin>
__global__ __launch_bounds__(256) void decode_step_f32(float* __restrict__ S,
                                                       float* __restrict__ z,
                                                       const Tin* __restrict__ q,
                                                       const Tin* __restrict__ k,
                                                       const Tin* __restrict__ v,
                                                       float* __restrict__ out, int d, int dv,
                                                       int g) {
  __shared__ float qs[64], ks[64], vs[256];
  __shared__ uint16_t pairs[2080];
  __shared__ float red[256][5];
  const int n = g * ((d / g) * (d / g + 1) / 2);
  const int bh = blockIdx.x;
  const int tid = threadIdx.x;
  build_pair_table(pairs, d, g);
  if (tid < d) {
    qs[tid] = load_f32(q, static_cast<long long>(bh) * d + tid);
    ks[tid] = load_f32(k, static_cast<long long>(bh) * d + tid);
  }
  for (int j = tid; j < dv; j += 256) vs[j] = load_f32(v, static_cast<long long>(bh) * dv + j);
  __syncthreads();
  float* Sh = S + static_cast<long long>(bh) * n * dv;
  float* zh = z + static_cast<long long>(bh) * n;
  float num[4] = {0.f, 0.f, 0.f, 0.f};
  float den = 0.f;
  int jbase = 0;
  const bool vec = (dv % 4 == 0) && (256 % (dv / 4) == 0);
  if (vec) {
    // float4 stream: thread owns columns [4*(tid % (dv/4)), +4) of rows
    // tid / (dv/4), + 256/(dv/4), ...
    const int g = dv / 4;
    const int rows_per_pass = 256 / g;
    jbase = 4 * (tid % g);
    const float v0 = vs[jbase + 0], v1 = vs[jbase + 1], v2 = vs[jbase + 2], v3 = vs[jbase + 3];
    auto row = [&](int f, float4 s) {
      const int a = pairs[f] & 0xFF, b = pairs[f] >> 8;
      const float pk = ks[a] * ks[b];
      const float pq = ((a == b) ? 1.f : 2.f) * qs[a] * qs[b];
      s.x += pk * v0;
      s.y += pk * v1;
      s.z += pk * v2;
      s.w += pk * v3;
      stream_store4(Sh + static_cast<long long>(f) * dv + jbase, s);
      num[0] += pq * s.x;
      num[1] += pq * s.y;
      num[2] += pq * s.z;
      num[3] += pq * s.w;
    };
    // kDecodeUnroll rows per thread in flight: their loads are issued together
    int f = tid / g;
    for (; f + (kDecodeUnroll - 1) * rows_per_pass < n; f += kDecodeUnroll * rows_per_pass) {
      float4 s[kDecodeUnroll];
#pragma unroll
      for (int u = 0; u < kDecodeUnroll; ++u)
        s[u] = stream_load4(Sh + static_cast<long long>(f + u * rows_per_pass) * dv + jbase);
#pragma unroll
      for (int u = 0; u < kDecodeUnroll; ++u) row(f + u * rows_per_pass, s[u]);
    }
    for (; f < n; f += rows_per_pass)
      row(f, stream_load4(Sh + static_cast<long long>(f) * dv + jbase));
  } else {
    const int rows_per_pass = 256 / dv;  // dv <= 256
    jbase = tid % dv;
    if (tid < rows_per_pass * dv) {
      for (int f = tid / dv; f < n; f += rows_per_pass) {
        int a = pairs[f] & 0xFF, b = pairs[f] >> 8;
        float pk = ks[a] * ks[b];
        float pq = ((a == b) ? 1.f : 2.f) * qs[a] * qs[b];
        float s = Sh[static_cast<long long>(f) * dv + jbase] + pk * vs[jbase];
        Sh[static_cast<long long>(f) * dv + jbase] = s;
        num[0] += pq * s;
      }
    }
  }
  for (int f = tid; f < n; f += 256) {
    int a = pairs[f] & 0xFF, b = pairs[f] >> 8;
    float zz = zh[f] + ks[a] * ks[b];
    zh[f] = zz;
    den += ((a == b) ? 1.f : 2.f) * qs[a] * qs[b] * zz;
  }
  red[tid][0] = num[0];
  red[tid][1] = num[1];
  red[tid][2] = num[2];
  red[tid][3] = num[3];
  red[tid][4] = den;
  __syncthreads();
  // denominator: tree over all threads
  for (int s = 128; s >= 1; s >>= 1) {
    if (tid < s) red[tid][4] += red[tid + s][4];
    __syncthreads();
  }
  const float D = red[0][4];
  if (vec) {
    const int g = dv / 4;
    if (tid < g) {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
      for (int t = tid; t < 256; t += g)
        for (int x = 0; x < 4; ++x) acc[x] += red[t][x];
      for (int x = 0; x < 4; ++x)
        out[static_cast<long long>(bh) * dv + 4 * tid + x] = (D > 0.f) ? acc[x] / D : 0.f;
    }
  } else {
    const int rows_per_pass = 256 / dv;
    if (tid < dv) {
      float acc = 0.f;
      for (int t = tid; t < rows_per_pass * dv; t += dv) acc += red[t][0];
      out[static_cast<long long>(bh) * dv + tid] = (D > 0.f) ? acc / D : 0.f;
    }
  }
}

// ---------------------------------------------------------------------------
// The same step with 1024 threads per head, the first rows' and z's loads issued
// before anything else, and k_a k_b and the weighted q_a q_b of every feature
// formed once, in LDS, while they are on their way: with few heads, one
// workgroup's latency is the step's (B1 H16 d64: 19.6 -> 13.3 us, near what one CU
// reads and writes; splitting a head over workgroups by value columns needs a
// second launch for z and took 17 us), and small heads (d = 32) are short enough
// for the setup to show.  6, 11 and 17 rows in flight per thread: 14.0, 13.3, 13.5
// us.  NT: state accesses past the caches, for states larger than they keep.
// grid BH, block 1024; dv a power of two from 4 to 256.
// ---------------------------------------------------------------------------
constexpr int kWideThreads = 1024;
constexpr int kWideUnroll = 11;  // rows per thread in flight
constexpr int kWideZ = 3;        // z values per thread (n <= 2080)

template <typename Tin, bool NT>
__global__ __launch_bounds__(kWideThreads) void decode_wide_f32(
    float* __restrict__ S, float* __restrict__ z, const Tin* __restrict__ q,
    const Tin* __restrict__ k, const Tin* __restrict__ v, float* __restrict__ out, int d, int dv,
    int g, unsigned inv_m) {
  __shared__ float qs[64], ks[64];
  __shared__ float2 pkq[2080];   // k_a k_b and w q_a q_b
  __shared__ float red[16][260];  // per wave: the columns' sums, then den
  const int m = d / g, nm = m * (m + 1) / 2, n = g * nm;
  const long long bh = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int gq = dv / 4, rows = kWideThreads / gq;  // 16-byte pieces per row, rows per pass
  const int r0 = tid / gq, col = 4 * (tid & (gq - 1));
  float* Sh = S + bh * n * dv + col;
  float* zh = z + bh * n;
  float4 s[kWideUnroll];
  auto fetch = [&](int f0) {
#pragma unroll
    for (int u = 0; u < kWideUnroll; ++u) {
      const float* p = Sh + min(f0 + u * rows, n - 1) * dv;
      s[u] = NT ? stream_load4(p) : *reinterpret_cast<const float4*>(p);
    }
  };
  if (tid < d) {
    qs[tid] = load_f32(q, bh * d + tid);
    ks[tid] = load_f32(k, bh * d + tid);
  }
  float zv[kWideZ];
#pragma unroll
  for (int u = 0; u < kWideZ; ++u) zv[u] = zh[min(tid + kWideThreads * u, n - 1)];
  float vv[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) vv[e] = load_f32(v, bh * dv + col + e);
  fetch(r0);
  __syncthreads();
  for (int i = tid; i < d * m; i += kWideThreads) {
    const int x = static_cast<int>((static_cast<unsigned>(i) * inv_m) >> 20);  // i / m
    const int b = i - x * m, blk = static_cast<int>((static_cast<unsigned>(x) * inv_m) >> 20);
    const int a = x - blk * m, y = blk * m + b;
    if (b >= a)
      pkq[blk * nm + packed_index(a, b, m)] =
          make_float2(ks[x] * ks[y], ((a == b) ? 1.f : 2.f) * qs[x] * qs[y]);
  }
  __syncthreads();
  float num[4] = {0.f, 0.f, 0.f, 0.f};
  for (int f0 = r0; f0 < n; f0 += kWideUnroll * rows) {
    if (f0 != r0) fetch(f0);
#pragma unroll
    for (int u = 0; u < kWideUnroll; ++u) {
      const int f = f0 + u * rows;
      if (f >= n) continue;  // its load read row n - 1 again
      const float2 p = pkq[f];
      s[u].x += p.x * vv[0];
      s[u].y += p.x * vv[1];
      s[u].z += p.x * vv[2];
      s[u].w += p.x * vv[3];
      if constexpr (NT) stream_store4(Sh + f * dv, s[u]);
      else *reinterpret_cast<float4*>(Sh + f * dv) = s[u];
      num[0] += p.y * s[u].x;
      num[1] += p.y * s[u].y;
      num[2] += p.y * s[u].z;
      num[3] += p.y * s[u].w;
    }
  }
  float den = 0.f;
#pragma unroll
  for (int u = 0; u < kWideZ; ++u) {
    const int f = tid + kWideThreads * u;
    if (f < n) {
      const float2 p = pkq[f];
      const float zz = zv[u] + p.x;
      zh[f] = zz;
      den += p.y * zz;
    }
  }
  // lanes of one column piece, then the waves
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    den += __shfl_xor(den, o);
    if (o >= gq) {
#pragma unroll
      for (int e = 0; e < 4; ++e) num[e] += __shfl_xor(num[e], o);
    }
  }
  if (lane < gq) {
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wv][col + e] = num[e];
  }
  if (lane == 0) red[wv][256] = den;
  __syncthreads();
  if (tid < dv) {
    float D = 0.f, x = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      D += red[w][256];
      x += red[w][tid];
    }
    out[bh * dv + tid] = (D > 0.f) ? x / D : 0.f;
  }
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
size_t fp32_forward_workspace(int BH, int T, int d, int dv, int C, int g) {
  const size_t n = static_cast<size_t>(g) * (d / g) * (d / g + 1) / 2;
  const size_t NC = (static_cast<size_t>(T) + C - 1) / C;
  return static_cast<size_t>(BH) * NC * (n * dv + n) * sizeof(float);
}

size_t fp32_forward_smem(int d, int C, int g) {
  const size_t n = static_cast<size_t>(g) * (d / g) * (d / g + 1) / 2;
  return (static_cast<size_t>(C) * d * 2 + static_cast<size_t>(C) * C + C) * sizeof(float) +
         n * sizeof(uint16_t);
}

template <typename Tin>
hipError_t launch_fp32_forward(const void* q, const void* k, const void* v, float* out, int BH,
                               int T, int d, int dv, int C, int g, void* ws, hipStream_t st,
                               hipEvent_t* ev) {
  const int n = g * ((d / g) * (d / g + 1) / 2);
  const int NC = (T + C - 1) / C;
  const long long rec = static_cast<long long>(n) * dv + n;
  float* states = static_cast<float*>(ws);
  const long long bh_stride = rec * NC;
  hipError_t e = record(ev, 0, st);
  if (e != hipSuccess) return e;
  if (quad32_fwd_ok(BH, T, d, dv, C, g)) {  // one launch, no states
    for (int i = 1; i < 3; ++i)
      if ((e = record(ev, i, st)) != hipSuccess) return e;
    if ((e = launch_quad32_fwd<Tin>(q, k, v, out, BH, T, d, dv, st)) != hipSuccess) return e;
    return record(ev, 3, st);
  }
  launch_chunk_state<Tin>(k, v, states, states + static_cast<long long>(n) * dv, BH, T, d, dv, C,
                          NC, g, bh_stride, rec, bh_stride, rec, st);
  if ((e = record(ev, 1, st)) != hipSuccess) return e;
  dim3 g2(static_cast<unsigned>((rec + kEB - 1) / kEB), BH);
  scan_exclusive<float, UnitWeight><<<g2, 256, 0, st>>>(states, states, NC, rec, bh_stride,
                                                        UnitWeight{});
  if ((e = record(ev, 2, st)) != hipSuccess) return e;
  const size_t shm = fp32_forward_smem(d, C, g);
  if (shm > 65536) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&chunk_out_f32<Tin>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       static_cast<int>(shm));
    if (e != hipSuccess) return e;
  }
  chunk_out_f32<Tin><<<dim3(NC, BH), 256, shm, st>>>(
      static_cast<const Tin*>(q), static_cast<const Tin*>(k), static_cast<const Tin*>(v), states,
      out, T, d, dv, C, g, bh_stride, rec);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return record(ev, 3, st);
}

template <typename Tin>
hipError_t launch_prefill(const void* k, const void* v, float* S, float* z, int BH, int T, int d,
                          int dv, int g, hipStream_t st) {
  const int n = g * ((d / g) * (d / g + 1) / 2);
  // one chunk covering all T tokens; S and z are separate arrays
  launch_chunk_state<Tin>(k, v, S, z, BH, T, d, dv, T, 1, g, static_cast<long long>(n) * dv, 0,
                          static_cast<long long>(n), 0, st);
  return hipGetLastError();
}

template <typename Tin>
hipError_t launch_decode(float* S, float* z, const void* q, const void* k, const void* v,
                         float* out, int BH, int d, int dv, int g, hipStream_t st) {
  // Measured (us, wide : 256 threads; d = 64, the same state each step / four in
  // turn): 64 heads (34 MB) 16 / 18 : 29 / 29 cached; 128 heads 29 / 30 : 33 / 33
  // and 256 heads (136 MB) 52 / 52 : 53 / 54 past the caches, 1024 heads 203 : 197;
  // d = 32 (135 KB per head) 1024 heads 50 : 58, 4096 heads 186 : 207.  Past the caches
  // heads of 2.1 MB (d = 64 dv = 256) take 75 : 67 (24 of them) to 95 : 86 (64), in the
  // caches 43 : 58 (16); heads of 1.2 MB (48, 256) 51 : 54 (48) and 56 : 58 (64).
  const int n = g * ((d / g) * (d / g + 1) / 2);
  const size_t head = static_cast<size_t>(n) * dv * sizeof(float), state = head * BH;
  const bool pow2 = dv >= 4 && dv <= 256 && (dv & (dv - 1)) == 0;
  // Heads of a few KB leave most of 1024 threads idle and, in large numbers, the
  // chip with one workgroup per CU (us, wide : 256 threads, fp32): d 8 dv 16 512 heads
  // 9 : 10, 1024 15 : 13, 16384 209 : 170; d 16 dv 32 (17 KB) 768 heads 14 : 13, 16384
  // 265 : 235; but d 24 dv 16 (19 KB) 1024 heads 18.5 : 18.9, 16384 280 : 295, d 16 dv
  // 64 (35 KB) 8192 heads 145 : 166.  For narrow values the 256-thread kernel ends in a
  // walk over 1024 / dv partial sums: dv 8 1024 heads 15.6 : 16.5, 1536 22.4 : 20.9;
  // dv 4 4096 heads 58 : 65, 16384 227 : 202.
  const bool few = BH <= max(512, 81920 / (dv * dv));
  // A launch holds fewer than 2^32 threads: 256 per head serve four times as many heads.
  const bool fits = static_cast<long long>(BH) * kWideThreads < (1LL << 32);
  if (pow2 && fits && (few || head >= (18u << 10)) &&
      (state <= (48u << 20) || (state <= (140u << 20) && head <= (1300u << 10)) ||
       head <= (160u << 10))) {
    const unsigned m = d / g, inv_m = ((1u << 20) + m - 1) / m;  // exact quotients below 64 m
    auto go = [&](auto nt) {
      decode_wide_f32<Tin, decltype(nt)::value><<<BH, kWideThreads, 0, st>>>(
          S, z, static_cast<const Tin*>(q), static_cast<const Tin*>(k), static_cast<const Tin*>(v),
          out, d, dv, g, inv_m);
    };
    if (state <= (48u << 20)) go(std::false_type{});
    else go(std::true_type{});
    return hipGetLastError();
  }
  decode_step_f32<Tin><<<BH, 256, 0, st>>>(S, z, static_cast<const Tin*>(q),
                                           static_cast<const Tin*>(k), static_cast<const Tin*>(v),
                                           out, d, dv, g);
  return hipGetLastError();
}

template hipError_t launch_fp32_forward<float>(const void*, const void*, const void*, float*, int,
                                               int, int, int, int, int, void*, hipStream_t,
                                               hipEvent_t*);
template hipError_t launch_fp32_forward<bf16_t>(const void*, const void*, const void*, float*, int,
                                                int, int, int, int, int, void*, hipStream_t,
                                                hipEvent_t*);
template hipError_t launch_prefill<float>(const void*, const void*, float*, float*, int, int,
                                          int, int, int, hipStream_t);
template hipError_t launch_prefill<bf16_t>(const void*, const void*, float*, float*, int, int,
                                           int, int, int, hipStream_t);
template hipError_t launch_decode<float>(float*, float*, const void*, const void*, const void*,
                                         float*, int, int, int, int, hipStream_t);
template hipError_t launch_decode<bf16_t>(float*, float*, const void*, const void*, const void*,
                                          float*, int, int, int, int, hipStream_t);

}  // namespace kata

#include "kata_quad32.hpp"
