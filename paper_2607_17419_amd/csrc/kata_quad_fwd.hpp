// kata_quad_fwd.hpp -- the causal KATA-M1 / M2 forward in the quadratic
// (flash-style) form on the bf16 matrix cores: d = 64 with one or two feature
// blocks, d = 32; dv = 64.
//
//   o_t = sum_{i <= t} w_ti v_i / D_t,  D_t = sum_{i <= t} w_ti,
//   w_ti = sum over blocks of (q_t . k_i)^2.
//
// Eight waves of one 32-query tile each, whose rows are B operands in registers
// (KS = 1), or four tiles each shared by two waves that take alternate halves of
// every stage's keys and add their sums in LDS (KS = 2: half the serial walk, for
// calls with few workgroups).  K and V rows come through LDS in stages of two
// key tiles per wave (direct global -> LDS copies, double buffered): K as rows (A
// operand of S^T = K Q^T), V through transposing reads as columns (A operand of
// O^T += V^T P), in the key order of the score accumulators, which are squared,
// rounded to bf16 and used as the B operand as they stand.  D sums the unrounded
// fp32 weights.
//
// Bound by the matrix rate: a tile pair is eight MFMAs (256 cycles) against 40
// vector instructions (160), the two score chains of a stage come first so that
// one tile's products run under the other's vector work, and 16 waves share a
// CU.  d = 64: B1 H16 T32768 1.83 ms (1.20 PFLOP/s, the rate of a large library
// product here), B8 H16 T4096 295 us; B1 H16 T4096 44 us (KS = 1: 63), where a
// four-wave form with a transposed copy of V took 74.  Stages of four tiles per
// wave measured 318 us, four-wave workgroups 306, two query tiles per wave 318 at
// B8 H16 T4096.
// (Kernels and launchers; part of kata_mfma.hip.)
#pragma once

#include <type_traits>

#include "kata_common.hpp"
#include "kata_internal.hpp"
#include "kata_quad.hpp"

namespace kata {

namespace {

// K and V rows of a stage of NKB 32-key tiles, tile after tile.
template <int D>
struct QuadStage {
  static constexpr int KT = 32 * D * 2;  // bytes of 32 K rows
  static constexpr int VT = 32 * 64 * 2;
};

template <int D, int NG, int KS>
__global__ __launch_bounds__(512, KS == 2 ? 4 : 2) void quad_fwd_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const uint16_t* __restrict__ v, float* __restrict__ out, float* __restrict__ den, int T, int BH,
    int NB) {
  using S = QuadStage<D>;
  constexpr int KZ = D / 16, NT = 2, NKB = NT * KS;  // tiles of a wave, of a stage
  constexpr int SB = NKB * (S::KT + S::VT);           // bytes of a stage
  constexpr int QT = 8 / KS;  // query tiles per workgroup
  __shared__ __attribute__((aligned(16))) char lds[2 * SB];
  // Workgroup id -> (head, query block), the longest walks (rank 0) first.  With a
  // multiple of eight heads a head stays on one XCD (id mod 8); ranks run up and
  // down in groups of four, so that the XCD's four shader engines, which get
  // workgroups in turn, get like work, and every other head runs the other way
  // round, so that the workgroups that land together on a CU add up alike (one
  // direction for all: 60 instead of 44 us at B1 H16 T4096).  Otherwise ranks are
  // the slow index.
  const int id = blockIdx.x;
  int bh, rank;
  if ((BH & 7) == 0) {
    const int per = (NB + 3) & ~3, j = (id >> 3) % per;
    bh = (id & 7) + 8 * ((id >> 3) / per);
    rank = (j & 4) ? j ^ 3 : j;
    if (rank >= NB) return;
    if (((BH >> 3) - 1 - ((id >> 3) / per)) & 1) rank = NB - 1 - rank;
  } else {
    bh = id % BH;
    rank = id / BH;
  }
  const int qb = NB - 1 - rank;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 31, h = lane >> 5;
  const long long hb = static_cast<long long>(bh) * T;
  const uint16_t* kh = k + hb * D;
  const uint16_t* vh = v + hb * 64;
  const QdOffsets of(lane);
  unsigned ro[KZ];
#pragma unroll
  for (int kz = 0; kz < KZ; ++kz)
    ro[kz] = D == 64 ? of.row[kz]
                     : static_cast<unsigned>(c * 64 + 16 * ((2 * kz + h) ^ qd_swz32(c)));
  const int qt = QT * qb + wave % QT;  // this wave's 32-query tile
  const int kg = wave / QT;            // its share of a stage's key tiles
  const int t = 32 * qt + c;
  bf16x8 qf[KZ];
#pragma unroll
  for (int kz = 0; kz < KZ; ++kz)
    qf[kz] = *reinterpret_cast<const bf16x8*>(q + (hb + min(t, T - 1)) * D + 16 * kz + 8 * h);
#pragma unroll
  for (int kz = 0; kz < KZ; ++kz) asm volatile("" ::"v"(qf[kz]));
  f32x16 acc[2] = {qd_zero(), qd_zero()};
  float dsum = 0.f;
  auto issue = [&](int st, char* buf) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < NKB; ++b) {
      const int r0 = st * 32 * NKB + 32 * b;
      char* t = buf + b * (S::KT + S::VT);
      if (wave >= 4) qd_stage(vh, r0, T, t + S::KT, wave & 3, lane);
      else if constexpr (D == 64) qd_stage(kh, r0, T, t, wave, lane);
      else if ((wave >> 1) == (b & 1)) qd_stage32(kh, r0, T, t, wave & 1, lane);
    }
  };
  const int last = min(QT * qb + QT - 1, (T - 1) / 32);  // last query (key) tile
  const int nst = last / NKB + 1;
  // tile b of a stage (KT + VT bytes each)
  auto scores = [&](const char* K, f32x16 (&s)[NG]) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      s[g] = qd_zero();
#pragma unroll
      for (int kz = 0; kz < KZ / NG; ++kz)
        s[g] = qd_mfma(*reinterpret_cast<const bf16x8*>(K + ro[g * (KZ / NG) + kz]),
                       qf[g * (KZ / NG) + kz], s[g]);
    }
  };
  auto weight = [&](const f32x16 (&s)[NG], int r) __attribute__((always_inline)) {
    float w = s[0][r] * s[0][r];
    if constexpr (NG == 2) w = fmaf(s[1][r], s[1][r], w);
    return w;
  };
  auto values = [&](const char* V, const uint32_t (&p)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int kv = 0; kv < 2; ++kv)
#pragma unroll
      for (int m = 0; m < 2; ++m)
        acc[m] = qd_mfma(of.cols(V + 2048 * kv, m), qd_frag(p + 4 * kv), acc[m]);
  };
  issue(0, lds);
  const char* buf = lds + kg * NT * (S::KT + S::VT);  // this wave's part of the current stage
  int flip = SB;
  auto next_stage = [&](int st) __attribute__((always_inline)) {
    wait_vmcnt<0>();
    lds_barrier();  // the stage is in; every wave is done with the other buffer
    if (st + 1 < nst) issue(st + 1, lds + ((st + 1) & 1) * SB);
  };
  // stages below the diagonal of every wave: straight-line code, the score
  // chains of all its tiles first
  const int nfull = QT * qb / NKB;
  int st = 0;
  for (; st < nfull; ++st) {
    next_stage(st);
    f32x16 s[NT][NG];
#pragma unroll
    for (int b = 0; b < NT; ++b) scores(buf + b * (S::KT + S::VT), s[b]);
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      uint32_t p[8];
      float part = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float x = weight(s[b], 2 * j), y = weight(s[b], 2 * j + 1);
        part += x + y;
        p[j] = pack_bf16x2(x, y);
      }
      dsum += part;
      values(buf + b * (S::KT + S::VT) + S::KT, p);
    }
    buf += flip;
    flip = -flip;
  }
  // the last stages, up to each wave's diagonal tile
  for (; st < nst; ++st) {
    next_stage(st);
    const int kt0 = st * NKB + kg * NT;
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      if (kt0 + b > qt) continue;  // wave-uniform
      const char* K = buf + b * (S::KT + S::VT);
      f32x16 s[NG];
      scores(K, s);
      // the diagonal tile: keys past the query (and past T) are masked
      const int lim = kt0 + b < qt ? 32 : c;
      uint32_t p[8];
      float part = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int ia = 8 * (j >> 1) + 4 * h + 2 * (j & 1);
        const float x = ia <= lim ? weight(s, 2 * j) : 0.f;
        const float y = ia + 1 <= lim ? weight(s, 2 * j + 1) : 0.f;
        part += x + y;
        p[j] = pack_bf16x2(x, y);
      }
      dsum += part;
      values(K + S::KT, p);
    }
    buf += flip;
    flip = -flip;
  }
  if constexpr (KS == 2) {  // the second half's sums through LDS
    float* red = reinterpret_cast<float*>(lds) + (wave % QT) * 33 * 64 + lane;
    static_assert(QT * 33 * 64 * 4 <= 2 * SB, "the sums fit the stage buffers");
    __syncthreads();
    if (kg == 1) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        red[64 * r] = acc[0][r];
        red[64 * (16 + r)] = acc[1][r];
      }
      red[64 * 32] = dsum;
    }
    __syncthreads();
    if (kg == 1) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc[0][r] += red[64 * r];
      acc[1][r] += red[64 * (16 + r)];
    }
    dsum += red[64 * 32];
  }
  const float Dt = dsum + __shfl_xor(dsum, 32);
  if (t >= T) return;
  if (den != nullptr && h == 0) den[hb + t] = Dt;
  qd_store(out + (hb + t) * 64, acc, h, Dt > 0.f ? 1.f / Dt : 0.f);
}

template <int D, int NG>
hipError_t run(const void* q, const void* k, const void* v, float* out, float* den, int BH, int T,
               hipStream_t st) {
  auto go = [&](auto ks) {
    constexpr int KS = decltype(ks)::value, QW = 256 / KS;
    const int NB = (T + QW - 1) / QW;
    const int nb = (BH & 7) == 0 ? (NB + 3) & ~3 : NB;
    quad_fwd_kernel<D, NG, KS><<<static_cast<unsigned>(BH) * nb, 512, 0, st>>>(
        static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k),
        static_cast<const uint16_t*>(v), out, den, T, BH, NB);
  };
  // Two waves per query tile where workgroups are few (us, KS 2 : 1): B1 H16 T1024
  // 13.5 : 19, T4096 44 : 63, B2 H16 T8192 272 : 290; B8 H16 T1024 35.5 : 33, B1 H16
  // T32768 2018 : 1865.
  const long long wgs = static_cast<long long>(BH) * ((T + 255) / 256);
  if (wgs < 512 || (wgs <= 1024 && T >= 4096)) go(std::integral_constant<int, 2>{});
  else go(std::integral_constant<int, 1>{});
  return hipGetLastError();
}

}  // namespace

// Quadratic time against the span pipeline's linear one, measured at 1, 2, 5, 16, 24,
// 33, 64, 100, 128, 250 and 512 heads (us, this form : spans of the default length).
// d = 64: 2 heads T2048 18 : 74, T6144 44 : 75; 16 heads T4096 43 : 86, T6144 83 : 92; 33
// heads T6144 184 : 180; 64 heads 315 : 314; 128 heads T1000 31 : 30, T4096 288 : 395,
// T6144 592 : 620; 250 heads T5000 858 : 960, T6144 1268 : 1191.  Two feature blocks: 16
// heads T5632 77 : 75; 24 heads T3584 53 : 75, T5632 117 : 93; 250 heads T3584 439 : 524,
// T5632 1097 : 812.  d = 32: 16 heads T4608 45 : 46; 24 heads T3072 32 : 45, T4608 63 :
// 49; 512 heads T3072 517 : 525.
bool quad_fwd_ok(int BH, int T, int d, int g) {
  if (d == 32) return T <= 3072 || (T <= 4608 && BH <= 16);
  if (g == 2) return T <= 3584 || (T <= 5632 && BH <= 16);
  return T <= (BH <= 128 ? 6144 : 5632);
}

hipError_t launch_quad_fwd(const void* q, const void* k, const void* v, float* out, float* den,
                           int BH, int T, int d, int g, hipStream_t st) {
  if (d == 32) return run<32, 1>(q, k, v, out, den, BH, T, st);
  return g == 2 ? run<64, 2>(q, k, v, out, den, BH, T, st)
                : run<64, 1>(q, k, v, out, den, BH, T, st);
}

}  // namespace kata
