// kata_bwd_quad.hpp -- gradients of the causal KATA-M1 forward in the quadratic
// (flash-style) form on the bf16 matrix cores: bf16 inputs, d = dv = 64, g = 1.
//
// With a_t = dout_t / D_t, b_t = -<dout_t, o_t> / D_t, s_ti = q_t . k_i and, for
// i <= t, c_ti = dL/dw_ti = <a_t, v_i> + b_t:
//   dq_t = 2 sum_i c_ti s_ti k_i,   dk_i = 2 sum_t c_ti s_ti q_t,
//   dv_i = sum_t s_ti^2 a_t,
// evaluated pair tile by pair tile, with no feature state.  A pair costs 10 d
// multiply-adds (the scores and c are formed on both sides, a_t as two bf16
// parts), a token through chunk states 10 n d (n = 2080 features),
// and the pair tiles stay on chip while every chunk record is written and
// read: B8 H16 T4096 takes 1.31 ms here (0.08 of it the coefficients) against
// 3.11 ms through chunk states, the MFMAs running at 1.13 PFLOP/s, which is
// the rate of a large library product on this part (1.2 PFLOP/s).
//
// Precision: scores and c_ti in fp32 (q, k, v exact in bf16; a_t as a bf16
// pair hi + lo, b_t in fp32 as the initial accumulator), c_ti s_ti and s_ti^2
// rounded to bf16 once as matrix operands, sums in fp32.
//
// One launch runs both gradients' workgroups, so that either fills the other's
// tail: the key side (dk, dv of 128 keys, walking the queries from its
// diagonal on) and the query side (dq of 128 queries, walking the keys up to
// its diagonal).  A wave owns 32 keys (queries): its own rows are B operands in
// registers, the rows walked come through LDS in 32-row stages (direct global
// -> LDS copies, double buffered) as A operands, both as rows and, through
// transposing reads, as columns.  The score tile's accumulator registers are
// then the B operand of the next product as they stand.  Two thirds of a
// wave's issue slots are MFMAs; three workgroups of four waves share a CU out
// of step, so that one's MFMAs run under another's vector work and barriers.
// (Kernels and launchers; part of kata_bwd.hip.)
#pragma once

#include <type_traits>

#include "kata_common.hpp"
#include "kata_internal.hpp"
#include "kata_quad.hpp"

namespace kata {

namespace {

constexpr int kQD = 64;               // d = dv
constexpr int kQWG = 128;             // keys (queries) per workgroup, 32 per wave
constexpr int kQST = 32;              // rows per LDS stage: one tile
constexpr int kQTile = kQST * kQD * 2;  // bytes of one staged operand
constexpr int kQStageK = 3 * kQTile + kQST * 4;  // key side: q, a hi, a lo rows, b
constexpr int kQStageQ = 2 * kQTile;             // query side: k, v rows

struct QuadArgs {
  const uint16_t *q, *k, *v, *ahi, *alo;
  const float* b;
  float *dq, *dk, *dv;
  int T;
};

// dk, dv of keys 128 kb .. + 127 of head bh.
__device__ __forceinline__ void qd_key_side(const QuadArgs& a, char* lds, int bh, int kb) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 31, h = lane >> 5;
  const int T = a.T;
  const long long hb = static_cast<long long>(bh) * T;
  const uint16_t* qh = a.q + hb * kQD;
  const uint16_t* hi = a.ahi + hb * kQD;
  const uint16_t* lo = a.alo + hb * kQD;
  const float* bh_ = a.b + hb;
  const int kt = 4 * kb + wave;  // this wave's 32-key tile
  const int key = 32 * kt + c;
  const QdOffsets of(lane);
  bf16x8 kf[4], vf[4];
  {
    const long long row = hb + min(key, T - 1);
#pragma unroll
    for (int kz = 0; kz < 4; ++kz) {
      kf[kz] = *reinterpret_cast<const bf16x8*>(a.k + row * kQD + 16 * kz + 8 * h);
      vf[kz] = *reinterpret_cast<const bf16x8*>(a.v + row * kQD + 16 * kz + 8 * h);
    }
  }
  f32x16 dk[2] = {qd_zero(), qd_zero()}, dv[2] = {qd_zero(), qd_zero()};
  const int nst = (T + kQST - 1) / kQST;
  auto issue = [&](int st, char* buf) __attribute__((always_inline)) {
    qd_stage(qh, st * kQST, T, buf, wave, lane);
    qd_stage(hi, st * kQST, T, buf + kQTile, wave, lane);
    qd_stage(lo, st * kQST, T, buf + 2 * kQTile, wave, lane);
    // b of the stage's rows, a 4-byte copy per lane
    if (wave == 0 && lane < kQST) {
      const uint32_t dst =
          static_cast<uint32_t>(reinterpret_cast<uintptr_t>((qd_lds_void_t*)(buf + 3 * kQTile)));
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                   :
                   : "v"(bh_ + min(st * kQST + lane, T - 1)), "s"(dst)
                   : "memory", "m0");
    }
  };
  // every compiler-issued load is back before the copies start
#pragma unroll
  for (int kz = 0; kz < 4; ++kz) asm volatile("" ::"v"(kf[kz]), "v"(vf[kz]));
  issue(4 * kb, lds);
  int cur = 0;
  for (int qt = 4 * kb; qt < nst; ++qt) {
    wait_vmcnt<0>();
    lds_barrier();  // the stage is in; every wave is done with the other buffer
    const char* Q = lds + cur * kQStageK;
    cur ^= 1;
    if (qt + 1 < nst) issue(qt + 1, lds + cur * kQStageK);
    if (qt < kt) continue;  // wave-uniform
    f32x16 s = qd_zero();
#pragma unroll
    for (int kz = 0; kz < 4; ++kz) s = qd_mfma(of.rows(Q, kz), kf[kz], s);
    f32x16 cw;
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const float4 bb = *reinterpret_cast<const float4*>(Q + 3 * kQTile +
                                                         4 * (8 * r4 + 4 * h));
      cw[4 * r4] = bb.x;
      cw[4 * r4 + 1] = bb.y;
      cw[4 * r4 + 2] = bb.z;
      cw[4 * r4 + 3] = bb.w;
    }
#pragma unroll
    for (int kz = 0; kz < 4; ++kz) cw = qd_mfma(of.rows(Q + kQTile, kz), vf[kz], cw);
#pragma unroll
    for (int kz = 0; kz < 4; ++kz) cw = qd_mfma(of.rows(Q + 2 * kQTile, kz), vf[kz], cw);
    uint32_t w[8], p[8];
    if (qt == kt || 32 * qt + 32 > T) {  // wave-uniform: the diagonal, or rows past T
      const int t0 = 32 * qt + 4 * h;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int ta = t0 + 8 * (j >> 1) + 2 * (j & 1), tb = ta + 1;
        const bool oa = ta >= key && ta < T, ob = tb >= key && tb < T;
        const float x = s[2 * j], y = s[2 * j + 1];
        w[j] = pack_bf16x2(oa ? x * x : 0.f, ob ? y * y : 0.f);
        p[j] = pack_bf16x2(oa ? x * cw[2 * j] : 0.f, ob ? y * cw[2 * j + 1] : 0.f);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float x = s[2 * j], y = s[2 * j + 1];
        w[j] = pack_bf16x2(x * x, y * y);
        p[j] = pack_bf16x2(x * cw[2 * j], y * cw[2 * j + 1]);
      }
    }
#pragma unroll
    for (int kv = 0; kv < 2; ++kv)
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        dk[m] = qd_mfma(of.cols(Q + 2048 * kv, m), qd_frag(p + 4 * kv), dk[m]);
        dv[m] = qd_mfma(of.cols(Q + kQTile + 2048 * kv, m), qd_frag(w + 4 * kv), dv[m]);
        dv[m] = qd_mfma(of.cols(Q + 2 * kQTile + 2048 * kv, m), qd_frag(w + 4 * kv), dv[m]);
      }
  }
  if (key < T) {
    qd_store(a.dk + (hb + key) * kQD, dk, h, 2.f);
    qd_store(a.dv + (hb + key) * kQD, dv, h, 1.f);
  }
}

// dq of queries 128 qb .. + 127 of head bh.
__device__ __forceinline__ void qd_query_side(const QuadArgs& a, char* lds, int bh, int qb) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 31, h = lane >> 5;
  const int T = a.T;
  const long long hb = static_cast<long long>(bh) * T;
  const uint16_t* kh = a.k + hb * kQD;
  const uint16_t* vh = a.v + hb * kQD;
  const int qt = 4 * qb + wave;  // this wave's 32-query tile
  const int t = 32 * qt + c;
  const QdOffsets of(lane);
  bf16x8 qf[4], hf[4], lf[4];
  const long long row = hb + min(t, T - 1);
#pragma unroll
  for (int kz = 0; kz < 4; ++kz) {
    qf[kz] = *reinterpret_cast<const bf16x8*>(a.q + row * kQD + 16 * kz + 8 * h);
    hf[kz] = *reinterpret_cast<const bf16x8*>(a.ahi + row * kQD + 16 * kz + 8 * h);
    lf[kz] = *reinterpret_cast<const bf16x8*>(a.alo + row * kQD + 16 * kz + 8 * h);
  }
  const float bt = a.b[row];
  f32x16 dq[2] = {qd_zero(), qd_zero()};
  auto issue = [&](int st, char* buf) __attribute__((always_inline)) {
    qd_stage(kh, st * kQST, T, buf, wave, lane);
    qd_stage(vh, st * kQST, T, buf + kQTile, wave, lane);
  };
#pragma unroll
  for (int kz = 0; kz < 4; ++kz) asm volatile("" ::"v"(qf[kz]), "v"(hf[kz]), "v"(lf[kz]));
  asm volatile("" ::"v"(bt));
  const int nst = min(4 * (qb + 1), (T + kQST - 1) / kQST);
  issue(0, lds);
  int cur = 0;
  for (int kt = 0; kt < nst; ++kt) {
    wait_vmcnt<0>();
    lds_barrier();
    const char* K = lds + cur * kQStageQ;
    cur ^= 1;
    if (kt + 1 < nst) issue(kt + 1, lds + cur * kQStageQ);
    if (kt > qt) continue;  // wave-uniform
    f32x16 s = qd_zero(), cw;
#pragma unroll
    for (int kz = 0; kz < 4; ++kz) s = qd_mfma(of.rows(K, kz), qf[kz], s);
#pragma unroll
    for (int r = 0; r < 16; ++r) cw[r] = bt;
#pragma unroll
    for (int kz = 0; kz < 4; ++kz) {
      const bf16x8 v = of.rows(K + kQTile, kz);
      cw = qd_mfma(v, hf[kz], cw);
      cw = qd_mfma(v, lf[kz], cw);
    }
    uint32_t p[8];
    if (kt == qt) {  // the diagonal: keys past the query (and past T) are masked
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int ia = 8 * (j >> 1) + 4 * h + 2 * (j & 1);
        p[j] = pack_bf16x2(ia <= c ? s[2 * j] * cw[2 * j] : 0.f,
                           ia + 1 <= c ? s[2 * j + 1] * cw[2 * j + 1] : 0.f);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        p[j] = pack_bf16x2(s[2 * j] * cw[2 * j], s[2 * j + 1] * cw[2 * j + 1]);
    }
#pragma unroll
    for (int kv = 0; kv < 2; ++kv)
#pragma unroll
      for (int m = 0; m < 2; ++m)
        dq[m] = qd_mfma(of.cols(K + 2048 * kv, m), qd_frag(p + 4 * kv), dq[m]);
  }
  if (t < T) qd_store(a.dq + (hb + t) * kQD, dq, h, 2.f);
}

// Workgroup id -> (head, side, rank), rank 0 being the longest walk of either
// side.  Workgroups go to the eight XCDs in turn and, inside one, to its four
// shader engines in turn, whatever is free, so work has to be equal over ids
// equal mod 32 (with key and query side on alternate ids two engines of every
// XCD got all the key sides: 1.36 instead of 1.23 ms at B8 H16 T4096).
// With a multiple of eight heads a head's workgroups share an XCD, whose L2
// then holds its rows: four key sides, four query sides, and so on, the ranks
// of a group of four running up and down in turn (NB4 = NB rounded up to four;
// ranks past NB exit).  The heads of an XCD follow each other but for its last
// kQTailHeads, whose groups of eight take turns, so that the launch ends with
// the shortest walks of several heads and not with all of one head: backward
// and forward at B1 H16 T4096 245 -> 222 us, B3 608 -> 577, B8 1507 -> 1477
// (2 heads: 222, 588, 1487; 8: 222, 578, 1487; all of them: 1537 at B8, more
// heads than an L2 holds).  Otherwise ranks are the slow index, so that
// neighbouring ids carry like work on every XCD.
constexpr int kQTailHeads = 4;
__global__ __launch_bounds__(256, 3) void bwd_quad_kernel(QuadArgs a, int BH, int NB) {
  __shared__ __attribute__((aligned(16))) char lds[2 * kQStageK];
  const int id = blockIdx.x;
  int bh, side, rank;
  if ((BH & 7) == 0) {
    const int per = 2 * ((NB + 3) & ~3), x = id >> 3;
    const int nh = BH >> 3, ni = min(nh, kQTailHeads), x0 = (nh - ni) * per;
    int j, hx;
    if (x < x0) {
      j = x % per;
      hx = x / per;
    } else {
      const int y = x - x0;
      j = (y & 7) + 8 * (y / 8 / ni);
      hx = nh - ni + y / 8 % ni;
    }
    bh = (id & 7) + 8 * hx;
    const int grp = j >> 3;
    side = (j >> 2) & 1;
    rank = 4 * grp + ((grp & 1) ? 3 - (j & 3) : (j & 3));
    if (rank >= NB) return;
  } else {
    bh = id % BH;
    side = (id / BH) & 1;
    rank = id / BH / 2;
  }
  if (side == 0) qd_key_side(a, lds, bh, rank);
  else qd_query_side(a, lds, bh, NB - 1 - rank);
}

// D_t = sum_{i <= t} s_ti^2 for callers without the forward's denominators:
// the query side's walk with the scores alone.
__global__ __launch_bounds__(256) void bwd_quad_den(const uint16_t* __restrict__ q,
                                                    const uint16_t* __restrict__ k,
                                                    float* __restrict__ den, int T, int NB) {
  __shared__ __attribute__((aligned(16))) char lds[2 * kQTile];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 31, h = lane >> 5;
  const int bh = blockIdx.x / NB, qb = NB - 1 - blockIdx.x % NB;
  const long long hb = static_cast<long long>(bh) * T;
  const uint16_t* kh = k + hb * kQD;
  const int qt = 4 * qb + wave, t = 32 * qt + c;
  const QdOffsets of(lane);
  bf16x8 qf[4];
#pragma unroll
  for (int kz = 0; kz < 4; ++kz)
    qf[kz] = *reinterpret_cast<const bf16x8*>(q + (hb + min(t, T - 1)) * kQD + 16 * kz + 8 * h);
#pragma unroll
  for (int kz = 0; kz < 4; ++kz) asm volatile("" ::"v"(qf[kz]));
  const int nst = min(4 * (qb + 1), (T + kQST - 1) / kQST);
  qd_stage(kh, 0, T, lds, wave, lane);
  int cur = 0;
  float D = 0.f;
  for (int kt = 0; kt < nst; ++kt) {
    wait_vmcnt<0>();
    lds_barrier();
    const char* buf = lds + cur * kQTile;
    cur ^= 1;
    if (kt + 1 < nst) qd_stage(kh, (kt + 1) * kQST, T, lds + cur * kQTile, wave, lane);
    if (kt > qt) continue;
    f32x16 s = qd_zero();
#pragma unroll
    for (int kz = 0; kz < 4; ++kz) s = qd_mfma(of.rows(buf, kz), qf[kz], s);
    float part = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bool ok = kt < qt || 8 * (r >> 2) + 4 * h + (r & 3) <= c;
      part += ok ? s[r] * s[r] : 0.f;
    }
    D += part;
  }
  D += __shfl_xor(D, 32);
  if (h == 0 && t < T) den[hb + t] = D;
}

// a_t = dout_t / D_t as a bf16 pair hi + lo and b_t = -<dout_t, o_t> / D_t in
// fp32 (zeros where D_t = 0).  Eight lanes per token, 8 columns each; reads
// and writes whole rows (HBM-bound).  grid ceil(rows / 32), block 256.
__global__ __launch_bounds__(256) void bwd_quad_coef(const float* __restrict__ o,
                                                     const float* __restrict__ dout,
                                                     const float* __restrict__ den,
                                                     uint16_t* __restrict__ ahi,
                                                     uint16_t* __restrict__ alo,
                                                     float* __restrict__ b, long long rows) {
  const int sub = threadIdx.x & 7;
  const long long row0 = static_cast<long long>(blockIdx.x) * 32 + (threadIdx.x >> 3);
  const long long row = row0 < rows ? row0 : rows - 1;
  const float D = den[row];
  const float inv = D > 0.f ? 1.f / D : 0.f;
  const float4* dp = reinterpret_cast<const float4*>(dout + row * kQD + 8 * sub);
  const float4* op = reinterpret_cast<const float4*>(o + row * kQD + 8 * sub);
  const float4 x0 = dp[0], x1 = dp[1], y0 = op[0], y1 = op[1];
  float go = x0.x * y0.x + x0.y * y0.y + x0.z * y0.z + x0.w * y0.w;
  go += x1.x * y1.x + x1.y * y1.y + x1.z * y1.z + x1.w * y1.w;
#pragma unroll
  for (int m = 4; m > 0; m >>= 1) go += __shfl_xor(go, m);
  if (row0 >= rows) return;
  const float av[8] = {x0.x * inv, x0.y * inv, x0.z * inv, x0.w * inv,
                       x1.x * inv, x1.y * inv, x1.z * inv, x1.w * inv};
  uint32_t hw[4], lw[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    hw[e] = pack_bf16x2(av[2 * e], av[2 * e + 1]);
    lw[e] = pack_bf16x2(av[2 * e] - bf16lo_f32(hw[e]), av[2 * e + 1] - bf16hi_f32(hw[e]));
  }
  *reinterpret_cast<uint4*>(ahi + row * kQD + 8 * sub) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
  *reinterpret_cast<uint4*>(alo + row * kQD + 8 * sub) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
  if (sub == 0) b[row] = -go * inv;
}

}  // namespace

// Quadratic time against the chunk states' linear one, measured at 1, 2, 5, 7, 8, 9, 15,
// 16, 17, 33, 64, 100 and 250 heads (us, with the denominators given): one head T4096
// 101 : 139, T6000 145 : 157, T8192 195 : 176; two heads T8192 199 : 182; eight heads T8192
// 347 : 617; 17 heads 631 : 1059; 100 heads 4095 : 4761 (64 heads T10240 3703 : 4160,
// T12288 5258 : 5000).  With few heads a workgroup's walk over T bounds the time, so they
// cross earlier; without the denominators one more score pass is due: one head T4096
// 145 : 147, 64 heads T8192 2781 : 3447.
bool bwd_quad_ok(int BH, int T) { return T <= 4096 || (T <= 8192 && BH >= 8); }

hipError_t launch_bwd_quad(const void* q, const void* k, const void* v, const float* out,
                           const float* dout, const float* den, float* dq, float* dk,
                           float* dv_out, int BH, int T, void* ws, hipStream_t st,
                           hipEvent_t* ev) {
  const long long rows = static_cast<long long>(BH) * T;
  const int NB = (T + kQWG - 1) / kQWG;
  uint16_t* ahi = static_cast<uint16_t*>(ws);
  uint16_t* alo = ahi + rows * kQD;
  float* b = reinterpret_cast<float*>(alo + rows * kQD);
  float* own_den = b + rows;
  const uint16_t* qp = static_cast<const uint16_t*>(q);
  const uint16_t* kp = static_cast<const uint16_t*>(k);
  hipError_t e;
  if ((e = record(ev, 0, st)) != hipSuccess) return e;
  if ((e = record(ev, 1, st)) != hipSuccess) return e;
  if ((e = record(ev, 2, st)) != hipSuccess) return e;
  if (den == nullptr) {
    bwd_quad_den<<<static_cast<unsigned>(BH) * NB, 256, 0, st>>>(qp, kp, own_den, T, NB);
    den = own_den;
  }
  bwd_quad_coef<<<static_cast<unsigned>((rows + 31) / 32), 256, 0, st>>>(out, dout, den, ahi, alo,
                                                                         b, rows);
  if ((e = record(ev, 3, st)) != hipSuccess) return e;
  if ((e = record(ev, 4, st)) != hipSuccess) return e;
  if ((e = record(ev, 5, st)) != hipSuccess) return e;
  const QuadArgs a{qp, kp, static_cast<const uint16_t*>(v), ahi, alo, b, dq, dk, dv_out, T};
  const int nb = (BH & 7) == 0 ? (NB + 3) & ~3 : NB;  // see the kernel's order of workgroups
  bwd_quad_kernel<<<static_cast<unsigned>(BH) * 2 * nb, 256, 0, st>>>(a, BH, NB);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return record(ev, 6, st);
}

}  // namespace kata
