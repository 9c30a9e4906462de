// kata_quad32.hpp -- KATA-M1 (one feature block) in the quadratic form with
// fp32 arithmetic on the fp32 matrix cores (v_mfma_f32_32x32x2_f32): forward and
// gradients for every shape of the fp32 paths with g = 1 (d <= 64; dv <= 256
// forward, dv <= 64 gradients; fp32 or bf16 inputs).
//
// A causal pair costs d + dv multiply-adds forward against 2 n dv per token
// through chunk states (n = d(d+1)/2), equal near T = 4200 at d = dv = 64, and it
// runs entirely in matrix instructions, where the chunk output reads a 2080 x
// 64 state per chunk into scalar products.  B1 H8 T1000 d64 fp32: forward 2990 ->
// 22 us, coefficients and gradients 66 us where the backward took 1045;
// B8 H16 T2048: forward 40.7 -> 0.60 ms (114 TFLOP/s of the 154 that a large fp32
// library product reaches), backward 16.3 -> 3.1 ms.
//
// A workgroup owns one tile of 32 queries (keys); its eight waves take the
// 32-row tiles of the walk in turn (wave w: tiles w, w + 8, ...), which keeps
// the longest serial chain short when a call has few heads, and add their
// sums through LDS in wave order at the end.  Operands come straight from
// global memory (L1 / L2): a 32 x 64 tile feeds 32 matrix instructions of 64
// cycles each, so the loads are a small part of the cycles and no staging or
// barrier stands between them.
//
// Row 0 of a head sees one key: its output is v_0 and its gradient zero up to
// the rounding residue of c_00 / D_0, the one row where D_t can be tiny and the
// residue visible.  Its output, s_00 and c_00 are formed in the order of operations
// of the chunk kernels, so that a call gives the same values there whichever
// form its length selects.
//
// Layout of v_mfma_f32_32x32x2_f32: lane (c = lane % 32, h = lane / 32) holds
// A[row c][k = h] and B[k = h][column c]; result row 8 (r / 4) + 4 h + r % 4,
// column c.  The order of k inside a sum is free: step i takes k = i and
// i + DP/2, so a lane reads its half row in consecutive pieces, and result
// register r is the B operand of a product over the result's rows, step r
// taking rows row(r, 0) and row(r, 1).
// (Kernels and launchers; part of kata_fp32.hip.)
#pragma once

#include <type_traits>

#include "kata_common.hpp"
#include "kata_internal.hpp"

namespace kata {

namespace {

constexpr int kW32 = 8;  // waves per workgroup

__device__ __forceinline__ f32x16 mf2(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int acc_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

// The rows of one head of q, k, v or a: T rows of w values, taken as WP values
// padded with zeros, through buffer loads whose range ends at the last row, so
// that rows past it read as zero and the loads of a tile share an address
// register.  EX: w = WP, half rows in 16-byte pieces; otherwise one value at a
// time.
template <typename Tin, int WP, bool EX>
struct HeadRows {
  static constexpr int SZ = static_cast<int>(sizeof(Tin));
  __amdgpu_buffer_rsrc_t rs;
  int w, rb;  // values and bytes of a row
  __device__ __forceinline__ HeadRows(const Tin* p, int T, int w_)
      : rs(__builtin_amdgcn_make_buffer_rsrc(const_cast<Tin*>(p), 0, T * w_ * SZ, 0x00020000)),
        w(EX ? WP : w_), rb((EX ? WP : w_) * SZ) {}
  __device__ __forceinline__ float load(int vo) const {
    if constexpr (SZ == 4)
      return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, vo, 0, 0));
    else
      return __uint_as_float(static_cast<uint32_t>(static_cast<uint16_t>(
                                 __builtin_amdgcn_raw_buffer_load_b16(rs, vo, 0, 0))) << 16);
  }
  // This lane's half (h) of a row.
  __device__ __forceinline__ void half(int row, int h, float (&x)[WP / 2]) const {
    const int vo = row * rb + h * (WP / 2) * SZ;
    if constexpr (EX) {
#pragma unroll
      for (int i = 0; i < WP / 2 * SZ / 16; ++i) {
        const uint4 u = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo + 16 * i, 0, 0));
        const uint32_t e[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if constexpr (SZ == 4) {
            x[4 * i + j] = __uint_as_float(e[j]);
          } else {
            x[8 * i + 2 * j] = bf16lo_f32(e[j]);
            x[8 * i + 2 * j + 1] = bf16hi_f32(e[j]);
          }
        }
      }
    } else {
      const int left = w - h * (WP / 2);  // values past the row: out of range, zero
#pragma unroll
      for (int i = 0; i < WP / 2; ++i) x[i] = load(i < left ? vo + i * SZ : -SZ);
    }
  }
  // Column j of one row (columns past w as in column()).
  __device__ __forceinline__ float at(int j, int row) const {
    return load(row * rb + min(j, w - 1) * SZ);
  }
  // Column j of rows r0 + acc_row(r, h).  Columns past w give another column:
  // they only reach result rows that are not stored.  The row is in the vector
  // offset throughout: the range check that makes rows past T - 1 read as zero
  // is specified for that offset (with the instruction's own), not for the
  // scalar one.
  __device__ __forceinline__ void column(int j, int r0, int h, float (&x)[16]) const {
    int vo = (r0 + 4 * h) * rb + min(j, w - 1) * SZ;
    if constexpr (!EX) asm("" : "+v"(vo));  // else a loop keeps all sixteen offsets in registers
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if constexpr (EX) {
        x[r] = load(vo + (8 * (r >> 2) + (r & 3)) * WP * SZ);
      } else {
        x[r] = load(vo);
        vo += (r & 3) == 3 ? 5 * rb : rb;
      }
    }
  }
};

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

// Orders this wave's LDS accesses before and after it (other waves take no part).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int KP>
__device__ __forceinline__ f32x16 dot_tile(const float (&a)[KP], const float (&b)[KP], f32x16 c) {
#pragma unroll
  for (int i = 0; i < KP; ++i) c = mf2(a[i], b[i], c);
  return c;
}

// acc += column j of the 32 rows of X from r0 on (x: this lane's, rows
// acc_row(r, h)) times the masked diagonal tile w, whose pairs of row and column
// c count where kUpTo ? row <= c : row >= c and are zero elsewhere.  A zero weight
// does not hide a non-finite x (0 Inf = NaN): a tile that has one adds its rows
// one at a time and keeps the sums of the columns that do not take the row, so
// that a non-finite value reaches the outputs that its pairs belong to and no
// others.  One wave of the workgroup has the diagonal tile: the weights pass
// through LDS (kDiagLds), the loop is kept rolled and x is read again, so that
// this path costs the other no registers (unrolled, with the weights in
// registers, it took 92 more in the forward at d = dv = 64).
constexpr int kDiagLds = 1024;  // floats from here on, past reduce_columns' own
template <bool kUpTo, typename Rows>
__device__ __forceinline__ void diagonal_products(const Rows& X, int j, int r0,
                                                  const float (&x)[16], const f32x16& w,
                                                  f32x16& acc, int c, int h, float* red) {
  float bad = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) bad += x[r] - x[r];  // 0, or NaN
  if (!__any(!(bad == 0.f))) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc = mf2(x[r], w[r], acc);
    return;
  }
  float* tile = red + kDiagLds;
  wave_lds_sync();  // the last call's reads
#pragma unroll
  for (int r = 0; r < 16; ++r) tile[r * 64 + 32 * h + c] = w[r];
  wave_lds_sync();
#pragma unroll 1
  for (int row = 0; row < 32; ++row) {
    const float xr = X.at(j, r0 + row);
    const float wr = tile[(4 * (row >> 3) + (row & 3)) * 64 + 32 * ((row >> 2) & 1) + c];
    const f32x16 sum = mf2(h ? 0.f : xr, h ? 0.f : wr, acc);
    const bool taken = kUpTo ? row <= c : row >= c;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = taken ? sum[e] : acc[e];
  }
}

// Adds the eight waves' tiles acc (result row j, column c) in wave order and
// writes fin(row j of column c, c) to out[c * w + j0 + j] for columns below nc
// and j0 + j < w.  Block-wide.
template <typename F>
__device__ __forceinline__ void reduce_store(float* red, const f32x16& acc, float* out, int w,
                                             int j0, int nc, F&& fin) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) red[(wv * 16 + r) * 64 + lane] = acc[r];
  __syncthreads();
  if (tid < 256) {  // four result rows of one column each
    const int r4 = tid >> 6, c = lane & 31, h = lane >> 5, j = j0 + 8 * r4 + 4 * h;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    for (int v = 0; v < kW32; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] += red[(v * 16 + 4 * r4 + e) * 64 + lane];
    if (c < nc) {
      float* o = out + static_cast<long long>(c) * w + j;
      if ((w & 3) == 0) {
        if (j < w) *reinterpret_cast<float4*>(o) = make_float4(fin(s[0], c), fin(s[1], c), fin(s[2], c), fin(s[3], c));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (j + e < w) o[e] = fin(s[e], c);
      }
    }
  }
}

// Sums x over the waves' lanes (both halves) per column into tot[32].
__device__ __forceinline__ void reduce_columns(float* red, float x, float* tot) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  x += __shfl_xor(x, 32);
  if (lane < 32) red[wv * 32 + lane] = x;
  __syncthreads();
  if (tid < 32) {
    float s = 0.f;
    for (int v = 0; v < kW32; ++v) s += red[v * 32 + tid];
    tot[tid] = s;
  }
  __syncthreads();
}

// Scores of the pairs t, i < 8, lane 8 t + i, summed in fp64.  In the first
// rows every score of a row can be tiny, D_t with them, and a sum rounded at
// the size of its terms then shows in o_t and, times 1 / s, in the gradients.
// Eight rows: of independent scores, D_t falls below a hundredth of its mean (a
// score's rounding then counts ten times) with probability 1e-2 in row 1, 2e-4 in
// row 3, 1e-7 in row 7 (chi-square of t + 1 degrees), and 64 pairs are one per lane.
template <typename Tin>
__device__ __forceinline__ float early_scores(const Tin* q, const Tin* k, int T, int d, int lane) {
  const Tin* qr = q + min(lane >> 3, T - 1) * d;
  const Tin* kr = k + min(lane & 7, T - 1) * d;
  double s = 0.0;
  __builtin_assume(d > 0);
#pragma unroll 8
  for (int x = 0; x < d; ++x)
    s = fma(static_cast<double>(to_f32(qr[x])), static_cast<double>(to_f32(kr[x])), s);
  return static_cast<float>(s);
}

// Puts values of lanes 8 t + i into the tile of rows and columns 0..31 whose
// columns are the queries (kQueryColumns) or the keys.
template <bool kQueryColumns>
__device__ __forceinline__ void put_early(f32x16& tile, float e, int c, int h) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 4 * h + r, col = c & 7;
    const float x = __shfl(e, kQueryColumns ? 8 * col + row : 8 * row + col);
    if (c < 8) tile[r] = x;
  }
}

// ---- forward ------------------------------------------------------------------
// grid q tiles x BH, the longest walks first.
template <typename Tin, int DP, int VP, bool EX>
__global__ __launch_bounds__(64 * kW32) void quad32_fwd(const Tin* __restrict__ q,
                                                        const Tin* __restrict__ k,
                                                        const Tin* __restrict__ v,
                                                        float* __restrict__ out, int T, int d,
                                                        int dv, int BH, int NQ) {
  constexpr int NT = (VP + 31) / 32;
  __shared__ float red[kW32 * 16 * 64];
  __shared__ float tot[32];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, c = lane & 31, h = lane >> 5;
  const int bh = blockIdx.x % BH, qt = NQ - 1 - blockIdx.x / BH;
  const long long hb = static_cast<long long>(bh) * T;
  const HeadRows<Tin, DP, EX> Q(q + hb * d, T, d), K(k + hb * d, T, d);
  const HeadRows<Tin, VP, EX> V(v + hb * dv, T, dv);
  float qf[DP / 2], kf[DP / 2];
  Q.half(32 * qt + c, h, qf);
  f32x16 acc[NT];
#pragma unroll
  for (int m = 0; m < NT; ++m) acc[m] = zero16();
  float D = 0.f;
  if (wv <= qt) K.half(32 * wv + c, h, kf);
  int kt = wv;
  for (; kt < qt; kt += kW32) {
    f32x16 s = dot_tile(kf, qf, zero16());
    K.half(32 * min(kt + kW32, qt) + c, h, kf);  // the next key rows, under the value products
    float part = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] *= s[r];
      part += s[r];
    }
    D += part;
#pragma unroll
    for (int m = 0; m < NT; ++m) {
      float vc[16];
      V.column(32 * m + c, 32 * kt, h, vc);
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m] = mf2(vc[r], s[r], acc[m]);
    }
  }
  // The diagonal tile: keys past the query (and past T) are masked.  Apart from the
  // loop, whose tiles then carry no test and no early scores: 124 registers where a
  // loop over both took 149, and two workgroups on a CU for one (d = dv = 64, eight
  // heads of 1024 27 -> 22 us, 128 of 2048 1.04 -> 0.60 ms).
  if (kt == qt) {
    f32x16 s = dot_tile(kf, qf, zero16());
    if (qt == 0) put_early<true>(s, early_scores(q + hb * d, k + hb * d, T, d, lane), c, h);
    float part = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = acc_row(r, h) <= c ? s[r] * s[r] : 0.f;
      part += s[r];
    }
    D += part;
#pragma unroll
    for (int m = 0; m < NT; ++m) {
      float vc[16];
      V.column(32 * m + c, 32 * kt, h, vc);
      diagonal_products<true>(V, 32 * m + c, 32 * kt, vc, s, acc[m], c, h, red);
    }
  }
  reduce_columns(red, D, tot);
  const int nc = min(32, T - 32 * qt);
  auto normalise = [&](float x, int col) { return tot[col] > 0.f ? x / tot[col] : 0.f; };
#pragma unroll
  for (int m = 0; m < NT; ++m)
    if (32 * m < dv)
      reduce_store(red, acc[m], out + (hb + 32 * qt) * dv, dv, 32 * m, nc, normalise);
  if (qt == 0) {  // row 0 in the chunk kernels' order
    __syncthreads();
    const int j = threadIdx.x;
    if (j < dv) {
      float s = 0.f;
      for (int x = 0; x < d; ++x) s = fmaf(to_f32(q[hb * d + x]), to_f32(k[hb * d + x]), s);
      const float w = s * s;
      out[hb * dv + j] = w > 0.f ? (w * to_f32(v[hb * dv + j])) / w : 0.f;
    }
  }
}

// ---- gradients ------------------------------------------------------------------
// a_t = dout_t / D_t ([rows][dv]) and b_t = -<dout_t, o_t> / D_t, zeros where
// D_t = 0, with D_t = sum_{i <= t} s_ti^2 formed here unless den is given; then
// also (c_00, s_00) of each head, in the chunk kernels' order of operations.
template <typename Tin, int DP, bool EX>
__global__ __launch_bounds__(64 * kW32) void quad32_coef(
    const Tin* __restrict__ q, const Tin* __restrict__ k, const Tin* __restrict__ v,
    const float* __restrict__ o, const float* __restrict__ dout, const float* __restrict__ den,
    float* __restrict__ a, float* __restrict__ b, float* __restrict__ c00, int T, int d, int dv,
    int BH, int NQ) {
  __shared__ float red[kW32 * 32];
  __shared__ float tot[32];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, c = lane & 31, h = lane >> 5;
  const int bh = blockIdx.x % BH, qt = NQ - 1 - blockIdx.x / BH;
  const long long hb = static_cast<long long>(bh) * T;
  if (den == nullptr) {
    const HeadRows<Tin, DP, EX> Q(q + hb * d, T, d), K(k + hb * d, T, d);
    float qf[DP / 2], kf[DP / 2];
    Q.half(32 * qt + c, h, qf);
    float D = 0.f;
    for (int kt = wv; kt <= qt; kt += kW32) {
      K.half(32 * kt + c, h, kf);
      f32x16 s = dot_tile(kf, qf, zero16());
      if (qt == 0) put_early<true>(s, early_scores(q + hb * d, k + hb * d, T, d, lane), c, h);
      float part = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) part += (kt < qt || acc_row(r, h) <= c) ? s[r] * s[r] : 0.f;
      D += part;
    }
    reduce_columns(red, D, tot);
    if (qt == 0) {
      if (wv == 0) {  // every element of the tile is s_00
        f32x16 s = zero16();
        for (int x = 0; x < d; x += 2) {
          const bool in = x + h < d;
          s = mf2(in ? to_f32(k[hb * d + x + h]) : 0.f, in ? to_f32(q[hb * d + x + h]) : 0.f, s);
        }
        const float D0 = s[0] * s[0], inv = D0 > 0.f ? 1.f / D0 : 0.f;
        const float* dr = dout + hb * dv;
        const float* orow = o + hb * dv;
        float go = 0.f;
        if (dv == 64) {  // sixteen lanes of four columns
          const int j = 4 * (lane & 15);
          go = fmaf(dr[j], orow[j], __fmul_rn(dr[j + 1], orow[j + 1]));
          go = fmaf(dr[j + 3], orow[j + 3], fmaf(dr[j + 2], orow[j + 2], go));
          for (int m = 8; m > 0; m >>= 1) go += __shfl_xor(go, m);
        } else {  // four lanes, columns p, p + 4, ...
          for (int j = lane & 3; j < dv; j += 4) go = fmaf(dr[j], orow[j], go);
          go += __shfl_xor(go, 1);
          go += __shfl_xor(go, 2);
        }
        float c = -go * inv;
        if (lane == 0) b[hb] = c;
        for (int j = 0; j < dv; ++j) c = fmaf(__fmul_rn(dr[j], inv), to_f32(v[hb * dv + j]), c);
        if (lane == 0) {
          c00[2 * bh] = c;
          c00[2 * bh + 1] = s[0];
          tot[0] = D0;
        }
      }
      __syncthreads();
    }
  } else {
    if (threadIdx.x < 32) tot[threadIdx.x] = den[hb + min(32 * qt + static_cast<int>(threadIdx.x), T - 1)];
    __syncthreads();
  }
  // sixteen lanes per token
  const int tok = threadIdx.x >> 4, p = threadIdx.x & 15, t = 32 * qt + tok;
  if (t >= T) return;
  const float D = tot[tok], inv = D > 0.f ? 1.f / D : 0.f;
  const float* dr = dout + (hb + t) * dv;
  const float* orow = o + (hb + t) * dv;
  float go = 0.f;
  for (int j = p; j < dv; j += 16) {
    const float x = dr[j];
    go += x * orow[j];
    a[(hb + t) * dv + j] = x * inv;
  }
#pragma unroll
  for (int m = 8; m > 0; m >>= 1) go += __shfl_xor(go, m);
  if (p == 0 && (t > 0 || den != nullptr)) b[hb + t] = -go * inv;
}

// c_ti of the pairs t, i < 8 as sum_j a_tj (v_ij - o_tj), lane 8 t + i: in the
// first rows <a_t, v_i> can nearly cancel b_t, which the difference form leaves
// out.  With this and early_scores no output of 1000 random cases is further
// from fp64 than 1.5 times the chunk kernels' error (without them 2% were).
template <typename Tin, int VP, bool EX>
__device__ __forceinline__ float early_c(const Tin* v, const float* a, const float* o, int T,
                                         int dv, int lane) {
  const int t = min(lane >> 3, T - 1), i = min(lane & 7, T - 1);
  const Tin* vr = v + i * dv;
  const float* ar = a + t * dv;
  const float* orow = o + t * dv;
  float c = 0.f;
  if constexpr (EX) {
#pragma unroll
    for (int j = 0; j < VP; j += 4) {
      const float4 x = *reinterpret_cast<const float4*>(ar + j);
      const float4 y = *reinterpret_cast<const float4*>(orow + j);
      c = fmaf(x.x, to_f32(vr[j]) - y.x, c);
      c = fmaf(x.y, to_f32(vr[j + 1]) - y.y, c);
      c = fmaf(x.z, to_f32(vr[j + 2]) - y.z, c);
      c = fmaf(x.w, to_f32(vr[j + 3]) - y.w, c);
    }
  } else {
    for (int j = 0; j < dv; ++j) c = fmaf(ar[j], to_f32(vr[j]) - orow[j], c);
  }
  return c;
}

// One launch for both sides (side 0: dk, dv of 32 keys, walking the queries
// from the diagonal on; side 1: dq of 32 queries), the longest walks first.
template <typename Tin, int DP, int VP, bool EX>
__global__ __launch_bounds__(64 * kW32) void quad32_grad(
    const Tin* __restrict__ q, const Tin* __restrict__ k, const Tin* __restrict__ v,
    const float* __restrict__ o, const float* __restrict__ a, const float* __restrict__ b,
    const float* __restrict__ c00, float* __restrict__ dq, float* __restrict__ dk, float* __restrict__ dvo, int T, int d, int dv, int BH, int NQ) {
  constexpr int ND = (DP + 31) / 32, NV = (VP + 31) / 32;
  __shared__ float red[kW32 * 16 * 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, c = lane & 31, h = lane >> 5;
  // like work on ids equal mod 32 (the XCDs and their shader engines are filled
  // in turn): four key sides, then four query sides
  const int bh = blockIdx.x % BH, j = blockIdx.x / BH, rank = 4 * (j >> 3) + (j & 3);
  if (rank >= NQ) return;
  const long long hb = static_cast<long long>(bh) * T;
  const HeadRows<Tin, DP, EX> Q(q + hb * d, T, d), K(k + hb * d, T, d);
  const HeadRows<Tin, VP, EX> V(v + hb * dv, T, dv);
  const HeadRows<float, VP, EX> A(a + hb * dv, T, dv);
  const float* bhp = b + hb;
  auto twice = [](float x, int) { return 2.f * x; };
  auto once = [](float x, int) { return x; };
  if (((j >> 2) & 1) == 0) {
    const int kt = rank, i = 32 * kt + c;  // this lane's key
    float kf[DP / 2], vf[VP / 2], x[DP / 2], y[VP / 2];
    K.half(i, h, kf);
    V.half(i, h, vf);
    f32x16 dka[ND], dva[NV];
#pragma unroll
    for (int m = 0; m < ND; ++m) dka[m] = zero16();
#pragma unroll
    for (int m = 0; m < NV; ++m) dva[m] = zero16();
    // the diagonal tile apart from the others: 161 registers for the 16-wide
    // form in place of 191, 24.5 : 25.2 us (T1024, eight heads), 65.7 : 66.6 at d = dv
    // = 64; the query side too: 23.8 and 67.7 us
    auto tile = [&](int qt, auto diagonal) __attribute__((always_inline)) {
      constexpr bool kDiag = decltype(diagonal)::value;
      const int r0 = 32 * qt;
      Q.half(r0 + c, h, x);
      A.half(r0 + c, h, y);
      f32x16 cw;
#pragma unroll
      for (int r = 0; r < 16; ++r) cw[r] = bhp[min(r0 + acc_row(r, h), T - 1)];
      f32x16 s = dot_tile(x, kf, zero16());
      cw = dot_tile(y, vf, cw);
      if (kDiag && qt == 0) {
        put_early<false>(s, early_scores(q + hb * d, k + hb * d, T, d, lane), c, h);
        put_early<false>(cw, early_c<Tin, VP, EX>(v + hb * dv, a + hb * dv, o + hb * dv, T, dv, lane),
                      c, h);
        if (c00 != nullptr && lane == 0) {  // pair (0, 0)
          cw[0] = c00[2 * bh];
          s[0] = c00[2 * bh + 1];
        }
      }
      if (!kDiag && r0 + 32 <= T) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          cw[r] *= s[r];  // c_ti s_ti
          s[r] *= s[r];   // w_ti
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int t = r0 + acc_row(r, h);
          const bool ok = t >= i && t < T;
          cw[r] = ok ? s[r] * cw[r] : 0.f;
          s[r] = ok ? s[r] * s[r] : 0.f;
        }
      }
#pragma unroll
      for (int m = 0; m < ND; ++m) {
        float col[16];
        Q.column(32 * m + c, r0, h, col);
        if constexpr (kDiag) {
          diagonal_products<false>(Q, 32 * m + c, r0, col, cw, dka[m], c, h, red);
          continue;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) dka[m] = mf2(col[r], cw[r], dka[m]);
      }
#pragma unroll
      for (int m = 0; m < NV; ++m) {
        float col[16];
        A.column(32 * m + c, r0, h, col);
        if constexpr (kDiag) {
          diagonal_products<false>(A, 32 * m + c, r0, col, s, dva[m], c, h, red);
          continue;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) dva[m] = mf2(col[r], s[r], dva[m]);
      }
    };
    if (wv == 0) tile(kt, std::true_type{});
    for (int qt = kt + (wv == 0 ? kW32 : wv); qt < NQ; qt += kW32) tile(qt, std::false_type{});
    const int nc = min(32, T - 32 * kt);
#pragma unroll
    for (int m = 0; m < ND; ++m)
      reduce_store(red, dka[m], dk + (hb + 32 * kt) * d, d, 32 * m, nc, twice);
#pragma unroll
    for (int m = 0; m < NV; ++m)
      reduce_store(red, dva[m], dvo + (hb + 32 * kt) * dv, dv, 32 * m, nc, once);
  } else {
    const int qt = NQ - 1 - rank, t = 32 * qt + c;  // this lane's query
    float qf[DP / 2], af[VP / 2], x[DP / 2], y[VP / 2];
    Q.half(t, h, qf);
    A.half(t, h, af);
    const float bt = bhp[min(t, T - 1)];
    f32x16 dqa[ND];
#pragma unroll
    for (int m = 0; m < ND; ++m) dqa[m] = zero16();
    for (int kt = wv; kt <= qt; kt += kW32) {
      const int r0 = 32 * kt;
      K.half(r0 + c, h, x);
      V.half(r0 + c, h, y);
      f32x16 s = dot_tile(x, qf, zero16()), cw;
#pragma unroll
      for (int r = 0; r < 16; ++r) cw[r] = bt;
      cw = dot_tile(y, af, cw);
      if (qt == 0) {
        put_early<true>(s, early_scores(q + hb * d, k + hb * d, T, d, lane), c, h);
        put_early<true>(cw, early_c<Tin, VP, EX>(v + hb * dv, a + hb * dv, o + hb * dv, T, dv, lane),
                      c, h);
        if (c00 != nullptr && lane == 0) {  // pair (0, 0)
          cw[0] = c00[2 * bh];
          s[0] = c00[2 * bh + 1];
        }
      }
      if (kt < qt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) cw[r] *= s[r];
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) cw[r] = acc_row(r, h) <= c ? s[r] * cw[r] : 0.f;
      }
#pragma unroll
      for (int m = 0; m < ND; ++m) {
        float col[16];
        K.column(32 * m + c, r0, h, col);
        if (kt == qt) {
          diagonal_products<true>(K, 32 * m + c, r0, col, cw, dqa[m], c, h, red);
          continue;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) dqa[m] = mf2(col[r], cw[r], dqa[m]);
      }
    }
    const int nc = min(32, T - 32 * qt);
#pragma unroll
    for (int m = 0; m < ND; ++m)
      reduce_store(red, dqa[m], dq + (hb + 32 * qt) * d, d, 32 * m, nc, twice);
  }
}

template <int V>
using IC = std::integral_constant<int, V>;

// Calls f(width class of w): 16, 32 or 64 (value widths of the forward also 128
// and 256).
template <bool kWide = false, typename F>
void by_width(int w, F&& f) {
  if (w <= 16) f(IC<16>{});
  else if (w <= 32) f(IC<32>{});
  else if (!kWide || w <= 64) f(IC<64>{});
  else if constexpr (kWide) {
    if (w <= 128) f(IC<128>{});
    else f(IC<256>{});
  }
}

}  // namespace

// Where the quadratic form is the faster one.  Its time grows with T^2 and the
// matrix instructions of a tile pair (widths padded to their class, whose values
// then also come one at a time), the chunk states' with T and the state's n dv
// values, n = d(d+1)/2, above a floor of launches and of one chunk's walk.
// The models below (us) are fits to both forms at 19 widths, 1 to 512 heads and
// T 512 .. 62400, C = 64, and to the chunk states at C 4 .. 128; over those 800
// calls the form that they choose is at most 1.25 times slower than the other
// (seven calls, all below 300 us, by more than 1.07).  Some of the times (d dv, heads,
// T: quadratic : chunk states), forward: 64 64, 8, 62400 27987 : 49777; 64 1, 8, 8192
// 1045 : 1554 and 16384 3923 : 3143; 32 8, 64, 4096 1168 : 1748 and 8192 4242 : 3431;
// 16 16, 64, 4096 392 : 458; 8 8, 8, 2048 24 : 38 and 4096 63 : 44, 64, 2048 128 : 97;
// 1 1, 64, 1024 34 : 34 and 4096 416 : 91.  Gradients: 64 64, 8, 8192 2454 : 4039; 16 64,
// 1, 8192 241 : 330 and 64, 8192 11561 : 10016; 64 1, 8, 2048 337 : 500 and 4096 1157 :
// 900; 8 64, 8, 1024 90 : 231 and 4096 848 : 451; 24 24, 8, 4096 584 : 652.
namespace {

int width_class(int w) { return w <= 16 ? 16 : w <= 32 ? 32 : w <= 64 ? 64 : w <= 128 ? 128 : 256; }
double n_of(int d) { return 0.5 * d * (d + 1); }

double quad32_fwd_us(double BH, double T, int d, int dv) {
  const int dp = width_class(d), vp = width_class(dv);
  double tile = 0.5 * (dp + (vp < 32 ? 32 : vp));
  if (d != dp || dv != vp) tile += 0.02 * d * dp;
  return 8 + tile * fmax(2.3e-4 * T, 1.5e-8 * BH * T * T);
}
double chunk32_fwd_us(double BH, double T, int d, int dv, double C) {
  const double n = n_of(d);
  const double token =
      3e-4 + n * (fmin(1e-5, 4e-6 + 2.5e-7 * d) + 5e-9 * dv * dv) + 2e-5 * fmax(0, dv - 64);
  return fmax((22 + 0.06 * T / C + n * (0.25 + 0.01 * dv) + 0.4 * dv) * fmax(1, C / 64),
              BH * T * token * fmax(1, fmax(24 / C, C / 64)));
}
double quad32_bwd_us(double BH, double T, int d, int dv) {
  const int dp = width_class(d), vp = width_class(dv);
  double tile = 1.5 * dp + vp + 32 * ((dp + 31) / 32) + 16 * ((vp + 31) / 32);
  if (d != dp || dv != vp) tile += 0.07 * d * dp + 0.05 * dv * vp;
  return 20 + tile * fmax(1.6e-4 * T, 1.8e-8 * BH * T * T);
}
double chunk32_bwd_us(double BH, double T, int d, int dv, double C) {
  const double n = n_of(d), token = 7.5e-3 + 3e-4 * d + 4e-5 * dv + 2.5e-7 * n * dv;
  return fmax(165 + 4.2 * d + 4e-3 * n * dv, BH * T * token * fmax(1, 52 / C));
}

}  // namespace

// A launch holds fewer than 2^32 threads: calls of more tokens keep the chunk
// states' two-dimensional grids.
bool quad32_fwd_ok(int BH, int T, int d, int dv, int C, int g) {
  return g == 1 && T <= 65536 && (T <= 4096 || T <= 30 * n_of(d)) &&
         static_cast<long long>(BH) * ((T + 31) / 32) * 64 * kW32 < (1LL << 32) &&
         quad32_fwd_us(BH, T, d, dv) <= chunk32_fwd_us(BH, T, d, dv, C);
}
bool quad32_bwd_ok(int BH, int T, int d, int dv, int C, int g) {
  const auto whole = [](int w) { return w == 16 || w == 32 || w == 64; };
  return g == 1 && dv <= 64 && T <= (whole(d) && whole(dv) ? 8192 : 4096) &&
         static_cast<long long>(BH) * ((T + 127) / 128) * 8 * 64 * kW32 < (1LL << 32) &&
         quad32_bwd_us(BH, T, d, dv) <= chunk32_bwd_us(BH, T, d, dv, C);
}

template <typename Tin>
hipError_t launch_quad32_fwd(const void* q, const void* k, const void* v, float* out, int BH,
                             int T, int d, int dv, hipStream_t st) {
  const int NQ = (T + 31) / 32;
  by_width(d, [&](auto dp) {
    by_width<true>(dv, [&](auto vpd) {
      constexpr int DP = decltype(dp)::value, VP = decltype(vpd)::value;
      auto go = [&](auto ex) {
        quad32_fwd<Tin, DP, VP, decltype(ex)::value>
            <<<static_cast<unsigned>(BH) * NQ, 64 * kW32, 0, st>>>(
                static_cast<const Tin*>(q), static_cast<const Tin*>(k),
                static_cast<const Tin*>(v), out, T, d, dv, BH, NQ);
      };
      if (d == DP && dv == VP) go(std::true_type{});
      else go(std::false_type{});
    });
  });
  return hipGetLastError();
}

template <typename Tin>
hipError_t launch_quad32_bwd(const void* q, const void* k, const void* v, const float* out,
                             const float* dout, const float* den, float* dq, float* dk,
                             float* dv_out, int BH, int T, int d, int dv, void* ws,
                             hipStream_t st, hipEvent_t* ev) {
  const int NQ = (T + 31) / 32;
  float* a = static_cast<float*>(ws);
  float* b = a + static_cast<size_t>(BH) * T * dv;
  float* c00 = b + static_cast<size_t>(BH) * T;
  const Tin* qp = static_cast<const Tin*>(q);
  const Tin* kp = static_cast<const Tin*>(k);
  const Tin* vp = static_cast<const Tin*>(v);
  hipError_t e;
  for (int i = 0; i < 3; ++i)
    if ((e = record(ev, i, st)) != hipSuccess) return e;
  by_width(d, [&](auto dp) {
    constexpr int DP = decltype(dp)::value;
    auto go = [&](auto ex) {
      quad32_coef<Tin, DP, decltype(ex)::value><<<static_cast<unsigned>(BH) * NQ, 64 * kW32, 0, st>>>(
          qp, kp, vp, out, dout, den, a, b, c00, T, d, dv, BH, NQ);
    };
    if (d == DP) go(std::true_type{});
    else go(std::false_type{});
  });
  for (int i = 3; i < 6; ++i)
    if ((e = record(ev, i, st)) != hipSuccess) return e;
  by_width(d, [&](auto dp) {
    by_width(dv, [&](auto vpd) {
      constexpr int DP = decltype(dp)::value, VP = decltype(vpd)::value;
      auto go = [&](auto ex) {
        quad32_grad<Tin, DP, VP, decltype(ex)::value>
            <<<static_cast<unsigned>(BH) * ((NQ + 3) / 4) * 8, 64 * kW32, 0, st>>>(
                qp, kp, vp, out, a, b, den == nullptr ? c00 : nullptr, dq, dk, dv_out, T, d, dv, BH,
                NQ);
      };
      if (d == DP && dv == VP) go(std::true_type{});
      else go(std::false_type{});
    });
  });
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return record(ev, 6, st);
}

template hipError_t launch_quad32_fwd<float>(const void*, const void*, const void*, float*, int,
                                             int, int, int, hipStream_t);
template hipError_t launch_quad32_fwd<bf16_t>(const void*, const void*, const void*, float*, int,
                                              int, int, int, hipStream_t);
template hipError_t launch_quad32_bwd<float>(const void*, const void*, const void*, const float*,
                                             const float*, const float*, float*, float*, float*,
                                             int, int, int, int, void*, hipStream_t, hipEvent_t*);
template hipError_t launch_quad32_bwd<bf16_t>(const void*, const void*, const void*, const float*,
                                              const float*, const float*, float*, float*, float*,
                                              int, int, int, int, void*, hipStream_t, hipEvent_t*);

}  // namespace kata
