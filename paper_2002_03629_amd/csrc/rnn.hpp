// Backward pass of a one-layer recurrent network as a Jacobi iteration (gfx950 only).
//
// Backpropagation through T time steps is feedforward computation (Appendix A.2): with d_t = dL/dh_t,
//     d_T = g_T,     d_t = g_t + W^T (sigmoid(z_{t+1}) * d_{t+1})          (softplus units, Appendix C.1),
// every state hangs on the one after it.  The standard backward pass takes the steps one by one
// (rnn_backward_seq_kernel); Jacobi iteration (Algorithm 1; "Jacobi_n" of Section 5.1 when cut after n passes)
// updates all steps at once from the previous iterate, which turns T dependent matrix-vector products into
// one [T, H] x [H, H] matrix product per pass (rnn_jacobi_kernel).
//
// Sequences are independent, so one workgroup owns one sequence for the whole call: the iterate lives in
// its LDS, the recurrent weights in registers, all passes and the forward-difference stop test run inside
// one launch.
#pragma once

#include "kernels.hpp"

namespace jm {

constexpr int RNN_WAVES = 8;
constexpr int RNN_MAX_H = 128;
constexpr int RNN_TILES_PER_WAVE = 2;

__device__ __forceinline__ float rnn_sigmoid_fast(float z);   // (with the recurrences, below)

struct RnnJacobiArgs {
  const float* W;        // [H, H], W[i][j] multiplies h_{t-1}[j] in unit i
  const float* z;        // [B, T, H] pre-activations of the forward pass
  const float* g;        // [B, T, H] direct loss gradients dl_t/dh_t
  const float* d_init;   // [B, T, H] initial iterate or NULL (zeros)
  float* d;              // [B, T, H] result
  int* iters;            // [B] or NULL
  int* converged;        // [B] or NULL: 1 = the forward difference met eps, 0 = the pass limit ended the iteration
  int B, T, H;
  int cap;               // pass limit, 1 .. T
  float eps;
  int x_bytes;           // distance of the second copy of X in LDS; 0: there is one
};

// fp32 value = hi + lo + O(2^-17 |value|), both parts bf16 (round to nearest even; gfx950 converts in hardware)
__device__ __forceinline__ void split_bf16(float v, bf16_t& hi, bf16_t& lo) {
  const __bf16 h = (__bf16)v;
  const __bf16 l = (__bf16)(v - (float)h);
  hi = __builtin_bit_cast(bf16_t, h);
  lo = __builtin_bit_cast(bf16_t, l);
}

// One pass is D_new = G + X W with X[t] = sigmoid(z[t+1]) * D_old[t+1]: a [Tp, Hp] x [Hp, Hp] product, Tp / Hp
// = T / H rounded up to 32.  gfx950 has no fast fp32 matrix path (fp32 MFMA runs at 1/16 of the bf16 rate), so
// both operands are split into two bf16 parts and a product is three bf16 MFMAs with fp32 accumulation
// (hi*hi + hi*lo + lo*hi; the dropped lo*lo term and the split residuals are ~2^-16 of a product).
// Wave w owns column tile (32 units) w % CT for good: its two W panels (hi, lo) stay in registers, as do G,
// sigmoid(z) and the current iterate of the (at most two) 32 x 32 tiles it owns.  The MFMA takes W^T as its row
// operand, so a lane holds 4 runs of 4 consecutive units of ONE time step: inputs come in 16-byte loads and the
// new X goes back to LDS in 8-byte pieces.  X lives in LDS as two bf16 arrays [time][unit], twice where it fits: a pass
// reads one copy and writes the other, so that there is one barrier a pass and one wave's update runs beside the
// other's products (they share a SIMD); with one copy all waves read, barrier, all waves write, barrier.
// The stop test asks whether any element moved by more than eps (one ballot); the first pass from zeros has no product.
// Bound by the two together: 48 MFMAs (0.64 us a wave, two to a SIMD) and ~450 other instructions a wave and pass.
// H = 128, 100 steps, 10 passes: one sequence 44.9 -> 39.3 us, 256
// 56 -> 49.9 us, of which about 12 us are the set-up.  Tried: every input requested at once ahead of the set-up (47.5 us),
// a wave's two tiles multiplied in turn (47.4).
template <int CT>
__global__ __launch_bounds__(RNN_WAVES * 64) void rnn_jacobi_kernel(RnnJacobiArgs a) {
  constexpr int Hp = 32 * CT;
  constexpr int KB = Hp / 16;            // MFMA K blocks (16 wide) per tile
  constexpr int LDX = Hp + 8;            // row pitch of X in bf16 elements (16 bytes of padding)
  constexpr int TW = RNN_TILES_PER_WAVE;
  extern __shared__ __align__(16) unsigned char rnn_lds[];
  __shared__ int moved_s[3];             // (pass k sets one, clears the next pass's, and may still read its own then)
  const int T = a.T, H = a.H;
  const int Tp = (T + 31) / 32 * 32, RT = Tp / 32;
  const int lo_off = Tp * LDX;                       // (elements) X's low parts behind its high ones
  int x_read = 0, x_write = a.x_bytes / 2;           // (elements) the copy a pass reads, the one it writes
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cl = lane & 31, hh = lane >> 5;
  const int seq = blockIdx.x;
  const size_t base = (size_t)seq * T * H;
  const bool vec_ok = (H % 4 == 0) && (((uintptr_t)a.g | (uintptr_t)a.z | (uintptr_t)a.d | (uintptr_t)a.d_init) % 16 == 0);

  const int c = wave % CT, q = wave / CT, nq = (RNN_WAVES - c + CT - 1) / CT;   // waves q = 0 .. nq-1 share column tile c

  // W panels: for K block m the lane holds W[k][unit], unit = 32 c + cl, k = hh * Hp/2 + 8 m .. + 8 (any
  // assignment of K to lanes works as long as the X reads below use the same one)
  uint4 whi[KB], wlo[KB];
  {
    const int unit = c * 32 + cl;
#pragma unroll
    for (int m = 0; m < KB; ++m) {
      bf16_t h8[8], l8[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = hh * (Hp / 2) + 8 * m + i;
        const float w = (k < H && unit < H) ? a.W[(size_t)k * H + unit] : 0.0f;
        split_bf16(w, h8[i], l8[i]);
      }
      whi[m] = make_uint4(h8[0] | (h8[1] << 16), h8[2] | (h8[3] << 16), h8[4] | (h8[5] << 16), h8[6] | (h8[7] << 16));
      wlo[m] = make_uint4(l8[0] | (l8[1] << 16), l8[2] | (l8[3] << 16), l8[4] | (l8[5] << 16), l8[6] | (l8[7] << 16));
    }
  }

  // this wave's tiles: row (time) tiles q, q + nq.  Accumulator element e = 4 jj + i of a tile is
  // (unit = 32 c + 8 jj + 4 hh + i, time = 32 r + cl).
  float G[TW][16], S[TW][16], D[TW][16];
  bool tile_ok[TW];
  auto load4f = [&](const float* p, size_t idx, int u0, bool row_ok, float (&o)[4]) {
    if (row_ok && vec_ok && u0 + 3 < H) {
      const float4 v = *(const float4*)(p + idx);
      o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = (row_ok && u0 + i < H) ? p[idx + i] : 0.0f;
    }
  };
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const int r = q + i * nq;
    tile_ok[i] = r < RT;
    const int t = 32 * r + cl;
    const bool row_ok = tile_ok[i] && t < T;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int u0 = 32 * c + 8 * jj + 4 * hh;
      const size_t idx = base + (size_t)t * H + u0;
      float gv[4], zv[4], dv[4] = {0.f, 0.f, 0.f, 0.f};
      load4f(a.g, idx, u0, row_ok, gv);
      load4f(a.z, idx, u0, row_ok, zv);
      if (a.d_init) load4f(a.d_init, idx, u0, row_ok, dv);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        G[i][4 * jj + e] = gv[e];
        S[i][4 * jj + e] = (row_ok && u0 + e < H) ? rnn_sigmoid_fast(zv[e]) : 0.0f;
        D[i][4 * jj + e] = dv[e];
      }
    }
  }
  // X[t-1][unit .. unit+3] = S[t] * D[t], both bf16 parts (see split_bf16), 8 bytes each
  auto store_x = [&](int copy, int i, int jj) {
    const int t = 32 * (q + i * nq) + cl;
    if (t >= 1 && t < T) {
      typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
      typedef float f32x4_t __attribute__((ext_vector_type(4)));
      const f32x4_t v = {S[i][4 * jj] * D[i][4 * jj], S[i][4 * jj + 1] * D[i][4 * jj + 1], S[i][4 * jj + 2] * D[i][4 * jj + 2],
                         S[i][4 * jj + 3] * D[i][4 * jj + 3]};
      const bf16x4_t hi = __builtin_convertvector(v, bf16x4_t);
      const bf16x4_t lo = __builtin_convertvector(v - __builtin_convertvector(hi, f32x4_t), bf16x4_t);
      bf16_t* x = (bf16_t*)rnn_lds + copy + (t - 1) * LDX + 32 * c + 8 * jj + 4 * hh;
      *(bf16x4_t*)x = hi;
      *(bf16x4_t*)(x + lo_off) = lo;
    }
  };

  for (int i = threadIdx.x; i < (4 * lo_off + a.x_bytes) / 16; i += RNN_WAVES * 64) ((uint4*)rnn_lds)[i] = make_uint4(0, 0, 0, 0);
  if (threadIdx.x < 3) moved_s[threadIdx.x] = 0;
  __syncthreads();
  if (a.d_init) {
#pragma unroll
    for (int i = 0; i < TW; ++i)
      if (tile_ok[i]) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) store_x(x_read, i, jj);
      }
  }
  __syncthreads();

  int k = 0, conv = 0, slot = 0;
  while (k < a.cap) {
    ++k;
    const int next_slot = slot == 2 ? 0 : slot + 1;
    // ---- acc^T = W^T X^T for the wave's tiles
    f32x16 acc[TW];
    const bool product = k > 1 || a.d_init;
#pragma unroll
    for (int i = 0; i < TW; ++i) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = 0.0f;
      if (tile_ok[i] && product) {
        const bf16_t* x = (const bf16_t*)rnn_lds + x_read + (32 * (q + i * nq) + cl) * LDX + hh * (Hp / 2);
#pragma unroll
        for (int m = 0; m < KB; ++m) {
          const bf16x8 xh = __builtin_bit_cast(bf16x8, *(const uint4*)(x + 8 * m));
          const bf16x8 xl = __builtin_bit_cast(bf16x8, *(const uint4*)(x + lo_off + 8 * m));
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, whi[m]), xl, acc[i], 0, 0, 0);
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wlo[m]), xh, acc[i], 0, 0, 0);
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, whi[m]), xh, acc[i], 0, 0, 0);
        }
      }
    }
    if (!a.x_bytes) __syncthreads();   // (uniform) every wave has read the old X
    // ---- D = G + acc, forward difference, X[t-1] = S[t] * D[t]
    bool moved = false;
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      if (tile_ok[i]) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float dn = G[i][4 * jj + e] + acc[i][4 * jj + e];
            moved |= !(fabsf(dn - D[i][4 * jj + e]) <= a.eps);          // (a NaN never counts as converged)
            D[i][4 * jj + e] = dn;
          }
          store_x(x_write, i, jj);
        }
      }
    }
    if (__any(moved) && lane == 0) moved_s[slot] = 1;
    if (threadIdx.x == 0) moved_s[next_slot] = 0;
    lds_barrier();
    if (!moved_s[slot]) {
      conv = 1;
      break;
    }
    slot = next_slot;
    const int other = x_read;
    x_read = x_write;
    x_write = other;
  }

#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const int t = 32 * (q + i * nq) + cl;
    if (tile_ok[i] && t < T) {
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int u0 = 32 * c + 8 * jj + 4 * hh;
        float* dst = a.d + base + (size_t)t * H + u0;
        if (vec_ok && u0 + 3 < H) {
          *(float4*)dst = make_float4(D[i][4 * jj], D[i][4 * jj + 1], D[i][4 * jj + 2], D[i][4 * jj + 3]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (u0 + e < H) dst[e] = D[i][4 * jj + e];
        }
      }
    }
  }
  if (threadIdx.x == 0) {
    if (a.iters) a.iters[seq] = k;
    if (a.converged) a.converged[seq] = conv;
  }
}

// ------------------------------------------------------------------------------------------------
// The two sequential recurrences (forward pass, standard backward pass): T dependent products of one vector with
// the recurrent matrix, fp32.
//
// One workgroup per sequence, and a step is as long as its chain of dependent instructions, so the chain is what is
// kept short.  16 lanes share 8 outputs: lane kk holds M[k][j] for its H / 16 values of k and all 8 outputs j in
// registers (so a value read from LDS feeds 8 products, and the 8 sums are independent chains), and the partial sums
// meet in registers by a transposing butterfly on DPP moves: three steps halve the number of outputs a lane still
// holds, the fourth adds the row's two halves.  No partial sum goes through LDS, and with the vector double-buffered
// a step has one barrier.  Inputs that do not hang on the recurrence are requested RNN_AHEAD steps early.
// What bounds a step: 64 fmas per lane (256 cycles, one wave per SIMD), then a chain of ~70 dependent instructions and
// one LDS round trip.  Against the form before it (half a column per thread, one product per LDS word, partial sums
// and two barriers through LDS, activations from the library's expf / log1pf of ~80 instructions), H = 128, 100 steps:
// forward 121 -> 49 us for one sequence, 129 -> 54 us for 256, 165 -> 107 us for 1024; standard backward pass
// 104 -> 46, 123 -> 48, 137 -> 103 us.  (With activations that round once or twice more, from the hardware's exp2 and
// log2, it was 42 / 47 / 92 and 42 / 44 / 95 us; their errors were two to three times the library's.)
// ------------------------------------------------------------------------------------------------
constexpr int RNN_AHEAD = 4;           // steps between the request of a step's inputs and their use

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_ROR8 = 0x128;

// exp(x) for -110 <= x <= 0 as hi + lo: x = n ln 2 + r with |r| <= ln 2 / 2, exp(r) = 1 + (r + r^2 s(r)) with s a
// least-maximum fit of degree 5 (2^-34), hi the rounded sum and lo what its rounding left out; with ALL also what the
// roundings of r and of the bracket left out.  The scaling by 2^n carries denormal results.
struct ExpParts {
  float hi, lo;
};
template <bool ALL>
__device__ __forceinline__ ExpParts exp_nonpositive(float x) {
#pragma clang fp contract(off)
  const float LN2_HI = 0.693147182f, LN2_LO = -1.90465421e-9f;
  const float n = rintf(x * 1.44269502f);
  const float r0 = fmaf(n, -LN2_HI, x), r = fmaf(n, -LN2_LO, r0), r2 = r * r;   // (r0 is exact)
  const float s = fmaf(fmaf(fmaf(r, 1.9790248e-4f, 1.3944759e-3f), r2, fmaf(r, 8.3334977e-3f, 4.1666295e-2f)), r2,
                       fmaf(r, 0.16666666f, 0.5f));
  const float t = fmaf(r2, s, r), e = 1.0f + t;
  float lo = t - (e - 1.0f);
  if (ALL) lo += fmaf(n, -LN2_LO, r0 - r) + fmaf(r2, s, r - t);
  const int k = (int)n;
  return {ldexpf(e, k), ldexpf(lo, k)};
}

// sigmoid(z) and softplus(z) from exp(-|z|); a NaN stays a NaN.  A quotient is the product with the hardware's reciprocal,
// corrected by its residual (which takes in what the rounding of the denominator and of the exponential left out), so
// that about one rounding is left.  Largest / mean error in units of 2^-24, z in [-20, -5], [-5, -1], [-1, 0.1], [0.1, 1],
// [1, 5]; below it 1 / (1 + expf(-z)) and log1pf(expf(z)) of the library, several times as many instructions:
//   sigmoid  1.35 / 0.375  1.25 / 0.369  1.20 / 0.372  1.04 / 0.400  0.79 / 0.273
//   library  2.58 / 0.524  2.17 / 0.521  2.14 / 0.611  1.87 / 0.529  1.68 / 0.521
//   softplus 1.00 / 0.362  1.03 / 0.363  1.17 / 0.367  1.06 / 0.366  1.00 / 0.365
//   library  2.25 / 0.472  2.15 / 0.485  1.87 / 0.451  1.61 / 0.424  1.35 / 0.382
__device__ __forceinline__ float rnn_sigmoid_fast(float z) {
#pragma clang fp contract(off)
  const float a = fabsf(z);
  const ExpParts e = exp_nonpositive<false>(a > 110.0f ? -110.0f : -a);
  const float d = 1.0f + e.hi, d_lo = ((1.0f - d) + e.hi) + e.lo;
  const float r = __builtin_amdgcn_rcpf(d);
  const float num = z >= 0.0f ? 1.0f : e.hi, num_lo = z >= 0.0f ? 0.0f : e.lo;
  const float q = num * r;
  return fmaf(fmaf(-q, d_lo, fmaf(-q, d, num) + num_lo), r, q);
}
// log(1 + e) = 2 atanh(t / 2) = t (1 + u (1 / 3 + u / 5 + ...)) with t = e / (1 + e / 2) and u = t^2 / 4 <= 1 / 9.
__device__ __forceinline__ float rnn_softplus_fast(float z) {
#pragma clang fp contract(off)
  const float a = fabsf(z);
  const ExpParts e = exp_nonpositive<true>(a > 110.0f ? -110.0f : -a);
  const float d = fmaf(e.hi, 0.5f, 1.0f), d_lo = fmaf(e.hi, 0.5f, 1.0f - d);
  const float r = __builtin_amdgcn_rcpf(d), t = e.hi * r;
  const float rest = fmaf(-t, d_lo, fmaf(-t, d, e.hi)) + e.lo * r;
  const float half = 0.5f * t, u = half * half;
  const float q = fmaf(fmaf(fmaf(fmaf(u, 0.12150466f, 0.10713829f), u, 0.14308442f), u, 0.19999439f), u, 0.33333337f);
  const float lo = fmaf(rest, r, t * u * q);
  const float m = z <= 0.0f ? 0.0f : z;
  const float sum = m + t, b = sum - m, err = (m - (sum - b)) + (t - b);   // (sum + err = m + t exactly)
  return z > 20.0f ? z : sum + (err + lo);
}

// Lane kk's k indices of an H = 32 CT wide vector: the reads of a row of 16 lanes are contiguous (16 bytes per lane
// for an even CT, 8 for an odd one).
template <int CT>
struct RnnStep {
  static constexpr int HP = 32 * CT, KL = HP / 16, RUN = CT % 2 == 0 ? 4 : 2, THREADS = 2 * HP;
  float m[KL][8];
  // which of a row's 8 outputs a lane ends up with (the butterfly's order: bits 2, 0, 1 of the lane number)
  __device__ __forceinline__ static int output_of(int lane) { return (lane & 4) + 2 * (lane & 1) + ((lane >> 1) & 1); }
  __device__ __forceinline__ static int k_of(int kk, int i) { return (i / RUN) * (16 * RUN) + kk * RUN + i % RUN; }
  // out[j] = sum_k v[k] (TRANSPOSED ? W[j][k] : W[k][j]) for the 8 outputs j0 .. j0 + 7
  template <bool TRANSPOSED>
  __device__ __forceinline__ void load(const float* W, int H, int j0, int kk) {
#pragma unroll
    for (int i = 0; i < KL; ++i)
#pragma unroll
      for (int o = 0; o < 8; ++o) {
        // (loads from an address that is always valid: no branch per element)
        const int k = k_of(kk, i), j = j0 + o, kc = min(k, H - 1), jc = min(j, H - 1);
        const float w = W[TRANSPOSED ? (size_t)jc * H + kc : (size_t)kc * H + jc];
        m[i][o] = k < H && j < H ? w : 0.0f;
      }
  }
  // the sum for output j0 + output_of(lane) (both halves of the row hold it)
  __device__ __forceinline__ float product(const float* v, int kk, int lane) const {
    float x[KL];
#pragma unroll
    for (int i = 0; i < KL; i += RUN) {
      if constexpr (RUN == 4) {
        const float4 t = *(const float4*)(v + k_of(kk, i));
        x[i] = t.x; x[i + 1] = t.y; x[i + 2] = t.z; x[i + 3] = t.w;
      } else {
        const float2 t = *(const float2*)(v + k_of(kk, i));
        x[i] = t.x; x[i + 1] = t.y;
      }
    }
    float s[8];
#pragma unroll
    for (int o = 0; o < 8; ++o) s[o] = x[0] * m[0][o];
#pragma unroll
    for (int i = 1; i < KL; ++i)
#pragma unroll
      for (int o = 0; o < 8; ++o) s[o] = fmaf(x[i], m[i][o], s[o]);
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
    float q[4], w[2];
#pragma unroll
    for (int o = 0; o < 4; ++o) q[o] = (b2 ? s[o + 4] : s[o]) + dpp_move<DPP_HALF_MIRROR>(b2 ? s[o] : s[o + 4]);
#pragma unroll
    for (int o = 0; o < 2; ++o) w[o] = (b0 ? q[o + 2] : q[o]) + dpp_move<DPP_XOR1>(b0 ? q[o] : q[o + 2]);
    const float t = (b1 ? w[1] : w[0]) + dpp_move<DPP_XOR2>(b1 ? w[0] : w[1]);
    return t + dpp_move<DPP_ROR8>(t);
  }
};

// Runs step(i, t) for t = first, first + dir, ... (T steps); i = place in a group of RNN_AHEAD steps, a constant after
// unrolling (it indexes registers).
template <typename F>
__device__ __forceinline__ void rnn_steps(int T, int first, int dir, F&& step) {
  int t = first, n = T;
  for (; n >= RNN_AHEAD; n -= RNN_AHEAD, t += RNN_AHEAD * dir)
    static_for<RNN_AHEAD>([&](auto I) { step(I, t + decltype(I)::value * dir); });
  static_for<RNN_AHEAD - 1>([&](auto I) {
    if (decltype(I)::value < n) step(I, t + decltype(I)::value * dir);
  });
}

// The standard backward pass (Section 5.1's "feedforward" baseline): T dependent steps, last step first.
// FULL: H = 32 CT, no lane without a unit.
template <int CT, bool FULL>
__global__ __launch_bounds__(RnnStep<CT>::THREADS) void rnn_backward_seq_kernel(const float* W, const float* z, const float* g,
                                                                                float* d, int T, int H) {
  __shared__ __align__(16) float v[2][RnnStep<CT>::HP];
  const int lane = threadIdx.x & 63, kk = lane & 15, j0 = (threadIdx.x >> 4) * 8;
  const int j = j0 + RnnStep<CT>::output_of(lane);
  const bool ok = FULL || j < H, first = (lane & 8) == 0;
  const float* zs = z + (size_t)blockIdx.x * T * H + (ok ? j : 0);
  const float* gs = g + (size_t)blockIdx.x * T * H + (ok ? j : 0);
  float* ds = d + (size_t)blockIdx.x * T * H + j;
  RnnStep<CT> m;
  m.template load<false>(W, H, j0, kk);
  float gn[RNN_AHEAD], zn[RNN_AHEAD];
#pragma unroll
  for (int i = 0; i < RNN_AHEAD; ++i) {
    const size_t o = (size_t)max(T - 2 - i, 0) * H;
    gn[i] = gs[o];
    zn[i] = zs[o];
  }
  if (first) {                                 // the last state is g, whatever W holds
    const size_t o = (size_t)(T - 1) * H;
    const float dj = gs[o];
    v[1][j] = ok ? rnn_sigmoid_fast(zs[o]) * dj : 0.0f;
    if (ok) ds[o] = dj;
  }
  __syncthreads();
  rnn_steps(T - 1, T - 2, -1, [&](auto I, int t) {
    constexpr int i = decltype(I)::value;
    const float gt = gn[i], st = rnn_sigmoid_fast(zn[i]);
    const size_t o = (size_t)max(t - RNN_AHEAD, 0) * H;
    gn[i] = gs[o];
    zn[i] = zs[o];
    const float dj = gt + m.product(v[(i + 1) & 1], kk, lane);
    if (first) {
      v[i & 1][j] = ok ? st * dj : 0.0f;       // the next (earlier) step reads sigmoid(z_t) * d_t
      if (ok) ds[(size_t)t * H] = dj;
    }
    lds_barrier();
  });
}

// Forward pass: z_t = W h_{t-1} + U x_t + b, h_t = softplus(z_t), one step after the other.  The part that does not
// hang on the recurrence, U x_t + b, is computed for all steps first and waits in z.
template <int CT, bool FULL>
__global__ __launch_bounds__(RnnStep<CT>::THREADS) void rnn_forward_kernel(const float* W, const float* U, const float* b, const float* x,
                                                                           const float* h0, float* z, float* h, int T, int H, int I) {
  constexpr int HP = RnnStep<CT>::HP;
  __shared__ __align__(16) float v[2][HP];
  const int lane = threadIdx.x & 63, kk = lane & 15, j0 = (threadIdx.x >> 4) * 8;
  const int j = j0 + RnnStep<CT>::output_of(lane);
  const bool ok = FULL || j < H, first = (lane & 8) == 0;
  float* zs = z + (size_t)blockIdx.x * T * H;
  RnnStep<CT> m;
  m.template load<true>(W, H, j0, kk);
  {
    const int ju = threadIdx.x % HP, half = threadIdx.x / HP;
    const float* xs = x + (size_t)blockIdx.x * T * I;
    if (FULL || ju < H) {
      const float bj = b[ju], u0 = U[(size_t)ju * I];
      for (int t0 = half; t0 < T; t0 += 2 * RNN_AHEAD) {
        float in[RNN_AHEAD];
#pragma unroll
        for (int i = 0; i < RNN_AHEAD; ++i) in[i] = fmaf(u0, xs[(size_t)min(t0 + 2 * i, T - 1) * I], bj);
        for (int c = 1; c < I; ++c) {
          const float u = U[(size_t)ju * I + c];
#pragma unroll
          for (int i = 0; i < RNN_AHEAD; ++i) in[i] = fmaf(u, xs[(size_t)min(t0 + 2 * i, T - 1) * I + c], in[i]);
        }
#pragma unroll
        for (int i = 0; i < RNN_AHEAD; ++i)
          if (t0 + 2 * i < T) zs[(size_t)(t0 + 2 * i) * H + ju] = in[i];
      }
    }
  }
  if (first) v[1][j] = ok && h0 ? h0[(size_t)blockIdx.x * H + j] : 0.0f;
  __syncthreads();
  const float* zin = zs + (ok ? j : 0);
  float* out = (first ? z : h) + (size_t)blockIdx.x * T * H + j;      // the row's two halves store one output each
  float in[RNN_AHEAD];
#pragma unroll
  for (int i = 0; i < RNN_AHEAD; ++i) in[i] = zin[(size_t)min(i, T - 1) * H];
  rnn_steps(T, 0, 1, [&](auto I_, int t) {
    constexpr int i = decltype(I_)::value;
    const float zt = in[i] + m.product(v[(i + 1) & 1], kk, lane);
    // (near the end the last step's own z is read again, possibly after it has been replaced: never used)
    in[i] = zin[(size_t)min(t + RNN_AHEAD, T - 1) * H];
    const float ht = rnn_softplus_fast(zt);
    if (first) v[i & 1][j] = ok ? ht : 0.0f;
    if (ok) out[(size_t)t * H] = first ? zt : ht;
    lds_barrier();
  });
}

// Parameter gradients from the states (Appendix A.2: "immediately computed" once they are known), with
// p_t = sigmoid(z_t) * d_t:   dW[i][j] = sum p_t[i] h_{t-1}[j],   dU[i][c] = sum p_t[i] x_t[c],   db[i] = sum p_t[i],
// sums over all steps of all sequences: a [H, B T] x [B T, H + I + 1] product in fp32.
//
// A workgroup owns a strip of 32 units i against all j, for a slice of the B T rows (blockIdx.x = strip, .y = slice):
// p of a row is then computed once per launch, and a strip's 32 x H sums fit a few accumulators.  The slice is walked
// in chunks of 64 rows that go through LDS, the next chunk's loads in flight (registers) while this one is multiplied
// with fp32 MFMA; wave w takes column tile w % CT and every (8 / CT)-th part of the chunk's rows.  dU and db ride
// along on the vector units from the same p (slot 0 of the eight columns of blockIdx.z = 0 is db, the rest inputs).
// Two workgroups to a compute unit fill each other's waits for a chunk.  With one slice the results
// are stored; with several every slice's sums go to a piece of static device memory and a kernel of its own adds them
// in slice order, so that two calls give the same bits.
// H = 128, 100 steps: 256 sequences 27.2 us for the product (29.7 with one workgroup to a compute unit and the library's
// exponential), 4.6 us for the addition, 4 us for taking a piece (in all, before: 33 us; 30 us when the slices were added by fp32 atomics in order of completion), one sequence 8.8 us; with a
// workgroup per 32 x 32 tile of dW over all rows (16 workgroups, loads waited for one by one) 2900 us and 11.8 us.
constexpr int GRAD_ROWS = 64;         // rows per chunk
constexpr int GRAD_SLOTS = 8;         // columns of [1, x] per blockIdx.z

// The slices' sums.  There are GRAD_PIECES pieces per GPU, held until the process ends.  A call with several slices takes
// a free one at its start and gives it back at its end, both on the GPU and in stream order, under a key that no other
// call in flight has: calls on any streams and threads, recorded ones too, never share a piece.  A call that finds none
// free adds its slices in one workgroup per strip instead: the same sums in the same order, without the spread over
// the chip.
constexpr int GRAD_PIECES = 4;
constexpr long long GRAD_PIECE_FLOATS = 10 << 18;      // 10 MiB: 128 slices of H = 128, I up to 28
__device__ float g_grad_piece[GRAD_PIECES][GRAD_PIECE_FLOATS];
constexpr int GRAD_KEY_SHIFT = 16;
// 0 = free, else the key of the call that holds the piece << GRAD_KEY_SHIFT + workgroups of its adding kernel that are
// through with it (at most GRAD_PIECE_FLOATS / 256)
__device__ unsigned long long g_grad_owner[GRAD_PIECES];

__global__ void rnn_grads_claim_kernel(unsigned long long key) {
  for (int i = 0; i < GRAD_PIECES; ++i)
    if (atomicCAS(&g_grad_owner[i], 0ull, key << GRAD_KEY_SHIFT) == 0ull) return;
}
// the piece that belongs to the call, or -1
__device__ __forceinline__ int rnn_grads_piece(unsigned long long key) {
  int piece = -1;
#pragma unroll
  for (int i = 0; i < GRAD_PIECES; ++i)
    if (__hip_atomic_load(&g_grad_owner[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> GRAD_KEY_SHIFT == key) piece = i;
  return piece;
}

// The slices are added in GRAD_GROUPS groups of consecutive ones, the groups' sums then in order: a thread of the adding
// kernel has all of a group's values (of four outputs) in flight at once.
constexpr int GRAD_GROUPS = 4;
__host__ __device__ constexpr int grad_group(int slices) { return (slices + GRAD_GROUPS - 1) / GRAD_GROUPS; }
__host__ __device__ constexpr long long grad_stride(int H, int I) { return ((long long)H * ((long long)H + I + 1) + 3) / 4 * 4; }

__global__ __launch_bounds__(64 * GRAD_GROUPS) void rnn_grads_add_kernel(unsigned long long key, int slices, int stride, int n_w, int n_u,
                                                                         int n_b, float* dW, float* dU, float* db) {
  __shared__ float4 part[GRAD_GROUPS][64];
  const int piece = rnn_grads_piece(key);
  if (piece < 0) return;                                 // (the results are in place)
  const int lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = 4 * (blockIdx.x * 64 + lane), group = grad_group(slices);
  const float4* p = (const float4*)(g_grad_piece[piece] + min(i, stride - 4));
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  const int end = min((g + 1) * group, slices);
  for (int s = g * group; s < end; s += 16) {
    float4 q[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) q[k] = p[(size_t)min(s + k, end - 1) * (stride / 4)];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (s + k < end) { v.x += q[k].x; v.y += q[k].y; v.z += q[k].z; v.w += q[k].w; }
  }
  part[g][lane] = v;
  __syncthreads();                                       // (everybody's part has been read)
  if (threadIdx.x == 64) {                               // the last workgroup frees the piece
    const unsigned long long n = __hip_atomic_fetch_add(&g_grad_owner[piece], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n + 1 == (key << GRAD_KEY_SHIFT) + gridDim.x)
      __hip_atomic_store(&g_grad_owner[piece], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (g == 0) {
#pragma unroll
    for (int k = 1; k < GRAD_GROUPS; ++k) {
      const float4 q = part[k][lane];
      v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
    }
    const float o[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = i + e;
      if (n < n_w + n_u + n_b) *(n < n_w ? dW + n : n < n_w + n_u ? dU + (n - n_w) : db + (n - n_w - n_u)) = o[e];
    }
  }
}

// (second launch bound: waves per SIMD, i.e. two workgroups to a compute unit)
template <int CT>
__global__ __launch_bounds__(RNN_WAVES * 64, 4) void rnn_param_grads_kernel(const float* z, const float* h, const float* x, const float* d,
                                                                         const float* h0, long long rows, int T, int H, int I,
                                                                         int slice_rows, int slices, unsigned long long key,
                                                                         float* dW, float* dU, float* db) {
  constexpr int Hp = 32 * CT, NQ = RNN_WAVES / CT;
  constexpr int LDH = Hp % 64 == 32 ? Hp : Hp + 32;       // rows k and k + 1 of a read sit 32 banks apart
  constexpr int STAGE = GRAD_ROWS * (LDH + 32 + GRAD_SLOTS), RED = RNN_WAVES * 32 * 33;
  __shared__ __align__(16) float lds[STAGE > RED ? STAGE : RED];
  float* Hs = lds;                                        // [64][LDH]  h_{t-1}
  float* Ps = lds + GRAD_ROWS * LDH;                      // [64][32]   p of the strip
  float* Xs = Ps + GRAD_ROWS * 32;                        // [64][8]    1 and inputs
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cl = lane & 31, hh = lane >> 5;
  const int u0 = blockIdx.x * 32;
  const bool gemm = blockIdx.z == 0;
  const int slot0 = blockIdx.z * GRAD_SLOTS;              // slot s of this block: s = 0: ones, else input s - 1
  const bool vec_ok = (H % 4 == 0) && (((uintptr_t)z | (uintptr_t)h | (uintptr_t)d | (uintptr_t)h0) % 16 == 0);

  auto load4 = [&](const float* p, int col, bool ok) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (ok && vec_ok && col + 3 < H) v = *(const float4*)(p + col);
    else if (ok) {
      if (col < H) v.x = p[col];
      if (col + 1 < H) v.y = p[col + 1];
      if (col + 2 < H) v.z = p[col + 2];
      if (col + 3 < H) v.w = p[col + 3];
    }
    return v;
  };
  float4 hv[CT], zv, dv;
  float xv;
  long long r_begin;
  int n_rows, t_begin;                                    // rows of the slice, step of its first one
  auto start = [&](int slice) {
    r_begin = (long long)slice * slice_rows;
    n_rows = (int)max(0LL, min((long long)slice_rows, rows - r_begin));
    t_begin = (int)(r_begin % T);
  };
  auto request = [&](int c) {                             // chunk c of the slice -> registers
    if (gemm) {
#pragma unroll
      for (int k = 0; k < CT; ++k) {
        const int e = (tid + k * RNN_WAVES * 64) * 4, row = c * GRAD_ROWS + e / Hp, col = e % Hp;
        const bool ok = row < n_rows;
        const long long r = r_begin + row;
        const bool first = (t_begin + row) % T == 0;
        const float* src = !first ? h + (r - 1) * H : (h0 ? h0 + (r / T) * H : nullptr);
        hv[k] = load4(src, col, ok && src != nullptr);
      }
    }
    {
      const int row = c * GRAD_ROWS + (tid >> 3), col = u0 + (tid & 7) * 4;
      const bool ok = row < n_rows;
      zv = load4(z + (r_begin + row) * H, col, ok);
      dv = load4(d + (r_begin + row) * H, col, ok);
      const int s = slot0 + (tid & 7);
      xv = ok && s <= I ? (s == 0 ? 1.0f : x[(r_begin + row) * I + s - 1]) : 0.0f;
    }
  };

  const int tj = wave % CT, q = wave / CT;                // (CT = 3: two waves without a part)
  const int unit = tid & 31, part = tid >> 5;             // [1, x] columns: thread (unit, 16th of the chunk's rows)
  constexpr int EPT = 32 * Hp / (RNN_WAVES * 64);         // elements of dW per thread
  float sum_w[EPT], sum_x = 0.0f, all_w[EPT], all_x = 0.0f;   // of a slice or a group of slices; of the groups before it
#pragma unroll
  for (int k = 0; k < EPT; ++k) sum_w[k] = all_w[k] = 0.0f;
  const int slice0 = blockIdx.y;
  start(slice0);
  request(0);
  // one workgroup of the strip to a slice, or (no piece) its first one to all of them
  const int piece = slices > 1 ? rnn_grads_piece(key) : -1;
  if (piece < 0 && slice0 > 0) return;
  const int slice1 = piece < 0 ? slices : slice0 + 1, group = grad_group(slices);
  for (int slice = slice0; slice < slice1; ++slice) {
    if (slice > slice0) {
      start(slice);
      request(0);
      if (slice % group == 0) {
#pragma unroll
        for (int k = 0; k < EPT; ++k) { all_w[k] += sum_w[k]; sum_w[k] = 0.0f; }
        all_x += sum_x;
        sum_x = 0.0f;
      }
    }
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
    float sums[GRAD_SLOTS];
#pragma unroll
    for (int s = 0; s < GRAD_SLOTS; ++s) sums[s] = 0.0f;
    const int n_chunks = (n_rows + GRAD_ROWS - 1) / GRAD_ROWS;
    for (int c = 0; c < n_chunks; ++c) {
      __syncthreads();                                    // the chunk before has been read
      if (gemm) {
#pragma unroll
        for (int k = 0; k < CT; ++k) {
          const int e = (tid + k * RNN_WAVES * 64) * 4;
          *(float4*)(Hs + (e / Hp) * LDH + e % Hp) = hv[k];
        }
      }
      *(float4*)(Ps + tid * 4) = make_float4(rnn_sigmoid_fast(zv.x) * dv.x, rnn_sigmoid_fast(zv.y) * dv.y,
                                             rnn_sigmoid_fast(zv.z) * dv.z, rnn_sigmoid_fast(zv.w) * dv.w);
      Xs[tid] = xv;
      __syncthreads();
      if (c + 1 < n_chunks) request(c + 1);
      if (gemm && q < NQ) {
#pragma unroll 4
        for (int m = 0; m < GRAD_ROWS / NQ; m += 2) {
          const int k = q * (GRAD_ROWS / NQ) + m + hh;
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(Ps[k * 32 + cl], Hs[k * LDH + 32 * tj + cl], acc, 0, 0, 0);
        }
      }
#pragma unroll
      for (int m = 0; m < GRAD_ROWS / 16; ++m) {
        const int k = part * (GRAD_ROWS / 16) + m;
        const float p = Ps[k * 32 + unit];
#pragma unroll
        for (int s = 0; s < GRAD_SLOTS; ++s) sums[s] = fmaf(p, Xs[k * GRAD_SLOTS + s], sums[s]);
      }
    }
    // acc[e] = element (row = 8 (e / 4) + 4 hh + e % 4 -> unit of the strip, col = cl -> unit of the column tile)
    __syncthreads();
    if (gemm) {
#pragma unroll
      for (int e = 0; e < 16; ++e) lds[(wave * 32 + 8 * (e >> 2) + 4 * hh + (e & 3)) * 33 + cl] = acc[e];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        const int e = tid + k * RNN_WAVES * 64, i = e / Hp, j = e % Hp;
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < NQ; ++w) s += lds[((w * CT + j / 32) * 32 + i) * 33 + j % 32];
        sum_w[k] += s;
      }
      __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < GRAD_SLOTS; ++s) lds[(part * GRAD_SLOTS + s) * 32 + unit] = sums[s];
    __syncthreads();
    if (tid < 32 * GRAD_SLOTS) {
      float s = 0.0f;
#pragma unroll
      for (int w = 0; w < 16; ++w) s += lds[(w * GRAD_SLOTS + (tid >> 5)) * 32 + (tid & 31)];
      sum_x += s;
    }
  }
  // (a piece: [slice][dW, dU, db])
  float* sums_w = piece < 0 ? dW : g_grad_piece[piece] + slice0 * grad_stride(H, I);
  float* sums_u = piece < 0 ? dU : sums_w + H * H;
  float* sums_b = piece < 0 ? db : sums_u + H * I;
  if (gemm) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const int e = tid + k * RNN_WAVES * 64, i = e / Hp, j = e % Hp;
      if (u0 + i < H && j < H) sums_w[(size_t)(u0 + i) * H + j] = all_w[k] + sum_w[k];
    }
  }
  if (tid < 32 * GRAD_SLOTS) {
    const int s = slot0 + (tid >> 5), u = u0 + (tid & 31);
    if (u < H && s <= I) *(s == 0 ? sums_b + u : sums_u + (size_t)u * I + s - 1) = all_x + sum_x;
  }
}

}  // namespace jm
