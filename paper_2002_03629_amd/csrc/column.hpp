// Block-wise forward substitution in one launch: GS-Jacobi blocks and the lean sequential sampler of a Bernoulli MLP
// (gfx950 only).
//
// Hidden units are sorted by degree, so the network is block lower triangular in the positions: the units of degree
// a .. b-1 and the outputs of positions [a, b) need the inputs before a, the hidden units of degree < a -- all final
// once the positions before a are -- and one another.  A workgroup owns COL_S samples for the whole call and walks the
// blocks:
//   1. all waves multiply the block's rows of every layer with the final inputs (a contraction over up to two thousand
//      inputs: matrix instructions, K split over the waves, weights streamed from L2, activations in LDS) and stage the
//      weights between the block's own units and positions in LDS;
//   2. one wave per sample solves the block: a lane owns one unit of every layer (and one position), its fp32
//      pre-activation in a register; a value that becomes known is broadcast and multiplied into the lanes that see it.
//      Sequential sampling draws one position after the other and adds what it changes; GS-Jacobi evaluates the
//      block from its base sums pass by pass until nothing changes.
// Every visible weight is read once per workgroup and call instead of once per pass, and nothing waits for another
// workgroup.  What bounds it: phase 2's chain of broadcasts and LDS reads (about 0.2 us per position) and, per block,
// the L2 latency of phase 1.
#pragma once

#include "kernels.hpp"

namespace jm {

constexpr int COL_S = 4;            // samples per workgroup: one per SIMD in phase 2, whose instruction issue bounds it
constexpr int COL_WAVES = 8;
constexpr int COL_UNITS = 64;       // units of one layer whose degree falls into a block, at most (one per lane)
constexpr int COL_POS = 32;         // positions of a block, at most
constexpr int COL_MAX_L = 3;        // hidden layers

struct ColumnArgs {
  const void* W[COL_MAX_L + 1];
  const float* bias[COL_MAX_L + 1];
  const int* cnt_lt[COL_MAX_L];     // [D + 2] units of degree < t (1-based degrees)
  int k_chunks[COL_MAX_L + 1];
  int lds_act[COL_MAX_L + 1];       // byte offsets into dynamic LDS: input of layer l, COL_S samples
  int lds_w[COL_MAX_L + 1];         // staged weights of layer l (float), input-major
  int lds_cnt[COL_MAX_L];
  int lds_red, lds_clear;           // partial sums of phase 1; bytes to clear at the start (inputs and staged weights)
  int lds_passes;                   // GS-Jacobi: [n_blocks] bytes, most passes of one of this workgroup's samples
  const int* bounds;                // sequential: block boundaries [n_blocks + 1]; NULL: blocks of `block` positions
  int n_blocks, block;
  int D, N;
  const float* noise;               // u[N, D]
  const uint8_t* x_init;            // GS-Jacobi: [N, D] or NULL
  uint8_t* x;                       // [N, D]
  int* iters;                       // GS-Jacobi: [N] passes
  // GS-Jacobi, device, zero between calls: finished workgroups and sample-passes; [n_blocks] most passes of a sample
  unsigned long long* ctr;
  int* block_passes;
  unsigned long long* host;         // pinned host memory: [0] passes, [1] sample-passes, [2] call_id when both are there
  unsigned long long call_id;
};

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ f32x4 col_mfma(const uint4& a, const uint4& b, f32x4 acc, bf16_t) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
__device__ __forceinline__ f32x4 col_mfma(const uint4& a, const uint4& b, f32x4 acc, float) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
}
__device__ __forceinline__ float col_value(float v, float) { return v; }
__device__ __forceinline__ float col_value(float v, bf16_t) { return bf16_to_f32(f32_to_bf16(v)); }   // as the layers store it

// Phase 1 of one layer: rows [row0, row0 + n_rows) (NT tiles of 16, the last one's surplus rows repeat the last row)
// times the first n_steps K steps of the input, this wave's share (steps wave, wave + COL_WAVES, ...), to
// red[wave][sample][red_row + row].  A K step is half a chunk (64 bytes per row): lane (row r, quarter q) holds piece
// (slot 2 (step % 2) + q / 2, half q % 2) of it.  Only COL_S of the 16 columns differ: lane r reads sample r % COL_S.
template <typename T, int NT>
__device__ __forceinline__ void col_product(const T* W, int k_chunks, const unsigned char* act, int row0, int n_rows,
                                            int n_steps, float* red, int red_pitch, int red_row) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, q = lane >> 4;
  const unsigned char* wp[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int row = row0 + min(16 * t + r, n_rows - 1);
    wp[t] = (const unsigned char*)W + (size_t)(row >> 5) * k_chunks * 4096 + (((q >> 1) * 2 + (q & 1)) * 32 + (row & 31)) * 16;
  }
  // (activations: 16-byte piece (chunk, half, slot) of sample s at ((chunk * 8 + half * 4 + slot) * COL_S + s) * 16)
  const unsigned char* ap = act + (((q & 1) * 4 + (q >> 1)) * COL_S + (r & (COL_S - 1))) * 16;
  f32x4 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto group = [&](auto CNT, int j0) {
    constexpr int cnt = decltype(CNT)::value;
    uint4 w[cnt][NT], x[cnt];
#pragma unroll
    for (int i = 0; i < cnt; ++i) {
      const int j = j0 + i * COL_WAVES;
#pragma unroll
      for (int t = 0; t < NT; ++t) w[i][t] = *(const uint4*)(wp[t] + (size_t)j * 2048);
    }
#pragma unroll
    for (int i = 0; i < cnt; ++i) {
      const int j = j0 + i * COL_WAVES;
      x[i] = *(const uint4*)(ap + ((j >> 1) * 8 + (j & 1) * 2) * COL_S * 16);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < cnt; ++i)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = col_mfma(w[i][t], x[i], acc[t], T{});
  };
  int j = wave;
  for (; j + 3 * COL_WAVES < n_steps; j += 4 * COL_WAVES) group(std::integral_constant<int, 4>{}, j);
  for (; j < n_steps; j += COL_WAVES) group(std::integral_constant<int, 1>{}, j);
  // acc[t][i]: row 16 t + 4 q + i, sample r
  if (r < COL_S) {
    float* dst = red + (size_t)(wave * COL_S + r) * red_pitch + red_row + 4 * q;
#pragma unroll
    for (int t = 0; t < NT; ++t) *(f32x4*)(dst + 16 * t) = acc[t];
  }
}

// Stage the weights of rows [row0, row0 + n_rows) x inputs [k0, k0 + n_k) as floats, ws[input * pitch + row]; inputs
// n_k .. up to a multiple of 8 are set to zero.
template <typename T>
__device__ __forceinline__ void col_stage(const T* W, int k_chunks, int row0, int n_rows, int k0, int n_k, float* ws,
                                          int pitch) {
  constexpr int EPL = Elem<T>::EPL, KC = 2 * EPL, P = 16 / (int)sizeof(T);
  const int p0 = k0 / P, n_pieces = n_k > 0 ? (k0 + n_k - 1) / P - p0 + 1 : 0;
  for (int i = threadIdx.x; i < n_pieces * pitch; i += COL_WAVES * 64) {
    const int row = i % pitch, k = (p0 + i / pitch) * P;
    if (row >= n_rows) continue;
    const int g = row0 + row, c = k / KC, kk = k % KC, h = kk / EPL, s = (kk % EPL) / P;
    const uint4 v = *(const uint4*)((const unsigned char*)W + ((size_t)(g >> 5) * k_chunks + c) * 4096 +
                                    ((s * 2 + h) * 32 + (g & 31)) * 16);
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < P; ++e) {
      const int kl = k + e - k0;
      float f;
      if constexpr (sizeof(T) == 2) f = __uint_as_float((e & 1) ? (u[e / 2] & 0xffff0000u) : (u[e / 2] << 16));
      else f = __uint_as_float(u[e]);
      if (kl >= 0 && kl < n_k) ws[kl * pitch + row] = f;
    }
  }
  const int n8 = (n_k + 7) & ~7;
  for (int i = threadIdx.x; i < (n8 - n_k) * pitch; i += COL_WAVES * 64) ws[n_k * pitch + i] = 0.f;
}

// sum + ws[u][lane] * h_u for the units u in [s, e): h_u sits in lane u of h
__device__ __forceinline__ float col_add_units(const float* ws, int pitch, int col, float h, int s, int e, float sum) {
  for (int u = s; u < e; u += 4) {
    // (requested before the first is used; rows past the range repeat its last one and are not multiplied)
    float w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = ws[min(u + i, e - 1) * pitch + col];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (u + i < e) sum = fmaf(w[i], __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(h), u + i)), sum);
  }
  return sum;
}
// the same over all units [0, n8), n8 a multiple of 8 (surplus rows and values are zero)
__device__ __forceinline__ float col_add_all(const float* ws, int pitch, int col, float h, int n8, float sum) {
  for (int u = 0; u < n8; u += 8) {
    float w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = ws[(u + i) * pitch + col];
#pragma unroll
    for (int i = 0; i < 8; ++i) sum = fmaf(w[i], __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(h), u + i)), sum);
  }
  return sum;
}

template <typename T, int L, bool SEQ>
__global__ __launch_bounds__(COL_WAVES * 64) void column_sampler_kernel(ColumnArgs p) {
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ unsigned long long passes_s[COL_S];
  __shared__ int block_passes_s[COL_S], all_passes_s, last_s;
  constexpr int NT_ = COL_WAVES * 64;
  constexpr int EPL = Elem<T>::EPL, KC = 2 * EPL, P = 16 / (int)sizeof(T);
  constexpr int RED = COL_UNITS * L + COL_POS;     // rows of a block over all layers
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int D = p.D;
  for (int i = threadIdx.x; i < p.lds_clear / 16; i += NT_) ((uint4*)lds)[i] = make_uint4(0, 0, 0, 0);
#pragma unroll
  for (int l = 0; l < L; ++l)
    for (int i = threadIdx.x; i < D + 2; i += NT_) ((int*)(lds + p.lds_cnt[l]))[i] = p.cnt_lt[l][i];
  __syncthreads();

  float* red = (float*)(lds + p.lds_red);
  const int n = blockIdx.x * COL_S + wave;         // phase 2: this wave's sample
  const bool solver = wave < COL_S && n < p.N;
  int my_passes = 0;
  // element (sample, k) of a layer's input in LDS (see col_product)
  auto put = [&](int l, int k, float v) {
    const int c = k / KC, kk = k % KC, h = kk / EPL, s = (kk % EPL) / P, e = kk % P;
    T* d = (T*)(lds + p.lds_act[l]) + ((c * 8 + h * 4 + s) * COL_S + wave) * P + e;
    *d = Elem<T>::from_f32(v);
  };

  for (int blk = 0; blk < p.n_blocks; ++blk) {
    const int a = p.bounds ? p.bounds[blk] : blk * p.block;
    const int b = p.bounds ? p.bounds[blk + 1] : min(D, a + p.block);
    const int nb = b - a;
    // (units of degree a .. b-1: layer l's slots [u0, u0 + nu))
    int u0[L], nu[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int* cn = (const int*)(lds + p.lds_cnt[l]);
      u0[l] = __builtin_amdgcn_readfirstlane(cn[a]);
      nu[l] = __builtin_amdgcn_readfirstlane(cn[b]) - u0[l];
    }
    // requested now, used in phase 2
    float uval = 0.f, bias[L + 1];
    unsigned long long init = 0;
    if (solver) {
      if (lane < nb) uval = p.noise[(size_t)n * D + a + lane];
      if (!SEQ && p.x_init) init = __ballot(lane < nb && p.x_init[(size_t)n * D + a + min(lane, nb - 1)] != 0);
    }
#pragma unroll
    for (int l = 0; l <= L; ++l) {
      const int first = l < L ? u0[l < L ? l : 0] : a, cnt = l < L ? nu[l < L ? l : 0] : nb;
      bias[l] = solver && lane < cnt ? p.bias[l][first + lane] : 0.f;
    }

    // ---- phase 1
    static_for<L + 1>([&](auto LL) {
      constexpr int l = LL;
      const int row0 = l < L ? u0[l < L ? l : 0] : a, rows = l < L ? nu[l < L ? l : 0] : nb;
      const int k0 = l == 0 ? a : u0[l > 0 ? l - 1 : 0], n_k = l == 0 ? nb : nu[l > 0 ? l - 1 : 0];
      // (a chunk's first step holds the columns 0 .. EPL/2 - 1 of its two halves, the second one the rest)
      const int rem = k0 % KC, steps = 2 * (k0 / KC) + (rem == 0 ? 0 : rem <= EPL / 2 ? 1 : 2);
      const T* W = (const T*)p.W[l];
      const unsigned char* act = lds + p.lds_act[l];
      const int tiles = (rows + 15) >> 4;
      if (tiles > 2) {
        if (tiles == 3) col_product<T, 3>(W, p.k_chunks[l], act, row0, rows, steps, red, RED, l * COL_UNITS);
        else col_product<T, 4>(W, p.k_chunks[l], act, row0, rows, steps, red, RED, l * COL_UNITS);
      } else if (tiles > 0) {
        if (tiles == 1) col_product<T, 1>(W, p.k_chunks[l], act, row0, rows, steps, red, RED, l * COL_UNITS);
        else col_product<T, 2>(W, p.k_chunks[l], act, row0, rows, steps, red, RED, l * COL_UNITS);
      }
      col_stage<T>(W, p.k_chunks[l], row0, rows, k0, n_k, (float*)(lds + p.lds_w[l]), l < L ? COL_UNITS : COL_POS);
    });
    __syncthreads();

    // ---- phase 2
    if (solver) {
      float pre[L + 1];
#pragma unroll
      for (int l = 0; l <= L; ++l) {
        const int cnt = l < L ? nu[l < L ? l : 0] : nb;
        float v = 0.f;
        if (lane < cnt) {
          const float* src = red + (size_t)wave * RED + l * COL_UNITS + lane;
#pragma unroll
          for (int w = 0; w < COL_WAVES; ++w) v += src[(size_t)w * COL_S * RED];
        }
        pre[l] = v + bias[l];
      }
      const int out_col = lane & (COL_POS - 1);
      unsigned mask = 0;                            // bit j: the symbol of position a + j
      if (SEQ) {
        int off[L];                                 // lane j: the first slot of degree a + j, relative to u0
#pragma unroll
        for (int l = 0; l < L; ++l) off[l] = ((const int*)(lds + p.lds_cnt[l]))[min(a + lane, b)] - u0[l];
        for (int j = 0; j < nb; ++j) {
          // units of degree a + j have all their inputs: into the next layer, or the logits
#pragma unroll
          for (int l = 0; l < L; ++l) {
            const int s = __builtin_amdgcn_readlane(off[l], j), e = __builtin_amdgcn_readlane(off[l], j + 1);
            const float h = col_value(fmaxf(pre[l], 0.f), T{});
            pre[l + 1] = col_add_units((const float*)(lds + p.lds_w[l + 1]), l + 1 < L ? COL_UNITS : COL_POS,
                                       l + 1 < L ? lane : out_col, h, s, e, pre[l + 1]);
          }
          const unsigned drawn = (unsigned)__ballot(uval < bernoulli_probability(pre[L]));
          if ((drawn >> j) & 1u) {
            mask |= 1u << j;
            pre[0] += ((const float*)(lds + p.lds_w[0]))[j * COL_UNITS + lane];
          }
        }
      } else {
        const unsigned live = nb == 32 ? 0xffffffffu : (1u << nb) - 1u;
        mask = (unsigned)init & live;
        float base[L + 1];
#pragma unroll
        for (int l = 0; l <= L; ++l) base[l] = pre[l];
        auto unit = [&](int l) { return lane < nu[l] ? col_value(fmaxf(pre[l], 0.f), T{}) : 0.f; };
        auto hidden = [&]() {                       // pre[l] from the block's symbols
          pre[0] = base[0];
          for (unsigned mm = mask; mm;) {
            const int j = __builtin_ctz(mm);
            mm &= mm - 1;
            const int j2 = mm ? __builtin_ctz(mm) : j;
            const bool two = mm != 0;
            mm &= mm - 1;                           // (0 & anything stays 0)
            const float w0 = ((const float*)(lds + p.lds_w[0]))[j * COL_UNITS + lane];
            const float w1 = ((const float*)(lds + p.lds_w[0]))[j2 * COL_UNITS + lane];
            pre[0] += w0;
            if (two) pre[0] += w1;
          }
#pragma unroll
          for (int l = 0; l + 1 < L; ++l)
            pre[l + 1] = col_add_all((const float*)(lds + p.lds_w[l + 1]), COL_UNITS, lane, unit(l), (nu[l] + 7) & ~7, base[l + 1]);
        };
        int k = 0;
        bool changed = true;
        while (changed && k < nb) {
          hidden();
          const float z = col_add_all((const float*)(lds + p.lds_w[L]), COL_POS, out_col,
                                      unit(L - 1), (nu[L - 1] + 7) & ~7, base[L]);
          const unsigned drawn = (unsigned)__ballot(uval < bernoulli_probability(z)) & live;
          changed = drawn != mask;
          mask = drawn;
          ++k;
        }
        if (changed) hidden();                      // (the last allowed pass still changed symbols: the units follow)
        my_passes += k;
        if (lane == 0) block_passes_s[wave] = k;
      }
      // ---- the block is final
      if (lane < nb) {
        const unsigned bit = (mask >> lane) & 1u;
        p.x[(size_t)n * D + a + lane] = (uint8_t)bit;
        put(0, a + lane, (float)bit);
      }
#pragma unroll
      for (int l = 0; l < L; ++l)
        if (lane < nu[l]) put(l + 1, u0[l] + lane, fmaxf(pre[l], 0.f));
    } else if (!SEQ && wave < COL_S && lane == 0) {
      block_passes_s[wave] = 0;
    }
    __syncthreads();
    if (!SEQ && threadIdx.x == 0) {
      int most = 0;
      for (int i = 0; i < COL_S; ++i) most = max(most, block_passes_s[i]);
      lds[p.lds_passes + blk] = (unsigned char)most;     // (<= COL_POS)
    }
  }

  if (!SEQ) {
    if (wave < COL_S && lane == 0) {
      passes_s[wave] = solver ? (unsigned long long)my_passes : 0ull;
      if (solver) p.iters[n] = my_passes;
    }
    __syncthreads();
    // A block takes as many passes as its slowest sample of the whole batch.  (Returning atomics, each performed before the
    // barrier: the workgroup that sees the full count sees every contribution.)
    for (int b = threadIdx.x; b < p.n_blocks; b += NT_) {
      const int o = __hip_atomic_fetch_max(&p.block_passes[b], (int)lds[p.lds_passes + b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("" ::"v"(o));
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long sum = 0;
      for (int i = 0; i < COL_S; ++i) sum += passes_s[i];
      unsigned long long o = __hip_atomic_fetch_add(&p.ctr[1], sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("" ::"v"(o));
      o = __hip_atomic_fetch_add(&p.ctr[0], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last_s = o == (unsigned long long)gridDim.x - 1;
      all_passes_s = 0;
    }
    __syncthreads();
    if (last_s) {                                    // (uniform) report, and leave the counters at zero
      int mine = 0;
      for (int b = threadIdx.x; b < p.n_blocks; b += NT_) mine += __hip_atomic_exchange(&p.block_passes[b], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (mine) atomicAdd(&all_passes_s, mine);
      __syncthreads();
      if (threadIdx.x == 0) {
        const unsigned long long sum = __hip_atomic_exchange(&p.ctr[1], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&p.ctr[0], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&p.host[0], (unsigned long long)all_passes_s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&p.host[1], sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&p.host[2], p.call_id, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
      }
    }
  }
}

}  // namespace jm
