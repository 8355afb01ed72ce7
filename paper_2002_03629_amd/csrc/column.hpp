// Block-wise forward substitution in one launch: GS-Jacobi blocks and the lean sequential sampler of a Bernoulli MLP
// (gfx950 only).
//
// Hidden units are sorted by degree, so the network is block lower triangular in the positions: the units of degree
// a .. b-1 and the outputs of positions [a, b) need the inputs before a, the hidden units of degree < a -- all final
// once the positions before a are -- and one another.  A workgroup owns COL_S samples for the whole call and walks the
// blocks with two kinds of waves:
//   * producers multiply the block's rows of every layer with the final inputs (a contraction over up to two thousand
//     inputs: matrix instructions, weights streamed from L2, activations in LDS) and stage the weights between the block's
//     own units and positions in LDS.  All of it but the inputs that the block before makes final (the late steps: a few K
//     steps, their weights requested ahead) is done while the block before is being solved;
//   * solvers, one wave per sample: a lane owns one unit of every layer (and one position), its fp32 pre-activation in a
//     register; a value that becomes known is broadcast and multiplied into the lanes that see it.  Sequential sampling draws
//     one position after the other and adds what it changes; GS-Jacobi evaluates the block from its base sums pass by pass
//     until nothing changes.
// Two barriers a block (of LDS traffic only: no store is waited for): the block's sums are there / the block is final.  Every
// visible weight is read once per workgroup and call instead of once per pass, and nothing waits for another workgroup.
// What bounds it: the solvers' dependent instructions (0.25 us per position; a GS-Jacobi pass of 16 positions and 41 units a
// layer 0.8 us) and, on short blocks, the producers' round trips (about 1 us each for all 8 waves' loads: 64 bytes a clock).
// 784 positions, 2 x 2000 units, bf16, batch 128: blocks of 16 442 -> 276 us, sequential 578 -> 274 us against one kind of
// waves taking both turns.  Tried: 4 producers with twice the loads in flight (344 and 458 us), the weights of a coming block
// asked for ahead of its turn so that they are in L2 (305 and 318).
#pragma once

#include "kernels.hpp"

namespace jm {

constexpr int COL_S = 4;            // samples per workgroup: one per SIMD in phase 2, whose instruction issue bounds it
constexpr int COL_PRODUCERS = 8;    // waves that multiply, two per SIMD
constexpr int COL_WAVES = COL_S + COL_PRODUCERS;
constexpr int COL_UNITS = 64;       // units of one layer whose degree falls into a block, at most (one per lane)
constexpr int COL_POS = 32;         // positions of a block, at most
constexpr int COL_Q = 4;            // sequential sampling: units of a position and layer whose weights are read ahead
constexpr int COL_SEQ_UNITS = COL_UNITS - COL_Q;   // ... and units of a block of several positions, at most
constexpr int COL_MAX_L = 3;        // hidden layers

struct ColumnArgs {
  const void* W[COL_MAX_L + 1];
  const float* bias[COL_MAX_L + 1];
  const int* cnt_lt[COL_MAX_L];     // [D + 2] units of degree < t (1-based degrees)
  int k_chunks[COL_MAX_L + 1];
  int lds_act[COL_MAX_L + 1];       // byte offsets into dynamic LDS: input of layer l, COL_S samples
  int lds_w[COL_MAX_L + 1];         // staged weights of layer l, input-major (see ColStage)
  int lds_w_bytes;                  // distance of the second buffer of them; 0: there is only one
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
__device__ __forceinline__ float col_value(float v, bf16_t) { return (float)(__bf16)v; }   // as the layers store it (v is no NaN)

// A block: positions [a, a + nb), and layer l's units of the degrees a .. a + nb - 1 in slots [u0[l], u0[l] + nu[l]).
template <int L>
struct ColBlock {
  int a, nb, u0[L], nu[L];
  __device__ __forceinline__ int row0(int l) const { return l < L ? u0[l < L ? l : 0] : a; }      // rows of layer l
  __device__ __forceinline__ int rows(int l) const { return l < L ? nu[l < L ? l : 0] : nb; }
  __device__ __forceinline__ int k0(int l) const { return l == 0 ? a : u0[l > 0 ? l - 1 : 0]; }   // its first input of the block
  __device__ __forceinline__ int n_k(int l) const { return l == 0 ? nb : nu[l > 0 ? l - 1 : 0]; }
};

// How the weights between a block's own units and positions lie in LDS: words (input, row), the rows at the pitch of a
// wave's lanes that hold them.  Sequential sampling adds one input at a time and takes floats; GS-Jacobi adds all of them,
// bf16 weights two inputs to a word (one instruction for both): the inputs 2 m and 2 m + 1 of the layer, so a block's first
// word may begin with an input before it and its last end with one behind it, which are multiplied with 0.
template <typename T, bool SEQ>
struct ColStage {
  static constexpr bool PAIRS = sizeof(T) == 2 && !SEQ;
  static constexpr int PER = PAIRS ? 2 : 1;                        // inputs of a word
  static constexpr int P = 16 / (int)sizeof(T);
  static constexpr int word_rows(int inputs) { return PAIRS ? inputs / 2 + 1 : inputs; }
  static __device__ __host__ constexpr int bytes(int inputs, int pitch) { return word_rows(inputs) * pitch * 4; }
  // the piece of inputs k .. k + P - 1 of a layer whose inputs of the block start at k0 (uniform), for row `row`
  static __device__ __forceinline__ void store(unsigned char* ws, int inputs, int pitch, int k0, int k, int row, const uint4& v) {
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
    uint32_t* dst = (uint32_t*)ws + row;
    auto put = [&](int word, uint32_t bits) {
      if (word >= 0 && word < word_rows(inputs)) dst[word * pitch] = bits;
    };
#pragma unroll
    for (int e = 0; e < P; e += PER) {
      if constexpr (PAIRS) put((k >> 1) - (k0 >> 1) + e / 2, u[e / 2]);
      else if constexpr (sizeof(T) == 4) put(k - k0 + e, u[e]);
      else put(k - k0 + e, (e & 1) ? u[e / 2] & 0xffff0000u : u[e / 2] << 16);
    }
  }
};

// max(v, 0), 0 for a NaN like fmaxf (which the compiler precedes by a second instruction, for signalling NaNs)
__device__ __forceinline__ float col_relu(float v) {
  float r;
  asm("v_max_f32 %0, 0, %1" : "=v"(r) : "v"(v));
  return r;
}
// u < sigmoid(z) as z > log(u / (1 - u)): the right-hand side does not wait for z.  Rounded once or twice, it is nearer to the exact
// line than the other kernels' sigmoid, which is within 1e-6; a draw can only differ from theirs there.  At the ends as they
// decide: their sigmoid is 0 from about log(2^-126) down, which u = 0 is not below (a logit of -1e4 never draws 1); u < 0 is below
// any, u >= 1 and a NaN below none.
__device__ __forceinline__ float col_threshold(float u) {
  const float t = logf((u == 0.0f ? 0x1p-126f : u) / (1.0f - u));
  return u < 0.0f ? -__builtin_inff() : t;
}

// max(v, 0) in lanes whose `top` is infinity, 0 in those where it is 0
__device__ __forceinline__ float col_relu_below(float v, float top) {
  float r;
  asm("v_med3_f32 %0, %1, 0, %2" : "=v"(r) : "v"(v), "v"(top));
  return r;
}
__device__ __forceinline__ float col_lane(float h, int u) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(h), u));
}

// sum + w_u h_u over the n inputs of a staged layer; h_u sits in lane u of h, 0 in the lanes past the last one.  The words of
// a group go to four sums, added at the end: one sum alone is a chain of dependent instructions, twice as long.  Root mean
// square error against 64 bits in units of 2^-24 (values of unit variance, bf16 weights of a fan-in of 2000), 2 / 16 / 41 / 64 inputs:
// 0.21 / 0.54 / 0.75 / 0.85, with one chain of fmas 0.22 / 0.62 / 1.00 / 1.25.
// `odd`: whether the first input is the second of its word.  ColHeld keeps a column of words in registers where all passes of
// a block need it.
template <typename T, int U>      // U inputs at most
struct ColHeld {
  using Stage = ColStage<T, false>;
  static constexpr bool PAIRS = Stage::PAIRS;
  static constexpr int G = PAIRS ? 4 : 8;                          // words of a group
  static constexpr int GROUPS = U / Stage::PER / G;
  uint32_t w[GROUPS][G], last;
  static __device__ __forceinline__ int words(int n, bool odd) { return PAIRS ? (n + (odd ? 2 : 1)) >> 1 : n; }
  __device__ __forceinline__ void load(const uint32_t* ws, int pitch, int n_words) {
    static_for<GROUPS>([&](auto g) {
      if (G * g < n_words) static_for<G>([&](auto i) { w[g][i] = ws[(G * g + i) * pitch]; });
    });
    if (PAIRS && n_words > GROUPS * G) last = ws[GROUPS * G * pitch];
  }
  template <typename F>
  static __device__ __forceinline__ float add(float h, int n_words, bool odd, float sum, F&& word) {
    float part[4] = {sum, 0.f, 0.f, 0.f};
    if constexpr (PAIRS) {
      typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
      // lane 2 m: the inputs of word m, which sit in the lanes 2 m and 2 m + 1, or (odd) 2 m - 1 and 2 m
      const float below = __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(h), 0x138 /* wave_shr:1 */, 0xf, 0xf, true));
      const float above = __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(h), 0x130 /* wave_shl:1 */, 0xf, 0xf, true));
      const bf16x2 pair = {(__bf16)(odd ? below : h), (__bf16)(odd ? h : above)};
      const uint32_t bits = __builtin_bit_cast(uint32_t, pair);
      auto dot = [&](uint32_t hu, uint32_t wu, float& v) {
        v = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, hu), __builtin_bit_cast(bf16x2, wu), v, false);
      };
      static_for<GROUPS>([&](auto g) {
        if (G * g < n_words) {
          uint32_t hu[G];
          static_for<G>([&](auto i) { hu[i] = __builtin_amdgcn_readlane(bits, 2 * (G * g + i)); });
          static_for<G>([&](auto i) { dot(hu[i], word(g, i), part[i % 4]); });
        }
      });
      if (n_words > GROUPS * G)                                     // (U inputs, odd: the last one alone in its word)
        dot(__builtin_amdgcn_readlane(bits, U - 1) >> 16, word(std::integral_constant<int, GROUPS>{}, std::integral_constant<int, 0>{}), part[0]);
    } else {
      static_for<GROUPS>([&](auto g) {
        if (G * g < n_words) {
          float hu[G];
          static_for<G>([&](auto i) { hu[i] = col_lane(h, G * g + i); });
          static_for<G>([&](auto i) { part[i % 4] = fmaf(__uint_as_float(word(g, i)), hu[i], part[i % 4]); });
        }
      });
    }
    return (part[0] + part[1]) + (part[2] + part[3]);
  }
  __device__ __forceinline__ float add(float h, int n_words, bool odd, float sum) const {
    return add(h, n_words, odd, sum, [&](auto g, auto i) {
      if constexpr (g == GROUPS) return last;
      else return w[g][i];
    });
  }
  static __device__ __forceinline__ float add_from(const uint32_t* ws, int pitch, float h, int n_words, bool odd, float sum) {
    return add(h, n_words, odd, sum, [&](auto g, auto i) { return ws[(G * g + i) * pitch]; });
  }
};

// The producers' side of a block (see the head of this file): what they carry from the one barrier to the other.  A K
// step is half a chunk (64 bytes per row): lane (row r, quarter q) of a 16 x 16 tile holds piece (slot 2 (step % 2) +
// q / 2, half q % 2) of it.  Only COL_S of the 16 columns differ: lane r reads sample r % COL_S.
// (A chunk's first step holds the columns 0 .. EPL/2 - 1 of its two halves, the second one the rest.)
template <typename T, int L, bool SEQ>
struct ColProducer {
  static constexpr int EPL = Elem<T>::EPL, KC = 2 * EPL, P = 16 / (int)sizeof(T);
  // steps between the chunk in which the block before starts and the block: chunks of at most KC - 1 + COL_UNITS columns
  static_assert(2 * ((KC - 1 + COL_UNITS) / KC) + 2 <= COL_PRODUCERS, "one late step to a wave");
  static constexpr int FLIGHT = 18;                          // loads of a wave on their way at a time
  static constexpr bool CARRY = L <= 2;                      // registers to carry requested weights from one barrier to the next
  static constexpr int RED = COL_UNITS * L + COL_POS;
  static constexpr int tiles(int l) { return (l < L ? COL_UNITS : COL_POS) / 16; }
  static constexpr int pitch(int l) { return l < L ? COL_UNITS : COL_POS; }
  static constexpr int inputs(int l) { return l == 0 ? COL_POS : COL_UNITS; }
  static constexpr int pieces(int l) { return ((l == 0 ? COL_POS : COL_UNITS) + P - 2) / P + 1; }
  // staging: the first waves serve layer 0, which has half the pieces, the others a layer each (L = 1: 2 and 6 of them, L = 2: 2, 3
  // and 3, L = 3: 2 each)
  static constexpr int stage_first(int l) { return l == 0 ? 0 : 2 + (COL_PRODUCERS - 2) * (l - 1) / L; }
  static constexpr int stage_waves(int l) { return stage_first(l + 1) - stage_first(l); }
  static constexpr int stage_loads(int l) { return (pieces(l) + stage_waves(l) - 1) / stage_waves(l); }
  static constexpr int most(int a, int b) { return a > b ? a : b; }
  static constexpr int STAGE = most(stage_loads(0), most(stage_loads(1), stage_loads(L)));

  f32x4 acc[L + 1][4];
  uint4 late_w[L + 1][4];
  uint4 staged[STAGE];

  static __device__ __forceinline__ int steps_before(int k0) {     // steps that hold the columns below k0
    const int rem = k0 % KC;
    return 2 * (k0 / KC) + (rem == 0 ? 0 : rem <= EPL / 2 ? 1 : 2);
  }
  static __device__ __forceinline__ int steps_whole(int k0) { return 2 * (k0 / KC); }   // of chunks entirely below k0

  // byte offset of a row's pieces of this lane from the start of step 0 (32 bits are enough: LDS holds COL_S samples' inputs of
  // every layer, so a layer has less than 20480 inputs and rows)
  static __device__ __forceinline__ uint32_t row_pieces(int k_chunks, int row) {
    const int q = (threadIdx.x & 63) >> 4;
    return (uint32_t)(row >> 5) * (uint32_t)k_chunks * 4096u + (uint32_t)((((q >> 1) * 2 + (q & 1)) * 32 + (row & 31)) * 16);
  }
  // (activations: 16-byte piece (chunk, half, slot) of sample s at ((chunk * 8 + half * 4 + slot) * COL_S + s) * 16)
  static __device__ __forceinline__ uint4 act_piece(const unsigned char* act, int step) {
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    return *(const uint4*)(act + (((step >> 1) * 8 + (step & 1) * 2 + (q & 1) * 4 + (q >> 1)) * COL_S + (r & (COL_S - 1))) * 16);
  }

  __device__ __forceinline__ void clear() {
    static_for<L + 1>([&](auto LL) {
      static_for<tiles(LL)>([&](auto TT) { acc[LL][TT] = f32x4{0.f, 0.f, 0.f, 0.f}; });
    });
  }

  // steps [j, end) of NT row tiles of layer l
  template <int l, int NT>
  __device__ __forceinline__ void product(const ColumnArgs& p, const unsigned char* lds, const ColBlock<L>& b, int j, int end) {
    constexpr int G = NT >= 3 ? FLIGHT / NT : 16 / NT;
    uint32_t wp[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) wp[t] = row_pieces(p.k_chunks[l], b.row0(l) + min(16 * t + (int)(threadIdx.x & 15), b.rows(l) - 1));
    const unsigned char* act = lds + p.lds_act[l];
    // N steps from j on: all requested, then multiplied (steps past the end repeat the last one and are not multiplied)
    auto group = [&](auto N) {
      uint4 w[N][NT];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const unsigned char* step = (const unsigned char*)p.W[l] + (size_t)min(j + i, end - 1) * 2048;
#pragma unroll
        for (int t = 0; t < NT; ++t) w[i][t] = *(const uint4*)(step + wp[t]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (j + i < end) {
          const uint4 x = act_piece(act, j + i);
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[l][t] = col_mfma(w[i][t], x, acc[l][t], T{});
        }
    };
    while (j < end) {
      if (end - j > G / 2) {
        group(std::integral_constant<int, G>{});
        j += G;
      } else {
        group(std::integral_constant<int, G / 2>{});
        j += G / 2;
      }
    }
  }

  // The contribution of the whole chunks that are final before block `cur` to the rows of block `b`.  The waves are dealt
  // to the layers by the loads these take (a layer split over all waves would cost every wave a round trip to memory per
  // layer), a layer's waves split its steps.
  __device__ __forceinline__ void early(const ColumnArgs& p, const unsigned char* lds, const ColBlock<L>& b, const ColBlock<L>& cur,
                                        int pw) {
    int loads[L + 1], waves[L + 1], left = COL_PRODUCERS;
#pragma unroll
    for (int l = 0; l <= L; ++l) {
      loads[l] = ((b.rows(l) + 15) >> 4) * steps_whole(cur.k0(l));
      waves[l] = loads[l] > 0;
      left -= waves[l];
    }
    clear();
    if (left == COL_PRODUCERS) return;                         // (nothing is final yet)
    for (; left > 0; --left) {                                 // the next one to the layer with the most loads to a wave
      int most = 0, n = loads[0], d = waves[0];
#pragma unroll
      for (int l = 1; l <= L; ++l)
        if (loads[l] * max(d, 1) > n * max(waves[l], 1)) {
          most = l;
          n = loads[l];
          d = waves[l];
        }
#pragma unroll
      for (int l = 0; l <= L; ++l) waves[l] += l == most;
    }
    // this wave's layer, and its steps of it: [steps i / w, steps (i + 1) / w), rounded, for the i-th of its w <= 8 waves.  (One wave's
    // end and the next one's start have to be the same number: an explicit fma, so that they are one operation on one set of
    // values however the two are compiled.  In whole numbers the call of 784 / 2 x 2000, blocks of 16, took 278.5 us for 276.)
    int layer = 0, i = pw;
#pragma unroll
    for (int l = 0; l < L; ++l)
      if (layer == l && i >= waves[l]) {
        i -= waves[l];
        layer = l + 1;
      }
    static_for<L + 1>([&](auto LL) {
      constexpr int l = LL;
      if (layer != l) return;                                  // (one layer to a wave: its sums alone take registers)
      clear();
      const int steps = steps_whole(cur.k0(l)), n = (b.rows(l) + 15) >> 4;
      const float per = (float)steps * __builtin_amdgcn_rcpf((float)max(waves[l], 1));
      auto cut = [&](int k) { return k >= waves[l] ? steps : (int)__builtin_fmaf(per, (float)k, 0.5f); };
      const int j = cut(i), end = cut(i + 1);
      if (n == 1) product<l, 1>(p, lds, b, j, end);
      else if (n == 2) product<l, 2>(p, lds, b, j, end);
      if constexpr (l < L) {
        if (n == 3) product<l, 3>(p, lds, b, j, end);
        else if (n == 4) product<l, 4>(p, lds, b, j, end);
      }
    });
  }

  // (which late step of a layer is a wave's: the layers' steps, up to four in bf16, lie beside one another)
  static __device__ __forceinline__ int late_step(int l, int pw) { return (pw - 3 * l) & (COL_PRODUCERS - 1); }
  // The rest of the inputs before block b, those that block `cur` makes final: requested ahead of the barrier ...
  __device__ __forceinline__ void late_request(const ColumnArgs& p, const ColBlock<L>& b, const ColBlock<L>& cur, int pw) {
    static_for<L + 1>([&](auto LL) {
      constexpr int l = LL;
      const int j = steps_whole(cur.k0(l)) + late_step(l, pw);
      static_for<tiles(l)>([&](auto TT) { late_w[l][TT] = make_uint4(0, 0, 0, 0); });   // (or the old values would count as live)
      if (b.rows(l) > 0 && j < steps_before(b.k0(l))) {
        static_for<tiles(l)>([&](auto TT) {
          constexpr int t = TT;
          if (16 * t < b.rows(l)) {
            const uint32_t wp = row_pieces(p.k_chunks[l], b.row0(l) + min(16 * t + (int)(threadIdx.x & 15), b.rows(l) - 1));
            late_w[l][t] = *(const uint4*)((const unsigned char*)p.W[l] + (size_t)j * 2048 + wp);
          }
        });
      }
    });
  }
  // ... and multiplied behind it; then all sums go to red[wave][sample][row].
  __device__ __forceinline__ void late_product(const ColumnArgs& p, const unsigned char* lds, const ColBlock<L>& b, const ColBlock<L>& cur,
                                               float* red, int pw) {
    static_for<L + 1>([&](auto LL) {
      constexpr int l = LL;
      const int j = steps_whole(cur.k0(l)) + late_step(l, pw), end = steps_before(b.k0(l));
      if (b.rows(l) > 0 && j < end) {
        const uint4 x = act_piece(lds + p.lds_act[l], j);
        static_for<tiles(l)>([&](auto TT) { acc[l][TT] = col_mfma(late_w[l][TT], x, acc[l][TT], T{}); });
      }
    });
    // acc[l][t][i]: row 16 t + 4 q + i, sample r
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    if (r < COL_S) {
      float* dst = red + (size_t)(pw * COL_S + r) * RED + 4 * q;
      static_for<L + 1>([&](auto LL) {
        static_for<tiles(LL)>([&](auto TT) { *(f32x4*)(dst + LL * COL_UNITS + 16 * TT) = acc[LL][TT]; });
      });
    }
  }

  // The weights between block b's own units and positions: requested, and written to LDS as ColStage has them.  A wave takes
  // whole pieces of one layer, a lane a row (rows past the last repeat it).
  template <typename F>
  __device__ __forceinline__ void stage_each(const ColBlock<L>& b, int pw, F&& piece_of) {
    static_for<L + 1>([&](auto LL) {
      constexpr int l = LL;
      if (pw < stage_first(l) || pw >= stage_first(l + 1) || b.rows(l) == 0) return;
      const int p0 = b.k0(l) / P + pw - stage_first(l), p1 = (b.k0(l) + b.n_k(l) + P - 1) / P;
      static_for<stage_loads(l)>([&](auto I) {
        if (p0 + I * stage_waves(l) < p1) piece_of(LL, I, p0 + I * stage_waves(l));
      });
    });
  }
  __device__ __forceinline__ void stage_request(const ColumnArgs& p, const ColBlock<L>& b, int pw) {
    static_for<STAGE>([&](auto I) { staged[I] = make_uint4(0, 0, 0, 0); });
    stage_each(b, pw, [&](auto LL, auto I, int piece) {
      constexpr int l = LL;
      const int g = b.row0(l) + min((int)(threadIdx.x & 63), b.rows(l) - 1);
      const uint32_t row = (uint32_t)(g >> 5) * (uint32_t)p.k_chunks[l] * 4096u + (uint32_t)(g & 31) * 16u;
      const int k = piece * P, c = k / KC, kk = k % KC, h = kk / EPL, s = (kk % EPL) / P;
      staged[I] = *(const uint4*)((const unsigned char*)p.W[l] + ((size_t)c * 4096 + (s * 2 + h) * 512) + row);
    });
  }
  __device__ __forceinline__ void stage_store(const ColumnArgs& p, unsigned char* lds, const ColBlock<L>& b, int buffer, int pw) {
    const int lane = threadIdx.x & 63;
    stage_each(b, pw, [&](auto LL, auto I, int piece) {
      constexpr int l = LL;
      if (pitch(l) == 64 || lane < pitch(l))
        ColStage<T, SEQ>::store(lds + p.lds_w[l] + buffer * p.lds_w_bytes, inputs(l), pitch(l), b.k0(l), piece * P, lane, staged[I]);
    });
  }
};

template <typename T, int L, bool SEQ>
__global__ __launch_bounds__(COL_WAVES * 64) void column_sampler_kernel(ColumnArgs p) {
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ unsigned long long passes_s[COL_S];
  __shared__ int block_passes_s[COL_S], all_passes_s, last_s;
  using Producer = ColProducer<T, L, SEQ>;
  constexpr int NT_ = COL_WAVES * 64;
  constexpr int P = 16 / (int)sizeof(T);
  constexpr int RED = Producer::RED;               // rows of a block over all layers
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int D = p.D;
  for (int i = threadIdx.x; i < p.lds_clear / 16; i += NT_) ((uint4*)lds)[i] = make_uint4(0, 0, 0, 0);
#pragma unroll
  for (int l = 0; l < L; ++l)
    for (int i = threadIdx.x; i < D + 2; i += NT_) ((int*)(lds + p.lds_cnt[l]))[i] = p.cnt_lt[l][i];
  __syncthreads();

  float* red = (float*)(lds + p.lds_red);
  const bool late_stage = p.lds_w_bytes == 0;      // one buffer of staged weights: written between the solvers' turns
  auto block_at = [&](int blk) {
    ColBlock<L> b;
    b.a = p.bounds ? p.bounds[blk] : blk * p.block;
    b.nb = (p.bounds ? p.bounds[blk + 1] : min(D, b.a + p.block)) - b.a;
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int* cn = (const int*)(lds + p.lds_cnt[l]);
      b.u0[l] = __builtin_amdgcn_readfirstlane(cn[b.a]);
      b.nu[l] = __builtin_amdgcn_readfirstlane(cn[b.a + b.nb]) - b.u0[l];
    }
    return b;
  };

  int my_passes = 0;
  const int n = blockIdx.x * COL_S + wave;         // solvers: this wave's sample
  const bool solver = wave < COL_S && n < p.N;
  if (wave >= COL_S) {
    // ---- producers: two barriers per block, like the solvers below
    const int pw = wave - COL_S;
    Producer pr;
    ColBlock<L> b = block_at(0), cur = b;          // (nothing lies before the first block)
    constexpr bool CARRY = Producer::CARRY;
    pr.stage_request(p, b, pw);
    pr.stage_store(p, lds, b, 0, pw);
    pr.clear();
    if (CARRY && !late_stage && p.n_blocks > 1) pr.stage_request(p, block_at(1), pw);
    for (int blk = 0; blk < p.n_blocks; ++blk) {
      if (late_stage && blk > 0) {
        if (!CARRY) pr.stage_request(p, b, pw);
        pr.stage_store(p, lds, b, 0, pw);
      }
      if (!CARRY) pr.late_request(p, b, cur, pw);
      pr.late_product(p, lds, b, cur, red, pw);
      lds_barrier();
      if (blk + 1 < p.n_blocks) {
        cur = b;
        b = block_at(blk + 1);
        if (!CARRY && !late_stage) pr.stage_request(p, b, pw);
        if (!late_stage) pr.stage_store(p, lds, b, (blk + 1) & 1, pw);
        pr.early(p, lds, b, cur, pw);
        if (CARRY) {
          pr.late_request(p, b, cur, pw);
          if (late_stage) pr.stage_request(p, b, pw);
          else if (blk + 2 < p.n_blocks) pr.stage_request(p, block_at(blk + 2), pw);
        }
      }
      lds_barrier();
    }
  } else {
    // ---- solvers
    __builtin_amdgcn_s_setprio(2);                 // (a SIMD's other wave, a producer, is not in a hurry)
    // element (sample, k) of a layer's input in LDS (see ColProducer::act_piece: pieces of P elements in order of k)
    auto put = [&](int l, unsigned k, float v) {
      *(T*)(lds + p.lds_act[l] + ((k / P) * COL_S + wave) * 16 + (k % P) * sizeof(T)) = Elem<T>::from_f32(v);
    };
    // a block's noise, biases and initial symbols, requested a block ahead
    ColBlock<L> b = block_at(0);
    float uval = 0.f, bias[L + 1];
    unsigned char init = 0;
    auto request = [&]() {
      uval = 0.f;
      init = 0;
#pragma unroll
      for (int l = 0; l <= L; ++l) bias[l] = 0.f;
      if (solver) {
        if (lane < b.nb) uval = p.noise[(size_t)n * D + b.a + lane];
        if (!SEQ && p.x_init && lane < b.nb) init = p.x_init[(size_t)n * D + b.a + lane];
#pragma unroll
        for (int l = 0; l <= L; ++l)
          if (lane < b.rows(l)) bias[l] = p.bias[l][b.row0(l) + lane];
      }
    };
    request();
    for (int blk = 0; blk < p.n_blocks; ++blk) {
      lds_barrier();
      if (solver) {
        const ColBlock<L> c = b;
        const int nb = c.nb;
        const float threshold = col_threshold(uval);
        const bool init_here = init != 0;
        float pre[L + 1];
#pragma unroll
        for (int l = 0; l <= L; ++l) {
          float v = 0.f;
          const float* src = red + (size_t)wave * RED + l * COL_UNITS + min(lane, max(c.rows(l) - 1, 0));
#pragma unroll
          for (int w = 0; w < COL_PRODUCERS; ++w) v += src[w * COL_S * RED];
          pre[l] = (lane < c.rows(l) ? v : 0.f) + bias[l];
        }
        if (blk + 1 < p.n_blocks) {
          b = block_at(blk + 1);
          request();
        }
        const int out_col = lane & (COL_POS - 1);
        const int buffer = (blk & 1) * p.lds_w_bytes;
        // this lane's column of the staged weights of layer l
        auto staged = [&](int l) { return (const uint32_t*)(lds + p.lds_w[l] + buffer) + (l < L ? lane : out_col); };
        unsigned mask;                              // bit j: the symbol of position a + j
        if constexpr (SEQ) {
          // lane j: the first slot of degree a + j, relative to u0
          int off[L];
#pragma unroll
          for (int l = 0; l < L; ++l) off[l] = ((const int*)(lds + p.lds_cnt[l]))[min(c.a + lane, c.a + nb)] - c.u0[l];
          // A position's weights -- of its units' first Q in every layer, and of its symbol -- are read from LDS while the
          // position before is worked on.  Rows past its last unit are read as well (whatever lies there is finite: staged
          // weights, sums, zeros) and multiplied with 0; s + Q <= COL_UNITS, see COL_SEQ_UNITS.
          constexpr int Q = COL_Q;
          struct Ahead {
            float w[L][Q], symbol, top[L];
            int s[L], e[L];
          };
          auto fetch = [&](int j) {
            Ahead f;
#pragma unroll
            for (int l = 0; l < L; ++l) {
              f.s[l] = __builtin_amdgcn_readlane(off[l], j);
              f.e[l] = __builtin_amdgcn_readlane(off[l], j + 1);
              f.top[l] = lane < f.e[l] ? __builtin_inff() : 0.f;
              const float* src = (const float*)staged(l + 1) + f.s[l] * Producer::pitch(l + 1);
#pragma unroll
              for (int i = 0; i < Q; ++i) f.w[l][i] = src[i * Producer::pitch(l + 1)];
            }
            f.symbol = ((const float*)staged(0))[j * COL_UNITS];
            return f;
          };
          auto step = [&](int j, const Ahead& f) {
            // units of degree a + j have all their inputs: into the next layer, or the logits
#pragma unroll
            for (int l = 0; l < L; ++l) {
              const float h = col_value(col_relu_below(pre[l], f.top[l]), T{});
              float hu[Q];
#pragma unroll
              for (int i = 0; i < Q; ++i) hu[i] = col_lane(h, f.s[l] + i);
#pragma unroll
              for (int i = 0; i < Q; ++i) pre[l + 1] = fmaf(f.w[l][i], hu[i], pre[l + 1]);
              for (int u = f.s[l] + Q; u < f.e[l]; u += Q) {
                const float* src = (const float*)staged(l + 1) + u * Producer::pitch(l + 1);
                float w[Q];
#pragma unroll
                for (int i = 0; i < Q; ++i) w[i] = src[i * Producer::pitch(l + 1)];
                // (only a block of one position has units past COL_SEQ_UNITS: the wave's lanes would start over)
                if (u + Q <= COL_UNITS) {
#pragma unroll
                  for (int i = 0; i < Q; ++i) pre[l + 1] = fmaf(w[i], col_lane(h, u + i), pre[l + 1]);
                } else {
#pragma unroll
                  for (int i = 0; i < Q; ++i)
                    if (u + i < f.e[l]) pre[l + 1] = fmaf(w[i], col_lane(h, u + i), pre[l + 1]);
                }
              }
            }
            const unsigned long long drawn = __ballot(pre[L] > threshold);
            pre[0] += (drawn >> j) & 1ull ? f.symbol : 0.f;
          };
          Ahead f0 = fetch(0);
          for (int j = 0;;) {
            const Ahead f1 = fetch(j + 1);
            step(j, f0);
            if (++j == nb) break;
            f0 = fetch(j + 1);
            step(j, f1);
            if (++j == nb) break;
          }
          // (a position's logit stands after its step: later units are no input of it, their weights are zero)
          mask = (unsigned)__ballot(pre[L] > threshold);
        } else {
          const unsigned live = nb == 32 ? 0xffffffffu : (1u << nb) - 1u;
          mask = (unsigned)__ballot(init_here) & live;
          float base[L + 1];
#pragma unroll
          for (int l = 0; l <= L; ++l) base[l] = pre[l];
          // what all passes of the block read stays in registers, as far as they go
          constexpr bool HELD = L <= (sizeof(T) == 2 ? 3 : 1);
          ColHeld<T, COL_POS> w_symbol;
          ColHeld<T, COL_UNITS> w[HELD ? L : 1];
          auto words = [&](int l) { return ColHeld<T, COL_UNITS>::words(c.n_k(l), c.k0(l) & 1); };
          w_symbol.load(staged(0), COL_UNITS, words(0));
          if constexpr (HELD) static_for<L>([&](auto LL) { w[LL].load(staged(LL + 1), Producer::pitch(LL + 1), words(LL + 1)); });
          auto add_units = [&](auto LL) {             // layer l + 1 from the units of layer l
            constexpr int l = LL;
            const float h = lane < c.nu[l] ? col_relu(pre[l]) : 0.f;
            if constexpr (HELD) return w[l].add(h, words(l + 1), c.k0(l + 1) & 1, base[l + 1]);
            else return ColHeld<T, COL_UNITS>::add_from(staged(l + 1), Producer::pitch(l + 1), h, words(l + 1), false, base[l + 1]);
          };
          auto hidden = [&]() {                       // pre[l] from the block's symbols
            pre[0] = w_symbol.add(lane < nb && ((mask >> (lane & 31)) & 1u) ? 1.f : 0.f, words(0), c.a & 1, base[0]);
            static_for<L - 1>([&](auto LL) { pre[LL + 1] = add_units(LL); });
          };
          int k = 0;
          bool changed = true;
          while (changed && k < nb) {
            hidden();
            const float z = add_units(std::integral_constant<int, L - 1>{});
            const unsigned drawn = (unsigned)__ballot(z > threshold) & live;
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
          p.x[(size_t)n * D + c.a + lane] = (uint8_t)bit;
          put(0, c.a + lane, (float)bit);
        }
#pragma unroll
        for (int l = 0; l < L; ++l)
          if (lane < c.nu[l]) put(l + 1, c.u0[l] + lane, fmaxf(pre[l], 0.f));
      } else if (!SEQ && lane == 0) {
        block_passes_s[wave] = 0;
      }
      lds_barrier();
      if (!SEQ && threadIdx.x == 0) {
        int most = 0;
        for (int i = 0; i < COL_S; ++i) most = max(most, block_passes_s[i]);
        lds[p.lds_passes + blk] = (unsigned char)most;     // (<= COL_POS)
      }
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
