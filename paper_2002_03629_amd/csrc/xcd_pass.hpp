// A whole Jacobi call on up to 256 samples in one launch, every XCD on its own eighth of the batch (gfx950 only).
//
// Per-layer launches cost 4 to 6 us each however little a layer has to do at such batches: the kernel boundary, then a
// chain of memory round trips (list, bounds and bias; weights and activations; the stop test).  Here the eight XCDs share
// nothing.  An XCD has at most 32 samples, one row tile, and 32 workgroups, one per compute unit; a workgroup keeps the same
// one or two unit tiles of every layer for the whole call, so whatever does not depend on the pass is read once -- bounds and
// biases into LDS, noise, symbols or states of its positions into registers -- and the weights of its next tiles are on
// their way while it waits for the others.  A layer is then: activations from L2, matrix instructions, partial sums through
// LDS, activations to L2, barrier.  No list is made: a sample that has stopped keeps its row, and is no longer redrawn.
// The stop test travels with the barrier: a workgroup's flag carries the rows it changed.
// Sums are taken in compute_tile's order (K chunks dealt to the waves, parts added in wave order), so states are those of the
// per-layer launches bit for bit.
// What bounds it: 2.3 us a layer (784 / 2 x 512 real, batch 100: activations and products 0.5, parts through LDS 0.3, epilogue
// 0.35, stores performed 0.1, barrier 1.1, of which the first poll waits for the weights requested ahead; polling before
// requesting moved 0.2 us from there to 0.45 us ahead of the sums).  That call 195 -> 102 us; 64 / 256 fp32, batch 16: 52 -> 38 us,
// half of which is the launch and the host's wait for the report.  Waiting is bounded and the grid drains if workgroups are not placed as assumed, as in xcd_sampler_kernel.
#pragma once

#include "kernels.hpp"

namespace jm {

constexpr int XP_GROUP = 32;             // workgroups of an XCD: one per compute unit
constexpr int XP_ROWS = TILE;            // samples of an XCD
constexpr int XP_MAX_TILES = 2 * XP_GROUP;   // unit tiles of a layer
constexpr int XP_B = 4, XP_A = 2;        // K chunks of a wave and tile whose weights are requested ahead: of the tile with the
                                         // longer prefix, and of the shorter one
constexpr int XP_VISIBLE = 24 << 20, XP_VISIBLE_FEW = 10 << 20;   // bytes of visible weights up to which it pays, and on batches below
constexpr int XP_FEW = 64;                                        // this (see run_xcd_pass)
constexpr int XP_PITCH = TILE + 2;

struct XcdPassArgs {
  PersistLayer layer[PERSIST_MAX_LAYERS];
  int L;                 // hidden layers; layer[L] is the output layer
  void* enc;
  int enc_chunks;
  unsigned row_bytes[PERSIST_MAX_LAYERS];   // bytes of the call's rows (whole tiles) in the buffer that layer l reads
  const float* noise;
  const void* x_init;    // symbols or states, NULL: zeros
  void* x;
  float eps;             // real states
  int N, D;
  int cap;               // pass limit (<= D)
  int flag_unconverged;
  int zero_start;        // started from zeros: the first pass's first layer is ReLU(bias)
  int* iters;            // [N]
  unsigned long long* slots;   // [XCDS][XP_GROUP] (barrier number, rows changed in the last output layer)
  unsigned* words;       // [XCDS][32]: [0] registered workgroups, [16] where the last call stopped counting barriers
  unsigned reg_base;
  int* flags;            // 2, 4: backed out
  unsigned spin_limit;
  int call_id;
  int* host_report;      // see PersistArgs
};

__device__ __forceinline__ int xp_or16(int v) {      // OR over a row of 16 lanes
  v |= __builtin_amdgcn_mov_dpp(v, 0x128 /* row_ror:8 */, 0xf, 0xf, true);
  v |= __builtin_amdgcn_mov_dpp(v, 0x124 /* row_ror:4 */, 0xf, 0xf, true);
  v |= __builtin_amdgcn_mov_dpp(v, 0x122 /* row_ror:2 */, 0xf, 0xf, true);
  v |= __builtin_amdgcn_mov_dpp(v, 0x121 /* row_ror:1 */, 0xf, 0xf, true);
  return v;
}

// 16 bytes that another compute unit of this XCD may have written: past this unit's L1 (sc1)
__device__ __forceinline__ uint4 xp_load16(__amdgpu_buffer_rsrc_t buf, unsigned offset) {
  typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
  const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(buf, (int)offset, 0, 16 /* sc1 */);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// (second launch bound: waves per SIMD, i.e. one workgroup per compute unit and up to 256 registers)
template <typename T, bool REAL>
__global__ __launch_bounds__(NW * 64, 2) void xcd_pass_kernel(XcdPassArgs p) {
  __shared__ float part[2][NW][TILE][XP_PITCH];
  __shared__ float bias_s[PERSIST_MAX_LAYERS][2][TILE];
  __shared__ int chunks_s[PERSIST_MAX_LAYERS][2];
  __shared__ int changed_s[NW];
  __shared__ int xcc_s, rank_s, ok_s, active_s;
  constexpr int NT = NW * 64;
  constexpr int KC = 2 * Elem<T>::EPL;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, h = lane >> 5;

  // ---- which XCD, and which of its workgroups (see xcd_sampler_kernel)
  if (threadIdx.x == 0) {
    unsigned id;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(id));
    id &= 0xf;
    xcc_s = (int)id;
    rank_s = id < XCDS ? (int)(__hip_atomic_fetch_add(p.words + (size_t)id * 32, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) -
                               p.reg_base)
                       : XP_GROUP;
  }
  __syncthreads();
  const int group = __builtin_amdgcn_readfirstlane(xcc_s), rank = __builtin_amdgcn_readfirstlane(rank_s);
  if (group >= XCDS || rank < 0 || rank >= XP_GROUP) {
    if (threadIdx.x == 0) {
      __hip_atomic_fetch_or(p.flags, 4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_or(p.host_report + 64, 4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return;
  }
  const int D = p.D, L = p.L;
  const int per = (p.N + XCDS - 1) / XCDS;               // <= XP_ROWS (host)
  const int first = group * per, count = max(0, min(per, p.N - first));
  int* report = p.host_report + group * 8;
  if (count == 0) {                                      // (barriers are per XCD: nobody waits for this one)
    if (rank == 0 && threadIdx.x == 0) {
      for (int i = 0; i < 5; ++i) __hip_atomic_store(report + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(report + 5, p.call_id, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return;
  }
  unsigned long long* slots = p.slots + (size_t)group * XP_GROUP;
  unsigned* epoch_word = p.words + (size_t)group * 32 + 16;
  unsigned epoch = *epoch_word;

  // ---- this workgroup's tiles: `rank`, and in layers of more than 32 tiles the one as far from the other end (K extents grow
  // with the unit, so the two together are about as long for every workgroup).  Tile 1 is the longer one; -1: none.
  auto tile_of = [&](int l, int which) {
    const int n = p.layer[l].n_tiles, far = n - 1 - rank;
    const bool two = far >= XP_GROUP;
    return which ? (two ? far : rank < n ? rank : -1) : (two ? rank : -1);
  };
  for (int l = 0; l <= L; ++l) {
    if (threadIdx.x < 2 * TILE) {
      const int which = threadIdx.x >> 5, c = threadIdx.x & 31, t = tile_of(l, which);
      bias_s[l][which][c] = t >= 0 ? p.layer[l].bias[t * TILE + c] : 0.f;
      if (c == 0) chunks_s[l][which] = t >= 0 ? (p.layer[l].tile_kend[t] + KC - 1) / KC : 0;
    }
  }

  // ---- the epilogue's share: row tid / 16, columns 2 (tid % 16) and the one behind it, of either tile
  const int e_row = threadIdx.x >> 4, e_col = 2 * (threadIdx.x & 15);
  const int e_sample = first + min(e_row, count - 1);
  constexpr int P_ = REAL ? 1 : 2;                       // positions of a thread and tile
  int pos[2];                                            // the first of them
  float noise[2][P_], state[2][P_];                      // (symbols as 0 / 1)
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const int t = tile_of(L, w);
    pos[w] = t < 0 ? D : REAL ? (t * TILE + e_col) >> 1 : t * TILE + e_col;
#pragma unroll
    for (int j = 0; j < P_; ++j) {
      noise[w][j] = state[w][j] = 0.f;
      if (pos[w] + j < D) {
        const size_t i = (size_t)e_sample * D + pos[w] + j;
        noise[w][j] = p.noise[i];
        if (p.x_init) state[w][j] = REAL ? ((const float*)p.x_init)[i] : (float)((const uint8_t*)p.x_init)[i];
      }
    }
  }
  // the network's input: x_init or zeros
  for (size_t i = (size_t)rank * NT + threadIdx.x; i < (size_t)count * D; i += (size_t)XP_GROUP * NT) {
    const int n = first + (int)(i / D), t = (int)(i % D);
    float v = 0.f;
    if (p.x_init) v = REAL ? ((const float*)p.x_init)[(size_t)n * D + t] : (float)((const uint8_t*)p.x_init)[(size_t)n * D + t];
    ((T*)p.enc)[frag_offset<T>(n, t, p.enc_chunks)] = Elem<T>::from_f32(v);
  }

  // ---- weights requested ahead of a layer
  uint4 wa[XP_A][4], wb[XP_B][4];
  const unsigned char *Wa = nullptr, *Wb = nullptr;      // (uniform; a lane's 16 bytes behind them)
  const unsigned lane16 = lane * 16;
  auto weight = [&](const unsigned char* W, int i, int s) { return *(const uint4*)(W + (size_t)i * (NW * 4096) + s * 1024 + lane16); };
  int n_a = 0, n_b = 0;                                  // this wave's K chunks (wave, wave + NW, ...) of the two tiles
  auto request = [&](int l) {
    const PersistLayer& ly = p.layer[l];
    const int ta = tile_of(l, 0), tb = tile_of(l, 1);
    n_a = (__builtin_amdgcn_readfirstlane(chunks_s[l][0]) - wave + NW - 1) / NW;
    n_b = (__builtin_amdgcn_readfirstlane(chunks_s[l][1]) - wave + NW - 1) / NW;
    Wa = (const unsigned char*)ly.W + ((size_t)max(ta, 0) * ly.k_chunks + wave) * 4096;
    Wb = (const unsigned char*)ly.W + ((size_t)max(tb, 0) * ly.k_chunks + wave) * 4096;
#pragma unroll
    for (int i = 0; i < XP_B; ++i)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        wb[i][s] = make_uint4(0, 0, 0, 0);
        if (i < n_b) wb[i][s] = weight(Wb, i, s);
      }
#pragma unroll
    for (int i = 0; i < XP_A; ++i)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        wa[i][s] = make_uint4(0, 0, 0, 0);
        if (i < n_a) wa[i][s] = weight(Wa, i, s);
      }
  };
  // ---- barrier among the XCD's workgroups: stores performed, flags, all flags seen; returns the rows that any of them
  // changed in the last output layer (in active_s), false when the wait ran out.  `next`: the layer behind it.  A wait that runs
  // out behind an output layer ends the call like a last pass (no rows changed): the others may have seen the barrier complete, it
  // may be the call's last one, after which the call is served, and then this workgroup's share of the result has to be there.
  // (Where it is not, the back-out flag has reached the host before any report of this workgroup.)
  int my_changed = 0;                                    // wave 0: the rows this workgroup changed
  auto barrier = [&](int next, bool output) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    epoch += 1;
    if (wave == 0) {
      if (output) {
        my_changed = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) my_changed |= changed_s[w];
      }
      if (lane == 0)
        __hip_atomic_store(slots + rank, (unsigned long long)(unsigned)my_changed << 32 | epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    request(next);
    if (wave == 0) {
      int ok = 1;
      unsigned spins = 0;
      unsigned long long v;
      for (;;) {
        v = __hip_atomic_load(slots + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__all((int)((unsigned)v - epoch) >= 0)) break;
        if (++spins > p.spin_limit ||
            ((spins & 255) == 0 && (__hip_atomic_load(p.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 6))) {
          if (lane == 0) {
            __hip_atomic_fetch_or(p.flags, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_or(p.host_report + 64, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          }
          ok = 0;
          break;
        }
      }
      // (read outside the branch: the last OR would be done for its one lane only)
      const int all = xp_or16((int)(v >> 32)), rows = __builtin_amdgcn_readlane(all, 0) | __builtin_amdgcn_readlane(all, 16);
      if (lane == 0) {
        ok_s = ok | (int)output;
        active_s = ok ? rows : 0;
      }
    }
    lds_barrier();
    return ok_s != 0;
  };

  // ---- one layer: this wave's share of the products into `part`
  auto product = [&](int l) {
    const PersistLayer& ly = p.layer[l];
    const void* A = l == 0 ? p.enc : p.layer[l - 1].out;
    const __amdgpu_buffer_rsrc_t buf = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, (int)p.row_bytes[l], 0x00027000);
    const int sample = first + min(r, count - 1);
    const unsigned base = ((unsigned)(sample >> 5) * (unsigned)ly.k_chunks * 256u + (unsigned)(h * 32 + (sample & 31)) + (unsigned)wave * 256u) * 16u;
    f32x16 acc_a, acc_b;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc_a[i] = acc_b[i] = 0.f;
    auto load = [&](int i, uint4 (&av)[4]) {
#pragma unroll
      for (int s = 0; s < 4; ++s) av[s] = xp_load16(buf, base + (unsigned)(i * NW) * 4096u + (unsigned)s * 1024u);
    };
    {
      const int n = max(n_a, n_b);
      uint4 av[XP_B][4];
#pragma unroll
      for (int i = 0; i < XP_B; ++i)
        if (i < n) load(i, av[i]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < XP_B; ++i) {
        if (i < n_b) mfma_chunk<T>(av[i], wb[i], acc_b);
        if (i < XP_A && i < n_a) mfma_chunk<T>(av[i], wa[i < XP_A ? i : 0], acc_a);
      }
    }
    // chunks not requested ahead (fp32; prefixes that are not complementary)
    auto rest = [&](int from, int n, const unsigned char* W, f32x16& acc) {
#pragma clang loop unroll(disable)
      for (int i = from; i < n; ++i) {
        uint4 av[4], w[4];
        load(i, av);
#pragma unroll
        for (int s = 0; s < 4; ++s) w[s] = weight(W, i, s);
        mfma_chunk<T>(av, w, acc);
      }
    };
    rest(XP_B, n_b, Wb, acc_b);
    rest(XP_A, n_a, Wa, acc_a);
    // acc[i]: row 8 (i / 4) + 4 h + i % 4 (sample), column r (unit)
#pragma unroll
    for (int i = 0; i < 16; ++i) part[1][wave][(i >> 2) * 8 + h * 4 + (i & 3)][r] = acc_b[i];
    if (tile_of(l, 0) >= 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) part[0][wave][(i >> 2) * 8 + h * 4 + (i & 3)][r] = acc_a[i];
    }
    lds_barrier();
  };
  auto sum = [&](int l, int which, float& v0, float& v1, bool none = false) {
    v0 = v1 = 0.f;
    if (!none) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float2 q = *(const float2*)&part[which][w][e_row][e_col];
        v0 += q.x;
        v1 += q.y;
      }
    }
    const float2 b = *(const float2*)&bias_s[l][which][e_col];
    v0 += b.x;
    v1 += b.y;
  };
  auto hidden = [&](int l, bool none) {
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const int t = tile_of(l, w);
      if (t < 0) continue;
      float v0, v1;
      sum(l, w, v0, v1, none);
      if (e_row < count) {
        T* dst = (T*)p.layer[l].out + frag_offset<T>(first + e_row, t * TILE + e_col, p.layer[l].out_chunks);
        const T a = Elem<T>::from_f32(fmaxf(v0, 0.f)), b = Elem<T>::from_f32(fmaxf(v1, 0.f));
        if constexpr (sizeof(T) == 2) *(uint32_t*)dst = (uint32_t)a | (uint32_t)b << 16;
        else *(float2*)dst = make_float2(a, b);
      }
    }
  };

  lds_barrier();                                         // (biases and bounds)
  int active = count == 32 ? -1 : (1 << count) - 1;
  int iters = 0;                                         // rank 0, lane i < 32: passes of row i
  int passes = 0, sample_passes = 0;
  bool unconverged = false;
  // One turn: layer l of pass k, or (l = -1) nothing but the barrier behind the set-up.  Started from zeros, the first layer
  // is ReLU(bias) whatever its weights, and needs neither.
  int k = 1, l = -1;
  bool none = p.zero_start != 0;
  if (none) l = 0;
  for (;;) {
    if (l >= 0 && !none) product(l);
    if (l == L) {
      const bool live = e_row < count && ((active >> e_row) & 1);
      bool moved = false;
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const int t = tile_of(L, w);
        if (t < 0) continue;
        float v[2];
        sum(L, w, v[0], v[1]);
#pragma unroll
        for (int j = 0; j < P_; ++j) {
          if (live && pos[w] + j < D) {
            float xn;
            if constexpr (REAL) {
              xn = v[0] + expf(fminf(fmaxf(v[1], LOGISTIC_A_LO), LOGISTIC_A_HI)) * noise[w][j];
              moved |= !(fabsf(xn - state[w][j]) <= p.eps);     // (a NaN counts as changed)
            } else {
              xn = noise[w][j] < bernoulli_probability(v[j]) ? 1.f : 0.f;
              moved |= xn != state[w][j];
            }
            if (xn != state[w][j]) {                            // (an unchanged state's encoding is in place)
              state[w][j] = xn;
              ((T*)p.enc)[frag_offset<T>(first + e_row, pos[w] + j, p.enc_chunks)] = Elem<T>::from_f32(xn);
            }
          }
        }
      }
      {
        const unsigned long long m = __ballot(moved);      // 16 lanes to a row
        if (lane == 0) {
          int rows = 0;
#pragma unroll
          for (int g = 0; g < 4; ++g) rows |= (m >> (16 * g) & 0xffffull) != 0 ? 1 << (4 * wave + g) : 0;
          changed_s[wave] = rows;
        }
      }
    } else if (l >= 0) {
      hidden(l, none);
    }
    none = false;
    const int next = l == L ? 0 : l + 1;
    if (!barrier(next, l == L)) return;
    if (l == L) {
      passes += 1;
      sample_passes += __builtin_popcount((unsigned)active);
      iters += (active >> (lane & 31)) & 1;
      active &= __builtin_amdgcn_readfirstlane(active_s);
      if (k == p.cap) unconverged = active != 0 && p.flag_unconverged;
      if (active == 0 || k == p.cap) break;
      ++k;
    }
    l = next;
  }

  // ---- the result, and the XCD's report by its first workgroup (the symbols are ordered like those of any launch: they are
  // there when the kernel has ended)
#pragma unroll
  for (int w = 0; w < 2; ++w)
#pragma unroll
    for (int j = 0; j < P_; ++j)
      if (e_row < count && pos[w] + j < D) {
        const size_t i = (size_t)e_sample * D + pos[w] + j;
        if constexpr (REAL) ((float*)p.x)[i] = state[w][j];
        else ((uint8_t*)p.x)[i] = (uint8_t)state[w][j];
      }
  if (rank == 0 && wave == 0) {
    if (lane < count) p.iters[first + lane] = iters;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0) {
      *epoch_word = epoch;
      __hip_atomic_store(report + 0, passes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(report + 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(report + 2, sample_passes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(report + 3, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(report + 4, unconverged ? 1 : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(report + 5, p.call_id, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

}  // namespace jm
