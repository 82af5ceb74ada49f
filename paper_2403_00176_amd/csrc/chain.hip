// A whole step of one-row work (the decode step: embedding, LayerNorm + projection, attention over the cache,
// projections, arg-max) as one kernel.
//
// Such a step is a chain of some 120 groups that each read a few MB of weights and one row of activations.  As kernels
// of their own they cost 5 to 10 us each: launch, one memory round trip for the row, one for the weights, and the
// drain; 0.85 ms per token for 0.13 ms of weight traffic.  Here one workgroup per CU stays for the whole step:
//   * a phase's weights do not depend on the phase before it, so every workgroup requests its share of the next
//     phase's weights (and of the cached keys and values) before it waits for the next phase's input;
//   * rows are exchanged as tagged words: 8 bytes holding two bf16 results (or one fp32 value) and the number of the
//     phase.  A producer writes its words through to memory, every consumer polls the words it needs.  No counter, no
//     separate flag, no cache maintenance: one exchange among 256 workgroups takes 1.5 - 1.9 us, against 2.8 us with a
//     flag per workgroup and 2.4 - 3.2 us for an empty kernel.  A producer's words have a 128-byte line of their own:
//     with several producers in one line (partial writes from different XCDs) the exchange takes 3 us.
// Workgroup w owns the rows w * rpw .. of every contraction; of its 8 computing waves, wave v takes the k segment
// v % nseg of 512 elements (one 16-byte load per lane and row), partial sums meet in LDS.  Attention: one workgroup per
// head and 128 keys leaves its unnormalised sum, maximum and weight; the contraction behind it combines them as it reads.
//
// Waiting inside a kernel needs all workgroups on the chip at once, and one fills a CU.  Nothing is assumed about that:
// every workgroup counts itself in before it sends its first words, and whoever waits for those words longer than
// CH_ARRIVE while some workgroup is missing calls the exchange off, in the word that holds the count, so that all agree.
// Nothing but words has been written by then.  The workgroups leave, the ones that come later find the mark, and the
// last of them computes the whole step by itself, with no one to wait for (10 ms instead of 0.4, but the same step);
// the host then launches group by group for CH_REST seconds.  Once everyone has counted in, all are on the chip to the
// end and no wait can be in vain; a limit of CH_POLLS polls stands against a broken machine: past it the row becomes NaN
// (so do the logits; the token is -1) and the next step of the process reports the failure.
// What keeps the workgroups from coming together for a while: kernels of other streams, streams whose CU mask is too
// narrow (not given this kernel), a second process on the device.  Launches of different streams of this process are
// ordered by an event, and of several processes that see each other's socket names only the first uses this kernel.
//
// One step of the 24-layer decoder (hidden 1024, FFN 4096, vocabulary 32000; 605 MB of weights) with 300 cached rows:
// 0.87 ms as 124 kernels, 0.36 ms as this one (1.7 TB/s of weights).  A layer takes 14.6 us: per exchange 0.8 - 1.2 us
// from the last producer's store to the row in LDS, 0.4 us more for a LayerNorm, 0.8 - 1.2 us from there to the store.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <sys/socket.h>
#include <sys/un.h>
#include <unistd.h>

#include <chrono>
#include <cstddef>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "chain.hpp"
#include "device_common.hpp"
#include "internal.hpp"

namespace sod2 {

typedef unsigned long long u64;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int CH_WAVES = 8, CH_IN = 8, CH_THREADS = (CH_WAVES + CH_IN) * 64;   // waves that compute, waves that wait for rows
constexpr int CH_U = 4;                                                    // 16-byte weight loads in flight per lane and phase
constexpr int CH_LN = 2;                                                   // waves that normalise a row
constexpr int CH_AHEAD = 2;                                                // phases whose weights are asked for ahead of time
constexpr int CH_PAR = CH_AHEAD + 3;                                       // phases whose parameters are kept: asked for CH_AHEAD + 1 ahead, read to a phase's end
constexpr int CH_KU = CHAIN_KEYS / 64;                                     // cached keys (and values) per thread
static_assert(2 * CH_KU == CH_U, "the keys and values of an attention part take the place of a contraction's weights");
constexpr int CH_LINE = 16;                                                // words of one producer: a 128-byte line
constexpr int CH_ATT = 80;                                                 // words of one attention part: 64 sums, maximum, weight
constexpr int CH_REGION = CHAIN_MAX_WG * CH_ATT;                           // words of one phase
constexpr int CH_RING = 16;                                                // phases before a region is written again
constexpr int CH_PART = 1024;                                              // partial sums of a phase in LDS
constexpr int CH_ARRIVE = 20000;                                           // microseconds the workgroups wait for one another to start
constexpr int CH_POLLS = 1 << 25;                                          // polls of one wait after that: upwards of 10 s
constexpr int CH_REST = 5;                                                 // seconds without this kernel after a step done by one workgroup
constexpr unsigned CH_OFF = 0x80000000u;                                   // in the count of arrivals: the exchange is off
constexpr int CH_ROW = CHAIN_MAX_WG * CH_LINE;                             // words of a row (two bf16 each) of the lone workgroup

struct ChainArgs {
  const ChainStep* steps;
  u64* mail;
  unsigned* here;                   // arrivals of this launch
  unsigned* here_next;              // of the next, cleared by this one
  uint32_t* rows;                   // CH_RING rows of a workgroup that does the step by itself
  unsigned* error;                  // pinned host words: [0] a wait ran past its limit, [1] a step was done by one workgroup
  unsigned arrive, polls;           // limits of the waits: ticks of the 100 MHz clock, polls
  char* ext[CHAIN_MAX_EXT];         // the caller's inputs and outputs of this launch
  int n_steps, lk;
  unsigned tag0;
};

__device__ __forceinline__ u64 mail_load(const u64* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void mail_store(u64* p, uint32_t payload, unsigned tag) {
  __hip_atomic_store(p, ((u64)tag << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the words at a.mail[at[0 .. n)] until all of them carry `tag`.  (All n are asked for together every time: a load under a
// condition of its own would be waited for on its own.)  first: the wait for the first row, words of every workgroup,
// which may not all be on the chip; *left is set when the exchange is off.  Past the limit of polls (*dead set) the words
// are NaN, of either type.
template <int n>
__device__ __forceinline__ void mail_wait(const ChainArgs& a, const uint32_t (&at)[n], unsigned tag, uint32_t (&v)[n], int* dead, bool first, int* left) {
  u64 w[n];
  unsigned spins = 0;
  u64 t0 = 0;
  for (;;) {
    bool all = true;
#pragma unroll
    for (int i = 0; i < n; ++i) w[i] = mail_load(a.mail + at[i]);
#pragma unroll
    for (int i = 0; i < n; ++i) all = all && (unsigned)(w[i] >> 32) == tag;
    if (all) break;
    if ((++spins & 255) == 0 || spins >= a.polls) {
      if (first) {
        unsigned here = __hip_atomic_load(a.here, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (here < gridDim.x) {                            // (someone is missing, and the exchange is on)
          const u64 now = wall_clock64();
          if (t0 == 0) t0 = now;
          if (now - t0 < a.arrive) continue;
          if (!__hip_atomic_compare_exchange_strong(a.here, &here, here | CH_OFF, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) continue;
          here |= CH_OFF;
        }
        if (here & CH_OFF) {
          __hip_atomic_store(left, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          break;
        }
      }
      if (spins >= a.polls || __hip_atomic_load(dead, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
        __hip_atomic_store(dead, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
        for (int i = 0; i < n; ++i) w[i] = 0x7fc07fc0u;
        break;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < n; ++i) v[i] = (uint32_t)w[i];
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <class T> __device__ __forceinline__ const T* unip(const void* p) {     // a pointer all lanes agree on, in scalar registers
  const u64 v = (u64)p;
  return (const T*)(((u64)(uint32_t)uni((int)(v >> 32)) << 32) | (uint32_t)uni((int)v));
}
// 16 bytes per lane from memory to LDS (lane l: base + 16 l); counted with the wave's other vector memory operations
__device__ __forceinline__ void ring_load(const void* p, uint32_t lds_wave_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_wave_base), "v"(p) : "memory");
}
__device__ __forceinline__ void ring_load4(const void* p, uint32_t lds_wave_base) {    // 4 bytes per lane
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_wave_base), "v"(p) : "memory");
}
__device__ __forceinline__ uint32_t lds_addr(void* p) { return (uint32_t)uni((int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)p); }
// LDS written before is visible after; global loads in flight stay in flight
__device__ __forceinline__ void wg_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
__device__ __forceinline__ float lo_f(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float hi_f(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }

// a.x b.x + a.y b.y + c of two bf16 pairs, in fp32
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}
__device__ __forceinline__ float add_halves(float v) {        // lane ^ 16 and lane ^ 32, without LDS
  typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
  u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// the sums of four values over the wave, value l & 3 in lane l: the first two exchanges halve the number of values
__device__ __forceinline__ float wave_sum4(const float (&d)[4], int lane) {
  const float e01 = ((lane & 1) ? d[1] : d[0]) + dpp_move<0xB1>(0.f, (lane & 1) ? d[0] : d[1]);
  const float e23 = ((lane & 1) ? d[3] : d[2]) + dpp_move<0xB1>(0.f, (lane & 1) ? d[2] : d[3]);
  float f = ((lane & 2) ? e23 : e01) + dpp_move<0x4E>(0.f, (lane & 2) ? e01 : e23);
  f += dpp_move<0x124>(0.f, f);                               // row_ror 4
  f += dpp_move<0x128>(0.f, f);                               // row_ror 8
  return add_halves(f);
}

// of two (value, index) pairs the larger value, the lower index among equals; 0x7fffffff: none
__device__ __forceinline__ void wave_argmax(float& v, int& i) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(v, o, 64);
    const int oi = __shfl_xor(i, o, 64);
    if (oi != 0x7fffffff && (i == 0x7fffffff || ov > v || (ov == v && oi < i))) { v = ov; i = oi; }
  }
}

// The whole step by one workgroup that waits for no other: 16 waves, a pair of rows or a head to a wave at a time.  Rows
// lie in a.rows, two values to a word; the values are those the exchanged rows would hold (sums in another order).
__device__ __forceinline__ void step_alone(const ChainArgs& a, const ChainStep* steps, char* const* ext, uint32_t* xw, float* part) {
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  constexpr int WAVES = CH_THREADS / 64;
  auto row_of = [&](int p) __attribute__((always_inline)) { return a.rows + (p & (CH_RING - 1)) * CH_ROW; };
  for (int p = 0; p < a.n_steps; ++p) {
    const ChainStep& s = steps[p];
    const int kind = uni(s.kind), n = uni(s.n);
    uint32_t* out = row_of(p);
    const uint32_t* in = row_of(uni(s.src));               // (a first phase has none and reads none)
    if (kind == CHAIN_GATHER) {
      auto row = [&](const void* table, int slot, long long rows, int i32) {
        const char* ix = ext[slot];
        long long id = i32 ? (long long)*(const int*)ix : *(const long long*)ix;
        id = id < 0 ? 0 : (id >= rows ? rows - 1 : id);
        return (const uint32_t*)((const bf16_t*)table + id * n);
      };
      for (int i = tid; i < n / 2; i += CH_THREADS) {
        uint32_t v = row(s.w, s.idx_ext, s.table_rows, s.idx_i32)[i];
        if (s.bias) {
          const uint32_t u = row(s.bias, s.idx2_ext, s.table2_rows, s.idx2_i32)[i];
          v = f2bf2(lo_f(v) + lo_f(u), hi_f(v) + hi_f(u));
        }
        out[i] = v;
      }
    } else if (kind == CHAIN_ATTN) {
      const int lk = a.lk + uni(s.lk_rel), ldw = uni(s.ldw), kg = lane >> 3, dc = lane & 7;
      const float scale = __uint_as_float(uni(__float_as_uint(s.scale))) * 1.4426950408889634f;
      for (int h = wave; h < n; h += WAVES) {
        const int col = h * 64 + dc * 8;
        u32x4 q, kn, vn;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          q[e] = in[((s.q_off + col) >> 1) + e];
          kn[e] = in[((s.k_off + col) >> 1) + e];
          vn[e] = in[((s.v_off + col) >> 1) + e];
        }
        float m = -INFINITY, l = 0.f, o[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int t0 = 0; t0 < lk; t0 += 8) {
          const int t = t0 + kg;
          u32x4 kr = kn, vr = vn;
          if (t < lk - 1) {
            kr = *(const u32x4*)((const bf16_t*)s.w + (long long)t * ldw + col);
            vr = *(const u32x4*)((const bf16_t*)s.bias + (long long)t * ldw + col);
          }
          float d = 0.f;
#pragma unroll
          for (int e = 0; e < 4; ++e) d = dot2(q[e], kr[e], d);
          d = octet_sum(d) * scale;
          if (t < lk) {
            const float mn = fmaxf(m, d), f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn);
            const float pr = d == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(d - mn);
            l = fmaf(l, f, pr);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              o[2 * e] = fmaf(o[2 * e], f, pr * lo_f(vr[e]));
              o[2 * e + 1] = fmaf(o[2 * e + 1], f, pr * hi_f(vr[e]));
            }
            m = mn;
          }
        }
        const float mx = wave_max(m), f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mx);
        l *= f;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] *= f;
#pragma unroll
        for (int x = 8; x < 64; x <<= 1) {
          l += __shfl_xor(l, x, 64);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] += __shfl_xor(o[e], x, 64);
        }
        if (kg == 0) {
          const float inv = 1.f / l;
#pragma unroll
          for (int e = 0; e < 4; ++e) out[(col >> 1) + e] = f2bf2(o[2 * e] * inv, o[2 * e + 1] * inv);
          *(u32x4*)((bf16_t*)s.w + (long long)(lk - 1) * ldw + col) = kn;       // the cache rows for later steps
          *(u32x4*)((bf16_t*)s.bias + (long long)(lk - 1) * ldw + col) = vn;
        }
      }
    } else {
      const int K = uni(s.k), words = K >> 1, ldw = uni(s.ldw), act1 = uni(s.act1), act2 = uni(s.act2), res = uni(s.res);
      if (s.gamma) {                                       // (K <= 1024: word 64 i + lane of the row, waves 0 .. 7 write one each)
        float d0 = 0.f;
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          v[i] = lane + 64 * i < words ? in[lane + 64 * i] : 0u;
          d0 += lo_f(v[i]) + hi_f(v[i]);
        }
        const float inv_k = 1.f / (float)K, mean = wave_sum(d0) * inv_k;
        d0 = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const bool on = lane + 64 * i < words;
          const float a0 = on ? lo_f(v[i]) - mean : 0.f, a1 = on ? hi_f(v[i]) - mean : 0.f;
          d0 = fmaf(a0, a0, fmaf(a1, a1, d0));
        }
        const float rstd = rsqrtf(wave_sum(d0) * inv_k + s.eps);
        const int i = wave * 64 + lane;
        if (i < words) {
          const uint32_t x = in[i], g = ((const uint32_t*)s.gamma)[i], b = ((const uint32_t*)s.beta)[i];
          xw[i] = f2bf2(fmaf((lo_f(x) - mean) * rstd, lo_f(g), lo_f(b)), fmaf((hi_f(x) - mean) * rstd, hi_f(g), hi_f(b)));
        }
      } else {
        for (int i = tid; i < words; i += CH_THREADS) xw[i] = in[i];
      }
      __syncthreads();
      float bv = -INFINITY;
      int bi = 0x7fffffff;
      for (int i = wave; 2 * i < n; i += WAVES) {
        const bf16_t* w = (const bf16_t*)s.w + 2ll * i * ldw;
        float d0 = 0.f, d1 = 0.f;
        for (int k = lane * 8; k < K; k += 512) {
          const u32x4 x = *(const u32x4*)&xw[k >> 1], w0 = *(const u32x4*)(w + k), w1 = *(const u32x4*)(w + ldw + k);
#pragma unroll
          for (int e = 0; e < 4; ++e) { d0 = dot2(x[e], w0[e], d0); d1 = dot2(x[e], w1[e], d1); }
        }
        const uint32_t b2 = s.bias ? ((const uint32_t*)s.bias)[i] : 0u;
        float v0 = apply_act(wave_sum(d0) * s.scale + lo_f(b2), act1), v1 = apply_act(wave_sum(d1) * s.scale + hi_f(b2), act1);
        if (res >= 0) {
          const uint32_t r = row_of(res)[i];
          v0 = apply_act(v0 + lo_f(r), act2);
          v1 = apply_act(v1 + hi_f(r), act2);
        }
        const uint32_t o = f2bf2(v0, v1);
        if (lane == 0) (s.out_ext >= 0 ? (uint32_t*)ext[s.out_ext] : out)[i] = o;
        if (bi == 0x7fffffff || lo_f(o) > bv) { bv = lo_f(o); bi = 2 * i; }
        if (hi_f(o) > bv) { bv = hi_f(o); bi = 2 * i + 1; }
      }
      if (s.arg_ext >= 0) {
        int* index = (int*)(part + WAVES);
        if (lane == 0) { part[wave] = bv; index[wave] = bi; }
        __syncthreads();
        if (tid == 0) {
          for (int v = 1; v < WAVES; ++v)
            if (index[v] != 0x7fffffff && (bi == 0x7fffffff || part[v] > bv || (part[v] == bv && index[v] < bi))) { bv = part[v]; bi = index[v]; }
          if (s.arg_i32) *(int*)ext[s.arg_ext] = bi;
          else *(long long*)ext[s.arg_ext] = bi;
        }
      }
    }
    __syncthreads();                                       // the row is there for everyone, and xw free
  }
  if (tid == 0) __hip_atomic_store(a.error + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The waves of a workgroup have one of two parts, because a wave's loads come back in order: a wave that polls must not
// have weights on their way.  Waves 8 .. 15 gather, wait for rows and leave them (normalised) in LDS; waves 0 .. 7 keep
// the weights of two phases on their way into a ring of LDS, multiply, and wave 0 finishes and sends the rows.  Two barriers per phase:
// row there, partial sums there.
__global__ __launch_bounds__(CH_THREADS, 4) void chain_kernel(ChainArgs a) {
  __shared__ ChainStep steps[CHAIN_MAX_STEPS];
  __shared__ __attribute__((aligned(16))) uint32_t xw[CHAIN_MAX_K / 2];    // the input row, two bf16 to a word
  __shared__ uint32_t own[CH_RING][64];                                    // this workgroup's part of the last rows (residuals)
  __shared__ __attribute__((aligned(16))) uint32_t lnw[CH_PAR][2][512];   // LayerNorm scale and shift on their way
  __shared__ uint32_t biasw[CH_PAR][64];                             // bias of this workgroup's rows on its way
  __shared__ __attribute__((aligned(16))) u32x4 ring[CH_WAVES][CH_AHEAD + 1][CH_U][64];   // weights (keys, values) on their way, each wave's own
  __shared__ __attribute__((aligned(16))) float part[CH_PART];
  __shared__ __attribute__((aligned(16))) uint32_t qkv[96];                // attention: the head's query, new key, new value
  __shared__ float am[CH_WAVES], al[CH_WAVES], ao[CH_WAVES][64];
  __shared__ uint32_t nowhere[64];
  __shared__ int dead, left;                               // a wait ran past its limit; the exchange is off
  __shared__ unsigned arrived;
  __shared__ char* ext[CHAIN_MAX_EXT];
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int wg = blockIdx.x, nwg = gridDim.x;
  for (int i = tid; i < a.n_steps * (int)(sizeof(ChainStep) / 16); i += CH_THREADS) ((uint4*)steps)[i] = ((const uint4*)a.steps)[i];
  if (tid == 0) {
    dead = left = 0;
    if (a.arrive == 0) __hip_atomic_fetch_or(a.here, CH_OFF, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    arrived = __hip_atomic_fetch_add(a.here, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (wg == 0) __hip_atomic_store(a.here_next, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int i = 0; i < CHAIN_MAX_EXT; ++i) ext[i] = a.ext[i];
  }
  __syncthreads();
  if (uni((int)arrived) < 0) {                             // the exchange is off: the last one to come does the step
    if ((uni((int)arrived) & 0x7fffffff) == nwg - 1) step_alone(a, steps, ext, xw, part);
    return;
  }

  // attention: parts per head; part head * splits + split of this workgroup, or -1
  auto attn_splits = [&](const ChainStep& s) __attribute__((always_inline)) { return (a.lk + uni(s.lk_rel) + CHAIN_KEYS - 1) / CHAIN_KEYS; };
  auto attn_part = [&](const ChainStep& s) __attribute__((always_inline)) {
    const int parts = uni(s.n) * attn_splits(s), every = nwg / parts, id = wg / every;
    return (wg % every == 0 && id < parts) ? id : -1;
  };
  auto region = [&](int p) __attribute__((always_inline)) { return (uint32_t)(p & (CH_RING - 1)) * CH_REGION; };   // in words of a.mail
  const int n_steps = a.n_steps;

  if (wave >= CH_WAVES) {
    // ------------------------------------------------------------------------------ rows in
    const int ct = tid - CH_WAVES * 64, cw = wave - CH_WAVES;
    // where word i (elements 2 i, 2 i + 1) of the row that phase p produced is
    auto word_of = [&](int p, int i) __attribute__((always_inline)) {
      const unsigned ppw = (unsigned)uni(steps[p].rpw) >> 1, g = (unsigned)i / ppw;
      return region(p) + (g * CH_LINE + (i - g * ppw));
    };
    for (int p = 0; p < n_steps; ++p) {
      const ChainStep& s = steps[p];
      const int kind = uni(s.kind), src = uni(s.src);
      if (kind == CHAIN_GATHER) {
        // one row of a table (and one of a second): every workgroup takes its own elements
        const int rpw = uni(s.rpw), n = uni(s.n), e = wg * rpw + 2 * ct;
        if (2 * ct < rpw && e < n) {
          auto row = [&](const void* table, int slot, long long rows, int i32) {
            const char* ix = ext[slot];
            long long id = i32 ? (long long)*(const int*)ix : *(const long long*)ix;
            id = id < 0 ? 0 : (id >= rows ? rows - 1 : id);
            return *(const uint32_t*)((const bf16_t*)table + id * n + e);
          };
          uint32_t v = row(s.w, s.idx_ext, s.table_rows, s.idx_i32);
          if (s.bias) {
            const uint32_t u = row(s.bias, s.idx2_ext, s.table2_rows, s.idx2_i32);
            v = f2bf2(lo_f(v) + lo_f(u), hi_f(v) + hi_f(u));
          }
          own[p & (CH_RING - 1)][ct] = v;
          mail_store(a.mail + region(p) + wg * CH_LINE + ct, v, a.tag0 + p);
        }
        wg_barrier();                                      // (the next phase's scale and shift have landed)
        continue;
      }
      if (kind == CHAIN_ATTN) {
        const int id = uni(attn_part(s));
        if (id < 0) continue;
        const int h = id / attn_splits(s);
        if (ct < 96) {
          const int which = ct >> 5, off = which == 0 ? s.q_off : (which == 1 ? s.k_off : s.v_off);
          uint32_t at[1] = {word_of(src, ((off + h * 64) >> 1) + (ct & 31))};
          uint32_t v[1];
          mail_wait<1>(a, at, a.tag0 + src, v, &dead, false, &left);
          qkv[ct] = v[0];
        }
        wg_barrier();
        wg_barrier();
        continue;
      }
      // a contraction's input row
      const int K = uni(s.k), words = K >> 1;
      if (uni(steps[src].kind) == CHAIN_ATTN) {
        // heads * 64 values: the parts of a head are combined by everyone who reads it
        const int splits = attn_splits(steps[src]);
        for (int i = ct; i < words; i += CH_IN * 64) {
          const uint32_t base = region(src) + ((2 * i) >> 6) * splits * CH_ATT;
          const int e = (2 * i) & 63;
          float m = -INFINITY, l = 0.f, o0 = 0.f, o1 = 0.f;
          for (int s0 = 0; s0 < splits; s0 += 4) {
            uint32_t at[16], v[16];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const uint32_t b = base + min(s0 + u, splits - 1) * CH_ATT;
              at[4 * u] = b + e; at[4 * u + 1] = b + e + 1; at[4 * u + 2] = b + 64; at[4 * u + 3] = b + 65;
            }
            mail_wait<16>(a, at, a.tag0 + src, v, &dead, false, &left);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (s0 + u >= splits) continue;
              const float mu = __uint_as_float(v[4 * u + 2]), mn = fmaxf(m, mu);
              const float f0 = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn);
              const float f1 = mu == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mu - mn);
              o0 = o0 * f0 + __uint_as_float(v[4 * u]) * f1;
              o1 = o1 * f0 + __uint_as_float(v[4 * u + 1]) * f1;
              l = l * f0 + __uint_as_float(v[4 * u + 3]) * f1;
              m = mn;
            }
          }
          const float inv = 1.f / l;
          xw[i] = f2bf2(o0 * inv, o1 * inv);
        }
      } else if (s.gamma) {
        // LayerNorm of the row (K <= 1024): a lane waits for 8 words, the statistics are lane moves; CH_LN waves do the
        // same and each leaves its share of the result
        if (cw < CH_LN) {
          uint32_t v[8], at[8];
          const float eps = __uint_as_float(uni(__float_as_uint(s.eps))), inv_k = 1.f / (float)K;
#pragma unroll
          for (int i = 0; i < 8; ++i) at[i] = word_of(src, min(lane + 64 * i, words - 1));
          // wave cw writes words 64 (4 cw + i) + lane (a branch per word would cost more than the word)
          static_assert(CH_LN == 2, "a half of the row per wave");
          uint32_t gm[4], bt[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            gm[i] = lnw[p % CH_PAR][0][64 * (4 * cw + i) + lane];
            bt[i] = lnw[p % CH_PAR][1][64 * (4 * cw + i) + lane];
          }
          float g0[4], g1[4], b0[4], b1[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) { g0[i] = lo_f(gm[i]); g1[i] = hi_f(gm[i]); b0[i] = lo_f(bt[i]); b1[i] = hi_f(bt[i]); }
          mail_wait<8>(a, at, a.tag0 + src, v, &dead, p == 1, &left);
          // the mean, then the squared distances from it, as the row kernels do it: a difference of two sums of squares
          // would lose digits, and overflow for rows whose distances do not
          if (words < 512) {
#pragma unroll
            for (int i = 0; i < 8; ++i) if (lane + 64 * i >= words) v[i] = 0u;
          }
          float d0 = 0.f, d1 = 0.f;
#pragma unroll
          for (int i = 0; i < 8; i += 2) {
            d0 = dot2(v[i], 0x3f803f80u, d0);              // bf16 ones
            d1 = dot2(v[i + 1], 0x3f803f80u, d1);
          }
          const float mean = wave_sum(d0 + d1) * inv_k;
          d0 = d1 = 0.f;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const bool in = words == 512 || lane + 64 * i < words;
            const float a0 = in ? lo_f(v[i]) - mean : 0.f, a1 = in ? hi_f(v[i]) - mean : 0.f;
            d0 = fmaf(a0, a0, d0);
            d1 = fmaf(a1, a1, d1);
          }
          const float rstd = rsqrtf(wave_sum(d0 + d1) * inv_k + eps);
          uint32_t u[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) u[i] = cw ? v[4 + i] : v[i];
#pragma unroll
          for (int i = 0; i < 4; ++i)                      // (what lies beyond K is not read)
            xw[64 * (4 * cw + i) + lane] = f2bf2(fmaf((lo_f(u[i]) - mean) * rstd, g0[i], b0[i]), fmaf((hi_f(u[i]) - mean) * rstd, g1[i], b1[i]));
        }
      } else {
        constexpr int PER = CHAIN_MAX_K / 2 / (CH_IN * 64);
        uint32_t at[PER], v[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) at[i] = word_of(src, min(ct + i * CH_IN * 64, words - 1));
        mail_wait<PER>(a, at, a.tag0 + src, v, &dead, p == 1, &left);
#pragma unroll
        for (int i = 0; i < PER; ++i) if (ct + i * CH_IN * 64 < words) xw[ct + i * CH_IN * 64] = v[i];
      }
      const int rpw = uni(s.rpw);
      wg_barrier();
      wg_barrier();
      if (p == 1 && uni(left)) break;
      if (uni(s.arg_ext) >= 0 && wg == 0 && cw == 0) {
        // arg-max: every workgroup's best pair
        float bv = -INFINITY;
        int bi = 0x7fffffff;
        const int waves = (rpw + 127) / 128;
        for (int i = lane; i < nwg * waves; i += 64) {
          const uint32_t line = region(p) + i / waves * CH_LINE + i % waves * 2;
          uint32_t at[2] = {line, line + 1};
          uint32_t v[2];
          mail_wait<2>(a, at, a.tag0 + p, v, &dead, false, &left);
          const float ov = __uint_as_float(v[0]);
          const int oi = (int)v[1];
          if (oi != 0x7fffffff && (bi == 0x7fffffff || ov > bv || (ov == bv && oi < bi))) { bv = ov; bi = oi; }
        }
        wave_argmax(bv, bi);
        if (__hip_atomic_load(&dead, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) bi = -1;
        if (lane == 0) {
          if (s.arg_i32) *(int*)ext[s.arg_ext] = bi;
          else *(long long*)ext[s.arg_ext] = bi;
        }
      }
    }
  } else {
    // ------------------------------------------------------------------------------ weights, products, rows out
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const uint32_t ring_base = lds_addr(&ring[wave][0][0][0]);
    // rows first + step j of this workgroup's part of a contraction, j = j0 .. j0 + CH_U - 1, this wave's k segment
    auto load_w = [&](const ChainStep& s, int j0, u32x4 (&d)[CH_U]) __attribute__((always_inline)) {
      const int sh = uni(s.seg_shift), rpw = uni(s.rpw), ldw = uni(s.ldw), n = uni(s.n);
      const int k = (wave & ((1 << sh) - 1)) * 512 + lane * 8, rows = k < uni(s.k) ? min(rpw, n - wg * rpw) : 0;
      const char* base = unip<char>(s.w) + (wg * rpw < n ? (long long)wg * rpw * ldw * 2 : 0);
#pragma unroll
      for (int j = 0; j < CH_U; ++j) {
        const int row = (wave >> sh) + (CH_WAVES >> sh) * (j0 + j);
        d[j] = *(const u32x4*)(base + (row < rows ? (uint32_t)(row * ldw + k) * 2u : 0u));
      }
    };
    // What phase p needs of memory: rows of its weights, or (attention) cached keys and values, straight into this wave's
    // ring in LDS.  Always the same number of loads, valid or not (an address that is not goes to the start), so that
    // waiting for one phase's leaves the later phases' on their way.  The addresses are worked out while the wave has
    // nothing else to do.
    // A phase's LayerNorm scale and shift (1 KB each to waves 1 .. 4) and bias (wave 5, 4 bytes a lane) go out one phase
    // before its weights: they have landed when the phase before it starts, so the waves that wait for rows find them.
    struct Plan { const char *w0, *w1, *par; uint32_t off[CH_U], par_off; };
    auto plan_params = [&](int p, Plan& f) __attribute__((always_inline)) {
      const ChainStep& s = steps[min(p, n_steps - 1)];
      const bool gemv = uni(s.kind) == CHAIN_GEMV;
      const char* par = wave <= 2 ? unip<char>(s.gamma) : (wave <= 4 ? unip<char>(s.beta) : unip<char>(s.bias));
      const int half = (wave - 1) & 1;                     // of the scale or shift: elements 512 half + 8 lane
      const bool ln = wave >= 1 && wave <= 4 && half * 512 + lane * 8 < uni(s.k);
      const bool bs = wave == 5 && 2 * lane < uni(s.rpw) && wg * uni(s.rpw) + 2 * lane < uni(s.n);
      const bool on = gemv && par && (ln || bs);
      f.par = (gemv && par) ? par : unip<char>(s.w);
      f.par_off = !on ? 0u : (wave == 5 ? (uint32_t)(wg * uni(s.rpw) + 2 * lane) * 2u : (uint32_t)(half * 512 + lane * 8) * 2u);
    };
    auto issue_params = [&](const Plan& f, int p) __attribute__((always_inline)) {
      const int slot = p % CH_PAR;
      // (the waves without a parameter load their line into a place nobody reads: the count stays the same)
      if (wave >= 1 && wave <= 4) ring_load(f.par + f.par_off, lds_addr(&lnw[slot][wave > 2][((wave - 1) & 1) * 256]));
      else ring_load4(f.par + f.par_off, lds_addr(wave == 5 ? &biasw[slot][0] : &nowhere[0]));
    };
    auto plan = [&](int p) __attribute__((always_inline)) {
      Plan f;
      const ChainStep& s = steps[min(p, n_steps - 1)];
      const int ldw = uni(s.ldw), n = uni(s.n);
      f.w0 = f.w1 = unip<char>(s.w);
      int first, step, rows, col;                          // loads of row first + j step < rows, element col
      bool attn = uni(s.kind) == CHAIN_ATTN;
      if (attn) {
        const int id = uni(attn_part(s)), splits = attn_splits(s), h = max(id, 0) / splits, sp = max(id, 0) - h * splits;
        first = sp * CHAIN_KEYS + (tid >> 3);
        step = 64;
        rows = id < 0 ? 0 : a.lk + uni(s.lk_rel) - 1;
        col = h * 64 + (tid & 7) * 8;
        f.w1 = unip<char>(s.bias);
      } else {
        const int rpw = uni(s.rpw), sh = uni(s.seg_shift);
        col = (wave & ((1 << sh) - 1)) * 512 + lane * 8;
        first = wave >> sh;
        step = CH_WAVES >> sh;
        rows = col < uni(s.k) ? min(rpw, n - wg * rpw) : 0;
        if (wg * rpw < n) f.w0 += (long long)wg * rpw * ldw * 2;
        f.w1 = f.w0;
      }
#pragma unroll
      for (int j = 0; j < CH_U; ++j) {
        const int row = first + step * (attn && j >= CH_KU ? j - CH_KU : j);
        f.off[j] = row < rows ? (uint32_t)(row * ldw + col) * 2u : 0u;
      }
      plan_params(p + 1, f);
      return f;
    };
    auto issue = [&](const Plan& f, int p) __attribute__((always_inline)) {
      const uint32_t slot = ring_base + (uint32_t)(p % (CH_AHEAD + 1)) * (CH_U * 1024);
#pragma unroll
      for (int j = 0; j < CH_U; ++j) ring_load((j >= CH_KU ? f.w1 : f.w0) + f.off[j], slot + j * 1024);
      issue_params(f, p + 1);
    };
    // phase p's loads have landed (those of the CH_AHEAD - 1 phases behind it need not): into registers
    auto take = [&](int p, u32x4 (&d)[CH_U]) __attribute__((always_inline)) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((CH_AHEAD - 1) * (CH_U + 1)) : "memory");
      const u32x4* r = &ring[wave][p % (CH_AHEAD + 1)][0][lane];
#pragma unroll
      for (int j = 0; j < CH_U; ++j) d[j] = r[j * 64];
    };

    auto attention = [&](int p, const ChainStep& s, int id, const u32x4 (&kv)[CH_U], const Plan& next) __attribute__((always_inline)) {
      const int splits = attn_splits(s), h = id / splits, sp = id - h * splits, lk = a.lk + uni(s.lk_rel);
      wg_barrier();
      issue(next, p + CH_AHEAD);
      // the cache rows for later steps
      if (sp == splits - 1 && tid < 16) {
        bf16_t* row = (tid < 8 ? (bf16_t*)s.w : (bf16_t*)s.bias) + (long long)(lk - 1) * s.ldw + h * 64 + (tid & 7) * 8;
        *(u32x4*)row = *(const u32x4*)&qkv[(tid < 8 ? 32 : 64) + (tid & 7) * 4];
      }
      const int kg = tid >> 3, dc = tid & 7;
      const u32x4 qv = *(const u32x4*)&qkv[dc * 4];
      const float scale = __uint_as_float(uni(__float_as_uint(s.scale))) * 1.4426950408889634f;
      const u32x4 kn = *(const u32x4*)&qkv[32 + dc * 4], vn = *(const u32x4*)&qkv[64 + dc * 4];
      float sc[CH_KU], mx = -INFINITY;
#pragma unroll
      for (int u = 0; u < CH_KU; ++u) {
        const int t = sp * CHAIN_KEYS + kg + 64 * u;
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) d = dot2(qv[e], t == lk - 1 ? kn[e] : kv[u][e], d);
        d = octet_sum(d);
        sc[u] = t < lk ? d * scale : -INFINITY;
        mx = fmaxf(mx, sc[u]);
      }
      mx = wave_max(mx);
      float l = 0.f, o[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < CH_KU; ++u) {
        const int t = sp * CHAIN_KEYS + kg + 64 * u;
        const float pr = t < lk ? __builtin_amdgcn_exp2f(sc[u] - mx) : 0.f;
        l += pr;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t vv = t == lk - 1 ? vn[e] : (t < lk ? kv[CH_KU + u][e] : 0u);
          o[2 * e] = fmaf(pr, lo_f(vv), o[2 * e]);
          o[2 * e + 1] = fmaf(pr, hi_f(vv), o[2 * e + 1]);
        }
      }
      // over the 8 key groups of the wave (lane bits 3 .. 5): every exchange adds two values' halves into one register,
      // so a lane ends with one of the 64 sums
      typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
      float h4[4], h2[2];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[e]), __float_as_uint(o[e + 4]), false, false);
        h4[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(h4[e]), __float_as_uint(h4[e + 2]), false, false);
        h2[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
      }
      ao[wave][dc * 8 + ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1)] =
          ((lane & 8) ? h2[1] : h2[0]) + dpp_move<0x128>(0.f, (lane & 8) ? h2[0] : h2[1]);
      l = add_halves(l + dpp_move<0x128>(0.f, l));
      if (lane == 0) { am[wave] = mx; al[wave] = l; }
      wg_barrier();
      if (wave == 0) {
        float m = am[0], ls = 0.f, os = 0.f;
#pragma unroll
        for (int v = 1; v < CH_WAVES; ++v) m = fmaxf(m, am[v]);
#pragma unroll
        for (int v = 0; v < CH_WAVES; ++v) {
          const float f = am[v] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(am[v] - m);
          ls = fmaf(al[v], f, ls);
          os = fmaf(ao[v][lane], f, os);
        }
        u64* out = a.mail + region(p) + id * CH_ATT;
        mail_store(out + lane, __float_as_uint(os), a.tag0 + p);
        if (lane < 2) mail_store(out + 64 + lane, __float_as_uint(lane ? ls : m), a.tag0 + p);
      }
    };

    auto phase = [&](int p) __attribute__((always_inline)) {
      const ChainStep& s = steps[p];
      const int kind = uni(s.kind);
      const Plan next = plan(p + CH_AHEAD);
      u32x4 cur[CH_U];
      take(p, cur);
      if (kind == CHAIN_ATTN) {
        const int id = uni(attn_part(s));
        if (id >= 0) attention(p, s, id, cur, next);
        else issue(next, p + CH_AHEAD);
        return;
      }
      if (kind == CHAIN_GATHER) {
        issue(next, p + CH_AHEAD);
        wg_barrier();
        return;
      }
      // everything of the table is in scalar registers before the row arrives: what follows the barrier is the critical path
      const int sh = uni(s.seg_shift), K = uni(s.k), rpw = uni(s.rpw), n = uni(s.n), res = uni(s.res), act1 = uni(s.act1), act2 = uni(s.act2);
      const bool has_bias = unip<bf16_t>(s.bias) != nullptr;
      const int out_ext = uni(s.out_ext), arg_ext = uni(s.arg_ext), rb = wave >> sh, rstep = CH_WAVES >> sh;
      const float scale = __uint_as_float(uni(__float_as_uint(s.scale)));
      const int k = (wave & ((1 << sh) - 1)) * 512 + lane * 8, row0 = wg * rpw + 2 * tid;
      const bool mine = 2 * tid < rpw && row0 < n;
      wg_barrier();
      u32x4 xv = *(const u32x4*)&xw[min(k, K - 8) >> 1];
      issue(next, p + CH_AHEAD);
      if (k >= K) xv = zero;
      auto dots = [&](int j0, const u32x4 (&h)[CH_U]) __attribute__((always_inline)) {
        float d[CH_U];
#pragma unroll
        for (int j = 0; j < CH_U; ++j) d[j] = dot2(xv[1], h[j][1], dot2(xv[0], h[j][0], 0.f)) + dot2(xv[3], h[j][3], dot2(xv[2], h[j][2], 0.f));
#pragma unroll
        for (int j = 0; j < CH_U; j += 4) {
          const float d4[4] = {d[j], d[j + 1], d[j + 2], d[j + 3]};
          const float t = wave_sum4(d4, lane);
          const int row = rb + rstep * (j0 + j + lane);
          if (lane < 4 && row < rpw) part[(row << sh) + (wave & ((1 << sh) - 1))] = t;
        }
      };
      if (p + 1 < n_steps) {                             // (one batch: checked when the table was made)
        dots(0, cur);
      } else {                                           // the last phase may be long; the other buffer is free
        const int J = (rpw + rstep - 1) / rstep;
        u32x4 other[CH_U];
        for (int j0 = 0; j0 < J; j0 += 2 * CH_U) {
          load_w(s, j0 + CH_U, other);
          dots(j0, cur);
          load_w(s, j0 + 2 * CH_U, cur);
          dots(j0 + CH_U, other);
        }
      }
      wg_barrier();
      if (wave * 128 < rpw) {                              // (the first wave; more of them only in a long last phase)
        float v0 = 0.f, v1 = 0.f;
        if (mine) {
          typedef float f32x4 __attribute__((ext_vector_type(4)));
          const f32x4* q = (const f32x4*)part;             // the segments of a row are neighbours: 2 << sh sums per lane
          if (sh == 1) {
            const f32x4 t = q[tid];
            v0 = t[0] + t[1];
            v1 = t[2] + t[3];
          } else if (sh == 3) {
            f32x4 t[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) t[c] = q[4 * tid + c];
            t[0] += t[1];
            t[2] += t[3];
            v0 = (t[0][0] + t[0][1]) + (t[0][2] + t[0][3]);
            v1 = (t[2][0] + t[2][1]) + (t[2][2] + t[2][3]);
          } else if (sh == 2) {
            const f32x4 t = q[2 * tid], u = q[2 * tid + 1];
            v0 = (t[0] + t[1]) + (t[2] + t[3]);
            v1 = (u[0] + u[1]) + (u[2] + u[3]);
          } else {
            v0 = part[2 * tid];
            v1 = part[2 * tid + 1];
          }
          const uint32_t b2 = has_bias ? biasw[p % CH_PAR][tid & 63] : 0u;      // (no bias where a workgroup has more than 128 rows)
          v0 = apply_act(v0 * scale + lo_f(b2), act1);
          v1 = apply_act(v1 * scale + hi_f(b2), act1);
          if (res >= 0) {
            const uint32_t r = own[res & (CH_RING - 1)][tid];
            v0 = apply_act(v0 + lo_f(r), act2);
            v1 = apply_act(v1 + hi_f(r), act2);
          }
          const uint32_t o = f2bf2(v0, v1);
          if (out_ext >= 0) *(uint32_t*)((bf16_t*)ext[out_ext] + row0) = o;
          else {
            mail_store(a.mail + region(p) + wg * CH_LINE + lane, o, a.tag0 + p);
            own[p & (CH_RING - 1)][lane] = o;
          }
          v0 = lo_f(o);
          v1 = hi_f(o);
        }
        if (arg_ext >= 0) {
          float bv = mine ? v0 : -INFINITY;
          int bi = mine ? row0 : 0x7fffffff;
          if (mine && v1 > bv) { bv = v1; bi = row0 + 1; }
          wave_argmax(bv, bi);
          if (lane < 2) mail_store(a.mail + region(p) + wg * CH_LINE + 2 * wave + lane, lane ? (uint32_t)bi : __float_as_uint(bv), a.tag0 + p);
        }
      }
    };

    {
      Plan f;
      plan_params(0, f);
      issue_params(f, 0);
    }
#pragma unroll
    for (int p = 0; p < CH_AHEAD; ++p) issue(plan(p), p);
    for (int p = 0; p < n_steps; ++p) {
      phase(p);
      if (p == 1 && uni(left)) break;                      // (words of a row that nobody reads have gone out, nothing else)
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // nothing of the ring is on its way when the workgroup ends
  }
  wg_barrier();
  if (tid == 0 && dead) __hip_atomic_store(a.error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------------
// the table's bytes ride in the kernel arguments (no copy engine, no host buffer that has to stay)
constexpr int CH_CHUNK = 3584;
struct ChainChunk { uint32_t w[CH_CHUNK / 4]; };
__global__ __launch_bounds__(256) void chain_table_kernel(uint32_t* dst, int words, ChainChunk c) {
  for (int i = threadIdx.x; i < words; i += 256) dst[i] = c.w[i];
}
__global__ __launch_bounds__(256) void chain_clear_kernel(u64* mail, long long n) {
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += 256ll * gridDim.x) mail[i] = 0;
}

constexpr int CH_TABLES = 8;       // sequences whose tables stay on the device; one more is uploaded again, 5 small launches a step (24 layers)
static __device__ __align__(256) u64 chain_mail[CH_RING * CH_REGION];
static __device__ __align__(256) ChainStep chain_tables[CH_TABLES][CHAIN_MAX_STEPS];
static __device__ __align__(256) unsigned chain_here[2][64];               // arrivals of this launch and the next
static __device__ __align__(256) uint32_t chain_rows[CH_RING * CH_ROW];

namespace {
struct ChainDevice {
  std::mutex mu;
  bool known = false;
  int n_cu = 0, owner = -1;                 // owner: the socket that holds the device's name, or -1
  std::chrono::steady_clock::time_point asked, again;      // asked for the name; when this kernel may be used again
  bool failed = false;
  u64* mail = nullptr;
  ChainStep* tables = nullptr;
  unsigned* here = nullptr;
  uint32_t* rows = nullptr;
  int turn = 0;                             // which count of arrivals the next launch takes
  unsigned* err_host = nullptr;
  unsigned* err_dev = nullptr;
  hipEvent_t last = nullptr;                // recorded behind the newest launch
  bool any = false;
  unsigned next_tag = 1;
  std::vector<ChainStep> held[CH_TABLES];   // what the device tables hold
  uint64_t used[CH_TABLES] = {}, clock = 0;
};
ChainDevice g_chain[64];

ChainDevice& chain_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) throw Error(SOD2_ERR_HIP, "current device could not be determined");
  return g_chain[dev];
}
void need(hipError_t e, const char* what) {
  if (e != hipSuccess) throw Error(SOD2_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}
// Addresses, a line of pinned memory and an event, once per device; false where they cannot be had (the groups run one by
// one then).  Another thread may be capturing a stream meanwhile, which forbids every thread calls like these unless it
// says that they are no part of the capture.
bool first_use(ChainDevice& d) {
  if (d.known) return true;
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  int dev = 0;
  void *mail = nullptr, *tables = nullptr, *here = nullptr, *rows = nullptr;
  bool ok = hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&d.n_cu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            hipGetSymbolAddress(&mail, HIP_SYMBOL(chain_mail)) == hipSuccess && hipGetSymbolAddress(&tables, HIP_SYMBOL(chain_tables)) == hipSuccess &&
            hipGetSymbolAddress(&here, HIP_SYMBOL(chain_here)) == hipSuccess && hipGetSymbolAddress(&rows, HIP_SYMBOL(chain_rows)) == hipSuccess;
  if (ok && !d.err_host) ok = hipHostMalloc((void**)&d.err_host, 64, hipHostMallocCoherent | hipHostMallocMapped) == hipSuccess;
  if (ok) ok = hipHostGetDevicePointer((void**)&d.err_dev, d.err_host, 0) == hipSuccess;
  if (ok && !d.last) ok = hipEventCreateWithFlags(&d.last, hipEventDisableTiming) == hipSuccess;
  if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (!ok) {
    (void)hipGetLastError();
    return false;
  }
  d.mail = (u64*)mail;
  d.tables = (ChainStep*)tables;
  d.here = (unsigned*)here;
  d.rows = (uint32_t*)rows;
  d.err_host[0] = d.err_host[1] = 0;
  d.known = true;
  return true;
}
}  // namespace

// Whether this process may run one-row steps as one kernel on the current device: it holds an abstract socket name (no
// file, gone with the process).  Asked again once a second while another process has it.  (Processes in different
// network namespaces do not see each other's names: their steps then meet, are called off and done by one workgroup, and
// both go on group by group for a while.)
static bool own_device(ChainDevice& d) {
  if (d.owner >= 0) return true;
  const auto now = std::chrono::steady_clock::now();
  if (d.asked.time_since_epoch().count() != 0 && now - d.asked < std::chrono::seconds(1)) return false;
  d.asked = now;
  int dev = 0;
  char bus[64] = {0};
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetPCIBusId(bus, sizeof bus, dev) != hipSuccess) return false;
  const std::string name = std::string("sod2-one-row-step-") + bus;
  sockaddr_un at{};
  at.sun_family = AF_UNIX;
  std::memcpy(at.sun_path + 1, name.data(), name.size());
  const int fd = socket(AF_UNIX, SOCK_DGRAM | SOCK_CLOEXEC, 0);
  if (fd < 0) return false;
  if (bind(fd, (const sockaddr*)&at, (socklen_t)(offsetof(sockaddr_un, sun_path) + 1 + name.size())) != 0) {
    close(fd);
    return false;
  }
  d.owner = fd;
  return true;
}

// a stream that may use only some of the CUs
static bool masked(hipStream_t s, int n_cu) {
  uint32_t mask[32] = {0};
  if (hipExtStreamGetCUMask(s, 32, mask) != hipSuccess) { (void)hipGetLastError(); return false; }
  int bits = 0;
  for (uint32_t m : mask) bits += __builtin_popcount(m);
  return bits > 0 && bits < n_cu;
}

// CUs of the current device: what a replay's table is dealt out to, whether the kernel can be had just now or not
int chain_cus() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return n;
}

// Workgroups a one-row step may have on stream s: one per CU, 0 where it is to be launched group by group.  Throws once
// if an earlier step could not be brought to its end.  (A stream of another device than the calling thread's current one
// launches kernels on its own device, where this device's exchange buffer and table have no business.)
int chain_workgroups(hipStream_t s) {
  if (!chain_takes(s)) return 0;
  if (s) {                                  // (the null stream is the current device's, with all its CUs)
    hipDevice_t of_stream = -1;
    int current = -2;
    if (hipStreamGetDevice(s, &of_stream) != hipSuccess || hipGetDevice(&current) != hipSuccess || of_stream != current) {
      (void)hipGetLastError();
      return 0;
    }
  }
  ChainDevice& d = chain_device();
  std::lock_guard<std::mutex> lock(d.mu);
  if (d.failed || !own_device(d) || !first_use(d)) return 0;
  if (__atomic_load_n(&d.err_host[0], __ATOMIC_RELAXED)) {
    d.failed = true;
    throw Error(SOD2_ERR_HIP, "an earlier one-row step waited too long for another workgroup: its logits are NaN, and what was computed from them "
                              "is not valid; such steps run group by group from now on");
  }
  const auto now = std::chrono::steady_clock::now();
  if (__atomic_exchange_n(&d.err_host[1], 0u, __ATOMIC_RELAXED)) d.again = now + std::chrono::seconds(CH_REST);
  return now < d.again || (s && masked(s, d.n_cu)) ? 0 : d.n_cu;
}

// One step on stream s.  ext: the caller's input and output pointers; lk: keys of the attention phases with lk_rel 0.
void chain_launch(const Chain& c, void* const* ext, int lk, hipStream_t s) {
  ChainDevice& d = chain_device();
  std::lock_guard<std::mutex> lock(d.mu);
  if (!d.known) throw Error(SOD2_ERR_HIP, "one-row step on a device that was not asked for one");
  // on the same stream too: a handle may by now be another stream's (destroyed and created again, or the per-thread one)
  if (d.any) need(hipStreamWaitEvent(s, d.last, 0), "ordering one-row steps of two streams");
  int slot = -1, oldest = 0;
  const size_t bytes = c.steps.size() * sizeof(ChainStep);
  for (int i = 0; i < CH_TABLES; ++i) {
    if (d.held[i].size() == c.steps.size() && std::memcmp(d.held[i].data(), c.steps.data(), bytes) == 0) slot = i;
    if (d.used[i] < d.used[oldest]) oldest = i;
  }
  if (slot < 0) {
    slot = oldest;                          // (launches run one after the other: nothing reads the old table any more)
    for (size_t at = 0; at < bytes; at += CH_CHUNK) {
      ChainChunk ch;
      const size_t n = std::min<size_t>(CH_CHUNK, bytes - at);
      std::memcpy(ch.w, (const char*)c.steps.data() + at, n);
      hipLaunchKernelGGL(chain_table_kernel, dim3(1), dim3(256), 0, s, (uint32_t*)((char*)(d.tables + (size_t)slot * CHAIN_MAX_STEPS) + at), (int)(n / 4), ch);
    }
    need(hipGetLastError(), "step table");
    d.held[slot] = c.steps;
  }
  d.used[slot] = ++d.clock;
  if (d.next_tag > 0xffffffffu - 2 * CHAIN_MAX_STEPS) {    // the tags start over: no word may carry an old one
    hipLaunchKernelGGL(chain_clear_kernel, dim3(256), dim3(256), 0, s, d.mail, (long long)CH_RING * CH_REGION);
    need(hipGetLastError(), "exchange buffer");
    d.next_tag = 1;
  }
  ChainArgs a;
  a.steps = d.tables + (size_t)slot * CHAIN_MAX_STEPS;
  a.mail = d.mail;
  a.here = d.here + 64 * d.turn;
  a.here_next = d.here + 64 * (d.turn ^ 1);
  a.rows = d.rows;
  a.error = d.err_dev;
  a.arrive = 100u * (unsigned)(c.arrive_us >= 0 ? c.arrive_us : CH_ARRIVE);
  a.polls = (unsigned)(c.polls >= 0 ? c.polls : CH_POLLS);
  for (int i = 0; i < CHAIN_MAX_EXT; ++i) a.ext[i] = i < c.n_ext ? (char*)ext[i] : nullptr;
  a.n_steps = (int)c.steps.size();
  a.lk = lk;
  a.tag0 = d.next_tag;
  d.next_tag += (unsigned)c.steps.size();
  hipLaunchKernelGGL(chain_kernel, dim3(c.workgroups), dim3(CH_THREADS), 0, s, a);
  need(hipGetLastError(), "one-row step");
  d.turn ^= 1;                              // (a launch that failed has counted nobody in)
  need(hipEventRecord(d.last, s), "one-row step");
  d.any = true;
}

// the rows that go to the caller's buffers are written two values at a time
bool chain_fits(const Chain& c, void* const* ext) {
  for (const ChainStep& s : c.steps)
    if (s.out_ext >= 0 && ((uintptr_t)ext[s.out_ext] & 3)) return false;
  return true;
}

// Whether the launches of one step form a chain this kernel can run, and its table.  `at` resolves weight and arena
// references; lk_grows: keys that later launches of the same table may add.
bool chain_build(const std::vector<Launch>& launches, int n_in, int n_out, const std::function<void*(const Ref&)>& at, int n_cu, int lk_grows,
                 Chain* out) {
  if (n_in + n_out > CHAIN_MAX_EXT) return false;
  struct Where { Ref ref; int64_t bytes; };
  std::vector<ChainStep> st;
  std::vector<Where> where;                  // storage each phase stands for
  auto ext_of = [&](const Ref& r) { return r.byte_off != 0 ? -1 : (r.space == SP_INPUT ? r.index : (r.space == SP_OUTPUT ? n_in + r.index : -1)); };
  auto same = [](const Ref& a, const Ref& b) { return a.space == b.space && a.index == b.index && a.byte_off == b.byte_off; };
  // the phase whose result is at r: the newest that touches that storage, and exactly it
  auto phase_at = [&](const Ref& r, int64_t bytes) {
    for (int q = (int)st.size() - 1; q >= 0; --q) {
      const Where& w = where[q];
      if (w.ref.space != r.space || w.ref.index != r.index) continue;
      if (w.ref.byte_off + w.bytes <= r.byte_off || r.byte_off + bytes <= w.ref.byte_off) continue;
      return same(w.ref, r) && w.bytes == bytes ? q : -1;
    }
    return -1;
  };
  auto al = [](const void* p, int n) { return ((uintptr_t)p & (n - 1)) == 0; };
  int lk0 = -1;
  for (size_t i = 0; i < launches.size(); ++i) {
    const Launch& L = launches[i];
    ChainStep s;
    std::memset(&s, 0, sizeof s);
    s.src = s.res = s.out_ext = s.arg_ext = s.idx_ext = s.idx2_ext = -1;
    s.scale = 1.f;
    if (L.empty) return false;
    if (L.kernel == K_GATHER) {
      const GatherArgs& g = L.u.gather;
      s.kind = CHAIN_GATHER;
      s.n = g.cols;
      s.w = at(L.r[0]);
      s.idx_ext = ext_of(L.r[1]);
      s.idx_i32 = g.idx_i32;
      s.table_rows = g.table_rows;
      if (g.rows != 1 || L.in_dtype != SOD2_BF16 || s.idx_ext < 0 || L.r[0].space != SP_WEIGHT || L.r[2].space != SP_ARENA || !al(s.w, 4) || g.cols % 2) return false;
      if (L.r[3].space != SP_NONE) {         // + the row gathered just before
        if (st.size() != 1 || st[0].kind != CHAIN_GATHER || st[0].bias || phase_at(L.r[3], 2ll * g.cols) != 0) return false;
        s.bias = st[0].w;
        s.idx2_ext = st[0].idx_ext;
        s.idx2_i32 = st[0].idx_i32;
        s.table2_rows = st[0].table_rows;
        st.clear();
        where.clear();
      }
      if (!st.empty() && L.r[3].space == SP_NONE) return false;
      st.push_back(s);
      where.push_back({L.r[2], 2ll * g.cols});
      continue;
    }
    if (L.kernel == K_GEMM) {
      const GemmArgs& g = L.u.gemm;
      const bool ln = L.r[5].space != SP_NONE;
      s.kind = CHAIN_GEMV;
      s.n = g.N; s.k = g.K; s.ldw = (int)g.b_sn;
      s.w = at(L.r[1]);
      s.bias = L.r[3].space == SP_NONE ? nullptr : at(L.r[3]);
      s.gamma = ln ? at(L.r[5]) : nullptr;
      s.beta = ln ? at(L.r[6]) : nullptr;
      s.eps = g.ln_eps; s.scale = g.scale; s.act1 = g.act1; s.act2 = g.act2;
      if (g.M != 1 || g.nb0 * g.nb1 != 1 || L.in_dtype != SOD2_BF16 || L.out_dtype != SOD2_BF16 || g.a_sk != 1 || g.b_sk != 1 || g.c_sn != 1 ||
          g.K % 8 || g.K > CHAIN_MAX_K || (ln && g.K > 1024) || g.b_sn % 8 || g.b_sn > (1 << 20) || g.N % 2 || L.post_ln || L.fold_read ||
          L.r[1].space != SP_WEIGHT || !al(s.w, 16) || !al(s.bias, 4) || !al(s.gamma, 16) || !al(s.beta, 16))
        return false;
      // (up to 1024 rows of a workgroup, 2 bytes an element: offsets stay within 32 bits)
      while ((512 << s.seg_shift) < g.K) ++s.seg_shift;
      if (st.empty()) return false;          // (a chain starts with an embedding row)
      s.src = (int)st.size() - 1;
      if (phase_at(L.r[0], 2ll * g.K) != s.src || st[s.src].out_ext >= 0) return false;
      if (ln && st[s.src].kind == CHAIN_ATTN) return false;      // (its parameters are asked for in the phase before)
      if (L.r[4].space != SP_NONE) {
        if (g.r_sn != 1) return false;
        s.res = phase_at(L.r[4], 2ll * g.N);
        if (s.res < 0 || st[s.res].kind == CHAIN_ATTN || st[s.res].out_ext >= 0 || s.src - s.res > CH_RING / 2) return false;
      }
      if (L.r[2].space == SP_OUTPUT) {
        s.out_ext = ext_of(L.r[2]);
        if (s.out_ext < 0) return false;
      } else if (L.r[2].space != SP_ARENA) {
        return false;
      }
      st.push_back(s);
      where.push_back({L.r[2], 2ll * g.N});
      continue;
    }
    if (L.kernel == K_ATTENTION) {
      const AttnArgs& t = L.u.attn;
      if (st.empty() || t.Lq != 1 || t.n_new != 1 || t.nb0 != 1 || t.q_sb1 != 64 || t.k_sb1 != 64 || t.v_sb1 != 64 || t.o_sb1 != 64) return false;
      s.kind = CHAIN_ATTN;
      s.src = (int)st.size() - 1;
      s.n = t.nb1;
      s.w = at(L.r[1]);
      s.bias = at(L.r[2]);
      s.ldw = t.nb1 * 64;                    // (the stride of a single cached row carries no meaning)
      if (t.Lk > 1 && (t.k_sn != s.ldw || t.v_sn != s.ldw)) return false;
      s.scale = t.scale;
      const Where& w = where[s.src];
      int* offs[3] = {&s.q_off, &s.k_off, &s.v_off};
      const Ref* refs[3] = {&L.r[0], &L.r[4], &L.r[5]};
      for (int k = 0; k < 3; ++k) {
        const int64_t off = refs[k]->byte_off - w.ref.byte_off;
        if (refs[k]->space != SP_ARENA || w.ref.space != SP_ARENA || off < 0 || off % 4 || off + t.nb1 * 128ll > w.bytes) return false;
        *offs[k] = (int)(off / 2);
      }
      if (st[s.src].kind != CHAIN_GEMV || L.r[1].space != SP_ARENA || L.r[2].space != SP_ARENA || L.r[3].space != SP_ARENA || !al(s.w, 16) || !al(s.bias, 16)) return false;
      if (lk0 < 0) lk0 = t.Lk;
      s.lk_rel = t.Lk - lk0;
      if (s.lk_rel != 0) return false;
      st.push_back(s);
      where.push_back({L.r[3], t.nb1 * 128ll});
      continue;
    }
    if (L.kernel == K_ARGMAX) {
      const ArgmaxArgs& g = L.u.argmax;
      if (st.empty() || st.back().kind != CHAIN_GEMV || st.back().out_ext < 0 || i + 1 != launches.size() || g.rows != 1 || g.cols != st.back().n ||
          !same(L.r[0], where.back().ref) || L.r[1].space != SP_OUTPUT || ext_of(L.r[1]) < 0)
        return false;
      st.back().arg_ext = ext_of(L.r[1]);
      st.back().arg_i32 = g.out_i32;
      continue;
    }
    return false;
  }
  if (st.size() < 8 || st.size() > (size_t)CHAIN_MAX_STEPS || st.back().out_ext < 0 || lk0 < 0) return false;   // (short chains: nothing to gain)
  // as many workgroups as the chip has CUs and every exchanged row deals out to in whole pairs; every workgroup then has
  // a part in every contraction, which bounds how far one can fall behind another to two phases: a region of the
  // exchange buffer (written again CH_RING phases later) is read by then (residuals reach back CH_RING / 2 at most)
  for (int nwg = n_cu / 64 * 64; nwg >= 64; nwg -= 64) {
    if (nwg > CHAIN_MAX_WG) continue;
    bool ok = true;
    for (size_t p = 0; p < st.size() && ok; ++p) {
      ChainStep& s = st[p];
      if (s.kind == CHAIN_ATTN) {
        ok = s.n * ((lk0 + lk_grows + CHAIN_KEYS - 1) / CHAIN_KEYS) <= nwg;
        continue;
      }
      s.rpw = ((s.n + nwg - 1) / nwg + 1) / 2 * 2;
      const bool last = p + 1 == st.size();
      if (!last) ok = s.rpw * nwg == s.n && s.rpw / 2 <= CH_LINE;
      ok = ok && s.rpw <= (last && !s.bias ? CH_WAVES * 128 : 128) && (s.kind == CHAIN_GATHER || s.rpw << s.seg_shift <= CH_PART);
      if (s.kind == CHAIN_GEMV && !last) ok = ok && s.rpw <= CH_U * (CH_WAVES >> s.seg_shift);
    }
    for (size_t p = 0; p + 1 < st.size() && ok; ++p)      // no two attention phases in a row (each follows its contraction)
      if (st[p].kind == CHAIN_ATTN && st[p + 1].kind != CHAIN_GEMV) ok = false;
    if (!ok) continue;
    out->steps = st;
    out->workgroups = nwg;
    out->n_ext = n_in + n_out;
    out->lk0 = lk0;
    return true;
  }
  return false;
}

}  // namespace sod2
