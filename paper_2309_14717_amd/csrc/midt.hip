// Adapter-free forward between the few-token kernels and the tiles of the dense one: up to 64 tokens
// (batched decoding, short prompts), every code width.
//
//   y = x . W~,   W~[i,j] = alpha[i/g,j] * code[i,j] + beta[i/g,j]      (Eq. 1 per group, Sec. 3.3)
//
// Operands and precision are the dense kernel's: x as fp16 rows at a power-of-two scale, W~ rebuilt
// around the mid code from two fp16 factors per (group, column) at a power-of-two scale, fp32
// accumulation.  What differs is where the work happens:
//   * W~ never passes through LDS.  A lane's operand of v_mfma_f32_16x16x32_f16 is eight consecutive
//     rows of one column -- one packed word of 4-bit codes -- so the lane that loads the word
//     rebuilds the operand in its own registers and uses it for every token tile.
//   * The fp16 factors are made here from alpha and beta (fp32 planes, fp16 pairs or the deployment
//     stream), so there is no factor launch and no second trip of the factors through memory.
//     The scale of a column is kept by the wavefront: it starts from the first groups it meets,
//     whose bound it brings where the factor job brings the whole column's, to [2^13, 2^14); should a
//     later group exceed 2^15 the accumulators of that column are rescaled (by a power of two:
//     exact).  No column's scale has to be known before, and none ends below the factor job's.
// What bounds it: the weight's bytes (135 MB of 8192 x 22016 at g = 32 are 25 us) and the issue time
// of the SIMDs, on which matrix and vector instructions take turns: per 16 columns x 32 rows 60
// cycles of rebuilding whatever the token count and 16 per sixteen tokens (20 us at 64 tokens).  The two add up: a
// wavefront has one unit of weights in flight, and x is staged again for every slab (180 MB beside the 135).  Counters
// at that size: 160 MB fetched, matrix cores busy for 19 % and vector instructions issued for 32 % of 47 us.  (A form with exact
// integer codes and alpha applied to the sums spends 24 more cycles per sixteen tokens and took
// 4.4 us instead of 2.8 per 256 x 256 weights at 64 tokens; beyond 64 tokens the dense kernel, which
// rebuilds a weight once for 256 rows, is the better one.)
//
// Decomposition.  A block of eight wavefronts owns a slab of 128 columns (64 per wavefront) for a run of
// units: 512 rows, a 128-row chunk per pair of wavefronts, whose sums meet in LDS at the end.  All
// (slab, unit) are laid out slab by slab and cut into equal runs, one per block, whatever the shape: a
// run may end one slab and begin the next.  A block works on its LAST slab first: what it cannot finish
// it publishes early (fp32 partial and a flag), and the slab whose end it holds comes last; it adds the
// partials of the blocks before it in their order and writes y.  (Slabs of 256 columns and 256 rows have
// twice the parts, each twice the size, for half as many blocks to add: 64 tokens of 22016 x 8192 took
// 55.4 us with them, 50 with these, 86 on the dense kernel with its factor launch.)  Waits are on
// lower-numbered blocks only and bounded (a wait that runs out gives NaN outputs and sets the
// workspace's status word); every order of summation is fixed by the shape.
// x goes through LDS by LDS-DMA, double-buffered, its 16-byte pieces XOR-swizzled by the token so
// that operand reads are conflict free.
#include <atomic>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "midt_plan.hpp"

namespace qalora {

namespace {

constexpr int MT_WAVES = 8;
constexpr int MT_THREADS = 64 * MT_WAVES;
constexpr uint32_t MT_SPIN_LIMIT = 1u << 18;  // bounded wait: the kernel always terminates
constexpr uint32_t kMtOob = 0xffff0000u;      // beyond every buffer: the range check returns zero
constexpr int MT_NT = 2;                      // cache policy "nontemporal": streamed once

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t mt_rsrc(const void* base, size_t bytes) {
  const uint32_t n = bytes > 0xffffffffull ? 0xffffffffu : (uint32_t)bytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)n, 0x00020000);
}
// LDS-only barrier: does not wait for the global loads that are in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int I, int N, typename Fn>
__device__ __forceinline__ void static_for(Fn&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Where alpha and beta come from
constexpr int FAC_F32 = 0;  // two fp32 planes [L, d_out]
constexpr int FAC_F16 = 1;  // one plane of words fp16 alpha | fp16 beta << 16
constexpr int FAC_DEP = 2;  // the factor units of the deployment stream (4-bit codes)

// Power of two that brings a bound m to [2^13, 2^14) (one for m = 0 or a non-finite m), as in the factor
// job; the limit above which a column is rescaled leaves fp16's largest value a factor of two away.
constexpr float kScaledLimit = 0x1p15f;
__device__ __forceinline__ float column_scale(float m) {
  const int E = (int)(__float_as_uint(m) >> 23) & 255;
  if (m == 0.0f || E == 255) return 1.0f;
  int e = 140 - E;
  e = e > 100 ? 100 : (e < -100 ? -100 : e);
  return __uint_as_float((uint32_t)(127 + e) << 23);
}
// 1 / s of a power of two s in [2^-100, 2^100]
__device__ __forceinline__ float inverse_pow2(float s) { return __uint_as_float((254u << 23) - __float_as_uint(s)); }

// Calls f with the x buffer the LDS-DMA is filling and the one being read as restrict-qualified
// pointers: they never overlap, and saying so keeps the compiler from draining the loads in front
// of every LDS read.
template <typename F>
__device__ __forceinline__ void with_x_buffers(unsigned char* __restrict__ dma, const unsigned char* __restrict__ rd, F&& f) {
  f(dma, rd);
}

}  // namespace

// TT: token tiles of sixteen
template <int NBITS, int FAC, int TT>
__global__ __launch_bounds__(MT_THREADS) void midt_kernel(const MidTArgs p) {
  static_assert(FAC != FAC_DEP || NBITS == 4, "the deployment stream holds 4-bit codes");
  constexpr int XCHUNK = TT * 16 * 256;    // bytes of one chunk of x
  constexpr int XBUF = MT_DEEP * XCHUNK;
  extern __shared__ __align__(16) unsigned char lds[];  // x [2][XBUF]
  __shared__ int poison;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, kb = lane >> 4;
  const int cg = wave & 1, deep = wave >> 1;
  const int C = p.d_in / 128;                    // chunks per slab
  const int CU = ceil_div(C, MT_DEEP);           // units per slab
  const int S = ceil_div(p.d_out, MT_SLAB);      // slabs
  const int L = p.d_in / p.group;
  const int sub_sh = p.group == 32 ? 0 : (p.group == 64 ? 1 : 2);  // log2 of 32-row steps per group
  const int ng = 4 >> sub_sh;                    // groups per chunk
  const int nb = gridDim.x, b = blockIdx.x;
  const int units = S * CU;
  auto run_begin = [&](int blk) { return (int)((unsigned)units * (unsigned)blk / (unsigned)nb); };  // below 2^31: checked on the host
  const int u0 = run_begin(b), u1 = run_begin(b + 1);
  const int s_first = u0 / CU, c_first = u0 - s_first * CU;
  const int s_last = (u1 - 1) / CU;
  if (tid == 0) poison = 0;

  const __amdgpu_buffer_rsrc_t rs_w = mt_rsrc(p.plane0, plane0_words(NBITS, p.d_in, p.d_out) * 4);
  const __amdgpu_buffer_rsrc_t rs_h = mt_rsrc(p.plane1, plane1_words(NBITS, p.d_in, p.d_out) * 4);
  const __amdgpu_buffer_rsrc_t rs_x = mt_rsrc(p.x16, (size_t)round_up(p.T, 256) * p.d_in * 2);
  const size_t fac_bytes = (size_t)L * p.d_out * 4;
  const int dep_units = sub_sh == 0 ? 6 : 5;
  const int cols64 = ceil_div(p.d_out, 64);
  const __amdgpu_buffer_rsrc_t rs_al =
      FAC == FAC_DEP ? mt_rsrc(p.stream, (size_t)cols64 * C * dep_units * 1024)
                     : mt_rsrc(FAC == FAC_F16 ? (const void*)p.fac16 : (const void*)p.alpha, fac_bytes);
  const __amdgpu_buffer_rsrc_t rs_be = mt_rsrc(p.beta, FAC == FAC_F32 ? fac_bytes : 0);
  const uint32_t row_b = (uint32_t)p.d_out * 4u;
  constexpr float mid = code_center<NBITS>();

  // extraction constants held in registers (see patch_code_pair_f16)
  uint32_t dq_mask = patch_code_mask<NBITS>(), dq_magic = 0x64006400u;
  if constexpr (NBITS != 3) {
    asm volatile("s_mov_b32 %0, %1" : "=s"(dq_mask) : "n"(patch_code_mask<NBITS>()));
    asm volatile("v_mov_b32 %0, 0x64006400" : "=v"(dq_magic));
  }
  const f32x4 zero4 = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // ---- the weight of a unit: lane (n, kb) has columns 4 n .. 4 n + 3 of the wavefront's 64 and, per
  // 32-row step, the rows 8 kb .. 8 kb + 7.  Positions past the matrix read zeros.
  u32x4 cw[4];
  uint32_t chi[NBITS == 3 ? 4 : 1];  // 3 bits: the high-bit word of column 4 n + kb
  u32x4 fa, fb;
  struct Pos {  // slab, unit inside it, end of the segment
    int s, c, ce;
  };
  const int jw = cg * 64 + 4 * n;
  auto load_step = [&](auto st_c, const Pos& q) {
    constexpr int st = decltype(st_c)::value;
    const int c = MT_DEEP * q.c + deep, j0 = q.s * MT_SLAB + jw;
    const bool live = c < C;
    constexpr uint32_t RPW = NBITS == 4 ? 4 : 2;  // plane-0 words per column and step
    const uint32_t vw = live && j0 < p.d_out ? (uint32_t)(NBITS == 4 ? kb : kb >> 1) * row_b + 4u * (uint32_t)j0 : kMtOob;
    const uint32_t cs = (uint32_t)(4 * min(c, C - 1) + st);
    cw[st] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, (int)vw, (int)(RPW * cs * row_b), MT_NT);
    if constexpr (NBITS == 3) {
      const uint32_t vh = live && j0 + kb < p.d_out ? 4u * (uint32_t)(j0 + kb) : kMtOob;
      chi[st] = __builtin_amdgcn_raw_buffer_load_b32(rs_h, (int)vh, (int)(cs * row_b), MT_NT);
    }
  };
  constexpr int NLOADS = (NBITS == 3 ? 8 : 4) + (FAC == FAC_F16 ? 1 : 2);  // of a unit, factors included
  // Factors of the unit's chunk.  Planes: lane (n, kb) takes group kb of its four columns.  Deployment
  // stream: all groups of column 4 n + kb (a record keeps a column's factors together).
  auto load_fac = [&](const Pos& q) {
    const int c = MT_DEEP * q.c + deep, j0 = q.s * MT_SLAB + jw;
    const bool live = c < C;
    const int cc = min(c, C - 1);
    if constexpr (FAC == FAC_DEP) {
      const int j = j0 + kb;
      const bool ok = live && j < p.d_out;
      const uint32_t v = ((uint32_t)cc * (uint32_t)cols64 + (uint32_t)(j >> 6)) * (uint32_t)(dep_units * 1024) + 4096u +
                         16u * (uint32_t)(j & 63);
      fa = __builtin_amdgcn_raw_buffer_load_b128(rs_al, (int)(ok ? v : kMtOob), 0, MT_NT);
      fb = __builtin_amdgcn_raw_buffer_load_b128(rs_al, (int)(ok && sub_sh == 0 ? v + 1024u : kMtOob), 0, MT_NT);
    } else {
      const uint32_t v = live && j0 < p.d_out && kb < ng ? (uint32_t)kb * row_b + 4u * (uint32_t)j0 : kMtOob;
      const uint32_t so = (uint32_t)(ng * cc) * row_b;
      fa = __builtin_amdgcn_raw_buffer_load_b128(rs_al, (int)v, (int)so, MT_NT);
      if constexpr (FAC == FAC_F32) fb = __builtin_amdgcn_raw_buffer_load_b128(rs_be, (int)v, (int)so, MT_NT);
    }
  };

  // ---- x: a wavefront's LDS-DMA load k fills 1 KB block 8 k + wave of the buffer = four token rows of one
  // chunk; lane i lands at byte 16 i of it, so it fetches the piece the swizzle (slot ^ token) puts
  // there.  (Row numbers count through the unit's chunks: 16 TT rows each.)
  auto load_x = [&](unsigned char* dst, const Pos& q) {
#pragma unroll
    for (int k = 0; k < 2 * TT; ++k) {
      const int r0 = 4 * (8 * k + wave), xc = r0 / (16 * TT), row = r0 - xc * (16 * TT) + (lane >> 4);
      const int c = min(MT_DEEP * q.c + xc, C - 1);  // (absent chunks of a slab's last unit: unused)
      const uint32_t off = (uint32_t)row * (uint32_t)p.d_in * 2u + 16u * (uint32_t)((lane & 15) ^ (row & 15));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void*)(dst + (8 * k + wave) * 1024),
                                               16, (int)off, (int)((uint32_t)c * 256u), 0, 0);
    }
  };
  const int x_lane = deep * XCHUNK + n * 256;

  f32x4 acc[TT][4];
  float sc[4];  // scale of the lane's columns 4 n + q (the same in all four lane groups)
  auto clear = [&]() {
    static_for<0, TT>([&](auto t) {
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[decltype(t)::value][q] = zero4;
    });
#pragma unroll
    for (int q = 0; q < 4; ++q) sc[q] = 0x1p100f;
  };
  clear();

  // A segment is complete: the four chunks' sums meet (in chunk order), pair `deep` of the wavefronts
  // finishing token tile `deep`; then publish, or finish the slab.  `area` is XBUF bytes of LDS nobody
  // uses now.
  auto flush = [&](int s, int ce, unsigned char* area) {
    const bool whole = s != s_first || c_first == 0;  // the segment starts at the slab's first unit
    int ftid = tid & 127;  // opaque: the addresses below are made when needed, not held across the units
    asm volatile("" : "+v"(ftid));
    static_for<0, TT>([&](auto t) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float inv = inverse_pow2(sc[q]);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[decltype(t)::value][q][r] *= inv;
      }
    });
    f32x4* ex = reinterpret_cast<f32x4*>(area);  // [tile of the round][chunk][q][128]; a tile's own pair keeps its sums
    constexpr int FIT0 = XBUF / (MT_DEEP * 4 * 128 * 16), FIT = FIT0 < TT ? FIT0 : TT;  // tiles per round
    static_assert(FIT >= 1, "a tile's sums fit");
    f32x4 sum[4];
    static_for<0, (TT + FIT - 1) / FIT>([&](auto rd_c) {
      constexpr int lo = decltype(rd_c)::value * FIT, hi = lo + FIT < TT ? lo + FIT : TT;
      static_for<lo, hi>([&](auto t) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          ex[(((decltype(t)::value - lo) * MT_DEEP + deep) * 4 + q) * 128 + ftid] = acc[decltype(t)::value][q];
      });
      lds_barrier();
      if (deep >= lo && deep < hi) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          sum[q] = ex[((deep - lo) * MT_DEEP * 4 + q) * 128 + ftid];
#pragma unroll
          for (int k = 1; k < MT_DEEP; ++k) sum[q] += ex[(((deep - lo) * MT_DEEP + k) * 4 + q) * 128 + ftid];
        }
      }
      lds_barrier();
    });
    constexpr uint32_t kBlockBytes = TT * 4 * 128 * 16;
    const __amdgpu_buffer_rsrc_t rs_p = mt_rsrc(p.partial, (size_t)nb * kBlockBytes);
    const uint32_t p_off = deep < TT ? (uint32_t)(deep * 4 * 128 + ftid) * 16u : kMtOob;  // + q * 2 KB
    if (ce < CU) {
      if (deep < TT) {
        const __amdgpu_buffer_rsrc_t own = own_partial(p.partial, b, kBlockBytes);
#pragma unroll
        for (int q = 0; q < 4; ++q) store_partial(own, __builtin_bit_cast(u32x4, sum[q]), p_off + (uint32_t)q * 2048u);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // every store of this wavefront has landed
      __syncthreads();
      if (tid == 0) __hip_atomic_store(p.flags + b, p.nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    bool bad = false;
    if (!whole) {
      int bf = b - 1;  // first block with units of this slab
      while (run_begin(bf) > s * CU) --bf;
      for (int i = bf + tid; i < b; i += MT_THREADS) {
        uint32_t spins = 0;
        bool timed_out = false;
        while (__hip_atomic_load(p.flags + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != p.nonce) {
          if (++spins > MT_SPIN_LIMIT) {
            poison = 1;
            timed_out = true;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
        // consumed: cleared, so that a replay of a captured launch waits for its own producers
        if (!timed_out)
          __hip_atomic_store(p.flags + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
          __hip_atomic_store(p.status, p.nonce | 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      bad = poison != 0;
      f32x4 tot[4] = {zero4, zero4, zero4, zero4};
      constexpr int PB = 8;  // producers whose loads are in flight together
#pragma nounroll
      for (int i0 = bf; i0 < b; i0 += PB) {
        u32x4 v[PB][4];
#pragma unroll
        for (int i = 0; i < PB; ++i) {
          const uint32_t off = i0 + i < b ? p_off : kMtOob;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            v[i][q] = __builtin_amdgcn_raw_buffer_load_b128(
                rs_p, (int)off, (int)((uint32_t)min(i0 + i, b) * kBlockBytes + (uint32_t)q * 2048u), kDeviceCoherent);
        }
#pragma unroll
        for (int i = 0; i < PB; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) tot[q] += __builtin_bit_cast(f32x4, v[i][q]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) sum[q] = tot[q] + sum[q];
    }
    const int f_n = ftid & 15, f_kb = (ftid >> 4) & 3;
    const int j0 = s * MT_SLAB + (ftid >> 6) * 64 + 4 * f_n;
    if (deep < TT && j0 < p.d_out) {
      float inv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) inv[r] = p.row_scale[min(16 * deep + 4 * f_kb + r, p.T - 1)].y;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int tok = 16 * deep + 4 * f_kb + r;
        if (tok < p.T) {
          const float iv = bad ? __builtin_nanf("") : inv[r];  // a wait ran out: make it loud
          const f32x4 v = {sum[0][r] * iv, sum[1][r] * iv, sum[2][r] * iv, sum[3][r] * iv};
          const size_t o = (size_t)tok * p.d_out + j0;
          if (p.out_bf16)
            *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(p.out) + o) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
          else
            *reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + o) = v;
        }
      }
    }
  };

  // One unit.  Its codes and factors are replaced by the next unit's (n1; clamped at the end of the run:
  // loaded again, unused) as soon as they are used, the codes step by step -- a unit is 2 us and
  // more of work, long enough for them to land.  x of the next unit goes to the other buffer.
  auto unit = [&](unsigned char* x_rd, unsigned char* x_dma, const Pos& at, const Pos& n1) {
    with_x_buffers(x_dma, x_rd, [&](unsigned char* dma, const unsigned char* rd) {
      load_x(dma, n1);
      __builtin_amdgcn_sched_barrier(0);
      const bool live = MT_DEEP * at.c + deep < C;
      // fp16 factor words fp16(alpha S) | fp16((beta + mid alpha) S) << 16, four per lane: element e is
      // group kb, column 4 n + e (planes) or the group of step e, column 4 n + kb (stream)
      uint32_t fw[4];
      {
        float al[4], be[4], cst[4], bound[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if constexpr (FAC == FAC_F16) {
            al[e] = (float)__builtin_bit_cast(_Float16, (uint16_t)(fa[e] & 0xffffu));
            be[e] = (float)__builtin_bit_cast(_Float16, (uint16_t)(fa[e] >> 16));
          } else {
            al[e] = __uint_as_float(fa[e]);
            be[e] = __uint_as_float(fb[e]);
          }
        }
        if constexpr (FAC == FAC_DEP) {  // a factor per step; group 64: alpha0 alpha1 beta0 beta1; 128: alpha beta - -
          if (sub_sh == 1) {
            be[0] = be[1] = al[2], be[2] = be[3] = al[3], al[2] = al[3] = al[1], al[1] = al[0];
            asm volatile("" : "+v"(be[0]));  // (a branch, not selects)
          } else if (sub_sh == 2) {
            be[0] = be[1] = be[2] = be[3] = al[1], al[1] = al[2] = al[3] = al[0];
            asm volatile("" : "+v"(be[0]));
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          cst[e] = __builtin_fmaf(mid, al[e], be[e]);
          bound[e] = __builtin_fmaf(mid, fabsf(al[e]), fabsf(cst[e]));
          // Values are complete before their registers are reloaded (here and below): were any use of the old
          // contents left behind a load, the new ones would land elsewhere and be copied back at the
          // end of the loop -- and the copy waits for every load in flight.
          asm volatile("" : "+v"(al[e]), "+v"(cst[e]), "+v"(bound[e]));
        }
        __builtin_amdgcn_sched_barrier(0);
        load_fac(n1);
        __builtin_amdgcn_sched_barrier(0);
        float own[4];  // the scales that go with the lane's four elements
        auto own_scales = [&]() {
          float lo = sc[0], hi = sc[2];
          if constexpr (FAC == FAC_DEP) {
            lo = (kb & 1) ? sc[1] : sc[0];
            hi = (kb & 1) ? sc[3] : sc[2];
            asm volatile("" : "+v"(lo), "+v"(hi));  // (two selects: merged into one they index an array in scratch memory)
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) own[e] = FAC == FAC_DEP ? ((kb & 2) ? hi : lo) : sc[e];
        };
        own_scales();
        bool over = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) over |= bound[e] * own[e] > kScaledLimit;
        if (__any(over)) {  // first unit of a segment, or a group beyond all before it
          float m[4];  // this chunk's bound of columns 4 n + q
          if constexpr (FAC == FAC_DEP) {
            const float mo = fmaxf(fmaxf(bound[0], bound[1]), fmaxf(bound[2], bound[3]));
#pragma unroll
            for (int q = 0; q < 4; ++q) m[q] = __shfl(mo, n + 16 * q, 64);
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              m[q] = fmaxf(bound[q], __shfl_xor(bound[q], 16, 64));
              m[q] = fmaxf(m[q], __shfl_xor(m[q], 32, 64));
            }
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float ns = m[q] * sc[q] > kScaledLimit ? column_scale(m[q]) : sc[q];
            const float ratio = ns * inverse_pow2(sc[q]);
            sc[q] = ns;
            static_for<0, TT>([&](auto t_c) {
#pragma unroll
              for (int r = 0; r < 4; ++r) acc[decltype(t_c)::value][q][r] *= ratio;
            });
          }
          own_scales();
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f32x2 v = {al[e] * own[e], cst[e] * own[e]};
          fw[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
        }
      }
      // the factor words of a step's columns (and, 3 bits, its high-bit words), handed round one step ahead
      uint32_t fwd[2][4], hw[2][NBITS == 3 ? 4 : 1];
      auto hand_round = [&](auto st_c) {
        constexpr int st = decltype(st_c)::value;
        const int u = st >> sub_sh;  // the step's group inside the chunk
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (FAC == FAC_DEP)
            fwd[st & 1][q] = (uint32_t)__builtin_amdgcn_ds_bpermute((n + 16 * q) * 4, (int)fw[st]);
          else
            fwd[st & 1][q] = (uint32_t)__builtin_amdgcn_ds_bpermute((n + 16 * u) * 4, (int)fw[q]);
          if constexpr (NBITS == 3) hw[st & 1][q] = (uint32_t)__builtin_amdgcn_ds_bpermute((n + 16 * q) * 4, (int)chi[st]);
        }
      };
      hand_round(std::integral_constant<int, 0>{});
      static_for<0, 4>([&](auto st_c) {
        constexpr int st = decltype(st_c)::value;
        const unsigned char* xp = rd + x_lane + (((4 * st + kb) ^ n) << 4);
        u32x4 xa[TT];  // requested before the operands are built
        static_for<0, TT>([&](auto t) { xa[decltype(t)::value] = *reinterpret_cast<const u32x4*>(xp + decltype(t)::value * 4096); });
        if constexpr (st < 3) hand_round(std::integral_constant<int, (st + 1) & 3>{});
        u32x4 ov[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f16x2 ab = __builtin_bit_cast(f16x2, fwd[st & 1][q]);
          const f16x2 a2 = {ab.x, ab.x}, b2 = {ab.y, ab.y};
          uint32_t w0 = cw[st][q], w1 = 0;
          if constexpr (NBITS != 4) w0 >>= 8 * (kb & 1);  // the lane's eight rows of the sixteen in a word
          if constexpr (NBITS == 3) w1 = hw[st & 1][q] >> (4 * kb);
#pragma unroll
          for (int m = 0; m < 4; ++m)
            ov[q][m] = __builtin_bit_cast(uint32_t, patch_code_pair_f16<NBITS>(w0, w1, m, dq_mask, dq_magic) * a2 + b2);
        }
        asm volatile("" : "+v"(ov[0]), "+v"(ov[1]), "+v"(ov[2]), "+v"(ov[3]));
        __builtin_amdgcn_sched_barrier(0);
        load_step(st_c, n1);
        __builtin_amdgcn_sched_barrier(0);
        if (live) {
          static_for<0, TT>([&](auto t_c) {
            constexpr int tt = decltype(t_c)::value;
#pragma unroll
            for (int q = 0; q < 4; ++q)
              acc[tt][q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, xa[tt]), __builtin_bit_cast(f16x8, ov[q]),
                                                                  acc[tt][q], 0, 0, 0);
          });
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    // the next unit's x was requested before this unit's other loads: once only those are in flight it
    // has landed
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NLOADS) : "memory");
    if (at.c + 1 == at.ce) {
      flush(at.s, at.ce, x_rd);
      clear();
    }
  };

  // segments run from the last slab of the run to the first
  auto next_of = [&](Pos q, int steps_left) {
    if (steps_left > 0 && ++q.c == q.ce) {
      --q.s;
      q.c = q.s == s_first ? c_first : 0;
      q.ce = CU;
    }
    return q;
  };
  Pos p0{s_last, s_last == s_first ? c_first : 0, u1 - s_last * CU};
  load_x(lds, p0);
  __builtin_amdgcn_sched_barrier(0);  // the wait counts on x being requested before the rest
  load_fac(p0);
  static_for<0, 4>([&](auto st) { load_step(st, p0); });
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NLOADS) : "memory");
  int x_cur = 0;
#pragma nounroll
  for (int left = u1 - u0 - 1; left >= 0; --left) {
    const Pos p1 = next_of(p0, left);
    unit(lds + x_cur, lds + (XBUF - x_cur), p0, p1);
    x_cur = XBUF - x_cur;
    p0 = p1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the last unit's prefetch
}

template <int NBITS, int FAC, int TT>
static hipError_t launch_tt(const MidTArgs& a, int blocks, hipStream_t st) {
  constexpr size_t smem = 2 * MT_DEEP * TT * 16 * 256;
  static std::atomic<uint64_t> granted{0};  // per instantiation
  if (hipError_t e = grant_dynamic_lds(reinterpret_cast<const void*>(midt_kernel<NBITS, FAC, TT>), (int)smem, granted);
      e != hipSuccess)
    return e;
  midt_kernel<NBITS, FAC, TT><<<blocks, MT_THREADS, smem, st>>>(a);
  return hipGetLastError();
}
template <int NBITS, int FAC>
static hipError_t launch_fac(const MidTArgs& a, int blocks, hipStream_t st) {
  const int tt = midt_tiles(a.T);
  if (tt == 2) return launch_tt<NBITS, FAC, 2>(a, blocks, st);
  return tt == 3 ? launch_tt<NBITS, FAC, 3>(a, blocks, st) : launch_tt<NBITS, FAC, 4>(a, blocks, st);
}

hipError_t launch_midt(int bits, const MidTArgs& args, int blocks, hipStream_t st) {
  MidTArgs a = args;
  if (a.T < 1 || a.T > MT_MAX_TOKENS || a.d_in % 128 != 0 || blocks < 1 || blocks > ST_MAX_BLOCKS) return hipErrorInvalidValue;
  if (a.group != 32 && a.group != 64 && a.group != 128) return hipErrorInvalidValue;
  if ((long)blocks > (long)ceil_div(a.d_out, MT_SLAB) * ceil_div(a.d_in / 128, MT_DEEP)) return hipErrorInvalidValue;  // no empty runs
  a.nonce = smallt_next_nonce();
  // measurement aid: this kernel is the forward contraction of its token range
  ProfileHook hook = g_profile_hook[0];
  g_profile_hook[0] = ProfileHook{nullptr, nullptr, nullptr};
  if (hook.start) (void)hipEventRecord(hook.start, st);
  hipError_t e = hipErrorInvalidValue;
  if (bits == 4)
    e = a.stream ? launch_fac<4, FAC_DEP>(a, blocks, st)
                 : (a.fac16 ? launch_fac<4, FAC_F16>(a, blocks, st) : launch_fac<4, FAC_F32>(a, blocks, st));
  else if (bits == 3 && !a.stream)
    e = a.fac16 ? launch_fac<3, FAC_F16>(a, blocks, st) : launch_fac<3, FAC_F32>(a, blocks, st);
  else if (bits == 2 && !a.stream)
    e = a.fac16 ? launch_fac<2, FAC_F16>(a, blocks, st) : launch_fac<2, FAC_F32>(a, blocks, st);
  if (hook.stop) (void)hipEventRecord(hook.stop, st);
  return e;
}

}  // namespace qalora
