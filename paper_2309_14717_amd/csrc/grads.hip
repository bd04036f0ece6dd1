// The adapter's gradients (derived from Alg. 1 with W frozen).  With P = pool_g(x), U = P A and dU = dy B^T,
//
//   dB = s U^T dy = s A^T Z,     dA = s P^T dU = s Z B^T,     Z = P^T dy  [L x d_out],
//
// so there are two ways, and grads_plan.hpp takes the shorter one for a call.
//
// By Z: dy meets one large product, whatever the rank and however many adapters share x.  Z costs 3 T L d_out
// multiply-adds (P goes through the bf16 matrix cores as three pieces, which hold all its bits), 3 / g of the dense
// backward's; what follows is L r d_out, in fp32 on v_mfma_f32_16x16x4_f32.
//   z_kernel       Z, in tiles of 128 groups x 128 columns and runs of tokens                     [slots][L][d_out]
//   finish_kernel  a block owns 128 groups x 32 columns: adds Z's partial sums in order, then its shares of
//                  dA [d_out / 32][L][r] and of dB [L / 128][r][d_out] (whole where L <= 128)
//   tail_kernel    adds the shares in order (and the slices of a split dx product, if there are any)
//   fused_kernel   the first two for few tokens: Z goes from the accumulators to LDS
//
// By U: where the rank is well below the groups (further below, with its kernels).
//
// 4096 tokens, rank 64: 4096 x 4096 by Z 23 + 12 + 5 us (with two pieces of P 19 + 11 + 5, but gradients ten times as far
// from the exact ones; each gradient from its own pass over dy, with B, U and P rounded to two pieces: 44).
// What bounds it: the chain of a step (loads, LDS, matrix work) on a unit that holds little else, then bytes: dy once (33.6
// MB for 4096 x 4096), P for every tile and Z's partial sums written and read (2 MB a slot there).  Counters of 4096 tokens of
// 4096 x 22016: 337 MB fetched (dy 180, P 3), matrix cores busy for 35 % of the launch.  Both of Z's operands have the contraction index (tokens) as their slow one: they
// are staged as they lie in memory and read transposed (ds_read_b64_tr_b16: a group of 16 lanes turns four rows
// of sixteen columns), so that no 16-bit gather or packing is left.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "grads_plan.hpp"
#include "kernels.hpp"
#include "split_sum.hpp"

namespace qalora {

namespace {
constexpr int GF_LD = 36;  // floats per LDS row of 32 columns
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

template <int NL, int NC, int NT = 256>
struct ZTile {  // how NT threads' wavefronts share a tile of NL rows (groups, or ranks) x NC columns
  static constexpr int kWavesL = NC < 128 ? NL / 32 : (NL >= 64 ? NT / 128 : 1);  // (32 columns and fewer than 128 rows: the rest idle)
  static constexpr int kWavesC = NC < 128 ? 1 : NT / 64 / kWavesL;
  static constexpr int TL = NL / kWavesL / 32, TC = NC / kWavesC / 32;
  // 16-bit elements per LDS row (a token): four rows of a transposed read in distinct banks
  static constexpr int P_LD = kPieces * NL + 16, Y_LD = NC + 16;
  static constexpr int kLds = GZ_T * (P_LD + Y_LD) * 2;
};

constexpr uint32_t kOob = 0xffff0000u;  // past every buffer below: reads zero
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)(bytes > kOob ? kOob : bytes), 0x00020000);
}

// Element i of four fp32 values from their pieces.
__device__ __forceinline__ float piece_sum(const uint2 (&w)[kPieces], int i) {
  float v = 0.0f;
#pragma unroll
  for (int h = 0; h < kPieces; ++h) {
    const uint32_t pair = i < 2 ? w[h].x : w[h].y;
    v += __uint_as_float(i & 1 ? pair & 0xffff0000u : pair << 16);
  }
  return v;
}

// LDS-only barrier: does not wait for the global loads that are in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Eight consecutive rows (tokens) of one column per lane, from LDS rows of `ld` elements: the operand of
// v_mfma_f32_32x32x16 whose 32 columns and 16 rows start at `tile`.
__device__ __forceinline__ bf16x8 read_columns(const uint16_t* tile, int ld, int lane) {
  const int i = lane & 15, row = 8 * (lane >> 5) + (i >> 2), col = 16 * ((lane >> 4) & 1) + 4 * (i & 3);
  const uint16_t* p = tile + row * ld + col;
  typedef __attribute__((address_space(3))) s16x4* lds_ptr;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * ld));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// acc += P[t0 .. t1)^T dy[t0 .. t1) of the NL rows from l0 (of L, P's pieces being Lp apart) and the NC columns from j0,
// by NT threads.  Rows and columns outside the matrix hold anything (the callers drop them).
template <int NL, int NC, int NT = 256>
__device__ __forceinline__ void z_tile(const uint16_t* P, int L, int Lp, const uint16_t* dy, int d_out, int l0, int j0,
                                       int t0, int t1, uint16_t* lds,
                                       f32x16 (&acc)[ZTile<NL, NC, NT>::TL][ZTile<NL, NC, NT>::TC]) {
  using G = ZTile<NL, NC, NT>;
  constexpr int P_LD = G::P_LD;
  constexpr int P_CH = NL / 8, P_LOADS = GZ_T * P_CH / NT, Y_CH = NC / 8, Y_LOADS = ceil_div(GZ_T * Y_CH, NT);
  uint16_t* ps = lds;
  uint16_t* ys = lds + GZ_T * P_LD;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wl = wave % G::kWavesL * G::TL * 32, wc = wave / G::kWavesL % G::kWavesC * G::TC * 32;
  // A lane's offsets inside a step are constants (groups and columns outside the matrix point past the buffer);
  // the buffers start at the step's first token and end with the last one's row, so later tokens read zero.
  const uint32_t p_row = (uint32_t)(kPieces * Lp) * 2u, y_row = (uint32_t)d_out * 2u;
  const int pr0 = tid / P_CH, pl = l0 + 8 * (tid % P_CH), yr0 = tid / Y_CH, yj = j0 + 8 * (tid % Y_CH);
  const bool y_mine = GZ_T * Y_CH >= NT || yr0 < GZ_T;  // (more threads than pieces of dy)
  const bool p_ok = pl < Lp, y_ok = yj < d_out && y_mine;
  uint32_t p_off = (uint32_t)pr0 * p_row + 2u * (uint32_t)pl, y_off = (uint32_t)yr0 * y_row + 2u * (uint32_t)yj;
  u32x4 pr[kPieces][P_LOADS], yr[Y_LOADS];  // the next step's, while this one is worked on
  auto fetch = [&](int t) {
    const size_t from = (size_t)min(t, t1), rows = (size_t)(t1 - (int)from);
    const __amdgpu_buffer_rsrc_t rs_p = rsrc(P + from * kPieces * Lp, rows * p_row);
    const __amdgpu_buffer_rsrc_t rs_y = rsrc(dy + from * d_out, rows * y_row);
    asm volatile("" : "+v"(p_off), "+v"(y_off));  // (a register for each load's offset, kept over the loop, is too many)
#pragma unroll
    for (int q = 0; q < P_LOADS; ++q)
#pragma unroll
      for (int h = 0; h < kPieces; ++h) {
        const uint32_t o = p_off + (uint32_t)(NT / P_CH * q) * p_row + 2u * (uint32_t)(h * Lp);
        pr[h][q] = __builtin_amdgcn_raw_buffer_load_b128(rs_p, (int)(p_ok ? o : kOob), 0, 0);
      }
#pragma unroll
    for (int q = 0; q < Y_LOADS; ++q) {
      const uint32_t o = y_off + (uint32_t)(NT / Y_CH * q) * y_row;
      yr[q] = __builtin_amdgcn_raw_buffer_load_b128(rs_y, (int)(y_ok ? o : kOob), 0, 0);
    }
  };
  const bool busy = l0 + wl < L && wave < G::kWavesL * G::kWavesC;
  fetch(t0);
  for (int t = t0; t < t1; t += GZ_T) {
#pragma unroll
    for (int q = 0; q < P_LOADS; ++q)
#pragma unroll
      for (int h = 0; h < kPieces; ++h)
        *reinterpret_cast<u32x4*>(ps + (pr0 + NT / P_CH * q) * P_LD + h * NL + pl - l0) = pr[h][q];
#pragma unroll
    for (int q = 0; q < Y_LOADS; ++q)
      if (y_mine) *reinterpret_cast<u32x4*>(ys + (yr0 + NT / Y_CH * q) * G::Y_LD + yj - j0) = yr[q];
    lds_barrier();
    fetch(t + GZ_T);  // (past the end: reads zero)
    if (busy) {
      // the operands of the next sixteen tokens are read while the matrix cores work on these (with 512 threads
      // there are no registers for both, and other wavefronts on the SIMD to work on)
      constexpr int D = NT > 256 && NC >= 128 ? 1 : 2;
      bf16x8 y[D][G::TC], p[D][kPieces][G::TL];
      auto read = [&](int kk) {
#pragma unroll
        for (int c = 0; c < G::TC; ++c) y[kk % D][c] = read_columns(ys + 16 * kk * G::Y_LD + wc + 32 * c, G::Y_LD, lane);
#pragma unroll
        for (int h = 0; h < kPieces; ++h)
#pragma unroll
          for (int l = 0; l < G::TL; ++l) p[kk % D][h][l] = read_columns(ps + 16 * kk * P_LD + h * NL + wl + 32 * l, P_LD, lane);
      };
      read(0);
#pragma unroll
      for (int kk = 0; kk < GZ_T / 16; ++kk) {
        if (kk + D - 1 < GZ_T / 16 && (D > 1 || kk > 0)) read(kk + D - 1);
        if constexpr (D > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < kPieces; ++h)
#pragma unroll
          for (int l = 0; l < G::TL; ++l)
#pragma unroll
            for (int c = 0; c < G::TC; ++c)
              acc[l][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[kk % D][h][l], y[kk % D][c], acc[l][c], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    lds_barrier();
  }
}

// What a block does with Z of its 128 groups x 32 columns: its shares of dB and dA.  The constructor requests
// the operands A (straight to LDS) and B, so that they arrive while Z is being made.
constexpr int kMaxRank = 128;
__host__ __device__ constexpr int finish_floats(int rank) {  // LDS: Z, B, A (and what the last row's padding lanes read)
  return GZ_L * GF_LD + round_up(rank, 16) * GF_LD + GZ_L * rank + 16;
}
template <int NW>
struct Finish {
  static constexpr int kTasks = 16 / NW;  // 16 x 16 tiles of dB per wavefront: rank / 16 of them x two
  static constexpr int kB = kMaxRank * GF_C / 64 / NW;
  const FinishArgs& a;
  const FinishPart& pt;
  const int pj0, l0, lane, wave, n, kq, mt;  // first column in the part; first group; mt: 16-row tiles of the rank
  float* zs;   // [GZ_L][GF_LD]: the caller's to fill, zero outside the matrix
  float* bs;   // [16 mt][GF_LD], zero outside the matrix
  float* as;   // [GZ_L][rank], zero outside the matrix
  float b[kB];

  __device__ __forceinline__ Finish(const FinishArgs& args, const FinishPart& part, int j0, int first_group, float* lds)
      : a(args), pt(part), pj0(j0 - part.col0), l0(first_group), lane(threadIdx.x & 63),
        wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)), n(lane & 15), kq(lane >> 4), mt((part.rank + 15) / 16),
        zs(lds), bs(lds + GZ_L * GF_LD), as(bs + 16 * mt * GF_LD) {
    // the rows of A are contiguous: a linear copy, zeros behind the last group
    const __amdgpu_buffer_rsrc_t rs = rsrc(pt.A + (size_t)l0 * pt.rank, (size_t)(a.L - l0) * pt.rank * 4);
    for (int i = wave * 64; i < GZ_L * pt.rank; i += NW * 64)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(as + i), 4, 4 * (i + lane), 0, 0, 0);
#pragma unroll
    for (int q = 0; q < kB; ++q) {
      const int idx = threadIdx.x + 64 * NW * q, k = idx / GF_C, c = idx % GF_C;
      b[q] = (k < pt.rank && pj0 + c < pt.d_out) ? pt.B[(size_t)k * pt.d_out + pj0 + c] : 0.0f;
    }
  }

  __device__ __forceinline__ void run() {
#pragma unroll
    for (int q = 0; q < kB; ++q) {
      const int idx = threadIdx.x + 64 * NW * q, k = idx / GF_C;
      if (k < 16 * mt) bs[k * GF_LD + idx % GF_C] = b[q];
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // A is in LDS
    __syncthreads();
    const int rows = min(GZ_L, a.L - l0);
    // A^T Z, groups in order (rows of the tile past the rank: other numbers of A, dropped)
    const bool whole = a.L <= GZ_L;
    float* dB = whole ? pt.dB : pt.db_part + (size_t)(l0 / GZ_L) * pt.rank * pt.d_out;
#pragma unroll
    for (int q = 0; q < kTasks; ++q) {
      const int task = wave + NW * q, k = 16 * (task >> 1) + n, c = 16 * (task & 1) + n;
      if (task < 2 * mt) {
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int i0 = 0; i0 < rows; i0 += 32) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int l = i0 + 4 * i + kq;
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(as[l * pt.rank + k], zs[l * GF_LD + c], acc, 0, 0, 0);
          }
        }
        if (pj0 + c < pt.d_out) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = 16 * (task >> 1) + 4 * kq + r;
            if (row < pt.rank) {
              float* o = dB + (size_t)row * pt.d_out + pj0 + c;
              *o = whole ? (a.accumulate ? *o : 0.0f) + pt.s * acc[r] : acc[r];
            }
          }
        }
      }
    }
    // Z B^T
    float* out = pt.da_part + (size_t)(pj0 / GF_C) * a.L * pt.rank;
    for (int lt = wave; 16 * lt < rows; lt += NW) {
      float zv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) zv[i] = zs[(16 * lt + n) * GF_LD + 4 * i + kq];
      for (int m0 = 0; m0 < mt; m0 += 2) {
        f32x4 acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int h = 0; h < 2; ++h)  // (an odd number of tiles: the last one twice)
            acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(zv[i], bs[(16 * min(m0 + h, mt - 1) + n) * GF_LD + 4 * i + kq], acc[h], 0, 0, 0);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int k = 16 * (m0 + h) + n;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int l = l0 + 16 * lt + 4 * kq + r;
            if (l < a.L && k < pt.rank) out[(size_t)l * pt.rank + k] = acc[h][r];
          }
        }
      }
    }
  }
};

__device__ __forceinline__ const FinishPart& part_of(const FinishArgs& a, int j0) {
  int pi = 0;
  for (int q = 1; q < a.n_parts; ++q)
    if (j0 >= a.part[q].col0) pi = q;
  return a.part[pi];
}
}  // namespace

// Equal runs of (tile, step) units, tile by tile: a tile that several blocks work on has a partial sum from each,
// in the slots 0, 1, ... in order.
// (NL: grads_group_tile)
// Tiles of 128 groups by eight wavefronts: a block per unit is two on a SIMD, of which one works while the other waits for
// loads, LDS or a barrier (by four: one; forward and backward of 4096 tokens, 4096 x 4096 308.9 us by four and 306.8 by
// eight, 1531 of 5120 x 13824 g 64 520.2 / 515.6; the same where two blocks share a unit, 2298 for the MLP block).
// (P as fp32 in memory, cut into pieces on the way to LDS, is a third fewer bytes but longer: the cutting is on every
// step's chain, 316.6 / 320.0 and 528.2 / 532.5 by four.)
constexpr int z_threads(int NL) { return NL < GZ_L ? 256 : 512; }
template <int NL>
__global__ __launch_bounds__(z_threads(NL), z_threads(NL) / 128) void z_kernel(const ZArgs a) {
  extern __shared__ __align__(16) uint16_t zlds[];
  using G = ZTile<NL, GZ_C, z_threads(NL)>;
  const int cols = ceil_div(a.d_out, GZ_C), lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wl = (wave % G::kWavesL) * G::TL * 32, wc = (wave / G::kWavesL) * G::TC * 32;
  const int b = (int)blockIdx.x, u1 = a.runs.first(b + 1);
  for (int u = a.runs.first(b); u < u1;) {
    const int tile = u / a.runs.steps, k0 = u - tile * a.runs.steps, k1 = min(a.runs.steps, k0 + u1 - u);
    const int j0 = tile % cols * GZ_C, l0 = tile / cols * GZ_L;
    f32x16 acc[G::TL][G::TC];
#pragma unroll
    for (int l = 0; l < G::TL; ++l)
#pragma unroll
      for (int c = 0; c < G::TC; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[l][c][r] = 0.0f;
    z_tile<NL, GZ_C, z_threads(NL)>(a.P, a.L, a.Lp, a.dy, a.d_out, l0, j0, k0 * GZ_T, min(a.T, k1 * GZ_T), zlds, acc);
    float* Z = a.Z + (size_t)(b - a.runs.owner(tile * a.runs.steps)) * a.L * a.d_out;
#pragma unroll
    for (int l = 0; l < G::TL; ++l)
#pragma unroll
      for (int c = 0; c < G::TC; ++c) {
        const int j = j0 + wc + 32 * c + (lane & 31);
        if (j < a.d_out) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = l0 + wl + 32 * l + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (row < a.L) Z[(size_t)row * a.d_out + j] = acc[l][c][r];
          }
        }
      }
    u += k1 - k0;
  }
}

constexpr int FINISH_WAVES = 8;
__global__ __launch_bounds__(64 * FINISH_WAVES) void finish_kernel(const FinishArgs a) {
  extern __shared__ __align__(16) float flds[];
  const int j0 = (int)blockIdx.x * GF_C, l0 = (int)blockIdx.y * GZ_L, tid = threadIdx.x;
  Finish<FINISH_WAVES> finish(a, part_of(a, j0), j0, l0, flds);
  constexpr int Q = GZ_L * GF_C / 4 / (64 * FINISH_WAVES);
  const f32x4* src[Q];  // (elements outside the matrix read its first and become zero)
  bool ok[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int idx = tid + 64 * FINISH_WAVES * q, l = l0 + (idx >> 3), j = j0 + 4 * (idx & 7);
    ok[q] = l < a.L && j < a.d_out;
    src[q] = reinterpret_cast<const f32x4*>(a.Z + (ok[q] ? (size_t)l * a.d_out + j : 0));
  }
  const int first = (int)blockIdx.y * ceil_div(a.d_out, GZ_C) + j0 / GZ_C;  // the tile, its units and their blocks
  const int slots = a.runs.owner((first + 1) * a.runs.steps - 1) - a.runs.owner(first * a.runs.steps) + 1;
  f32x4 v[Q];
  sum_slices<8>(src, (size_t)a.L * a.d_out / 4, slots, v);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int idx = tid + 64 * FINISH_WAVES * q;
    *reinterpret_cast<f32x4*>(finish.zs + (idx >> 3) * GF_LD + 4 * (idx & 7)) = ok[q] ? v[q] : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  finish.run();
}

// (128 groups: eight wavefronts here too, of which four hold Z; all stage its operands and share what follows.  Forward and
// backward by four / by eight, us: 115 tokens of 3968 x 1504, rank 128 85.6 / 79.2; 248 of 6912 x 1912, rank 128 111.2 / 106.7;
// 311 of 9728 x 1408, g 128 rank 64 97.8 / 94.2; 25 of 13568 x 896, rank 16 71.0 / 70.1.)
template <int NL>
__global__ __launch_bounds__(z_threads(NL)) void fused_kernel(const ZArgs z, const FinishArgs a) {
  extern __shared__ __align__(16) uint16_t zlds[];
  using G = ZTile<NL, GF_C, z_threads(NL)>;
  const int j0 = (int)blockIdx.x * GF_C, l0 = (int)blockIdx.y * GZ_L, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Finish<z_threads(NL) / 64> finish(a, part_of(a, j0), j0, l0, reinterpret_cast<float*>(zlds + G::kLds / 2));
  f32x16 acc[1][1];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.0f;
  z_tile<NL, GF_C, z_threads(NL)>(z.P, z.L, z.Lp, z.dy, z.d_out, l0, j0, 0, z.T, zlds, acc);
  const int c = lane & 31;
  if (wave < GZ_L / 32) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = 32 * wave + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      finish.zs[row * GF_LD + c] = (l0 + row < a.L && j0 + c < a.d_out) ? acc[0][0][r] : 0.0f;
    }
  }
  finish.run();
}

// ---- by way of U = P A and dU = dy B^T ---------------------------------------------------------------------------
// dB = s U^T dy and dA = s P^T dU: T d_out r products twice instead of T d_out L once.  The operands of the bf16 matrix
// cores are the three pieces of U and of B (B's are cut on the way to LDS, by every block of tokens); P A and P^T dU are
// small and stay in fp32.
//   du_kernel  blocks of tokens x a run of columns: dU's partial sums; a wavefront per 16 tokens x 16 ranks: U, as pieces
//   db_kernel  runs of (128 columns, 64 tokens) as in z_kernel, U in P's place: dB's partial sums; blocks of
//              128 groups x a run of tokens: shares of dA, from the sums of dU
//   tail_kernel
// 1000 tokens of 13824 x 13824, rank 128 (432 groups): 32 + 29 + 10 us, by Z 69 + 71 + 20; 20 of them 20 + 14 + 8 and
// 14 + 64 + 26; 4096 of 11008 x 4096 rank 64 25 + 20 + 6 and 61 + 14 + 6; 4096 of 4096 x 4096 19 + 18 + 5 and
// 23 + 12 + 5.  Bound by dy's bytes, twice, and by B's, read from L2 by every block of tokens (22016 columns, rank 64,
// 4096 tokens: 361 MB of B in blocks of 64 tokens, 102 us; in blocks of 256 90 MB, 64 us).
constexpr int GU_LD = 72;    // 16-bit elements per LDS row of 64 columns
constexpr int GA_LD = 144;   // floats per LDS row of 128 groups or ranks: four rows in distinct banks

// How the wavefronts of a dU block share its tokens (32 each) and ranks.  Long batches: 256 tokens, so that B is read and
// cut into pieces for fewer tiles; else 64.
template <int NL, bool LONG>  // NL: ranks, rounded up: 32, 64 or 128
struct DuTile {
  static constexpr int kWavesT = LONG ? 8 : 2, kWavesR = LONG ? 1 : 2, kThreads = 64 * kWavesT * kWavesR;
  static constexpr int kTokens = 32 * kWavesT;
  static constexpr int kTiles = NL / 32;                                    // of 32 ranks
  static constexpr int kPer = kTiles > kWavesR ? kTiles / kWavesR : 1;      // of them per wavefront
  static constexpr int kLds = (kTokens + kPieces * NL) * GU_LD * 2;
};

// Partial sums of dU of a block's tokens over a run of a part's columns.
template <int NL, bool LONG>
__device__ __forceinline__ void du_block(const UArgs& a, const UPart& pt, int t0, int slice, uint16_t* lds) {
  using G = DuTile<NL, LONG>;
  constexpr int Y_LOADS = G::kTokens * 8 / G::kThreads, B_LOADS = NL * 16 / G::kThreads;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wt = 32 * (wave / G::kWavesR), wr = wave % G::kWavesR;
  const int j0 = slice * pt.du_steps * 64, j1 = min(pt.d_out, j0 + pt.du_steps * 64);
  uint16_t* ys = lds;
  uint16_t* bs = lds + G::kTokens * GU_LD;  // [kPieces][NL][GU_LD]
  const size_t rows = (size_t)min(G::kTokens, a.T - t0);
  const __amdgpu_buffer_rsrc_t rs_y = rsrc(a.dy + (size_t)t0 * a.d_out, rows * a.d_out * 2);
  const __amdgpu_buffer_rsrc_t rs_b = rsrc(pt.B, (size_t)pt.rank * pt.d_out * 4);
  constexpr int D = LONG && NL < 128 ? 1 : 2;  // steps in flight
  u32x4 yr[D][Y_LOADS];
  f32x4 br[D][B_LOADS];
  auto fetch = [&](auto s_c, int j) {  // columns past the run read zero
    constexpr int s = decltype(s_c)::value;
#pragma unroll
    for (int q = 0; q < Y_LOADS; ++q) {
      const int idx = tid + G::kThreads * q, c = j + 8 * (idx & 7);
      const uint32_t o = ((uint32_t)(idx >> 3) * (uint32_t)a.d_out + (uint32_t)(pt.col0 + c)) * 2u;
      yr[s][q] = __builtin_amdgcn_raw_buffer_load_b128(rs_y, (int)(c < j1 ? o : kOob), 0, 0);
    }
#pragma unroll
    for (int q = 0; q < B_LOADS; ++q) {
      const int idx = tid + G::kThreads * q, c = j + 4 * (idx & 15), k = idx >> 4;
      const uint32_t o = ((uint32_t)k * (uint32_t)pt.d_out + (uint32_t)c) * 4u;
      br[s][q] = __builtin_bit_cast(
          f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_b, (int)(c < j1 && k < pt.rank ? o : kOob), 0, 0));
    }
  };
  f32x16 acc[G::kPer];
#pragma unroll
  for (int m = 0; m < G::kPer; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[m][r] = 0.0f;
  auto step = [&](auto s_c, int j) {
    constexpr int s = decltype(s_c)::value;
#pragma unroll
    for (int q = 0; q < Y_LOADS; ++q) {
      const int idx = tid + G::kThreads * q;
      *reinterpret_cast<u32x4*>(ys + (idx >> 3) * GU_LD + 8 * (idx & 7)) = yr[s][q];
    }
#pragma unroll
    for (int q = 0; q < B_LOADS; ++q) {
      const int idx = tid + G::kThreads * q;
      uint16_t piece[4][kPieces];
#pragma unroll
      for (int c = 0; c < 4; ++c) split_bf16(br[s][q][c], piece[c]);
#pragma unroll
      for (int h = 0; h < kPieces; ++h) {
        const uint2 v = {piece[0][h] | (uint32_t)piece[1][h] << 16, piece[2][h] | (uint32_t)piece[3][h] << 16};
        *reinterpret_cast<uint2*>(bs + (h * NL + (idx >> 4)) * GU_LD + 4 * (idx & 15)) = v;
      }
    }
    lds_barrier();
    fetch(s_c, j + 64 * D);
    if (wr < G::kTiles) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const int at = 16 * kk + 8 * (lane >> 5);
        const bf16x8 y = *reinterpret_cast<const bf16x8*>(ys + (wt + (lane & 31)) * GU_LD + at);
#pragma unroll
        for (int h = 0; h < kPieces; ++h)
#pragma unroll
          for (int m = 0; m < G::kPer; ++m) {
            const bf16x8 b = *reinterpret_cast<const bf16x8*>(bs + (h * NL + 32 * (wr + G::kWavesR * m) + (lane & 31)) * GU_LD + at);
            acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(y, b, acc[m], 0, 0, 0);
          }
      }
    }
    lds_barrier();
  };
  using zero = std::integral_constant<int, 0>;
  using last = std::integral_constant<int, D - 1>;
  fetch(zero{}, j0);
  if constexpr (D > 1) fetch(last{}, j0 + 64);
  for (int j = j0; j < j1; j += 64 * D) {
    step(zero{}, j);
    if constexpr (D > 1)
      if (j + 64 < j1) step(last{}, j + 64);
  }
  if (wr >= G::kTiles) return;
  float* out = pt.du + (size_t)slice * a.T * pt.ld;
#pragma unroll
  for (int m = 0; m < G::kPer; ++m) {
    const int k = 32 * (wr + G::kWavesR * m) + (lane & 31);
    if (k < pt.ld) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int t = t0 + wt + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (t < a.T) out[(size_t)t * pt.ld + k] = acc[m][r];
      }
    }
  }
}

// U = P A of sixteen tokens and ranks per wavefront, groups in order, as pieces.
template <int CH>  // sixteen groups each: a batch of loads, the next one in flight behind it
__device__ __forceinline__ void u_block(const UArgs& a, const UPart& pt, int t0, int k0) {
  const int lane = threadIdx.x & 63, n = lane & 15, kq = lane >> 4, k = k0 + n;
  const uint32_t p_row = (uint32_t)(kPieces * a.Lp) * 2u, a_row = (uint32_t)pt.rank * 4u;
  // (groups and tokens past the last one read zero, and so do ranks)
  const __amdgpu_buffer_rsrc_t rs_p = rsrc(a.P + (size_t)t0 * kPieces * a.Lp, (size_t)min(16, a.T - t0) * p_row);
  const __amdgpu_buffer_rsrc_t rs_a = rsrc(pt.A, (size_t)a.L * a_row);
  uint2 pv[2][CH][kPieces];
  float av[2][CH][4];
  auto fetch = [&](auto s_c, int l0) {
    constexpr int s = decltype(s_c)::value;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int l = l0 + 16 * c + 4 * kq;
      const uint32_t po = (uint32_t)n * p_row + 2u * (uint32_t)l, ao = (uint32_t)l * a_row + 4u * (uint32_t)k;
#pragma unroll
      for (int h = 0; h < kPieces; ++h)
        pv[s][c][h] = __builtin_bit_cast(
            uint2, __builtin_amdgcn_raw_buffer_load_b64(rs_p, (int)(l < a.Lp ? po + 2u * (uint32_t)(h * a.Lp) : kOob), 0, 0));
#pragma unroll
      for (int i = 0; i < 4; ++i)
        av[s][c][i] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(rs_a, (int)(k < pt.rank ? ao + (uint32_t)i * a_row : kOob), 0, 0));
    }
  };
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  auto use = [&](auto s_c) {
    constexpr int s = decltype(s_c)::value;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(piece_sum(pv[s][c], i), av[s][c][i], acc, 0, 0, 0);
  };
  const std::integral_constant<int, 0> zero;
  const std::integral_constant<int, 1> one;
  fetch(zero, 0);
  for (int l0 = 0; l0 < a.L; l0 += 32 * CH) {
    fetch(one, l0 + 16 * CH);  // (past the end: zero)
    use(zero);
    fetch(zero, l0 + 32 * CH);
    use(one);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int t = t0 + 4 * kq + r;
    if (t < a.T && k < pt.ld) {
      uint16_t piece[kPieces];
      split_bf16(acc[r], piece);
#pragma unroll
      for (int h = 0; h < kPieces; ++h) pt.U[((size_t)t * kPieces + h) * pt.ld + k] = piece[h];
    }
  }
}

template <int NL, bool LONG>
__global__ __launch_bounds__((DuTile<NL, LONG>::kThreads), (LONG && NL < 128 ? 4 : 2)) void du_kernel(const UArgs a) {
  extern __shared__ __align__(16) uint16_t zlds[];
  constexpr int kTokens = DuTile<NL, LONG>::kTokens, kWaves = DuTile<NL, LONG>::kThreads / 64;
  int b = (int)blockIdx.x;
  // U first: few instructions and long waits, under everything else
  for (int q = 0; q < a.n_parts; ++q) {
    const int kt = ceil_div(a.part[q].rank, 16), n = ceil_div(ceil_div(a.T, 16) * kt, kWaves);
    if (b < n) {
      const int task = b * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
      if (16 * (task / kt) < a.T) u_block<LONG && NL < 128 ? 2 : 4>(a, a.part[q], 16 * (task / kt), 16 * (task % kt));
      return;
    }
    b -= n;
  }
  for (int q = 0; q < a.n_parts; ++q) {
    const int n = ceil_div(a.T, kTokens) * a.part[q].du_slices;
    if (b < n) {
      du_block<NL, LONG>(a, a.part[q], b / a.part[q].du_slices * kTokens, b % a.part[q].du_slices, zlds);
      return;
    }
    b -= n;
  }
}

// A share of dA: P^T dU of 128 groups over a run of tokens.
__device__ __forceinline__ void da_block(const UArgs& a, const UPart& pt, int l0, int run, float* lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, kq = lane >> 4, wl = 32 * wave, mt = ceil_div(pt.rank, 16);
  float* ps = lds;                  // [GA_T][GA_LD]: groups
  float* us = lds + GA_T * GA_LD;   // ranks
  const int t1 = min(a.T, (run + 1) * a.da_tokens);
  f32x4 acc[2][kMaxRank / 16];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int m = 0; m < kMaxRank / 16; ++m) acc[i][m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int quads = pt.ld / 4;
  for (int t0 = run * a.da_tokens; t0 < t1; t0 += GA_T) {
#pragma unroll
    for (int q = 0; q < GA_T * 16 / 256; ++q) {  // eight groups of a token each
      const int idx = tid + 256 * q, t = t0 + (idx >> 4), l = l0 + 8 * (idx & 15);
      u32x4 v[kPieces] = {};
      if (t < t1 && l < a.Lp) {
#pragma unroll
        for (int h = 0; h < kPieces; ++h)
          v[h] = *reinterpret_cast<const u32x4*>(a.P + ((size_t)t * kPieces + h) * a.Lp + l);
      }
      float* o = ps + (idx >> 4) * GA_LD + 8 * (idx & 15);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint2 w[kPieces] = {{v[0][2 * e], v[0][2 * e + 1]}, {v[1][2 * e], v[1][2 * e + 1]}, {v[2][2 * e], v[2][2 * e + 1]}};
        *reinterpret_cast<f32x4*>(o + 4 * e) = f32x4{piece_sum(w, 0), piece_sum(w, 1), piece_sum(w, 2), piece_sum(w, 3)};
      }
    }
    for (int idx = tid; idx < GA_T * quads; idx += 256) {
      const int row = idx / quads, c = 4 * (idx % quads);
      f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
      if (t0 + row < t1)
        v = sum_slices<8>(reinterpret_cast<const f32x4*>(pt.du + (size_t)(t0 + row) * pt.ld + c), (size_t)a.T * pt.ld / 4,
                          pt.du_slices);
      *reinterpret_cast<f32x4*>(us + row * GA_LD + c) = v;
    }
    __syncthreads();
    if (l0 + wl < a.L) {
#pragma unroll 2
      for (int i = 0; i < GA_T; i += 4) {
        const float p0 = ps[(i + kq) * GA_LD + wl + n], p1 = ps[(i + kq) * GA_LD + wl + 16 + n];
#pragma unroll
        for (int m = 0; m < kMaxRank / 16; ++m)
          if (m < mt) {  // (ranks past the last one: other numbers, dropped)
            const float u = us[(i + kq) * GA_LD + 16 * m + n];
            acc[0][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(p0, u, acc[0][m], 0, 0, 0);
            acc[1][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(p1, u, acc[1][m], 0, 0, 0);
          }
      }
    }
    __syncthreads();
  }
  float* out = pt.da_part + (size_t)run * a.L * pt.rank;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int m = 0; m < kMaxRank / 16; ++m) {
      const int k = 16 * m + n;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = l0 + wl + 16 * i + 4 * kq + r;
        if (l < a.L && k < pt.rank) out[(size_t)l * pt.rank + k] = acc[i][m][r];
      }
    }
}

template <int NL>
__global__ __launch_bounds__(256, 2) void db_kernel(const UArgs a) {
  extern __shared__ __align__(16) uint16_t zlds[];
  using G = ZTile<NL, GZ_C>;
  int b = (int)blockIdx.x;
  const int da = a.n_parts * a.da_shares * ceil_div(a.L, GZ_L);
  if (b < da) {
    const int tiles = ceil_div(a.L, GZ_L), per = tiles * a.da_shares;
    da_block(a, a.part[b / per], b % per / a.da_shares * GZ_L, b % a.da_shares, reinterpret_cast<float*>(zlds));
    return;
  }
  b -= da;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wl = (wave % G::kWavesL) * G::TL * 32, wc = (wave / G::kWavesL) * G::TC * 32;
  const int u1 = a.runs.first(b + 1);
  for (int u = a.runs.first(b); u < u1;) {
    const int tile = u / a.runs.steps, k0 = u - tile * a.runs.steps, k1 = min(a.runs.steps, k0 + u1 - u);
    int pi = 0;
    for (int q = 1; q < a.n_parts; ++q)
      if (tile >= a.part[q].tile0) pi = q;
    const UPart& pt = a.part[pi];
    const int j0 = (tile - pt.tile0) * GZ_C;
    f32x16 acc[G::TL][G::TC];
#pragma unroll
    for (int l = 0; l < G::TL; ++l)
#pragma unroll
      for (int c = 0; c < G::TC; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[l][c][r] = 0.0f;
    z_tile<NL, GZ_C>(pt.U, pt.rank, pt.ld, a.dy, a.d_out, 0, pt.col0 + j0, k0 * GZ_T, min(a.T, k1 * GZ_T), zlds, acc);
    float* out = pt.db_part + (size_t)(b - a.runs.owner(tile * a.runs.steps)) * pt.rank * pt.d_out;
#pragma unroll
    for (int l = 0; l < G::TL; ++l)
#pragma unroll
      for (int c = 0; c < G::TC; ++c) {
        const int j = j0 + wc + 32 * c + (lane & 31);
        if (j < pt.d_out) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int k = wl + 32 * l + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (k < pt.rank) out[(size_t)k * pt.d_out + j] = acc[l][c][r];
          }
        }
      }
    u += k1 - k0;
  }
}

// dA of every part: 64 elements per block, sixteen wavefronts with every sixteenth share each, added in a
// fixed order; then the sums that are a handful of copies each (dB's shares, the slices of dx), an element quad
// per thread.
constexpr int TAIL_WAVES = 16;
__global__ __launch_bounds__(64 * TAIL_WAVES) void tail_kernel(const TailArgs a) {
  __shared__ float part[TAIL_WAVES][64];
  int bid = blockIdx.x;
  if (bid >= a.da_blocks) {
    int si = 0;
    for (int q = 1; q < a.n_sums; ++q)
      if (bid >= a.sum[q].block0) si = q;
    const TailSum& ts = a.sum[si];
    const size_t i = (size_t)(bid - ts.block0) * (64 * TAIL_WAVES) + threadIdx.x;
    if (i >= ts.sum.n4) return;
    if (!ts.gradient) {
      split_sum_one(ts.sum, i);
    } else {
      int slices = ts.sum.slices;
      if (ts.runs.blocks > 0) {  // as many as blocks worked on the element's columns
        const int tile = ts.tile0 + (int)(i % (ts.d_out / 4)) * 4 / GZ_C;
        slices = ts.runs.owner((tile + 1) * ts.runs.steps - 1) - ts.runs.owner(tile * ts.runs.steps) + 1;
      }
      const f32x4 v = sum_slices(reinterpret_cast<const f32x4*>(ts.sum.partial) + i, ts.sum.n4, slices);
      f32x4* o = static_cast<f32x4*>(ts.sum.out) + i;
      const f32x4 was = a.accumulate ? *o : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int c = 0; c < 4; ++c) (*o)[c] = was[c] + ts.s * v[c];
    }
    return;
  }
  int pi = 0;
  for (int q = 1; q < a.n_parts; ++q)
    if (bid >= a.part[q].block0) pi = q;
  const TailPart& pt = a.part[pi];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const size_t e = (size_t)(bid - pt.block0) * 64 + lane;
  float sum = 0.0f;
  if (e < pt.n) {
    constexpr int B = 8;  // shares in flight
    for (int p0 = wave; p0 < pt.shares; p0 += B * TAIL_WAVES) {
      float v[B];
#pragma unroll
      for (int q = 0; q < B; ++q) v[q] = p0 + q * TAIL_WAVES < pt.shares ? pt.da_part[(size_t)(p0 + q * TAIL_WAVES) * pt.n + e] : 0.0f;
#pragma unroll
      for (int q = 0; q < B; ++q) sum += v[q];
    }
  }
  part[wave][lane] = sum;
  __syncthreads();
  if (wave == 0 && e < pt.n) {
    float v = part[0][lane];
#pragma unroll
    for (int q = 1; q < TAIL_WAVES; ++q) v += part[q][lane];
    pt.dA[e] = (a.accumulate ? pt.dA[e] : 0.0f) + pt.s * v;
  }
}

template <typename K>
static hipError_t grant(K kernel, size_t smem, std::atomic<uint64_t>& granted) {
  return smem > 48 * 1024 ? grant_dynamic_lds(reinterpret_cast<const void*>(kernel), (int)smem, granted) : hipSuccess;
}

template <int NL>
static hipError_t launch_z(const GradsPlan& plan, const ZArgs& z, const FinishArgs& f, hipStream_t st) {
  int max_rank = 0;
  for (int q = 0; q < f.n_parts; ++q) max_rank = std::max(max_rank, f.part[q].rank);
  const size_t finish = (size_t)finish_floats(max_rank) * 4, most = (size_t)finish_floats(kMaxRank) * 4;
  const dim3 blocks(ceil_div(f.d_out, GF_C), ceil_div(f.L, GZ_L));
  if (plan.form == GRADS_FUSED) {
    constexpr size_t lds = ZTile<NL, GF_C>::kLds;
    static std::atomic<uint64_t> granted{0};
    if (hipError_t e = grant(fused_kernel<NL>, lds + most, granted); e != hipSuccess) return e;
    fused_kernel<NL><<<blocks, z_threads(NL), lds + finish, st>>>(z, f);
    return hipGetLastError();
  }
  constexpr size_t lds = ZTile<NL, GZ_C>::kLds;
  static std::atomic<uint64_t> granted_z{0}, granted_f{0};
  if (hipError_t e = grant(z_kernel<NL>, lds, granted_z); e != hipSuccess) return e;
  if (hipError_t e = grant(finish_kernel, most, granted_f); e != hipSuccess) return e;
  z_kernel<NL><<<plan.runs.blocks, z_threads(NL), lds, st>>>(z);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  finish_kernel<<<blocks, 64 * FINISH_WAVES, finish, st>>>(f);
  return hipGetLastError();
}

hipError_t launch_grads(const GradsPlan& plan, const ZArgs& z, const FinishArgs& f, hipStream_t st) {
  const int rows = grads_group_tile(f.L);
  return rows == 32 ? launch_z<32>(plan, z, f, st) : (rows == 64 ? launch_z<64>(plan, z, f, st) : launch_z<GZ_L>(plan, z, f, st));
}

template <int NL, bool LONG>
static hipError_t launch_du(const UArgs& a, hipStream_t st) {
  using G = DuTile<NL, LONG>;
  static std::atomic<uint64_t> granted{0};
  if (hipError_t e = grant(du_kernel<NL, LONG>, G::kLds, granted); e != hipSuccess) return e;
  int blocks = 0;
  for (int q = 0; q < a.n_parts; ++q)
    blocks += ceil_div(ceil_div(a.T, 16) * ceil_div(a.part[q].rank, 16), G::kThreads / 64) +
              ceil_div(a.T, G::kTokens) * a.part[q].du_slices;
  du_kernel<NL, LONG><<<blocks, G::kThreads, G::kLds, st>>>(a);
  return hipGetLastError();
}
template <int NL>
static hipError_t launch_by_u(const GradsPlan& plan, const UArgs& a, hipStream_t st) {
  if (hipError_t e = plan.du_long ? launch_du<NL, true>(a, st) : launch_du<NL, false>(a, st); e != hipSuccess) return e;
  static std::atomic<uint64_t> granted{0};
  constexpr size_t lds = std::max<size_t>(ZTile<NL, GZ_C>::kLds, 2 * GA_T * GA_LD * 4);
  if (hipError_t e = grant(db_kernel<NL>, lds, granted); e != hipSuccess) return e;
  db_kernel<NL><<<a.n_parts * a.da_shares * ceil_div(a.L, GZ_L) + a.runs.blocks, 256, lds, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_grads_by_u(const GradsPlan& plan, const UArgs& a, hipStream_t st) {
  return plan.rank_tile == 32 ? launch_by_u<32>(plan, a, st)
                              : (plan.rank_tile == 64 ? launch_by_u<64>(plan, a, st) : launch_by_u<128>(plan, a, st));
}

hipError_t launch_tail(TailArgs t, hipStream_t st) {
  t.da_blocks = 0;
  for (int q = 0; q < t.n_parts; ++q) {
    t.part[q].block0 = t.da_blocks;
    t.da_blocks += (int)((t.part[q].n + 63) / 64);
  }
  int blocks = t.da_blocks;
  for (int q = 0; q < t.n_sums; ++q) {
    t.sum[q].block0 = blocks;
    blocks += (int)((t.sum[q].sum.n4 + 64 * TAIL_WAVES - 1) / (64 * TAIL_WAVES));
  }
  if (blocks == 0) return hipSuccess;
  tail_kernel<<<blocks, 64 * TAIL_WAVES, 0, st>>>(t);
  return hipGetLastError();
}

}  // namespace qalora
