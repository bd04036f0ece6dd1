// The adapter's gradients (derived from Alg. 1 with W frozen).  With P = pool_g(x) and U = P A,
//
//   dB = s U^T dy = s A^T Z,     dA = s P^T (dy B^T) = s Z B^T,     Z = P^T dy  [L x d_out],
//
// so dy meets only one large product, whatever the rank and however many adapters share x, and neither
// U nor dU = s dy B^T is formed.  Z costs 3 T L d_out multiply-adds (P goes through the bf16 matrix cores as
// three pieces, which hold all its bits), 3 / g of the dense backward's; what follows is L r d_out, in fp32 on
// v_mfma_f32_16x16x4_f32.
//
//   z_kernel       Z, in tiles of 128 groups x 128 columns and runs of tokens                     [slots][L][d_out]
//   finish_kernel  a block owns 128 groups x 32 columns: adds Z's partial sums in order, then its shares of
//                  dA [d_out / 32][L][r] and of dB [L / 128][r][d_out] (whole where L <= 128)
//   tail_kernel    adds the shares in order (and the slices of a split dx product, if there are any)
//   fused_kernel   the first two for few tokens: Z goes from the accumulators to LDS
//
// 4096 tokens, rank 64: 4096 x 4096 19 + 11 + 5 us (dU, dB, dA and their sums one after the other, each from its own
// pass over dy, took 44); a gate | up layer of 4096 x 22016 67 + 25 + 5 (143).
// What bounds it: bytes of dy once (33.6 MB for 4096 x 4096) and Z's partial sums written and read (2 MB a slot there);
// the matrix work is small.  Both of Z's operands have the contraction index (tokens) as their slow one: they
// are staged as they lie in memory and read transposed (ds_read_b64_tr_b16: a group of 16 lanes turns four rows
// of sixteen columns), so that no 16-bit gather or packing is left.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"
#include "split_sum.hpp"

namespace qalora {

namespace {
constexpr int GZ_L = 128;  // groups per tile
constexpr int GZ_C = 128;  // columns per tile of z_kernel
constexpr int GF_C = 32;   // columns per block of finish_kernel and fused_kernel
constexpr int GF_LD = 36;  // floats per LDS row of 32 columns
constexpr int P_LD = kPieces * GZ_L + 16;  // 16-bit elements per LDS row of P: four rows of a transposed read in distinct banks
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int GZ_T = 64;   // tokens per step
template <int NC>
struct ZTile {  // how four wavefronts share a tile of 128 groups x NC columns
  static constexpr int kWavesC = NC >= 128 ? 2 : 1;
  static constexpr int kWavesL = 4 / kWavesC;
  static constexpr int TL = GZ_L / kWavesL / 32, TC = NC / kWavesC / 32;
  static constexpr int Y_LD = NC + 16;
  static constexpr int kLds = GZ_T * (P_LD + Y_LD) * 2;
};


constexpr uint32_t kOob = 0xffff0000u;  // past every buffer below: reads zero
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)(bytes > kOob ? kOob : bytes), 0x00020000);
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

// acc += P[t0 .. t1)^T dy[t0 .. t1) of the 128 groups from l0 and the NC columns from j0, by 256 threads.
// Groups and columns outside the matrix hold anything (the callers drop them).
template <int NC>
__device__ __forceinline__ void z_tile(const ZArgs& a, int l0, int j0, int t0, int t1, uint16_t* lds,
                                       f32x16 (&acc)[ZTile<NC>::TL][ZTile<NC>::TC]) {
  using G = ZTile<NC>;
  constexpr int P_CH = GZ_L / 8, P_LOADS = GZ_T * P_CH / 256, Y_CH = NC / 8, Y_LOADS = GZ_T * Y_CH / 256;
  uint16_t* ps = lds;
  uint16_t* ys = lds + GZ_T * P_LD;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wl = (wave % G::kWavesL) * G::TL * 32, wc = (wave / G::kWavesL) * G::TC * 32;
  // A lane's offsets inside a step are constants (groups and columns outside the matrix point past the buffer);
  // the buffers start at the step's first token and end with the last one's row, so later tokens read zero.
  const uint32_t p_row = (uint32_t)(kPieces * a.Lp) * 2u, y_row = (uint32_t)a.d_out * 2u;
  const int pr0 = tid / P_CH, pl = l0 + 8 * (tid % P_CH), yr0 = tid / Y_CH, yj = j0 + 8 * (tid % Y_CH);
  const bool p_ok = pl < a.Lp, y_ok = yj < a.d_out;
  uint32_t p_off = (uint32_t)pr0 * p_row + 2u * (uint32_t)pl, y_off = (uint32_t)yr0 * y_row + 2u * (uint32_t)yj;
  u32x4 pr[kPieces][P_LOADS], yr[Y_LOADS];  // the next step's, while this one is worked on
  auto fetch = [&](int t) {
    const size_t from = (size_t)min(t, t1), rows = (size_t)(t1 - (int)from);
    const __amdgpu_buffer_rsrc_t rs_p = rsrc(a.P + from * kPieces * a.Lp, rows * p_row);
    const __amdgpu_buffer_rsrc_t rs_y = rsrc(a.dy + from * a.d_out, rows * y_row);
    asm volatile("" : "+v"(p_off), "+v"(y_off));  // (a register for each load's offset, kept over the loop, is too many)
#pragma unroll
    for (int q = 0; q < P_LOADS; ++q)
#pragma unroll
      for (int h = 0; h < kPieces; ++h) {
        const uint32_t o = p_off + (uint32_t)(256 / P_CH * q) * p_row + 2u * (uint32_t)(h * a.Lp);
        pr[h][q] = __builtin_amdgcn_raw_buffer_load_b128(rs_p, (int)(p_ok ? o : kOob), 0, 0);
      }
#pragma unroll
    for (int q = 0; q < Y_LOADS; ++q) {
      const uint32_t o = y_off + (uint32_t)(256 / Y_CH * q) * y_row;
      yr[q] = __builtin_amdgcn_raw_buffer_load_b128(rs_y, (int)(y_ok ? o : kOob), 0, 0);
    }
  };
  const bool busy = l0 + wl < a.L;
  fetch(t0);
  for (int t = t0; t < t1; t += GZ_T) {
#pragma unroll
    for (int q = 0; q < P_LOADS; ++q)
#pragma unroll
      for (int h = 0; h < kPieces; ++h)
        *reinterpret_cast<u32x4*>(ps + (pr0 + 256 / P_CH * q) * P_LD + h * GZ_L + pl - l0) = pr[h][q];
#pragma unroll
    for (int q = 0; q < Y_LOADS; ++q)
      *reinterpret_cast<u32x4*>(ys + (yr0 + 256 / Y_CH * q) * G::Y_LD + yj - j0) = yr[q];
    lds_barrier();
    fetch(t + GZ_T);  // (past the end: reads zero)
    if (busy) {
      // the operands of the next sixteen tokens are read while the matrix cores work on these
      bf16x8 y[2][G::TC], p[2][kPieces][G::TL];
      auto read = [&](int kk) {
#pragma unroll
        for (int c = 0; c < G::TC; ++c) y[kk & 1][c] = read_columns(ys + 16 * kk * G::Y_LD + wc + 32 * c, G::Y_LD, lane);
#pragma unroll
        for (int h = 0; h < kPieces; ++h)
#pragma unroll
          for (int l = 0; l < G::TL; ++l) p[kk & 1][h][l] = read_columns(ps + 16 * kk * P_LD + h * GZ_L + wl + 32 * l, P_LD, lane);
      };
      read(0);
#pragma unroll
      for (int kk = 0; kk < GZ_T / 16; ++kk) {
        if (kk + 1 < GZ_T / 16) read(kk + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < kPieces; ++h)
#pragma unroll
          for (int l = 0; l < G::TL; ++l)
#pragma unroll
            for (int c = 0; c < G::TC; ++c)
              acc[l][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[kk & 1][h][l], y[kk & 1][c], acc[l][c], 0, 0, 0);
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
__global__ __launch_bounds__(256, 2) void z_kernel(const ZArgs a) {
  extern __shared__ __align__(16) uint16_t zlds[];
  using G = ZTile<GZ_C>;
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
    z_tile<GZ_C>(a, l0, j0, k0 * GZ_T, min(a.T, k1 * GZ_T), zlds, acc);
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

__global__ __launch_bounds__(256) void fused_kernel(const ZArgs z, const FinishArgs a) {
  extern __shared__ __align__(16) uint16_t zlds[];
  using G = ZTile<GF_C>;
  const int j0 = (int)blockIdx.x * GF_C, l0 = (int)blockIdx.y * GZ_L, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Finish<4> finish(a, part_of(a, j0), j0, l0, reinterpret_cast<float*>(zlds + G::kLds / 2));
  f32x16 acc[1][1];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.0f;
  z_tile<GF_C>(z, l0, j0, 0, z.T, zlds, acc);
  const int c = lane & 31;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 32 * wave + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    finish.zs[row * GF_LD + c] = (l0 + row < a.L && j0 + c < a.d_out) ? acc[0][0][r] : 0.0f;
  }
  finish.run();
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
      const f32x4 v = sum_slices(reinterpret_cast<const f32x4*>(ts.sum.partial) + i, ts.sum.n4, ts.sum.slices);
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

int grads_da_shares(int d_out) { return ceil_div(d_out, GF_C); }
int grads_db_shares(int L) { return L <= GZ_L ? 0 : ceil_div(L, GZ_L); }

// Few tokens and no more blocks than compute units: one launch (forward and backward of 64 tokens, 1024 x 1024
// rank 16: 37.7 us against 42.1 with two; 512 of 4096 x 4096 rank 64: 107 / 112; 1024 of 2048 x 2048: 86.9 / 85.1;
// 128 of 4096 x 11008, 344 blocks: 108.6 / 106.5).
// Blocks of z_kernel: one per compute unit, two where the runs are long -- a unit with two blocks takes 1.2 us per
// step instead of 1.4, but twice as many partial sums are written and read again (4096 tokens: 4096 x 22016
// 66 us against 98, 4096 x 4096 20.3 + 13.2 with their sums against 18.8 + 10.6).
GradsPlan grads_plan(int T, int L, int d_out) {
  GradsPlan p{};
  const int steps = ceil_div(T, GZ_T), tiles = ceil_div(d_out, GZ_C) * ceil_div(L, GZ_L);
  p.fused = T <= 640 && ceil_div(d_out, GF_C) * ceil_div(L, GZ_L) <= 256;
  if (p.fused) return p;
  const long units = (long)steps * tiles;
  p.runs.steps = steps;
  p.runs.units = (int)units;
  p.runs.blocks = (int)std::min(units, units > 8192 ? 512L : 256L);
  p.slots = std::min(steps, ceil_div(p.runs.blocks, tiles) + 1);
  return p;
}

template <typename K>
static hipError_t grant(K kernel, size_t smem, std::atomic<uint64_t>& granted) {
  return smem > 48 * 1024 ? grant_dynamic_lds(reinterpret_cast<const void*>(kernel), (int)smem, granted) : hipSuccess;
}

hipError_t launch_grads(const GradsPlan& plan, const ZArgs& z, const FinishArgs& f, hipStream_t st) {
  int max_rank = 0;
  for (int q = 0; q < f.n_parts; ++q) max_rank = std::max(max_rank, f.part[q].rank);
  const size_t finish = (size_t)finish_floats(max_rank) * 4, most = (size_t)finish_floats(kMaxRank) * 4;
  const dim3 blocks(ceil_div(f.d_out, GF_C), ceil_div(f.L, GZ_L));
  if (plan.fused) {
    static std::atomic<uint64_t> granted{0};
    if (hipError_t e = grant(fused_kernel, ZTile<GF_C>::kLds + most, granted); e != hipSuccess) return e;
    fused_kernel<<<blocks, 256, ZTile<GF_C>::kLds + finish, st>>>(z, f);
    return hipGetLastError();
  }
  static std::atomic<uint64_t> granted_z{0}, granted_f{0};
  if (hipError_t e = grant(z_kernel, ZTile<GZ_C>::kLds, granted_z); e != hipSuccess) return e;
  if (hipError_t e = grant(finish_kernel, most, granted_f); e != hipSuccess) return e;
  z_kernel<<<plan.runs.blocks, 256, ZTile<GZ_C>::kLds, st>>>(z);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  finish_kernel<<<blocks, 64 * FINISH_WAVES, finish, st>>>(f);
  return hipGetLastError();
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
