// Error-compensated code selection: the role the post-training quantizer plays in the paper's
// experiments (Sec. 4.1, quantization settings; App. B.1: the layer takes whatever codes, scales
// and zeros that quantizer hands over).  The published procedure, restated for W [d_in x d_out]
// with groups down the input rows: the rows are quantized in order; the error a row leaves,
// divided by the diagonal of U (the upper Cholesky factor of the inverse input Hessian,
// H^-1 = U^T U), is spread over the rows not yet quantized with the weights U[i, r], so that
// the output error tr((W - W~)^T H (W - W~)) shrinks; a group's beta and alpha are taken, by
// Eq. 1's min-max recipe, from the group's rows as they stand when its first row is reached;
// rows beyond the current block of kBlock rows receive the block's errors in one lazy update.
//
// The operation order is part of the definition (fp32, fused multiply-adds, every sum in
// ascending row order), so the codes are reproducible bit for bit:
//   inside a block of 128 rows   w_r <- fma(-U[i,r], e_i, w_r)            for i = first row .. r - 1
//   beyond it, once per block    w_r <- w_r - (fma chain from 0 over the block's 128 rows)
// Both are chains v_mfma_f32_16x16x4_f32 computes exactly: that instruction adds its four
// products one after the other, k ascending, each with one rounding (checked on the device
// against fmaf, subnormals included; the bit-exact tests stand on it).
//
// What bounds it: d_in dependent rows (a rounding, a division by U[i,i] and an update each) and
// d_in^2 d_out / 2 multiply-adds.  A block of four wavefronts, one per SIMD, owns 16 columns -- one
// matrix tile; 256 blocks for a 4096-column layer -- and runs the two side by side:
//   * ONE wavefront walks the rows of the current 128-row panel.  Sixteen rows at a time are
//     held whole in every lane's registers (lane = column; the four lane groups repeat each
//     other), so a row costs no barrier, no LDS round trip and no cross-lane step; the sixteen
//     rows' errors then go to the panel's later rows as matrix instructions.
//   * THREE wavefronts meanwhile bring the NEXT panel up to date with all finished blocks
//     (left-looking: W is read once, the blocks' errors are kept instead and re-read as matrix
//     operands), so that only the newest block's errors remain to be applied when the walker
//     is done.  (Four of them, one sharing the walker's SIMD, are slower: vector and matrix
//     instructions of a SIMD take turns, so that SIMD's times add up.)
// Two barriers per panel.
// The divisions of the walk.  e = t / U[i,i] is a product with the reciprocal in two parts and one
// remainder step (Markstein's theorem: with the correctly rounded reciprocal and a quotient
// within one unit in the last place the result is the correctly rounded quotient, while nothing
// under- or overflows).  The code needs the quotient (w - beta) / alpha only up to rounding to an
// integer: a product with a reciprocal within one unit in the last place is within three units, and
// decides the same integer unless it lies next to a tie.  Sixteen rows in which some operand
// leaves the range where this holds, or some quotient comes near a tie, are done again with
// real divisions.
// The walker is the longer part up to about 2048 rows and stays issue bound there: about 170 cycles per row, 500 to
// 1900 per sixteen rows for the matrix work behind them.  Its panel's triangle of U lies in LDS (loads of U by the
// walker itself took 860 cycles per sixteen rows), a new group's min-max crosses lanes in registers and its division
// by the number of levels needs no division (1160 cycles per group before, 300 now): 42 -> 34 thousand cycles per panel.
// INT4 g = 32, us: 4096 x 4096 10130 with 16 columns x 64 row lanes, a barrier per row and two LDS operands per
// multiply-add; 920 with a walker and updaters, 860 with the walker of today; 2048 x 4096 397 -> 340; 1024 x 4096
// 182 -> 149; 512 x 2048 91 -> 76.  (Updaters that work ahead on later panels while the walker is the longer part:
// 940 and 3 % off the smaller ones; their panels' way to memory and back costs what the even load saves.)
#include <type_traits>

#include "common.hpp"
#include "compensate_addr.hpp"
#include "kernels.hpp"

namespace qalora {

namespace {
constexpr int kBlock = kCompBlock;
constexpr int kCols = 16;                // columns per thread block
constexpr int kTiles = kBlock / 16;      // 16-row tiles of a panel
constexpr int kUpd = 3;                  // updating wavefronts: three tiles (48 rows) each, the last one two
constexpr int kThreads = 64 * (kUpd + 1);
constexpr int kTrLd = 20;                // floats per column of the transposed sub-block (16 + 4: bank spread)

struct CompArgs {
  const float* W;
  const float* U;
  int d_in, d_out, g;
  float* err;        // errors of finished blocks: 16-row blocks of a column block, [kb][column][4] each
  uint32_t* plane0;
  uint32_t* plane1;
  float* alpha;
  float* beta;
};

// f(integral_constant<I>), ..., f(integral_constant<N - 1>): loops over register arrays whose indices must
// stay constants (left to the optimiser, the row loops below were rolled up again and the
// registers indexed at run time)
template <int I, int N, typename Fn>
__device__ __forceinline__ void static_for(Fn&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr uint32_t kOob = 0xffff0000u;  // past every buffer below: reads zero
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)(bytes > kOob ? kOob : bytes), 0x00020000);
}
__device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
}
__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
}

// LDS-only barrier: does not wait for the global loads that are in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// f over the four rows of sixteen lanes, in every lane (two exchanges in registers)
template <typename F>
__device__ __forceinline__ float over_rows(float v, F&& f) {
  const uint32_t w = __float_as_uint(v);
  const auto h = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  const uint32_t m = __float_as_uint(f(__uint_as_float(h[0]), __uint_as_float(h[1])));
  const auto g = __builtin_amdgcn_permlane32_swap(m, m, false, false);
  return f(__uint_as_float(g[0]), __uint_as_float(g[1]));
}

// |v| in [2^-60, 2^60]
__device__ __forceinline__ bool in_safe_range(float v) { return fabsf(v) >= 0x1p-60f && fabsf(v) <= 0x1p60f; }
}  // namespace

template <int NBITS>
__global__ __launch_bounds__(kThreads, 2) void compensate_kernel(const CompArgs p) {
  __shared__ f32x4 tile[kTiles * 64];  // the panel to be walked, as matrix accumulator fragments
  __shared__ f32x4 errs[kTiles * 64];  // the walked panel's errors, as matrix operand fragments
  __shared__ float tr[kCols * kTrLd];  // the walker's sixteen rows, column by column
  // U of the walked panel: 16 x 16 blocks (s, t >= s), and room for a row of seven read past the last one
  __shared__ __align__(16) float up[(kTiles * (kTiles + 1) / 2 + kTiles - 1) * 256];
  __shared__ f32x2 rcp[kBlock];        // 1 / U[i,i] of the panel's rows: rounded, and what is left of it
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool walker = wave == kUpd;
  const int n = lane & 15, kb = lane >> 4;  // column; rows 4 kb + r of a fragment
  const int d_in = p.d_in, d_out = p.d_out, g = p.g;
  const uint32_t row_b = (uint32_t)d_in * 4u;  // bytes of a row of U
  const int j0 = blockIdx.x * kCols, j = j0 + n;
  const int nc = min(kCols, d_out - j0);  // 16, or 8 at the right edge
  const bool col_ok = n < nc;
  const float* __restrict__ U = p.U;
  // this column block's share of the error store; a fragment of 16 rows is 16 nc floats
  float* err = p.err + (size_t)j0 * d_in;
  const int e_lane = (kb * nc + min(n, nc - 1)) * 4;
  const int panels = ceil_div(d_in, kBlock);

  // An updating wavefront's 16 NT rows are dealt to its NT tiles in turn -- row m of tile h is
  // r0 + NT m + h -- so that a lane's NT elements of a row of U are adjacent (one load).
  auto load_w = [&](auto nt_c, int r0, f32x4* v) {  // zeros outside the matrix
    constexpr int NT = decltype(nt_c)::value;
#pragma unroll
    for (int h = 0; h < NT; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = r0 + NT * (4 * kb + r) + h;
        v[h][r] = (row < d_in && col_ok) ? p.W[(size_t)row * d_out + j] : 0.0f;
      }
  };
  // ... into the walker's fragments: row 16 t + 4 k + r of the panel at lane (n, k) of tile t
  float* tile_f = reinterpret_cast<float*>(tile);
  auto store_tile = [&](auto nt_c, const f32x4* v) {
    constexpr int NT = decltype(nt_c)::value;
#pragma unroll
    for (int h = 0; h < NT; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 48 * wave + NT * (4 * kb + r) + h;
        tile_f[((row >> 4) * 64 + 16 * ((row >> 2) & 3) + n) * 4 + (row & 3)] = v[h][r];
      }
  };

  if (!walker) {
    auto update = [&](auto nt_c) __attribute__((always_inline)) {
      constexpr int NT = decltype(nt_c)::value;
      f32x4 cur[NT], nxt[NT];  // the tiles being brought up to date; W of the ones after
      float u[kTiles][4][NT];  // U of one block of rows, eight pieces of 16
      f32x4 ev[kTiles];        // the block's errors
      const uint32_t e_off = 4u * (uint32_t)e_lane, e_step = 64u * (uint32_t)nc;  // bytes
      auto rs_u = [&](int blk) { return rsrc(U + (size_t)blk * kBlock * d_in, (size_t)comp_block_rows(d_in, blk) * row_b); };
      auto rs_e = [&](int blk) { return rsrc(err + (size_t)blk * kBlock * nc, (size_t)kTiles * e_step); };
      // U operand: lane (row m = n of the tiles, kb) supplies U[i + 4 q + kb][r0 + NT n + h]; columns
      // outside the matrix are some other element of U (or zero): they reach rows outside the matrix only
      auto u_offset = [&](int r0) { return comp_update_lane(row_b, NT, r0, n, kb); };
      auto load_u = [&](int k, __amdgpu_buffer_rsrc_t r, uint32_t off) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t so = comp_update_row(row_b, k, q);
          if constexpr (NT == 3) {
            const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(r, (int)off, (int)so, 0);
#pragma unroll
            for (int h = 0; h < 3; ++h) u[k][q][h] = __uint_as_float(v[h]);
          } else {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, (int)so, 0);
#pragma unroll
            for (int h = 0; h < 2; ++h) u[k][q][h] = __uint_as_float(v[h]);
          }
        }
      };
      load_w(nt_c, 48 * wave, cur);
      store_tile(nt_c, cur);
      int r0 = kBlock + 48 * wave;
      uint32_t u_off = u_offset(r0);
      load_w(nt_c, r0, cur);
      if (comp_updates(panels)) {
#pragma unroll
        for (int k = 0; k < kTiles; ++k) load_u(k, rs_u(0), u_off);
      }
      lds_barrier();  // the first panel is in place
      for (int pn = 0; pn < panels; ++pn) {
        // (rows past the end of a ragged last panel come to hold sums over whatever their columns' loads of U
        // returned; the walker takes them through its sixteen rows and stores nothing of them)
        const bool work = pn + 1 < panels;
        if (work) {
          // a piece's registers are reloaded for the next block as soon as it has been used, so a
          // whole block of loads is in flight
          for (int blk = 0; blk < pn; ++blk) {
            f32x4 acc[NT];
#pragma unroll
            for (int h = 0; h < NT; ++h) acc[h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            // U ends with block pn; its errors are not known yet: the last known block's are loaded again
            const __amdgpu_buffer_rsrc_t ru = rs_u(blk + 1), re = rs_e(min(blk + 1, pn - 1));
#pragma unroll
            for (int k = 0; k < kTiles; ++k) {
#pragma unroll
              for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int h = 0; h < NT; ++h)
                  acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(u[k][q][h], ev[k][q], acc[h], 0, 0, 0);
              __builtin_amdgcn_sched_barrier(0);
              load_u(k, ru, u_off);
              ev[k] = load4(re, e_off, (uint32_t)k * e_step);
              __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int h = 0; h < NT; ++h)
#pragma unroll
              for (int r = 0; r < 4; ++r) cur[h][r] = __fsub_rn(cur[h][r], acc[h][r]);
          }
        }
        lds_barrier();  // block pn's errors are known
        if (work) {
          // block pn, and the loads the next panel starts with
          r0 += kBlock;
          u_off = u_offset(r0);
          load_w(nt_c, r0, nxt);
          const __amdgpu_buffer_rsrc_t ru = rs_u(0), re = rs_e(0);
          f32x4 acc[NT];
#pragma unroll
          for (int h = 0; h < NT; ++h) acc[h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
          f32x4 el[kTiles];
#pragma unroll
          for (int k = 0; k < kTiles; ++k) el[k] = errs[k * 64 + lane];
#pragma unroll
          for (int k = 0; k < kTiles; ++k) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int h = 0; h < NT; ++h)
                acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(u[k][q][h], el[k][q], acc[h], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            load_u(k, ru, u_off);
            ev[k] = load4(re, e_off, (uint32_t)k * e_step);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int h = 0; h < NT; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) cur[h][r] = __fsub_rn(cur[h][r], acc[h][r]);
          store_tile(nt_c, cur);
#pragma unroll
          for (int h = 0; h < NT; ++h) cur[h] = nxt[h];
        }
        lds_barrier();  // the next panel is in place
      }
    };
    if (wave + 1 < kUpd) update(std::integral_constant<int, 3>{});
    else update(std::integral_constant<int, 2>{});
    return;
  }

  // ---- the walker ---------------------------------------------------------------------------
  // The panel's triangle of U goes straight to LDS (a 16 x 16 block per load, 16 bytes a lane) while the updating
  // wavefronts bring the panel itself into place: walking it needs no other memory.  Rows and columns outside the
  // matrix read zero.
  constexpr auto block_of = [](int s, int t) { return (s * (2 * kTiles + 1 - s) / 2 + t - s) * 256; };
  auto fetch_u = [&](int pn) {
    const int rows = comp_block_rows(d_in, pn), c0 = pn * kBlock + 4 * (lane & 3);
    const __amdgpu_buffer_rsrc_t r = rsrc(U + (size_t)pn * kBlock * d_in, (size_t)rows * row_b);
#pragma unroll
    for (int s = 0; s < kTiles; ++s) {
      const uint32_t row = comp_walk_row(row_b, rows, s, lane >> 4) + (uint32_t)((lane >> 2) & 3) * row_b + 4u * (uint32_t)c0;
#pragma unroll
      for (int t = s; t < kTiles; ++t)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(up + block_of(s, t)), 16,
                                                 (int)(c0 + 16 * t < d_in ? row + 64u * (uint32_t)t : kOob), 0, 0, 0);
    }
  };
  fetch_u(0);
  lds_barrier();  // the first panel is in place
  float a = 1.0f, b = 0.0f, ya = 1.0f;  // walker: the column's current group: alpha, beta, 1 / alpha
  for (int pn = 0; pn < panels; ++pn) {
    const int i1 = pn * kBlock;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // its triangle of U too
    bool odd = false;  // a diagonal element outside the reciprocal's range
#pragma unroll
    for (int h = 0; h < kBlock / 64; ++h) {
      const int i = 64 * h + lane, s = i >> 4;
      const float d = i1 + i < d_in ? up[s * (2 * kTiles + 1 - s) / 2 * 256 + (i & 15) * 17] : 1.0f;
      const float y = __fdiv_rn(1.0f, d);
      rcp[i] = f32x2{y, __fmul_rn(__fmaf_rn(-d, y, 1.0f), y)};
      odd |= !(d >= 0x1p-40f && d <= 0x1p40f);
    }
    const bool any_odd = __any(odd);
    f32x4 pt[kTiles];  // pt[t]: tile s + t of the panel, rotating with the sub-block s
#pragma unroll
    for (int t = 0; t < kTiles; ++t) pt[t] = tile[t * 64 + lane];
    uint32_t hiword = 0;  // 3 bits: the high-bit word, two sub-blocks per word
    for (int s = 0; s < kTiles; ++s) {
      const int row0 = i1 + 16 * s;
      if (row0 >= d_in) break;
      *reinterpret_cast<f32x4*>(tr + n * kTrLd + 4 * kb) = pt[0];
      const float* us = up + block_of(s, s);
      // U of this sub-block's rows against the panel's later tiles: requested now, used after the walk (tiles past
      // the panel: other blocks' numbers, unused)
      float au[kTiles - 1][4];
#pragma unroll
      for (int t = 1; t < kTiles; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) au[t - 1][q] = us[t * 256 + q * 64 + lane];
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" ::: "memory");  // one wavefront: its LDS accesses complete in order

      f32x4 eb;  // the sixteen errors as the matrix operand: lane (column n, kb) supplies rows 4 q + kb
      uint32_t word0 = 0, word1 = 0;
      float a_s, b_s, ya_s;  // the group state after the sixteen rows
      uint32_t hi_s;
      auto walk = [&](auto fast_c) __attribute__((always_inline)) -> bool {  // true: an operand left the safe range
        constexpr bool FAST = decltype(fast_c)::value;
        float w[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(tr + n * kTrLd + 4 * q);
#pragma unroll
          for (int r = 0; r < 4; ++r) w[4 * q + r] = v[r];
        }
        a_s = a, b_s = b, ya_s = ya, hi_s = hiword;
        word0 = word1 = 0;
        bool bad = !in_safe_range(a);
        // |t| in [2^-60, 2^60] or +0 (as bits rotated left by one, less one: +0 comes out largest, -0
        // smallest), and how near the quotients come to a tie
        uint32_t tmin = 0xffffffffu;
        float tmax = 0.0f, dmax = 0.0f;
        const float levels = (float)((1 << NBITS) - 1);
        f32x4 ur[3][4];  // the row's piece of U and the next two's, requested two rows ahead
        f32x2 ry[3];
        auto fetch_row = [&](auto i_c) {
          constexpr int i = decltype(i_c)::value;
          static_for<i / 4, 4>([&](auto q) {
            ur[i % 3][decltype(q)::value] = *reinterpret_cast<const f32x4*>(us + 16 * i + 4 * decltype(q)::value);
          });
          ry[i % 3] = rcp[16 * s + i];
        };
        fetch_row(std::integral_constant<int, 0>{});
        fetch_row(std::integral_constant<int, 1>{});
        static_for<0, 16>([&](auto i_c) {
          constexpr int i = decltype(i_c)::value;
          if constexpr (i + 2 < 16) fetch_row(std::integral_constant<int, i + 2>{});
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (i == 0 || i == 8) {
            if ((row0 + i) % g == 0) {  // a new group: min-max of its rows as they stand (Eq. 1)
              float mn, mx;
              if (i == 8 || g == 8) {
                mn = mx = w[i];
                static_for<1, 8>([&](auto q_c) {
                  constexpr int q = i < 9 ? i + decltype(q_c)::value : 15;
                  mn = w[q] < mn ? w[q] : mn;
                  mx = w[q] > mx ? w[q] : mx;
                });
              } else {
                const int nt = g >> 4;
                mn = mx = pt[0][0];
                static_for<0, kTiles>([&](auto t_c) {
                  constexpr int t = decltype(t_c)::value;
                  if (t < nt) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                      mn = fminf(mn, pt[t][r]);
                      mx = fmaxf(mx, pt[t][r]);
                    }
                  }
                });
                mn = over_rows(mn, [](float p, float q) { return fminf(p, q); });
                mx = over_rows(mx, [](float p, float q) { return fmaxf(p, q); });
                if (w[i] != w[i]) mn = mx = w[i];  // a NaN in the group's first row stays (as above), others are passed over
                if (__any(mn == 0.0f)) {  // a minimum of zero keeps the sign of the first zero of the group
                  int key = 1 << 20;
                  static_for<0, kTiles>([&](auto t_c) {
                    constexpr int t = decltype(t_c)::value;
                    if (t < nt) {
#pragma unroll
                      for (int r = 0; r < 4; ++r)
                        if (pt[t][r] == 0.0f)
                          key = min(key, 2 * (16 * t + r) + (int)(__float_as_uint(pt[t][r]) >> 31));
                    }
                  });
                  key += 8 * kb;  // the lane's rows are 4 kb + r of each tile
                  key = min(key, __shfl_xor(key, 16, 64));
                  key = min(key, __shfl_xor(key, 32, 64));
                  if (mn == 0.0f) mn = (key & 1) ? -0.0f : 0.0f;
                }
              }
              // (one product and one remainder step give the rounded quotient for each of these divisors: checked for
              // all significands; the reciprocal of alpha is within a unit in the last place)
              const float range = __fsub_rn(mx, mn);
              constexpr float kInverse = 1.0f / (float)((1 << NBITS) - 1);
              const float q0 = __fmul_rn(range, kInverse);
              a_s = __fmaf_rn(__fmaf_rn(-levels, q0, range), kInverse, q0);
              if (__any(!in_safe_range(range))) a_s = __fdiv_rn(range, levels);
              if (!(a_s > 0.0f)) a_s = 0x1p-60f;
              b_s = mn;
              ya_s = __builtin_amdgcn_rcpf(a_s);
              bad |= !in_safe_range(a_s);
              if (kb == 0 && col_ok && row0 + i < d_in) {
                const size_t o = (size_t)((row0 + i) / g) * d_out + j;
                p.alpha[o] = a_s;
                p.beta[o] = b_s;
              }
            }
          }
          const float x = __fsub_rn(w[i], b_s);
          float rq, q;
          if constexpr (FAST) {
            const float q0 = __fmul_rn(x, ya_s), rn = rintf(q0);
            dmax = fmaxf(dmax, fabsf(__fsub_rn(q0, rn)));
            rq = __builtin_amdgcn_fmed3f(rn, 0.0f, levels);
          } else {
            rq = rintf(__fdiv_rn(x, a_s));
            if (!(rq >= 0.0f)) rq = 0.0f;
            if (rq > levels) rq = levels;
          }
          const float t = __fsub_rn(w[i], __fmaf_rn(a_s, rq, b_s));
          const float d = ur[i % 3][i / 4][i % 4];
          if constexpr (FAST) {
            const float q1 = __fmaf_rn(t, ry[i % 3][0], __fmul_rn(t, ry[i % 3][1]));
            q = __fmaf_rn(__fmaf_rn(-d, q1, t), ry[i % 3][0], q1);
            const uint32_t tb = __float_as_uint(t);
            tmin = min(tmin, ((tb << 1) | (tb >> 31)) - 1u);
            tmax = fmaxf(tmax, fabsf(t));
          } else {
            q = __fdiv_rn(t, d);
          }
          eb[i >> 2] = (i & 3) == 0 || kb == (i & 3) ? q : eb[i >> 2];
          static_for<i + 1, 16>([&](auto r_c) {
            constexpr int r = decltype(r_c)::value;
            w[r] = __fmaf_rn(-ur[i % 3][r / 4][r % 4], q, w[r]);
          });
          // (the parts of a fetched row that no update needs stay allocated until here: given to another fetch
          // sooner, that fetch would first wait for this one's data)
          static_for<i / 4, 4>([&](auto q_c) {
            const f32x4 part = ur[i % 3][decltype(q_c)::value];
            asm volatile("" ::"v"(part));
          });
          const f32x2 inverse = ry[i % 3];
          asm volatile("" ::"v"(inverse));
          const uint32_t c = (uint32_t)(int)rq;
          if constexpr (NBITS == 4) {
            constexpr int ps = 4 * ((i & 7) >> 1) + 16 * (i & 1);
            if constexpr (i < 8) word0 |= c << ps;
            else word1 |= c << ps;
          } else {
            word0 |= (c & 3u) << (2 * (i >> 1) + 16 * (i & 1));
            if constexpr (NBITS == 3) hi_s |= (c >> 2) << ((i >> 1) + 16 * (i & 1) + 8 * (s & 1));
          }
        });
        // (2^-60 has the bits 67 << 23; a quotient of up to 31 carries an error below 2^-17, larger
        // ones are clamped whichever way they round)
        return bad || tmin < (67u << 24) - 1u || !(tmax <= 0x1p60f) || !(dmax < 0.5f - 0x1p-16f);
      };
      if (any_odd || __any(walk(std::true_type{}))) walk(std::false_type{});
      a = a_s, b = b_s, ya = ya_s, hiword = hi_s;

      errs[s * 64 + lane] = eb;
      if (pn + 1 < panels && col_ok) *reinterpret_cast<f32x4*>(err + (size_t)(row0 >> 4) * 16 * nc + e_lane) = eb;
      if (col_ok) {
        if constexpr (NBITS == 4) {
          if (kb < 2 && row0 + 8 * kb < d_in) p.plane0[(size_t)(row0 / 8 + kb) * d_out + j] = kb ? word1 : word0;
        } else {
          if (kb == 0) p.plane0[(size_t)(row0 / 16) * d_out + j] = word0;
          if constexpr (NBITS == 3)
            if (kb == 1 && (s & 1)) p.plane1[(size_t)(row0 / 32) * d_out + j] = hiword;
        }
      }
      if (s & 1) hiword = 0;
      // ... onto the panel's later tiles, exactly as many as there are (the switch keeps the
      // chains of different tiles interleaved without computing absent ones)
      f32x4 ne;
#pragma unroll
      for (int q = 0; q < 4; ++q) ne[q] = -eb[q];
      auto behind = [&](auto nt_c) {
        constexpr int NT = decltype(nt_c)::value;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int t = 1; t <= NT; ++t)
            pt[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(au[t - 1][q], ne[q], pt[t], 0, 0, 0);
      };
      switch (kTiles - 1 - s) {
        case 7: behind(std::integral_constant<int, 7>{}); break;
        case 6: behind(std::integral_constant<int, 6>{}); break;
        case 5: behind(std::integral_constant<int, 5>{}); break;
        case 4: behind(std::integral_constant<int, 4>{}); break;
        case 3: behind(std::integral_constant<int, 3>{}); break;
        case 2: behind(std::integral_constant<int, 2>{}); break;
        case 1: behind(std::integral_constant<int, 1>{}); break;
        default: break;
      }
#pragma unroll
      for (int t = 0; t + 1 < kTiles; ++t) pt[t] = pt[t + 1];
    }
    // block pn's errors are known: in LDS, and (for this block's later loads) in the error store
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (pn + 1 < panels) fetch_u(pn + 1);
    lds_barrier();  // the next panel is in place
  }
}

// err: d_in * d_out fp32 of scratch.  g must divide 128.
hipError_t launch_compensate(const float* W, const float* U, int d_in, int d_out, int bits, int g,
                             float* err, void* packed, float* alpha, float* beta, hipStream_t st) {
  if (kBlock % g != 0 || d_out % 8 != 0 || d_in % 8 != 0) return hipErrorInvalidValue;
  CompArgs a{};
  a.W = W;
  a.U = U;
  a.d_in = d_in;
  a.d_out = d_out;
  a.g = g;
  a.err = err;
  a.plane0 = static_cast<uint32_t*>(packed);
  a.plane1 = a.plane0 + plane0_words(bits, d_in, d_out);
  a.alpha = alpha;
  a.beta = beta;
  const int grid = ceil_div(d_out, kCols);
  if (bits == 4) compensate_kernel<4><<<grid, kThreads, 0, st>>>(a);
  else if (bits == 3) compensate_kernel<3><<<grid, kThreads, 0, st>>>(a);
  else compensate_kernel<2><<<grid, kThreads, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace qalora
