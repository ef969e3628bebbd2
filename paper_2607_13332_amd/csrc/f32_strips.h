// Column-strip kernel over the columns of float32 matrices (see the comment
// at the kernel): the weight re-projection W <- U (U^T W) and, in its FG
// mode, the reparameterized layer's factor gradient.  Included by the
// translation units that instantiate it (its launcher is explicitly
// instantiated for 1..4 and 5..8 k tiles in two units that compile in
// parallel) and by the one that dispatches.
#pragma once

#include "ssn_device.h"
#include "ssn_launch.h"

#include <type_traits>

namespace ssn {

// ===========================================================================
// Weight re-projection W <- U (U^T W) with float32 storage (the original SSN's
// step after each optimizer update, sections 4.1 and 6.1).
//
// Products: every float32 operand is split into three bf16 planes that hold
// its 24 bits (split3_bf16x8) and a product takes the six plane pairs that
// leave out at most 2^-24 of it, on the bf16 matrix cores: 6 instructions of 16x16x32 (96
// cycles) do the work of 8 of 16x16x4 in float32 (256 cycles).  The five
// small pairs of a K step are summed on their own and added to the running
// sum once, so a running sum is rounded twice per 32 products (the float32
// MFMA rounds it once per product).
//
// The columns of all matrices of a batch form one sequence of strips of
// 16 NT columns; RS waves of a block own a strip (they share its rows) and a
// block owns cs <= 8 / RS strips.  W never goes through LDS: lane (n16, g)
// loads the NT consecutive columns NT n16 .. of rows 8 g + e (e = 0..7) of a
// 32-row step, 4 rows x 64 NT contiguous bytes per instruction, and column
// tile i of the MFMAs is the columns NT n16 + i, so the eight values it
// holds of a column are that column's B operand as they are.
// Pass 1, T = U^T W: U's planes are staged per block in A-operand order,
// double buffered, one barrier per SR steps (thread task: 8 rows of one
// column, so any k is read whole); W runs two steps ahead in registers.
// With RS > 1 the partial sums of a strip's waves are added through LDS in a
// fixed order.  Lane (n16, g) then holds T[16 kt + 4 g + r][its column of
// tile i].
// Pass 2, W = U T: K slot (g, e) of K step s stands for coordinate
// 32 s + 4 g + e (e < 4) and 32 s + 16 + 4 g + e - 4, so T stays in the
// registers that pass 1 left it in (split once), U's planes are staged in
// that order, and a lane ends with rows 4 g + r of its NT columns: stored as
// they are, 4 rows x 64 NT contiguous bytes per instruction (non-temporal).
// A wave whose T the planes cannot vouch for (planes_unsure: an infinity or
// NaN in W or U, an element below 2^-80) redoes both passes with float32 MFMAs
// straight from memory, which propagate infinities and NaN as float32
// arithmetic does.
//
// Bound: HBM, W read once and written once.  Measured on MI355X against the
// kernel that multiplied float32 operands and passed W through LDS: 4 x
// (5120^2, 5120 x 18432) at k = 51 1597 -> 771 us (5.0 TB/s, the rate of a
// large copy); 4 x (4096^2, 4096 x 14336) at k = 64 845 -> 544 us; error
// against 64 bits at 2048^2, k = 51 3.2e-7 -> 1.3e-7.
//
// FG: the reparameterized layer's factor gradient (section 4.1, Eq. (3)),
// dZp = H^T GT, with H [N, din] as the single matrix of the batch, GT [N, k]
// in place of U and N rows in place of d (any N): pass 1 alone, then
// T = GT^T H is written transposed to fg_out [din, k].
// ===========================================================================
struct ColumnBatchF32 {
  float* W[kMaxBatch];
  int32_t n[kMaxBatch];
  int32_t first[kMaxBatch + 1];        // prefix sums of ceil(n / strip width)
  int32_t count;
  int32_t strips;                      // total strips of the batch
  int32_t cs;                          // strips per block
};

constexpr int kS32Waves = 8;
// 32-row steps per staged chunk of pass 1 (every wave of a strip has one at
// least), and rows per chunk of pass 2: U's planes take 48 KB of LDS at the
// widest k of either line, 96 KB where more waves share a strip's rows; there
// pass 1 has one buffer (and a second barrier per chunk) instead of two.
constexpr int s32_steps(int kt, int rs) { return kt <= 4 ? (rs > 4 ? rs : 4) : (rs > 2 ? rs : 2); }
constexpr int s32_rows2(int kt) { return kt <= 4 ? 128 : 64; }
constexpr int cmax3(int a, int b, int c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }

template <int NT>
struct StripVec;
template <>
struct StripVec<4> { typedef f32x4 T; };
template <>
struct StripVec<2> { typedef f32x2 T; };
template <>
struct StripVec<1> { typedef float T __attribute__((ext_vector_type(1))); };

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

template <int KT, int NT, int RS, bool FG>
__global__ __launch_bounds__(64 * kS32Waves) void project_weights_f32_mfma(
    ColumnBatchF32 cb, const float* __restrict__ U, int rows, int k,
    float* __restrict__ fg_out) {
  static_assert((NT == 1 || NT == 2 || NT == 4) && (RS == 1 || RS == 2 || RS == 4 || RS == 8), "strip shape");
  typedef typename StripVec<NT>::T vec;
  constexpr int T = 64 * kS32Waves, K = 16 * KT, KS2 = (KT + 1) / 2;
  constexpr int SR = s32_steps(KT, RS), PS = SR / RS, R2 = s32_rows2(KT);
  static_assert(PS >= 1, "every wave of a strip has a step of each chunk");
  constexpr int F1 = SR * KT * 3 * 64;             // 16-byte pieces of a pass-1 buffer
  constexpr int NB1 = F1 * 32 > 98304 ? 1 : 2;     // pass-1 buffers
  constexpr int F2 = (R2 / 16) * KS2 * 3 * 64;     // and of a pass-2 buffer
  constexpr int FR = RS > 1 ? kS32Waves * KT * NT * 64 : 0;   // partial T of 8 waves
  __shared__ u32x4 smem[cmax3(NB1 * F1, 2 * F2, FR)];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n16 = lane & 15, g = lane >> 4;
  const int grp = wave / RS, rs = wave % RS;
  // XCD order: neighbouring blocks' columns on one XCD (blocks go to the 8
  // XCDs round robin; gridDim.x is a multiple of 8)
  const int bx = (int)((blockIdx.x % 8u) * (gridDim.x / 8u) + blockIdx.x / 8u);
  const int strip = bx * cb.cs + grp;
  const bool active = grp < cb.cs && strip < cb.strips;   // wave-uniform
  int b = 0;
  while (b + 1 < cb.count && (active ? strip : 0) >= cb.first[b + 1]) ++b;
  const int64_t ld = cb.n[b];
  const int64_t colw = (int64_t)((active ? strip : 0) - cb.first[b]) * (16 * NT) + NT * n16;
  const bool on = active && colw < ld;            // n % 4 == 0: all NT columns or none
  float* const wcol = cb.W[b] + (on ? colw : 0);

  const int nsteps = FG ? (rows + 31) / 32 : rows / 32;
  const int nch1 = (nsteps + SR - 1) / SR, nch2 = (rows + R2 - 1) / R2;

  // U of pass 1: task q is column q % K of the 8 rows q / K of the chunk
  constexpr int NT1 = SR * 4 * K, TP1 = (NT1 + T - 1) / T;
  float u1[TP1][8];
  auto load_u1 = [&](int c) {
#pragma unroll
    for (int i = 0; i < TP1; ++i) {
      // Tasks past the chunk's last, columns past k and rows past the end
      // load something in range: their planes meet no W, or make rows k .. K
      // - 1 of T, which pass 2 multiplies by zero.  FG's last step may be
      // ragged: its rows past the end are zero.
      const int q = NT1 % T == 0 ? tid + T * i : min(tid + T * i, NT1 - 1);
      const int col = min(q % K, k - 1), r0 = c * (SR * 32) + 8 * (q / K);
      if constexpr (FG) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = U[(int64_t)min(r0 + e, rows - 1) * k + col];
          u1[i][e] = r0 + e < rows ? x : 0.f;
        }
      } else {
        const float* src = U + (int64_t)min(r0, rows - 8) * k + col;
#pragma unroll
        for (int e = 0; e < 8; ++e) u1[i][e] = src[e * k];
      }
    }
  };
  auto store_u1 = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TP1; ++i) {
      const int q = tid + T * i, col = q % K, rg = q / K;
      u32x4 h, m, l;
      split3_bf16x8(u1[i], h, m, l);
      if (NT1 % T == 0 || q < NT1) {
        u32x4* dst = smem + buf * F1 + ((rg >> 2) * KT + (col >> 4)) * 192 + 16 * (rg & 3) + (col & 15);
        dst[0] = h;
        dst[64] = m;
        dst[128] = l;
      }
    }
  };
  // U of pass 2: task q is piece q % (4 KS2) of row q / (4 KS2), piece p = 4 s +
  // g' the coordinates 32 s + 4 g' + 0..3 and 32 s + 16 + 4 g' + 0..3; within
  // a fragment the slot of (row m, g') is XORed with p, so that the pieces
  // of one row go to different banks
  constexpr int PPR = 4 * KS2, NT2 = R2 * PPR, TP2 = (NT2 + T - 1) / T;
  float u2[TP2][8];
  const int64_t total = (int64_t)rows * k;
  auto load_u2 = [&](int c) {
#pragma unroll
    for (int i = 0; i < TP2; ++i) {
      const int q = NT2 % T == 0 ? tid + T * i : min(tid + T * i, NT2 - 1);
      const int row = min(c * R2 + q / PPR, rows - 1), p = q % PPR;
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const int c0 = 32 * (p >> 2) + 4 * (p & 3) + 16 * hf;
        const int64_t o = (int64_t)row * k + c0;
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
        if (o + 4 <= total) {                     // into the next row, past k
          v = *(const f32x4_a4*)(U + o);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (o + e < total) v[e] = U[o + e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) u2[i][4 * hf + e] = c0 + e < k ? v[e] : 0.f;
      }
    }
  };
  auto store_u2 = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TP2; ++i) {
      const int q = tid + T * i, row = q / PPR, p = q % PPR;
      u32x4 h, m, l;
      split3_bf16x8(u2[i], h, m, l);
      if (NT2 % T == 0 || q < NT2) {
        u32x4* dst = smem + buf * F2 + ((row >> 4) * KS2 + (p >> 2)) * 192 + 16 * (p & 3) +
                     ((row & 15) ^ (p & 15));
        dst[0] = h;
        dst[64] = m;
        dst[128] = l;
      }
    }
  };

  // The whole computation, for waves with a strip (ON) and for those that
  // only stage U and keep the barriers.
  auto run = [&](auto ONc) {
    constexpr bool ON = decltype(ONc)::value;
    // ---- pass 1: T = U^T W ----
    f32x4 acc[KT][NT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int i = 0; i < NT; ++i) acc[kt][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    vec wv[2][8];
    // step j of this wave: rows 32 (rs + RS j) + 8 g + e (past the end: the
    // last row again, against zero rows of U)
    auto load_w = [&](int j, vec(&v)[8]) {
      const int st = min(rs + RS * j, nsteps - 1);
      if constexpr (FG) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[e] = __builtin_nontemporal_load(
              (const vec*)(wcol + (int64_t)min(32 * st + 8 * g + e, rows - 1) * ld));
      } else {
        const float* src = wcol + (int64_t)(32 * st + 8 * g) * ld;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = __builtin_nontemporal_load((const vec*)(src + e * ld));
      }
    };
    auto step1 = [&](int c, int p, int j, auto Sc) {
      constexpr int S = decltype(Sc)::value;
      u32x4 wh[NT], wm[NT], wl[NT];
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = wv[S][e][i];
        split3_bf16x8(v, wh[i], wm[i], wl[i]);
      }
      load_w(j + 2, wv[S]);
      const int sl = rs + RS * p;                 // step within the chunk
      if (c * SR + sl < nsteps) {
        const u32x4* ub = smem + c % NB1 * F1 + sl * (KT * 192) + lane;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
          const u32x4 uh = ub[kt * 192], um = ub[kt * 192 + 64], ul = ub[kt * 192 + 128];
          f32x4 t[NT];
#pragma unroll
          for (int i = 0; i < NT; ++i) t[i] = mfma16x16x32(ul, wh[i], f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
          for (int i = 0; i < NT; ++i) t[i] = mfma16x16x32(uh, wl[i], t[i]);
#pragma unroll
          for (int i = 0; i < NT; ++i) t[i] = mfma16x16x32(um, wm[i], t[i]);
#pragma unroll
          for (int i = 0; i < NT; ++i) t[i] = mfma16x16x32(um, wh[i], t[i]);
#pragma unroll
          for (int i = 0; i < NT; ++i) t[i] = mfma16x16x32(uh, wm[i], t[i]);
#pragma unroll
          for (int i = 0; i < NT; ++i) acc[kt][i] = mfma16x16x32(uh, wh[i], acc[kt][i]);
#pragma unroll
          for (int i = 0; i < NT; ++i) acc[kt][i] += t[i];
        }
      }
    };
    // chunk c in buffer c % NB1; P0: parity of this wave's first step of it
    auto chunk1 = [&](int c, auto P0c) {
      constexpr int P0 = decltype(P0c)::value;
      load_u1(min(c + 1, nch1 - 1));
      if constexpr (ON) {
        if constexpr (PS == 1) {
          step1(c, 0, c, std::integral_constant<int, P0>{});
        } else {
#pragma unroll
          for (int p = 0; p < PS; p += 2) {
            step1(c, p, c * PS + p, std::integral_constant<int, 0>{});
            step1(c, p + 1, c * PS + p + 1, std::integral_constant<int, 1>{});
          }
        }
      }
      if constexpr (NB1 == 1) __syncthreads();    // every wave is done with chunk c
      store_u1((c + 1) % NB1);
      __syncthreads();
    };
    if (nch1 > 0) {
      load_u1(0);
      if constexpr (ON) {
        load_w(0, wv[0]);
        load_w(1, wv[1]);
      }
      store_u1(0);
      __syncthreads();
      int c = 0;
      if constexpr (PS == 1) {
        for (; c + 1 < nch1; c += 2) {
          chunk1(c, std::integral_constant<int, 0>{});
          chunk1(c + 1, std::integral_constant<int, 1>{});
        }
        if (c < nch1) chunk1(c, std::integral_constant<int, 0>{});
      } else {
        for (; c < nch1; ++c) chunk1(c, std::integral_constant<int, 0>{});
      }
    }

    if constexpr (RS > 1) {
      // partial T of wave w at red[(w KT NT + e) 64 + lane], element
      // e = kt NT + i.  Wave rs of a strip adds the partials of elements
      // e = rs mod RS in wave order and stores the total over the first
      // partial; every wave of the strip then reads the totals.
      constexpr int E = KT * NT, NE = (E + RS - 1) / RS;
      f32x4* const red = (f32x4*)smem;
      const int w0 = grp * RS;
      if constexpr (ON) {
#pragma unroll
        for (int e = 0; e < E; ++e) red[(wave * E + e) * 64 + lane] = acc[e / NT][e % NT];
      }
      __syncthreads();
      f32x4 tot[NE];
      if constexpr (ON) {
#pragma unroll
        for (int i = 0; i < NE; ++i) {
          const int e = rs + RS * i;
          if (e < E) {
            f32x4 s = red[(w0 * E + e) * 64 + lane];
#pragma unroll
            for (int r2 = 1; r2 < RS; ++r2) s += red[((w0 + r2) * E + e) * 64 + lane];
            tot[i] = s;
          }
        }
      }
      __syncthreads();                            // every partial read
      if constexpr (ON) {
#pragma unroll
        for (int i = 0; i < NE; ++i) {
          const int e = rs + RS * i;
          if (e < E) red[(w0 * E + e) * 64 + lane] = tot[i];
        }
      }
      __syncthreads();
      if constexpr (ON) {
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e / NT][e % NT] = red[(w0 * E + e) * 64 + lane];
      }
      __syncthreads();                            // totals read before pass 2 stages U
    }

    // an element of T that the planes cannot vouch for (rows past k repeat
    // row k - 1): the strip's T again, in float32
    bool bad = false;
    if constexpr (ON) {
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) bad |= planes_unsure(acc[kt][i][r]);
      bad = __any(bad);
      if (bad) {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int i = 0; i < NT; ++i) acc[kt][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int r0 = 0; r0 < rows; r0 += 4) {
          const int row = r0 + g;
          const bool ok = row < rows;
          vec w = *(const vec*)(wcol + (int64_t)(ok ? row : 0) * ld);
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) {
            const float a = (ok && 16 * kt + n16 < k) ? U[(int64_t)row * k + 16 * kt + n16] : 0.f;
#pragma unroll
            for (int i = 0; i < NT; ++i)
              acc[kt][i] = mfma16x16x4f32(a, ok ? (float)w[i] : 0.f, acc[kt][i]);
          }
        }
      }
    }

    if constexpr (FG) {
      // dZp row NT n16 + i (of din), columns 16 kt + 4 g + r (of k); one wave
      // of the strip writes
      if (ON && rs == 0 && on) {
        const bool v16 = k % 4 == 0 && ((uintptr_t)fg_out & 15u) == 0;
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) {
            const int kc = 16 * kt + 4 * g;
            float* dst = fg_out + (colw + i) * k + kc;
            if (v16 && kc < k) {
              *(f32x4*)dst = acc[kt][i];
            } else {
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (kc + r < k) dst[r] = acc[kt][i][r];
            }
          }
      }
    } else {
      // ---- pass 2: W = U T ----
      // rows 16 rt + 4 g + r of the chunk, this lane's NT columns
      auto put = [&](int row, const f32x4(&o)[NT]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          vec v;
#pragma unroll
          for (int i = 0; i < NT; ++i) v[i] = o[i][r];
          __builtin_nontemporal_store(v, (vec*)(wcol + (int64_t)(row + r) * ld));
        }
      };
      // every chunk of rows, with its U staged: tile(c) does this wave's rows
      auto sweep = [&](auto tile) {
        load_u2(0);
        store_u2(0);
        __syncthreads();
        for (int c = 0; c < nch2; ++c) {
          load_u2(min(c + 1, nch2 - 1));
          tile(c);
          store_u2((c + 1) & 1);
          __syncthreads();
        }
      };
      if constexpr (ON) {
        if (bad) {
          sweep([&](int c) {
            for (int rt = rs; rt < R2 / 16; rt += RS) {
              const int r0 = c * R2 + 16 * rt;
              if (r0 >= rows) break;
              f32x4 o[NT];
#pragma unroll
              for (int i = 0; i < NT; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                  // both operands zero past k, where T may hold 0 x infinity
                  const int col = 16 * kt + 4 * g + s;
                  const float a = col < k ? U[(int64_t)(r0 + n16) * k + col] : 0.f;
#pragma unroll
                  for (int i = 0; i < NT; ++i)
                    o[i] = mfma16x16x4f32(a, col < k ? acc[kt][i][s] : 0.f, o[i]);
                }
              if (on) put(r0 + 4 * g, o);
            }
          });
        } else {
          u32x4 th[KS2][NT], tm[KS2][NT], tl[KS2][NT];
#pragma unroll
          for (int s = 0; s < KS2; ++s)
#pragma unroll
            for (int i = 0; i < NT; ++i) {
              float v[8];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                v[e] = acc[2 * s][i][e];
                v[4 + e] = 2 * s + 1 < KT ? acc[2 * s + 1 < KT ? 2 * s + 1 : 0][i][e] : 0.f;
              }
              split3_bf16x8(v, th[s][i], tm[s][i], tl[s][i]);
            }
          auto row_tile = [&](int c, int rt, f32x4(&o)[NT]) {
            const u32x4* ub = smem + (c & 1) * F2 + rt * (KS2 * 192);
            f32x4 t[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) {
              t[i] = f32x4{0.f, 0.f, 0.f, 0.f};
              o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int s = 0; s < KS2; ++s) {
              const u32x4* us = ub + s * 192 + 16 * g + (n16 ^ (4 * s + g));
              const u32x4 uh = us[0], um = us[64], ul = us[128];
#pragma unroll
              for (int i = 0; i < NT; ++i) t[i] = mfma16x16x32(ul, th[s][i], t[i]);
#pragma unroll
              for (int i = 0; i < NT; ++i) t[i] = mfma16x16x32(uh, tl[s][i], t[i]);
#pragma unroll
              for (int i = 0; i < NT; ++i) t[i] = mfma16x16x32(um, tm[s][i], t[i]);
#pragma unroll
              for (int i = 0; i < NT; ++i) t[i] = mfma16x16x32(um, th[s][i], t[i]);
#pragma unroll
              for (int i = 0; i < NT; ++i) t[i] = mfma16x16x32(uh, tm[s][i], t[i]);
#pragma unroll
              for (int i = 0; i < NT; ++i) o[i] = mfma16x16x32(uh, th[s][i], o[i]);
            }
#pragma unroll
            for (int i = 0; i < NT; ++i) o[i] += t[i];
          };
          if (__all(on) && rows % R2 == 0) {
            // whole chunks and columns: every store unconditional
            sweep([&](int c) {
#pragma unroll
              for (int q = 0; q < R2 / 16 / RS; ++q) {
                const int rt = rs + RS * q;
                f32x4 o[NT];
                row_tile(c, rt, o);
                put(c * R2 + 16 * rt + 4 * g, o);
              }
            });
          } else {
            sweep([&](int c) {
              for (int rt = rs; rt < R2 / 16; rt += RS) {
                if (c * R2 + 16 * rt >= rows) break;
                f32x4 o[NT];
                row_tile(c, rt, o);
                if (on) put(c * R2 + 16 * rt + 4 * g, o);
              }
            });
          }
        }
      } else {
        sweep([](int) {});
      }
    }
  };
  if (active)
    run(std::true_type{});
  else
    run(std::false_type{});
}

template <int KT, int NT, int RS, bool FG>
static hipError_t launch_weights_f32_cfg(ColumnBatchF32& cb, const float* U, int rows, int k,
                                         float* fg_out, int64_t want, hipStream_t st) {
  int32_t acc = 0;
  for (int b = 0; b < cb.count; ++b) {
    cb.first[b] = acc;
    acc += (int32_t)(((int64_t)cb.n[b] + 16 * NT - 1) / (16 * NT));
  }
  for (int b = cb.count; b <= kMaxBatch; ++b) cb.first[b] = acc;
  cb.strips = acc;
  // strips per block: as even as possible over rounds of `want` blocks
  const int64_t most = kS32Waves / RS, rounds = (acc + want * most - 1) / (want * most);
  const int64_t cs = (acc + want * rounds - 1) / (want * rounds);
  cb.cs = (int32_t)(cs < 1 ? 1 : (cs > most ? most : cs));
  // a multiple of 8 blocks (blocks past the last strip only keep the barriers)
  const unsigned grid = ((unsigned)((acc + cb.cs - 1) / cb.cs) + 7u) & ~7u;
  hipLaunchKernelGGL((project_weights_f32_mfma<KT, NT, RS, FG>), dim3(grid), dim3(64 * kS32Waves), 0, st,
                     cb, U, rows, k, fg_out);
  return hipGetLastError();
}

// Strip shapes by the columns each compute unit gets: enough waves per unit
// to keep loads in flight and all four SIMDs on the matrix cores (wide
// strips, one wave each, for large batches; narrower strips whose rows are
// shared by several waves for small ones).  Measured on MI355X against the
// float32-product kernel (us): 2048^2, k = 40 40.9 -> 36.7 (8 waves per
// 16-column strip; with 4 48); 4096^2, k = 64 109 -> 81; 4096 x 14336 262 ->
// 138; 4096 x (4096 + 14336) 309 -> 174; 5120 x (5120 + 18432), k = 51 547
// -> 237; k = 128, 2048^2 82 -> 67 and 4 x (5120^2, 5120 x 18432) 3737 ->
// 1461; k <= 16, whose products are few, 4 x (2048^2, 2048 x 7168) 112 ->
// 110, 4 x (4096^2, 4096 x 14336) 400 -> 416 (five waves on 231 units; other
// strip shapes and an even spread over 256 units 412 to 466).
template <int KT, bool FG>
hipError_t launch_weights_f32_kt(ColumnBatchF32& cb, const float* U, int rows, int k, float* fg_out,
                                 hipStream_t st) {
  const int64_t cus = device_cu_count();
  int64_t cols = 0;
  for (int b = 0; b < cb.count; ++b) cols += cb.n[b];
  const int64_t per = (cols + cus - 1) / cus;
  if constexpr (KT <= 4) {
    if (per > 256) return launch_weights_f32_cfg<KT, 4, 1, FG>(cb, U, rows, k, fg_out, cus, st);
    if (per > 128) return launch_weights_f32_cfg<KT, 4, 2, FG>(cb, U, rows, k, fg_out, cus, st);
    if (per > 64) return launch_weights_f32_cfg<KT, 4, 4, FG>(cb, U, rows, k, fg_out, cus, st);
    if (per > 32) return launch_weights_f32_cfg<KT, 2, 4, FG>(cb, U, rows, k, fg_out, cus, st);
    if (per > 16) return launch_weights_f32_cfg<KT, 1, 4, FG>(cb, U, rows, k, fg_out, cus, st);
    return launch_weights_f32_cfg<KT, 1, 8, FG>(cb, U, rows, k, fg_out, cus, st);
  } else {
    if (per > 128) return launch_weights_f32_cfg<KT, 2, 1, FG>(cb, U, rows, k, fg_out, cus, st);
    if (per > 64) return launch_weights_f32_cfg<KT, 2, 2, FG>(cb, U, rows, k, fg_out, cus, st);
    if (per > 32) return launch_weights_f32_cfg<KT, 1, 2, FG>(cb, U, rows, k, fg_out, cus, st);
    return launch_weights_f32_cfg<KT, 1, 4, FG>(cb, U, rows, k, fg_out, cus, st);
  }
}

// Explicitly instantiated in f32_strips_a.hip (KT 1..4) and f32_strips_b.hip
// (KT 5..8); the dispatching unit declares them extern.
#define SSN_STRIPS_F32_KT(KT, FG)                                                           \
  template hipError_t launch_weights_f32_kt<KT, FG>(ColumnBatchF32&, const float*, int, int, \
                                                    float*, hipStream_t)
#define SSN_STRIPS_F32_KT_EXTERN(KT, FG) extern SSN_STRIPS_F32_KT(KT, FG)

}  // namespace ssn
