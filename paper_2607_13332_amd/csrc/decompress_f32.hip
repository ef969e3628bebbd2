// decompress / gradient expansion with float32 storage on the bf16 matrix
// cores (contract over k): Y = E[ids] + Z U^T, Y = Z U^T, or Y = Z[ids] U^T.
//
// Paper: section 4.1, Eq. (2) -- reconstruction of the activation from its
// coordinates, and G_Z U^T for the gradient at the sender.
#include "ssn_device.h"
#include "ssn_launch.h"

namespace ssn {

constexpr int kExp32Waves = 4;
// 16-column tiles per wave: three planes of 4 tiles' rows of U take 48
// registers per K step, and at four K steps only 2 tiles fit
constexpr int exp32_tiles(int ks) { return ks == 4 ? 2 : 4; }

typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
template <int NTL>
struct TileVec;
template <>
struct TileVec<4> { typedef f32x4 T; };
template <>
struct TileVec<2> { typedef f32x2 T; };

// ===========================================================================
// What bounds it: the bytes of Y (and of the gathered rows of E); the float32
// matrix instructions would not keep up with them (16x16x4: 32 cycles for
// what six bf16 16x16x32 do in 12).  Every float32 operand is split exactly
// into three bf16 planes and a product takes the six plane pairs that leave
// out at most 2^-24 of it, the five small pairs of all K steps first.  The
// large ones go on from their sum, or (one K step, where one rounding more
// counts) are summed apart and added once.  bf16 coordinates (ZB) are one
// plane, three pairs.  Float32 coordinates are split scaled by 2^16, so that
// the smallest gradient keeps its bits; U's planes are not (an entry below
// 2^-110 is off by 2^-133 at most): the scale alone took a short launch's start
// 6 % longer (N = 5000, d = 1024, k = 72 expansion 12.6 -> 13.4 us).
//
// A wave owns 16 NTL columns of Y whose rows of U stay in registers, split
// once, as MFMA B fragments; the block walks its range of tokens in tiles of
// 16.  Column n of B tile tt is column NTL n + tt of the wave's, so that lane
// (n16, g) ends with NTL consecutive columns of tokens 4 g + j: a store moves
// 4 rows x 64 NTL contiguous bytes, and the rows of E arrive in the same
// shape.  Coordinates are staged by the block, ST tiles at a time and one
// 8-coordinate piece per thread, split there, into LDS in A-fragment order
// (cell n16 of K group c at n16 ^ c); double buffered, one barrier per stage.
//
// Columns past k: the K group at column c0 reads the window [o, o + 8), o =
// min(c0, kz - 8), of the rows of both U and Z, with U's elements below c0
// zeroed (the group before carries them), so every load is a whole piece
// inside its row for any kz >= 8.
//
// A tile with a result that is not finite (an infinity or NaN in Z or U, or
// an overflow) is computed again in plain float32, which propagates them.
// Tokens past N recompute token N - 1 and store the same bytes there.
// ===========================================================================
template <int KS, bool HAS_E, bool GZ, bool ZB>
__global__ __launch_bounds__(64 * kExp32Waves, 2) void decompress_cols_f32(
    const float* __restrict__ Zc, const uint16_t* __restrict__ Zb, const int32_t* __restrict__ ids,
    const float* __restrict__ E, const float* __restrict__ U, float* __restrict__ Y, int64_t N, int d,
    int k, int64_t V, int kz, int nd, int ranges, int per, int more) {
  static_assert(!(HAS_E && GZ), "gathered coordinates carry no additive embedding");
  constexpr int NW = kExp32Waves, NT = 64 * NW, NTL = exp32_tiles(KS), CW = 16 * NTL;
  typedef typename TileVec<NTL>::T vec;
  constexpr int ST = KS == 1 ? 4 : (KS == 2 ? 2 : 1);   // tiles per stage
  constexpr int PIECES = ST * 64 * KS;                  // 8-coordinate pieces per stage
  static_assert(PIECES <= NT, "one piece per thread");
  constexpr int NP = ZB ? 1 : 3;                        // planes of Z
  constexpr int UPITCH = 36;                            // floats per row of the U tile
  constexpr int UR = CW / 8;                            // 8-row loads of a K step of U
  __shared__ u32x4 zl[2][ST][KS][NP][kWave];
  __shared__ f32x4 ut[NW][CW * UPITCH / 4];             // one K step of a wave's rows of U

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n16 = lane & 15, g = lane >> 4;

  // Block -> (token range, column group); consecutive work items share a
  // token range and are given to one XCD (workgroups go to the 8 in turn).
  const int nb = nd * ranges, q8 = nb >> 3, r8 = nb & 7;
  const int xcd = blockIdx.x & 7, xj = blockIdx.x >> 3;
  const int w = xcd * q8 + (xcd < r8 ? xcd : r8) + xj;
  const int range = w / nd;
  // (unsigned: the last block's columns may pass 2^31)
  const uint32_t colw = (uint32_t)((w - range * nd) * NW + wave) * CW;
  const bool live = colw < (uint32_t)d;          // others only help with the staging
  const int col0 = live ? (int)colw : 0;
  // per or per + 1 tiles (divided on the host: a 64-bit division here took
  // about as long as the smallest launches' loads)
  const int n = per + (range < more ? 1 : 0);
  const int64_t tok0 = 16 * ((int64_t)range * per + (range < more ? range : more));
  auto clamp_token = [&](int64_t t) { return t < N ? t : N - 1; };
  auto window = [&](int c0) { return c0 + 8 <= kz ? c0 : (kz >= 8 ? kz - 8 : 0); };

  // ---- staging of the coordinates: the thread's piece ----
  const int piece = PIECES == NT || tid < PIECES ? tid : PIECES - 1;
  const int prow = piece / (4 * KS), pc = piece % (4 * KS);
  const int po = window(8 * pc), pdst = 16 * (pc & 3) + ((prow & 15) ^ pc);
  u32x4 zr[2];
  auto ptoken = [&](int j) { return clamp_token(tok0 + 16 * (int64_t)ST * j + prow); };
  auto load_z = [&](int64_t zrow) __attribute__((always_inline)) {
    if (KS > 1 || kz >= 8) {
      if constexpr (ZB) {
        zr[0] = *(const u32x4_a2*)(Zb + zrow + po);
      } else {
        zr[0] = __builtin_bit_cast(u32x4, *(const f32x4_a4*)(Zc + zrow + po));
        zr[1] = __builtin_bit_cast(u32x4, *(const f32x4_a4*)(Zc + zrow + po + 4));
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool on = 8 * pc + e < kz;
        if constexpr (ZB) {
          const uint32_t x = on ? (uint32_t)Zb[zrow + e] : 0u;
          zr[0][e >> 1] = (e & 1) ? (zr[0][e >> 1] | (x << 16)) : x;
        } else {
          zr[e >> 2][e & 3] = on ? __float_as_uint(Zc[zrow + e]) : 0u;
        }
      }
    }
  };
  auto store_z = [&](int buf) __attribute__((always_inline)) {
    if (PIECES == NT || tid < PIECES) {
      u32x4(*dst)[kWave] = zl[buf][prow >> 4][pc >> 2];
      if constexpr (ZB) {
        dst[0][pdst] = zr[0];
      } else {
        float v[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) v[m] = __uint_as_float(zr[m >> 2][m & 3]);
        u32x4 h, m, l;
        split3_bf16x8<true>(v, h, m, l);
        dst[0][pdst] = h;
        dst[NP > 1 ? 1 : 0][pdst] = m;
        dst[NP > 2 ? 2 : 0][pdst] = l;
      }
    }
  };

  // rows of E of one tile (instruction j: tokens 4 g + j), one tile ahead,
  // their ids two
  vec er[4];
  int32_t idr[4];
  auto load_ids = [&](int i, int32_t (&id)[4]) __attribute__((always_inline)) {
    const int64_t t = tok0 + 16 * (int64_t)(i < n ? i : n - 1) + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) id[j] = ids[clamp_token(t + j)];
  };
  auto load_e = [&](const int32_t (&id)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      er[j] = *(const vec*)(E + clamp_id(id[j], V) * d + col0 + NTL * n16);
  };

  const int nst = (n + ST - 1) / ST;
  auto last = [&](int j) { return j < nst ? j : nst - 1; };
  int32_t zid = 0;                               // GZ: the piece's table row, next stage
  int32_t first[4];
  if constexpr (GZ) {
    const int32_t a = ids[ptoken(0)];
    zid = ids[ptoken(last(1))];
    load_z(clamp_id(a, V) * kz);
  } else {
    if constexpr (HAS_E) {
      load_ids(0, first);
      load_ids(1, idr);
    }
    load_z(ptoken(0) * kz);
  }
  // ---- U: per K step 8 rows x 128 bytes an instruction, through a
  // wave-private LDS tile ----
  f32x4 uraw[KS][UR];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int c0 = 32 * s + 8 * ((lane & 7) >> 1), o = window(c0) + 4 * (lane & 1);
#pragma unroll
    for (int r = 0; r < UR; ++r) {
      const float* p = U + (int64_t)(col0 + 8 * r + (lane >> 3)) * k + o;
      if (KS > 1 || kz >= 8) {
        uraw[s][r] = *(const f32x4_a4*)p;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) uraw[s][r][e] = c0 + 4 * (lane & 1) + e < kz ? p[e] : 0.f;
      }
    }
  }
  if constexpr (HAS_E) load_e(first);
  u32x4 ub[KS][NTL][3];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int c0 = 32 * s + 8 * ((lane & 7) >> 1);
    const int nz = (kz < 8 ? 0 : c0 - window(c0)) - 4 * (lane & 1);   // leading elements to drop
#pragma unroll
    for (int r = 0; r < UR; ++r) {
      f32x4 v = uraw[s][r];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = e < nz ? 0.f : v[e];
      ut[wave][((8 * r + (lane >> 3)) * UPITCH + 4 * (lane & 7)) / 4] = v;
    }
    wave_lds_order();
#pragma unroll
    for (int tt = 0; tt < NTL; ++tt) {
      const f32x4* src = &ut[wave][((NTL * n16 + tt) * UPITCH + 8 * g) / 4];
      const f32x4 a = src[0], b = src[1];
      const float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
      split3_bf16x8(v, ub[s][tt][0], ub[s][tt][1], ub[s][tt][2]);
    }
    wave_lds_order();
  }
  store_z(0);

  auto step = [&](int i, const u32x4 (&zt)[KS][NP][kWave]) __attribute__((always_inline)) {
    f32x4 acc[NTL];
#pragma unroll
    for (int tt = 0; tt < NTL; ++tt) acc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int cell = 16 * g + (n16 ^ (4 * s + g));
      const u32x4 zh = zt[s][0][cell];
#pragma unroll
      for (int tt = 0; tt < NTL; ++tt) acc[tt] = mfma16x16x32(zh, ub[s][tt][2], acc[tt]);
      if constexpr (!ZB) {
        const u32x4 zm = zt[s][NP > 1 ? 1 : 0][cell], zo = zt[s][NP > 2 ? 2 : 0][cell];
#pragma unroll
        for (int tt = 0; tt < NTL; ++tt) acc[tt] = mfma16x16x32(zo, ub[s][tt][0], acc[tt]);
#pragma unroll
        for (int tt = 0; tt < NTL; ++tt) acc[tt] = mfma16x16x32(zm, ub[s][tt][1], acc[tt]);
#pragma unroll
        for (int tt = 0; tt < NTL; ++tt) acc[tt] = mfma16x16x32(zm, ub[s][tt][0], acc[tt]);
      }
#pragma unroll
      for (int tt = 0; tt < NTL; ++tt) acc[tt] = mfma16x16x32(zh, ub[s][tt][1], acc[tt]);
    }
    if constexpr (KS == 1) {
      const u32x4 zh = zt[0][0][16 * g + (n16 ^ g)];
#pragma unroll
      for (int tt = 0; tt < NTL; ++tt) acc[tt] += mfma16x16x32(zh, ub[0][tt][0], f32x4{0.f, 0.f, 0.f, 0.f});
    } else {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const u32x4 zh = zt[s][0][16 * g + (n16 ^ (4 * s + g))];
#pragma unroll
        for (int tt = 0; tt < NTL; ++tt) acc[tt] = mfma16x16x32(zh, ub[s][tt][0], acc[tt]);
      }
    }
    // float32 coordinates entered scaled
    constexpr float unscale = ZB ? 1.f : 1.f / kPlanesScale;
    const int64_t t = tok0 + 16 * (int64_t)i + 4 * g;
    float z = 0.f;
#pragma unroll
    for (int tt = 0; tt < NTL; ++tt) {
#pragma unroll
      for (int j = 0; j < 4; ++j) z = fmaf(acc[tt][j], 0.f, z);
      acc[tt] *= unscale;
    }
    if (__any(z != 0.f)) {
      // not finite: the tile again, in float32 from memory
#pragma unroll
      for (int tt = 0; tt < NTL; ++tt) acc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
      int64_t zrow[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t tj = clamp_token(t + j);
        zrow[j] = (GZ ? clamp_id(ids[tj], V) : tj) * kz;
      }
#pragma clang loop unroll(disable)
      for (int c = 0; c < kz; ++c) {
#pragma unroll
        for (int tt = 0; tt < NTL; ++tt) {
          const float u = U[(int64_t)(col0 + NTL * n16 + tt) * k + c];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[tt][j] = fmaf(ZB ? bf16_to_f32(Zb[zrow[j] + c]) : Zc[zrow[j] + c], u, acc[tt][j]);
        }
      }
    }
    vec y[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int tt = 0; tt < NTL; ++tt) y[j][tt] = acc[tt][j];
      if constexpr (HAS_E) y[j] += er[j];
    }
    if constexpr (HAS_E) {
      load_e(idr);
      load_ids(i + 2, idr);
    }
    if (live) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        __builtin_nontemporal_store(y[j], (vec*)(Y + clamp_token(t + j) * d + col0 + NTL * n16));
    }
  };
#pragma clang loop unroll(disable)
  for (int j = 0; j < nst; ++j) {
    if constexpr (GZ) {
      load_z(clamp_id(zid, V) * kz);
      zid = ids[ptoken(last(j + 2))];
    } else {
      load_z(ptoken(last(j + 1)) * kz);
    }
    __syncthreads();
#pragma clang loop unroll(disable)
    for (int q = 0; q < ST && j * ST + q < n; ++q) step(j * ST + q, zl[j & 1][q]);
    store_z((j + 1) & 1);
  }
}

// Two blocks per compute unit (two waves per SIMD), each with an equal range
// of the 16-token tiles; one block per unit where two would have about one
// tile each, so that half the blocks fetch and split U (N = 2048, d = 1024, k
// = 48 expansion 98 -> 85 hundredths of the time of float32 instructions, N =
// 1500, d = 576 97 -> 86; with two tiles each it loses, N = 4096, d = 1024 84
// -> 85, decompress 91 -> 98).
template <int KS, bool HAS_E, bool GZ, bool ZB>
static hipError_t launch_cols(int64_t N, int d, int k, int64_t V, const float* Zc, const uint16_t* Zb,
                              const int32_t* ids, const float* E, const float* U, float* Y, int kz,
                              hipStream_t st) {
  constexpr int BC = kExp32Waves * 16 * exp32_tiles(KS);
  const int64_t tiles = (N + 15) / 16, nd = ((int64_t)d + BC - 1) / BC;
  int64_t ranges = 2 * (int64_t)device_cu_count() / nd;
  if (4 * tiles <= 5 * ranges) ranges /= 2;
  ranges = ranges < 1 ? 1 : (ranges < tiles ? ranges : tiles);
  hipLaunchKernelGGL((decompress_cols_f32<KS, HAS_E, GZ, ZB>), dim3((unsigned)(nd * ranges)),
                     dim3(64 * kExp32Waves), 0, st, Zc, Zb, ids, E, U, Y, N, d, k, V, kz, (int)nd,
                     (int)ranges, (int)(tiles / ranges), (int)(tiles % ranges));
  return hipGetLastError();
}

template <int KS>
static hipError_t launch_cols_ks(int64_t N, int d, int k, int64_t V, const float* Zc,
                                 const uint16_t* Zb, const int32_t* ids, const float* E,
                                 const float* U, float* Y, bool gather_z, int kz, hipStream_t st) {
  if (gather_z) return launch_cols<KS, false, true, false>(N, d, k, V, Zc, Zb, ids, E, U, Y, kz, st);
  if (E)
    return Zb ? launch_cols<KS, true, false, true>(N, d, k, V, Zc, Zb, ids, E, U, Y, kz, st)
              : launch_cols<KS, true, false, false>(N, d, k, V, Zc, Zb, ids, E, U, Y, kz, st);
  return Zb ? launch_cols<KS, false, false, true>(N, d, k, V, Zc, Zb, ids, E, U, Y, kz, st)
            : launch_cols<KS, false, false, false>(N, d, k, V, Zc, Zb, ids, E, U, Y, kz, st);
}

// Where float32 instructions on U as it is stored (decompress_f32_chunks) beat
// planes in registers: few coordinates, and fewer output elements than pay
// for a wave's start.  Measured in us, chunks against columns, with E / without:
//   k = 8:  N = 512, d = 256 4.3 / 5.3 and 4.1 / 4.7; N = 4096, d = 1024 7.6 /
//           9.5 and 5.8 / 7.0; N = 3000, d = 2048 100 : 110 and 100 : 111
//           (relative); N = 3000, d = 4096 100 : 104 and 100 : 88
//   k = 24: N = 3000, d = 576 100 : 131 and 100 : 111; N = 1500, d = 2048 100 :
//           100 and 120 : 100
// and further where their grid is one full round of blocks (N = 4096, 8192):
//   k = 8:  N = 8192, d = 2048 100 : 108 and 100 : 92; N = 2048, d = 5120 100 :
//           123 and 100 : 115; a stage's step at N = 5000, d = 5120, no full
//           round, 178 / 168
//   k = 24: N = 2048, d = 5120 with E 100 : 110, without 100 : 98.
static bool decompress_f32_uses_chunks(int64_t N, int64_t d, int64_t ku, bool has_e) {
  const int64_t out = N * d;
  if (ku >= 32) return false;
  if (out <= (int64_t)1 << (ku <= 16 ? 23 : 21)) return true;
  if (!has_e && (ku > 16 || out > 5 * ((int64_t)1 << 21))) return false;
  return out < (int64_t)1 << 25 && decompress_chunks_fill(N, d);
}

hipError_t launch_decompress_f32(int64_t N, int64_t d, int64_t k, int64_t V, const float* Z,
                                 const int32_t* ids, const float* E, const float* U, float* Y,
                                 bool gather_z, hipStream_t st, const uint16_t* Zb, int kz) {
  const int dd = (int)d, ku = (int)k;
  if (decompress_f32_uses_chunks(N, d, k, E != nullptr))
    return launch_decompress_f32_chunks(N, dd, V, Z, ids, E, U, Y, gather_z, st, Zb, kz, ku);
  switch ((kz + 31) / 32) {
    case 1: return launch_cols_ks<1>(N, dd, ku, V, Z, Zb, ids, E, U, Y, gather_z, kz, st);
    case 2: return launch_cols_ks<2>(N, dd, ku, V, Z, Zb, ids, E, U, Y, gather_z, kz, st);
    case 3: return launch_cols_ks<3>(N, dd, ku, V, Z, Zb, ids, E, U, Y, gather_z, kz, st);
    default: return launch_cols_ks<4>(N, dd, ku, V, Z, Zb, ids, E, U, Y, gather_z, kz, st);
  }
}

}  // namespace ssn
