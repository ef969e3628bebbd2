// decompress / gradient expansion with bf16 storage on the matrix cores
// (contract over k): Y = E[ids] + Z U^T, Y = Z U^T, or Y = Z[ids] U^T.
//
// Paper: section 4.1, Eq. (2) -- reconstruction of the activation from its
// coordinates, and G_Z U^T for the gradient at the sender.
#include "ssn_device.h"
#include "ssn_launch.h"


namespace ssn {

constexpr int kExpandWaves = 4;                     // waves per block
constexpr int kExpandCols = 128;                    // columns of d per wave
constexpr int kExpandBlockCols = kExpandWaves * kExpandCols;

typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));

// ===========================================================================
// What bounds it: the bytes of Y (and of the gathered rows of E), so the loop
// over tokens touches nothing else but the coordinates.  A wave owns 128
// columns of Y: the 128 rows of U that they need stay in registers as MFMA B
// fragments for the whole kernel (32 KS registers, KS = ceil(k / 32) K
// steps), and the block walks its range of tokens in tiles of 16.  Column n
// of B tile tt is column 8 n + tt of the wave's 128, so that lane (n16, g)
// ends with columns 8 n16 .. + 7 of tokens 4 g + j: store j moves 4 rows x
// 256 contiguous bytes straight from the accumulators, and the rows of E
// arrive in the same shape.  (With the tokens on the lanes' fast axis, 16
// rows x 64 bytes an instruction, every lane is a cache line lookup of its
// own: measured twice as slow.)
//
// The coordinates are staged by the whole block, ST tiles at a time and one
// 8-coordinate piece per thread, into LDS in A-fragment order (cell n16 of
// K group c is stored at n16 ^ c, which spreads both sides over the banks);
// double buffered, one barrier per stage.  Float32 coordinates are split
// there into bf16 hi + lo parts, two MFMAs each, which keeps about float32
// accuracy; bf16 coordinates (ZB) are exact in the hi part.
//
// Columns past k: the last K group of 8 would read past the row, so the group
// at column c0 reads the window [o, o + 8), o = min(c0, kz - 8), of the rows
// of both U and Z, and U's elements below c0 (which the group before carries)
// are zeroed once.  Every load is then a whole, possibly unaligned, 16-byte
// piece inside its row, for any kz >= 8.
//
// Rows of E are requested a tile ahead (their ids two; two and four measured
// no faster at any N), coordinates a stage ahead, always before the stores of
// the tile in hand: loads and stores share one in-order counter, so no wait
// covers a younger store.
// Tokens past N recompute token N - 1 and store the same bytes there.
// ===========================================================================
template <int KS, bool HAS_E, bool GZ, bool ZB, bool TS>
__global__ __launch_bounds__(64 * kExpandWaves, 2) void decompress_cols_bf16(
    const float* __restrict__ Zc, const uint16_t* __restrict__ Zb, const int32_t* __restrict__ ids,
    const uint16_t* __restrict__ E, const uint16_t* __restrict__ U, uint16_t* __restrict__ Y,
    int64_t N, int d, int k, int64_t V, int kz, int nd, int ranges, int per, int more) {
  static_assert(!(HAS_E && GZ), "gathered coordinates carry no additive embedding");
  constexpr int NW = kExpandWaves, NT = 64 * NW;
  constexpr int ST = TS || KS == 1 ? NW : (KS == 2 ? 2 : 1);   // tiles per stage
  constexpr int PIECES = ST * 64 * KS;                  // 8-coordinate pieces per stage
  constexpr int PPT = (PIECES + NT - 1) / NT;           // per thread
  constexpr int NP = ZB ? 1 : 2;                        // parts: hi (and lo)
  static_assert(PPT == 1 || PIECES % NT == 0, "whole rounds of pieces");
  __shared__ u32x4 zl[2][ST][KS][NP][kWave];
  // U on its way to the lanes: one K step of each wave's rows, or (TS) all of
  // the block's
  __shared__ u32x4 ut[TS ? KS : NW][4 * kExpandCols];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n16 = lane & 15, g = lane >> 4;

  // Block -> (token range, group of 512 columns).  Workgroups go to the 8
  // XCDs in turn; consecutive work items, which share a token range (and so
  // the range's coordinates and ids in L2), are given to one XCD.
  const int nb = nd * ranges, q8 = nb >> 3, r8 = nb & 7;
  const int xcd = blockIdx.x & 7, xj = blockIdx.x >> 3;
  const int w = xcd * q8 + (xcd < r8 ? xcd : r8) + xj;
  const int range = w / nd;
  // waves past the last column only help with the staging
  // (unsigned: the last block's columns may pass 2^31)
  const uint32_t colw = (uint32_t)((w - range * nd) * (TS ? 1 : NW) + (TS ? 0 : wave)) * kExpandCols;
  const bool live = TS || colw < (uint32_t)d;
  const int col0 = live ? (int)colw : 0;
  // per or per + 1 tiles (divided on the host: a 64-bit division here took
  // about as long as the smallest launches' loads)
  const int n = per + (range < more ? 1 : 0);
  const int64_t tok0 = 16 * ((int64_t)range * per + (range < more ? range : more));
  auto clamp_token = [&](int64_t t) { return t < N ? t : N - 1; };

  // ---- U: B fragments of the wave's 128 columns.  Per K step they arrive as
  // 16 rows x 64 bytes per instruction (4 lanes to a row) and change lanes
  // through a wave-private LDS tile: cell (row, c) at (4 row + c) ^ (row / 8),
  // which spreads the reads of rows 8 n16 + tt over the banks ----
  u32x4 ub[KS][8];
  constexpr int UR = TS ? 8 / NW : 8;            // 16-row loads of this wave
  const int ur0 = TS ? UR * wave : 0;
  auto load_u = [&]() __attribute__((always_inline)) {
    const int c = lane & 3;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int c0 = 32 * s + 8 * c;
      const int o = c0 + 8 <= kz ? c0 : (kz >= 8 ? kz - 8 : 0);
#pragma unroll
      for (int r = 0; r < UR; ++r) {
        const uint16_t* p = U + (int64_t)(col0 + 16 * (ur0 + r) + (lane >> 2)) * k + o;
        if (KS > 1 || kz >= 8) {
          ub[s][r] = *(const u32x4_a2*)p;
        } else {
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            const uint32_t lo = c0 + 2 * m < kz ? (uint32_t)p[2 * m] : 0u;
            const uint32_t hi = c0 + 2 * m + 1 < kz ? (uint32_t)p[2 * m + 1] : 0u;
            ub[s][r][m] = lo | (hi << 16);
          }
        }
      }
    }
  };
  auto park_u = [&](int s, u32x4* tile) __attribute__((always_inline)) {
    const int c0 = 32 * s + 8 * (lane & 3);
    const int nz = c0 + 8 <= kz || kz < 8 ? 0 : c0 - (kz - 8);   // leading elements to drop
#pragma unroll
    for (int r = 0; r < UR; ++r) {
      u32x4 v = ub[s][r];
#pragma unroll
      for (int m = 0; m < 4; ++m)
        v[m] = 2 * m + 1 < nz ? 0u : (2 * m < nz ? v[m] & 0xFFFF0000u : v[m]);
      tile[(64 * (ur0 + r) + lane) ^ (2 * (ur0 + r) + (lane >> 5))] = v;
    }
  };
  auto take_u = [&](int s, const u32x4* tile) __attribute__((always_inline)) {
#pragma unroll
    for (int tt = 0; tt < 8; ++tt) ub[s][tt] = tile[(32 * n16 + 4 * tt + g) ^ n16];
  };

  // ---- staging: thread tid moves pieces tid + NT q of a stage: coordinates
  // [po, po + 8) of token prow + q PR (threads past the last piece repeat it
  // and do not store) ----
  constexpr int PR = NT / (4 * KS);
  static_assert(PPT == 1 || NT % (4 * KS) == 0, "a thread's pieces share their columns");
  const int piece = PIECES % NT == 0 || tid < PIECES ? tid : PIECES - 1;
  const int prow = piece / (4 * KS), pc = piece % (4 * KS);
  const int po = 8 * pc + 8 <= kz ? 8 * pc : (kz >= 8 ? kz - 8 : 0);
  struct ZPiece {
    u32x4 v[NP];
  };
  auto ptoken = [&](int j, int q) {       // the token of the thread's piece q in stage j
    return clamp_token(tok0 + 16 * (int64_t)ST * j + prow + PR * q);
  };
  auto load_z = [&](int64_t zrow, ZPiece& z) __attribute__((always_inline)) {
    if (KS > 1 || kz >= 8) {
      if constexpr (ZB) {
        z.v[0] = *(const u32x4_a2*)(Zb + zrow + po);
      } else {
        z.v[0] = __builtin_bit_cast(u32x4, *(const f32x4_a4*)(Zc + zrow + po));
        z.v[1] = __builtin_bit_cast(u32x4, *(const f32x4_a4*)(Zc + zrow + po + 4));
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool on = 8 * pc + e < kz;
        if constexpr (ZB) {
          const uint32_t x = on ? (uint32_t)Zb[zrow + e] : 0u;
          z.v[0][e >> 1] = (e & 1) ? (z.v[0][e >> 1] | (x << 16)) : x;
        } else {
          z.v[e >> 2][e & 3] = on ? __float_as_uint(Zc[zrow + e]) : 0u;
        }
      }
    }
  };
  auto store_z = [&](int buf, int q, const ZPiece& z) __attribute__((always_inline)) {
    if (PIECES % NT == 0 || tid < PIECES) {
      const int row = prow + PR * q, pdst = 16 * (pc & 3) + ((row & 15) ^ pc);
      u32x4(*dst)[kWave] = zl[buf][row >> 4][pc >> 2];
      if constexpr (ZB) {
        dst[0][pdst] = z.v[0];
      } else {
        float v[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) v[m] = __uint_as_float(z.v[m >> 2][m & 3]);
        u32x4 hi, lo;
        split_bf16x8(v, hi, lo);
        dst[0][pdst] = hi;
        dst[NP - 1][pdst] = lo;
      }
    }
  };

  // rows of E of one tile: instruction j covers tokens 4 g + j
  struct ETile {
    u32x4 v[4];
  };
  struct Ids {
    int32_t v[4];
  };
  auto load_ids = [&](int i, Ids& id) __attribute__((always_inline)) {
    const int64_t t = tok0 + 16 * (int64_t)(i < n ? i : n - 1) + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) id.v[j] = ids[clamp_token(t + j)];
  };
  auto load_e = [&](const Ids& id, ETile& e) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      e.v[j] = *(const u32x4*)(E + clamp_id(id.v[j], V) * d + col0 + 8 * n16);
  };

  const int nst = (n + ST - 1) / ST;
  // the wave's q-th tile of the range: every tile, or (TS) every NW-th
  auto tile_of = [&](int q) { return TS ? NW * q + wave : q; };
  auto last = [&](int j) { return j < nst ? j : nst - 1; };
  ZPiece zr[PPT];
  int32_t zid[PPT];                              // GZ: the pieces' table rows, next stage
  ETile er;                                      // HAS_E: rows of the next tile,
  Ids idr;                                       // and the ids of the one after
  Ids first;
  if constexpr (GZ) {
    int32_t zf[PPT];
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
      zf[q] = ids[ptoken(0, q)];
      zid[q] = ids[ptoken(last(1), q)];
    }
    load_u();
#pragma unroll
    for (int q = 0; q < PPT; ++q) load_z(clamp_id(zf[q], V) * kz, zr[q]);
  } else {
    if constexpr (HAS_E) {
      load_ids(tile_of(0), first);
      load_ids(tile_of(1), idr);
    }
#pragma unroll
    for (int q = 0; q < PPT; ++q) load_z(ptoken(0, q) * kz, zr[q]);
    // the ids were asked for before U, so the embedding rows wait for them alone
    load_u();
    if constexpr (HAS_E) load_e(first, er);
  }
  if constexpr (TS) {
#pragma unroll
    for (int s = 0; s < KS; ++s) park_u(s, ut[s]);
  } else {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      park_u(s, ut[wave]);
      wave_lds_order();
      take_u(s, ut[wave]);
      wave_lds_order();
    }
  }
#pragma unroll
  for (int q = 0; q < PPT; ++q) store_z(0, q, zr[q]);
  if constexpr (TS) {
    __syncthreads();
#pragma unroll
    for (int s = 0; s < KS; ++s) take_u(s, ut[s]);
  }

  auto step = [&](int i, const u32x4 (&zt)[KS][NP][kWave]) __attribute__((always_inline)) {
    f32x4 acc[8];
#pragma unroll
    for (int tt = 0; tt < 8; ++tt) acc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int cell = 16 * g + (n16 ^ (4 * s + g));
      const u32x4 zhi = zt[s][0][cell];
      u32x4 zlo;
      if constexpr (!ZB) zlo = zt[s][NP - 1][cell];
#pragma unroll
      for (int tt = 0; tt < 8; ++tt) acc[tt] = mfma16x16x32(zhi, ub[s][tt], acc[tt]);
      if constexpr (!ZB) {
#pragma unroll
        for (int tt = 0; tt < 8; ++tt) acc[tt] = mfma16x16x32(zlo, ub[s][tt], acc[tt]);
      }
    }
    u32x4 y[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float v[8];
#pragma unroll
      for (int tt = 0; tt < 8; ++tt) v[tt] = acc[tt][j];
      if constexpr (HAS_E) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          v[2 * m] += lo_bf16(er.v[j][m]);
          v[2 * m + 1] += hi_bf16(er.v[j][m]);
        }
      }
      y[j] = u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]),
                   pack_bf16x2(v[6], v[7])};
    }
    if constexpr (HAS_E) {
      if (!TS || i + NW < n) {
        load_e(idr, er);
        load_ids(i + (TS ? 2 * NW : 2), idr);
      }
    }
    const int64_t t = tok0 + 16 * (int64_t)i + 4 * g;
    if (live) {
#pragma unroll
      for (int j = 0; j < 4; ++j) stg<true>(Y + clamp_token(t + j) * d + col0 + 8 * n16, y[j]);
    }
  };
  // Few copies of the step (at most a stage's two tiles, one stage for both
  // buffers): a short launch runs them from cold instruction memory, and six
  // copies, 16 KB, lost at N = 4096 what the kernel gains.
#pragma clang loop unroll(disable)
  for (int j = 0; j < nst; ++j) {
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
      if constexpr (GZ) {
        load_z(clamp_id(zid[q], V) * kz, zr[q]);
        zid[q] = ids[ptoken(last(j + 2), q)];
      } else {
        if (!TS || j + 1 < nst) load_z(ptoken(last(j + 1), q) * kz, zr[q]);
      }
    }
    __syncthreads();
    if constexpr (TS) {
      const int i = j * ST + wave;
      if (i < n) step(i, zl[j & 1][wave]);
    } else {
#pragma clang loop unroll_count(ST <= 2 ? ST : 1)
      for (int q = 0; q < ST; ++q)
        if (j * ST + q < n) step(j * ST + q, zl[j & 1][q]);
    }
#pragma unroll
    for (int q = 0; q < PPT; ++q)
      if (!TS || j + 1 < nst) store_z((j + 1) & 1, q, zr[q]);
  }
}

int64_t decompress_cols_ranges(int64_t d) {
  const int64_t r = 2 * (int64_t)device_cu_count() / ((d + kExpandBlockCols - 1) / kExpandBlockCols);
  return r < 1 ? 1 : r;
}

// One block per slot (two blocks per compute unit: two waves per SIMD), each
// with an equal range of the 16-token tiles.  With at most 2.75 tiles to a
// range the waves of a block share 128 columns and split the tokens (TS), so
// that each block fetches a quarter of the rows of U for four times the
// tokens: N = 2048, d = 2048, k = 40 decompress 7.6 -> 6.1 us, expansion 6.6
// -> 5.4; with more tiles 512 columns win for their longer rows and fewer
// reads of Z.  Whole stage steps, TS / 512 columns in us: 2.2 tiles (N = 9000,
// d = 1024) k = 8 34.7 / 36.1, k = 64 40.4 / 41.7; 2.4 tiles 36.7 / 37.8 and 41.6
// / 42.8; 2.9 tiles (N = 3000, d = 4096) 44.9 / 43.3 and 57.0 / 55.5, (N =
// 12205, d = 1024) 43.2 / 42.5 and 46.6 / 47.5.  k > 64 takes the columns
// always (U's registers).
template <int KS, bool HAS_E, bool GZ, bool ZB>
static hipError_t launch_cols(int64_t N, int d, int k, int64_t V, const float* Zc,
                              const uint16_t* Zb, const int32_t* ids, const void* E, const void* U,
                              void* Y, int kz, hipStream_t st) {
  const int64_t tiles = (N + 15) / 16, slots = 2 * (int64_t)device_cu_count();
  auto ranges_of = [&](int64_t nd, int64_t most) {
    const int64_t r = slots / nd < 1 ? 1 : slots / nd;
    return r < most ? r : most;
  };
  int64_t nd = ((int64_t)d + kExpandBlockCols - 1) / kExpandBlockCols;
  int64_t ranges = decompress_cols_ranges(d) < tiles ? decompress_cols_ranges(d) : tiles;
  if constexpr (KS <= 2) {
    if (4 * tiles <= 11 * ranges) {
      nd = d / kExpandCols;
      ranges = ranges_of(nd, (tiles + kExpandWaves - 1) / kExpandWaves);
      hipLaunchKernelGGL((decompress_cols_bf16<KS, HAS_E, GZ, ZB, true>), dim3((unsigned)(nd * ranges)),
                         dim3(64 * kExpandWaves), 0, st, Zc, Zb, ids, (const uint16_t*)E,
                         (const uint16_t*)U, (uint16_t*)Y, N, d, k, V, kz, (int)nd, (int)ranges,
                     (int)(tiles / ranges), (int)(tiles % ranges));
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((decompress_cols_bf16<KS, HAS_E, GZ, ZB, false>), dim3((unsigned)(nd * ranges)),
                     dim3(64 * kExpandWaves), 0, st, Zc, Zb, ids, (const uint16_t*)E,
                     (const uint16_t*)U, (uint16_t*)Y, N, d, k, V, kz, (int)nd, (int)ranges,
                     (int)(tiles / ranges), (int)(tiles % ranges));
  return hipGetLastError();
}

template <int KS>
static hipError_t launch_cols_ks(int64_t N, int d, int k, int64_t V, const float* Zc,
                                 const uint16_t* Zb, const int32_t* ids, const void* E,
                                 const void* U, void* Y, bool gather_z, int kz, hipStream_t st) {
  if (gather_z) return launch_cols<KS, false, true, false>(N, d, k, V, Zc, Zb, ids, E, U, Y, kz, st);
  if (E)
    return Zb ? launch_cols<KS, true, false, true>(N, d, k, V, Zc, Zb, ids, E, U, Y, kz, st)
              : launch_cols<KS, true, false, false>(N, d, k, V, Zc, Zb, ids, E, U, Y, kz, st);
  return Zb ? launch_cols<KS, false, false, true>(N, d, k, V, Zc, Zb, ids, E, U, Y, kz, st)
            : launch_cols<KS, false, false, false>(N, d, k, V, Zc, Zb, ids, E, U, Y, kz, st);
}

hipError_t launch_decompress_bf16(int64_t N, int64_t d, int64_t k, int64_t V, const float* Zc,
                                  const int32_t* ids, const void* E, const void* U, void* Y,
                                  bool gather_z, hipStream_t st, const uint16_t* Zb, int kz) {
  const int dd = (int)d, ku = (int)k;
  switch ((kz + 31) / 32) {
    case 1: return launch_cols_ks<1>(N, dd, ku, V, Zc, Zb, ids, E, U, Y, gather_z, kz, st);
    case 2: return launch_cols_ks<2>(N, dd, ku, V, Zc, Zb, ids, E, U, Y, gather_z, kz, st);
    case 3: return launch_cols_ks<3>(N, dd, ku, V, Zc, Zb, ids, E, U, Y, gather_z, kz, st);
    default: return launch_cols_ks<4>(N, dd, ku, V, Zc, Zb, ids, E, U, Y, gather_z, kz, st);
  }
}

}  // namespace ssn
