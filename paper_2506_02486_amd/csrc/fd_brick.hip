// fd_brick.hip -- the forward update and the gradient pass of grids that the caches
// hold (gfx950).
//
// A grid of up to about 14 million points has its four arrays (16 bytes per point) in
// the L2 and last-level caches between steps, which stream them at 7-8 TB/s, and its
// step is over in 4-35 us: too short for a z march, whose blocks spend a few
// microseconds filling a nine-plane register queue and then wait one memory round trip
// per plane, and bound by the vector-memory path (25 loads per point, 112 bytes
// through L1) for one thread per point.  Here a block owns one brick of 32 or 64 x 16
// points and KZ planes and issues all its loads at once:
//   * a lane holds 4 consecutive x points (16-byte accesses) of the KZ planes and of
//     the 4 planes above and below them in registers: its z neighbours;
//   * the KZ planes and their x/y halos go through LDS, one barrier per brick: the x
//     and y neighbours.  Centre planes and halos are loaded first, so that the x and y
//     terms are computed while the z planes and the pointwise operands arrive;
//   * about 35 bytes per point pass L1 (KZ = 2), most of them hits in L2.
// Order of the bricks: an XCD takes a run of consecutive ones, whose u planes overlap by 8
// of 10 planes and 8 of 24 rows and are to be found in its 4 MB of L2.  With x, y, z
// order a layer of two planes puts 16 planes (10 of u, 3 x 2 others) between a plane's
// uses, more than L2 holds from about 50000 points per plane on, so larger planes are
// taken as bands of rows, each swept through z before the next (338 x 226 x 146 44.2 us
// per step -> 31.6, 512 x 128 x 128 27.5 -> 22.5, 224^3 31.3 -> 30.4).
//
// The arithmetic is that of the marching kernels, term for term and in the same order
// (centre, x pairs, y pairs, z pairs; the damped form only where eta != 0; the source,
// residual and receiver epilogues), so every kernel gives the same bits.
//
// KZ = 2 planes: 112-118 VGPRs, 16 waves per CU.  4 planes read less (26 bytes per
// point) but take 218 VGPRs and half the waves: slower from 64^3 to 224^3 (160^3: 16.0
// us against 13.5).  One plane on grids of at most 2^20 points, which leave CUs idle
// otherwise (80^3: 4.5 us against 4.8).  8 lanes (32 points, 128 threads) where 64-wide
// bricks would cover a tenth more of the x extent than 32-wide ones, 16 lanes (64
// points, 256 threads, fewer x halos) elsewhere with two planes: 192^3 20.1 us (16 lanes)
// against 20.6, 160^3 13.7 against 13.2, 224^3 32.4 against 30.9.  Bricks of one plane are
// 32 points wide (brick_lanes says why).
//
// Measured (us per step in the native loop, sponge 16, before / after; before: one
// thread per point up to 160^3, 64 x 32 marching tiles at 192^3, 16-byte marching lanes
// above): 80^3 5.83 / 4.48, 96^3 6.72 / 5.36, 128^3 9.83 / 7.97, 141 x 119 x 133 15.5 /
// 9.6, 160^3 19.5 / 13.2, 192^3 26.2 / 20.1, 336 x 150 x 174 31.3 / 24.7, 224^3 37.7 /
// 30.4 (5.9 TB/s of the 16 bytes per point), 240^3 44.5 / 40.1; 256^3 (268 MB, past the
// last-level cache) would be 49.5 / 59.6.  A launch of an empty kernel in the same loop takes 2.4 us.
// The exchange form (all twelve faces): 96^3 9.80 / 7.35, 128^3 14.3 / 9.45, 160^3 25.5
// / 16.0, 224^3 47.0 / 37.8, 256^3 54.8 / 67.9.
//
// Exchange form (XCH): a float4 outside the interior is read from the receive buffer of
// its face (whole float4s: nx is a multiple of 4) and the faces of the result are
// written by the lanes that own them, so the exchange step is one launch.
#include <stdint.h>

#include <algorithm>

#include "fd_internal.h"

namespace fd {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int TROWS = 16;  // y rows of a brick

// FWD: the update.  GRAD: the gradient pass.  KEEP: the update, which also writes its
// stencil sum s_n = L u^n + f^n.  ACC: the update of the reverse sweep (u = b^{n+1}, up =
// b^{n+2}), which also adds the gradient terms of the s it is given (why: fd_stencil4.hip).
// 128^3: KEEP 8.7 us, ACC 14.8, update 8.0 (before, 64 x 32 marching tiles and one thread
// per point: 12.4 forward, 11.6 + 12.4 + a 2.7 us residual launch per reverse step); a
// gradient over 96 steps, checkpoints every 32: 4.85 -> 2.87 ms.
enum BrickMode { B_FWD = 0, B_GRAD = 1, B_KEEP = 2, B_ACC = 3 };

struct BrickArgs {
  Geo g;
  Coef c;
  const float* u;   // u^n (stencil field)
  const float* up;  // u^{n-1}  (GRAD: a^{n+1})
  const float* q;   // vdt2     (GRAD: the accumulator, as un)
  float* un;        // u^{n+1}; may alias up
  const float* ex;
  const float* ey;
  const float* ez;
  int tiles_x, tiles_y;
  // order of the bricks: x fastest, then the y rows of a band (band rows of bricks), then
  // z, then the bands; span: rows of bricks in a band (band x layers of z); mx, mspan,
  // mband, mlast: ceil(2^31 / d) of tiles_x, span, band and the last band's rows
  int band, span;
  unsigned mx, mspan, mband, mlast;
  int si, sj, sk;   // source point (si < 0: none)
  float sw;
  // receivers on plane rk (rk < 0: none): rmap[j * nx + i] is the receiver index of
  // point (i, j, rk) or -1; rrow takes u^{n+1} there, or (RADD) is added there, scaled
  // by vdt2 / (1+eta)
  int rk;
  const int32_t* rmap;
  float* rrow;
  // KEEP: s_n is written to keep.  ACC: g_acc += up s2 (if s2) + u s1
  float* keep;
  const float* s1;
  const float* s2;
  float* g_acc;
};
struct BrickFaces {
  const float* in[6];
  float* out[6];
};

__device__ __forceinline__ int remap_brick(int bid, int nb) {
  const int per = nb >> 3;
  if (bid < (per << 3)) return (bid & 7) * per + (bid >> 3);
  return bid;
}

__device__ __forceinline__ f4 ld4(const char* base, unsigned boff) {
  return *reinterpret_cast<const f4*>(base + boff);
}

template <int LANES, int KZ, bool SPONGE, bool XCH, BrickMode MODE, bool RADD>
__device__ __forceinline__ void brick_block(const BrickArgs& p, const BrickFaces& fc,
                                            const int bx, const int by, const int bz,
                                            const int t) {
  constexpr bool GRAD = MODE == B_GRAD, KEEP = MODE == B_KEEP, ACC = MODE == B_ACC;
  constexpr int BT = LANES * TROWS;
  constexpr int TX = 4 * LANES;
  constexpr int LX = TX + 8;
  constexpr int LY = TROWS + 8;
  constexpr int HY = 8 * LANES;         // float4 of y halo per plane
  constexpr int HX = 2 * TROWS;         // float4 of x halo per plane
  constexpr int HP = HY + HX;
  constexpr int HN = (HP * KZ + BT - 1) / BT;  // halo float4 a thread loads
  __shared__ __attribute__((aligned(16))) float sm[KZ * LY * LX];

  const int lx = t % LANES, ty = t / LANES;
  const int nx = p.g.nx, ny = p.g.ny, nz = p.g.nz, sy = p.g.sy;
  const long long szb = 4LL * p.g.sz;
  const int x0 = bx * TX, y0 = by * TROWS, kb = bz * KZ;
  const int x = x0 + 4 * lx, y = y0 + ty;

  auto boff = [&](int xx, int yy) -> unsigned {
    return 4u * (unsigned)((yy + 4) * sy + (xx + 4));
  };
  const int xcl_in = (nx + 3) & ~3, xcl_halo = nx & ~3;
  auto xcl = [&](int yy) { return yy < ny ? xcl_in : xcl_halo; };
  auto cell = [&](int xx, int yy) -> unsigned {
    const int yz = min(yy, ny + 3);
    return boff(min(xx, xcl(yz)), yz);
  };
  const long long org_c = p.g.org - 4LL * sy - 4;
  // planes kb - 4 .. kb + KZ + 3 of the field (clamped to the last halo plane)
  const char* F[KZ + 8];
  F[0] = reinterpret_cast<const char*>(p.u + org_c) + (long long)(kb - 4) * szb;
#pragma unroll
  for (int s = 1; s < KZ + 8; ++s) F[s] = F[s - 1] + (kb - 4 + s <= nz + 3 ? szb : 0);
  // exchange form: the face buffer that holds the float4 at (xx, yy) of plane k, or
  // (neither outside the interior, or outside on both axes) u itself
  auto xcell = [&](const char* plane, int xx, int yy, int k) -> const char* {
    const bool yin = yy >= 0 && yy < ny;
    if (xx < 0 && yin) return reinterpret_cast<const char*>(fc.in[0]) + 16ull * ((size_t)k * ny + yy);
    if (xx >= nx && yin) return reinterpret_cast<const char*>(fc.in[1]) + 16ull * ((size_t)k * ny + yy);
    if (xx >= 0 && xx < nx && yy < 0)
      return reinterpret_cast<const char*>(fc.in[2]) + 4ull * (((size_t)k * 4 + (yy + 4)) * nx + xx);
    if (xx >= 0 && xx < nx && yy >= ny && yy < ny + 4)
      return reinterpret_cast<const char*>(fc.in[3]) + 4ull * (((size_t)k * 4 + (yy - ny)) * nx + xx);
    return plane + cell(xx, yy);
  };
  const int yp = min(y, ny - 1), xp = min(x, (nx - 1) & ~3);
  const unsigned co = cell(x, y), po = boff(xp, yp);
  auto zplane = [&](int s) -> f4 {
    if constexpr (XCH) {
      const int k = kb - 4 + s;
      if (k < 0)
        return *reinterpret_cast<const f4*>(fc.in[4] + ((size_t)(k + 4) * ny + yp) * nx + xp);
      if (k >= nz)
        return *reinterpret_cast<const f4*>(fc.in[5] + ((size_t)(min(k, nz + 3) - nz) * ny + yp) * nx + xp);
    }
    return ld4(F[s], co);
  };

  // ---- loads: the brick's planes and their halos first
  f4 zc[KZ + 8];
#pragma unroll
  for (int s = 0; s < KZ; ++s) {
    if constexpr (XCH)
      zc[s + 4] = kb + s < nz ? *reinterpret_cast<const f4*>(xcell(F[s + 4], x, y, kb + s)) : zplane(s + 4);
    else
      zc[s + 4] = ld4(F[s + 4], co);
  }
  f4 hv[HN];
  int hl[HN];
#pragma unroll
  for (int h = 0; h < HN; ++h) {
    const int id = HP * KZ % BT == 0 ? t + h * BT : min(t + h * BT, HP * KZ - 1);
    const int s = id / HP, r = id - s * HP;
    int hx, hy;
    if (r < HY) {
      const int row = r / LANES;
      hx = x0 + 4 * (r % LANES);
      hy = row < 4 ? y0 - 4 + row : y0 + TROWS + (row - 4);
    } else {
      const int e = r - HY;
      hx = (e & 1) ? x0 + TX : x0 - 4;
      hy = y0 + (e >> 1);
    }
    hl[h] = s * (LY * LX) + (hy - y0 + 4) * LX + (hx - x0 + 4);
    const int kk = min(s, nz - 1 - kb);
    if constexpr (XCH)
      hv[h] = *reinterpret_cast<const f4*>(xcell(F[4] + (long long)kk * szb, hx, hy, kb + kk));
    else
      hv[h] = ld4(F[4], (unsigned)kk * (unsigned)szb + cell(hx, hy));
  }
  __builtin_amdgcn_sched_barrier(0);
  // ---- the planes above and below the brick
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    zc[3 - s] = zplane(3 - s);
    zc[KZ + 4 + s] = zplane(KZ + 4 + s);
  }
  // ---- pointwise operands
  f4 pa[KZ], pb[KZ];
  {
    const char* A = reinterpret_cast<const char*>(p.up + org_c) + (long long)kb * szb;
    const char* B = reinterpret_cast<const char*>(p.q + org_c) + (long long)kb * szb;
#pragma unroll
    for (int s = 0; s < KZ; ++s) {
      pa[s] = ld4(A, po);
      pb[s] = ld4(B, po);
      A += kb + s + 1 < nz ? szb : 0;
      B += kb + s + 1 < nz ? szb : 0;
    }
  }
  f4 s1v[KZ], s2v[KZ], gv[KZ];
  if constexpr (ACC) {
    const char* S1 = reinterpret_cast<const char*>(p.s1 + org_c) + (long long)kb * szb;
    const char* S2 = reinterpret_cast<const char*>((p.s2 ? p.s2 : p.s1) + org_c) + (long long)kb * szb;
    const char* G0 = reinterpret_cast<const char*>(p.g_acc + org_c) + (long long)kb * szb;
#pragma unroll
    for (int s = 0; s < KZ; ++s) {
      const long long o = kb + s < nz ? s * szb : 0;
      s1v[s] = ld4(S1 + o, po);
      s2v[s] = ld4(S2 + o, po);
      gv[s] = ld4(G0 + o, po);
    }
  }
  float exc[4] = {0.f, 0.f, 0.f, 0.f}, eyr = 0.f;
  float ezk[KZ];
  bool damp_xy = false;
#pragma unroll
  for (int s = 0; s < KZ; ++s) ezk[s] = 0.f;
  if constexpr (SPONGE) {
#pragma unroll
    for (int e = 0; e < 4; ++e) exc[e] = p.ex[min(x + e, nx - 1)];
    eyr = p.ey[yp];
#pragma unroll
    for (int s = 0; s < KZ; ++s) ezk[s] = p.ez[min(kb + s, nz - 1)];
    damp_xy = exc[0] != 0.f || exc[1] != 0.f || exc[2] != 0.f || exc[3] != 0.f || eyr != 0.f;
  }
  const bool rec_brick = !GRAD && p.rk >= kb && p.rk < kb + KZ;
  int rix[4] = {-1, -1, -1, -1};
  float rval[4] = {0.f, 0.f, 0.f, 0.f};
  if (rec_brick) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = p.rmap[(long long)yp * nx + min(x + e, nx - 1)];
      rix[e] = x + e < nx && y < ny ? r : -1;
    }
    if constexpr (RADD) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (rix[e] >= 0) rval[e] = p.rrow[rix[e]];
    }
  }

  __builtin_amdgcn_sched_barrier(0);
  // ---- stage the brick
#pragma unroll
  for (int s = 0; s < KZ; ++s)
    *reinterpret_cast<f4*>(sm + s * (LY * LX) + (4 + ty) * LX + 4 + 4 * lx) = zc[s + 4];
#pragma unroll
  for (int h = 0; h < HN; ++h)
    if (HP * KZ % BT == 0 || t + h * BT < HP * KZ) *reinterpret_cast<f4*>(sm + hl[h]) = hv[h];
  __syncthreads();

  const Coef& c = p.c;
  const bool src_tile = p.si >= x0 && p.si < x0 + TX && p.sj >= y0 && p.sj < y0 + TROWS &&
                        p.sk >= kb && p.sk < kb + KZ;
  const bool act = x < nx && y < ny, full = x + 4 <= nx && y < ny;
  const unsigned cb = boff(x, y);
  // x and y terms of every plane, while the z planes and pointwise operands arrive
  f4 lap[KZ];
#pragma unroll
  for (int s = 0; s < KZ; ++s) {
    const float* m0 = sm + s * (LY * LX) + (4 + ty) * LX + 4 + 4 * lx;
    const f4 lf = *reinterpret_cast<const f4*>(m0 - 4);
    const f4 rt = *reinterpret_cast<const f4*>(m0 + 4);
    const f4 uc = zc[s + 4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      auto X = [&](int o) -> float {
        const int j = e + o;
        return j < 0 ? lf[j + 4] : (j > 3 ? rt[j - 4] : uc[j]);
      };
      float l = c.cc * uc[e];
#pragma unroll
      for (int m = 1; m <= 4; ++m) l += c.cx[m] * (X(m) + X(-m));
      lap[s][e] = l;
    }
#pragma unroll
    for (int m = 1; m <= 4; ++m) {
      const f4 yu = *reinterpret_cast<const f4*>(m0 + m * LX);
      const f4 yd = *reinterpret_cast<const f4*>(m0 - m * LX);
#pragma unroll
      for (int e = 0; e < 4; ++e) lap[s][e] += c.cy[m] * (yu[e] + yd[e]);
    }
  }
#pragma unroll
  for (int s = 0; s < KZ; ++s) {
    const int k = kb + s;
    const f4 uc = zc[s + 4];
    const f4 ua = pa[s], ub = pb[s];
    f4 eta = {0.f, 0.f, 0.f, 0.f};
    const bool damped = SPONGE && (damp_xy || ezk[s] != 0.f);
    const bool src_plane = src_tile && k == p.sk;
    f4 v4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float l = lap[s][e];
#pragma unroll
      for (int m = 1; m <= 4; ++m) l += c.cz[m] * (zc[s + 4 + m][e] + zc[s + 4 - m][e]);
      // s_n = L u + f: f is added where it is 0 too (that decides the sign of a zero), as
      // in the gradient mode of the marching kernels
      if constexpr (GRAD || KEEP)
        lap[s][e] = l + (src_plane && x + e == p.si && y == p.sj ? p.sw : 0.f);
      if constexpr (!GRAD) v4[e] = 2.f * uc[e] - ua[e] + ub[e] * l;
      if constexpr (ACC) {
        if (p.s2) gv[s][e] += ua[e] * s2v[s][e];
        gv[s][e] += uc[e] * s1v[s][e];
      }
    }
    if constexpr (GRAD) {
      // g += D a (L u + f)
      f4 da = ua;
      if (damped) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          eta[e] = exc[e] + eyr + ezk[s];
          if (eta[e] != 0.f) da[e] = __builtin_amdgcn_rcpf(1.f + eta[e]) * ua[e];
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) v4[e] = ub[e] + da[e] * lap[s][e];
    } else {
      if (damped) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          eta[e] = exc[e] + eyr + ezk[s];
          const float w = (v4[e] + eta[e] * ua[e]) * __builtin_amdgcn_rcpf(1.f + eta[e]);
          v4[e] = eta[e] != 0.f ? w : v4[e];
        }
      }
      if (src_plane) {
        const int e = p.si - x;
        if (e >= 0 && e < 4 && y == p.sj) {
#pragma clang fp contract(off)
          const float qs = e == 0 ? ub[0] : e == 1 ? ub[1] : e == 2 ? ub[2] : ub[3];
          const float es = e == 0 ? eta[0] : e == 1 ? eta[1] : e == 2 ? eta[2] : eta[3];
          const float a = qs * p.sw / (1.f + es);
          v4[0] = e == 0 ? v4[0] + a : v4[0];
          v4[1] = e == 1 ? v4[1] + a : v4[1];
          v4[2] = e == 2 ? v4[2] + a : v4[2];
          v4[3] = e == 3 ? v4[3] + a : v4[3];
        }
      }
      if (rec_brick && k == p.rk) {
        if constexpr (RADD) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
#pragma clang fp contract(off)
            if (rix[e] >= 0) v4[e] += rval[e] * (ub[e] / (1.f + eta[e]));
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (rix[e] >= 0) p.rrow[rix[e]] = v4[e];
        }
      }
    }
    if (k >= nz) continue;
    float* d = reinterpret_cast<float*>(reinterpret_cast<char*>(p.un + org_c) + (long long)k * szb + cb);
    if (full) {
      *reinterpret_cast<f4*>(d) = v4;  // a plain store: the next step reads it from cache
      if constexpr (KEEP)
        __builtin_nontemporal_store(
            lap[s], reinterpret_cast<f4*>(reinterpret_cast<char*>(p.keep + org_c) + (long long)k * szb + cb));
      if constexpr (ACC)
        *reinterpret_cast<f4*>(reinterpret_cast<char*>(p.g_acc + org_c) + (long long)k * szb + cb) = gv[s];
      if constexpr (XCH) {
        const size_t kk = (size_t)k;
        if (x == 0) *reinterpret_cast<f4*>(fc.out[0] + (kk * ny + y) * 4) = v4;
        if (x == nx - 4) *reinterpret_cast<f4*>(fc.out[1] + (kk * ny + y) * 4) = v4;
        if (y < 4) *reinterpret_cast<f4*>(fc.out[2] + (kk * 4 + y) * nx + x) = v4;
        if (y >= ny - 4) *reinterpret_cast<f4*>(fc.out[3] + (kk * 4 + (y - (ny - 4))) * nx + x) = v4;
        if (k < 4) *reinterpret_cast<f4*>(fc.out[4] + (kk * ny + y) * nx + x) = v4;
        if (k >= nz - 4) *reinterpret_cast<f4*>(fc.out[5] + ((kk - (nz - 4)) * ny + y) * nx + x) = v4;
      }
    } else if (act) {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (x + e < nx) d[e] = v4[e];
      if constexpr (KEEP || ACC) {
        float* d2 = reinterpret_cast<float*>(
            reinterpret_cast<char*>((KEEP ? p.keep : p.g_acc) + org_c) + (long long)k * szb + cb);
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (x + e < nx) d2[e] = KEEP ? lap[s][e] : gv[s][e];
      }
    }
  }
}

// Tile of block `logical` of the grid p describes.
__device__ __forceinline__ void brick_tile(const BrickArgs& p, unsigned logical, int* bx, int* by,
                                           int* bz) {
  const unsigned rest = (unsigned)(((uint64_t)logical * p.mx) >> 31);
  const unsigned band = (unsigned)(((uint64_t)rest * p.mspan) >> 31);
  const unsigned in = rest - band * (unsigned)p.span;
  const int left = p.tiles_y - (int)band * p.band;
  const unsigned rows = (unsigned)min(p.band, left);
  const unsigned z = (unsigned)(((uint64_t)in * (left < p.band ? p.mlast : p.mband)) >> 31);
  *bx = (int)(logical - rest * (unsigned)p.tiles_x);
  *by = (int)(band * (unsigned)p.band + in - z * rows);
  *bz = (int)z;
}

// waves per SIMD the register budget must allow: 16 waves per CU, 12 where two planes
// with a further operand or two per point would spill at that
constexpr int brick_waves(int kz, BrickMode mode) {
  return kz > 1 && (mode == B_GRAD || mode == B_ACC) ? 3 : 4;
}

template <int LANES, int KZ, bool SPONGE, bool XCH, BrickMode MODE, bool RADD>
__global__ void __launch_bounds__(LANES * TROWS, brick_waves(KZ, MODE))
    brick_kernel(BrickArgs p, BrickFaces fc) {
  int bx, by, bz;
  brick_tile(p, (unsigned)remap_brick(blockIdx.x, gridDim.x), &bx, &by, &bz);
  brick_block<LANES, KZ, SPONGE, XCH, MODE, RADD>(p, fc, bx, by, bz, threadIdx.x);
}

// One step of several grids in one launch, their parameters in the kernel arguments:
// grid i owns blocks [start[i], start[i+1]).
struct BrickMulti {
  int start[kBrickMulti + 1];
  BrickArgs grid[kBrickMulti];
};

template <int KZ>
__global__ void __launch_bounds__(8 * TROWS, brick_waves(KZ, B_FWD))
    brick_multi_kernel(BrickMulti A) {
  const int b = remap_brick(blockIdx.x, gridDim.x);
  // the grid that owns block b: all starts compared at once (unused ones lie past the
  // last block; a search would wait for one kernel-argument load after another)
  int i = 0;
#pragma unroll
  for (int j = 1; j < kBrickMulti; ++j) i += b >= A.start[j];
  const BrickArgs& p = A.grid[i];
  int bx, by, bz;
  brick_tile(p, (unsigned)(b - A.start[i]), &bx, &by, &bz);
  brick_block<8, KZ, true, false, B_FWD, false>(p, BrickFaces{}, bx, by, bz, threadIdx.x);
}

// Grids up to this many points take one plane per brick: with two, a 64^3 grid has 256
// blocks of 128 threads (one per CU) and finishes later.
constexpr long long kOnePlanePoints = 1LL << 20;

int brick_planes(long long points) { return points <= kOnePlanePoints ? 1 : 2; }
int brick_planes(const Geo& g) { return brick_planes((long long)g.nx * g.ny * g.nz); }

// 16 lanes (64 points) where 64-wide bricks cover at most a tenth more than 32-wide
// ones (the figures are at the top of this file).  One-plane bricks, whose grids leave CUs
// idle, always 8: twice the blocks; us per step, 16 lanes / 8: 392 x 53 x 32 6.9 / 6.3 (one
// thread per point 5.8-6.2), 64 x 64 x 200 5.0 / 4.5, 120 x 109 x 68 6.5 / 6.2, 128 x 64 x 64
// 4.7 / 4.6; over 44 grids of 0.45 to 1 million points a mean of 1.05, the worst (36 x 90 x
// 238) 0.97.
int brick_lanes(const Geo& g) {
  if (brick_planes(g) == 1) return 8;
  const int c64 = (g.nx + 63) / 64 * 64, c32 = (g.nx + 31) / 32 * 32;
  return 10 * c64 <= 11 * c32 ? 16 : 8;
}

unsigned magic31(int d) { return (unsigned)(((1ull << 31) + d - 1) / d); }

// Rows of bricks per band of the order (see the top) for planes of rows x width points
// (the bricks' extent): equal bands of about kBandPoints, of any size for planes of at
// most kWholePoints.  us per step, whole planes / bands of 2, 4, 6 or 8 rows: 338 x 226 x
// 146 44.2 / 32.5, 31.9, 31.7, -; 512 x 128 x 128 27.5 / 22.5, 22.7, 23.5, -; 256 x 256 x
// 200 42.4 / 36.9, 35.7, 36.1, 37.1; 512 x 200 x 136 62.2 / 37.5, 37.2, 40.8, 45.3; 192^3
// 20.4 / 20.9, 20.3, 20.1, -; 96 x 300 x 300 (29k points a plane) 24.6 / 26.8, 25.8, 25.5, -.
constexpr int kBandPoints = 24576, kWholePoints = 32768;

int brick_band(int width, int rows) {
  const int row = TROWS * width;
  if ((long long)rows * row <= kWholePoints) return rows;
  const int most = std::max(1, (kBandPoints + row / 2) / row);
  const int bands = (rows + most - 1) / most;
  return (rows + bands - 1) / bands;
}

BrickArgs brick_args(const Geo& g, const Coef& c, const float* up, const float* u, float* un,
                     const float* q, const float* ex, const float* ey, const float* ez,
                     const fd_source* src, const RecPlane* rp, int lanes, int kz) {
  BrickArgs p{};
  p.g = g;
  p.c = c;
  p.u = u;
  p.up = up;
  p.q = q;
  p.un = un;
  p.ex = ex;
  p.ey = ey;
  p.ez = ez;
  p.tiles_x = (g.nx + 4 * lanes - 1) / (4 * lanes);
  p.tiles_y = (g.ny + TROWS - 1) / TROWS;
  p.band = brick_band(p.tiles_x * 4 * lanes, p.tiles_y);
  p.span = p.band * ((g.nz + kz - 1) / kz);
  p.mx = magic31(p.tiles_x);
  p.mspan = magic31(p.span);
  p.mband = magic31(p.band);
  const int last = p.tiles_y % p.band;
  p.mlast = magic31(last ? last : p.band);
  p.si = p.sj = p.sk = -1;
  if (src) {
    p.si = src->i;
    p.sj = src->j;
    p.sk = src->k;
    p.sw = src->w;
  }
  p.rk = -1;
  if (rp && rp->map) {
    p.rmap = rp->map;
    p.rk = rp->k;
    p.rrow = rp->row;
  }
  return p;
}

template <bool SPONGE, bool XCH, BrickMode MODE, bool RADD>
hipError_t launch_bricks(const BrickArgs& p, const BrickFaces& fc, int lanes, hipStream_t s) {
  const int kz = brick_planes(p.g);
  const long long nb = (long long)p.tiles_x * p.tiles_y * ((p.g.nz + kz - 1) / kz);
  if (nb <= 0 || nb > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)nb), block((unsigned)(lanes * TROWS));
#define FD_BRICK(L, K) \
  hipLaunchKernelGGL((brick_kernel<L, K, SPONGE, XCH, MODE, RADD>), grid, block, 0, s, p, fc)
  if (kz == 1) FD_BRICK(8, 1);  // (brick_lanes)
  else if (lanes == 8) FD_BRICK(8, 2);
  else FD_BRICK(16, 2);
#undef FD_BRICK
  return hipGetLastError();
}

bool aligned16(const void* ptr) { return ((uintptr_t)ptr & 15u) == 0; }

}  // namespace

bool brick_grid(const Geo& g, long long most) {
  if (tile_override() != 0) return false;
  if (g.sy % 4 || g.sz % 4 || g.org % 4) return false;
  const long long points = (long long)g.nx * g.ny * g.nz;
  if (points > most) return false;
  // bricks that cover more than twice the grid (extents far below 32 x 16) waste what
  // the other kernels' shapes do not
  const long long tx = (g.nx + 31) / 32, ty = (g.ny + TROWS - 1) / TROWS;
  if (tx * 32 * ty * TROWS > 2LL * g.nx * g.ny) return false;
  if (tx * 32 * ty * TROWS * g.nz > kBrickCover) return false;
  // the divisions of brick_tile are exact while dividend x divisor stays below 2^31
  // (blocks by tiles_x, rows of bricks by a band's)
  const long long kz = brick_planes(g), rows = ty * ((g.nz + kz - 1) / kz);
  return tx * rows * tx < (1LL << 31) && rows * rows < (1LL << 31);
}

bool brick_step(const Geo& g, bool faces, long long most) {
  const long long lanes = (long long)((g.nx + 63) / 64 * 64) * g.ny * g.nz;
  if (lanes <= (faces ? kBrickLeastFaces : kBrickLeast)) return false;
  if (faces && (g.nx % 4 || g.ny < 4 || g.nz < 4)) return false;
  return brick_grid(g, most);
}

bool brick_takes(const Geo& g, const float* const arrays[4], long long most,
                 const float* const* in, float* const* out) {
  if (!brick_step(g, in != nullptr, most)) return false;
  for (int i = 0; i < 4; ++i)
    if (!arrays[i] || !aligned16(arrays[i])) return false;
  for (int f = 0; in && f < 6; ++f)
    if (!in[f] || !out[f] || !aligned16(in[f]) || !aligned16(out[f])) return false;
  return true;
}

hipError_t launch_brick(const Geo& g, const Coef& c, const float* up, const float* u, float* un,
                        const float* q, const float* ex, const float* ey, const float* ez,
                        const fd_source* src, const RecPlane* rp, hipStream_t s,
                        const float* const* in, float* const* out) {
  const int lanes = brick_lanes(g);
  const BrickArgs p = brick_args(g, c, up, u, un, q, ex, ey, ez, src, rp, lanes, brick_planes(g));
  const bool radd = rp && rp->map && rp->add;
  BrickFaces fc{};
  if (in) {
    if (radd) return hipErrorInvalidValue;  // exchange: records only
    for (int f = 0; f < 6; ++f) {
      fc.in[f] = in[f];
      fc.out[f] = out[f];
    }
    return ex ? launch_bricks<true, true, B_FWD, false>(p, fc, lanes, s)
              : launch_bricks<false, true, B_FWD, false>(p, fc, lanes, s);
  }
  if (radd)
    return ex ? launch_bricks<true, false, B_FWD, true>(p, fc, lanes, s)
              : launch_bricks<false, false, B_FWD, true>(p, fc, lanes, s);
  return ex ? launch_bricks<true, false, B_FWD, false>(p, fc, lanes, s)
            : launch_bricks<false, false, B_FWD, false>(p, fc, lanes, s);
}

hipError_t launch_grad_brick(const Geo& g, const Coef& c, const float* u, const float* an1,
                             float* gq, const float* ex, const float* ey, const float* ez,
                             const fd_source* src, hipStream_t s) {
  const int lanes = brick_lanes(g);
  const BrickArgs p = brick_args(g, c, an1, u, gq, gq, ex, ey, ez, src, nullptr, lanes, brick_planes(g));
  return ex ? launch_bricks<true, false, B_GRAD, false>(p, BrickFaces{}, lanes, s)
            : launch_bricks<false, false, B_GRAD, false>(p, BrickFaces{}, lanes, s);
}

hipError_t launch_keep_brick(const Geo& g, const Coef& c, const float* up, const float* u,
                             float* un, const float* q, const float* ex, const float* ey,
                             const float* ez, const fd_source* src, const RecPlane* rp,
                             float* keep, hipStream_t s) {
  const int lanes = brick_lanes(g);
  BrickArgs p = brick_args(g, c, up, u, un, q, ex, ey, ez, src, rp, lanes, brick_planes(g));
  p.keep = keep;
  return ex ? launch_bricks<true, false, B_KEEP, false>(p, BrickFaces{}, lanes, s)
            : launch_bricks<false, false, B_KEEP, false>(p, BrickFaces{}, lanes, s);
}

hipError_t launch_acc_brick(const Geo& g, const Coef& c, const float* up, const float* u, float* un,
                            const float* q, const float* ex, const float* ey, const float* ez,
                            const RecPlane* rp, const float* s1, const float* s2, float* g_acc,
                            hipStream_t s) {
  const int lanes = brick_lanes(g);
  BrickArgs p = brick_args(g, c, up, u, un, q, ex, ey, ez, nullptr, rp, lanes, brick_planes(g));
  p.s1 = s1;
  p.s2 = s2;
  p.g_acc = g_acc;
  return ex ? launch_bricks<true, false, B_ACC, true>(p, BrickFaces{}, lanes, s)
            : launch_bricks<false, false, B_ACC, true>(p, BrickFaces{}, lanes, s);
}

hipError_t launch_brick_multi(const WideStep* steps, int n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n > kBrickMulti) return hipErrorInvalidValue;
  long long points = 0;
  for (int i = 0; i < n; ++i) points += (long long)steps[i].g.nx * steps[i].g.ny * steps[i].g.nz;
  const int kz = brick_planes(points);
  BrickMulti A;
  long long nb = 0;
  for (int i = 0; i < n; ++i) {
    const WideStep& w = steps[i];
    A.start[i] = (int)nb;
    A.grid[i] = brick_args(w.g, w.c, w.up, w.u, w.un, w.q, w.ex, w.ey, w.ez, &w.src, &w.rec, 8, kz);
    nb += (long long)A.grid[i].tiles_x * A.grid[i].tiles_y * ((w.g.nz + kz - 1) / kz);
    if (nb > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  }
  for (int i = n; i <= kBrickMulti; ++i) A.start[i] = (int)nb;
  const dim3 grid((unsigned)nb), block(8 * TROWS);
  if (kz == 1) hipLaunchKernelGGL(brick_multi_kernel<1>, grid, block, 0, s, A);
  else hipLaunchKernelGGL(brick_multi_kernel<2>, grid, block, 0, s, A);
  return hipGetLastError();
}

}  // namespace fd
