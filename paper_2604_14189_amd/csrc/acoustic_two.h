// Acoustic step of a piece of 64 columns x 8 rows in items of two columns (the
// recurrence of acoustic.hip with the same operations in the same order, so the
// same bits), for NX >= 2 and any P: the pieces that the four-column items of
// acoustic_wide.hip do not fit. Device code.
//
// Such a step is bound by latency, of the chain load -> LDS -> memory variables ->
// LDS -> update: all loads of a thread are issued before the first use, and every
// thread stages its own cells and at most two 2-column items of each halo (no
// index division, no loop).
#pragma once

#include "fd.h"
#include "internal.h"

namespace sweep {

// Steps of encoded shots (kMany): the sources of a shot, one a lane (64 from k0 on;
// -1: none), loaded with the fields.
__device__ __forceinline__ int lane_source(const AcStep& a, int shot, int k0) {
  const int k = k0 + (int)(threadIdx.x & 63);
  return k < a.nsrc ? a.src_cell[(size_t)shot * a.nsrc + k] : -1;
}
// f(cell, sample) for each source of the shot in the cells [lo, lo + n) of this wave's
// rows, in their order (coincident sources add up as one after the other). Every wave
// has all of its lanes here. A loop over the sources in every lane, as one source per
// shot has it (where it is the faster one by 3 % in odd sizes), took 80 ns a source
// and piece: 1080 x 380 cells, 64 shots of 32 sources, 189 us a forward step, now 86
// (144 by tile sets).
template <class F>
__device__ __forceinline__ void each_source(const AcStep& a, int shot, int sc, int lo, int n, F f) {
  for (int k0 = 0; k0 < a.nsrc; k0 += 64) {
    if (k0) sc = lane_source(a, shot, k0);
    for (unsigned long long m = __ballot(sc >= lo && sc < lo + n); m; m &= m - 1) {
      const int k = __builtin_ctzll(m);
      f(__builtin_amdgcn_readlane(sc, k),
        a.w * a.wavelet[((size_t)shot * a.nsrc + k0 + k) * a.nt + a.n]);
    }
  }
}

namespace two {

typedef float f2 __attribute__((ext_vector_type(2)));
// rows and strips start at any 4-byte address when NX or P is odd
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
constexpr f2 kZero = {0.0f, 0.0f};
constexpr int kGZ = 8;  // rows of a piece

// Two consecutive floats at element i of a work-group-uniform base (32-bit
// byte offset, as u32at).
__device__ __forceinline__ f2 ld2(const float* f, unsigned i) {
  return *reinterpret_cast<const f2u*>(reinterpret_cast<const char*>(f) + i * 4u);
}
__device__ __forceinline__ void st2(float* f, unsigned i, f2 v) {
  *reinterpret_cast<f2u*>(reinterpret_cast<char*>(f) + i * 4u) = v;
}
__device__ __forceinline__ f2 lds2(const float* s) { return *reinterpret_cast<const f2*>(s); }
__device__ __forceinline__ void put2(float* s, f2 v) { *reinterpret_cast<f2*>(s) = v; }
__device__ __forceinline__ f2 fma2(f2 a, f2 b, f2 c) {
  return f2{fmaf(a.x, b.x, c.x), fmaf(a.y, b.y, c.y)};
}
__device__ __forceinline__ f2 fma2(float a, f2 b, f2 c) { return fma2(f2{a, a}, b, c); }

// The 2 cells c of an LDS row and the 4 on either side.
struct XWin {
  float w[10];
  __device__ __forceinline__ XWin(const float* at, f2 c) {
    const f2 a = lds2(at - 4), b = lds2(at - 2), d = lds2(at + 2), e = lds2(at + 4);
    const float v[10] = {a.x, a.y, b.x, b.y, c.x, c.y, d.x, d.y, e.x, e.y};
#pragma unroll
    for (int i = 0; i < 10; ++i) w[i] = v[i];
  }
  // D2', the operations of d2c: f_{i-k} - f_i is the exact negative of the
  // difference formed at i - k, so adding it is subtracting that one
  __device__ __forceinline__ f2 d2() const {
    float s[2];
#pragma unroll
    for (int k = 1; k <= 4; ++k) {
      const float ak = k == 1 ? kA1 : k == 2 ? kA2 : k == 3 ? kA3 : kA4;
      float e[6];
#pragma unroll
      for (int i = 0; i < 2 + k; ++i) e[i] = w[4 + i] - w[4 + i - k];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float d = e[j + k] - e[j];
        s[j] = k == 1 ? ak * d : fmaf(ak, d, s[j]);
      }
    }
    return f2{s[0], s[1]};
  }
  __device__ __forceinline__ f2 d1() const {
    return f2{d1c(w[5], w[3], w[6], w[2], w[7], w[1], w[8], w[0]),
              d1c(w[6], w[4], w[7], w[3], w[8], w[2], w[9], w[1])};
  }
};
// The 2 cells c of an LDS column pair and the 4 rows (st floats apart) on
// either side; D2' and D1' along z.
struct ZWin {
  f2 c, p[4], m[4];
  __device__ __forceinline__ ZWin(const float* at, int st) {
    c = lds2(at);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      p[k] = lds2(at + (k + 1) * st);
      m[k] = lds2(at - (k + 1) * st);
    }
  }
  __device__ __forceinline__ f2 d2() const {
    return f2{d2c(c.x, p[0].x, m[0].x, p[1].x, m[1].x, p[2].x, m[2].x, p[3].x, m[3].x),
              d2c(c.y, p[0].y, m[0].y, p[1].y, m[1].y, p[2].y, m[2].y, p[3].y, m[3].y)};
  }
  __device__ __forceinline__ f2 d1() const {
    return f2{d1c(p[0].x, m[0].x, p[1].x, m[1].x, p[2].x, m[2].x, p[3].x, m[3].x),
              d1c(p[0].y, m[0].y, p[1].y, m[1].y, p[2].y, m[2].y, p[3].y, m[3].y)};
  }
};

// One piece of one shot: rows z0 .. z0+7, columns x0 .. x0+63; the thread's
// columns are gx, gx+1 and its row gz. kOdd: NX or P is odd, so that a 2-column
// item may lie across the right edge or a strip's edge; otherwise it is inside
// or outside as a whole. Loads come from a valid address and are selected
// afterwards (no branch); the other column's value read across a strip's edge
// is some other memory variable of the row.
template <bool kOdd>
struct Piece {
  int NX, NZ, P, P2, x0, z0;

  __device__ __forceinline__ bool in(int gz, int gx) const {
    return (unsigned)gz < (unsigned)NZ && (unsigned)gx < (unsigned)NX;
  }
  // keeps the columns of v for which the first (ok0) and second (ok1) hold
  __device__ __forceinline__ static f2 sel(bool ok0, bool ok1, f2 v, f2 u = kZero) {
    return f2{ok0 ? v.x : u.x, ok1 ? v.y : u.y};
  }
  // f at row gz, columns gx and gx+1, 0 outside the grid
  __device__ __forceinline__ f2 get(const float* f, int gz, int gx) const {
    if (!kOdd) {
      const bool ok = in(gz, gx);
      return sel(ok, ok, ld2(f, ok ? (unsigned)(gz * NX + gx) : 0u));
    }
    const bool ok0 = in(gz, gx), ok1 = in(gz, gx + 1);
    // the item across the right edge is read one column further left (there is one:
    // NX >= 2)
    const int sh = ok0 && !ok1 ? 1 : 0;
    const f2 v = ld2(f, ok0 || ok1 ? (unsigned)max(gz * NX + gx - sh, 0) : 0u);
    return sel(ok0, ok1, f2{sh ? v.y : v.x, v.y});
  }
  __device__ __forceinline__ void set(float* f, int gz, int gx, f2 v) const {
    const unsigned i = (unsigned)(gz * NX + gx);
    if (in(gz, gx) && (!kOdd || gx + 1 < NX))
      st2(f, i, v);
    else if (kOdd && in(gz, gx))
      u32at(f, i) = v.x;
  }
  // whether column gx (+ j) of row gz is in an x strip
  __device__ __forceinline__ bool xin(int gz, int gx) const {
    return in(gz, gx) && (gx < P || gx >= NX - P);
  }
  // offset of columns gx, gx+1 in an x-strip array and the memory variable there
  // (q0, q1: which of them are in a strip), 0 elsewhere
  __device__ __forceinline__ unsigned xoff(int gz, int gx) const {
    return (unsigned)(gz * P2 + (gx < P ? gx : gx - (NX - P2)));
  }
  __device__ __forceinline__ f2 getx(const float* m, int gz, int gx, bool q0, bool q1) const {
    if (!kOdd) return sel(q0, q0, ld2(m, q0 ? xoff(gz, gx) : 0u));
    const unsigned i = q0 || q1 ? xoff(gz, gx) : 0u;
    return sel(q0, q1, f2{u32at(m, i), u32at(m, q1 ? i + 1 : 0u)});
  }
  __device__ __forceinline__ void setx(float* m, int gz, int gx, bool q0, bool q1, f2 v) const {
    const unsigned i = xoff(gz, gx);
    if (!kOdd) {
      if (q0) st2(m, i, v);
    } else {
      if (q0) u32at(m, i) = v.x;
      if (q1) u32at(m, i + 1) = v.y;
    }
  }
  // z-strip row of gz (-1: none) and the memory variable there
  __device__ __forceinline__ int zrow(int gz) const {
    return (unsigned)gz < (unsigned)NZ ? zstrip_row(gz, NZ, P) : -1;
  }
  __device__ __forceinline__ f2 getz(const float* m, int row, int gx) const {
    const bool ok = row >= 0 && gx < NX;
    if (!kOdd) return sel(ok, ok, ld2(m, ok ? (unsigned)(row * NX + gx) : 0u));
    const bool ok1 = row >= 0 && gx + 1 < NX;
    const unsigned i = ok ? (unsigned)(row * NX + gx) : 0u;
    return sel(ok, ok1, f2{u32at(m, i), u32at(m, ok1 ? i + 1 : 0u)});
  }
  __device__ __forceinline__ void setz(float* m, int row, int gx, f2 v) const {
    if (row < 0 || gx >= NX) return;
    if (!kOdd || gx + 1 < NX)
      st2(m, (unsigned)(row * NX + gx), v);
    else
      u32at(m, (unsigned)(row * NX + gx)) = v.x;
  }
  // C-PML coefficients of columns gx, gx+1 (0 outside the grid) and of row gz
  __device__ __forceinline__ f2 xco(const float* t, int gx) const {
    const bool ok = (unsigned)gx < (unsigned)NX, ok1 = (unsigned)(gx + 1) < (unsigned)NX;
    if (!kOdd) return sel(ok, ok, ld2(t, ok ? (unsigned)gx : 0u));
    return sel(ok, ok1, f2{u32at(t, ok ? (unsigned)gx : 0u), u32at(t, ok1 ? gx + 1u : 0u)});
  }
  __device__ __forceinline__ float zco(const float* t, int gz) const {
    return u32at(t, (unsigned)min(max(gz, 0), NZ - 1));
  }
};

// Staged arrays of a piece with x strips within 4 columns (HX) / z strips within
// 4 rows (HZ): along such an axis the field has a halo of 8 cells (the memory
// variables are formed on a 4-cell ring), else of 4.
template <bool HX, bool HZ>
struct GridGeom {
  static constexpr int hx = HX ? 8 : 4, hz = HZ ? 8 : 4;
  static constexpr int BW = kTX + 2 * hx, BH = kGZ + 2 * hz;
  static constexpr int XW = kTX + 8, ZH = kGZ + 8;
  static constexpr int NPX = HX ? kGZ * XW : 0, NPZ = HZ ? ZH * kTX : 0;
  static constexpr int kFwd = BW * BH + NPX + NPZ;
  static constexpr int kAdj = kGZ * BW + BH * kTX + NPX + NPZ;
  // halo rows a thread stages (8 rows of 32 items for each), and whether it
  // stages a side item: hx of them (hx / 2 on each side) in every row
  static constexpr int KZ = 2 * hz / 8;
  static constexpr int NXF = hx * BH;   // forward: all box rows (with the corners)
  static constexpr int NXA = hx * kGZ;  // adjoint: the piece's rows
};
constexpr int grid_lds(bool adj) {
  return adj ? GridGeom<true, true>::kAdj : GridGeom<true, true>::kFwd;
}
static_assert(GridGeom<true, true>::NXF <= kThreads, "one side item for each thread");

// Box row of halo row r (0 .. 2 hz - 1), box column of side item q.
template <class G>
__device__ __forceinline__ int halo_row(int r) { return r < G::hz ? r : r + kGZ; }
template <class G>
__device__ __forceinline__ int side_col(int q) {
  return q < G::hx / 2 ? 2 * q : kTX + 2 * q;
}

template <bool HX, bool HZ, bool kBorn, bool kMany, bool kOdd>
__device__ __forceinline__ void grid_fwd(const AcStep& a, const Piece<kOdd>& p, int shot,
                                         int tile, int row0, float* lds) {
  using G = GridGeom<HX, HZ>;
  constexpr int BW = G::BW, hx = G::hx, hz = G::hz, XW = G::XW;
  float* sb = lds;
  float* spx = lds + BW * G::BH;
  float* spz = spx + G::NPX;
  const int tid = threadIdx.x, lx = 2 * (tid & 31), zr = tid >> 5;
  const int gx = p.x0 + lx, gz = p.z0 + zr;
  const size_t plane = (size_t)p.NX * p.NZ;
  const float* cur = a.cur + shot * plane;
  const size_t xso = (size_t)shot * p.NZ * p.P2, zso = (size_t)shot * p.P2 * p.NX;

  // all loads of the step
  const int* ro = a.rec_off + (size_t)shot * a.ntiles + tile;
  const int e0 = ro[0], e1 = a.gathers ? ro[1] : 0;
  bool src = false;  // a source in this piece's rows (work-group-uniform)
  int lsrc = -1;
  if constexpr (kMany)
    lsrc = lane_source(a, shot, 0);
  else if constexpr (!kBorn)
    for (int k = 0; k < a.nsrc; ++k) {
      const int c = a.src_cell[shot * a.nsrc + k];
      src = src || (c >= p.z0 * p.NX && c < (p.z0 + kGZ) * p.NX);
    }
  const f2 own = p.get(cur, gz, gx);
  f2 zh[G::KZ], xh = kZero;
#pragma unroll
  for (int k = 0; k < G::KZ; ++k)
    zh[k] = p.get(cur, p.z0 - hz + halo_row<G>(zr + 8 * k), gx);
  const int sr = tid / hx, sc = side_col<G>(tid % hx);
  if (tid < G::NXF) xh = p.get(cur, p.z0 - hz + sr, p.x0 - hx + sc);
  const f2 pp = p.get(a.prev + shot * plane, gz, gx);
  const f2 cs = p.get(a.Cs, gz, gx);
  f2 bd = kZero, bb = kZero;
  if constexpr (kBorn) {
    bd = p.get(a.bdC, gz, gx);
    bb = p.get(a.bB + shot * plane, gz, gx);
  }
  // rings of the memory variables: columns x0-4 .. x0-1, x0+64 .. x0+67 of the
  // piece's rows (4 items a row, threads 0 .. 31) and rows z0-4 .. z0-1, z0+8 ..
  // z0+11 (one item for each thread)
  const int rr = tid >> 2, rc = (tid & 3) < 2 ? 2 * (tid & 3) - 4 : kTX + 2 * (tid & 3) - 4;
  const int rz = zr < 4 ? zr - 4 : zr + 4;
  bool q0 = false, q1 = false, h0 = false, h1 = false;
  f2 px, ex, axv, bxv, pxh, axh, bxh;
  if constexpr (HX) {
    q0 = p.xin(gz, gx);
    q1 = kOdd ? p.xin(gz, gx + 1) : q0;
    axv = p.xco(a.ax, gx);
    bxv = p.xco(a.bx, gx);
    px = p.getx(a.psx_in + xso, gz, gx, q0, q1);
    ex = p.getx(a.zex_in + xso, gz, gx, q0, q1);
    if (tid < 4 * kGZ) {
      h0 = p.xin(p.z0 + rr, p.x0 + rc);
      h1 = kOdd ? p.xin(p.z0 + rr, p.x0 + rc + 1) : h0;
      axh = p.xco(a.ax, p.x0 + rc);
      bxh = p.xco(a.bx, p.x0 + rc);
      pxh = p.getx(a.psx_in + xso, p.z0 + rr, p.x0 + rc, h0, h1);
    }
  }
  int row = -1, rowh = -1;
  f2 pz, ez, pzh;
  float az = 0.0f, bz = 0.0f, azh = 0.0f, bzh = 0.0f;
  if constexpr (HZ) {
    row = p.zrow(gz);
    rowh = p.zrow(p.z0 + rz);
    az = p.zco(a.az, gz);
    bz = p.zco(a.bz, gz);
    azh = p.zco(a.az, p.z0 + rz);
    bzh = p.zco(a.bz, p.z0 + rz);
    pz = p.getz(a.psz_in + zso, row, gx);
    ez = p.getz(a.zez_in + zso, row, gx);
    pzh = p.getz(a.psz_in + zso, rowh, gx);
  }
  int2 en = make_int2(0, 0);
  if (e0 + tid < e1) en = a.rec_ent[e0 + tid];

  put2(&sb[(zr + hz) * BW + hx + lx], own);
#pragma unroll
  for (int k = 0; k < G::KZ; ++k) put2(&sb[halo_row<G>(zr + 8 * k) * BW + hx + lx], zh[k]);
  if (tid < G::NXF) put2(&sb[sr * BW + sc], xh);
  __syncthreads();

  const float* at = &sb[(zr + hz) * BW + hx + lx];
  f2 Bx, Bz;
  {
    const XWin xw(at, own);
    Bx = xw.d2();
    if constexpr (HX) {
      // psi_x^n = b psi_x^{n-1} + a D1x' p^n in the strips
      const f2 ps = fma2(axv, xw.d1(), bxv * px);
      p.setx(a.psx_out + xso, gz, gx, q0, q1, ps);
      px = p.sel(q0, q1, ps);
      put2(&spx[zr * XW + 4 + lx], px);
      if (tid < 4 * kGZ) {
        const float* hat = &sb[(rr + hz) * BW + hx + rc];
        const f2 ph = fma2(axh, XWin(hat, lds2(hat)).d1(), bxh * pxh);
        put2(&spx[rr * XW + 4 + rc], p.sel(h0, h1, ph));
      }
    }
  }
  {
    const ZWin zw(at, BW);
    Bz = zw.d2();
    if constexpr (HZ) {
      const f2 ps = fma2(az, zw.d1(), bz * pz);
      p.setz(a.psz_out + zso, row, gx, ps);
      put2(&spz[(zr + 4) * kTX + lx], p.sel(row >= 0, row >= 0, ps));
      const f2 ph = fma2(azh, ZWin(&sb[(rz + hz) * BW + hx + lx], BW).d1(), bzh * pzh);
      put2(&spz[(rz + 4) * kTX + lx], p.sel(rowh >= 0, rowh >= 0, ph));
    }
  }
  if constexpr (HX || HZ) __syncthreads();
  if constexpr (HX) {
    Bx = Bx + XWin(&spx[zr * XW + 4 + lx], px).d1();
    const f2 ze = fma2(axv, Bx, bxv * ex);
    p.setx(a.zex_out + xso, gz, gx, q0, q1, ze);
    Bx = p.sel(q0, q1, Bx + ze, Bx);
  }
  if constexpr (HZ) {
    Bz = Bz + ZWin(&spz[(zr + 4) * kTX + lx], kTX).d1();
    const f2 ze = fma2(az, Bz, bz * ez);
    p.setz(a.zez_out + zso, row, gx, ze);
    Bz = p.sel(row >= 0, row >= 0, Bz + ze, Bz);
  }
  const f2 B = Bx + Bz;
  f2 out = fma2(cs, B, 2.0f * own - pp);
  if constexpr (kBorn) out = out + bd * bb;
  if constexpr (kMany)
    each_source(a, shot, lsrc, (p.z0 + (zr & ~1)) * p.NX, 2 * p.NX, [&](int cell, float sw) {
      const int d = cell - (gz * p.NX + gx);
      if (d == 0 && gx < p.NX) out.x += sw;
      if (d == 1 && gx + 1 < p.NX) out.y += sw;
    });
  if (src)
    for (int k = 0; k < a.nsrc; ++k) {
      const int d = a.src_cell[shot * a.nsrc + k] - (gz * p.NX + gx);
      const float sw = a.w * a.wavelet[((size_t)shot * a.nsrc + k) * a.nt + a.n];
      if (d == 0 && gx < p.NX) out.x += sw;
      if (d == 1 && gx + 1 < p.NX) out.y += sw;
    }
  p.set(a.next + shot * plane, gz, gx, out);
  if (a.B_out) p.set(a.B_out + shot * plane, gz, gx, B);
  if (e1 > e0) {  // the receivers of the tile in this piece's rows
    if constexpr (!(HX || HZ)) __syncthreads();  // sb is read until here
    put2(&sb[zr * kTX + lx], out);
    __syncthreads();
    float* dst = a.gathers + ((size_t)shot * a.nt + a.n) * a.nrec;
    for (int e = e0 + tid; e < e1; e += kThreads) {
      if (e >= e0 + kThreads) en = a.rec_ent[e];
      const int r = (en.x >> 6) - row0;
      if (r >= 0 && r < kGZ) dst[en.y] = sb[en.x - row0 * kTX];
    }
  }
}

template <bool HX, bool HZ, bool kOdd>
__device__ __forceinline__ void grid_adj(const AcStep& a, const Piece<kOdd>& p, int shot,
                                         int tile, int row0, float* lds) {
  using G = GridGeom<HX, HZ>;
  constexpr int BW = G::BW, hx = G::hx, hz = G::hz, XW = G::XW;
  float* sqx = lds;                 // Qbar_x: the piece's rows, columns x0-hx ..
  float* sqz = lds + kGZ * BW;      // Qbar_z: rows z0-hz .., the piece's columns
  float* stx = sqz + G::BH * kTX;   // a psbar on the rings
  float* stz = stx + G::NPX;
  const int tid = threadIdx.x, lx = 2 * (tid & 31), zr = tid >> 5;
  const int gx = p.x0 + lx, gz = p.z0 + zr;
  const size_t plane = (size_t)p.NX * p.NZ;
  const float* cur = a.cur + shot * plane;
  const size_t xso = (size_t)shot * p.NZ * p.P2, zso = (size_t)shot * p.P2 * p.NX;

  const int* ro = a.rec_off + (size_t)shot * a.ntiles + tile;
  const int e0 = ro[0], e1 = a.resid && a.n >= 1 ? ro[1] : 0;
  const float* rs = a.resid + ((size_t)shot * a.nt + (a.n - 1)) * a.nrec;
  const f2 l1 = p.get(cur, gz, gx);
  const f2 cs = p.get(a.Cs, gz, gx);
  f2 zl[G::KZ], zc[G::KZ], zz[G::KZ], xl = kZero, xc = kZero, xz = kZero, xa = kZero;
  float za[G::KZ];
  int zq[G::KZ];
#pragma unroll
  for (int k = 0; k < G::KZ; ++k) {
    const int hr = p.z0 - hz + halo_row<G>(zr + 8 * k);
    zl[k] = p.get(cur, hr, gx);
    zc[k] = p.get(a.Cs, hr, gx);
    if constexpr (HZ) {
      zq[k] = p.zrow(hr);
      za[k] = p.zco(a.az, hr);
      zz[k] = p.getz(a.zez_in + zso, zq[k], gx);
    }
  }
  const int sr = tid / hx, sc = side_col<G>(tid % hx), sgx = p.x0 - hx + sc;
  bool s0 = false, s1 = false;
  if (tid < G::NXA) {
    xl = p.get(cur, p.z0 + sr, sgx);
    xc = p.get(a.Cs, p.z0 + sr, sgx);
    if constexpr (HX) {
      s0 = p.xin(p.z0 + sr, sgx);
      s1 = kOdd ? p.xin(p.z0 + sr, sgx + 1) : s0;
      xz = p.getx(a.zex_in + xso, p.z0 + sr, sgx, s0, s1);
      xa = p.xco(a.ax, sgx);
    }
  }
  const int rr = tid >> 2, rc = (tid & 3) < 2 ? 2 * (tid & 3) - 4 : kTX + 2 * (tid & 3) - 4;
  const int rz = zr < 4 ? zr - 4 : zr + 4;
  bool q0 = false, q1 = false, h0 = false, h1 = false;
  f2 px, ex, axv, bxv, pxh, axh;
  if constexpr (HX) {
    q0 = p.xin(gz, gx);
    q1 = kOdd ? p.xin(gz, gx + 1) : q0;
    axv = p.xco(a.ax, gx);
    bxv = p.xco(a.bx, gx);
    px = p.getx(a.psx_in + xso, gz, gx, q0, q1);
    ex = p.getx(a.zex_in + xso, gz, gx, q0, q1);
    if (tid < 4 * kGZ) {
      h0 = p.xin(p.z0 + rr, p.x0 + rc);
      h1 = kOdd ? p.xin(p.z0 + rr, p.x0 + rc + 1) : h0;
      axh = p.xco(a.ax, p.x0 + rc);
      pxh = p.getx(a.psx_in + xso, p.z0 + rr, p.x0 + rc, h0, h1);
    }
  }
  int row = -1, rowh = -1;
  f2 pz, ez, pzh;
  float az = 0.0f, bz = 0.0f, azh = 0.0f;
  if constexpr (HZ) {
    row = p.zrow(gz);
    rowh = p.zrow(p.z0 + rz);
    az = p.zco(a.az, gz);
    bz = p.zco(a.bz, gz);
    azh = p.zco(a.az, p.z0 + rz);
    pz = p.getz(a.psz_in + zso, row, gx);
    ez = p.getz(a.zez_in + zso, row, gx);
    pzh = p.getz(a.psz_in + zso, rowh, gx);
  }
  const f2 l2 = p.get(a.prev + shot * plane, gz, gx);
  const f2 bb = p.get(a.B_in + shot * plane, gz, gx);
  f2 gg = kZero;
  if (!a.g_init) gg = p.get(a.g + shot * plane, gz, gx);
  int2 en = make_int2(0, 0);
  if (e0 + tid < e1) en = a.rec_ent[e0 + tid];

  // Qbar = q + a zbar, zbar = Z + q (q = Cs lambda) where the axis has a strip
  f2 qx = cs * l1, qz = qx;
  if constexpr (HX) {
    const f2 zbar = ex + qx;
    p.setx(a.zex_out + xso, gz, gx, q0, q1, bxv * zbar);
    qx = p.sel(q0, q1, qx + axv * zbar, qx);
  }
  if constexpr (HZ) {
    const f2 zbar = ez + qz;
    p.setz(a.zez_out + zso, row, gx, bz * zbar);
    qz = p.sel(row >= 0, row >= 0, qz + az * zbar, qz);
  }
  put2(&sqx[zr * BW + hx + lx], qx);
  put2(&sqz[(zr + hz) * kTX + lx], qz);
#pragma unroll
  for (int k = 0; k < G::KZ; ++k) {
    f2 v = zc[k] * zl[k];
    if constexpr (HZ) v = p.sel(zq[k] >= 0, zq[k] >= 0, v + za[k] * (zz[k] + v), v);
    put2(&sqz[halo_row<G>(zr + 8 * k) * kTX + lx], v);
  }
  if (tid < G::NXA) {
    f2 v = xc * xl;
    if constexpr (HX) v = p.sel(s0, s1, v + xa * (xz + v), v);
    put2(&sqx[sr * BW + sc], v);
  }
  __syncthreads();

  f2 out = 2.0f * l1 - l2;
  {
    const XWin xw(&sqx[zr * BW + hx + lx], qx);
    out = out + xw.d2();
    if constexpr (HX) {
      const f2 psb = px - xw.d1();
      p.setx(a.psx_out + xso, gz, gx, q0, q1, bxv * psb);
      px = p.sel(q0, q1, axv * psb);
      put2(&stx[zr * XW + 4 + lx], px);
      if (tid < 4 * kGZ) {
        const float* hat = &sqx[rr * BW + hx + rc];
        const f2 ph = pxh - XWin(hat, lds2(hat)).d1();
        put2(&stx[rr * XW + 4 + rc], p.sel(h0, h1, axh * ph));
      }
    }
  }
  {
    const ZWin zw(&sqz[(zr + hz) * kTX + lx], kTX);
    out = out + zw.d2();
    if constexpr (HZ) {
      const f2 psb = pz - zw.d1();
      p.setz(a.psz_out + zso, row, gx, bz * psb);
      put2(&stz[(zr + 4) * kTX + lx], p.sel(row >= 0, row >= 0, az * psb));
      const f2 ph = pzh - ZWin(&sqz[(rz + hz) * kTX + lx], kTX).d1();
      put2(&stz[(rz + 4) * kTX + lx], p.sel(rowh >= 0, rowh >= 0, azh * ph));
    }
  }
  if constexpr (HX || HZ) __syncthreads();
  if constexpr (HX) out = out - XWin(&stx[zr * XW + 4 + lx], px).d1();
  if constexpr (HZ) out = out - ZWin(&stz[(zr + 4) * kTX + lx], kTX).d1();
  const f2 gb = l1 * bb;
  p.set(a.g + shot * plane, gz, gx, a.g_init ? gb : gg + gb);
  if (e1 > e0) {  // r_{n-1} at this piece's receivers; a cell's first entry adds all of them
    if constexpr (!(HX || HZ)) __syncthreads();  // sqx and sqz are read until here
    put2(&sqz[zr * kTX + lx], out);
    __syncthreads();
    for (int e = e0 + tid; e < e1; e += kThreads) {
      if (e >= e0 + kThreads) en = a.rec_ent[e];
      const int r = (en.x >> 6) - row0;
      if (r < 0 || r >= kGZ || (e > e0 && a.rec_ent[e - 1].x == en.x)) continue;
      float acc = sqz[en.x - row0 * kTX];
      acc += rs[en.y];
      for (int k = e + 1; k < e1 && a.rec_ent[k].x == en.x; ++k) acc += rs[a.rec_ent[k].y];
      sqz[en.x - row0 * kTX] = acc;
    }
    __syncthreads();
    out = lds2(&sqz[zr * kTX + lx]);
  }
  p.set(a.next + shot * plane, gz, gx, out);
}

// The piece at columns x0, rows z0 of a shot: row0 its first row in the tile.
template <GridStep kKind, bool kOdd>
__device__ __forceinline__ void piece(const AcStep& a, int shot, int tile, int x0, int z0,
                                      int row0, float* lds) {
  Piece<kOdd> p;
  p.NX = a.NX;
  p.NZ = a.NZ;
  p.P = a.P;
  p.P2 = 2 * a.P;
  p.x0 = x0;
  p.z0 = z0;
  if (p.z0 >= p.NZ) return;
  const bool hx = p.P > 0 && (p.x0 - 4 < p.P || p.x0 + kTX + 4 > p.NX - p.P);
  const bool hz = p.P > 0 && (p.z0 - 4 < p.P || p.z0 + kGZ + 4 > p.NZ - p.P);
#define SWEEP_PIECE(HX, HZ)                                                           \
  do {                                                                                \
    if constexpr (kKind == kGridAdj)                                                  \
      grid_adj<HX, HZ>(a, p, shot, tile, row0, lds);                           \
    else                                                                              \
      grid_fwd<HX, HZ, kKind == kGridBorn, kKind == kGridEncoded>(a, p, shot, tile, \
                                                                  row0, lds);  \
  } while (0)
  if (hx && hz)
    SWEEP_PIECE(true, true);
  else if (hx)
    SWEEP_PIECE(true, false);
  else if (hz)
    SWEEP_PIECE(false, true);
  else
    SWEEP_PIECE(false, false);
#undef SWEEP_PIECE
}

}  // namespace two
}  // namespace sweep
