// Acoustic steps over the whole padded grid in one launch, in items of four
// columns (the recurrence of acoustic.hip with the same operations in the same
// order, so the same bits). us a step on 1080 x 380 cells, forward and adjoint: 32
// shots 42 and 74 against 65 and 95 by tile sets (64 shots in two groups: 84 and
// 149 against 122 and 175), 1 shot 5.5 and 6.7 against 6.5 and 7.6 in items of two
// columns.
//
// A work-group takes a piece of 64 columns x 16 rows, a thread four columns of a
// row: every field is one 16-byte access a thread, the differences along x are
// shared between the four cells, and those along z read 16 bytes of LDS a row.
// Every thread stages its own cells; the halo rows are one item a thread (half of
// the threads away from a z strip) and the side columns are left to one wave.
// Where NX and P are multiples of 4, an item is inside the grid, and inside a strip,
// as a whole. Other sizes take two-column items (acoustic_two.h) in the pieces near
// an x strip or the right edge and four-column ones, at any 4-byte address, in the
// others: 459 x 245 cells, 11 shots, 13.0 and 17.6 us a step (456 cells across: 9.0
// and 12.9; by tile sets 23.8 and 29.8). Calls with thousands of two-column pieces,
// which keep a full GPU busier than the tile sets do, go by those (api.hip).
//
// The fields are read and written without the non-temporal hint: those of a few
// dozen shots stay in the last-level cache from step to step. B' and the gradient
// partials are used once a step and carry it in the four-column pieces; the
// two-column ones read and write them plainly.
#include <algorithm>

#include "acoustic_two.h"
#include "fd.h"
#include "internal.h"

namespace sweep {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
// rows start at any 4-byte address where NX is not a multiple of 4
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr f4 kZ4 = {0.0f, 0.0f, 0.0f, 0.0f};
constexpr int kWZ = 16;  // rows of a piece
static_assert(kThreads == kWZ * kTX / 4, "four cells per thread");

// Four floats at element i of a work-group-uniform base (32-bit byte offset, as
// u32at), plain and with the non-temporal hint.
__device__ __forceinline__ const f4u* at4(const float* f, unsigned i) {
  return reinterpret_cast<const f4u*>(reinterpret_cast<const char*>(f) + i * 4u);
}
__device__ __forceinline__ f4u* at4(float* f, unsigned i) {
  return reinterpret_cast<f4u*>(reinterpret_cast<char*>(f) + i * 4u);
}
__device__ __forceinline__ f4 lds4(const float* s) { return *reinterpret_cast<const f4*>(s); }
__device__ __forceinline__ void put4(float* s, f4 v) { *reinterpret_cast<f4*>(s) = v; }
__device__ __forceinline__ f4 fma4(f4 a, f4 b, f4 c) {
  return f4{fmaf(a.x, b.x, c.x), fmaf(a.y, b.y, c.y), fmaf(a.z, b.z, c.z), fmaf(a.w, b.w, c.w)};
}
__device__ __forceinline__ f4 fma4(float a, f4 b, f4 c) { return fma4(f4{a, a, a, a}, b, c); }
__device__ __forceinline__ f4 sel(bool ok, f4 v, f4 u = kZ4) {
  return f4{ok ? v.x : u.x, ok ? v.y : u.y, ok ? v.z : u.z, ok ? v.w : u.w};
}

// The four cells c of an LDS row (at their address) and the four on either side:
// D2' and D1' along x, the operations of d2c and d1c.
struct XWin {
  float w[12];
  __device__ __forceinline__ XWin(const float* at, f4 c) {
    const f4 l = lds4(at - 4), r = lds4(at + 4);
    const float v[12] = {l.x, l.y, l.z, l.w, c.x, c.y, c.z, c.w, r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 12; ++i) w[i] = v[i];
  }
  // f_{i-k} - f_i is the exact negative of the difference formed at i - k, so
  // adding it is subtracting that one
  __device__ __forceinline__ f4 d2() const {
    f4 s;
#pragma unroll
    for (int k = 1; k <= 4; ++k) {
      const float ak = k == 1 ? kA1 : k == 2 ? kA2 : k == 3 ? kA3 : kA4;
      float e[8];
#pragma unroll
      for (int i = 0; i < 4 + k; ++i) e[i] = w[4 + i] - w[4 + i - k];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float d = e[j + k] - e[j];
        s[j] = k == 1 ? ak * d : fmaf(ak, d, s[j]);
      }
    }
    return s;
  }
  __device__ __forceinline__ f4 d1() const {
    f4 s;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      s[j] = d1c(w[5 + j], w[3 + j], w[6 + j], w[2 + j], w[7 + j], w[1 + j], w[8 + j], w[j]);
    return s;
  }
};

// D2' and D1' along z of the cells c of an LDS column group (rows st floats
// apart).
__device__ __forceinline__ void zboth(const float* at, int st, f4 c, f4& d2, f4& d1) {
#pragma unroll
  for (int k = 1; k <= 4; ++k) {
    const float ak = k == 1 ? kA1 : k == 2 ? kA2 : k == 3 ? kA3 : kA4;
    const float bk = k == 1 ? kB1 : k == 2 ? kB2 : k == 3 ? kB3 : kB4;
    const f4 p = lds4(at + k * st), m = lds4(at - k * st);
    const f4 s = (p - c) + (m - c), d = p - m;
    d2 = k == 1 ? ak * s : fma4(ak, s, d2);
    d1 = k == 1 ? bk * d : fma4(bk, d, d1);
  }
}
__device__ __forceinline__ f4 zd2(const float* at, int st, f4 c) {
  f4 a, b;
  zboth(at, st, c, a, b);
  return a;
}
__device__ __forceinline__ f4 zd1(const float* at, int st) {
  f4 a, b;
  zboth(at, st, kZ4, a, b);
  return b;
}

// One piece of one shot: rows z0 .. z0+15, columns x0 .. x0+63. kFull: the piece
// and 4 cells around it lie inside the grid. Guarded loads come from a valid
// address and are selected afterwards (no branch).
template <bool kFull>
struct Piece {
  int NX, NZ, P, P2, x0, z0;
  __device__ __forceinline__ bool in(int z, int x) const {
    return (unsigned)z < (unsigned)NZ && (unsigned)x < (unsigned)NX;
  }
  __device__ __forceinline__ f4 get(const float* f, int z, int x) const {
    if (kFull) return *at4(f, (unsigned)(z * NX + x));
    const bool ok = in(z, x);
    return sel(ok, *at4(f, ok ? (unsigned)(z * NX + x) : 0u));
  }
  __device__ __forceinline__ f4 get_nt(const float* f, int z, int x) const {
    return __builtin_nontemporal_load(at4(f, kFull || in(z, x) ? (unsigned)(z * NX + x) : 0u));
  }
  __device__ __forceinline__ void set(float* f, int z, int x, f4 v) const {
    if (kFull || in(z, x)) *at4(f, (unsigned)(z * NX + x)) = v;
  }
  __device__ __forceinline__ void set_nt(float* f, int z, int x, f4 v) const {
    if (kFull || in(z, x)) __builtin_nontemporal_store(v, at4(f, (unsigned)(z * NX + x)));
  }
  // x strips: whether columns x .. x+3 of row z are in one; the memory variable
  // there (0 elsewhere)
  __device__ __forceinline__ bool xin(int z, int x) const {
    return in(z, x) && (x < P || x >= NX - P);
  }
  __device__ __forceinline__ unsigned xoff(int z, int x) const {
    return (unsigned)(z * P2 + (x < P ? x : x - (NX - P2)));
  }
  __device__ __forceinline__ f4 getx(const float* m, int z, int x, bool q) const {
    return sel(q, *at4(m, q ? xoff(z, x) : 0u));
  }
  __device__ __forceinline__ void setx(float* m, int z, int x, bool q, f4 v) const {
    if (q) *at4(m, xoff(z, x)) = v;
  }
  // z strips: the strip row of z at columns x .. x+3 (-1: none)
  __device__ __forceinline__ int zrow(int z, int x) const {
    return in(z, x) ? zstrip_row(z, NZ, P) : -1;
  }
  __device__ __forceinline__ f4 getz(const float* m, int row, int x) const {
    return sel(row >= 0, *at4(m, row >= 0 ? (unsigned)(row * NX + x) : 0u));
  }
  __device__ __forceinline__ void setz(float* m, int row, int x, f4 v) const {
    if (row >= 0) *at4(m, (unsigned)(row * NX + x)) = v;
  }
  // C-PML coefficients of columns x .. x+3 and of row z (any value outside)
  __device__ __forceinline__ f4 xco(const float* t, int x) const {
    return *at4(t, (unsigned)x < (unsigned)NX ? (unsigned)x : 0u);
  }
  __device__ __forceinline__ float zco(const float* t, int z) const {
    return u32at(t, (unsigned)min(max(z, 0), NZ - 1));
  }
};

// Staged arrays of a piece with x strips within 4 columns (HX) / z strips within
// 4 rows (HZ): along such an axis the field has a halo of 8 cells (the memory
// variables are formed on a 4-cell ring), else of 4.
template <bool HX, bool HZ>
struct WideGeom {
  static constexpr int hx = HX ? 8 : 4, hz = HZ ? 8 : 4;
  static constexpr int BW = kTX + 2 * hx, BH = kWZ + 2 * hz;
  static constexpr int XW = kTX + 8, ZH = kWZ + 8;
  static constexpr int NPX = HX ? kWZ * XW : 0, NPZ = HZ ? ZH * kTX : 0;
  static constexpr int kFwd = BW * BH + NPX + NPZ;
  static constexpr int kAdj = kWZ * BW + BH * kTX + NPX + NPZ;
  static constexpr int NZH = 2 * hz * (kTX / 4);   // items of the halo rows
  static constexpr int NXH = hx / 2 * kWZ;         // side items of the piece's rows
  static_assert(NZH <= kThreads && NXH <= 64, "one halo item for each thread");
};
constexpr int wide_lds(bool adj) {
  return adj ? WideGeom<true, true>::kAdj : WideGeom<true, true>::kFwd;
}

// A thread's cells and halo items. Halo rows: item tid (box row zb). Side items:
// the last wave (row sr of the piece, box column sc). Rings: the x ring's items
// (4 columns left, 4 right, row rr) belong to threads 128 .. 159, the z ring's
// (row rz of the piece) to threads below 128.
template <class G>
struct Cells {
  int lx, zr, zb, sr, sc, rr, rc, rz;
  bool zh, xh, xr, zring;
  __device__ __forceinline__ Cells() {
    const int tid = threadIdx.x;
    lx = 4 * (tid & 15);
    zr = tid >> 4;
    zh = tid < G::NZH;
    zb = zr < G::hz ? zr : zr + kWZ;
    const int s = tid - 192;
    xh = s >= 0 && s < G::NXH;
    constexpr int n = G::hx / 2;  // side items of a row
    sr = (s & 63) / n;
    const int q = (s & 63) % n;
    sc = q < n / 2 ? 4 * q : kTX + 4 * q;
    xr = tid >= 128 && tid < 128 + 2 * kWZ;
    rr = (tid >> 1) & 15;
    rc = tid & 1 ? kTX : -4;
    zring = tid < 128;
    rz = zr < 4 ? zr - 4 : zr - 4 + kWZ;
  }
};

template <bool HX, bool HZ, bool kFull, bool kBorn, bool kMany>
__device__ __forceinline__ void wide_fwd(const AcStep& a, const Piece<kFull>& p, int shot,
                                         int tile, int row0, float* lds) {
  using G = WideGeom<HX, HZ>;
  constexpr int BW = G::BW, hx = G::hx, hz = G::hz, XW = G::XW;
  float* sb = lds;
  float* spx = lds + BW * G::BH;
  float* spz = spx + G::NPX;
  const Cells<G> c;
  const int tid = threadIdx.x, gx = p.x0 + c.lx, gz = p.z0 + c.zr;
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
      const int q = a.src_cell[shot * a.nsrc + k];
      src = src || (q >= p.z0 * p.NX && q < (p.z0 + kWZ) * p.NX);
    }
  const f4 own = p.get(cur, gz, gx);
  f4 zh = kZ4, xh = kZ4;
  if (G::NZH == kThreads || c.zh) zh = p.get(cur, p.z0 - hz + c.zb, gx);
  if (c.xh) xh = p.get(cur, p.z0 + c.sr, p.x0 - hx + c.sc);
  const f4 pp = p.get(a.prev + shot * plane, gz, gx);
  const f4 cs = p.get(a.Cs, gz, gx);
  f4 bd = kZ4, bb = kZ4;
  if constexpr (kBorn) {
    bd = p.get(a.bdC, gz, gx);
    bb = p.get_nt(a.bB + shot * plane, gz, gx);
  }
  bool q = false, h = false;
  f4 px, ex, axv, bxv, pxh = kZ4, axh = kZ4, bxh = kZ4;
  if constexpr (HX) {
    q = p.xin(gz, gx);
    px = p.getx(a.psx_in + xso, gz, gx, q);
    axv = p.xco(a.ax, gx);
    bxv = p.xco(a.bx, gx);
    if (c.xr) {
      h = p.xin(p.z0 + c.rr, p.x0 + c.rc);
      pxh = p.getx(a.psx_in + xso, p.z0 + c.rr, p.x0 + c.rc, h);
      axh = p.xco(a.ax, p.x0 + c.rc);
      bxh = p.xco(a.bx, p.x0 + c.rc);
    }
  }
  int row = -1, rowh = -1;
  f4 pz, ez, pzh = kZ4;
  float az = 0.0f, bz = 0.0f, azh = 0.0f, bzh = 0.0f;
  if constexpr (HZ) {
    row = p.zrow(gz, gx);
    pz = p.getz(a.psz_in + zso, row, gx);
    az = p.zco(a.az, gz);
    bz = p.zco(a.bz, gz);
    if (c.zring) {
      rowh = p.zrow(p.z0 + c.rz, gx);
      pzh = p.getz(a.psz_in + zso, rowh, gx);
      azh = p.zco(a.az, p.z0 + c.rz);
      bzh = p.zco(a.bz, p.z0 + c.rz);
    }
  }

  float* const at = &sb[(c.zr + hz) * BW + hx + c.lx];
  put4(at, own);
  if (G::NZH == kThreads || c.zh) put4(&sb[c.zb * BW + hx + c.lx], zh);
  if (c.xh) put4(&sb[(c.sr + hz) * BW + c.sc], xh);
  __syncthreads();
  // needed after the second barrier only: in flight over the first derivatives
  if constexpr (HX) ex = p.getx(a.zex_in + xso, gz, gx, q);
  if constexpr (HZ) ez = p.getz(a.zez_in + zso, row, gx);

  f4 Bx, Bz, d1;
  {
    const XWin xw(at, own);
    Bx = xw.d2();
    if constexpr (HX) {
      // psi_x^n = b psi_x^{n-1} + a D1x' p^n in the strips
      const f4 ps = fma4(axv, xw.d1(), bxv * px);
      p.setx(a.psx_out + xso, gz, gx, q, ps);
      px = sel(q, ps);
      put4(&spx[c.zr * XW + 4 + c.lx], px);
      if (c.xr) {
        const float* hat = &sb[(c.rr + hz) * BW + hx + c.rc];
        const f4 ph = fma4(axh, XWin(hat, lds4(hat)).d1(), bxh * pxh);
        put4(&spx[c.rr * XW + 4 + c.rc], sel(h, ph));
      }
    }
  }
  zboth(at, BW, own, Bz, d1);
  if constexpr (HZ) {
    const f4 ps = fma4(az, d1, bz * pz);
    p.setz(a.psz_out + zso, row, gx, ps);
    put4(&spz[(c.zr + 4) * kTX + c.lx], sel(row >= 0, ps));
    if (c.zring) {
      const f4 ph = fma4(azh, zd1(&sb[(c.rz + hz) * BW + hx + c.lx], BW), bzh * pzh);
      put4(&spz[(c.rz + 4) * kTX + c.lx], sel(rowh >= 0, ph));
    }
  }
  if constexpr (HX || HZ) __syncthreads();
  if constexpr (HX) {
    Bx = Bx + XWin(&spx[c.zr * XW + 4 + c.lx], px).d1();
    const f4 ze = fma4(axv, Bx, bxv * ex);
    p.setx(a.zex_out + xso, gz, gx, q, ze);
    Bx = sel(q, Bx + ze, Bx);
  }
  if constexpr (HZ) {
    Bz = Bz + zd1(&spz[(c.zr + 4) * kTX + c.lx], kTX);
    const f4 ze = fma4(az, Bz, bz * ez);
    p.setz(a.zez_out + zso, row, gx, ze);
    Bz = sel(row >= 0, Bz + ze, Bz);
  }
  const f4 B = Bx + Bz;
  f4 out = fma4(cs, B, 2.0f * own - pp);
  if constexpr (kBorn) out = out + bd * bb;
  if constexpr (kMany)
    each_source(a, shot, lsrc, (p.z0 + (c.zr & ~3)) * p.NX, 4 * p.NX, [&](int cell, float sw) {
      const int d = cell - (gz * p.NX + gx);
      if ((unsigned)d < 4u && gx < p.NX) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (d == j) out[j] += sw;
      }
    });
  if (src)
    for (int k = 0; k < a.nsrc; ++k) {
      const int d = a.src_cell[shot * a.nsrc + k] - (gz * p.NX + gx);
      const float sw = a.w * a.wavelet[((size_t)shot * a.nsrc + k) * a.nt + a.n];
      if ((unsigned)d < 4u && gx < p.NX) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (d == j) out[j] += sw;
      }
    }
  p.set(a.next + shot * plane, gz, gx, out);
  if (a.B_out) p.set_nt(a.B_out + shot * plane, gz, gx, B);
  if (e1 > e0) {  // the receivers of the tile in this piece's rows
    __syncthreads();  // sb is read until here
    put4(&sb[c.zr * kTX + c.lx], out);
    __syncthreads();
    float* dst = a.gathers + ((size_t)shot * a.nt + a.n) * a.nrec;
    for (int e = e0 + tid; e < e1; e += kThreads) {
      const int2 en = a.rec_ent[e];
      const int r = (en.x >> 6) - row0;
      if (r >= 0 && r < kWZ) dst[en.y] = sb[en.x - row0 * kTX];
    }
  }
}

template <bool HX, bool HZ, bool kFull>
__device__ __forceinline__ void wide_adj(const AcStep& a, const Piece<kFull>& p, int shot,
                                         int tile, int row0, float* lds) {
  using G = WideGeom<HX, HZ>;
  constexpr int BW = G::BW, hx = G::hx, hz = G::hz, XW = G::XW;
  float* sqx = lds;                 // Qbar_x: the piece's rows, columns x0-hx ..
  float* sqz = lds + kWZ * BW;      // Qbar_z: rows z0-hz .., the piece's columns
  float* stx = sqz + G::BH * kTX;   // a psbar on the rings
  float* stz = stx + G::NPX;
  const Cells<G> c;
  const int tid = threadIdx.x, gx = p.x0 + c.lx, gz = p.z0 + c.zr;
  const size_t plane = (size_t)p.NX * p.NZ;
  const float* cur = a.cur + shot * plane;
  const size_t xso = (size_t)shot * p.NZ * p.P2, zso = (size_t)shot * p.P2 * p.NX;

  const int* ro = a.rec_off + (size_t)shot * a.ntiles + tile;
  const int e0 = ro[0], e1 = a.resid && a.n >= 1 ? ro[1] : 0;
  const f4 l1 = p.get(cur, gz, gx);
  const f4 cs = p.get(a.Cs, gz, gx);
  // halo rows and side columns: lambda, Cs, Z
  f4 zl = kZ4, zc = kZ4, zz = kZ4, xl = kZ4, xc = kZ4, xz = kZ4, xa = kZ4;
  float za = 0.0f;
  int zq = -1;
  bool s = false;
  if (G::NZH == kThreads || c.zh) {
    const int hr = p.z0 - hz + c.zb;
    zl = p.get(cur, hr, gx);
    zc = p.get(a.Cs, hr, gx);
    if constexpr (HZ) {
      zq = p.zrow(hr, gx);
      zz = p.getz(a.zez_in + zso, zq, gx);
      za = p.zco(a.az, hr);
    }
  }
  if (c.xh) {
    const int sx = p.x0 - hx + c.sc;
    xl = p.get(cur, p.z0 + c.sr, sx);
    xc = p.get(a.Cs, p.z0 + c.sr, sx);
    if constexpr (HX) {
      s = p.xin(p.z0 + c.sr, sx);
      xz = p.getx(a.zex_in + xso, p.z0 + c.sr, sx, s);
      xa = p.xco(a.ax, sx);
    }
  }
  bool q = false, h = false;
  f4 px, ex, axv, bxv, pxh = kZ4, axh = kZ4;
  if constexpr (HX) {
    q = p.xin(gz, gx);
    px = p.getx(a.psx_in + xso, gz, gx, q);
    ex = p.getx(a.zex_in + xso, gz, gx, q);
    axv = p.xco(a.ax, gx);
    bxv = p.xco(a.bx, gx);
    if (c.xr) {
      h = p.xin(p.z0 + c.rr, p.x0 + c.rc);
      pxh = p.getx(a.psx_in + xso, p.z0 + c.rr, p.x0 + c.rc, h);
      axh = p.xco(a.ax, p.x0 + c.rc);
    }
  }
  int row = -1, rowh = -1;
  f4 pz, ez, pzh = kZ4;
  float az = 0.0f, bz = 0.0f, azh = 0.0f;
  if constexpr (HZ) {
    row = p.zrow(gz, gx);
    pz = p.getz(a.psz_in + zso, row, gx);
    ez = p.getz(a.zez_in + zso, row, gx);
    az = p.zco(a.az, gz);
    bz = p.zco(a.bz, gz);
    if (c.zring) {
      rowh = p.zrow(p.z0 + c.rz, gx);
      pzh = p.getz(a.psz_in + zso, rowh, gx);
      azh = p.zco(a.az, p.z0 + c.rz);
    }
  }
  const f4 l2 = p.get(a.prev + shot * plane, gz, gx);
  const f4 bb = p.get_nt(a.B_in + shot * plane, gz, gx);
  f4 gg = kZ4;
  if (!a.g_init) gg = p.get_nt(a.g + shot * plane, gz, gx);

  // Qbar = q + a zbar, zbar = Z + q (q = Cs lambda) where the axis has a strip
  f4 qx = cs * l1, qz = qx;
  if constexpr (HX) {
    const f4 zbar = ex + qx;
    p.setx(a.zex_out + xso, gz, gx, q, bxv * zbar);
    qx = sel(q, qx + axv * zbar, qx);
  }
  if constexpr (HZ) {
    const f4 zbar = ez + qz;
    p.setz(a.zez_out + zso, row, gx, bz * zbar);
    qz = sel(row >= 0, qz + az * zbar, qz);
  }
  float* const atx = &sqx[c.zr * BW + hx + c.lx];
  float* const atz = &sqz[(c.zr + hz) * kTX + c.lx];
  put4(atx, qx);
  put4(atz, qz);
  if (G::NZH == kThreads || c.zh) {
    f4 v = zc * zl;
    if constexpr (HZ) v = sel(zq >= 0, v + za * (zz + v), v);
    put4(&sqz[c.zb * kTX + c.lx], v);
  }
  if (c.xh) {
    f4 v = xc * xl;
    if constexpr (HX) v = sel(s, v + xa * (xz + v), v);
    put4(&sqx[c.sr * BW + c.sc], v);
  }
  __syncthreads();

  f4 out = 2.0f * l1 - l2;
  {
    const XWin xw(atx, qx);
    out = out + xw.d2();
    if constexpr (HX) {
      const f4 psb = px - xw.d1();
      p.setx(a.psx_out + xso, gz, gx, q, bxv * psb);
      px = sel(q, axv * psb);
      put4(&stx[c.zr * XW + 4 + c.lx], px);
      if (c.xr) {
        const float* hat = &sqx[c.rr * BW + hx + c.rc];
        const f4 ph = pxh - XWin(hat, lds4(hat)).d1();
        put4(&stx[c.rr * XW + 4 + c.rc], sel(h, axh * ph));
      }
    }
  }
  f4 d2, d1;
  zboth(atz, kTX, qz, d2, d1);
  out = out + d2;
  if constexpr (HZ) {
    const f4 psb = pz - d1;
    p.setz(a.psz_out + zso, row, gx, bz * psb);
    put4(&stz[(c.zr + 4) * kTX + c.lx], sel(row >= 0, az * psb));
    if (c.zring) {
      const f4 ph = pzh - zd1(&sqz[(c.rz + hz) * kTX + c.lx], kTX);
      put4(&stz[(c.rz + 4) * kTX + c.lx], sel(rowh >= 0, azh * ph));
    }
  }
  if constexpr (HX || HZ) __syncthreads();
  if constexpr (HX) out = out - XWin(&stx[c.zr * XW + 4 + c.lx], px).d1();
  if constexpr (HZ) out = out - zd1(&stz[(c.zr + 4) * kTX + c.lx], kTX);
  const f4 gb = l1 * bb;
  p.set_nt(a.g + shot * plane, gz, gx, a.g_init ? gb : gg + gb);
  if (e1 > e0) {  // r_{n-1} at this piece's receivers; a cell's first entry adds all of them
    const float* rs = a.resid + ((size_t)shot * a.nt + (a.n - 1)) * a.nrec;
    __syncthreads();  // sqx and sqz are read until here
    put4(&sqz[c.zr * kTX + c.lx], out);
    __syncthreads();
    for (int e = e0 + tid; e < e1; e += kThreads) {
      const int2 en = a.rec_ent[e];
      const int r = (en.x >> 6) - row0;
      if (r < 0 || r >= kWZ || (e > e0 && a.rec_ent[e - 1].x == en.x)) continue;
      float acc = sqz[en.x - row0 * kTX];
      acc += rs[en.y];
      for (int k = e + 1; k < e1 && a.rec_ent[k].x == en.x; ++k) acc += rs[a.rec_ent[k].y];
      sqz[en.x - row0 * kTX] = acc;
    }
    __syncthreads();
    out = lds4(&sqz[c.zr * kTX + c.lx]);
  }
  p.set(a.next + shot * plane, gz, gx, out);
}

// Tile columns [c0, c1) whose cells are all more than 4 cells from an x strip and
// from the grid's edge.
__host__ __device__ inline void free_columns(int NX, int P, int tiles_x, int& c0, int& c1) {
  const int lo = P > 0 ? P + 4 : 4, hi = NX - lo;  // columns [lo, hi) are free of both
  c0 = (lo + kTX - 1) / kTX;
  c1 = hi / kTX;
  // a few such columns are not worth the taller pieces, which a small grid waits
  // for (170 x 97 cells, 3 shots: 1 column of 3, 6 % slower a gradient)
  if (2 * (c1 - c0) < tiles_x) c0 = c1 = 0;
}

// Pieces of a shot: tile columns [c0, c1) take 64 x 16 pieces of four-column
// items, the others (none where NX and P are multiples of 4) 64 x 8 pieces of
// two-column ones.
struct Pieces {
  int c0, c1, tiles_x, rows;  // rows: 16-row pieces along z
  __host__ __device__ Pieces(const AcStep& a, bool aligned) {
    tiles_x = a.tiles_x;
    rows = a.ntiles / tiles_x * (a.tz / kWZ);
    c0 = 0;
    c1 = tiles_x;
    if (!aligned) free_columns(a.NX, a.P, tiles_x, c0, c1);
  }
  __host__ __device__ int four() const { return rows * (c1 - c0); }
  __host__ __device__ int blocks() const { return four() + 2 * rows * (tiles_x - (c1 - c0)); }
};

template <GridStep kKind, int kUnit>
__device__ __forceinline__ void wide_piece(const AcStep& a, int l, float* lds) {
  const Pieces n(a, kUnit == 4);
  const int per = n.blocks(), shot = l / per, t = l - shot * per, four = n.four();
  const int NX = a.NX, NZ = a.NZ, P = a.P;
  if (kUnit != 4 && t >= four) {
    const int w = n.tiles_x - (n.c1 - n.c0), u = t - four, row = u / w, c = u - row * w;
    const int col = c < n.c0 ? c : c + (n.c1 - n.c0), z = row * two::kGZ, tz = z / a.tz;
    two::piece<kKind, kUnit == 1>(a, shot, tz * n.tiles_x + col, col * kTX, z, z - tz * a.tz, lds);
    return;
  }
  const int w = n.c1 - n.c0, row = t / w, col = n.c0 + t - row * w;
  const int x0 = col * kTX, z0 = row * kWZ, tz = z0 / a.tz;
  const int tile = tz * n.tiles_x + col, row0 = z0 - tz * a.tz;
  if (z0 >= NZ) return;
  const bool hx = kUnit == 4 && P > 0 && (x0 - 4 < P || x0 + kTX + 4 > NX - P);
  const bool hz = P > 0 && (z0 - 4 < P || z0 + kWZ + 4 > NZ - P);
  const bool full = x0 >= 4 && x0 + kTX + 4 <= NX && z0 >= 4 && z0 + kWZ + 4 <= NZ;
#define SWEEP_PIECE(HX, HZ, FULL)                                               \
  do {                                                                          \
    const Piece<FULL> p{NX, NZ, P, 2 * P, x0, z0};                              \
    if constexpr (kKind == kGridAdj)                                            \
      wide_adj<HX, HZ, FULL>(a, p, shot, tile, row0, lds);                      \
    else                                                                        \
      wide_fwd<HX, HZ, FULL, kKind == kGridBorn, kKind == kGridEncoded>(        \
          a, p, shot, tile, row0, lds);                                         \
  } while (0)
  if constexpr (kUnit == 4) {
    if (hx && hz) {
      SWEEP_PIECE(true, true, false);
      return;
    }
    if (hx) {
      SWEEP_PIECE(true, false, false);
      return;
    }
  }
  if (hz)
    SWEEP_PIECE(false, true, false);
  else if (full)
    SWEEP_PIECE(false, false, true);
  else
    SWEEP_PIECE(false, false, false);
#undef SWEEP_PIECE
}

constexpr int lds_floats(GridStep kind, bool aligned) {
  const int w = wide_lds(kind == kGridAdj), t = two::grid_lds(kind == kGridAdj);
  return aligned || w > t ? w : t;
}

// The corner pieces set the registers: 124 forward and 112 in reverse, 4 waves a
// SIMD (127 with encoded shots), and 131 in a Born step, 3 waves. Held to 96 for 5 waves, forward and reverse
// spill and 32 shots take 50 and 78 us.
template <GridStep kKind, int kUnit>
__global__ __launch_bounds__(kThreads) void ac_wide_kernel(AcStep a) {
  __shared__ __attribute__((aligned(16))) float lds[lds_floats(kKind, kUnit == 4)];
  wide_piece<kKind, kUnit>(a, xcd_spread(blockIdx.x, gridDim.x), lds);
}

// Several plans in one launch (AcBatch); the least aligned one chooses the code.
template <GridStep kKind, int kUnit>
__global__ __launch_bounds__(kThreads) void ac_wide_batch_kernel(AcBatch b) {
  __shared__ __attribute__((aligned(16))) float lds[lds_floats(kKind, kUnit == 4)];
  int f = xcd_spread(blockIdx.x, gridDim.x), q = 0;
  while (q + 1 < b.nplans && f >= b.base[q + 1]) ++q;
  wide_piece<kKind, kUnit>(b.step[q], f - b.base[q], lds);
}

int wide_blocks(const AcStep& a, bool aligned) { return Pieces(a, aligned).blocks() * a.nshots; }

template <int kUnit>
void launch_wide(const AcStep& a, GridStep kind, hipStream_t s) {
  const dim3 g(wide_blocks(a, kUnit == 4)), t(kThreads);
  switch (kind) {
    case kGridFwd: hipLaunchKernelGGL((ac_wide_kernel<kGridFwd, kUnit>), g, t, 0, s, a); break;
    case kGridAdj: hipLaunchKernelGGL((ac_wide_kernel<kGridAdj, kUnit>), g, t, 0, s, a); break;
    case kGridEncoded:
      hipLaunchKernelGGL((ac_wide_kernel<kGridEncoded, kUnit>), g, t, 0, s, a);
      break;
    default: hipLaunchKernelGGL((ac_wide_kernel<kGridBorn, kUnit>), g, t, 0, s, a); break;
  }
}

template <int kUnit>
void launch_wide_batch(const AcBatch& b, GridStep kind, hipStream_t s) {
  const dim3 g(b.base[b.nplans]), t(kThreads);
  if (kind == kGridAdj)
    hipLaunchKernelGGL((ac_wide_batch_kernel<kGridAdj, kUnit>), g, t, 0, s, b);
  else
    hipLaunchKernelGGL((ac_wide_batch_kernel<kGridFwd, kUnit>), g, t, 0, s, b);
}

int check_wide(const AcStep& a, GridStep kind) {
  if (a.tz % kWZ != 0) {
    set_error("one-launch step: the tile height must be a multiple of 16");
    return SWEEP_EINVAL;
  }
  if (a.NX < 2) {
    set_error("one-launch step: the grid must be two columns wide at least");
    return SWEEP_EINVAL;
  }
  if (kind == kGridBorn && (!a.bdC || !a.bB)) {
    set_error("Born step without its perturbation operands");
    return SWEEP_EINVAL;
  }
  return SWEEP_OK;
}

}  // namespace

int ac_wide_unit(int NX, int P) { return (NX | P) & 1 ? 1 : (NX | P) & 2 ? 2 : 4; }

int ac_wide_two(int NX, int NZ, int P) {
  const int tiles_x = (NX + kTX - 1) / kTX;
  int c0, c1;
  free_columns(NX, P, tiles_x, c0, c1);
  return (NZ + two::kGZ - 1) / two::kGZ * (tiles_x - (c1 - c0));
}

int ac_launch_wide(const AcStep& a, GridStep kind, hipStream_t s) {
  const int rc = check_wide(a, kind);
  if (rc) return rc;
  if (kind == kGridFwd && a.nsrc > 1) kind = kGridEncoded;
  switch (ac_wide_unit(a.NX, a.P)) {
    case 4: launch_wide<4>(a, kind, s); break;
    case 2: launch_wide<2>(a, kind, s); break;
    default: launch_wide<1>(a, kind, s);
  }
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

int ac_launch_wide_batch(const AcStep* steps, int n, GridStep kind, hipStream_t s) {
  AcBatch b;
  for (int q = 0; q < n;) {
    b.nplans = 0;
    b.base[0] = 0;
    const int q0 = q;
    int unit = 4;
    for (; q < n && b.nplans < kPlansPerLaunch; ++q) {
      const int rc = check_wide(steps[q], kind);
      if (rc) return rc;
      b.step[b.nplans++] = steps[q];
      unit = std::min(unit, ac_wide_unit(steps[q].NX, steps[q].P));
    }
    for (int k = 0; k < b.nplans; ++k)
      b.base[k + 1] = b.base[k] + wide_blocks(steps[q0 + k], unit == 4);
    switch (unit) {
      case 4: launch_wide_batch<4>(b, kind, s); break;
      case 2: launch_wide_batch<2>(b, kind, s); break;
      default: launch_wide_batch<1>(b, kind, s);
    }
  }
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

}  // namespace sweep
