// Elastic step kernels for gfx950: the isotropic velocity-stress system
// (Sec. 3.5, Eq. 12) on a staggered grid, 4th order in space, with C-PML and an
// optional free surface, and the exact transpose of that recurrence.
//
// Nodes of the values stored at [j][i]: txx, tzz at (i, j); vx at (i+1/2, j);
// vz at (i, j+1/2); txz at (i+1/2, j+1/2). Derivatives (c1 = 9/8, c2 = -1/24):
//   Dx+ f = c1 (f[i+1]-f[i]) + c2 (f[i+2]-f[i-1])    integer -> half
//   Dx- g = c1 (g[i]-g[i-1]) + c2 (g[i+1]-g[i-2])    half -> integer
// zero outside the grid; along z at a free surface the stress images
// tzz[-k] = -tzz[k], txz[-k-1] = -txz[k] are folded into the first rows and the
// velocity z-derivatives that would reach above the surface fall back to the
// 2nd-order difference. Each of the eight derivatives carries a C-PML memory
// variable psi <- b psi + a D f, stored over the whole grid but touched only
// where a != 0.
//
// Forward step: velocity kernel (vx, vz), stress kernel (txx, tzz, txz,
// explosive source; it also gathers the receivers). Every step kernel has a fluid variant
// (kFluid, the first-order acoustic system at vs = 0): there mu = 0, so txz
// stays 0, and the shear stress, its four memory variables and the mu
// partials of the adjoint enter only through products with 0. The variant
// drops them; every other value is formed by the same operations, so it gives
// the elastic kernels' results at vs = 0 while moving about a fifth fewer
// bytes forward and a quarter fewer in reverse. Reverse step (gather form of the
// transpose): adjoint-stress kernel (updates the velocity adjoints from the
// stress adjoints and injects the residuals), adjoint-velocity kernel. Away from the
// surface the transposes are (Dx+)^T = -Dx-, (Dx-)^T = -Dx+ (and along z); on the
// first four rows below a free surface they use tap tables derived on the host
// from the forward taps.
#include "elastic.h"
#include "finish.h"

namespace sweep {
namespace {

constexpr float C1 = 9.0f / 8.0f;
constexpr float C2 = -1.0f / 24.0f;

// ---------------------------------------------------------------------------
// Tiles: 64 columns x 16 rows per work-group; thread t owns the four columns
// 4 (t & 15) .. + 3 of row t / 16, so a field is one 16-byte access a thread and
// a wave covers four rows. What a kernel differentiates is staged in LDS, zero
// outside the grid: every thread stages its own cells (and keeps them in
// registers), one wave the two rows above and below the tile and another the two
// columns left and right of it. Which waves these are rotates with the
// work-group, so that no SIMD takes all the halos. A plane that is differentiated
// along one axis only has the halo of that axis only.
//
// The steps move 7 to 16 planes per cell and are bound by memory. Forward they
// run near a stream of the same planes; in reverse a work-group's chain (loads,
// LDS, update) leaves part of the bandwidth idle. 16-byte items instead of one
// column a thread halve the memory instructions and the address arithmetic. The
// fields of up to about 200 MB of shots stay in the last-level cache from kernel
// to kernel, so what is used once a step (traces, gradient partials) passes by it
// with the non-temporal hint: on 680 x 380 cells and 32 shots the traced stress
// step takes 56 us with the hint on the traces and 92 us without, the reverse
// stress step 117 us with it on traces and partials and 135 us without. On the
// fields themselves the hint costs 10 to 30 %.
// us a launch on 660 x 330 cells, 32 shots, mean over a gradient that stores half
// of its segments, with one column a thread and no hints -> now: velocity 55 ->
// 43, stress 66 -> 52, reverse stress 136 -> 102, reverse velocity 112 -> 82.
// ---------------------------------------------------------------------------
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
// rows start at any 4-byte address when NX is odd
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr f2 kZ2 = {0.0f, 0.0f};
constexpr f4 kZ4 = {0.0f, 0.0f, 0.0f, 0.0f};
constexpr int kElTZ = kElTileRows;
constexpr int kElXP = kTX + 8;     // row pitch of a plane with an x halo: column c at 4 + c
constexpr int kElZH = kElTZ + 4;   // rows of a plane with a z halo: row r at 2 + r
static_assert(kThreads == kElTZ * kTX / 4, "four cells per thread");

__device__ __forceinline__ f4 ld4(const float* f, unsigned i) {
  return *reinterpret_cast<const f4u*>(reinterpret_cast<const char*>(f) + i * 4u);
}
__device__ __forceinline__ f2 ld2(const float* f, unsigned i) {
  return *reinterpret_cast<const f2u*>(reinterpret_cast<const char*>(f) + i * 4u);
}
__device__ __forceinline__ void st4(float* f, unsigned i, f4 v) {
  *reinterpret_cast<f4u*>(reinterpret_cast<char*>(f) + i * 4u) = v;
}
// the same with the non-temporal hint
__device__ __forceinline__ f4 ld4_nt(const float* f, unsigned i) {
  return __builtin_nontemporal_load(
      reinterpret_cast<const f4u*>(reinterpret_cast<const char*>(f) + i * 4u));
}
__device__ __forceinline__ void st4_nt(float* f, unsigned i, f4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<f4u*>(reinterpret_cast<char*>(f) + i * 4u));
}
__device__ __forceinline__ f4 lds4(const float* s) { return *reinterpret_cast<const f4*>(s); }
__device__ __forceinline__ f2 lds2(const float* s) { return *reinterpret_cast<const f2*>(s); }
__device__ __forceinline__ void put4(float* s, f4 v) { *reinterpret_cast<f4*>(s) = v; }
__device__ __forceinline__ void put2(float* s, f2 v) { *reinterpret_cast<f2*>(s) = v; }
__device__ __forceinline__ float fma_(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ f2 fma_(f2 a, f2 b, f2 c) {
  return f2{fmaf(a.x, b.x, c.x), fmaf(a.y, b.y, c.y)};
}
__device__ __forceinline__ f4 fma_(f4 a, f4 b, f4 c) {
  return f4{fmaf(a.x, b.x, c.x), fmaf(a.y, b.y, c.y), fmaf(a.z, b.z, c.z), fmaf(a.w, b.w, c.w)};
}
__device__ __forceinline__ f4 fma_(float a, f4 b, f4 c) { return fma_(f4{a, a, a, a}, b, c); }
// c != 0 ? a : b, per column
__device__ __forceinline__ float pick(float c, float a, float b) { return c != 0.0f ? a : b; }
__device__ __forceinline__ f2 pick(f2 c, f2 a, f2 b) {
  return f2{pick(c.x, a.x, b.x), pick(c.y, a.y, b.y)};
}
__device__ __forceinline__ f4 pick(f4 c, f4 a, f4 b) {
  return f4{pick(c.x, a.x, b.x), pick(c.y, a.y, b.y), pick(c.z, a.z, b.z), pick(c.w, a.w, b.w)};
}
__device__ __forceinline__ f4 pick(float c, f4 a, f4 b) { return c != 0.0f ? a : b; }

// The two first derivatives along x of a staged row (times h) at the four own
// columns c, whose LDS address is `at`:
// plus  Dx+ f = c1 (f[i+1] - f[i]) + c2 (f[i+2] - f[i-1]), minus Dx- likewise.
struct XWin {
  float w[8];
  __device__ __forceinline__ XWin(const float* at, f4 c) {
    const f2 l = lds2(at - 2), r = lds2(at + 4);
    const float v[8] = {l.x, l.y, c.x, c.y, c.z, c.w, r.x, r.y};
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = v[i];
  }
  __device__ __forceinline__ float d(int i) const {
    return fmaf(C2, w[i + 3] - w[i], C1 * (w[i + 2] - w[i + 1]));
  }
  __device__ __forceinline__ f4 plus() const { return f4{d(1), d(2), d(3), d(4)}; }
  __device__ __forceinline__ f4 minus() const { return f4{d(0), d(1), d(2), d(3)}; }
};
// Rows j-2 .. j+2 of a staged column group (row pitch st), own row c: Dz+, Dz-.
__device__ __forceinline__ f4 zplus(const float* at, int st, f4 c) {
  return fma_(C2, lds4(at + 2 * st) - lds4(at - st), C1 * (lds4(at + st) - c));
}
__device__ __forceinline__ f4 zminus(const float* at, int st, f4 c) {
  const f4 m1 = lds4(at - st);
  return fma_(C2, lds4(at + st) - lds4(at - 2 * st), C1 * (c - m1));
}
// z derivatives with the free-surface rules on rows 0 and 1 (fs: this wave has
// the rows 0..3 under a free surface; j the thread's row)
__device__ __forceinline__ f4 dz_tzz(const float* at, int st, f4 c, bool fs, int j) {
  if (fs && j == 0)  // tzz[-1] = -tzz[1]
    return fma_(C2, lds4(at + 2 * st), fma_(C1 + C2, lds4(at + st), -C1 * c));
  return zplus(at, st, c);
}
__device__ __forceinline__ f4 dz_txz(const float* at, int st, f4 c, bool fs, int j) {
  if (fs && j == 0)  // txz[-1] = -txz[0], txz[-2] = -txz[1]
    return fma_(2.0f * C2, lds4(at + st), 2.0f * C1 * c);
  if (fs && j == 1)  // txz[-1] = -txz[0]
    return fma_(C2, lds4(at + st), fma_(-C1 + C2, lds4(at - st), C1 * c));
  return zminus(at, st, c);
}
__device__ __forceinline__ f4 dz_vx(const float* at, int st, f4 c, bool fs, int j) {
  if (fs && j == 0) return lds4(at + st) - c;
  return zplus(at, st, c);
}
__device__ __forceinline__ f4 dz_vz(const float* at, int st, f4 c, bool fs, int j) {
  if (fs && j == 0) return kZ4;
  if (fs && j == 1) return c - lds4(at - st);
  return zminus(at, st, c);
}

// The tile of this work-group (1-D launch over tiles x shots) and this thread's
// cells of it. kCols: what the right edge can cut. 4: NX is a multiple of 4, an
// item of four columns (two in a column halo) is inside or outside as a whole.
// 2: it is not; tiles that lie inside the grid (kFull) move four columns at a time
// all the same, at any 4-byte address, and so do those at the right edge, which
// read the item there from further left and shift it (column by column, these tiles
// set the time of a small launch: velocity, 459 x 245 cells, 11 shots, 16.7 us,
// shifted 9.7). 1: NX < 4, columns one by one. Guarded loads come from a valid
// address and are selected afterwards (no branch).
template <int kCols, bool kFull>
struct Tile {
  int NX, NZ, P, top, x0, z0;
  size_t so;      // first cell of the shot
  int shot;
  int wave, c;    // wave (uniform), first own column in the tile
  int gx, gz, r;  // first own column and row in the grid, row in the tile

  static __device__ __forceinline__ void origin(const ElStep& a, int f, int& x0, int& z0,
                                                int& shot) {
    const int tx = (a.NX + kTX - 1) / kTX, tz = (a.NZ + kElTZ - 1) / kElTZ;
    shot = f / (tx * tz);
    const int t = f - shot * (tx * tz);
    z0 = (t / tx) * kElTZ;
    x0 = (t % tx) * kTX;
  }
  __device__ __forceinline__ Tile(const ElStep& a, int x, int z, int s)
      : NX(a.NX), NZ(a.NZ), P(a.P), top(a.top), x0(x), z0(z), shot(s) {
    so = (size_t)shot * ((size_t)NX * NZ);
    wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    c = (int)(threadIdx.x & 15) * 4;
    r = wave * 4 + ((int)(threadIdx.x & 63) >> 4);
    gx = x0 + c;
    gz = z0 + r;
  }
  __device__ __forceinline__ bool zin(int z) const { return (unsigned)z < (unsigned)NZ; }
  __device__ __forceinline__ bool xin(int x) const { return (unsigned)x < (unsigned)NX; }
  // f at row z, columns x .. x+3 (x within the tile); 0 outside the grid or where !q
  __device__ __forceinline__ f4 get(const float* f, int z, int x, bool q = true) const {
    if (kCols == 4 || kFull) {
      const bool ok = q && zin(z) && (kFull || xin(x));
      const f4 v = ld4(f, ok ? (unsigned)(z * NX + x) : 0u);
      return f4{ok ? v.x : 0.0f, ok ? v.y : 0.0f, ok ? v.z : 0.0f, ok ? v.w : 0.0f};
    }
    if (kCols == 2) {
      const bool ok = q && zin(z) && xin(x);
      const int xs = min(x, NX - 4), sh = ok ? x - xs : 4;
      f4 v = ld4(f, ok ? (unsigned)(z * NX + xs) : 0u);
      if (sh & 1) v = f4{v.y, v.z, v.w, 0.0f};
      if (sh & 2) v = f4{v.z, v.w, 0.0f, 0.0f};
      return sh & 4 ? kZ4 : v;
    }
    const f2 a = part(f, z, x, q), b = part(f, z, x + 2, q);
    return f4{a.x, a.y, b.x, b.y};
  }
  // two columns, of a column halo too
  __device__ __forceinline__ f2 part(const float* f, int z, int x, bool q = true) const {
    if (kCols == 4) {
      const bool ok = q && zin(z) && xin(x);
      const f2 v = ld2(f, ok ? (unsigned)(z * NX + x) : 0u);
      return f2{ok ? v.x : 0.0f, ok ? v.y : 0.0f};
    }
    const bool o0 = q && zin(z) && xin(x), o1 = q && zin(z) && xin(x + 1);
    const float v0 = u32at(f, o0 ? (unsigned)(z * NX + x) : 0u);
    const float v1 = u32at(f, o1 ? (unsigned)(z * NX + x + 1) : 0u);
    return f2{o0 ? v0 : 0.0f, o1 ? v1 : 0.0f};
  }
  __device__ __forceinline__ f4 own(const float* f) const { return get(f, gz, gx); }
  // own cells with the non-temporal hint (no selection: what lies outside the
  // grid is not used); the right edge's parts go without it
  __device__ __forceinline__ f4 own_nt(const float* f) const {
    if (!(kCols == 4 || kFull)) return own(f);
    return ld4_nt(f, zin(gz) && (kFull || xin(gx)) ? (unsigned)(gz * NX + gx) : 0u);
  }
  __device__ __forceinline__ void put_nt(float* f, f4 v) const {
    if (!(kCols == 4 || kFull))
      put(f, v);
    else if (zin(gz) && (kFull || xin(gx)))
      st4_nt(f, (unsigned)(gz * NX + gx), v);
  }
  __device__ __forceinline__ void put(float* f, f4 v) const {
    if (!zin(gz)) return;
    const unsigned k = (unsigned)(gz * NX + gx);
    if (kFull || gx + 4 <= NX) {
      st4(f, k, v);
    } else if (kCols != 4) {
      if (xin(gx)) u32at(f, k) = v.x;
      if (xin(gx + 1)) u32at(f, k + 1) = v.y;
      if (xin(gx + 2)) u32at(f, k + 2) = v.z;
    }
  }
  // a table along x, z (0 outside the grid)
  __device__ __forceinline__ f4 tabx(const float* t) const { return get(t, 0, gx); }
  __device__ __forceinline__ float tabz(const float* t, int z) const {
    return ldz32(t, zin(z) ? (unsigned)z : 0u, zin(z));
  }
  // C-PML: no coefficient is other than 0 outside columns [0, P) and
  // [NX - 1 - P, NX), rows [0, top) and [NZ - 1 - P, NZ) (half nodes lie half a
  // cell further). Whether the tile's columns -2 .. 65 (its rows z .. z+n-1) touch
  // those, and whether n columns from x (row z) do.
  __device__ __forceinline__ bool xs() const {
    return P > 0 && (x0 - 2 < P || x0 + kTX + 2 > NX - 1 - P);
  }
  __device__ __forceinline__ bool zs(int z, int n) const {
    return z < top || (P > 0 && z + n > NZ - 1 - P);
  }
  __device__ __forceinline__ bool xq(int x, int n) const { return x < P || x + n > NX - 1 - P; }
  // halo of this wave: 0 the rows, 1 the columns, other: none
  __device__ __forceinline__ int role() const { return (wave + (int)blockIdx.x) & 3; }
  // row halo item (64 lanes): grid row and LDS row; columns as the own ones
  __device__ __forceinline__ void row_item(int& z, int& lr) const {
    const int h = (int)(threadIdx.x & 63) >> 4;
    lr = h < 2 ? h : kElTZ + h;
    z = z0 - 2 + lr;
  }
  // column halo item (32 lanes): grid row and column, LDS row and column
  __device__ __forceinline__ bool col_item(int& z, int& x, int& lr, int& lc) const {
    const int l = threadIdx.x & 63;
    lr = (l >> 1) & 15;
    z = z0 + lr;
    x = l & 1 ? x0 + kTX : x0 - 2;
    lc = l & 1 ? kTX + 4 : 2;
    return l < 32;
  }
};

// Runs body<kFull>(tile) for the tile f.
#define EL_DISPATCH(BODY)                                                     \
  do {                                                                        \
    int x0, z0, shot;                                                         \
    Tile<kCols, true>::origin(a, f, x0, z0, shot);                            \
    if (kCols != 4 && x0 + kTX <= a.NX)                                       \
      BODY<kCols, true, kFluid>(a, Tile<kCols, true>(a, x0, z0, shot), sb);   \
    else                                                                      \
      BODY<kCols, false, kFluid>(a, Tile<kCols, false>(a, x0, z0, shot), sb); \
  } while (0)

// The stress update is txx += dt (cxx_x exx + cxx_z ezz), tzz += dt (czz_x exx +
// czz_z ezz). Away from a free surface cxx_x = czz_z = lambda + 2 mu and
// cxx_z = czz_x = lambda; on the free-surface row cxx_x = M and the other three
// are 0. So czz_x = cxx_z everywhere, and czz_z (of row j) follows from cxx_x:
// the kernels read two coefficient planes instead of four.
__device__ __forceinline__ f4 czz_z(const ElStep& a, int j, f4 cxx_x) {
  return a.fs && j == 0 ? kZ4 : cxx_x;
}

// C-PML update of the own cells with a preloaded memory variable: psi <- b psi +
// a G where a != 0 (stored with its unchanged neighbours), returns G + psi; G
// elsewhere. On: whether the wave has a cell where a != 0 may hold, q: the item.
template <class T, class A>
__device__ __forceinline__ f4 cpml(const T& t, float* psi, bool on, bool q, f4 G, A a, A b, f4 p0) {
  if (!on) return G;
  const f4 p = fma_(a, G, b * p0);
  if (q) t.put(psi, pick(a, p, p0));
  return pick(a, G + p, G);
}

// ---------------------------------------------------------------------------
// forward: velocity update  vx += dt bx (Dx+ txx + Dz- txz), vz += dt bz (Dx- txz + Dz+ tzz)
// ---------------------------------------------------------------------------
constexpr int kVelLds = kElTZ * kElXP + kElZH * kTX;  // txx, tzz; txz after them

template <int kCols, bool kFull, bool kFluid>
__device__ __forceinline__ void el_vel(const ElStep& a, const Tile<kCols, kFull>& t, float* sb) {
  float* const sxx = sb;
  float* const szz = sb + kElTZ * kElXP;
  float* const sxz = sb + kVelLds;
  const size_t so = t.so;
  const f4 txx = t.own(a.txx + so), tzz = t.own(a.tzz + so);
  const f4 txz = kFluid ? kZ4 : t.own(a.txz + so);
  const int role = t.role();
  f4 h0 = kZ4, h1 = kZ4;
  int hz, hx, lr, lc = 0;
  bool hc = false;
  if (role == 0) {
    t.row_item(hz, lr);
    h0 = t.get(a.tzz + so, hz, t.gx);
    if (!kFluid) h1 = t.get(a.txz + so, hz, t.gx);
  } else if (role == 1) {
    hc = t.col_item(hz, hx, lr, lc);
    const f2 u = t.part(a.txx + so, hz, hx, hc);
    h0 = f4{u.x, u.y, 0.0f, 0.0f};
    if (!kFluid) {
      const f2 w = t.part(a.txz + so, hz, hx, hc);
      h1 = f4{w.x, w.y, 0.0f, 0.0f};
    }
  }
  const f4 ovx = t.own(a.vx + so), ovz = t.own(a.vz + so), bx = t.own(a.bx), bz = t.own(a.bz);
  const bool xs = t.xs(), zs = t.zs(t.z0 + t.wave * 4, 4);
  const bool xq = t.xq(t.gx, 4), zq = t.zs(t.gz, 1);
  f4 axh = kZ4, bxh = kZ4, axi = kZ4, bxi = kZ4, p0 = kZ4, p1 = kZ4, p2 = kZ4, p3 = kZ4;
  float azi = 0.0f, bzi = 0.0f, azh = 0.0f, bzh = 0.0f;
  if (xs) {
    p0 = t.get(a.ps[0] + so, t.gz, t.gx, xq);
    axh = t.tabx(a.axh);
    bxh = t.tabx(a.bxh);
    if (!kFluid) {
      p2 = t.get(a.ps[2] + so, t.gz, t.gx, xq);
      axi = t.tabx(a.axi);
      bxi = t.tabx(a.bxi);
    }
  }
  if (zs) {
    p3 = t.get(a.ps[3] + so, t.gz, t.gx, zq);
    azh = t.tabz(a.azh, t.gz);
    bzh = t.tabz(a.bzh, t.gz);
    if (!kFluid) {
      p1 = t.get(a.ps[1] + so, t.gz, t.gx, zq);
      azi = t.tabz(a.azi, t.gz);
      bzi = t.tabz(a.bzi, t.gz);
    }
  }
  float* const oxx = sxx + t.r * kElXP + 4 + t.c;
  float* const ozz = szz + (t.r + 2) * kTX + t.c;
  float* const oxz = sxz + (t.r + 2) * kElXP + 4 + t.c;
  put4(oxx, txx);
  put4(ozz, tzz);
  if (!kFluid) put4(oxz, txz);
  if (role == 0) {
    put4(szz + lr * kTX + t.c, h0);
    if (!kFluid) put4(sxz + lr * kElXP + 4 + t.c, h1);
  } else if (hc) {
    put2(sxx + lr * kElXP + lc, f2{h0.x, h0.y});
    if (!kFluid) put2(sxz + (lr + 2) * kElXP + lc, f2{h1.x, h1.y});
  }
  __syncthreads();
  const bool fs = a.fs && t.z0 == 0 && t.wave == 0;
  const float ih = a.ih;
  const f4 Ga = XWin(oxx, txx).plus() * ih;
  const f4 Gd = dz_tzz(ozz, kTX, tzz, fs, t.gz) * ih;
  f4 fvx = cpml(t, a.ps[0] + so, xs, xq, Ga, axh, bxh, p0);
  f4 fvz = cpml(t, a.ps[3] + so, zs, zq, Gd, azh, bzh, p3);
  if (!kFluid) {
    const f4 Gb = dz_txz(oxz, kElXP, txz, fs, t.gz) * ih;
    const f4 Gc = XWin(oxz, txz).minus() * ih;
    fvx = fvx + cpml(t, a.ps[1] + so, zs, zq, Gb, azi, bzi, p1);
    fvz = cpml(t, a.ps[2] + so, xs, xq, Gc, axi, bxi, p2) + fvz;
  }
  t.put(a.vx + so, fma_(a.dt * bx, fvx, ovx));
  t.put(a.vz + so, fma_(a.dt * bz, fvz, ovz));
  if (a.tr[0]) {
    t.put_nt(a.tr[0] + so, fvx);
    t.put_nt(a.tr[1] + so, fvz);
  }
}

template <int kCols, bool kFluid>
__global__ __launch_bounds__(kThreads) void el_vel_kernel(ElStep a) {
  __shared__ __attribute__((aligned(16))) float sb[kVelLds + (kFluid ? 0 : kElZH * kElXP)];
  const int f = xcd_spread(blockIdx.x, gridDim.x);
  EL_DISPATCH(el_vel);
}

// ---------------------------------------------------------------------------
// forward: stress update, explosive source and, in the work-groups after the
// tiles', gathers[shot][n][r] = (vx, vz) at the receiver cell (v^{n+1/2}, which
// this kernel reads only)
// ---------------------------------------------------------------------------
template <int kCols, bool kFull, bool kFluid>
__device__ __forceinline__ void el_str(const ElStep& a, const Tile<kCols, kFull>& t, float* sb) {
  float* const svx = sb;
  float* const svz = sb + kElZH * kElXP;
  const size_t so = t.so;
  const f4 vx = t.own(a.vx + so), vz = t.own(a.vz + so);
  const int role = t.role();
  f4 h0 = kZ4, h1 = kZ4;
  int hz, hx, lr, lc = 0;
  bool hc = false;
  if (role == 0) {
    t.row_item(hz, lr);
    h1 = t.get(a.vz + so, hz, t.gx);
    if (!kFluid) h0 = t.get(a.vx + so, hz, t.gx);
  } else if (role == 1) {
    hc = t.col_item(hz, hx, lr, lc);
    const f2 u = t.part(a.vx + so, hz, hx, hc);
    h0 = f4{u.x, u.y, 0.0f, 0.0f};
    if (!kFluid) {
      const f2 w = t.part(a.vz + so, hz, hx, hc);
      h1 = f4{w.x, w.y, 0.0f, 0.0f};
    }
  }
  const f4 otxx = t.own(a.txx + so), otzz = t.own(a.tzz + so);
  const f4 otxz = kFluid ? kZ4 : t.own(a.txz + so);
  const f4 cxx_x = t.own(a.cxx_x), cxx_z = t.own(a.cxx_z);
  const f4 mxz = kFluid ? kZ4 : t.own(a.mxz);
  const bool xs = t.xs(), zs = t.zs(t.z0 + t.wave * 4, 4);
  const bool xq = t.xq(t.gx, 4), zq = t.zs(t.gz, 1);
  f4 axi = kZ4, bxi = kZ4, axh = kZ4, bxh = kZ4, p4 = kZ4, p5 = kZ4, p6 = kZ4, p7 = kZ4;
  float azi = 0.0f, bzi = 0.0f, azh = 0.0f, bzh = 0.0f;
  if (xs) {
    p4 = t.get(a.ps[4] + so, t.gz, t.gx, xq);
    axi = t.tabx(a.axi);
    bxi = t.tabx(a.bxi);
    if (!kFluid) {
      p7 = t.get(a.ps[7] + so, t.gz, t.gx, xq);
      axh = t.tabx(a.axh);
      bxh = t.tabx(a.bxh);
    }
  }
  if (zs) {
    p5 = t.get(a.ps[5] + so, t.gz, t.gx, zq);
    azi = t.tabz(a.azi, t.gz);
    bzi = t.tabz(a.bzi, t.gz);
    if (!kFluid) {
      p6 = t.get(a.ps[6] + so, t.gz, t.gx, zq);
      azh = t.tabz(a.azh, t.gz);
      bzh = t.tabz(a.bzh, t.gz);
    }
  }
  const int src = a.src_cell[t.shot];
  const float sw = a.w * a.wavelet[(size_t)t.shot * a.nt + a.n];
  float* const ox = svx + (t.r + 2) * kElXP + 4 + t.c;
  float* const oz = svz + (t.r + 2) * kElXP + 4 + t.c;
  put4(ox, vx);
  put4(oz, vz);
  if (role == 0) {
    put4(svz + lr * kElXP + 4 + t.c, h1);
    if (!kFluid) put4(svx + lr * kElXP + 4 + t.c, h0);
  } else if (hc) {
    put2(svx + (lr + 2) * kElXP + lc, f2{h0.x, h0.y});
    if (!kFluid) put2(svz + (lr + 2) * kElXP + lc, f2{h1.x, h1.y});
  }
  __syncthreads();
  const bool fs = a.fs && t.z0 == 0 && t.wave == 0;
  const float ih = a.ih, dt = a.dt;
  const f4 Ge = XWin(ox, vx).minus() * ih;
  const f4 Gf = dz_vz(oz, kElXP, vz, fs, t.gz) * ih;
  const f4 exx = cpml(t, a.ps[4] + so, xs, xq, Ge, axi, bxi, p4);
  const f4 ezz = cpml(t, a.ps[5] + so, zs, zq, Gf, azi, bzi, p5);
  f4 txx = otxx + dt * fma_(cxx_x, exx, cxx_z * ezz);
  f4 tzz = otzz + dt * fma_(cxx_z, exx, czz_z(a, t.gz, cxx_x) * ezz);
  const int sc = src - (t.gz * t.NX + t.gx);
  if ((unsigned)sc < 4u && t.xin(t.gx + sc)) {
    const float sz = sw * u32at(a.smask, (unsigned)src);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q == sc) {
        txx[q] += sw;
        tzz[q] += sz;
      }
  }
  t.put(a.txx + so, txx);
  t.put(a.tzz + so, tzz);
  f4 exz = kZ4;
  if (!kFluid) {
    const f4 Gg = dz_vx(ox, kElXP, vx, fs, t.gz) * ih;
    const f4 Gh = XWin(oz, vz).plus() * ih;
    exz = cpml(t, a.ps[6] + so, zs, zq, Gg, azh, bzh, p6) +
          cpml(t, a.ps[7] + so, xs, xq, Gh, axh, bxh, p7);
    t.put(a.txz + so, fma_(dt * mxz, exz, otxz));
  }
  if (a.tr[2]) {
    t.put_nt(a.tr[2] + so, exx);
    t.put_nt(a.tr[3] + so, ezz);
    if (!kFluid) t.put_nt(a.tr[4] + so, exz);
  }
}

template <int kCols, bool kFluid>
__global__ __launch_bounds__(kThreads) void el_str_kernel(ElStep a, int ntiles) {
  __shared__ __attribute__((aligned(16))) float sb[2 * kElZH * kElXP];
  if ((int)blockIdx.x >= ntiles) {
    const size_t t = (size_t)(blockIdx.x - ntiles) * kThreads + threadIdx.x;
    if (t >= (size_t)a.nshots * a.nrec) return;
    const int s = (int)(t / a.nrec), r = (int)(t - (size_t)s * a.nrec);
    const size_t k = (size_t)s * ((size_t)a.NX * a.NZ) + a.rec_cell[t];
    float* d = a.gathers + (((size_t)s * a.nt + a.n) * a.nrec + r) * 2;
    d[0] = a.vx[k];
    d[1] = a.vz[k];
    return;
  }
  const int f = xcd_spread(blockIdx.x, ntiles);
  EL_DISPATCH(el_str);
}

// ---------------------------------------------------------------------------
// Reverse step. With ebar = dt (stress coefficient) x (stress adjoint) and the
// C-PML adjoint t = Psi + ebar, the derivative input adjoint is ebar + a t and
// Psi <- b t. The velocity adjoints collect the transposed derivatives of those.
// ---------------------------------------------------------------------------

// Transposed z-derivative of a staged plane (column group `at`, own row c, row
// pitch kTX) at row j: standard (-Dz- or -Dz+) away from a free surface,
// otherwise (fs: the wave of the first four rows) the host-derived taps, whose
// offsets lie within two rows.
__device__ __forceinline__ f4 dzT(const ElStep& a, int kind, const float* at, f4 c, bool fs, int j,
                                  bool minus_dzm) {
  if (fs) {
    f4 acc = kZ4;
    const int n = a.tt_cnt[kind][j & 3];
    for (int e = 0; e < n; ++e)
      acc = fma_(a.tt_w[kind][j & 3][e], lds4(at + a.tt_off[kind][j & 3][e] * kTX), acc);
    return acc;
  }
  return minus_dzm ? -zminus(at, kTX, c) : -zplus(at, kTX, c);
}

// Derivative-input adjoint e + a (q + e) where a != 0, e elsewhere.
template <class F, class A>
__device__ __forceinline__ F adj_in(A a, F q, F e) {
  return pick(a, fma_(a, q + e, e), e);
}

// The memory-variable adjoint b (q + e) of the own cells (0 where a = 0, where
// it is never used).
template <class T, class A>
__device__ __forceinline__ void adj_psi(const T& t, float* out, bool on, bool q, A a, A b, f4 q0,
                                        f4 e) {
  if (on && q) t.put(out, pick(a, b * (q0 + e), kZ4));
}

constexpr int kAdjX = kElTZ * kElXP, kAdjZ = kElZH * kTX;  // LDS planes with an x, a z halo

// Velocity adjoints from the stress adjoints, coefficient gradients, then the
// residuals of the receivers in the tile.
template <int kCols, bool kFull, bool kFluid>
__device__ __forceinline__ void el_adj_s(const ElStep& a, const Tile<kCols, kFull>& t, float* sb) {
  float* const sbe = sb;                  // exx input, x halo
  float* const sbf = sb + kAdjX;          // ezz input, z halo
  float* const sbg = sbf + kAdjZ;         // Dz vx of exz, z halo
  float* const sbh = sbg + kAdjZ;         // Dx vz of exz, x halo
  const size_t so = t.so;
  const float dt = a.dt, ih = a.ih;
  const int role = t.role();
  const bool xs = t.xs();
  // this thread's halo item: stress adjoints, coefficients, memory variables
  f4 hs0 = kZ4, hs1 = kZ4, hs2 = kZ4, hc0 = kZ4, hc1 = kZ4, hc2 = kZ4, hq0 = kZ4, hq1 = kZ4;
  f4 ha0 = kZ4, ha1 = kZ4;
  int hz, hx, lr, lc = 0;
  bool hc = false;
  if (role == 0) {
    t.row_item(hz, lr);
    hs0 = t.get(a.txx + so, hz, t.gx);
    hs1 = t.get(a.tzz + so, hz, t.gx);
    hc0 = t.get(a.cxx_x, hz, t.gx);
    hc1 = t.get(a.cxx_z, hz, t.gx);
    if (!kFluid) {
      hs2 = t.get(a.txz + so, hz, t.gx);
      hc2 = t.get(a.mxz, hz, t.gx);
    }
    if (t.zs(t.z0 - 2, 2) || t.zs(t.z0 + kElTZ, 2)) {
      const bool q = t.zs(hz, 1);
      hq0 = t.get(a.ps_in[5] + so, hz, t.gx, q);
      ha0.x = t.tabz(a.azi, hz);
      if (!kFluid) {
        hq1 = t.get(a.ps_in[6] + so, hz, t.gx, q);
        ha1.x = t.tabz(a.azh, hz);
      }
    }
  } else if (role == 1) {
    hc = t.col_item(hz, hx, lr, lc);
    auto two = [&](const float* f, bool q) {
      const f2 v = t.part(f, hz, hx, hc && q);
      return f4{v.x, v.y, 0.0f, 0.0f};
    };
    hs0 = two(a.txx + so, true);
    hs1 = two(a.tzz + so, true);
    hc0 = two(a.cxx_x, true);
    hc1 = two(a.cxx_z, true);
    if (!kFluid) {
      hs2 = two(a.txz + so, true);
      hc2 = two(a.mxz, true);
    }
    if (xs) {
      const bool q = t.xq(hx, 2);
      const f2 u = t.part(a.axi, 0, hx, hc);
      hq0 = two(a.ps_in[4] + so, q);
      ha0 = f4{u.x, u.y, 0.0f, 0.0f};
      if (!kFluid) {
        const f2 w = t.part(a.axh, 0, hx, hc);
        hq1 = two(a.ps_in[7] + so, q);
        ha1 = f4{w.x, w.y, 0.0f, 0.0f};
      }
    }
  }
  const f4 txx = t.own(a.txx + so), tzz = t.own(a.tzz + so);
  const f4 cxx_x = t.own(a.cxx_x), cxx_z = t.own(a.cxx_z);
  const f4 txz = kFluid ? kZ4 : t.own(a.txz + so), mxz = kFluid ? kZ4 : t.own(a.mxz);
  const bool zs = t.zs(t.z0 + t.wave * 4, 4);
  const bool xq = t.xq(t.gx, 4), zq = t.zs(t.gz, 1);
  f4 axi = kZ4, axh = kZ4, q4 = kZ4, q5 = kZ4, q6 = kZ4, q7 = kZ4;
  float azi = 0.0f, azh = 0.0f;
  if (xs) {
    q4 = t.get(a.ps_in[4] + so, t.gz, t.gx, xq);
    axi = t.tabx(a.axi);
    if (!kFluid) {
      q7 = t.get(a.ps_in[7] + so, t.gz, t.gx, xq);
      axh = t.tabx(a.axh);
    }
  }
  if (zs) {
    q5 = t.get(a.ps_in[5] + so, t.gz, t.gx, zq);
    azi = t.tabz(a.azi, t.gz);
    if (!kFluid) {
      q6 = t.get(a.ps_in[6] + so, t.gz, t.gx, zq);
      azh = t.tabz(a.azh, t.gz);
    }
  }
  // the shot's receivers in the tile's rows (all of them where there are too few
  // for a directory)
  const int4* const rs = a.rec_sorted + (size_t)t.shot * a.nrec;
  const int e0 = a.rec_dir ? rs[t.z0 / kElTZ].w : 0;
  const int e1 = a.rec_dir ? rs[t.z0 / kElTZ + 1].w : a.nrec;

  // the halo's planes: rows ezz (czz_z = cxx_x there) and Dz vx, columns exx, Dx vz
  if (role == 0) {
    put4(sbf + lr * kTX + t.c, adj_in(ha0.x, hq0, dt * fma_(hc1, hs0, hc0 * hs1)));
    if (!kFluid) put4(sbg + lr * kTX + t.c, adj_in(ha1.x, hq1, dt * hc2 * hs2));
  } else if (hc) {
    const f4 he = adj_in(ha0, hq0, dt * fma_(hc0, hs0, hc1 * hs1));
    put2(sbe + lr * kElXP + lc, f2{he.x, he.y});
    if (!kFluid) {
      const f4 hh = adj_in(ha1, hq1, dt * hc2 * hs2);
      put2(sbh + lr * kElXP + lc, f2{hh.x, hh.y});
    }
  }
  const f4 ex = dt * fma_(cxx_x, txx, cxx_z * tzz);
  const f4 ez = dt * fma_(cxx_z, txx, czz_z(a, t.gz, cxx_x) * tzz);
  const f4 exz = dt * mxz * txz;
  const f4 be = adj_in(axi, q4, ex), bf = adj_in(azi, q5, ez);
  const f4 bg = adj_in(azh, q6, exz), bh = adj_in(axh, q7, exz);
  float* const oe = sbe + t.r * kElXP + 4 + t.c;
  float* const of = sbf + (t.r + 2) * kTX + t.c;
  float* const og = sbg + (t.r + 2) * kTX + t.c;
  float* const oh = sbh + t.r * kElXP + 4 + t.c;
  put4(oe, be);
  put4(of, bf);
  if (!kFluid) {
    put4(og, bg);
    put4(oh, bh);
  }
  // memory-variable adjoints
  if (xs) {
    adj_psi(t, a.ps_out[4] + so, xs, xq, axi, t.tabx(a.bxi), q4, ex);
    if (!kFluid) adj_psi(t, a.ps_out[7] + so, xs, xq, axh, t.tabx(a.bxh), q7, exz);
  }
  if (zs) {
    adj_psi(t, a.ps_out[5] + so, zs, zq, azi, t.tabz(a.bzi, t.gz), q5, ez);
    if (!kFluid) adj_psi(t, a.ps_out[6] + so, zs, zq, azh, t.tabz(a.bzh, t.gz), q6, exz);
  }
  const bool gacc = !a.g_init;
  const f4 ovx = t.own(a.vx + so), ovz = t.own(a.vz + so);
  const f4 fexx = t.own_nt(a.trc[2] + so), fezz = t.own_nt(a.trc[3] + so);
  const f4 fexz = kFluid ? kZ4 : t.own_nt(a.trc[4] + so);
  f4 g0 = kZ4, g1 = kZ4, g2 = kZ4;
  if (gacc) {
    g0 = t.own_nt(a.g[0] + so);
    if (!kFluid) {
      g1 = t.own_nt(a.g[1] + so);
      g2 = t.own_nt(a.g[2] + so);
    }
  }
  __syncthreads();
  const bool fs = a.fs && t.z0 == 0 && t.wave == 0;
  // Vx += (Dx-)^T gbe + (Dz+ of vx)^T gbg ;  (Dx-)^T = -Dx+
  // Vz += (Dz- of vz)^T gbf + (Dx+)^T gbh ;  (Dx+)^T = -Dx-
  // (the exz terms are absent in a fluid)
  f4 dvx = -XWin(oe, be).plus();
  f4 dvz = dzT(a, 3, of, bf, fs, t.gz, false);
  if (!kFluid) {
    dvx = dvx + dzT(a, 2, og, bg, fs, t.gz, true);
    dvz = dvz + -XWin(oh, bh).minus();
  }
  t.put(a.vx + so, ovx + dvx * ih);
  t.put(a.vz + so, ovz + dvz * ih);

  // coefficient gradients
  f4 glam = dt * (txx + tzz) * (fexx + fezz);
  f4 gmu = 2.0f * dt * fma_(txx, fexx, tzz * fezz);
  if (fs && t.gz == 0) {
    // txx += dt M exx with M = 4 mu (lambda + mu) / (lambda + 2 mu)
    const f4 gM = dt * txx * fexx;
    glam = gM * t.tabx(a.dM_dl);
    gmu = gM * t.tabx(a.dM_dm);
  }
  // a fluid has no mu partials (the gradient finish weighs them by vs = 0;
  // their planes stay zero)
  const f4 gmxz = dt * txz * fexz;
  g0 = gacc ? g0 + glam : glam;
  g1 = gacc ? g1 + gmu : gmu;
  g2 = gacc ? g2 + gmxz : gmxz;
  t.put_nt(a.g[0] + so, g0);
  if (!kFluid) {
    t.put_nt(a.g[1] + so, g1);
    t.put_nt(a.g[2] + so, g2);
  }

  // residual injection into the velocity adjoints just written (receivers sorted
  // by (cell, r); the first of each run of equal cells adds the whole run in order)
  if (e1 > e0) {
    __syncthreads();
    for (int e = e0 + (int)threadIdx.x; e < e1; e += kThreads) {
      const int cell = rs[e].y, z = cell / t.NX, x = cell - z * t.NX;
      if ((unsigned)(x - t.x0) >= (unsigned)kTX || (unsigned)(z - t.z0) >= (unsigned)kElTZ ||
          (e > e0 && rs[e - 1].y == cell))
        continue;
      float ax = a.vx[so + cell], az = a.vz[so + cell];
      for (int q = e; q < e1 && rs[q].y == cell; ++q) {
        const float* s = a.resid + (((size_t)t.shot * a.nt + a.n) * a.nrec + rs[q].z) * 2;
        ax += s[0];
        az += s[1];
      }
      a.vx[so + cell] = ax;
      a.vz[so + cell] = az;
    }
  }
}

template <int kCols, bool kFluid>
__global__ __launch_bounds__(kThreads) void el_adj_s_kernel(ElStep a) {
  __shared__ __attribute__((aligned(16))) float sb[(kFluid ? 1 : 2) * (kAdjX + kAdjZ)];
  const int f = xcd_spread(blockIdx.x, gridDim.x);
  EL_DISPATCH(el_adj_s);
}

// Stress adjoints from the velocity adjoints, buoyancy gradients. Derivative-
// input adjoints of the velocity step: gba (Dx txx of vx), gbb (Dz txz of vx),
// gbc (Dx txz of vz), gbd (Dz tzz of vz); a fluid has gba and gbd only.
template <int kCols, bool kFull, bool kFluid>
__device__ __forceinline__ void el_adj_v(const ElStep& a, const Tile<kCols, kFull>& t, float* sb) {
  float* const sba = sb;           // x halo
  float* const sbd = sb + kAdjX;   // z halo
  float* const sbb = sbd + kAdjZ;  // z halo
  float* const sbc = sbb + kAdjZ;  // x halo
  const size_t so = t.so;
  const float dt = a.dt, ih = a.ih;
  const int role = t.role();
  const bool xs = t.xs();
  f4 hvx = kZ4, hvz = kZ4, hbx = kZ4, hbz = kZ4, hq0 = kZ4, hq1 = kZ4, ha0 = kZ4, ha1 = kZ4;
  int hz, hx, lr, lc = 0;
  bool hc = false;
  if (role == 0) {  // gbd, gbb
    t.row_item(hz, lr);
    hvz = t.get(a.vz + so, hz, t.gx);
    hbz = t.get(a.bz, hz, t.gx);
    if (!kFluid) {
      hvx = t.get(a.vx + so, hz, t.gx);
      hbx = t.get(a.bx, hz, t.gx);
    }
    if (t.zs(t.z0 - 2, 2) || t.zs(t.z0 + kElTZ, 2)) {
      const bool q = t.zs(hz, 1);
      hq0 = t.get(a.ps_in[3] + so, hz, t.gx, q);
      ha0.x = t.tabz(a.azh, hz);
      if (!kFluid) {
        hq1 = t.get(a.ps_in[1] + so, hz, t.gx, q);
        ha1.x = t.tabz(a.azi, hz);
      }
    }
  } else if (role == 1) {  // gba, gbc
    hc = t.col_item(hz, hx, lr, lc);
    auto two = [&](const float* f, bool q) {
      const f2 v = t.part(f, hz, hx, hc && q);
      return f4{v.x, v.y, 0.0f, 0.0f};
    };
    hvx = two(a.vx + so, true);
    hbx = two(a.bx, true);
    if (!kFluid) {
      hvz = two(a.vz + so, true);
      hbz = two(a.bz, true);
    }
    if (xs) {
      const bool q = t.xq(hx, 2);
      const f2 u = t.part(a.axh, 0, hx, hc);
      hq0 = two(a.ps_in[0] + so, q);
      ha0 = f4{u.x, u.y, 0.0f, 0.0f};
      if (!kFluid) {
        const f2 w = t.part(a.axi, 0, hx, hc);
        hq1 = two(a.ps_in[2] + so, q);
        ha1 = f4{w.x, w.y, 0.0f, 0.0f};
      }
    }
  }
  const f4 vx = t.own(a.vx + so), vz = t.own(a.vz + so), bx = t.own(a.bx), bz = t.own(a.bz);
  const bool zs = t.zs(t.z0 + t.wave * 4, 4);
  const bool xq = t.xq(t.gx, 4), zq = t.zs(t.gz, 1);
  f4 axh = kZ4, axi = kZ4, q0 = kZ4, q1 = kZ4, q2 = kZ4, q3 = kZ4;
  float azi = 0.0f, azh = 0.0f;
  if (xs) {
    q0 = t.get(a.ps_in[0] + so, t.gz, t.gx, xq);
    axh = t.tabx(a.axh);
    if (!kFluid) {
      q2 = t.get(a.ps_in[2] + so, t.gz, t.gx, xq);
      axi = t.tabx(a.axi);
    }
  }
  if (zs) {
    q3 = t.get(a.ps_in[3] + so, t.gz, t.gx, zq);
    azh = t.tabz(a.azh, t.gz);
    if (!kFluid) {
      q1 = t.get(a.ps_in[1] + so, t.gz, t.gx, zq);
      azi = t.tabz(a.azi, t.gz);
    }
  }
  if (role == 0) {
    put4(sbd + lr * kTX + t.c, adj_in(ha0.x, hq0, dt * hbz * hvz));
    if (!kFluid) put4(sbb + lr * kTX + t.c, adj_in(ha1.x, hq1, dt * hbx * hvx));
  } else if (hc) {
    const f4 h0 = adj_in(ha0, hq0, dt * hbx * hvx);
    put2(sba + lr * kElXP + lc, f2{h0.x, h0.y});
    if (!kFluid) {
      const f4 h2 = adj_in(ha1, hq1, dt * hbz * hvz);
      put2(sbc + lr * kElXP + lc, f2{h2.x, h2.y});
    }
  }
  const f4 kx = dt * bx * vx, kz = dt * bz * vz;
  const f4 ba = adj_in(axh, q0, kx), bb = adj_in(azi, q1, kx);
  const f4 bc = adj_in(axi, q2, kz), bd = adj_in(azh, q3, kz);
  float* const oa = sba + t.r * kElXP + 4 + t.c;
  float* const od = sbd + (t.r + 2) * kTX + t.c;
  float* const ob = sbb + (t.r + 2) * kTX + t.c;
  float* const oc = sbc + t.r * kElXP + 4 + t.c;
  put4(oa, ba);
  put4(od, bd);
  if (!kFluid) {
    put4(ob, bb);
    put4(oc, bc);
  }
  if (xs) {
    adj_psi(t, a.ps_out[0] + so, xs, xq, axh, t.tabx(a.bxh), q0, kx);
    if (!kFluid) adj_psi(t, a.ps_out[2] + so, xs, xq, axi, t.tabx(a.bxi), q2, kz);
  }
  if (zs) {
    adj_psi(t, a.ps_out[3] + so, zs, zq, azh, t.tabz(a.bzh, t.gz), q3, kz);
    if (!kFluid) adj_psi(t, a.ps_out[1] + so, zs, zq, azi, t.tabz(a.bzi, t.gz), q1, kx);
  }
  const bool gacc = !a.g_init;
  const f4 otxx = t.own(a.txx + so), otzz = t.own(a.tzz + so);
  const f4 otxz = kFluid ? kZ4 : t.own(a.txz + so);
  const f4 f0 = t.own_nt(a.trc[0] + so), f1 = t.own_nt(a.trc[1] + so);
  f4 g3 = kZ4, g4 = kZ4;
  if (gacc) {
    g3 = t.own_nt(a.g[3] + so);
    g4 = t.own_nt(a.g[4] + so);
  }
  __syncthreads();
  const bool fs = a.fs && t.z0 == 0 && t.wave == 0;
  // Txx += (Dx+)^T gba = -Dx- gba ;  Tzz += (Dz+ of tzz)^T gbd
  t.put(a.txx + so, otxx + -XWin(oa, ba).minus() * ih);
  t.put(a.tzz + so, otzz + dzT(a, 0, od, bd, fs, t.gz, true) * ih);
  // Txz += (Dz- of txz)^T gbb + (Dx-)^T gbc = ... - Dx+ gbc (a fluid's txz
  // adjoint reaches nothing: its only use is weighed by mu = 0)
  if (!kFluid)
    t.put(a.txz + so, otxz + (dzT(a, 1, ob, bb, fs, t.gz, false) + -XWin(oc, bc).plus()) * ih);

  const f4 gbx = dt * vx * f0, gbz = dt * vz * f1;
  g3 = gacc ? g3 + gbx : gbx;
  g4 = gacc ? g4 + gbz : gbz;
  t.put_nt(a.g[3] + so, g3);
  t.put_nt(a.g[4] + so, g4);
}

template <int kCols, bool kFluid>
__global__ __launch_bounds__(kThreads) void el_adj_v_kernel(ElStep a) {
  __shared__ __attribute__((aligned(16))) float sb[(kFluid ? 1 : 2) * (kAdjX + kAdjZ)];
  const int f = xcd_spread(blockIdx.x, gridDim.x);
  EL_DISPATCH(el_adj_v);
}

// ---------------------------------------------------------------------------
// Material preparation: padded vp, vs, rho, lambda, mu; buoyancies; harmonic
// mu at txz nodes; stress coefficients (free-surface row uses M); C-PML tables.
// A fluid model holds (vp, rho) and has vs = 0.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double el_vs(const float* model, size_t mn, size_t m, int fluid) {
  return fluid ? 0.0 : (double)model[mn + m];
}
__device__ __forceinline__ double el_rho(const float* model, size_t mn, size_t m, int fluid) {
  return (double)model[(fluid ? 1 : 2) * mn + m];
}

__global__ void el_prep_kernel(const float* model, ElCoef c, int nx, int nz, int P, int top,
                               int NX, int NZ, int fs, int fluid) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (i >= NX || j >= NZ) return;
  const size_t mn = (size_t)nx * nz;
  const int ii = min(max(i - P, 0), nx - 1), jj = min(max(j - top, 0), nz - 1);
  const size_t m = (size_t)jj * nx + ii, k = (size_t)j * NX + i;
  const double vp = model[m], vs = el_vs(model, mn, m, fluid), rho = el_rho(model, mn, m, fluid);
  const double mu = rho * vs * vs, lam = rho * (vp * vp - 2.0 * vs * vs);
  c.vp[k] = (float)vp;
  c.vs[k] = (float)vs;
  c.rho[k] = (float)rho;
  c.lam[k] = (float)lam;
  c.mu[k] = (float)mu;
  if (fs && j == 0) {
    const double d = lam + 2.0 * mu;
    c.cxx_x[k] = d > 0 ? (float)(4.0 * mu * (lam + mu) / d) : 0.0f;
    c.cxx_z[k] = c.czz_x[k] = c.czz_z[k] = 0.0f;
    c.smask[k] = 0.0f;
    c.dM_dl[i] = d > 0 ? (float)(4.0 * mu * mu / (d * d)) : 0.0f;
    c.dM_dm[i] = d > 0 ? (float)(4.0 * (lam * lam + 2.0 * lam * mu + 2.0 * mu * mu) / (d * d)) : 0.0f;
  } else {
    c.cxx_x[k] = c.czz_z[k] = (float)(lam + 2.0 * mu);
    c.cxx_z[k] = c.czz_x[k] = (float)lam;
    c.smask[k] = 1.0f;
  }
}

// buoyancies and the harmonic-mean shear modulus need neighbouring cells: a
// second pass over the padded grid (values re-read from the edge-replicated model)
__device__ __forceinline__ size_t el_model_index(int i, int j, int nx, int nz, int P, int top) {
  const int mi = min(max(i - P, 0), nx - 1), mj = min(max(j - top, 0), nz - 1);
  return (size_t)mj * nx + mi;
}

__global__ void el_prep2_kernel(const float* model, ElCoef c, int nx, int nz, int P, int top,
                                int NX, int NZ, int fluid) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (i >= NX || j >= NZ) return;
  const size_t mn = (size_t)nx * nz;
  auto rho_at = [&](int ii, int jj) -> double {
    return el_rho(model, mn, el_model_index(ii, jj, nx, nz, P, top), fluid);
  };
  auto mu_at = [&](int ii, int jj) -> double {
    const size_t m = el_model_index(ii, jj, nx, nz, P, top);
    const double vs = el_vs(model, mn, m, fluid), rho = el_rho(model, mn, m, fluid);
    return rho * vs * vs;
  };
  const int i1 = min(i + 1, NX - 1), j1 = min(j + 1, NZ - 1);
  const size_t k = (size_t)j * NX + i;
  const double r0 = rho_at(i, j);
  c.bx[k] = (float)(2.0 / (r0 + rho_at(i1, j)));
  c.bz[k] = (float)(2.0 / (r0 + rho_at(i, j1)));
  const double m00 = mu_at(i, j), m10 = mu_at(i1, j), m01 = mu_at(i, j1), m11 = mu_at(i1, j1);
  c.mxz[k] = (m00 > 0 && m10 > 0 && m01 > 0 && m11 > 0)
                 ? (float)(4.0 / (1.0 / m00 + 1.0 / m10 + 1.0 / m01 + 1.0 / m11))
                 : 0.0f;
}

// C-PML coefficients at node x = i + shift of an axis of n cells with lo / hi pads
__device__ void el_pml(int i, double shift, int n, int lo, int hi, double h, double dt,
                       double vmax, double f0, double R, float* a, float* b) {
  const double x = i + shift;
  double xi = 0.0, L = 1.0;
  if (lo > 0 && x < lo) {
    xi = (lo - x) * h;
    L = lo * h;
  } else if (hi > 0 && x > n - 1 - hi) {
    xi = (x - (n - 1 - hi)) * h;
    L = hi * h;
  }
  if (xi > L) xi = L;
  const double d0 = -3.0 * vmax * log(R) / (2.0 * L);
  const double d = xi > 0.0 ? d0 * (xi / L) * (xi / L) : 0.0;
  const double alpha = M_PI * f0 * (1.0 - xi / L);
  const double bb = exp(-(d + alpha) * dt);
  b[i] = (float)bb;
  a[i] = d > 0.0 ? (float)(d / (d + alpha) * (bb - 1.0)) : 0.0f;
}

__global__ void el_tables_kernel(ElCoef c, int NX, int NZ, int P, int top, double h, double dt,
                                 double vmax, double f0, double R) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < NX) {
    el_pml(i, 0.0, NX, P, P, h, dt, vmax, f0, R, c.axi, c.bxi);
    el_pml(i, 0.5, NX, P, P, h, dt, vmax, f0, R, c.axh, c.bxh);
  }
  if (i < NZ) {
    el_pml(i, 0.0, NZ, top, P, h, dt, vmax, f0, R, c.azi, c.bzi);
    el_pml(i, 0.5, NZ, top, P, h, dt, vmax, f0, R, c.azh, c.bzh);
  }
}

// tot_q += sum over shots of the FP32 partial q (q = 0..4), float64
__global__ void el_fold_kernel(double* tot, const float* gpart, int nshots, size_t plane) {
  const size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int q = blockIdx.y;
  if (c >= plane) return;
  double acc = tot[q * plane + c];
  for (int s = 0; s < nshots; ++s) acc += (double)gpart[((size_t)q * nshots + s) * plane + c];
  tot[q * plane + c] = acc;
}

// Chain rule on the padded grid for one padded cell:
//   lambda = rho (vp^2 - 2 vs^2), mu = rho vs^2; mu_xz = harmonic mean of 4 mu;
//   b = 2/(rho_a + rho_b). Returns (gvp, gvs, grho).
__device__ void el_chain_cell(const double* tot, size_t plane, const ElCoef& c, int i, int j,
                              int NX, int NZ, double* out) {
  const size_t q = (size_t)j * NX + i;
  double gl = tot[q], gm = tot[plane + q], gr = 0.0;
  const double muq = c.mu[q];
  // contributions of the txz nodes and buoyancy nodes whose stencil uses cell q
  for (int dj = -1; dj <= 0; ++dj)
    for (int di = -1; di <= 0; ++di) {
      const int ki = i + di, kj = j + dj;
      if (ki < 0 || kj < 0) continue;
      const int k1i = min(ki + 1, NX - 1), k1j = min(kj + 1, NZ - 1);
      const size_t k = (size_t)kj * NX + ki;
      // multiplicity of q among the four mu cells of txz node k
      const int mult = (ki == i && kj == j) + (k1i == i && kj == j) + (ki == i && k1j == j) +
                       (k1i == i && k1j == j);
      const double mxz = c.mxz[k];
      if (mult && mxz > 0.0 && muq > 0.0)
        gm += mult * tot[2 * plane + k] * mxz * mxz / (4.0 * muq * muq);
      // buoyancy bx at k uses rho at (ki, kj) and (k1i, kj); bz at (ki, kj), (ki, k1j)
      if (kj == j) {
        const int mb = (ki == i) + (k1i == i);
        const double b = c.bx[k];
        gr += mb * tot[3 * plane + k] * (-0.5 * b * b);
      }
      if (ki == i) {
        const int mb = (kj == j) + (k1j == j);
        const double b = c.bz[k];
        gr += mb * tot[4 * plane + k] * (-0.5 * b * b);
      }
    }
  const double vp = c.vp[q], vs = c.vs[q], rho = c.rho[q];
  out[0] = gl * 2.0 * rho * vp;
  out[1] = gl * (-4.0 * rho * vs) + gm * 2.0 * rho * vs;
  out[2] = gl * (vp * vp - 2.0 * vs * vs) + gm * vs * vs + gr;
}

// dJ/d(model) of a model cell: the chain rule summed over the padded cells that
// repeat it. The border takes a wave per cell: with a thread per cell a corner's
// (P + 1)^2 terms were the kernel's time (660 x 330 cells, P = 30: 1.3 ms, now 56 us).
__global__ __launch_bounds__(256) void el_finish_kernel(const double* tot, ElCoef c, float* grad,
                                                        int nx, int nz, int P, int top, int NX,
                                                        int NZ, int fluid) {
  int ii, jj, lane, nl;
  if (!finish_cell(nx, nz, ii, jj, lane, nl)) return;
  const size_t plane = (size_t)NX * NZ;
  const int i0 = ii == 0 ? 0 : ii + P, i1 = ii == nx - 1 ? NX - 1 : ii + P;
  const int j0 = jj == 0 ? 0 : jj + top, j1 = jj == nz - 1 ? NZ - 1 : jj + top;
  const int w = i1 - i0 + 1, n = w * (j1 - j0 + 1);
  double acc[3] = {0.0, 0.0, 0.0};
  for (int t = lane; t < n; t += nl) {
    double o[3];
    el_chain_cell(tot, plane, c, i0 + t % w, j0 + t / w, NX, NZ, o);
    acc[0] += o[0];
    acc[1] += o[1];
    acc[2] += o[2];
  }
  for (double& v : acc) v = finish_sum(v, nl);
  if (lane) return;
  const size_t mn = (size_t)nx * nz, m = (size_t)jj * nx + ii;
  grad[m] = (float)acc[0];
  if (fluid) {  // (vp, rho); the vs term vanishes at vs = 0
    grad[mn + m] = (float)acc[2];
  } else {
    grad[mn + m] = (float)acc[1];
    grad[2 * mn + m] = (float)acc[2];
  }
}

int tiles_of(const ElStep& a) {
  return ((a.NX + kTX - 1) / kTX) * ((a.NZ + kElTZ - 1) / kElTZ) * a.nshots;
}

template <int kCols, bool kFluid>
void launch_fwd(const ElStep& a, hipStream_t s) {
  const int n = tiles_of(a);
  const int rec = a.gathers ? (int)(((size_t)a.nshots * a.nrec + kThreads - 1) / kThreads) : 0;
  hipLaunchKernelGGL((el_vel_kernel<kCols, kFluid>), dim3(n), dim3(kThreads), 0, s, a);
  hipLaunchKernelGGL((el_str_kernel<kCols, kFluid>), dim3(n + rec), dim3(kThreads), 0, s, a, n);
}
template <int kCols, bool kFluid>
void launch_adj(const ElStep& a, hipStream_t s) {
  const int n = tiles_of(a);
  hipLaunchKernelGGL((el_adj_s_kernel<kCols, kFluid>), dim3(n), dim3(kThreads), 0, s, a);
  hipLaunchKernelGGL((el_adj_v_kernel<kCols, kFluid>), dim3(n), dim3(kThreads), 0, s, a);
}
template <int kCols>
void launch(const ElStep& a, bool adj, hipStream_t s) {
  if (adj)
    a.fluid ? launch_adj<kCols, true>(a, s) : launch_adj<kCols, false>(a, s);
  else
    a.fluid ? launch_fwd<kCols, true>(a, s) : launch_fwd<kCols, false>(a, s);
}
int launch(const ElStep& a, bool adj, hipStream_t s, hipEvent_t* ev) {
  if (ev) SWEEP_HIP(hipEventRecord(ev[0], s));
  if (a.NX % 4 == 0)
    launch<4>(a, adj, s);
  else if (a.NX >= 4)
    launch<2>(a, adj, s);
  else
    launch<1>(a, adj, s);
  if (ev) SWEEP_HIP(hipEventRecord(ev[1], s));
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

}  // namespace

int el_launch_prep(const float* model, const ElCoef& c, int nx, int nz, int P, int fs, int fluid,
                   double h, double dt, double vmax, double f0, double R, hipStream_t s) {
  const int top = fs ? 0 : P;
  const int NX = nx + 2 * P, NZ = nz + top + P;
  hipLaunchKernelGGL(el_prep_kernel, dim3((NX + 255) / 256, NZ), dim3(256), 0, s, model, c, nx,
                     nz, P, top, NX, NZ, fs, fluid);
  hipLaunchKernelGGL(el_prep2_kernel, dim3((NX + 255) / 256, NZ), dim3(256), 0, s, model, c, nx,
                     nz, P, top, NX, NZ, fluid);
  const int nmax = NX > NZ ? NX : NZ;
  hipLaunchKernelGGL(el_tables_kernel, dim3((nmax + 255) / 256), dim3(256), 0, s, c, NX, NZ, P,
                     top, h, dt, vmax, f0, R);
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

int el_launch_fwd(const ElStep& a, hipStream_t s, hipEvent_t* ev) { return launch(a, false, s, ev); }

int el_launch_adj(const ElStep& a, hipStream_t s, hipEvent_t* ev) { return launch(a, true, s, ev); }

int el_launch_fold(double* tot, const float* gpart, int nshots, size_t plane, hipStream_t s) {
  hipLaunchKernelGGL(el_fold_kernel, dim3((unsigned)((plane + 255) / 256), 5), dim3(256), 0, s,
                     tot, gpart, nshots, plane);
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

int el_launch_finish(const double* tot, const ElCoef& c, float* grad, int nx, int nz, int P,
                     int fs, int fluid, hipStream_t s) {
  const int top = fs ? 0 : P;
  const int NX = nx + 2 * P, NZ = nz + top + P;
  hipLaunchKernelGGL(el_finish_kernel, finish_grid(nx, nz), dim3(256), 0, s, tot, c, grad,
                     nx, nz, P, top, NX, NZ, fluid);
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

}  // namespace sweep
