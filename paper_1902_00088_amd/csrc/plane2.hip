// 2D stage, filter, analysis and refinement kernels over whole blocks or halves of blocks
// (gfx950): advection on blocks of 33^2 or 17^2 points, Navier-Stokes (four fields, halo 4) on
// 33^2.
//
// As in column3.hip, the owner of a tile point (the finest leaf holding it on its own
// lattice, Sec. 2.2 and Sec. 2.5) only depends on its zone along each axis -- before the
// block, its first node, the first half, the middle node, the second half, its last node,
// beyond -- so a workgroup resolves the owners of 7^2 zones once, and a thread forms the
// addresses of its few tile points with one look-up each and has all their loads (every
// field) in flight together.
#include "device.hpp"

#include <hip/hip_runtime.h>
#include <algorithm>

namespace mrb {

namespace {

constexpr int NZ = 7;   // zones per axis

template <int BS>
__device__ __forceinline__ constexpr int zone_of(int t) {
  constexpr int M = (BS - 1) / 2;
  return t < 0 ? 0 : (t == 0 ? 1 : (t < M ? 2 : (t == M ? 3 : (t < 2 * M ? 4 : (t == 2 * M ? 5 : 6)))));
}

// Tile of a block's rows [y0, y0 + SY) (all columns) with a halo of HW, and the coarse
// lattice (even points up to HW + 3 beyond) that predictions read
template <int BS, int NF, int HW, int SY, int TPB>
struct Tile2 {
  static constexpr int NP = BS * BS, TW = BS + 2 * HW, TH = SY + 2 * HW, TSZ = TW * TH, H = HW + 3;
  static constexpr int RG = TPB / TW, NR = (TH + RG - 1) / RG;   // row groups, rows per thread
  static constexpr int ROWS = SY + 2 * H;   // rows of the owner table
  static constexpr int CW = (BS + 2 * H + 1) / 2, CH = (SY + 2 * H + 1) / 2, CSZ = CW * CH;
  static_assert(RG >= 1, "a tile row fits the workgroup");
  __device__ static __forceinline__ int first_even(int r0) { return (r0 - H + 1) & ~1; }
};

// Owner of the points of a row and a zone along x, the row folded into its base: rows
// y0 - H .. y0 + SY - 1 + H of a tile.  A coarser owner (sh 2) holds even points only.
template <int ROWS>
struct Rows2 {
  unsigned long long m[2][NZ];   // entries whose box holds the zone, per axis
  SEnt se[64];
  SEnt tab[ROWS * NZ];           // x zone fastest
};

// owners of the tile's rows (see zone_table in column3.hip)
template <int BS, int NF, int TPB, int ROWS>
__device__ __forceinline__ void row_table(Rows2<ROWS>& z, const BlockDesc& d, const NbEntry* ent, int stride, int first) {
  constexpr int M = (BS - 1) / 2, NP = BS * BS;
  const int lane = threadIdx.x & 63;
  NbEntry E{};
  if (lane < stride) E = ent[lane];
  const bool live = lane < d.n_ent;
  const int ext = E.dl > 0 ? M : (E.dl == 0 ? BS - 1 : 2 * (BS - 1));
  for (int q = threadIdx.x >> 6; q < 2 * NZ; q += TPB / 64) {
    const int a = q / NZ, k = q % NZ;
    const int t = k == 0 ? -1 : (k == 1 ? 0 : (k == 2 ? 1 : (k == 3 ? M : (k == 4 ? M + 1 : (k == 5 ? 2 * M : 2 * M + 1)))));
    const int l = t - (a == 0 ? E.o[0] : E.o[1]);
    const unsigned long long mm = __ballot(live && l >= 0 && l <= ext);
    if (lane == 0) z.m[a][k] = mm;
  }
  if (threadIdx.x < 64) {
    const int sh = 1 - E.dl;
    z.se[lane] = SEnt{E.slot * NF * NP - (((2 * E.o[0]) >> sh) + BS * ((2 * E.o[1]) >> sh)), sh};
  }
  __syncthreads();
  for (int p = threadIdx.x; p < ROWS * NZ; p += TPB) {
    const int ty = first + p / NZ;
    const unsigned long long c = z.m[0][p % NZ] & z.m[1][zone_of<BS>(ty)];
    const SEnt e = z.se[c ? 63 - __clzll((long long)c) : 0];
    z.tab[p] = SEnt{e.base + BS * ((2 * ty) >> e.sh), e.sh};
  }
  __syncthreads();
}

// This thread's tile points (column x, rows rg + i RG): values of every field, owned or
// predicted, in registers.  carr: LDS of 2 NF CSZ values (the coarse lattice and its odd
// points along x), used by blocks with coarser neighbours only.  load(address, field's offset)
// fetches a stored point, val(fetched, field) turns it into the tile's value.
template <int BS, int NF, int HW, int SY, int TPB, typename TT>
struct Gather2 {
  using T2 = Tile2<BS, NF, HW, SY, TPB>;
  TT v[T2::NR][NF];
  int x, rg;
  unsigned in;   // bit i: row i lies in the tile

  template <typename Z, typename LOAD, typename VAL>
  __device__ __forceinline__ void run(TT* carr, const Z& zn, int self, bool hasc, int y0, int cnty, const LOAD& load,
                                      const VAL& val) {
    constexpr int NR = T2::NR, TW = T2::TW, RG = T2::RG, CW = T2::CW, CSZ = T2::CSZ, NP = T2::NP, H = T2::H;
    using R = typename LOAD::type;   // what a load returns (u, and the slope where there is one)
    const int tid = threadIdx.x;
    x = tid % TW;
    rg = tid / TW;
    const int tx = x - HW, zx = zone_of<BS>(tx), cx0 = T2::first_even(0), cy0 = T2::first_even(y0);
    unsigned held = 0;
    in = 0;
    int ad[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int r = rg + RG * i, ty = y0 - HW + r;
      const SEnt E = zn.tab[zx + NZ * min(r + 3, T2::ROWS - 1)];
      const bool ok = rg < RG && r < cnty + 2 * HW, h = E.sh < 2 || ((tx | ty) & 1) == 0;
      if (ok) in |= 1u << i;
      if (h) held |= 1u << i;
      // (points nobody holds, and rows past the tile, load the block's first node)
      ad[i] = ok && h ? E.base + ((2 * tx) >> E.sh) : self;
    }
    R raw[NR][NF];
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int f = 0; f < NF; ++f) raw[i][f] = load(ad[i], f * NP);
    if (hasc) {
      // coarse-lattice points outside the tile
      for (int p = tid; p < CSZ; p += TPB) {
        const int sx = cx0 + 2 * (p % CW), sy = cy0 + 2 * (p / CW);
        const bool inside = sx >= -HW && sx < BS + HW && sy >= y0 - HW && sy < y0 + cnty + HW;
        if (inside || sx > BS - 1 + H || sy > y0 + cnty - 1 + H || sy < y0 - H) continue;
        const SEnt E = zn.tab[zone_of<BS>(sx) + NZ * (sy - y0 + H)];
        const int a = E.base + ((2 * sx) >> E.sh);
        R q[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) q[f] = load(a, f * NP);
#pragma unroll
        for (int f = 0; f < NF; ++f) carr[f * CSZ + p] = val(q[f], f);
      }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int f = 0; f < NF; ++f) v[i][f] = val(raw[i][f], f);
    if (!hasc) return;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int ty = y0 - HW + rg + RG * i;
      if (((in >> i) & 1u) && ((tx | ty) & 1) == 0) {
#pragma unroll
        for (int f = 0; f < NF; ++f) carr[f * CSZ + (tx - cx0) / 2 + CW * ((ty - cy0) / 2)] = v[i][f];
      }
    }
    __syncthreads();
    // the points between two coarse ones along x (entry i: between coarse points i + 1, i + 2)
    TT* codd = carr + NF * CSZ;
    for (int p = tid; p < NF * CSZ; p += TPB) {
      if (p % CW >= CW - 3) continue;
      codd[p] = P4(carr[p], carr[p + 1], carr[p + 2], carr[p + 3]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int ty = y0 - HW + rg + RG * i;
      if (((held >> i) & 1u) || !((in >> i) & 1u)) continue;
      const int dx = tx - cx0, dy = ty - cy0;
      const TT* c = ((tx & 1) ? codd + (dx - 3) / 2 : carr + dx / 2) + CW * ((ty & 1) ? (dy - 3) / 2 : dy / 2);
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const TT* q = c + f * CSZ;
        v[i][f] = (ty & 1) ? P4(q[0], q[CW], q[2 * CW], q[3 * CW]) : q[0];
      }
    }
  }
};

// sources: u alone, or u and the previous slope
struct LoadU {
  using type = double;
  const double* u;
  __device__ __forceinline__ type operator()(int i, int o) const { return (u + o)[(unsigned)i]; }
};
template <typename KT>
struct UK {
  double u;
  KT k;
};
template <typename KT>
struct LoadUK {
  using type = UK<KT>;
  const double* u;
  const KT* k;
  __device__ __forceinline__ type operator()(int i, int o) const { return type{(u + o)[(unsigned)i], (k + o)[(unsigned)i]}; }
};

// stage value from what was loaded, minus the field offset in FP32 tiles
template <typename TT>
struct StageValue {
  double alpha;
  const double* off;
  __device__ __forceinline__ TT fin(double y, int f) const {
    if constexpr (sizeof(TT) == 4) return (TT)(y - off[f]);
    else return y;
  }
  __device__ __forceinline__ TT operator()(double u, int f) const { return fin(u, f); }
  template <typename KT>
  __device__ __forceinline__ TT operator()(const UK<KT>& q, int f) const { return fin(q.u + alpha * (double)q.k, f); }
};

template <typename KT, typename F>
__device__ __forceinline__ void with_source(const StageArgs& A, const F& f) {
  if (A.stage == 1) f(LoadU{A.u});
  else f(LoadUK<KT>{A.u, (const KT*)A.kprev});
}

// ---------------------------------------------------------------------------
// Advection stage (constant velocity or swirl) of a whole block per workgroup, one (17^2) or
// four (33^2) tile points per thread.  Latency bound: the descriptor and entry row, the owner
// table, one round of loads, LDS, the update; so the workgroup size trades rounds against
// blocks in flight.  740 to 2,900 blocks of 33^2 FP64: 12.9 us a stage with 384 threads (13.7
// with 256, 15.8 with 576) against 22.3 us for a tile gathered point by point; 40 blocks of
// 17^2: 5.3 us with 448 (5.8 with 256) against 6.5 us.
// ---------------------------------------------------------------------------
template <int BS, int TPB, typename TT, typename KT>
__global__ void __launch_bounds__(TPB) k_stage2(StageArgs A) {
  constexpr int HW = 2;
  using G = Gather2<BS, 1, HW, BS, TPB, TT>;
  using T2 = typename G::T2;
  constexpr int TW = T2::TW, NP = T2::NP;
  __shared__ Rows2<T2::ROWS> zn;
  __shared__ double sw[4 * BS];
  __shared__ TT tile[T2::TSZ];
  __shared__ TT carr[2 * T2::CSZ];
  const XcdWork it(A.topo.h.n_blocks);   // one work item per workgroup
  if (!it.ok()) return;
  const int tid = threadIdx.x;
  const int b = A.order ? A.topo.list()[it.w] : it.w;
  const BlockDesc d = A.topo.blk()[b];
  const bool swirl = A.ph.kind == 1;
  if (swirl) {
    // table slices at the block's nodes: s2(x), s(x), s2(y), s(y)
    const int nl = A.lt.nl[d.level], shift = A.ph.jmax - d.level;
    for (int q = tid; q < 4 * BS; q += TPB) {
      const int k = q / BS, l = q % BS;
      int gg = (k < 2 ? d.c[0] : d.c[1]) * (BS - 1) + l;
      if (gg >= nl) gg -= nl;
      gg <<= shift;
      sw[q] = (k & 1) ? A.ph.s[gg] : A.ph.s2[gg];
    }
  }
  row_table<BS, 1, TPB>(zn, d, A.topo.nb(b), A.topo.h.nb_stride, -T2::H);
  const int base = d.slot * NP;
  G g;
  const StageValue<TT> val{A.alpha, A.off};
  with_source<KT>(A, [&](const auto& src) { g.run(carr, zn, base, d.n_coarse > 0, 0, BS, src, val); });
#pragma unroll
  for (int i = 0; i < T2::NR; ++i)
    if ((g.in >> i) & 1u) tile[g.x + TW * (g.rg + T2::RG * i)] = g.v[i][0];
  __syncthreads();
  TT r;
  if constexpr (sizeof(TT) == 8) r = A.lt.r[d.level];
  else r = A.lt.rf[d.level];
  const int node0 = base;
  constexpr int NU = (NP + TPB - 1) / TPB;
  double e1[NU], e2[NU], e3[NU], eu[NU];
  if (A.stage == 4) {
#pragma unroll
    for (int q = 0; q < NU; ++q) {
      const int p = node0 + min(tid + q * TPB, NP - 1);
      e1[q] = (double)((const KT*)A.k1)[p];
      e2[q] = (double)((const KT*)A.k2)[p];
      e3[q] = (double)((const KT*)A.k3)[p];
      eu[q] = A.u[p];
    }
  }
#pragma unroll
  for (int q = 0; q < NU; ++q) {
    const int p = tid + q * TPB;
    if (p >= NP) continue;
    const int ly = p / BS, lx = p - ly * BS;
    const TT* T = tile + lx + HW + TW * (ly + HW);
    const TT dx = D4(T[-2], T[-1], T[1], T[2], r);
    const TT dy = D4(T[-2 * TW], T[-TW], T[TW], T[2 * TW], r);
    TT kv;
    if (swirl) {
      const double U = (sw[lx] * sw[3 * BS + ly]) * A.cfac;
      const double W = -((sw[2 * BS + ly] * sw[BS + lx]) * A.cfac);
      kv = -(((TT)U * dx) + ((TT)W * dy));
    } else {
      TT acc = (TT)A.ph.c[0] * dx;
      acc = acc + (TT)A.ph.c[1] * dy;
      kv = -acc;
    }
    if (A.stage < 4) ((KT*)A.kout)[node0 + p] = (KT)kv;
    else A.unew[node0 + p] = eu[q] + A.h6 * ((e1[q] + (double)kv) + 2.0 * (e2[q] + e3[q]));
  }
}

// ---------------------------------------------------------------------------
// Navier-Stokes stage (primitive variables rho, u, v, p) of half or a third of a block per
// workgroup (SY rows, one node per thread).  The tile is FP64, CT the arithmetic type
// (see ns_fluxes in kernels.hip, whose operations these are, point by point).  p / rho is
// formed once per tile point (it had cost eight FP64 divisions per flux point), and a
// node's gradients, stresses and momentum factors pass from its fluxes to its right-hand
// side in registers.  Thirds, mixed, are bound by vector instructions (3,800 of a wave a third,
// 70% of a compute unit's cycles), LDS (52%, a quarter of it bank conflicts) and memory (260 MB,
// 50 us) together, overlapped by the two to four workgroups that fit a compute unit's LDS; FP64
// issues half of the time and waits for LDS as long.  2,944 blocks on five levels: 89 us a stage
// mixed against 244 us for whole blocks of 256 threads; 1,024 blocks FP64: 42 against 76 us.
// ---------------------------------------------------------------------------
constexpr int NB = 33;
constexpr int ns_parts(int sy) { return (NB + sy - 1) / sy; }

template <typename CT>
__device__ __forceinline__ CT D4d(double um2, double um1, double up1, double up2, CT r) {
  if constexpr (sizeof(CT) == 8) return D4(um2, um1, up1, up2, r);
  else return (8.0f * (CT)(up1 - um1) - (CT)(up2 - um2)) * r;
}

// SHARE: the coarse lattice lies where the tile comes to lie and the heat fluxes take the place
// of the normal stresses once these are read, three barriers more, for one workgroup more in the
// compute unit's LDS (thirds of blocks, mixed: 39 KB instead of 53)
template <typename KT, typename CT, bool SHARE, int SY, int T>
struct NsLds {
  using T2 = Tile2<NB, 4, 4, SY, T>;
  static constexpr int FX = NB + 4, FY = SY + 4;            // flux points -2 .. 34, -2 .. cnt + 1
  static constexpr int NXX = FX * SY, NYY = NB * FY, NXY = FX * FY;
  static constexpr size_t tile = sizeof(double) * T2::TSZ * 5;   // four fields and p / rho
  static constexpr size_t flux = sizeof(CT) * ((SHARE ? 1 : 2) * (NXX + NYY) + NXY), lat = sizeof(double) * 2 * 4 * T2::CSZ;
  static constexpr size_t bytes = tile + (SHARE || flux > lat ? flux : lat);
  static_assert(lat <= tile, "the lattice is dead before the tile (SHARE) or the fluxes are written");
};

template <typename KT, typename CT, bool SHARE, int SY, int T>
__global__ void __launch_bounds__(T) k_stage_ns(StageArgs A) {
  using L = NsLds<KT, CT, SHARE, SY, T>;
  using G = Gather2<NB, 4, 4, SY, T, double>;
  using T2 = typename G::T2;
  constexpr int TW = T2::TW, TSZ = T2::TSZ, NP = T2::NP, HW = 4, FX = L::FX;
  __shared__ Rows2<T2::ROWS> zn;
  extern __shared__ __align__(16) char smem[];
  double* tile = reinterpret_cast<double*>(smem);
  double* Tt = tile + 4 * TSZ;                       // p / rho
  double* carr = SHARE ? tile : Tt + TSZ;
  CT* txy = reinterpret_cast<CT*>(Tt + TSZ);         // x -2..34, y -2..18
  CT* txx = txy + L::NXY;                            // x -2..34, y 0..16
  CT* tyy = txx + L::NXX;                            // x 0..32, y -2..18
  CT* qx = SHARE ? txx : tyy + L::NYY;
  CT* qy = SHARE ? tyy : qx + L::NXX;
  const XcdWork it(ns_parts(SY) * A.topo.h.n_blocks);       // one work item per workgroup
  if (!it.ok()) return;
  const int tid = threadIdx.x, part = it.w % ns_parts(SY);
  const int b = A.order ? A.topo.list()[it.w / ns_parts(SY)] : it.w / ns_parts(SY);
  const BlockDesc d = A.topo.blk()[b];
  const int y0 = part * SY, cnty = min(SY, NB - y0);
  row_table<NB, 4, T>(zn, d, A.topo.nb(b), A.topo.h.nb_stride, y0 - T2::H);
  const int base = d.slot * 4 * NP;
  {
    G g;
    const StageValue<double> val{A.alpha, A.off};
    with_source<KT>(A, [&](const auto& src) { g.run(carr, zn, base, d.n_coarse > 0, y0, cnty, src, val); });
    if (SHARE && d.n_coarse > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < T2::NR; ++i) {
      if (!((g.in >> i) & 1u)) continue;
      const int q = g.x + TW * (g.rg + T2::RG * i);
#pragma unroll
      for (int f = 0; f < 4; ++f) tile[f * TSZ + q] = g.v[i][f];
      Tt[q] = g.v[i][3] / g.v[i][0];
    }
  }
  __syncthreads();
  CT mu, kap, gam, c23, r;
  mu = (CT)A.ph.mu;
  kap = (CT)A.ph.kap;
  gam = (CT)A.ph.gamma;
  c23 = (CT)(2.0 / 3.0);
  if constexpr (sizeof(CT) == 8) r = A.lt.r[d.level];
  else r = A.lt.rf[d.level];
  const double *fr = tile, *fu = tile + TSZ, *fv = tile + 2 * TSZ, *fp = tile + 3 * TSZ;
  auto Dx = [&](const double* F, int q) { return D4d<CT>(F[q - 2], F[q - 1], F[q + 1], F[q + 2], r); };
  auto Dy = [&](const double* F, int q) { return D4d<CT>(F[q - 2 * TW], F[q - TW], F[q + TW], F[q + 2 * TW], r); };
  // Stresses and heat flux, each where a derivative along x or y reads it: at the thread's
  // own node, whose velocity gradients, stresses and momentum factors stay in registers for
  // the right-hand side, then at the points beside the region (two per side and row).
  static_assert(NB * SY <= T, "one region node per thread");
  const int nn = NB * cnty;
  const bool mine = tid < nn;
  const int ly = mine ? tid / NB : 0, lx = mine ? tid - ly * NB : 0;
  const int q = lx + HW + TW * (ly + HW);
  const int wx = lx + 2 + FX * ly, wy = lx + NB * (ly + 2), wc = lx + 2 + FX * (ly + 2);
  CT ux, uy, vx, vy, sxx, syy, sxy;
  double um[4], vm[4];   // u along x, v along y (the momentum derivatives' factors)
  if (mine) {
    um[0] = fu[q - 2]; um[1] = fu[q - 1]; um[2] = fu[q + 1]; um[3] = fu[q + 2];
    vm[0] = fv[q - 2 * TW]; vm[1] = fv[q - TW]; vm[2] = fv[q + TW]; vm[3] = fv[q + 2 * TW];
    ux = D4d<CT>(um[0], um[1], um[2], um[3], r);
    vy = D4d<CT>(vm[0], vm[1], vm[2], vm[3], r);
    uy = Dy(fu, q);
    vx = Dx(fv, q);
    const CT div = ux + vy;
    sxx = mu * (CT(2) * ux - c23 * div);
    syy = mu * (CT(2) * vy - c23 * div);
    sxy = mu * (uy + vx);
    txx[wx] = sxx;
    tyy[wy] = syy;
    txy[wc] = sxy;
  }
  // beside the region along x (xs) or y
  const int sp = T - 1 - tid, nside = 4 * cnty;    // the last waves have fewer own nodes
  const bool side = sp < nside + 4 * NB, xs = sp < nside;
  const int sk = xs ? sp % 4 : (sp - nside) / NB;
  const int fx = xs ? (sk < 2 ? sk - 2 : NB - 2 + sk) : (sp - nside) % NB;
  const int fy = xs ? sp / 4 : (sk < 2 ? sk - 2 : cnty - 2 + sk);
  const int s = fx + HW + TW * (fy + HW), ws = xs ? fx + 2 + FX * fy : fx + NB * (fy + 2);
  if (side) {
    const CT ax = Dx(fu, s), ay = Dy(fu, s), bx = Dx(fv, s), by = Dy(fv, s);
    const CT div = ax + by;
    txy[fx + 2 + FX * (fy + 2)] = mu * (ay + bx);
    if (xs) txx[ws] = mu * (CT(2) * ax - c23 * div);
    else tyy[ws] = mu * (CT(2) * by - c23 * div);
  }
  auto heat = [&]() {
    if (mine) {
      qx[wx] = -(kap * Dx(Tt, q));
      qy[wy] = -(kap * Dy(Tt, q));
    }
    if (side) {
      if (xs) qx[ws] = -(kap * Dx(Tt, s));
      else qy[ws] = -(kap * Dy(Tt, s));
    }
  };
  auto dxw = [&](const CT* w, int i) { return D4(w[i - 2], w[i - 1], w[i + 1], w[i + 2], r); };
  auto dyw = [&](const CT* w, int i, int t) { return D4(w[i - 2 * t], w[i - t], w[i + t], w[i + 2 * t], r); };
  if constexpr (!SHARE) heat();
  __syncthreads();
  CT dtxx, dtxy_y, dtxy_x, dtyy;
  if (mine) {
    dtxx = dxw(txx, wx);
    dtyy = dyw(tyy, wy, NB);
    dtxy_y = dyw(txy, wc, FX);
    dtxy_x = dxw(txy, wc);
  }
  if constexpr (SHARE) {
    __syncthreads();
    heat();
    __syncthreads();
  }
  if (mine) {
    const size_t node = (size_t)base + lx + NB * (y0 + ly);
    const CT rho = (CT)fr[q], uu = (CT)fu[q], vv = (CT)fv[q], pp = (CT)fp[q];
    const CT px = Dx(fp, q), py = Dy(fp, q);
    const CT dmx = D4d<CT>(fr[q - 2] * um[0], fr[q - 1] * um[1], fr[q + 1] * um[2], fr[q + 2] * um[3], r);
    const CT dmy = D4d<CT>(fr[q - 2 * TW] * vm[0], fr[q - TW] * vm[1], fr[q + TW] * vm[2], fr[q + 2 * TW] * vm[3], r);
    const CT dqx = dxw(qx, wx), dqy = dyw(qy, wy, NB);
    CT kv[4];
    kv[0] = -(dmx + dmy);
    kv[1] = -(uu * ux + vv * uy) - px / rho + (dtxx + dtxy_y) / rho;
    kv[2] = -(uu * vx + vv * vy) - py / rho + (dtxy_x + dtyy) / rho;
    const CT phi = sxx * ux + sxy * (uy + vx) + syy * vy;
    const CT divq = dqx + dqy;
    kv[3] = -(uu * px + vv * py) - gam * pp * (ux + vy) + (gam - CT(1)) * (phi - divq);
    if (A.stage < 4) {
#pragma unroll
      for (int f = 0; f < 4; ++f) ((KT*)A.kout + f * NP)[node] = (KT)kv[f];
    } else {
      // The update's operands, requested together once the right-hand side's registers are
      // free (held through it they cost more in resident waves than their latency does)
      __builtin_amdgcn_sched_barrier(0);
      KT e1[4], e2[4], e3[4];
      double eu[4];
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        e1[f] = ((const KT*)A.k1 + f * NP)[node];
        e2[f] = ((const KT*)A.k2 + f * NP)[node];
        e3[f] = ((const KT*)A.k3 + f * NP)[node];
        eu[f] = (A.u + f * NP)[node];
      }
#pragma unroll
      for (int f = 0; f < 4; ++f)
        (A.unew + f * NP)[node] = eu[f] + A.h6 * (((double)e1[f] + (double)kv[f]) + 2.0 * ((double)e2[f] + (double)e3[f]));
    }
  }
}

// ---------------------------------------------------------------------------
// Shock-capturing filter after a time step (formulas at FilterArgs), half or a third of a
// block per workgroup: per axis the pressure sensor of one point more than the region on either
// side, then the switched second-order fluxes.  Vector instructions fill 64% of a compute
// unit's cycles (two divisions a sensor), LDS 39%.  2,944 blocks: 68 us (205 MB of block data,
// 3.0 TB/s) against 149 us for whole blocks of 256 threads, one per compute unit.
// ---------------------------------------------------------------------------
constexpr int FHW = 3;   // p is read up to 3 beyond the region, the other fields 1

template <int SY, int T>
struct FilterLds {
  using T2 = Tile2<NB, 4, FHW, SY, T>;
  static constexpr int NX = (NB + 2) * SY, NY = NB * (SY + 2);
  static constexpr size_t tile = sizeof(double) * 4 * T2::TSZ, sens = sizeof(double) * (NX + NY),
                          lat = sizeof(double) * 2 * 4 * T2::CSZ;
  static constexpr size_t bytes = tile + (sens > lat ? sens : lat);   // (the lattice is dead before the sensors)
};

struct FilterValue {
  __device__ __forceinline__ double operator()(double u, int) const { return u; }
};

template <int SY, int T>
__global__ void __launch_bounds__(T) k_filter2(FilterArgs A) {
  using G = Gather2<NB, 4, FHW, SY, T, double>;
  using T2 = typename G::T2;
  constexpr int TW = T2::TW, TSZ = T2::TSZ, NP = T2::NP, SXW = NB + 2;
  __shared__ Rows2<T2::ROWS> zn;
  extern __shared__ __align__(16) char smem[];
  double* tile = reinterpret_cast<double*>(smem);
  double* carr = tile + 4 * TSZ;
  double* sx = carr;                     // sensor along x at x = -1..33, y = 0..cnt-1
  double* sy = sx + FilterLds<SY, T>::NX;       // sensor along y at x = 0..32, y = -1..cnt
  const XcdWork it(ns_parts(SY) * A.topo.h.n_blocks);
  if (!it.ok()) return;
  const int tid = threadIdx.x, part = it.w % ns_parts(SY), b = it.w / ns_parts(SY);
  const BlockDesc d = A.topo.blk()[b];
  const int y0 = part * SY, cnty = min(SY, NB - y0);
  row_table<NB, 4, T>(zn, d, A.topo.nb(b), A.topo.h.nb_stride, y0 - T2::H);
  const int base = d.slot * 4 * NP;
  {
    G g;
    g.run(carr, zn, base, d.n_coarse > 0, y0, cnty, LoadU{A.u}, FilterValue{});
#pragma unroll
    for (int i = 0; i < T2::NR; ++i) {
      if (!((g.in >> i) & 1u)) continue;
#pragma unroll
      for (int f = 0; f < 4; ++f) tile[f * TSZ + g.x + TW * (g.rg + T2::RG * i)] = g.v[i][f];
    }
  }
  __syncthreads();
  const double* P = tile + 3 * TSZ;
  auto sens = [&](int q, int st) -> double {
    auto Dp = [&](int c) { return ((-P[c + st] + 2.0 * P[c]) - P[c - st]) * 0.25; };
    const double d0 = Dp(q), dp = Dp(q + st), dm = Dp(q - st);
    const double m = ((d0 - dp) * (d0 - dp) + (d0 - dm) * (d0 - dm)) * 0.5;
    const double p0 = P[q];
    const double r = m / (p0 * p0) + 1e-16;
    const double sv = 1.0 - A.rth / r;
    return sv > 0.0 ? sv : 0.0;
  };
  for (int p = tid; p < SXW * cnty + NB * (cnty + 2); p += T) {
    if (p < SXW * cnty) {
      const int y = p / SXW, x = p - y * SXW;
      sx[p] = sens(x - 1 + FHW + TW * (y + FHW), 1);
    } else {
      const int r = p - SXW * cnty, y = r / NB, x = r - y * NB;
      sy[r] = sens(x + FHW + TW * (y - 1 + FHW), TW);
    }
  }
  __syncthreads();
  static_assert(NB * SY <= T, "one node per thread");
  if (tid < NB * cnty) {
    const int y = tid / NB, x = tid - y * NB;
    const double sx0 = sx[(x + 1) + SXW * y], sy0 = sy[x + NB * (y + 1)];
    const double sxm = (sx[x + SXW * y] + sx0) * 0.5, sxp = (sx0 + sx[(x + 2) + SXW * y]) * 0.5;
    const double sym = (sy[x + NB * y] + sy0) * 0.5, syp = (sy0 + sy[x + NB * (y + 2)]) * 0.5;
    const double* Q = tile + x + FHW + TW * (y + FHW);
    double* out = A.unew + (size_t)base + x + NB * (y0 + y);
#pragma unroll
    for (int f = 0; f < 4; ++f, Q += TSZ) {
      const double q = Q[0];
      const double fxp = -(Q[1] - q) * 0.25, fxm = -(q - Q[-1]) * 0.25;
      const double fyp = -(Q[TW] - q) * 0.25, fym = -(q - Q[-TW]) * 0.25;
      out[f * NP] = q - ((sxp * fxp - sxm * fxm) + (syp * fyp - sym * fym));
    }
  }
}

// ---------------------------------------------------------------------------
// Prediction over a block's 33^2 (17^2) points from an EW^2 array of every second one and one
// more around them (the even points of the block, or the parent's points under a child): the
// points between two along x are formed once (od), a point off the rows combines four of them.
// ---------------------------------------------------------------------------
template <int BS>
struct Half2 {
  static constexpr int M = (BS - 1) / 2, EW = M + 3, NE = EW * EW, NOUT = 4 * EW - 4;
};

template <int BS, int NF, int TPB>
__device__ __forceinline__ void fill_odd2(double* od, const double* ev) {
  constexpr int EW = Half2<BS>::EW, M = Half2<BS>::M;
  for (int p = threadIdx.x; p < NF * EW * M; p += TPB) {
    const double* e = ev + p % M + EW * (p / M);
    od[p % M + EW * (p / M)] = P4(e[0], e[1], e[2], e[3]);
  }
}

template <int BS>
__device__ __forceinline__ double half_value(const double* ev, const double* od, int x, int y) {
  constexpr int EW = Half2<BS>::EW;
  const double* c = ((x & 1) ? od + x / 2 : ev + x / 2 + 1) + EW * (y / 2);
  return (y & 1) ? P4(c[0], c[EW], c[2 * EW], c[3 * EW]) : c[EW];
}

// ---------------------------------------------------------------------------
// Analysis of a whole block per workgroup (operations and stores as k_mr in kernels.hip):
// a thread owns a few of the block's points, LDS holds only the even points and their odd
// neighbours along x (6 KB a field, so that eight blocks of one field share a compute unit).
// Bound by vector instructions on large grids (80% of a compute unit's cycles; 4,096 blocks,
// 36 MB: 15.6 us against 39.7 for a tile in LDS) and by its chain of loads on small ones (740
// to 2,900 blocks: 7.4 against 12.9 us; four fields, 740 to 2,900 blocks on five levels: 21.6
// against 40.4 us).
// ---------------------------------------------------------------------------
template <int BS, int NF, int TPB>
__global__ void __launch_bounds__(TPB) k_mr2(MrArgs A) {
  using HB = Half2<BS>;
  constexpr int NP = BS * BS, EW = HB::EW, NE = HB::NE, RG = TPB / BS, NR = (BS + RG - 1) / RG, ROWS = BS + 4;
  static_assert(TPB >= HB::NOUT, "one even point outside the block per thread");
  __shared__ Rows2<ROWS> zn;
  __shared__ double ev[NF * NE], od[NF * NE];
  __shared__ double red[TPB / 64][NF];
  const XcdWork it(A.topo.h.n_blocks);   // one work item per workgroup
  if (!it.ok()) return;
  const int tid = threadIdx.x, b = it.w;
  const BlockDesc d = A.topo.blk()[b];
  const int sm = A.smap ? A.smap[b] : -1;
  row_table<BS, NF, TPB>(zn, d, A.topo.nb(b), A.topo.h.nb_stride, -2);
  const int base = d.slot * NF * NP;
  const int x = tid % BS, rg = tid / BS, zx = zone_of<BS>(x);
  double v[NR][NF];
  unsigned in = 0, fine = 0;   // rows of the block; those a finer neighbour owns
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int y = rg + RG * i;
    const bool ok = rg < RG && y < BS;
    const SEnt E = zn.tab[zx + NZ * (min(y, BS - 1) + 2)];
    if (ok) in |= 1u << i;
    if (ok && E.sh == 0) fine |= 1u << i;
    const int ad = ok ? E.base + ((2 * x) >> E.sh) : base;
#pragma unroll
    for (int f = 0; f < NF; ++f) v[i][f] = (A.u + f * NP)[(unsigned)ad];
  }
  double ov[NF];
  int oi = 0;
  if (tid < HB::NOUT) {
    // even points outside the block: the first and last rows, then the first and last columns
    const int r = tid - 2 * EW;
    const int cx = tid < 2 * EW ? tid % EW : (r & 1) * (EW - 1), cy = tid < 2 * EW ? (tid / EW) * (EW - 1) : 1 + r / 2;
    const int sx = 2 * cx - 2, sy = 2 * cy - 2;
    const SEnt E = zn.tab[zone_of<BS>(sx) + NZ * (sy + 2)];
    const int ad = E.base + ((2 * sx) >> E.sh);
    oi = cx + EW * cy;
#pragma unroll
    for (int f = 0; f < NF; ++f) ov[f] = (A.u + f * NP)[(unsigned)ad];
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int y = rg + RG * i;
    if (((in >> i) & 1u) && ((x | y) & 1) == 0) {
#pragma unroll
      for (int f = 0; f < NF; ++f) ev[f * NE + x / 2 + 1 + EW * (y / 2 + 1)] = v[i][f];
    }
    // redundant nodes owned by a finer neighbour: store the synchronised value
    if ((fine >> i) & 1u) {
#pragma unroll
      for (int f = 0; f < NF; ++f) (A.u + f * NP)[(unsigned)(base + x + BS * y)] = v[i][f];
    }
  }
  if (tid < HB::NOUT) {
#pragma unroll
    for (int f = 0; f < NF; ++f) ev[f * NE + oi] = ov[f];
  }
  __syncthreads();
  fill_odd2<BS, NF, TPB>(od, ev);
  __syncthreads();
  // |details| as unsigned bits, whose maximum NaN propagates through (zero at even points)
  unsigned long long m[NF] = {};
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int y = rg + RG * i;
    if (!((in >> i) & 1u) || ((x | y) & 1) == 0) continue;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const double dv = fabs(v[i][f] - half_value<BS>(ev + f * NE, od + f * NE, x, y));
      m[f] = umax64(m[f], (unsigned long long)__double_as_longlong(dv));
    }
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const double w = wave_nanmax(__longlong_as_double((long long)m[f]));
    if ((tid & 63) == 0) red[tid >> 6][f] = w;
  }
  __syncthreads();
  if (tid == 0) {
    bool coarse = d.level > 1;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      double w = red[0][f];
#pragma unroll
      for (int q = 1; q < TPB / 64; ++q) w = nanmax(w, red[q][f]);
      A.maxd[(size_t)b * NF + f] = w;
      if (!(w < A.thr[f])) coarse = false;
    }
    A.flags[b] = coarse ? (int8_t)-1 : (int8_t)0;
  }
  if (sm >= 0) {
    // the block is child `ch` of a speculated family: the mother's nodes it supplies (see
    // k_mr3 in column3.hip)
    const int ch = sm & 7, mbase = (sm >> 3) * NF * NP;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int y = rg + RG * i;
      if (!((in >> i) & 1u) || ((x | y) & 1) || ((ch & 1) && x == 0) || ((ch & 2) && y == 0)) continue;
      const int mn = x / 2 + (ch & 1) * HB::M + BS * (y / 2 + ((ch >> 1) & 1) * HB::M);
      const bool from_tile = !(x == 0 || y == 0 || x == BS - 1 || y == BS - 1) || ((fine >> i) & 1u);
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        double* u = A.u + f * NP;
        u[(unsigned)(mbase + mn)] = from_tile ? v[i][f] : u[(unsigned)(base + x + BS * y)];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Refinement, one workgroup per child of a parent (the child's nodes take the
// synchronised value at level l+1: a finer neighbour's stored value where one holds the node,
// else the parent's value at even nodes or its prediction at odd ones):
// LDS holds the synchronised parent points the child needs, its half of the parent and one
// point around.  Bound by its stores.  740 to 2,900 blocks of one field: 11.6 us against 15.1
// for a tile; of four fields: 27.0 against 43.6 us.
// ---------------------------------------------------------------------------
template <int BS, int NF, int TPB>
__global__ void __launch_bounds__(TPB) k_refine2(RefineArgs A) {
  using HB = Half2<BS>;
  constexpr int NP = BS * BS, M = HB::M, EW = HB::EW, NE = HB::NE, RG = TPB / BS, NR = (BS + RG - 1) / RG;
  constexpr int LW = M / 2 + 5, NL = LW * LW, ROWS = 2 * LW - 1;   // the parent's coarse lattice
  constexpr int RE = (NE + TPB - 1) / TPB;
  static_assert(TPB >= NL && TPB >= 2 * EW, "one lattice point per thread");
  __shared__ Rows2<ROWS> zn;
  __shared__ double ev[NF * NE], od[NF * NE];   // od first holds the lattice
  static_assert(NL <= NE, "the lattice fits od");
  const XcdWork it(A.topo.h.n_ref * 4);   // one work item per workgroup
  if (!it.ok()) return;
  const int tid = threadIdx.x, ri = it.w >> 2, ch = it.w & 3, bx = ch & 1, by = ch >> 1;
  const BlockDesc d = A.topo.pblk()[ri];
  const int obase = A.topo.ref()[ri].child[ch] * NF * NP;
  const int l0 = M * bx - 4, l1 = M * by - 4;   // first lattice point
  row_table<BS, NF, TPB>(zn, d, A.topo.pnb(ri), A.topo.h.pnb_stride, l1);
  // finer entries come last in the list
  const bool hasc = d.n_coarse > 0, hasf = d.n_ent > 0 && zn.se[d.n_ent - 1].sh == 0;
  const int base = d.slot * NF * NP;
  auto owner = [&](int sx, int sy) { return zn.tab[zone_of<BS>(sx) + NZ * (sy - l1)]; };
  double pv[RE][NF];
#pragma unroll
  for (int q = 0; q < RE; ++q) {
    const int p = min(tid + q * TPB, NE - 1);
    const int sx = l0 + 3 + p % EW, sy = l1 + 3 + p / EW;
    const SEnt E = owner(sx, sy);
    const int ad = E.sh < 2 || ((sx | sy) & 1) == 0 ? E.base + ((2 * sx) >> E.sh) : base;   // (unheld: predicted below)
#pragma unroll
    for (int f = 0; f < NF; ++f) pv[q][f] = (A.u + f * NP)[(unsigned)ad];
  }
  double lv[NF];
  if (hasc) {
    const int p = min(tid, NL - 1), sx = l0 + 2 * (p % LW), sy = l1 + 2 * (p / LW);
    const SEnt E = owner(sx, sy);
    const int ad = E.base + ((2 * sx) >> E.sh);
#pragma unroll
    for (int f = 0; f < NF; ++f) lv[f] = (A.u + f * NP)[(unsigned)ad];
  }
  const int x = tid % BS, rg = tid / BS;
  // odd nodes of the parent's boundary that a finer leaf holds take its value: their address
  int fa[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) fa[i] = -1;
  if (hasf) {
    // zone of a fine coordinate Q (parent coordinate Q / 2)
    auto fz = [](int Q) { return Q == 0 ? 1 : (Q < BS - 1 ? 2 : (Q == BS - 1 ? 3 : (Q < 2 * (BS - 1) ? 4 : 5))); };
    const int lane = tid & 63;
    const unsigned long long fmask = __ballot(lane < d.n_ent && zn.se[lane].sh == 0);
    const int Qx = x + (BS - 1) * bx;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int y = min(rg + RG * i, BS - 1), Qy = y + (BS - 1) * by;
      const unsigned long long c = zn.m[0][fz(Qx)] & zn.m[1][fz(Qy)] & fmask;
      const bool rim = Qx == 0 || Qx == 2 * (BS - 1) || Qy == 0 || Qy == 2 * (BS - 1);
      if (rim && ((x | y) & 1) && c) fa[i] = zn.se[__ffsll((long long)c) - 1].base + Qx + BS * Qy;
    }
  }
#pragma unroll
  for (int q = 0; q < RE; ++q) {
    const int p = tid + q * TPB;
    if (p < NE) {
#pragma unroll
      for (int f = 0; f < NF; ++f) ev[f * NE + p] = pv[q][f];
    }
  }
  if (hasc) {
    if (tid < NL) {
#pragma unroll
      for (int f = 0; f < NF; ++f) od[f * NE + tid] = lv[f];
    }
    __syncthreads();
    // parent points inside a coarser neighbour, off its lattice: only the row and the column
    // one point outside the parent can hold any
    if (tid < 2 * EW) {
      const bool col = tid >= EW;
      const int k = tid % EW, e0 = bx ? EW - 1 : 0, e1 = by ? EW - 1 : 0;
      const int c0 = col ? e0 : k, c1 = col ? k : e1;
      const int sx = l0 + 3 + c0, sy = l1 + 3 + c1;
      if (owner(sx, sy).sh == 2 && ((sx | sy) & 1)) {
        const int t0 = c0 + 3, t1 = c1 + 3;   // from the lattice's first point
        const int px = t0 & 1, py = t1 & 1;
        const double* c = od + (px ? (t0 - 3) / 2 : t0 / 2) + LW * (py ? (t1 - 3) / 2 : t1 / 2);
#pragma unroll
        for (int f = 0; f < NF; ++f, c += NE) {
          auto row = [&](const double* q) { return px ? P4(q[0], q[1], q[2], q[3]) : q[0]; };
          ev[f * NE + c0 + EW * c1] = py ? P4(row(c), row(c + LW), row(c + 2 * LW), row(c + 3 * LW)) : row(c);
        }
      }
    }
  }
  __syncthreads();
  fill_odd2<BS, NF, TPB>(od, ev);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int y = rg + RG * i;
    if (rg >= RG || y >= BS) continue;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      double* u = A.u + f * NP;
      double w = half_value<BS>(ev + f * NE, od + f * NE, x, y);
      if (fa[i] >= 0) w = u[(unsigned)fa[i]];
      u[(unsigned)(obase + x + BS * y)] = w;
    }
  }
}

// one workgroup per work item (XcdWork deals them out from a multiple of 8)
template <typename K, typename Arg>
hipError_t go2(K kern, int items, size_t lds, int threads, hipStream_t st, const Arg& a) {
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(std::max(8, (items + 7) & ~7)), dim3(threads), lds, st, a);
  return hipGetLastError();
}

template <typename KT, typename CT, bool SHARE, int SY, int T>
hipError_t go_ns(int n, hipStream_t st, const StageArgs& a) {
  return go2(k_stage_ns<KT, CT, SHARE, SY, T>, ns_parts(SY) * n, NsLds<KT, CT, SHARE, SY, T>::bytes, T, st, a);
}

}  // namespace

hipError_t launch_stage2(const Shape& s, int precision, int ncu, const StageArgs& a, hipStream_t st) {
  const int n = a.topo.h.n_blocks;
  if (s.nf == 4) {
    if (zone_form(s, precision, n, ncu).parts == 3) {
      if (precision == 0) return go_ns<double, double, false, 11, kNsThirds>(n, st, a);
      return go_ns<float, float, true, 11, kNsThirdsMixed>(n, st, a);
    }
    if (precision == 0) return go_ns<double, double, false, 17, kNsThreads>(n, st, a);
    return go_ns<float, float, false, 17, kNsThreads>(n, st, a);
  }
  if (s.bs == 33) {
    if (precision == 0) return go2(k_stage2<33, 384, double, double>, n, 0, 384, st, a);
    return go2(k_stage2<33, 384, float, float>, n, 0, 384, st, a);
  }
  if (precision == 0) return go2(k_stage2<17, 448, double, double>, n, 0, 448, st, a);
  return go2(k_stage2<17, 448, float, float>, n, 0, 448, st, a);
}

// The analysis takes 256 threads a block unless tuning asks for more (4,096 blocks of 33^2:
// 15.6 us with 256, 20.3 with 512, 33.6 with 576; 100 blocks of four fields: 10.9, 10.1 with
// 512, 12.8 with 1,024), the one round of 17^2 points a multiple of 64 that holds them; the
// refinement 256 (one field: 11.6 us against 12.2 with 512) or 512 (four: 27.0 against 27.6
// with 256 and 36.9 with 576).
hipError_t launch_mr2(const Shape& s, int tpb, const MrArgs& a, hipStream_t st) {
  const int n = a.topo.h.n_blocks;
  if (s.bs == 17) return tpb == 256 ? go2(k_mr2<17, 1, 320>, n, 0, 320, st, a) : hipErrorInvalidValue;
  if (tpb == 256) return s.nf == 4 ? go2(k_mr2<33, 4, 256>, n, 0, 256, st, a) : go2(k_mr2<33, 1, 256>, n, 0, 256, st, a);
  if (tpb == 512) return s.nf == 4 ? go2(k_mr2<33, 4, 512>, n, 0, 512, st, a) : go2(k_mr2<33, 1, 512>, n, 0, 512, st, a);
  if (tpb == 1024)
    return s.nf == 4 ? go2(k_mr2<33, 4, 1024>, n, 0, 1024, st, a) : go2(k_mr2<33, 1, 1024>, n, 0, 1024, st, a);
  return hipErrorInvalidValue;
}

hipError_t launch_refine2(const Shape& s, const RefineArgs& a, hipStream_t st) {
  const int n = 4 * a.topo.h.n_ref;
  if (s.nf == 4) return go2(k_refine2<33, 4, 512>, n, 0, 512, st, a);
  if (s.bs == 33) return go2(k_refine2<33, 1, 256>, n, 0, 256, st, a);
  return go2(k_refine2<17, 1, 320>, n, 0, 320, st, a);
}

// (halves and thirds as in the stage: thirds are 2% faster on 2,944 blocks, 68 us, and 5% on
// 1,024, 25 us)
hipError_t launch_filter(int ncu, const FilterArgs& a, hipStream_t st) {
  const int n = a.topo.h.n_blocks;
  if (n > ncu) return go2(k_filter2<11, 448>, ns_parts(11) * n, FilterLds<11, 448>::bytes, 448, st, a);
  return go2(k_filter2<17, kNsThreads>, ns_parts(17) * n, FilterLds<17, kNsThreads>::bytes, kNsThreads, st, a);
}

}  // namespace mrb
