// Kernels on whole 3D blocks of 17^3 points (one field, halo 2): the RK stage, the
// multiresolution analysis and the refinement, a column along z per thread (gfx950).
//
// The owner of a tile point -- the finest leaf holding it on its own lattice (Sec. 2.2,
// Sec. 2.5) -- only depends on the point's zone along each axis: before the block, its
// first node, the first half, the middle node, the second half, its last node, beyond
// (every neighbour's box starts and ends on one of the three nodes named).  So a
// workgroup resolves the owners of the 7^3 zones once (one zone per thread) instead of
// the owners of 21^3 points: a thread keeps its (x, y) zone and walks z with one table
// look-up per zone and a multiply-add per point.
//
// Neighbours along z are the thread's own registers; only the x and y neighbours go
// through LDS.  Predictions (Sec. 2.3, tensor product x -> y -> z) reuse the same order:
// a column forms its x-y predictions once per coarse plane and combines them along z.
#include "device.hpp"

#include <hip/hip_runtime.h>
#include <algorithm>

namespace mrb {

namespace {

constexpr int B = 17, NP = B * B * B;   // points per axis and block
constexpr int NZ = 7;                   // zones per axis

__device__ __forceinline__ constexpr int zone_of(int t) {
  return t < 0 ? 0 : (t == 0 ? 1 : (t < 8 ? 2 : (t == 8 ? 3 : (t < 16 ? 4 : (t == 16 ? 5 : 6)))));
}

struct Zones {
  unsigned long long m[3][NZ];   // entries whose box holds the zone, per axis
  SEnt se[64];
  SEnt tab[NZ * NZ * NZ];        // owner of each zone, x fastest
};

// The owners of a block's zones: the highest entry (finer ones come last) holding a zone
// along all three axes.  A coarser owner holds the zone's even points only (its lattice);
// the others have no holder and are predicted.  A workgroup of whole waves, at least 343
// threads for one table entry each; the entry row is loaded without waiting for the
// descriptor (`stride` entries are in bounds, those past n_ent are unused).
template <int TPB>
__device__ __forceinline__ void zone_table(Zones& z, const BlockDesc& d, const NbEntry* ent, int stride) {
  const int lane = threadIdx.x & 63;
  NbEntry E{};
  if (lane < stride) E = ent[lane];
  const bool live = lane < d.n_ent;
  const int ext = E.dl > 0 ? (B - 1) / 2 : (E.dl == 0 ? B - 1 : 2 * (B - 1));
  for (int q = threadIdx.x >> 6; q < 3 * NZ; q += TPB / 64) {
    const int a = q / NZ, k = q % NZ;
    const int t = k == 0 ? -1 : (k == 1 ? 0 : (k == 2 ? 1 : (k == 3 ? 8 : (k == 4 ? 9 : (k == 5 ? 16 : 17)))));
    const int l = t - (a == 0 ? E.o[0] : (a == 1 ? E.o[1] : E.o[2]));
    const unsigned long long mm = __ballot(live && l >= 0 && l <= ext);
    if (lane == 0) z.m[a][k] = mm;
  }
  if (threadIdx.x < 64) {
    const int sh = 1 - E.dl;
    z.se[lane] = SEnt{E.slot * NP - (((2 * E.o[0]) >> sh) + B * ((2 * E.o[1]) >> sh) + B * B * ((2 * E.o[2]) >> sh)), sh};
  }
  __syncthreads();
  for (int p = threadIdx.x; p < NZ * NZ * NZ; p += TPB) {
    const unsigned long long c = z.m[0][p % NZ] & z.m[1][(p / NZ) % NZ] & z.m[2][p / (NZ * NZ)];
    z.tab[p] = z.se[c ? 63 - __clzll((long long)c) : 0];
  }
  __syncthreads();
}

// address of the point t with owner E
__device__ __forceinline__ int addr_of(const SEnt& E, int x, int y, int z) {
  return E.base + ((2 * x) >> E.sh) + B * ((2 * y) >> E.sh) + B * B * ((2 * z) >> E.sh);
}
__device__ __forceinline__ SEnt owner_of(const Zones& z, int x, int y, int zz) {
  return z.tab[zone_of(x) + NZ * zone_of(y) + NZ * NZ * zone_of(zz)];
}

// Predictions of a column from a coarse array (W points per axis, x fastest): the points
// between two coarse ones along x are formed once for the workgroup, in an array `odd` of
// the same strides (entry i: between coarse points i + 1 and i + 2), so a column reads one
// point of a plane, or four along y.
template <int W, int N, int TPB, typename T>
__device__ __forceinline__ void fill_odd(T* odd, const T* c) {
  for (int p = threadIdx.x; p < N * W * W; p += TPB) {
    const int o = p % N + W * (p / N);
    odd[o] = P4(c[o], c[o + 1], c[o + 2], c[o + 3]);
  }
}

// x-y prediction at plane k of the column whose first row is at c
template <bool PY, int W, typename T>
__device__ __forceinline__ T plane_value(const T* c, int k) {
  const T* p = c + W * W * k;
  return PY ? P4(p[0], p[W], p[2 * W], p[3 * W]) : p[0];
}

// ---------------------------------------------------------------------------
// RK stage of whole blocks.  448 threads: one of the 21 x 21 columns of block + halo
// each (columns outside the block along both x and y feed the predictions only).  The
// tile kernel it replaces spent 21,000 vector instructions of a wave on a block, half of them
// on owners resolved point by point; this one spends 7,000 (40% of a compute unit's cycles;
// LDS 23%).  What bounds it now is memory: lines of
// 128 bytes for x-halo segments of two points, and the rounds of latency of a workgroup
// (14 to 18 us, two per compute unit; three are no faster, since their blocks outgrow the
// XCD's L2).  1,793 blocks on three levels: 55 us a stage mixed and 83 us FP64 on average,
// 4.2 TB/s counted, against 114 and 306 us.
// ---------------------------------------------------------------------------
constexpr int ST = kColumnThreads;
constexpr int TW = B + 4, NCOL = TW * TW;
constexpr int CW = 13;                  // coarse-lattice array: even points -4 .. 20
constexpr int NSHELL = CW * CW * CW - 11 * 11 * 11;   // of them outside -2 .. 18

// predicted values of a column (first row at c): a column of the block needs the points
// beyond it along z, a halo column the points beside the block; cm: the coarse zones
template <bool PY, typename TT>
__device__ __forceinline__ void predict_column(TT* v, const TT* c, bool own, unsigned cm) {
  auto plane = [&](int k) { return plane_value<PY, CW>(c, k); };
  // (selects, not stores under a condition: the column has to stay in registers)
  if (own) {
    const bool lo = cm & 1, hi = cm & 64;
    TT m2 = v[0], m1 = v[1], p1 = v[19], p2 = v[20];   // z = -2, -1, 17, 18
    if (lo) {
      const TT w0 = plane(0), w1 = plane(1), w2 = plane(2), w3 = plane(3);
      m2 = w1;
      m1 = P4(w0, w1, w2, w3);
    }
    if (hi) {
      const TT w0 = plane(9), w1 = plane(10), w2 = plane(11), w3 = plane(12);
      p1 = P4(w0, w1, w2, w3);
      p2 = w2;
    }
    v[0] = m2;
    v[1] = m1;
    v[19] = p1;
    v[20] = p2;
  } else {
    TT w0 = plane(1), w1 = plane(2), w2 = plane(3);
#pragma unroll
    for (int m = 0; m <= 8; ++m) {    // z = 2 m and 2 m + 1
      const TT w3 = m < 8 ? plane(m + 4) : w2;
      v[2 * m + 2] = cm & (1u << zone_of(2 * m)) ? w1 : v[2 * m + 2];
      if (m < 8) v[2 * m + 3] = cm & (1u << zone_of(2 * m + 1)) ? P4(w0, w1, w2, w3) : v[2 * m + 3];
      w0 = w1;
      w1 = w2;
      w2 = w3;
    }
  }
}

// k1 and k2 in the update, their last use: FP64 slopes are loaded past the caches, which
// the neighbours' halos need (87.5 against 91.1 us); FP32 ones are faster through them
__device__ __forceinline__ double last_use(const double* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ float last_use(const float* p) { return *p; }

template <typename TT, typename KT, bool HASK, int PARTS>
__global__ void __launch_bounds__(ST, 4) k_stage3(StageArgs A) {
  __shared__ Zones zn;
  extern __shared__ __align__(16) char smem[];
  TT* tile = reinterpret_cast<TT*>(smem);   // [17 planes][NCOL]
  TT* carr = tile;                          // coarse lattice and its odd points along x:
  TT* codd = carr + CW * CW * CW;           // dead before the tile is written
  const int tid = threadIdx.x;
  // the block's own columns first (17 x 17), then the ones beside it along y, along x, and
  // along both: own columns fill whole waves, which alone run the update
  constexpr int N1 = B * B, N2 = N1 + 4 * B, N3 = N2 + 4 * B;
  const bool live = tid < NCOL, own = tid < N1, side = tid >= N1 && tid < N3;
  auto beside = [](int i) { return i < 2 ? i - 2 : B - 2 + i; };   // -2, -1, 17, 18
  const int tx = tid < N1 ? tid % B : (tid < N2 ? (tid - N1) % B : (live ? beside((tid - N2) % 4) : 0));
  const int ty = tid < N1 ? tid / B
                          : (tid < N2 ? beside((tid - N1) / B)
                                      : (tid < N3 ? (tid - N2) / 4 : (live ? beside((tid - N3) / 4) : 0)));
  const int col = tx + 2 + TW * (ty + 2);
  const bool even = ((tx | ty) & 1) == 0;
  const int nblk = A.topo.h.n_blocks, stage = A.stage;
  const double off = A.off[0], alpha = A.alpha;
  const XcdWork it(nblk);   // one work item per workgroup
  if (!it.ok()) return;
  const int b = A.order ? A.topo.list()[it.w] : it.w;
  const BlockDesc d = A.topo.blk()[b];
  zone_table<ST>(zn, d, A.topo.nb(b), A.topo.h.nb_stride);
  const bool hasc = d.n_coarse > 0;
  const int base = d.slot * NP;
  const KT* kp = (const KT*)A.kprev;
  const SEnt* ct = zn.tab + zone_of(tx) + NZ * zone_of(ty);   // the column's zones, NZ * NZ apart
  unsigned cm = 0;   // coarse zones
#pragma unroll
  for (int k = 0; k < NZ; ++k)
    if (ct[NZ * NZ * k].sh == 2) cm |= 1u << k;
  TT v[TW];
  auto value = [&](double u, double k) -> TT {
    const double y = HASK ? u + alpha * k : u;
    if constexpr (sizeof(TT) == 4) return (TT)(y - off);
    else return y;
  };
  // the coarse lattice's shell (even points beyond the columns at hand), requested first
  constexpr int RS = (NSHELL + ST - 1) / ST;
  double su[RS];
  KT sk[RS];
  int so[RS];
  if (hasc) {
#pragma unroll
    for (int q = 0; q < RS; ++q) {
      const int p = min(tid + q * ST, NSHELL - 1);
      int cx, cy, cz;
      if (p < 2 * CW * CW) {
        const int r = p % (CW * CW);
        cz = p < CW * CW ? 0 : CW - 1;
        cy = r / CW;
        cx = r % CW;
      } else if (p < 2 * CW * CW + 2 * 11 * CW) {
        const int r = (p - 2 * CW * CW) % (11 * CW);
        cy = p - 2 * CW * CW < 11 * CW ? 0 : CW - 1;
        cz = 1 + r / CW;
        cx = r % CW;
      } else {
        const int r0 = p - 2 * CW * CW - 2 * 11 * CW, r = r0 % 121;
        cx = r0 < 121 ? 0 : CW - 1;
        cz = 1 + r / 11;
        cy = 1 + r % 11;
      }
      const int sx = 2 * cx - 4, sy = 2 * cy - 4, sz = 2 * cz - 4;
      const int a = addr_of(owner_of(zn, sx, sy, sz), sx, sy, sz);
      so[q] = cx + CW * cy + CW * CW * cz;
      su[q] = A.u[a];
      if (HASK) sk[q] = kp[a];
    }
  }
  // in PARTS rounds, every load of a round in flight at once; points that nobody needs or
  // holds load the block's first node and are dropped
  const bool needh = own || (hasc && even), needs = needh || side;
#pragma unroll
  for (int part = 0; part < PARTS; ++part) {
    constexpr int N = (TW + PARTS - 1) / PARTS;
    const int i0 = N * part, n = min(N, TW - i0), k0 = zone_of(i0 - 2), k1 = zone_of(i0 + n - 3);
    double uu[N];
    KT kk[N];
    int ad[N], cb[NZ], sh[NZ];
#pragma unroll
    for (int k = k0; k <= k1; ++k) {
      const SEnt E = ct[NZ * NZ * k];
      cb[k] = E.base + ((2 * tx) >> E.sh) + B * ((2 * ty) >> E.sh);
      sh[k] = E.sh;
    }
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const int z = i0 + i - 2, k = zone_of(z);
      const bool held = !((cm >> k) & 1u) || (even && (z & 1) == 0);
      const bool need = z >= 0 && z < B ? needs : needh;
      ad[i] = held && need ? cb[k] + B * B * ((2 * z) >> sh[k]) : base;
    }
#pragma unroll
    for (int i = 0; i < n; ++i) {
      uu[i] = A.u[ad[i]];
      if (HASK) kk[i] = kp[ad[i]];
    }
#pragma unroll
    for (int i = 0; i < n; ++i) v[i0 + i] = value(uu[i], HASK ? (double)kk[i] : 0.0);
  }
  if (hasc) {
    // the coarse lattice: even points of the columns at hand, then the shell around them
    if (live && even) {
      TT* c = carr + (tx + 4) / 2 + CW * ((ty + 4) / 2) + CW * CW;
#pragma unroll
      for (int k = 0; k < 11; ++k) c[CW * CW * k] = v[2 * k];
    }
#pragma unroll
    for (int q = 0; q < RS; ++q)   // (a repeated last point holds the same value)
      carr[so[q]] = value(su[q], HASK ? (double)sk[q] : 0.0);
    __syncthreads();
    fill_odd<CW, 10, ST>(codd, carr);
    __syncthreads();
    const unsigned need = own ? cm & 0x41u : (side ? cm & 0x3Eu : 0u);
    if (need) {
      const TT* c = (tx & 1) ? codd + (tx + 1) / 2 : carr + (tx + 4) / 2;
      if (ty & 1) predict_column<true>(v, c + CW * ((ty + 1) / 2), own, need);
      else predict_column<false>(v, c + CW * ((ty + 4) / 2), own, need);
    }
    __syncthreads();
  }
  if (own || side) {
#pragma unroll
    for (int z = 0; z < B; ++z) tile[z * NCOL + col] = v[z + 2];
  }
  __syncthreads();
  if (own) {
    TT r;
    if constexpr (sizeof(TT) == 8) r = A.lt.r[d.level];
    else r = A.lt.rf[d.level];
    const TT c0 = (TT)A.ph.c[0], c1 = (TT)A.ph.c[1], c2 = (TT)A.ph.c[2];
    const size_t node0 = (size_t)base + tx + B * ty;
    const TT* T = tile + col;
    auto rhs = [&](int z) -> TT {
      const TT* p = T + z * NCOL;
      TT acc = c0 * D4(p[-2], p[-1], p[1], p[2], r);
      acc = acc + c1 * D4(p[-2 * TW], p[-TW], p[TW], p[2 * TW], r);
      acc = acc + c2 * D4(v[z], v[z + 1], v[z + 3], v[z + 4], r);
      return -acc;
    };
    if (stage < 4) {
      KT* ko = (KT*)A.kout + node0;
#pragma unroll
      for (int z = 0; z < B; ++z) ko[B * B * z] = (KT)rhs(z);
    } else {
      // the update's operands, a few nodes at a time, requested before they are used
      constexpr int NB = 4;
      const KT *q1 = (const KT*)A.k1 + node0, *q2 = (const KT*)A.k2 + node0, *q3 = (const KT*)A.k3 + node0;
      const double* qu = A.u + node0;
#pragma unroll
      for (int z0 = 0; z0 < B; z0 += NB) {
        double e1[NB], e2[NB], e3[NB], eu[NB];
#pragma unroll
        for (int e = 0; e < NB; ++e) {
          if (z0 + e >= B) continue;
          const int o = B * B * (z0 + e);
          e1[e] = (double)last_use(q1 + o);
          e2[e] = (double)last_use(q2 + o);
          e3[e] = (double)q3[o];
          eu[e] = qu[o];
        }
#pragma unroll
        for (int e = 0; e < NB; ++e) {
          if (z0 + e >= B) continue;
          const double k4 = (double)rhs(z0 + e);
          A.unew[node0 + B * B * (z0 + e)] = eu[e] + A.h6 * ((e1[e] + k4) + 2.0 * (e2[e] + e3[e]));
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// multiresolution analysis of whole blocks: details d = u - P(R(u)), maximum, flag, the
// synchronised values of redundant nodes finer neighbours own, and the mothers' nodes of
// a speculated coarsening.  320 threads: one of the block's 17 x 17 columns each; LDS
// holds the even points up to 2 beyond the block only (the prediction's inputs), 25 KB
// against 53 KB for a tile, and a column's details read 55 of them where a stencil per
// point read 290.  1,793 blocks: 30 us (2.4 TB/s of block data) against 123 us.
// ---------------------------------------------------------------------------
constexpr int MT = 320;                 // threads of the analysis and refinement kernels
constexpr int EW = 11, NEV = EW * EW * EW;   // even points -2 .. 18

// details of a column (first row at c): maximum of |v - prediction| as unsigned bits, which
// NaN propagates through; skip: the column's even points are coarse points themselves
template <bool PY>
__device__ __forceinline__ unsigned long long column_details(const double* v, const double* c, bool skip) {
  auto plane = [&](int k) { return plane_value<PY, EW>(c, k); };
  unsigned long long m = 0;
  auto take = [&](double dv) { m = umax64(m, (unsigned long long)__double_as_longlong(fabs(dv))); };
  double w0 = plane(0), w1 = plane(1), w2 = plane(2);
#pragma unroll
  for (int k = 0; k <= 8; ++k) {   // z = 2 k and 2 k + 1
    const double w3 = k < 8 ? plane(k + 3) : w2;
    if (PY || !skip) take(v[2 * k] - w1);
    if (k < 8) take(v[2 * k + 1] - P4(w0, w1, w2, w3));
    w0 = w1;
    w1 = w2;
    w2 = w3;
  }
  return m;
}

__global__ void __launch_bounds__(MT, 3) k_mr3(MrArgs A) {
  __shared__ Zones zn;
  __shared__ double ev[NEV], od[NEV];
  __shared__ double red[MT / 64];
  const int tid = threadIdx.x;
  const bool own = tid < B * B;
  const int col = own ? tid : 0, tx = col % B, ty = col / B;
  const bool even = ((tx | ty) & 1) == 0, rim = tx == 0 || ty == 0 || tx == B - 1 || ty == B - 1;
  const int nblk = A.topo.h.n_blocks;
  const XcdWork it(nblk);   // one work item per workgroup
  if (!it.ok()) return;
  const int b = it.w;
  const BlockDesc d = A.topo.blk()[b];
  const int sm = A.smap ? A.smap[b] : -1;
  zone_table<MT>(zn, d, A.topo.nb(b), A.topo.h.nb_stride);
  const int base = d.slot * NP;
  int cb[5], sh[5];
  unsigned fine = 0;   // zones (of 1 .. 5) a finer neighbour owns
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const SEnt E = zn.tab[zone_of(tx) + NZ * zone_of(ty) + NZ * NZ * (k + 1)];
    cb[k] = E.base + ((2 * tx) >> E.sh) + B * ((2 * ty) >> E.sh);
    sh[k] = E.sh;
    if (E.sh == 0) fine |= 1u << k;
  }
  double v[B];
#pragma unroll
  for (int z = 0; z < B; ++z) {
    const int k = zone_of(z) - 1;
    v[z] = A.u[cb[k] + B * B * ((2 * z) >> sh[k])];
  }
  // even points outside the block (602), two rounds
  constexpr int NOUT = NEV - 9 * 9 * 9, R = (NOUT + MT - 1) / MT;
  double ov[R];
  int oi[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int p = min(tid + q * MT, NOUT - 1);
    int cx, cy, cz;
    if (p < 242) {
      const int r = p % 121;
      cz = p < 121 ? 0 : EW - 1;
      cy = r / EW;
      cx = r % EW;
    } else if (p < 242 + 198) {
      const int r = (p - 242) % 99;
      cy = p - 242 < 99 ? 0 : EW - 1;
      cz = 1 + r / EW;
      cx = r % EW;
    } else {
      const int r = (p - 440) % 81;
      cx = p - 440 < 81 ? 0 : EW - 1;
      cz = 1 + r / 9;
      cy = 1 + r % 9;
    }
    const int sx = 2 * cx - 2, sy = 2 * cy - 2, sz = 2 * cz - 2;
    oi[q] = cx + EW * cy + EW * EW * cz;
    ov[q] = A.u[addr_of(owner_of(zn, sx, sy, sz), sx, sy, sz)];
  }
  if (own && even) {
#pragma unroll
    for (int k = 0; k < 9; ++k) ev[tx / 2 + 1 + EW * (ty / 2 + 1) + EW * EW * (k + 1)] = v[2 * k];
  }
#pragma unroll
  for (int q = 0; q < R; ++q) ev[oi[q]] = ov[q];   // (a repeated last point holds the same value)
  // redundant nodes owned by a finer neighbour: store the synchronised value
  if (own && fine) {
#pragma unroll
    for (int z = 0; z < B; ++z) {
      const int k = zone_of(z) - 1;
      if ((rim || z == 0 || z == B - 1) && ((fine >> k) & 1u)) A.u[base + tx + B * ty + B * B * z] = v[z];
    }
  }
  __syncthreads();
  fill_odd<EW, 8, MT>(od, ev);
  __syncthreads();
  unsigned long long m = 0;
  if (own) {
    const double* c = (tx & 1) ? od + tx / 2 : ev + tx / 2 + 1;
    if (ty & 1) m = column_details<true>(v, c + EW * (ty / 2), false);
    else m = column_details<false>(v, c + EW * (ty / 2 + 1), even);
  }
  const double wm = wave_nanmax(__longlong_as_double((long long)m));
  if ((tid & 63) == 0) red[tid >> 6] = wm;
  __syncthreads();
  if (tid == 0) {
    double v0 = red[0];
#pragma unroll
    for (int q = 1; q < MT / 64; ++q) v0 = nanmax(v0, red[q]);
    A.maxd[b] = v0;
    A.flags[b] = d.level > 1 && v0 < A.thr[0] ? (int8_t)-1 : (int8_t)0;
  }
  if (sm >= 0 && own && even) {
    // the block is child `ch` of a speculated family: the mother's nodes it supplies (a
    // node shared by several children comes from the lowest child index), with the values
    // the block holds after the write-back above
    const int ch = sm & 7;
    const size_t mbase = (size_t)(sm >> 3) * NP;
    const bool skip = ((ch & 1) && tx == 0) || ((ch & 2) && ty == 0);
    const int mx = tx / 2 + (ch & 1) * 8, my = ty / 2 + ((ch >> 1) & 1) * 8, mz = ((ch >> 2) & 1) * 8;
#pragma unroll
    for (int z = 0; z < B; z += 2) {
      if (skip || ((ch & 4) && z == 0)) continue;
      const int k = zone_of(z) - 1;
      const bool from_tile = !(rim || z == 0 || z == B - 1) || ((fine >> k) & 1u);
      const double val = from_tile ? v[z] : A.u[base + tx + B * ty + B * B * z];
      A.u[mbase + mx + B * my + B * B * (mz + z / 2)] = val;
    }
  }
}

// ---------------------------------------------------------------------------
// refinement, one workgroup per child of a parent: LDS holds the synchronised parent
// points the child needs (11^3: its half of the parent and one point around), and every
// thread interpolates one of the child's 17 x 17 columns.  Nodes on the parent's boundary
// that a finer leaf holds are copied in a pass of their own, all loads in flight, so no
// column waits for them.  428 parents to 3,424 children: 66 us (its stores, 135 MB) against
// 111 us for sub-tiles of children; 8 and 29 parents, a whole call: 19 and 26 us against 24
// and 48.
// ---------------------------------------------------------------------------
constexpr int LW = 9;                   // coarse lattice of a parent beside coarser leaves

// a column of the child (first row at c) stored at out; held: zones along z (of the fine
// coordinate) where a finer leaf holds the column's nodes on the parent's boundary, which
// are left out (rim: every node of the column lies on it)
template <bool PY>
__device__ __forceinline__ void refine_column(const double* c, double* out, unsigned held, bool rim, bool even, int bit) {
  auto plane = [&](int k) { return plane_value<PY, EW>(c, k); };
  double w0 = plane(0), w1 = plane(1), w2 = plane(2);
#pragma unroll
  for (int z = 0; z < B; ++z) {
    double w3 = w2, val = w1;
    if (z & 1) {
      w3 = plane(z / 2 + 3);
      val = P4(w0, w1, w2, w3);
    }
    // zone of the fine coordinate z + 16 bit (in the parent's units: half of it)
    const unsigned zb = z == 0 ? (bit ? 8u : 2u) : (z == B - 1 ? (bit ? 32u : 8u) : (bit ? 16u : 4u));
    const bool bnd = rim || (z == 0 && !bit) || (z == B - 1 && bit);
    const bool keep = (held & zb) && bnd && !(even && (z & 1) == 0);
    if (!keep) out[B * B * z] = val;
    if (z & 1) {
      w0 = w1;
      w1 = w2;
      w2 = w3;
    }
  }
}

__global__ void __launch_bounds__(MT, 4) k_refine3(RefineArgs A) {
  __shared__ Zones zn;
  __shared__ SEnt fin[NZ * NZ * NZ];   // first finer holder of a zone (sh 1: none)
  __shared__ double ev[NEV], od[NEV];
  __shared__ double lat[LW * LW * LW];
  const int tid = threadIdx.x;
  const bool own = tid < B * B;
  const int col = own ? tid : 0, x = col % B, y = col / B;
  // zone of a fine coordinate Q (parent coordinate Q / 2)
  auto fz = [](int Q) { return Q == 0 ? 1 : (Q < 16 ? 2 : (Q == 16 ? 3 : (Q < 32 ? 4 : 5))); };
  const int nref = A.topo.h.n_ref;
  const XcdWork it(nref * 8);   // one work item per workgroup
  if (!it.ok()) return;
  const int ri = it.w >> 3, ch = it.w & 7;
  const BlockDesc d = A.topo.pblk()[ri];
  const int cslot = A.topo.ref()[ri].child[ch];
  zone_table<MT>(zn, d, A.topo.pnb(ri), A.topo.h.pnb_stride);
  // finer entries come last in the list: the second table is needed only then
  const bool hasf = d.n_ent > 0 && zn.se[d.n_ent - 1].sh == 0;
  const int bx = ch & 1, by = (ch >> 1) & 1, bz = (ch >> 2) & 1;
  const bool hasc = d.n_coarse > 0;
  const int p0 = 8 * bx - 1, p1 = 8 * by - 1, p2 = 8 * bz - 1;   // first parent point
  constexpr int R = (NEV + MT - 1) / MT;
  double pv[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int p = min(tid + q * MT, NEV - 1);
    const int sx = p0 + p % EW, sy = p1 + (p / EW) % EW, sz = p2 + p / (EW * EW);
    const SEnt E = owner_of(zn, sx, sy, sz);
    const bool held = E.sh < 2 || ((sx | sy | sz) & 1) == 0;
    pv[q] = A.u[held ? addr_of(E, sx, sy, sz) : d.slot * NP];   // (unheld: predicted below)
  }
  constexpr int RL = (LW * LW * LW + MT - 1) / MT;
  double lv[RL];
  if (hasc) {
    // the parent's even points around the child's half: 9^3 from -4 (or 4) on
#pragma unroll
    for (int q = 0; q < RL; ++q) {
      const int p = min(tid + q * MT, LW * LW * LW - 1);
      const int sx = 8 * bx - 4 + 2 * (p % LW), sy = 8 * by - 4 + 2 * ((p / LW) % LW),
                sz = 8 * bz - 4 + 2 * (p / (LW * LW));
      lv[q] = A.u[addr_of(owner_of(zn, sx, sy, sz), sx, sy, sz)];
    }
  }
#pragma unroll
  for (int q = 0; q < R; ++q) ev[min(tid + q * MT, NEV - 1)] = pv[q];
  if (hasc) {
#pragma unroll
    for (int q = 0; q < RL; ++q) lat[min(tid + q * MT, LW * LW * LW - 1)] = lv[q];
  }
  if (hasf) {
    const int lane = tid & 63;
    const unsigned long long fmask = __ballot(lane < d.n_ent && zn.se[lane].sh == 0);
    for (int p = tid; p < NZ * NZ * NZ; p += MT) {
      const unsigned long long c = zn.m[0][p % NZ] & zn.m[1][(p / NZ) % NZ] & zn.m[2][p / (NZ * NZ)] & fmask;
      fin[p] = c ? zn.se[__ffsll((long long)c) - 1] : SEnt{0, 1};
    }
  }
  __syncthreads();
  if (hasc) {
    // parent points inside a coarser neighbour, off its lattice: only the three planes one
    // point outside the parent can hold any
#pragma unroll 1
    for (int p = tid; p < 3 * EW * EW; p += MT) {
      const int ax = p / (EW * EW), r = p % (EW * EW), i = r % EW, j = r / EW;
      const int e = (ax == 0 ? bx : (ax == 1 ? by : bz)) ? EW - 1 : 0;
      const int c0 = ax == 0 ? e : i, c1 = ax == 1 ? e : (ax == 0 ? i : j), c2 = ax == 2 ? e : j;
      const int sx = p0 + c0, sy = p1 + c1, sz = p2 + c2;
      const SEnt E = owner_of(zn, sx, sy, sz);
      if (E.sh < 2 || ((sx | sy | sz) & 1) == 0) continue;
      const int l0 = c0 + 3, l1 = c1 + 3, l2 = c2 + 3;   // from the lattice's first point
      const int px = l0 & 1, py = l1 & 1, pz = l2 & 1;
      const double* c = lat + (px ? (l0 - 3) / 2 : l0 / 2) + LW * (py ? (l1 - 3) / 2 : l1 / 2) +
                        LW * LW * (pz ? (l2 - 3) / 2 : l2 / 2);
      auto row = [&](const double* q) { return px ? P4(q[0], q[1], q[2], q[3]) : q[0]; };
      auto plane = [&](const double* q) {
        return py ? P4(row(q), row(q + LW), row(q + 2 * LW), row(q + 3 * LW)) : row(q);
      };
      ev[c0 + EW * c1 + EW * EW * c2] =
          pz ? P4(plane(c), plane(c + LW * LW), plane(c + 2 * LW * LW), plane(c + 3 * LW * LW)) : plane(c);
    }
    __syncthreads();
  }
  fill_odd<EW, 8, MT>(od, ev);
  __syncthreads();
  double* const out = A.u + (size_t)cslot * NP;
  if (own) {
    const int Qx = x + 16 * bx, Qy = y + 16 * by;
    const bool rim = Qx == 0 || Qx == 32 || Qy == 0 || Qy == 32, even = ((x | y) & 1) == 0;
    unsigned held = 0;
    if (hasf) {
      const SEnt* f = fin + fz(Qx) + NZ * fz(Qy);
#pragma unroll
      for (int k = 1; k < 6; ++k)
        if (f[NZ * NZ * k].sh == 0) held |= 1u << k;
    }
    const double* c = (x & 1) ? od + x / 2 : ev + x / 2 + 1;
    if (y & 1) refine_column<true>(c + EW * (y / 2), out + col, held, rim, even, bz);
    else refine_column<false>(c + EW * (y / 2 + 1), out + col, held, rim, even, bz);
  }
  if (hasf) {
    // the odd nodes of the parent's boundary that a finer leaf holds take its values
    constexpr int RF = (3 * B * B + MT - 1) / MT;
    double fv[RF];
    int fn[RF];
#pragma unroll
    for (int q = 0; q < RF; ++q) {
      const int p = tid + q * MT;
      const int ax = p / (B * B), r = p % (B * B), i = r % B, j = r / B;
      const int e = (ax == 0 ? bx : (ax == 1 ? by : bz)) ? B - 1 : 0;
      const int c0 = ax == 0 ? e : i, c1 = ax == 1 ? e : (ax == 0 ? i : j), c2 = ax == 2 ? e : j;
      const int Qx = c0 + 16 * bx, Qy = c1 + 16 * by, Qz = c2 + 16 * bz;
      const SEnt E = fin[fz(Qx) + NZ * fz(Qy) + NZ * NZ * fz(Qz)];
      const bool take = ax < 3 && E.sh == 0 && ((c0 | c1 | c2) & 1);
      fn[q] = take ? c0 + B * c1 + B * B * c2 : -1;
      fv[q] = A.u[take ? E.base + Qx + B * Qy + B * B * Qz : d.slot * NP];
    }
#pragma unroll
    for (int q = 0; q < RF; ++q)
      if (fn[q] >= 0) out[fn[q]] = fv[q];
  }
  __syncthreads();
}

// one workgroup per work item (XcdWork deals them out from a multiple of 8)
template <typename K, typename Arg>
hipError_t go3(K kern, int items, size_t lds, int threads, hipStream_t st, const Arg& a) {
  hipLaunchKernelGGL(kern, dim3(std::max(8, (items + 7) & ~7)), dim3(threads), lds, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_stage3(int precision, const StageArgs& a, hipStream_t st) {
  constexpr size_t pts = (size_t)B * NCOL;
  static_assert(pts >= (size_t)2 * CW * CW * CW, "the coarse lattice shares the tile's LDS");
  const int n = a.topo.h.n_blocks;
  if (precision == 0)
    return a.stage > 1 ? go3(k_stage3<double, double, true, 2>, n, pts * sizeof(double), ST, st, a)
                       : go3(k_stage3<double, double, false, 1>, n, pts * sizeof(double), ST, st, a);
  return a.stage > 1 ? go3(k_stage3<float, float, true, 1>, n, pts * sizeof(float), ST, st, a)
                     : go3(k_stage3<float, float, false, 1>, n, pts * sizeof(float), ST, st, a);
}

hipError_t launch_mr3(const MrArgs& a, hipStream_t st) { return go3(k_mr3, a.topo.h.n_blocks, 0, MT, st, a); }

hipError_t launch_refine3(const RefineArgs& a, hipStream_t st) { return go3(k_refine3, 8 * a.topo.h.n_ref, 0, MT, st, a); }

}  // namespace mrb
