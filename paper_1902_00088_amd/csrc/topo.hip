// Device-resident topology transitions of the multiresolution step (gfx950): the
// safety-zone refinement plan (Sec. 2.1 item 1), the coarsening plan with its
// completeness and gradedness fixed point (Sec. 2.3, last paragraph; Sec. 2.2 graded
// grid) and the neighbour entries of the new grid, so that a step needs no host
// planning.  The results are the host planner's: the same forest order (Morton), the
// same slots from the same free stack, the same entries in the same order.
//
// Layout: every grid lives in an arena of fixed capacity (header, block descriptors,
// entry rows of a fixed stride, refinement parents with their entry rows, refinement
// and coarsening plans); a dense index holds, for every possible block of every level,
// the pool slot of the leaf there or -1; the free pool slots form a stack.
//
// All of this is small integer work on a few thousand blocks: a launch costs its chain of
// dependent loads (0.6 to 0.8 us each) and not its bytes.  So the index holds slots (an
// entry needs no second look-up), a family is known by its first member's position (no
// numbering pass), positions after a transition follow from the number of parents or live
// families before a block (flags counted by every workgroup for itself: 1 bit or byte per
// block, instead of scans in one workgroup), and pushes to the free stack wait for the
// launch after the one that pops.  Per step of an adaptive 2D run (740 to 2,900 blocks, the
// refinement, two analyses, one coarsening): 129 -> 45 us in these kernels.
#include "internal.hpp"

#include <hip/hip_runtime.h>

namespace mrb {

namespace {

// coordinates and origins along z are 0 in 2D: loops over axes run to 3, unrolled
__device__ __forceinline__ int cell_of(const DevTopoArgs& A, int l, const int* c) {
  int k = A.cell_off[l] + c[0] + (c[1] << l);
  if (A.dim > 2) k += c[2] << (2 * l);
  return k;
}

__device__ __forceinline__ int wrapl(int a, int l) { return a & ((1 << l) - 1); }

// flags set (bytes 0 or 1) before position `end` (a multiple of 8) of a byte array, or bits
// set in `end` words: the sum over the workgroup of 256 threads, in every thread
__device__ __forceinline__ int wg_count(const unsigned long long* w, int words) {
  __shared__ int part[4];
  int s = 0;
  for (int i = threadIdx.x; i < words; i += blockDim.x) s += __popcll(w[i]);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  return part[0] + part[1] + part[2] + part[3];
}

}  // namespace

// ---------------------------------------------------------------------------
// refinement plan: every block below jmax becomes its 2^dim children in its place of the
// forest order; child ch of the r-th parent takes free[top-1-(r*nch+ch)], and the parents'
// slots are pushed in forest order by k_entries.  Writes the new grid's block descriptors
// (entries come later), the refinement plan (children's slots, the parents' descriptors)
// and the dense index.  One thread per (block, child); the parents before a workgroup are
// counted from the flags that k_entries left (4,096 blocks: 16 bytes a thread).
// 372 blocks of 3D: 24 -> 4.8 us, and the two index launches it takes in were 6 more.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_plan_refine(DevTopoArgs A) {
  const int n = A.old_h.n_blocks, nch = A.nch, t = threadIdx.x;
  const int per = 256 / nch, base = blockIdx.x * per;   // per = 64 or 32 blocks
  const unsigned long long* isp = (const unsigned long long*)A.isp;
  const int before = wg_count(isp, base / 8);
  const int b = base + t / nch, ch = t % nch;
  if (b >= n) return;
  int ri = before;
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    const int k = b - base - 8 * w;   // flags of this word that lie before b
    if (k > 0) ri += __popcll(isp[base / 8 + w] & (k < 8 ? (1ull << (8 * k)) - 1ull : ~0ull));
  }
  const BlockDesc d = ((const BlockDesc*)(A.old_base + A.old_h.off_blk))[b];
  BlockDesc* nb = (BlockDesc*)(A.new_base + A.new_h.off_blk);
  const int pos = b + (nch - 1) * ri;
  BlockDesc k = d;
  k.nb_begin = k.n_ent = k.n_coarse = 0;
  if (d.level >= A.jmax) {
    if (ch == 0) nb[pos] = k;
    return;
  }
  k.slot = A.free_stack[A.free_top - 1 - (ri * nch + ch)];
  k.level = d.level + 1;
  for (int a = 0; a < 3; ++a) k.c[a] = 2 * d.c[a] + ((ch >> a) & 1);
  nb[pos + ch] = k;
  A.cells[cell_of(A, k.level, k.c)] = k.slot;
  RefineDesc* rd = (RefineDesc*)(A.new_base + A.new_h.off_ref);
  rd[ri].child[ch] = k.slot;
  if (ch + nch < 8) rd[ri].child[ch + nch] = -1;
  if (ch == 0) {
    A.cells[cell_of(A, d.level, d.c)] = -1;
    ((BlockDesc*)(A.new_base + A.new_h.off_pblk))[ri] = d;
    A.fam[ri] = b;   // parent r -> old block (for the entry-row copy)
  }
}

// ---------------------------------------------------------------------------
// coarsening plan, in three launches.  Complete families whose 2^dim members
// (consecutive in forest order) are all flagged -1 are the candidates.  A candidate
// must go while a finer leaf touching one of its members is not in a live candidate
// (the greatest such set: a demotion only removes a family that no valid subset can
// hold, so the order of demotions does not matter).  The number of live families, read
// back by the host, decides whether the fourth launch (k_coarsen_apply) follows.
// Scratch: fam[slot] (position of the first member of the slot's candidate family or -1),
// dead[position] (0: first member of a live candidate), live (bits of dead == 0), edge
// count, any candidates, edges (family, family it needs).  The count and the flag are zero
// before a plan and left zero by it.
// A step whose plan finds nothing to merge takes 30 -> 12 us (adaptive 2D, 740 to 2,900 blocks).
// ---------------------------------------------------------------------------
namespace {
__device__ __forceinline__ bool family_first(const DevTopoArgs& A, const BlockDesc* ob, int n, int b) {
  const BlockDesc d = ob[b];
  if (d.level < 2 || A.flags[b] != -1) return false;
  for (int a = 0; a < 3; ++a)
    if (d.c[a] & 1) return false;
  if (b + A.nch > n) return false;
  bool all = true;   // no early way out: the members' loads are issued together
#pragma unroll
  for (int ch = 1; ch < 8; ++ch) {
    if (ch >= A.nch) break;
    const BlockDesc e = ob[b + ch];
    all = all && e.level == d.level && A.flags[b + ch] == -1;
    for (int a = 0; a < 3; ++a) all = all && e.c[a] == d.c[a] + ((ch >> a) & 1);
  }
  return all;
}
}  // namespace

// 1 (whole grid): the candidate family of every block, and whether its detail norms are
// finite
__global__ void __launch_bounds__(256) k_coarsen_candidates(DevTopoArgs A) {
  const int n = A.old_h.n_blocks;
  const BlockDesc* ob = (const BlockDesc*)(A.old_base + A.old_h.off_blk);
  int bad = 0, any = 0;
  for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < n; b += gridDim.x * blockDim.x) {
    const BlockDesc d = ob[b];
    int ch = 0;
    for (int a = 0; a < 3; ++a) ch |= (d.c[a] & 1) << a;
    const int f = b - ch;   // the members stand in child order
    const bool cand = f >= 0 && family_first(A, ob, n, f);
    A.fam[d.slot] = cand ? f : -1;
    A.dead[b] = cand && ch == 0 ? 0 : 1;
    if (cand) any = 1;
    for (int q = 0; q < A.nf; ++q)
      if (!isfinite(A.maxd[(size_t)b * A.nf + q])) bad = 1;
  }
  if (any) A.edges[1] = 1;
  if (bad) atomicOr(A.err, 2);   // a non-finite detail norm
}

// 2 (whole grid): one lane per (member, entry slot), 16 or 64 lanes a member: a finer leaf
// outside every candidate kills the member's family; one inside a candidate becomes an
// edge (one counter update per wave)
__global__ void __launch_bounds__(256) k_coarsen_edges(DevTopoArgs A) {
  if (A.edges[1] == 0) return;   // no candidates
  const int n = A.old_h.n_blocks, S = A.old_h.nb_stride;
  const BlockDesc* ob = (const BlockDesc*)(A.old_base + A.old_h.off_blk);
  const NbEntry* nb = (const NbEntry*)(A.old_base + A.old_h.off_nb);
  const int gl = S <= 16 ? 16 : 64, per = 64 / gl, lane = threadIdx.x & 63, e = lane % gl;
  const int waves = gridDim.x * (blockDim.x >> 6);
  for (int w = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); w * per < n; w += waves) {
    const int m = w * per + lane / gl;
    int f = -1, g = -1;
    if (m < n && e < S) {
      const BlockDesc M = ob[m];
      const NbEntry E = nb[(size_t)m * S + e];
      const int fm = A.fam[M.slot];
      if (fm >= 0 && e < M.n_ent && E.dl > 0) {
        f = fm;
        g = A.fam[E.slot];
        if (g < 0) A.dead[f] = 1;
      }
    }
    const bool edge = g >= 0 && g != f;
    const unsigned long long who = __ballot(edge);
    if (who == 0) continue;
    int k = 0;
    if (lane == 0) k = atomicAdd(&A.edges[0], __popcll(who));
    k = __shfl(k, 0, 64) + __popcll(who & ((1ull << lane) - 1ull));
    if (edge) {
      A.edges[2 + 2 * k] = f;
      A.edges[3 + 2 * k] = g;
    }
  }
}

// 3 (one workgroup): the fixed point over the edges, the live families' bits and counts.
// The flags stay in LDS (a byte a block) up to kAliveLds blocks, else in dead.
__global__ void __launch_bounds__(1024) k_coarsen_fix(DevTopoArgs A) {
  __shared__ int fams[kMaxLevels];
  __shared__ int changed, total;
  __shared__ unsigned char alive_lds[kAliveLds];
  const int n = A.old_h.n_blocks, t = threadIdx.x, T = blockDim.x;
  const BlockDesc* ob = (const BlockDesc*)(A.old_base + A.old_h.off_blk);
  const int nedge = A.edges[0], any = A.edges[1];
  int m = 0;
  if (any) {
    const bool lds = n <= kAliveLds;
    int* dead = A.dead;
    if (t < kMaxLevels) fams[t] = 0;
    if (t == 0) total = 0;
    if (lds)
      for (int q = t; q < n; q += T) alive_lds[q] = dead[q] ? 0 : 1;
    __syncthreads();
    auto alive = [&](int q) -> bool { return lds ? alive_lds[q] != 0 : dead[q] == 0; };
    while (nedge > 0) {
      if (t == 0) changed = 0;
      __syncthreads();
      for (int k = t; k < nedge; k += T) {
        const int f = A.edges[2 + 2 * k], g = A.edges[3 + 2 * k];
        if (alive(f) && !alive(g)) {
          if (lds) alive_lds[f] = 0;
          else dead[f] = 1;
          changed = 1;
        }
      }
      __syncthreads();
      if (!changed) break;
      __syncthreads();
    }
    for (int q0 = 0; q0 < n; q0 += T) {
      const int q = q0 + t;
      const bool a = q < n && alive(q);
      const unsigned long long who = __ballot(a);
      if ((t & 63) == 0 && q < n) {
        A.live[q >> 6] = who;
        if (who) atomicAdd(&total, __popcll(who));
      }
      if (a) atomicAdd(&fams[ob[q].level], 1);
    }
    __syncthreads();
    m = total;
    if (t < kMaxLevels) A.out[4 + t] = fams[t];
  }
  if (t == 0) {
    // errors of this plan and of the entry builds since the last one, reported and cleared
    int err = atomicExch(A.err, 0);
    if (m > A.free_top) {
      err |= 4;   // the mothers need more free slots than the pool has
      m = 0;
    }
    A.out[0] = m;
    A.out[1] = n - m * (A.nch - 1);
    A.out[2] = A.free_top - m + m * A.nch;
    A.out[3] = err;
    A.edges[0] = 0;
    A.edges[1] = 0;
  }
}

// 4 (whole grid, m live families): the new forest and the dense index.  Every live family's
// mother takes its first child's place in the forest order; mother k takes free[top-m+k],
// and k_entries pushes the children's slots.  The families before a workgroup are counted
// from the live bits.
__global__ void __launch_bounds__(256) k_coarsen_apply(DevTopoArgs A) {
  const int n = A.old_h.n_blocks, nch = A.nch, m = A.new_h.n_fam;
  const int base = blockIdx.x * 256, b = base + threadIdx.x;
  const BlockDesc* ob = (const BlockDesc*)(A.old_base + A.old_h.off_blk);
  int k = wg_count(A.live, base / 64);
  if (b >= n) return;
  for (int w = base / 64; w < b / 64; ++w) k += __popcll(A.live[w]);
  k += __popcll(A.live[b / 64] & ((1ull << (b & 63)) - 1ull));
  BlockDesc d = ob[b];
  const int f = A.fam[d.slot];
  const bool gone = f >= 0 && (A.live[f >> 6] >> (f & 63) & 1ull);
  if (gone) {
    A.cells[cell_of(A, d.level, d.c)] = -1;
    if (f != b) return;
    FamilyDesc F;
    F.parent = A.free_stack[A.free_top - m + k];
    for (int ch = 0; ch < 8; ++ch) F.child[ch] = ch < nch ? ob[b + ch].slot : -1;
    ((FamilyDesc*)(A.new_base + A.new_h.off_fam))[k] = F;
    d.slot = F.parent;
    d.level -= 1;
    for (int a = 0; a < 3; ++a) d.c[a] >>= 1;
    A.cells[cell_of(A, d.level, d.c)] = d.slot;
  }
  d.nb_begin = 0;
  d.n_ent = 0;
  d.n_coarse = 0;
  ((BlockDesc*)(A.new_base + A.new_h.off_blk))[b - (nch - 1) * k] = d;
}

// the dense index of a new grid (its cells hold -1 before)
__global__ void __launch_bounds__(256) k_index(DevTopoArgs A) {
  const BlockDesc* bd = (const BlockDesc*)(A.new_base + A.new_h.off_blk);
  for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < A.new_h.n_blocks; b += gridDim.x * blockDim.x) {
    const BlockDesc d = bd[b];
    A.cells[cell_of(A, d.level, d.c)] = d.slot;
  }
}

// ---------------------------------------------------------------------------
// neighbour entries of the new grid, 16 (2D) or 32 (3D) lanes per block: lane q takes
// direction q of the 3^dim block neighbourhood (x fastest) -- a same-level leaf, else the
// coarser leaf covering that position (once per distinct leaf and image), else the finer
// leaves touching the block there -- and the group writes them in the order the kernels
// rely on: coarser, the block itself, same level, finer, each in direction order.  A lane
// looks up all six cells that can matter at once, so that a block costs two dependent
// loads.  Items past the blocks copy the refinement parents' entry rows and push the slots
// that the refinement or the coarsening has freed.
// 2,976 blocks of 3D: 25 -> 5.6 us; 740 to 2,900 of 2D: 17 -> 4.6.
// ---------------------------------------------------------------------------
template <int DIM>
__global__ void __launch_bounds__(256) k_entries(DevTopoArgs A) {
  constexpr int GL = DIM == 2 ? 16 : 32, ND = DIM == 2 ? 9 : 27, CEN = ND / 2, PER = 256 / GL;
  const int lane = threadIdx.x % GL, sh = (threadIdx.x & 63) & ~(GL - 1);
  const int nblk = A.new_h.n_blocks, nref = A.new_h.n_ref, nfam = A.new_h.n_fam, S = A.new_h.nb_stride;
  BlockDesc* bd = (BlockDesc*)(A.new_base + A.new_h.off_blk);
  for (int w = blockIdx.x * PER + threadIdx.x / GL; w < nblk + nref + nfam; w += gridDim.x * PER) {
    if (w >= nblk + nref) {
      // family k: children to free[top - m + (m*nch - 1 - (k*nch + ch))]
      const int k = w - nblk - nref;
      const FamilyDesc* fd = (const FamilyDesc*)(A.new_base + A.new_h.off_fam);
      if (lane < (1 << DIM))
        A.free_stack[A.free_top - nfam + ((nfam - k) << DIM) - 1 - lane] = fd[k].child[lane];
      continue;
    }
    if (w >= nblk) {
      // refinement parent r: its slot is free, its entry row that of the grid before
      const int r = w - nblk;
      const NbEntry* src = (const NbEntry*)(A.old_base + A.old_h.off_nb) + (size_t)A.fam[r] * A.old_h.nb_stride;
      NbEntry* dst = (NbEntry*)(A.new_base + A.new_h.off_pnb) + (size_t)r * A.new_h.pnb_stride;
      for (int e = lane; e < A.old_h.nb_stride; e += GL) dst[e] = src[e];
      if (lane == 0)
        A.free_stack[A.free_top - (nref << DIM) + r] = ((const BlockDesc*)(A.new_base + A.new_h.off_pblk))[r].slot;
      continue;
    }
    const BlockDesc L = bd[w];
    const int l = L.level, bs1 = A.bs - 1;
    const bool act = lane < ND && lane != CEN;
    int dlt[3] = {lane % 3 - 1, lane / 3 % 3 - 1, DIM > 2 ? lane / 9 - 1 : 0};
    // same level; coarser (the parent cell of that position); finer: the children of that
    // cell on the block's side, 2^(axes with dlt = 0) of them
    int cn[3] = {0, 0, 0}, wc[3] = {0, 0, 0}, pc[3] = {0, 0, 0}, wp[3] = {0, 0, 0};
    int nz = 0;
    bool first = true;   // the first direction that reaches this parent cell
    for (int a = 0; a < DIM; ++a) {
      cn[a] = L.c[a] + dlt[a];
      wc[a] = wrapl(cn[a], l);
      pc[a] = cn[a] >> 1;   // floor division
      wp[a] = l > 1 ? wrapl(pc[a], l - 1) : 0;
      nz += dlt[a] == 0;
      if (dlt[a] == ((L.c[a] & 1) ? 0 : 1)) first = false;
    }
    const int ncand = 1 << nz;
    int beta[4][3] = {};
    int sslot = -1, cslot = -1, fslot[4] = {-1, -1, -1, -1};
    if (act) {
      sslot = A.cells[cell_of(A, l, wc)];
      if (l > 1) cslot = A.cells[cell_of(A, l - 1, wp)];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        int q = i, fc[3] = {0, 0, 0};
        for (int a = 0; a < DIM; ++a) {
          beta[i][a] = dlt[a] == 0 ? q & 1 : (dlt[a] < 0 ? 1 : 0);
          if (dlt[a] == 0) q >>= 1;
          fc[a] = 2 * wc[a] + beta[i][a];
        }
        if (l < A.jmax && i < ncand) fslot[i] = A.cells[cell_of(A, l + 1, fc)];
      }
    }
    if (sslot >= 0) cslot = -1;
    const bool keep_c = act && cslot >= 0 && first;
    const bool fine = act && sslot < 0 && cslot < 0;
    bool hole = false;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (fine && i < ncand && fslot[i] < 0) hole = true;
    // positions in the row: counts over the group's lanes below this one
    const unsigned long long all = (GL == 32 ? 0xffffffffull : 0xffffull) << sh;
    const unsigned long long below = ((1ull << lane) - 1ull) << sh;
    const unsigned long long bc = __ballot(keep_c), bsm = __ballot(act && sslot >= 0);
    const unsigned long long f1 = __ballot(fine && nz == 0), f2 = __ballot(fine && nz == 1),
                             f4 = __ballot(fine && nz == 2), bh = __ballot(hole);
    const int ncoarse = __popcll(bc & all), nsame = __popcll(bsm & all);
    const int nfine = __popcll(f1 & all) + 2 * __popcll(f2 & all) + 4 * __popcll(f4 & all);
    const int fpre = __popcll(f1 & below) + 2 * __popcll(f2 & below) + 4 * __popcll(f4 & below);
    const int nent = ncoarse + 1 + nsame + nfine;
    if (lane == 0) A.isp[w] = l < A.jmax ? 1 : 0;
    if ((bh & all) != 0 || nent > S) {
      if (lane == 0) atomicOr(A.err, 1);   // not graded, or a hole
      continue;
    }
    NbEntry* row = (NbEntry*)(A.new_base + A.new_h.off_nb) + (size_t)w * S;
    NbEntry e;
    e.o[0] = e.o[1] = e.o[2] = 0;
    if (keep_c) {
      e.slot = cslot;
      e.dl = -1;
      for (int a = 0; a < DIM; ++a) e.o[a] = (int8_t)((2 * pc[a] - L.c[a]) * bs1);
      row[__popcll(bc & below)] = e;
    } else if (act && sslot >= 0) {
      e.slot = sslot;
      e.dl = 0;
      for (int a = 0; a < DIM; ++a) e.o[a] = (int8_t)(dlt[a] * bs1);
      row[ncoarse + 1 + __popcll(bsm & below)] = e;
    } else if (fine) {
      e.dl = 1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i >= ncand) break;
        e.slot = fslot[i];
        for (int a = 0; a < DIM; ++a) e.o[a] = (int8_t)(dlt[a] * bs1 + beta[i][a] * (bs1 / 2));
        row[ncoarse + 1 + nsame + fpre + i] = e;
      }
    } else if (lane == CEN) {
      e.slot = L.slot;
      e.dl = 0;
      row[ncoarse] = e;
      BlockDesc d = L;
      d.nb_begin = w * S;
      d.n_ent = nent;
      d.n_coarse = ncoarse;
      bd[w] = d;
    }
  }
}

// fill n ints with a value
__global__ void __launch_bounds__(256) k_fill_int(int* p, size_t n, int v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

namespace {
// one thread (or `lanes` of them) per item, bounded: the whole-grid kernels stride
int item_grid(long items, int lanes) {
  const long g = (items * lanes + 255) / 256;
  return (int)(g < 1 ? 1 : g > 65536 ? 65536 : g);
}
}  // namespace

hipError_t launch_plan_refine(const DevTopoArgs& a, hipStream_t st) {
  const int per = 256 / a.nch;
  hipLaunchKernelGGL(k_plan_refine, dim3((a.old_h.n_blocks + per - 1) / per), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_plan_coarsen(const DevTopoArgs& a, hipStream_t st) {
  const int n = a.old_h.n_blocks;
  hipLaunchKernelGGL(k_coarsen_candidates, dim3(item_grid(n, 1)), dim3(256), 0, st, a);
  hipLaunchKernelGGL(k_coarsen_edges, dim3(item_grid(n, a.old_h.nb_stride <= 16 ? 16 : 64)), dim3(256), 0, st, a);
  hipLaunchKernelGGL(k_coarsen_fix, dim3(1), dim3(1024), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_coarsen_apply(const DevTopoArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_coarsen_apply, dim3((a.old_h.n_blocks + 255) / 256), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_index(const DevTopoArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_index, dim3(item_grid(a.new_h.n_blocks, 1)), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_entries(const DevTopoArgs& a, hipStream_t st) {
  const long items = (long)a.new_h.n_blocks + a.new_h.n_ref + a.new_h.n_fam;
  if (a.dim == 2) hipLaunchKernelGGL(k_entries<2>, dim3(item_grid(items, 16)), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(k_entries<3>, dim3(item_grid(items, 32)), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_fill_int(int* p, size_t n, int v, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int grid = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  hipLaunchKernelGGL(k_fill_int, dim3(grid), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

}  // namespace mrb
