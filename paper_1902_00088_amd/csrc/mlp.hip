// Learned refinement predictor on the GPU: block features (8 x 8 average pool of
// every field of the synchronised block), a nin -> 64 -> 64 -> 3 MLP with GELU,
// class-weighted softmax cross-entropy, backward pass and Adam.  FP32 arithmetic;
// the per-parameter gradient reduction over the batch accumulates in FP64 in a
// fixed order (deterministic, no atomics).  The layers are tiny (a batch of 1024 is
// ~60 MFLOP), so launches and dependent loads set the time: two launches per training
// batch, matrix instructions for the contractions.  The parameter vector layout is
// W1[nin][64], b1[64], W2[64][64], b2[64], W3[64][3], b3[3].
#include "internal.hpp"
#include "mlp.hpp"

#include <hip/hip_runtime.h>

namespace mrb {

namespace {

constexpr int HID = 64, NOUT = 3;

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

struct Off {
  int w1, b1, w2, b2, w3, b3, n;
  __device__ __host__ explicit Off(int nin) {
    w1 = 0;
    b1 = nin * HID;
    w2 = b1 + HID;
    b2 = w2 + HID * HID;
    w3 = b2 + HID;
    b3 = w3 + HID * NOUT;
    n = b3 + NOUT;
  }
};

// features of every block: gather the synchronised block (no halo) and average each
// field over 8 x 8 bins of w = (bs-1)/8 nodes (y outer, x inner, FP64)
template <int BS>
__global__ void __launch_bounds__(256) k_pool(MlpPoolArgs A) {
  constexpr int NPT = BS * BS;
  constexpr int W = (BS - 1) / 8;
  extern __shared__ __align__(16) char smem[];
  double* tile = reinterpret_cast<double*>(smem);
  const int nblk = A.topo.h.n_blocks;
  for (int b = blockIdx.x; b < nblk; b += gridDim.x) {
    const BlockDesc d = A.topo.blk()[b];
    // owner of each node: the block itself except on its boundary, where a finer
    // neighbour may hold the node; a same-level neighbour holds equal values
    for (int p = threadIdx.x; p < A.nf * NPT; p += blockDim.x) {
      const int f = p / NPT, q = p % NPT, x = q % BS, y = q / BS;
      double v = A.u[((size_t)d.slot * A.nf + f) * NPT + q];
      if (x == 0 || y == 0 || x == BS - 1 || y == BS - 1) {
        for (int e = 0; e < d.n_ent; ++e) {
          const NbEntry E = A.topo.nb(b)[e];
          if (E.dl <= 0) continue;
          const int lx = x - E.o[0], ly = y - E.o[1];
          if (lx >= 0 && lx <= (BS - 1) / 2 && ly >= 0 && ly <= (BS - 1) / 2) {
            v = A.u[((size_t)E.slot * A.nf + f) * NPT + 2 * lx + BS * 2 * ly];
            break;
          }
        }
      }
      tile[p] = v;
    }
    __syncthreads();
    for (int p = threadIdx.x; p < A.nf * 64; p += blockDim.x) {
      const int f = p / 64, bin = p % 64, bx = bin % 8, by = bin / 8;
      double s = 0.0;
      for (int y = by * W; y < by * W + W; ++y)
        for (int x = bx * W; x < bx * W + W; ++x) s = s + tile[f * NPT + y * BS + x];
      A.feat[(size_t)b * A.nf * 64 + p] = (float)(s / (double)(W * W));
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Forward pass (and, with TRAIN, loss and deltas) of 16 samples per workgroup.  The
// layers are contractions over the inputs, so they run on the FP32 matrix cores
// (16 x 16 x 4): the rows of a tile are the samples, wave w owns hidden units
// 16w .. 16w + 15.  A lane of group q = lane / 16 takes reduction index 16 q + t at step
// t of a 64-wide slice, so that it reads its activations (LDS) and, for the transposed
// product of the backward pass, its weights (cache) four floats at a time.  The tile's
// accumulators keep z1 and z2 in registers from the forward to the backward part.  A
// batch of 1,024 samples is 64 workgroups of four waves: latency bound (weights through
// L2), so every weight and input is requested up front; 1,024 x 256 inputs with loss and
// deltas take 10.7 us, against 76 us for one wave per sample with a serial loop over the
// inputs plus 4.5 us each for the loss's and the deltas' launches.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int MS = 16;             // samples per workgroup
constexpr int AST = HID + 4;       // LDS row stride of the activations (bank spread)

// This lane's weights of one 64-wide slice: column b (stride bstride) in k, or with a
// stride of 1 its row of the transposed weights
__device__ __forceinline__ void wload(float* bv, const float* b, int bstride) {
  const int q = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int t = 0; t < 16; ++t) bv[t] = b[(16 * q + t) * bstride];
}

// acc += A B over one 64-wide slice: A's row (this lane's sample) at arow, B from wload
__device__ __forceinline__ f32x4 mm64(f32x4 acc, const float* arow, const float* bv) {
  const int q = (threadIdx.x & 63) >> 4;
  f32x4 av[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) av[t] = *(const f32x4*)(arow + 16 * q + 4 * t);
#pragma unroll
  for (int t = 0; t < 16; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t >> 2][t & 3], bv[t], acc, 0, 0, 0);
  return acc;
}

// NS: 64-wide slices of the inputs (one per field).  A wave's weights are loaded once, all
// in flight together, before the samples.
template <bool TRAIN, int NS>
__global__ void __launch_bounds__(256) k_fwd(MlpArgs A) {
  extern __shared__ __align__(16) char smem[];
  const Off o(A.nin);
  constexpr int NIN = 64 * NS, XST = NIN + 4;
  float* xs = reinterpret_cast<float*>(smem);       // [MS][nin + 4] normalised features
  float* a1s = xs + MS * XST;                       // [MS][AST]; later dz2
  float* a2s = a1s + MS * AST;
  float* ls = a2s + MS * AST;                       // [MS][4] logits, then dL/dlogits
  float* w3s = ls + MS * 4;                         // [HID][NOUT] output weights
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int col = lane & 15, q = lane >> 4, j = 16 * w + col;
  float v1[NS][16], v2[16], v2t[16];
#pragma unroll
  for (int k = 0; k < NS; ++k) wload(v1[k], A.p + o.w1 + k * 64 * HID + j, HID);
  wload(v2, A.p + o.w2 + j, HID);
  if (TRAIN) wload(v2t, A.p + o.w2 + j * HID, 1);
  const float b1 = A.p[o.b1 + j], b2 = A.p[o.b2 + j];
  if (tid < HID * NOUT) w3s[tid] = A.p[o.w3 + tid];
  for (int s0 = blockIdx.x * MS; s0 < A.n; s0 += gridDim.x * MS) {
    // (rows past the batch hold zeros; their results are not stored)
    // (every input of the workgroup requested before the first is used)
    constexpr int RI = 4 / NS;   // rows per round of 256 threads
    const int k = tid % NIN, f = k / 64;
    const float mean = A.mean[f], sd = A.std[f];
    float xv[MS / RI];
#pragma unroll
    for (int i = 0; i < MS / RI; ++i)
      xv[i] = A.x[(size_t)min(s0 + i * RI + tid / NIN, A.n - 1) * NIN + k];
#pragma unroll
    for (int i = 0; i < MS / RI; ++i) {
      const int r = i * RI + tid / NIN;
      const float xn = s0 + r < A.n ? (xv[i] - mean) / sd : 0.0f;
      if (TRAIN && s0 + r < A.n) A.xn[(size_t)(s0 + r) * NIN + k] = xn;
      xs[r * XST + k] = xn;
    }
    __syncthreads();
    // accumulator element v of a lane: sample 4 q + v, hidden unit j
    f32x4 z1 = {b1, b1, b1, b1};
#pragma unroll
    for (int k = 0; k < NS; ++k) z1 = mm64(z1, xs + col * XST + 64 * k, v1[k]);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 4 * q + v;
      const float g = gelu(z1[v]);
      a1s[r * AST + j] = g;
      if (TRAIN && s0 + r < A.n) A.a1[(size_t)(s0 + r) * HID + j] = g;
    }
    __syncthreads();
    f32x4 z2 = {b2, b2, b2, b2};
    z2 = mm64(z2, a1s + col * AST, v2);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 4 * q + v;
      const float g = gelu(z2[v]);
      a2s[r * AST + j] = g;
      if (TRAIN && s0 + r < A.n) A.a2[(size_t)(s0 + r) * HID + j] = g;
    }
    __syncthreads();
    if (tid < MS * NOUT) {
      const int r = tid / NOUT, c = tid % NOUT;
      float l = A.p[o.b3 + c];
#pragma unroll 16
      for (int k = 0; k < HID; ++k) l = l + a2s[r * AST + k] * w3s[k * NOUT + c];
      ls[r * 4 + c] = l;
      if (s0 + r < A.n) A.logits[(size_t)(s0 + r) * NOUT + c] = l;
    }
    __syncthreads();
    if constexpr (TRAIN) {
      // weighted softmax cross-entropy: per-sample loss and dL/dlogits
      if (tid < MS) {
        float dl[NOUT] = {0.0f, 0.0f, 0.0f};
        if (s0 + tid < A.n) {
          const int b = s0 + tid;
          const float* l = ls + tid * 4;
          const float m = fmaxf(l[0], fmaxf(l[1], l[2]));
          const float e0 = expf(l[0] - m), e1 = expf(l[1] - m), e2 = expf(l[2] - m);
          const float s = e0 + e1 + e2;
          const float pr[3] = {e0 / s, e1 / s, e2 / s};
          const int y = A.y[b];
          const float cw = A.classw[y];
          A.loss[b] = -logf(y == 0 ? pr[0] : (y == 1 ? pr[1] : pr[2])) * cw * A.inv_wsum;
          for (int c = 0; c < NOUT; ++c) {
            dl[c] = (pr[c] - (c == y ? 1.0f : 0.0f)) * (cw * A.inv_wsum);
            A.dl[(size_t)b * NOUT + c] = dl[c];
          }
        }
        for (int c = 0; c < NOUT; ++c) ls[tid * 4 + c] = dl[c];
      }
      __syncthreads();
      // dz2 (into a1s, last read two barriers ago), then dz1 = (dz2 W2^T) gelu'(z1)
      const float w30 = w3s[j * NOUT], w31 = w3s[j * NOUT + 1], w32 = w3s[j * NOUT + 2];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 4 * q + v;
        const float* dl = ls + r * 4;
        float da2 = 0.0f;
        da2 = da2 + dl[0] * w30;
        da2 = da2 + dl[1] * w31;
        da2 = da2 + dl[2] * w32;
        const float d2 = da2 * gelu_grad(z2[v]);
        a1s[r * AST + j] = d2;
        if (s0 + r < A.n) A.dz2[(size_t)(s0 + r) * HID + j] = d2;
      }
      __syncthreads();
      f32x4 da1 = {0.0f, 0.0f, 0.0f, 0.0f};
      da1 = mm64(da1, a1s + col * AST, v2t);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 4 * q + v;
        if (s0 + r < A.n) A.dz1[(size_t)(s0 + r) * HID + j] = da1[v] * gelu_grad(z1[v]);
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Parameter gradients, and with `adam` their Adam update.  Each weight matrix's
// gradient is X^T D over the batch: FP64 matrix cores (16 x 16 x 4) on the FP32 factors
// (their products are exact in FP64), one workgroup per 16 x 16 tile of a weight matrix
// or 16 biases (X = 1), the batch split over its 16 waves and the partial sums added in
// wave order, so the result does not depend on scheduling.  Latency bound: 93 workgroups
// (four fields), 64 samples a wave; a batch of 1,024 takes 6.7 us with the update
// folded in, against 269 us for one thread per parameter walking the whole batch (and
// 4.7 us for the update's own launch).
// ---------------------------------------------------------------------------
constexpr int GW = 16;    // waves per workgroup

__global__ void __launch_bounds__(64 * GW) k_wgrad(MlpArgs A, MlpAdamArgs D) {
  __shared__ double part[GW][256];
  const Off o(A.nin);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, col = lane & 15, q = lane >> 4;
  // this workgroup's tile: factors X [n][xs] (null: ones) at column x0, D [n][ds] at d0
  // (dn live columns), gradient g[g0 + row * gs + column]
  const int n1 = (A.nin / 16) * 4;
  int t = blockIdx.x;
  const float *X = nullptr, *Dz;
  int xs = 0, x0 = 0, ds = HID, d0, dn = 16, g0, gs = HID;
  if (t < n1) {
    X = A.xn; xs = A.nin; x0 = 16 * (t / 4); Dz = A.dz1; d0 = 16 * (t % 4); g0 = o.w1 + x0 * HID + d0;
  } else if ((t -= n1) < 16) {
    X = A.a1; xs = HID; x0 = 16 * (t / 4); Dz = A.dz2; d0 = 16 * (t % 4); g0 = o.w2 + x0 * HID + d0;
  } else if ((t -= 16) < 4) {
    X = A.a2; xs = HID; x0 = 16 * t; Dz = A.dl; ds = NOUT; d0 = 0; dn = NOUT; g0 = o.w3 + x0 * NOUT; gs = NOUT;
  } else if ((t -= 4) < 4) {
    Dz = A.dz1; d0 = 16 * t; g0 = o.b1 + d0;
  } else if ((t -= 4) < 4) {
    Dz = A.dz2; d0 = 16 * t; g0 = o.b2 + d0;
  } else {
    Dz = A.dl; ds = NOUT; d0 = 0; dn = NOUT; g0 = o.b3;
  }
  // this thread's parameter of the tile (the first 256 threads), its Adam state requested
  // before the sums need it
  const int prow = threadIdx.x >> 4, pc = threadIdx.x & 15, p = g0 + prow * gs + pc;
  const bool mine = threadIdx.x < 256 && pc < dn && (X || prow == 0);
  float pm = 0.0f, pv = 0.0f, pp = 0.0f;
  if (mine && D.p) {
    pm = D.m[p];
    pv = D.v[p];
    pp = D.p[p];
  }
  const int chunk = ((A.n + 4 * GW - 1) / (4 * GW)) * 4;   // samples per wave
  const int b0 = w * chunk, b1 = min(A.n, b0 + chunk);
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  const float* Xp = X ? X : Dz;   // (a bias loads the other factor and discards it)
  const int xc = X ? x0 + col : d0;
  if (!X) xs = ds;
  constexpr int U = 16;
  for (int b = b0; b < b1; b += 4 * U) {
    float xv[U], dv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // this lane's sample of the step (past the share's end, the batch's last, dropped)
      const int s = min(b + 4 * u + q, A.n - 1);
      xv[u] = Xp[(size_t)s * xs + xc];
      dv[u] = Dz[(size_t)s * ds + d0 + min(col, dn - 1)];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = b + 4 * u + q < b1;
      xv[u] = ok ? (X ? xv[u] : 1.0f) : 0.0f;
      dv[u] = ok && col < dn ? dv[u] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)xv[u], (double)dv[u], acc, 0, 0, 0);
  }
  // accumulator element v of a lane: row 4 v + q, column col
#pragma unroll
  for (int v = 0; v < 4; ++v) part[w][(4 * v + q) * 16 + col] = acc[v];
  __syncthreads();
  if (mine) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < GW; ++k) s += part[k][threadIdx.x];
    const float g = (float)s;
    A.g[p] = g;
    if (D.p) {
      const float m = D.b1 * pm + (1.0f - D.b1) * g;
      const float v = D.b2 * pv + (1.0f - D.b2) * g * g;
      D.m[p] = m;
      D.v[p] = v;
      D.p[p] = pp - D.lr * (m / D.bc1) / (sqrtf(v / D.bc2) + D.eps);
    }
  }
}

// prediction from logits: argmax class and its softmax probability
__global__ void __launch_bounds__(256) k_pred(const float* logits, int n, int8_t* pred, float* pmax) {
  for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < n; b += gridDim.x * blockDim.x) {
    const float* l = logits + (size_t)b * NOUT;
    int c = 0;
    if (l[1] > l[c]) c = 1;
    if (l[2] > l[c]) c = 2;
    const float s = expf(l[0] - l[c]) + expf(l[1] - l[c]) + expf(l[2] - l[c]);
    pred[b] = (int8_t)c;
    pmax[b] = 1.0f / s;
  }
}

}  // namespace

int mlp_param_count(int nin) { return Off(nin).n; }

hipError_t launch_pred(const float* logits, int n, int8_t* pred, float* pmax, hipStream_t st) {
  const int g = (n + 255) / 256;
  hipLaunchKernelGGL(k_pred, dim3(g > 0 ? g : 1), dim3(256), 0, st, logits, n, pred, pmax);
  return hipGetLastError();
}

hipError_t launch_pool(int bs, int grid, const MlpPoolArgs& a, hipStream_t st) {
  const size_t lds = sizeof(double) * a.nf * bs * bs;
  if (bs == 33) hipLaunchKernelGGL(k_pool<33>, dim3(grid), dim3(256), lds, st, a);
  else if (bs == 17) hipLaunchKernelGGL(k_pool<17>, dim3(grid), dim3(256), lds, st, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// workgroups and dynamic LDS of the forward kernel
static void fwd_shape(const MlpArgs& a, int* grid, size_t* lds) {
  const int g = (a.n + MS - 1) / MS;
  *grid = g < 4096 ? (g > 0 ? g : 1) : 4096;
  *lds = sizeof(float) * ((size_t)MS * (a.nin + 4) + 2 * MS * AST + MS * 4 + HID * NOUT);
}

template <bool TRAIN>
static hipError_t fwd_go(const MlpArgs& a, hipStream_t st) {
  int grid;
  size_t lds;
  fwd_shape(a, &grid, &lds);
  if (a.nin == 64) hipLaunchKernelGGL((k_fwd<TRAIN, 1>), dim3(grid), dim3(256), lds, st, a);
  else if (a.nin == 256) hipLaunchKernelGGL((k_fwd<TRAIN, 4>), dim3(grid), dim3(256), lds, st, a);
  else return hipErrorInvalidValue;   // one or four fields
  return hipGetLastError();
}

hipError_t launch_mlp_forward(const MlpArgs& a, hipStream_t st) { return fwd_go<false>(a, st); }

hipError_t launch_mlp_train(const MlpArgs& a, const MlpAdamArgs& adam, hipStream_t st) {
  hipError_t e = fwd_go<true>(a, st);
  if (e != hipSuccess) return e;
  const int tiles = (a.nin / 16) * 4 + 16 + 4 + 4 + 4 + 1;   // W1, W2, W3, b1, b2, b3
  hipLaunchKernelGGL(k_wgrad, dim3(tiles), dim3(64 * GW), 0, st, a, adam);
  return hipGetLastError();
}

}  // namespace mrb
