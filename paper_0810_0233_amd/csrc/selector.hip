// selector.hip -- learned per-smallest-cell choice of local order and opening
// angle, and the pieces it is trained from.
//
// The paper chooses (p_m, alpha_m) once for a whole system from timing and the
// error estimate [alpha/(2-alpha)]^p (Sec. 4).  Here a small MLP predicts, for
// every smallest cell, log10 of the relative RMS field error of that cell for
// each candidate pair (p, theta) in {2..6} x {0.3..0.7}; the cheapest pair
// whose prediction meets the bound (with a margin) is used for that cell.  The
// levels above keep the plan's fixed (p, theta); a cell's theta re-splits its
// own candidates into near and far cells and its p truncates its local
// expansion.  Features, network forward/backward, optimiser and selection all
// run in the kernels below.
#include <algorithm>
#include <cmath>

#include "plan.hpp"

namespace ccfmm {

constexpr int kIn = CCFMM_MLP_IN, kH = CCFMM_MLP_HIDDEN, kOut = CCFMM_MLP_OUT;
constexpr int kParams = kH * kIn + kH + kH * kH + kH + kOut * kH + kOut;
// packed parameter offsets: W1 [kH][kIn], b1, W2 [kH][kH], b2, W3 [kOut][kH], b3
constexpr int oW1 = 0, ob1 = oW1 + kH * kIn, oW2 = ob1 + kH, ob2 = oW2 + kH * kH, oW3 = ob2 + kH,
              ob3 = oW3 + kOut * kH;
static_assert(ob3 + kOut == kParams, "parameter packing");

__device__ constexpr double kThetaSet[5] = {0.3, 0.4, 0.5, 0.6, 0.7};

// ---------------------------------------------------------------- per-cell data
__global__ void k_leaf_ids(int64_t n, const int32_t* __restrict__ dleaf, const int32_t* __restrict__ perm,
                           int32_t* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[perm[i]] = dleaf[i];
}

// per cell: sum over its dipoles and the configurations of |H - Href|^2 and |Href|^2
__global__ void k_leaf_err(int32_t nl, int64_t n, int nb, const int32_t* __restrict__ lstart,
                           const int32_t* __restrict__ lcount, const int32_t* __restrict__ perm,
                           const double* __restrict__ H, const double* __restrict__ Href, double* num, double* den) {
  const int l = blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= nl) return;
  double a = 0.0, b2 = 0.0;
  for (int k = 0; k < lcount[l]; k++) {
    const int64_t i = perm[lstart[l] + k];
    for (int b = 0; b < nb; b++) {
      const int64_t o = ((int64_t)b * n + i) * 3;
      for (int c = 0; c < 3; c++) {
        const double d = H[o + c] - Href[o + c];
        a += d * d;
        b2 += Href[o + c] * Href[o + c];
      }
    }
  }
  num[l] = a;
  den[l] = b2;
}

// Eight features of a smallest cell (computed on the fixed-parameter lists):
// log2(1+count), log2(1+near sources), near cells/64, far cells/64, |mean m|,
// moment variance, log2 of count over mean near occupancy, level/16.
__global__ void k_leaf_features(int32_t nl, int64_t n, int nb, int L, const int32_t* __restrict__ lstart,
                                const int32_t* __restrict__ lcount, const int32_t* __restrict__ near_ptr,
                                const int32_t* __restrict__ near_idx, const int32_t* __restrict__ far_ptr,
                                const int32_t* __restrict__ perm, const double* __restrict__ m, float* feat) {
  const int l = blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= nl) return;
  const int c = lcount[l];
  int64_t nsrc = 0;
  const int nnear = near_ptr[l + 1] - near_ptr[l];
  for (int e = near_ptr[l]; e < near_ptr[l + 1]; e++) nsrc += lcount[near_idx[e]];
  const int nfar = far_ptr[l + 1] - far_ptr[l];
  double sx = 0, sy = 0, sz = 0, s2 = 0;
  for (int k = 0; k < c; k++) {
    const int64_t i = perm[lstart[l] + k];
    for (int b = 0; b < nb; b++) {
      const double* mi = m + ((int64_t)b * n + i) * 3;
      sx += mi[0];
      sy += mi[1];
      sz += mi[2];
      s2 += mi[0] * mi[0] + mi[1] * mi[1] + mi[2] * mi[2];
    }
  }
  const double cnt = (double)c * nb;
  const double mx = sx / cnt, my = sy / cnt, mz = sz / cnt;
  const double mm = sqrt(mx * mx + my * my + mz * mz);
  const double var = s2 / cnt - mm * mm;
  const double mean_near = (double)nsrc / (double)max(1, nnear);
  float* f = feat + (int64_t)l * kIn;
  f[0] = (float)log2(1.0 + c);
  f[1] = (float)log2(1.0 + (double)nsrc);
  f[2] = (float)(nnear / 64.0);
  f[3] = (float)(nfar / 64.0);
  f[4] = (float)mm;
  f[5] = (float)var;
  f[6] = (float)(log2(1.0 + c) - log2(1.0 + mean_near));
  f[7] = (float)(L / 16.0);
}

// ---------------------------------------------------------------- MLP
__device__ __forceinline__ void mlp_row(const float* __restrict__ P, const float* x, float* a1, float* a2, float* y) {
  for (int j = 0; j < kH; j++) {
    float s = P[ob1 + j];
    for (int i = 0; i < kIn; i++) s += P[oW1 + j * kIn + i] * x[i];
    a1[j] = s > 0.f ? s : 0.f;
  }
  for (int j = 0; j < kH; j++) {
    float s = P[ob2 + j];
    for (int i = 0; i < kH; i++) s += P[oW2 + j * kH + i] * a1[i];
    a2[j] = s > 0.f ? s : 0.f;
  }
  for (int o = 0; o < kOut; o++) {
    float s = P[ob3 + o];
    for (int i = 0; i < kH; i++) s += P[oW3 + o * kH + i] * a2[i];
    y[o] = s;
  }
}

__global__ void __launch_bounds__(64) k_mlp_forward(const float* __restrict__ params, int64_t rows,
                                                    const float* __restrict__ x, float* __restrict__ y) {
  __shared__ float P[kParams];
  for (int q = threadIdx.x; q < kParams; q += blockDim.x) P[q] = params[q];
  __syncthreads();
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  float a1[kH], a2[kH], xr[kIn];
  for (int i = 0; i < kIn; i++) xr[i] = x[r * kIn + i];
  mlp_row(P, xr, a1, a2, y + r * kOut);
}

// Masked squared error: loss = sum mask (y - t)^2 / 2 / max(1, sum mask).
// A block takes kGR rows through the forward pass, the back-propagated deltas
// and its share of every parameter gradient, activations and weights in LDS; a
// wavefront works on 8 rows of a layer with one unit per lane, so a weight is
// read once for 8 rows and the activations are broadcast reads.  Gradients and
// loss are formed unscaled: the normalisation (a sum over the whole mask) is
// applied by the second kernel, which adds the blocks' shares in a fixed order
// in FP64, so no pass over the mask comes first.  8,192 rows: a step took 223
// us in four kernels (90 of them one block summing the mask, 97 with one
// thread per row in a quarter of each block's threads).
constexpr int kGR = 32;        // rows per gradient block
constexpr int kGA = kH + 4;    // padded row of activations (16-byte rows)
constexpr int kGW = kH + 1;    // padded row of weights
struct GradShare {
  double loss, mask;
};

__global__ void __launch_bounds__(256) k_mlp_grad_part(const float* __restrict__ params, int64_t rows,
                                                       const float* __restrict__ x, const float* __restrict__ t,
                                                       const float* __restrict__ mask, float* __restrict__ part,
                                                       GradShare* __restrict__ share) {
  __shared__ __attribute__((aligned(16))) float a1[kGR][kGA], a2[kGR][kGA], d1[kGR][kGA], d2[kGR][kGA];
  __shared__ float sx[kGR][kIn], sdy[kGR][kOut + 3], w2[kH][kGW], w3[kOut][kGW];
  __shared__ double sl[256], sm[256];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kGR;
  for (int q = tid; q < kH * kH; q += 256) w2[q / kH][q % kH] = params[oW2 + q];
  for (int q = tid; q < kOut * kH; q += 256) w3[q / kH][q % kH] = params[oW3 + q];
  for (int q = tid; q < kGR * kIn; q += 256) sx[q / kIn][q % kIn] = r0 + q / kIn < rows ? x[r0 * kIn + q] : 0.f;
  float w1[kIn];
#pragma unroll
  for (int i = 0; i < kIn; i++) w1[i] = params[oW1 + lane * kIn + i];
  const float c1 = params[ob1 + lane], c2 = params[ob2 + lane];
  __syncthreads();
  const int rb = 8 * w;  // this wavefront's rows; lane = unit
#pragma unroll
  for (int r = 0; r < 8; r++) {
    float s = c1;
#pragma unroll
    for (int i = 0; i < kIn; i++) s += w1[i] * sx[rb + r][i];
    a1[rb + r][lane] = s > 0.f ? s : 0.f;
  }
  __syncthreads();
  {
    float s[8];
#pragma unroll
    for (int r = 0; r < 8; r++) s[r] = c2;
    for (int i = 0; i < kH; i += 4) {
      float wv[4];
#pragma unroll
      for (int u = 0; u < 4; u++) wv[u] = w2[lane][i + u];
#pragma unroll
      for (int r = 0; r < 8; r++) {
        const float4 v = *reinterpret_cast<const float4*>(&a1[rb + r][i]);
        s[r] += wv[0] * v.x;
        s[r] += wv[1] * v.y;
        s[r] += wv[2] * v.z;
        s[r] += wv[3] * v.w;
      }
    }
#pragma unroll
    for (int r = 0; r < 8; r++) a2[rb + r][lane] = s[r] > 0.f ? s[r] : 0.f;
  }
  __syncthreads();
  double l = 0.0, mk = 0.0;
  {  // outputs: half a wavefront per 4 rows
    const int o = tid & 31, rq = 4 * (tid >> 5);
    if (o < kOut) {
      float s[4];
#pragma unroll
      for (int r = 0; r < 4; r++) s[r] = params[ob3 + o];
      for (int i = 0; i < kH; i++) {
        const float wv = w3[o][i];
#pragma unroll
        for (int r = 0; r < 4; r++) s[r] += wv * a2[rq + r][i];
      }
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int64_t row = r0 + rq + r;
        float dy = 0.f;
        if (row < rows) {
          const float e = s[r] - t[row * kOut + o];
          const float wm = mask[row * kOut + o];
          l += 0.5 * (double)wm * (double)e * (double)e;
          mk += (double)wm;
          dy = wm * e;
        }
        sdy[rq + r][o] = dy;
      }
    }
  }
  sl[tid] = l;
  sm[tid] = mk;
  __syncthreads();
  {
    float s[8];
#pragma unroll
    for (int r = 0; r < 8; r++) s[r] = 0.f;
    for (int o = 0; o < kOut; o++) {
      const float wv = w3[o][lane];
#pragma unroll
      for (int r = 0; r < 8; r++) s[r] += wv * sdy[rb + r][o];
    }
#pragma unroll
    for (int r = 0; r < 8; r++) d2[rb + r][lane] = a2[rb + r][lane] > 0.f ? s[r] : 0.f;
  }
  for (int off = 128; off > 0; off >>= 1) {
    __syncthreads();
    if (tid < off) {
      sl[tid] += sl[tid + off];
      sm[tid] += sm[tid + off];
    }
  }
  __syncthreads();
  {
    float s[8];
#pragma unroll
    for (int r = 0; r < 8; r++) s[r] = 0.f;
    for (int j = 0; j < kH; j += 4) {
      float wv[4];
#pragma unroll
      for (int u = 0; u < 4; u++) wv[u] = w2[j + u][lane];
#pragma unroll
      for (int r = 0; r < 8; r++) {
        const float4 v = *reinterpret_cast<const float4*>(&d2[rb + r][j]);
        s[r] += wv[0] * v.x;
        s[r] += wv[1] * v.y;
        s[r] += wv[2] * v.z;
        s[r] += wv[3] * v.w;
      }
    }
#pragma unroll
    for (int r = 0; r < 8; r++) d1[rb + r][lane] = a1[rb + r][lane] > 0.f ? s[r] : 0.f;
  }
  __syncthreads();
  float* g = part + (int64_t)blockIdx.x * kParams;
  {  // W2: a 4 x 4 tile per thread
    const int j0 = 4 * (tid >> 4), i0 = 4 * (tid & 15);
    float s[4][4] = {};
    for (int r = 0; r < kGR; r++) {
      const float4 u = *reinterpret_cast<const float4*>(&d2[r][j0]);
      const float4 v = *reinterpret_cast<const float4*>(&a1[r][i0]);
      const float uu[4] = {u.x, u.y, u.z, u.w}, vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int p = 0; p < 4; p++)
#pragma unroll
        for (int q = 0; q < 4; q++) s[p][q] += uu[p] * vv[q];
    }
#pragma unroll
    for (int p = 0; p < 4; p++)
#pragma unroll
      for (int q = 0; q < 4; q++) g[oW2 + (j0 + p) * kH + i0 + q] = s[p][q];
  }
  {  // W3 (and b3): outputs w, w + 4, ... of input unit `lane`
    constexpr int NO = (kOut + 3) / 4;
    float s[NO] = {}, sb[NO] = {};
    for (int r = 0; r < kGR; r++) {
      const float v = a2[r][lane];
#pragma unroll
      for (int q = 0; q < NO; q++) {
        const float dy = w + 4 * q < kOut ? sdy[r][w + 4 * q] : 0.f;
        s[q] += dy * v;
        sb[q] += dy;
      }
    }
#pragma unroll
    for (int q = 0; q < NO; q++) {
      const int o = w + 4 * q;
      if (o < kOut) {
        g[oW3 + o * kH + lane] = s[q];
        if (lane == 0) g[ob3 + o] = sb[q];
      }
    }
  }
  {  // W1: inputs 2 w and 2 w + 1 of unit `lane`; b1 and b2 beside them
    float s0 = 0.f, s1 = 0.f, sb = 0.f;
    for (int r = 0; r < kGR; r++) {
      const float v = d1[r][lane];
      s0 += v * sx[r][2 * w];
      s1 += v * sx[r][2 * w + 1];
      sb += w == 1 ? d2[r][lane] : v;
    }
    g[oW1 + lane * kIn + 2 * w] = s0;
    g[oW1 + lane * kIn + 2 * w + 1] = s1;
    if (w < 2) g[(w == 0 ? ob1 : ob2) + lane] = sb;
  }
  if (tid == 0) share[blockIdx.x] = GradShare{sl[0], sm[0]};
}

// 64 parameters per block, 16 wavefronts that take every 16th block's share;
// the sums, in a fixed order, are scaled by 1 / max(1, sum mask)
__global__ void __launch_bounds__(1024) k_mlp_grad_sum(int nblk, const float* __restrict__ part,
                                                       const GradShare* __restrict__ share, float* __restrict__ grad,
                                                       float* __restrict__ loss) {
  __shared__ double sg[16][64], sl[1024], sm[1024];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int q = blockIdx.x * 64 + lane;
  double g = 0.0, l = 0.0, m = 0.0;
  if (q < kParams)
    for (int b = w; b < nblk; b += 16) g += (double)part[(int64_t)b * kParams + q];
  for (int b = tid; b < nblk; b += 1024) {
    l += share[b].loss;
    m += share[b].mask;
  }
  sg[w][lane] = g;
  sl[tid] = l;
  sm[tid] = m;
  for (int off = 512; off > 0; off >>= 1) {
    __syncthreads();
    if (tid < off) {
      sl[tid] += sl[tid + off];
      sm[tid] += sm[tid + off];
    }
  }
  __syncthreads();
  const double inv = 1.0 / (sm[0] > 1.0 ? sm[0] : 1.0);
  if (w == 0 && q < kParams) {
    double s = 0.0;
    for (int k = 0; k < 16; k++) s += sg[k][lane];
    grad[q] = (float)(s * inv);
  }
  if (blockIdx.x == 0 && tid == 0 && loss) loss[0] = (float)(sl[0] * inv);
}

// Adam step (bias-corrected), one thread per parameter.
__global__ void k_adam(float* __restrict__ params, const float* __restrict__ grad, float* __restrict__ m1,
                       float* __restrict__ m2, int step, float lr, float b1, float b2, float eps) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= kParams) return;
  const float g = grad[q];
  const float a = b1 * m1[q] + (1.f - b1) * g;
  const float v = b2 * m2[q] + (1.f - b2) * g * g;
  m1[q] = a;
  m2[q] = v;
  const float ah = a / (1.f - powf(b1, (float)step));
  const float vh = v / (1.f - powf(b2, (float)step));
  params[q] -= lr * ah / (sqrtf(vh) + eps);
}

// ---------------------------------------------------------------- selection
struct SelectArgs {
  const int32_t* parent;      // smallest level
  const int32_t* coord;
  const int32_t* pnear_ptr;   // level above
  const int32_t* pnear_idx;
  const int32_t* pchild;
  const int32_t* lcount;      // smallest cells
  int32_t nl;
  int L;
  double log_bound;           // log10(err_bound) - margin
  double cost_far;            // cost of one far (M2L) cell relative to one dipole pair
  double far_share[5];        // share of that cost a cell of order 2..6 takes (its M2L rows)
  int pmax;
};

__device__ __forceinline__ bool near_test(const LevelGeom& lg, double th2, int dx, int dy, int dz) {
#pragma clang fp contract(off)
  const double ax = (double)dx * lg.g[0];
  const double ay = (double)dy * lg.g[1];
  const double az = (double)dz * lg.g[2];
  double D = ax * ax;
  D = D + ay * ay;
  D = D + az * az;
  double R = lg.g[0] * lg.g[0];
  R = R + lg.g[1] * lg.g[1];
  R = R + lg.g[2] * lg.g[2];
  return !(th2 * D >= R);
}

// Per cell and candidate (p, theta): the work it costs, in direct-pair
// units: own dipoles x near source dipoles at that angle, plus cost_far per
// far cell (scaled by the share of the M2L rows order p needs), plus the smooth field at order p (an FMA triple per monomial of
// degree <= p-1 and own dipole, weighed against the ~23 vector operations of
// one pair).  Candidates above the plan's order cost +inf (never chosen).
constexpr double kL2PPairFrac = 3.0 / 23.0;

__global__ void k_cand_costs(SelectArgs a, TreeGeom G, double* __restrict__ cost) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= a.nl) return;
  const LevelGeom& lg = G.lev[a.L];
  double th2[5];
  for (int q = 0; q < 5; q++) th2[q] = kThetaSet[q] * kThetaSet[q];
  double near_src[5] = {0, 0, 0, 0, 0}, far_cells[5] = {0, 0, 0, 0, 0};
  const int pc = a.parent[c];
  const int cx = a.coord[3 * c], cy = a.coord[3 * c + 1], cz = a.coord[3 * c + 2];
  for (int e = a.pnear_ptr[pc]; e < a.pnear_ptr[pc + 1]; e++) {
    for (int s = 0; s < 2; s++) {
      const int X = a.pchild[2 * a.pnear_idx[e] + s];
      if (X < 0) continue;
      const int dx = a.coord[3 * X] - cx, dy = a.coord[3 * X + 1] - cy, dz = a.coord[3 * X + 2] - cz;
      for (int q = 0; q < 5; q++) {
        if (near_test(lg, th2[q], dx, dy, dz))
          near_src[q] += a.lcount[X];
        else
          far_cells[q] += 1.0;
      }
    }
  }
  const double own = a.lcount[c];
  for (int p = 2; p <= 6; p++)
    for (int q = 0; q < 5; q++) {
      const double l2p = own * kL2PPairFrac * (double)ncoef(p - 1);
      cost[(int64_t)c * kOut + (p - 2) * 5 + q] =
          p > a.pmax ? INFINITY : own * near_src[q] + a.cost_far * a.far_share[p - 2] * far_cells[q] + l2p;
    }
}

// The candidate of cell c for multiplier lam: the least cost + lam E, with
// E = F_c 10^(2 y) the cell's predicted squared field error (F_c its squared
// fixed-parameter field, y the predicted log10 relative error); ties go to
// the smaller E.  lam < 0 asks for the most accurate candidate (ties to the
// higher order, then the smaller angle).
__device__ __forceinline__ int lagrange_pick(int c, double lam, const double* __restrict__ cost,
                                             const float* __restrict__ pred, const double* __restrict__ F,
                                             double& e_out) {
  int best = -1;
  double bv = INFINITY, be = INFINITY;
  const double f = F[c];
  for (int k = 0; k < kOut; k++) {
    const double ck = cost[(int64_t)c * kOut + k];
    if (!(ck < INFINITY)) continue;
    const double ek = f * exp10(2.0 * (double)pred[(int64_t)c * kOut + k]);
    bool take;
    if (lam < 0.0)  // equal predictions: the higher order, then the smaller angle (k = 5 (p - 2) + angle)
      take = ek < be || (ek == be && (best < 0 || k / 5 > best / 5 || (k / 5 == best / 5 && k % 5 < best % 5)));
    else {
      const double v = lam > 0.0 ? ck + lam * ek : ck;
      take = v < bv || (v == bv && ek < be);
      if (take) bv = v;
    }
    if (take) {
      be = ek;
      best = k;
    }
  }
  e_out = be;
  return best;
}

constexpr int kLagBlocks = 256;

// partial sums (fixed order) of the chosen cells' predicted squared errors
__global__ void __launch_bounds__(256) k_lagrange_sum(int nl, double lam, const double* __restrict__ cost,
                                                      const float* __restrict__ pred, const double* __restrict__ F,
                                                      double* __restrict__ part) {
  __shared__ double se[256];
  double e = 0.0;
  for (int c = blockIdx.x * 256 + threadIdx.x; c < nl; c += gridDim.x * 256) {
    double ec;
    (void)lagrange_pick(c, lam, cost, pred, F, ec);
    e += ec;
  }
  se[threadIdx.x] = e;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) se[threadIdx.x] += se[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = se[0];
}

// the final choice for multiplier lam
__global__ void k_lagrange_choose(int nl, double lam, const double* __restrict__ cost, const float* __restrict__ pred,
                                  const double* __restrict__ F, int32_t* out_p, double* out_theta, int32_t* hist) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nl) return;
  double ec;
  const int k = lagrange_pick(c, lam, cost, pred, F, ec);
  out_p[c] = 2 + k / 5;
  out_theta[c] = kThetaSet[k % 5];
  atomicAdd(&hist[k], 1);
}

__global__ void k_diff_sums(int64_t count, const double* __restrict__ A, const double* __restrict__ B, double* part) {
  __shared__ double s1[256], s2[256];
  double a = 0.0, b = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) {
    const double d = A[i] - B[i];
    a += d * d;
    b += B[i] * B[i];
  }
  s1[threadIdx.x] = a;
  s2[threadIdx.x] = b;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) {
      s1[threadIdx.x] += s1[threadIdx.x + off];
      s2[threadIdx.x] += s2[threadIdx.x + off];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = s1[0];
    part[2 * blockIdx.x + 1] = s2[0];
  }
}

// dst[idx[t]] = src[t] for rows of 3 doubles (the direct sum at sampled
// dipoles placed into a field array)
__global__ void k_scatter_rows(int64_t nt, const int64_t* __restrict__ idx, const double* __restrict__ src,
                               double* __restrict__ dst) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nt) return;
  const int64_t i = idx[t];
  dst[3 * i] = src[3 * t];
  dst[3 * i + 1] = src[3 * t + 1];
  dst[3 * i + 2] = src[3 * t + 2];
}

// ---------------------------------------------------------------- launchers
void run_scatter_rows(int64_t nt, const int64_t* d_idx, const double* d_src, double* d_dst, hipStream_t st) {
  if (nt <= 0) return;
  k_scatter_rows<<<ceil_div(nt, 256), 256, 0, st>>>(nt, d_idx, d_src, d_dst);
  CCFMM_HIP(hipGetLastError());
}

void run_leaf_ids(Plan& P, int32_t* d_out, hipStream_t st) {
  k_leaf_ids<<<ceil_div(P.n, 256), 256, 0, st>>>(P.n, P.dleaf.as<int32_t>(), P.perm.as<int32_t>(), d_out);
  CCFMM_HIP(hipGetLastError());
}

void run_leaf_errors(Plan& P, int nb, const double* d_H, const double* d_Href, double* d_num, double* d_den,
                     hipStream_t st) {
  const int nl = P.lev[P.L]->ncells;
  k_leaf_err<<<ceil_div(nl, 128), 128, 0, st>>>(nl, P.n, nb, P.lstart.as<int32_t>(), P.lcount.as<int32_t>(),
                                                 P.perm.as<int32_t>(), d_H, d_Href, d_num, d_den);
  CCFMM_HIP(hipGetLastError());
}

void run_leaf_features(Plan& P, int nb, const double* d_m, float* d_feat, hipStream_t st) {
  LevelData& D = *P.lev[P.L];
  const int nl = D.ncells;
  k_leaf_features<<<ceil_div(nl, 128), 128, 0, st>>>(nl, P.n, nb, P.L, P.lstart.as<int32_t>(),
                                                     P.lcount.as<int32_t>(), D.near_ptr.as<int32_t>(),
                                                     D.near_idx.as<int32_t>(), D.far_ptr.as<int32_t>(),
                                                     P.perm.as<int32_t>(), d_m, d_feat);
  CCFMM_HIP(hipGetLastError());
}

void run_mlp_forward(const float* d_params, int64_t rows, const float* d_x, float* d_y, hipStream_t st) {
  if (rows <= 0) return;
  k_mlp_forward<<<ceil_div(rows, 64), 64, 0, st>>>(d_params, rows, d_x, d_y);
  CCFMM_HIP(hipGetLastError());
}

size_t mlp_grad_bytes(int64_t rows) {
  return (sizeof(GradShare) + sizeof(float) * kParams) * (size_t)std::max(1, ceil_div(rows, kGR));
}

void run_mlp_loss_grad(const float* d_params, int64_t rows, const float* d_x, const float* d_t, const float* d_mask,
                       float* d_grad, float* d_loss, DevBuf& tmp, hipStream_t st) {
  const int nblk = std::max(1, ceil_div(rows, kGR));
  char* buf = reinterpret_cast<char*>(tmp.ensure(mlp_grad_bytes(rows)));
  GradShare* share = reinterpret_cast<GradShare*>(buf);
  float* part = reinterpret_cast<float*>(share + nblk);
  k_mlp_grad_part<<<nblk, 256, 0, st>>>(d_params, rows, d_x, d_t, d_mask, part, share);
  CCFMM_HIP(hipGetLastError());
  k_mlp_grad_sum<<<ceil_div(kParams, 64), 1024, 0, st>>>(nblk, part, share, d_grad, d_loss);
  CCFMM_HIP(hipGetLastError());
}

void run_mlp_adam(float* d_params, const float* d_grad, float* d_m1, float* d_m2, int step, float lr,
                  hipStream_t st) {
  k_adam<<<ceil_div(kParams, 256), 256, 0, st>>>(d_params, d_grad, d_m1, d_m2, step, lr, 0.9f, 0.999f, 1e-8f);
  CCFMM_HIP(hipGetLastError());
}

// features -> network -> per-cell choice for a global error budget; returns
// the choice histogram and the predicted relative RMS error of the choice.
// d_F: per-cell squared field of the fixed-parameter evaluation (device [nl]).
// The choice minimises the total cost subject to
//   sum_c F_c 10^(2 y_c) <= 10^(2 log_bound) sum_c F_c,
// the predicted global relative RMS error within the bound: per cell the
// least cost + lam F_c 10^(2 y_c), the multiplier lam found by bisection in
// log10 lam (a fixed sequence of steps, so the choice is reproducible).  If
// the cheapest candidates already meet the budget they are taken; if even the
// most accurate ones miss it, those are taken and the judge decides.
void run_select(Plan& P, const float* d_params, double log_bound, double cost_far, int nb, const double* d_m,
                const double* d_F, int32_t* d_p, double* d_theta, std::vector<int32_t>& hist, double* pred_err,
                hipStream_t st) {
  LevelData& D = *P.lev[P.L];
  LevelData& U = *P.lev[P.L > 0 ? P.L - 1 : 0];
  const int nl = D.ncells;
  if (P.L == 0) fail(CCFMM_EINVAL, "the tree has a single cell: nothing to select");
  const size_t fbytes = (sizeof(float) * (size_t)nl * (kIn + kOut) + 255) & ~(size_t)255;
  const size_t cbytes = sizeof(double) * (size_t)nl * kOut;
  char* buf = reinterpret_cast<char*>(P.scratch2.ensure(fbytes + cbytes + sizeof(double) * kLagBlocks));
  float* feat = reinterpret_cast<float*>(buf);
  float* pred = feat + (size_t)nl * kIn;
  double* cost = reinterpret_cast<double*>(buf + fbytes);
  double* part = cost + (size_t)nl * kOut;
  P.flags.ensure(256);  // flags, then the 25 choice counters
  int32_t* dh = reinterpret_cast<int32_t*>(P.flags.as<char>() + 64);
  CCFMM_HIP(hipMemsetAsync(dh, 0, sizeof(int32_t) * kOut, st));
  run_leaf_features(P, nb, d_m, feat, st);
  run_mlp_forward(d_params, nl, feat, pred, st);
  SelectArgs a;
  a.parent = D.parent.as<int32_t>();
  a.coord = D.coord.as<int32_t>();
  a.pnear_ptr = U.near_ptr.as<int32_t>();
  a.pnear_idx = U.near_idx.as<int32_t>();
  a.pchild = U.child.as<int32_t>();
  a.lcount = P.lcount.as<int32_t>();
  a.nl = nl;
  a.L = P.L;
  a.log_bound = log_bound;
  a.cost_far = cost_far;
  a.pmax = std::min(P.p, 6);
  for (int q = 2; q <= 6; q++) a.far_share[q - 2] = m2l_row_share(P, q);
  k_cand_costs<<<ceil_div(nl, 128), 128, 0, st>>>(a, P.geo, cost);
  CCFMM_HIP(hipGetLastError());
  std::vector<double> hF(nl);
  CCFMM_HIP(hipMemcpyAsync(hF.data(), d_F, sizeof(double) * nl, hipMemcpyDeviceToHost, st));
  CCFMM_HIP(hipStreamSynchronize(st));
  double Ftot = 0.0;
  for (double f : hF) Ftot += f;
  const double budget = std::pow(10.0, 2.0 * log_bound) * Ftot;
  std::vector<double> hp(kLagBlocks);
  auto predicted = [&](double lam) {
    k_lagrange_sum<<<kLagBlocks, 256, 0, st>>>(nl, lam, cost, pred, d_F, part);
    CCFMM_HIP(hipGetLastError());
    CCFMM_HIP(hipMemcpyAsync(hp.data(), part, sizeof(double) * kLagBlocks, hipMemcpyDeviceToHost, st));
    CCFMM_HIP(hipStreamSynchronize(st));
    double e = 0.0;
    for (double v : hp) e += v;
    return e;
  };
  double lam;
  if (predicted(-1.0) > budget) {
    lam = -1.0;
  } else if (predicted(0.0) <= budget) {
    lam = 0.0;
  } else {
    double lo = -300.0, hi = 300.0;  // log10 lam: infeasible at lo, feasible at hi
    for (int it = 0; it < 64; it++) {
      const double mid = 0.5 * (lo + hi);
      if (predicted(std::pow(10.0, mid)) <= budget)
        hi = mid;
      else
        lo = mid;
    }
    lam = std::pow(10.0, hi);
  }
  const double e_final = predicted(lam);
  if (pred_err) *pred_err = Ftot > 0.0 ? std::sqrt(e_final / Ftot) : 0.0;
  k_lagrange_choose<<<ceil_div(nl, 128), 128, 0, st>>>(nl, lam, cost, pred, d_F, d_p, d_theta, dh);
  CCFMM_HIP(hipGetLastError());
  hist.assign(kOut, 0);
  CCFMM_HIP(hipMemcpyAsync(hist.data(), dh, sizeof(int32_t) * kOut, hipMemcpyDeviceToHost, st));
  CCFMM_HIP(hipStreamSynchronize(st));
}

double run_rel_rms(const double* d_A, const double* d_B, int64_t count, DevBuf& tmp, hipStream_t st) {
  const int nblk = (int)std::min<int64_t>(512, std::max<int64_t>(1, count / 256));
  double* part = reinterpret_cast<double*>(tmp.ensure(sizeof(double) * 2 * nblk));
  k_diff_sums<<<nblk, 256, 0, st>>>(count, d_A, d_B, part);
  CCFMM_HIP(hipGetLastError());
  std::vector<double> h(2 * nblk);
  CCFMM_HIP(hipMemcpyAsync(h.data(), part, sizeof(double) * 2 * nblk, hipMemcpyDeviceToHost, st));
  CCFMM_HIP(hipStreamSynchronize(st));
  double a = 0.0, b = 0.0;
  for (int i = 0; i < nblk; i++) {
    a += h[2 * i];
    b += h[2 * i + 1];
  }
  return b > 0.0 ? std::sqrt(a / b) : 0.0;
}

}  // namespace ccfmm
