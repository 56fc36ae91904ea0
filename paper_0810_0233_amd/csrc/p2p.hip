// p2p.hip -- the field at the dipoles: smooth part from the local expansion
// (Eq. H, with H = -grad V) plus the direct sum over the near smallest cells
// (Eq. H2, read as the field of source dipole j: (3 (m_j.u) u - m_j)/r^3, pairs
// at zero separation skipped), accumulated in FP64 and written in the
// caller's dipole order.
//
// One wavefront per chunk of <= 64 dipoles of one smallest cell.  The c
// dipoles of a chunk are split as c = a + b (a the largest power of two <= c):
// the first a get G1 = 64/a lanes each, the other b get G2 = floor(64/b)
// lanes each, so nearly every lane works in both roles whatever c is.  The
// lanes of a dipole split the sources, and their partial fields are combined
// at the end (butterflies in the first role, a segmented tree in the second).  Sources are staged 64 at a time in LDS,
// packed from consecutive near cells (each shifted by the integer offset of its
// cell so all coordinates stay cell-relative) and padded with null sources
// (zero moment, far away) that add exactly zero, so every lane runs the same
// trip count; the next batch is loaded while the current one is summed.
#include <mutex>
#include <type_traits>

#include "near.hpp"

namespace ccfmm {

// One staged source: position (cell-relative, shifted to the target cell) and
// moment, padded to 8 elements so a lane reads it with two 16-byte loads.
template <typename T>
struct alignas(8 * sizeof(T)) P2PSrc {
  T x, y, z, mx, my, mz, p0, p1;
};
// FP32 residuals of a staged position (exact position = x + lx, ...)
template <typename T>
struct alignas(4 * sizeof(T)) P2PLo {
  T x, y, z, p;
};
// A target dipole: position and its residual (zero in FP64)
template <typename T>
struct P2PTgt {
  T x, y, z, lx, ly, lz;
};

// Small systems (kSplit): with fewer chunks than a few wavefronts per SIMD the
// near field's time is that of one wavefront walking its near list, so the
// wavefronts of a block share chunks: `split` of them take a contiguous part of
// the list each, and their sums are added in part order through LDS.
struct SplitItem {
  int64_t item;
  int part;
};
template <bool kSplit>
__device__ __forceinline__ SplitItem split_item(int64_t blk, int w, int split) {
  if (!kSplit) return {blk * kP2PWaves + w, 0};
  return {blk * (kP2PWaves / split) + w / split, w % split};
}
// this part's share of the list [e0, e1)
__device__ __forceinline__ void split_range(int part, int split, int& e0, int& e1) {
  const int n = e1 - e0, b = e0;
  e0 = b + (int)((int64_t)n * part / split);
  e1 = b + (int)((int64_t)n * (part + 1) / split);
}
// v of part 0 += v of the parts 1 .. split - 1 (every wavefront of the block
// calls this; buf holds 3 x 64 doubles per wavefront, row_bytes apart)
__device__ __forceinline__ void split_sum(double (&v)[3], char* buf, int row_bytes, int w, int lane, int part,
                                          int split) {
  double* mine = reinterpret_cast<double*>(buf + (size_t)w * row_bytes);
  __syncthreads();
  if (part > 0) {
#pragma unroll
    for (int c = 0; c < 3; c++) mine[64 * c + lane] = v[c];
  }
  __syncthreads();
  if (part == 0) {
    for (int q = 1; q < split; q++) {
      const double* o = reinterpret_cast<const double*>(buf + (size_t)(w + q) * row_bytes);
#pragma unroll
      for (int c = 0; c < 3; c++) v[c] += o[64 * c + lane];
    }
  }
}

// One source on one target: f += (3 (m.r) r / r^2 - m) / r^3, written as
// inv3 * (k r - m) with k = 3 (m.r) / r^2.  Only the target's own cell can
// hold a source at zero separation (a position determines its cell), so only
// that cell pays for the test.  With kAcc the separation is formed as
// (hi_t - hi_s) + (lo_t - lo_s): the first difference is exact for close
// points, so r keeps its digits however close the pair (own and adjacent
// cells only; elsewhere r is at least a cell side).
template <typename T, bool kSelf, bool kAcc>
__device__ __forceinline__ void p2p_pair(const P2PSrc<T>& s, const P2PLo<T>* l, const P2PTgt<T>& t, T& fx, T& fy,
                                         T& fz) {
  T rx = t.x - s.x, ry = t.y - s.y, rz = t.z - s.z;
  if (kAcc) {
    const P2PLo<T> q = *l;
    rx += t.lx - q.x;
    ry += t.ly - q.y;
    rz += t.lz - q.z;
  }
  const T r2 = rx * rx + ry * ry + rz * rz;
  T inv = rsqrt_t<T>(r2);
  if (kSelf) inv = (r2 > (T)0) ? inv : (T)0;
  const T inv2 = inv * inv;
  const T inv3 = inv2 * inv;
  const T mr = s.mx * rx + s.my * ry + s.mz * rz;
  const T k = ((T)3 * inv2) * mr;
  fx += inv3 * (k * rx - s.mx);
  fy += inv3 * (k * ry - s.my);
  fz += inv3 * (k * rz - s.mz);
}

// K sources q = sub, sub + G, ... of the staged batch for one target.
template <typename T, int G, bool kSelf, bool kAcc>
__device__ __forceinline__ void p2p_run(const P2PSrc<T>* __restrict__ src, const P2PLo<T>* __restrict__ lo, int sub,
                                        int K, const P2PTgt<T>& t, T& fx, T& fy, T& fz) {
  const P2PSrc<T>* q = src + sub;
  const P2PLo<T>* ql = lo + sub;
  int k = 0;
  for (; k + 4 <= K; k += 4, q += 4 * G, ql += 4 * G) {
#pragma unroll
    for (int u = 0; u < 4; u++) p2p_pair<T, kSelf, kAcc>(q[u * G], ql + u * G, t, fx, fy, fz);
  }
  for (; k < K; k++, q += G, ql += G) p2p_pair<T, kSelf, kAcc>(q[0], ql, t, fx, fy, fz);
}

// G lanes per target: a power of two (first role) or floor(64 / b) for the b
// targets of the second role.  A lane reads slots sub + k G < K G, which can
// pass the 64 staged sources by up to 20 (G = 21): those slots hold null
// sources.
constexpr int kP2PPad = 24;

template <typename T, bool kSelf, bool kAcc>
__device__ __forceinline__ void p2p_role(const P2PSrc<T>* __restrict__ src, const P2PLo<T>* __restrict__ lo, int G,
                                         int sub, int nsrc, const P2PTgt<T>& t, T& fx, T& fy, T& fz) {
  const int K = (nsrc + G - 1) / G;
  switch (G) {
    case 1: p2p_run<T, 1, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 2: p2p_run<T, 2, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 3: p2p_run<T, 3, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 4: p2p_run<T, 4, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 5: p2p_run<T, 5, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 6: p2p_run<T, 6, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 7: p2p_run<T, 7, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 8: p2p_run<T, 8, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 9: p2p_run<T, 9, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 10: p2p_run<T, 10, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 12: p2p_run<T, 12, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 16: p2p_run<T, 16, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 21: p2p_run<T, 21, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    case 32: p2p_run<T, 32, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
    default: p2p_run<T, 64, kSelf, kAcc>(src, lo, sub, K, t, fx, fy, fz); break;
  }
}

// ------------------------------------------------------------ smooth field
// Gradient of the local expansion of a dipole's cell, degree by degree up to the
// cell's order, from the monomials y^k / k! (factors px, py, pz).
template <typename T, int P>
struct SmoothMono {
  T px[P], py[P], pz[P];
  __device__ __forceinline__ SmoothMono(T yx, T yy, T yz) {
    px[0] = py[0] = pz[0] = (T)1;
#pragma unroll
    for (int j = 1; j < P; j++) {
      const T inv = (T)(1.0 / j);
      px[j] = px[j - 1] * yx * inv;
      py[j] = py[j - 1] * yy * inv;
      pz[j] = pz[j - 1] * yz * inv;
    }
  }
  __device__ __forceinline__ void gradient(const T* __restrict__ v, int pl, T (&e)[3]) const {
    e[0] = e[1] = e[2] = (T)0;
#pragma unroll
    for (int d = 0; d < P; d++) {
      if (d >= pl) break;
#pragma unroll
      for (int k = ncoef(d - 1); k < ncoef(d); k++) {
        const int kx = kMI.x[k], ky = kMI.y[k], kz = kMI.z[k];
        const T mono = px[kx] * py[ky] * pz[kz];
        e[0] += v[midx(kx + 1, ky, kz) - 1] * mono;
        e[1] += v[midx(kx, ky + 1, kz) - 1] * mono;
        e[2] += v[midx(kx, ky, kz + 1) - 1] * mono;
      }
    }
  }
};

// Smooth field of one dipole from its cell's local expansion,
// H_a = -sum_{|k| <= pl-1} Vt_{k+e_a} yt^k / k!, plus the near field.
template <typename T, int P>
__device__ __forceinline__ void l2p_write(const T* __restrict__ v, int pl, T yx, T yy, T yz, double hx, double hy,
                                          double hz, double s3, double* __restrict__ Ho) {
  const SmoothMono<T, P> mono(yx, yy, yz);
  T e[3];
  mono.gradient(v, pl, e);
  Ho[0] = s3 * (hx - (double)e[0]);
  Ho[1] = s3 * (hy - (double)e[1]);
  Ho[2] = s3 * (hz - (double)e[2]);
}

// ------------------------------------------------------------ one configuration
// The near field of one configuration alone (written, not added): the smooth
// field is added by k_l2p_one.  kSplit: the wavefronts of a block share
// chunks (near_split).
// FP32 asks for 6 waves per SIMD, which spills a few registers (44 bytes a
// lane, held in the caches); at 5 waves nothing spills but the 2^20-dipole
// ferrofluid's near field took 3.15 ms instead of 3.03.
template <typename T, bool kSplit>
__global__ void __launch_bounds__(64 * kP2PWaves, sizeof(T) == 4 ? 6 : 2) k_p2p_one(P2PArgs a, const T* __restrict__ y,
                                                                                 const T* __restrict__ msort,
                                                                                 double* __restrict__ H) {
  constexpr bool kLo = std::is_same<T, float>::value;  // FP32 keeps residuals for close pairs
  __shared__ P2PSrc<T> sS[kP2PWaves][64 + kP2PPad];
  __shared__ P2PLo<T> sL[kP2PWaves][kLo ? 64 + kP2PPad : 1];
  // the wave index is uniform: say so, so chunk data, counts and loop bounds
  // live in scalar registers and branch on scalar conditions
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t blk = xcd_run_block(gridDim.x, blockIdx.x);
  const SplitItem si = split_item<kSplit>(blk, w, a.split);
  const int b = blockIdx.y;
  const bool live = si.item < *a.nchunks;
  if (!kSplit && !live) return;  // (kSplit: every wavefront reaches the barriers of the sums)
  const P2PChunk ch = a.chunks[live ? si.item : 0];
  const int n = (int)a.n;
  const int c = ch.count;
  int A = 1;
  while (2 * A <= c) A <<= 1;
  const int B = c - A;
  const int G1 = 64 / A, G2 = B > 0 ? 64 / B : 64;  // G2 in {1..10, 12, 16, 21, 32, 64}
  const int t1 = lane / G1, sub1 = lane % G1;
  const int t2 = A + lane / G2, sub2 = lane % G2;
  const bool act2 = B > 0 && t2 < c;
  const int64_t i1 = ch.first + t1, i2 = ch.first + (act2 ? t2 : 0);
  const T x1 = y[i1], y1 = y[n + i1], z1 = y[2 * n + i1];
  const T x2 = y[i2], y2 = y[n + i2], z2 = y[2 * n + i2];
  P2PTgt<T> tg1{x1, y1, z1, (T)0, (T)0, (T)0}, tg2{x2, y2, z2, (T)0, (T)0, (T)0};
  if constexpr (kLo) {
    tg1.lx = (T)a.ylo[i1];
    tg1.ly = (T)a.ylo[n + i1];
    tg1.lz = (T)a.ylo[2 * n + i1];
    tg2.lx = (T)a.ylo[i2];
    tg2.ly = (T)a.ylo[n + i2];
    tg2.lz = (T)a.ylo[2 * n + i2];
  }
  const T* mb = msort + (int64_t)b * 3 * n;
  const int cx = a.coord[3 * ch.leaf], cy = a.coord[3 * ch.leaf + 1], cz = a.coord[3 * ch.leaf + 2];
  P2PSrc<T>* src = sS[w];
  P2PLo<T>* srclo = sL[w];
  if (lane < kP2PPad) {  // null sources past the batch (read by strides that do not divide 64)
    P2PSrc<T> z;
    z.x = z.y = z.z = (T)1e4;
    z.mx = z.my = z.mz = z.p0 = z.p1 = (T)0;
    src[64 + lane] = z;
    if constexpr (kLo) {
      P2PLo<T> zl;
      zl.x = zl.y = zl.z = zl.p = (T)0;
      srclo[64 + lane] = zl;
    }
  }
  int e0 = a.near_ptr[ch.leaf], e1 = a.near_ptr[ch.leaf + 1];
  if (kSplit) {
    split_range(si.part, a.split, e0, e1);
    if (!live) e1 = e0;
  }
  // Near-list metadata, 64 entries at a time, one entry per lane: first sorted
  // dipole, count, and the cell offset in cell-relative units.  The batch
  // builder below reads it back with readlane (no dependent loads per cell).
  int wb = e0;
  int mstart = 0, mcnt = 0, mself = 0, madj = 0;
  T mox = (T)0, moy = (T)0, moz = (T)0;
  auto load_meta = [&](int base) {
    const int e = base + lane;
    mcnt = 0;
    mself = 0;
    madj = 0;
    if (e < e1) {
      const int S = a.near_idx[e];
      mstart = a.lstart[S];
      mcnt = a.lcount[S];
      mself = S == ch.leaf;
      madj = abs(a.coord[3 * S] - cx) <= 1 && abs(a.coord[3 * S + 1] - cy) <= 1 && abs(a.coord[3 * S + 2] - cz) <= 1;
      mox = (T)((a.coord[3 * S] - cx) * a.g[0]);
      moy = (T)((a.coord[3 * S + 1] - cy) * a.g[1]);
      moz = (T)((a.coord[3 * S + 2] - cz) * a.g[2]);
    }
  };
  load_meta(wb);
  // Batches of up to 64 sources drawn from consecutive near cells (a cell
  // may be split between batches); (e, off) is the cursor.
  int e = e0, off = 0;
  struct Batch {
    int filled;
    bool self;
    bool adj;    // holds the target cell or a neighbour of it (close pairs possible)
    bool valid;  // this lane's slot holds a source
    int64_t j;   // its sorted index
    T ox, oy, oz;
  };
  auto next_batch = [&]() -> Batch {
    Batch bt;
    bt.filled = 0;
    bt.self = false;
    bt.adj = false;
    bt.valid = false;
    bt.j = 0;
    bt.ox = bt.oy = bt.oz = (T)0;
    while (bt.filled < 64 && e < e1) {
      if (e - wb >= 64) {
        wb = e;
        load_meta(wb);
      }
      const int k = e - wb;
      const int cnt = __builtin_amdgcn_readlane(mcnt, k);
      const int st = __builtin_amdgcn_readlane(mstart, k);
      const int take = min(64 - bt.filled, cnt - off);
      if (lane >= bt.filled && lane < bt.filled + take) {
        bt.valid = true;
        bt.j = st + off + (lane - bt.filled);
        bt.ox = __builtin_bit_cast(T, readlane_t(mox, k));
        bt.oy = __builtin_bit_cast(T, readlane_t(moy, k));
        bt.oz = __builtin_bit_cast(T, readlane_t(moz, k));
      }
      bt.self = bt.self || __builtin_amdgcn_readlane(mself, k);
      bt.adj = bt.adj || __builtin_amdgcn_readlane(madj, k);
      bt.filled += take;
      off += take;
      if (off == cnt) {
        e++;
        off = 0;
      }
    }
    return bt;
  };
  // A source shifted into the target cell's frame: hi + o is rounded; with
  // |o| >= |hi| (o a nonzero multiple of the cell side, |hi| at most half of
  // it) the rounding error is exactly hi - ((hi + o) - o), which joins the
  // stored residual.  Returned by value (no address-taken temporaries).
  auto load_src = [&](const Batch& bt) -> P2PSrc<T> {
    P2PSrc<T> q;
    if (bt.valid) {
      const int64_t j = bt.j;
      q.x = y[j] + bt.ox;
      q.y = y[n + j] + bt.oy;
      q.z = y[2 * n + j] + bt.oz;
      q.mx = mb[j];
      q.my = mb[n + j];
      q.mz = mb[2 * n + j];
    } else {  // null source: zero moment, far from every target
      q.x = q.y = q.z = (T)1e4;
      q.mx = q.my = q.mz = (T)0;
    }
    q.p0 = q.p1 = (T)0;
    return q;
  };
  auto load_lo = [&](const Batch& bt, const P2PSrc<T>& q) -> P2PLo<T> {
    P2PLo<T> l;
    l.x = l.y = l.z = l.p = (T)0;
    if (kLo && bt.adj && bt.valid) {
      const int64_t j = bt.j;
      l.x = (y[j] - (q.x - bt.ox)) + (T)a.ylo[j];
      l.y = (y[n + j] - (q.y - bt.oy)) + (T)a.ylo[n + j];
      l.z = (y[2 * n + j] - (q.z - bt.oz)) + (T)a.ylo[2 * n + j];
    }
    return l;
  };
  double hx1 = 0.0, hy1 = 0.0, hz1 = 0.0, hx2 = 0.0, hy2 = 0.0, hz2 = 0.0;  // near field, cell-relative units
  Batch cur = next_batch();
  P2PSrc<T> qc = load_src(cur);
  P2PLo<T> lc = load_lo(cur, qc);
  while (cur.filled > 0) {
    src[lane] = qc;
    if (kLo && cur.adj) srclo[lane] = lc;
    wave_lds_sync();
    // the next batch's loads fly while this one is summed
    const Batch nxt = next_batch();
    const P2PSrc<T> qn = load_src(nxt);
    const P2PLo<T> ln = load_lo(nxt, qn);
    const int nsrc = cur.filled;
    T fx1 = (T)0, fy1 = (T)0, fz1 = (T)0, fx2 = (T)0, fy2 = (T)0, fz2 = (T)0;
    if (cur.self) {
      p2p_role<T, true, kLo>(src, srclo, G1, sub1, nsrc, tg1, fx1, fy1, fz1);
      if (B > 0) p2p_role<T, true, kLo>(src, srclo, G2, sub2, nsrc, tg2, fx2, fy2, fz2);
    } else if (kLo && cur.adj) {
      p2p_role<T, false, kLo>(src, srclo, G1, sub1, nsrc, tg1, fx1, fy1, fz1);
      if (B > 0) p2p_role<T, false, kLo>(src, srclo, G2, sub2, nsrc, tg2, fx2, fy2, fz2);
    } else {
      p2p_role<T, false, false>(src, srclo, G1, sub1, nsrc, tg1, fx1, fy1, fz1);
      if (B > 0) p2p_role<T, false, false>(src, srclo, G2, sub2, nsrc, tg2, fx2, fy2, fz2);
    }
    wave_lds_sync();
    hx1 += (double)fx1;
    hy1 += (double)fy1;
    hz1 += (double)fz1;
    hx2 += (double)fx2;
    hy2 += (double)fy2;
    hz2 += (double)fz2;
    cur = nxt;
    qc = qn;
    lc = ln;
  }
  // combine the lanes of each dipole (they are contiguous: lane = t G + sub)
  for (int off = 1; off < G1; off <<= 1) {
    hx1 += __shfl_xor(hx1, off);
    hy1 += __shfl_xor(hy1, off);
    hz1 += __shfl_xor(hz1, off);
  }
  // second role: G2 need not be a power of two; a segmented tree leaves each
  // dipole's sum in its first lane (sub2 = 0, the one that writes)
  for (int off = 1; off < G2; off <<= 1) {
    const double ox = __shfl_down(hx2, off), oy = __shfl_down(hy2, off), oz = __shfl_down(hz2, off);
    if (sub2 + off < G2) {
      hx2 += ox;
      hy2 += oy;
      hz2 += oz;
    }
  }
  if constexpr (kSplit) {
    double v1[3] = {hx1, hy1, hz1}, v2[3] = {hx2, hy2, hz2};
    static_assert(sizeof(sS[0]) >= 3 * 64 * sizeof(double), "the sums need the staging rows' room");
    split_sum(v1, reinterpret_cast<char*>(&sS[0][0]), (int)sizeof(sS[0]), w, lane, si.part, a.split);
    split_sum(v2, reinterpret_cast<char*>(&sS[0][0]), (int)sizeof(sS[0]), w, lane, si.part, a.split);
    if (si.part > 0 || !live) return;
    hx1 = v1[0], hy1 = v1[1], hz1 = v1[2];
    hx2 = v2[0], hy2 = v2[1], hz2 = v2[2];
  }
  const double s3 = a.inv_s3;
  if (sub1 == 0) {
    double* o = H + ((int64_t)b * n + a.perm[i1]) * 3;
    o[0] = s3 * hx1;
    o[1] = s3 * hy1;
    o[2] = s3 * hz1;
  }
  if (act2 && sub2 == 0) {
    double* o = H + ((int64_t)b * n + a.perm[i2]) * 3;
    o[0] = s3 * hx2;
    o[1] = s3 * hy2;
    o[2] = s3 * hz2;
  }
}

// ------------------------------------------------------------ a few configurations
// Near field of several configurations on the vector units: FP64 plans, and in
// mixed ones two configurations of large plans, plans without room for the FP16
// form and configurations that it leaves (P2PArgs::range).  The geometry of a pair -- separation, reciprocal distance, r^-2 and r^-3 -- is the same for
// every configuration, so it is formed once and applied to KB configurations
// held by the same lane: about 13 + 10 KB operations per pair instead of
// 23 KB (in FP64 about 24 + 9 KB; vector and matrix-core FP64 run at the same
// rate here and do not overlap, so FP64 uses this form for every batch size).  One wavefront per chunk of <= 64 target dipoles of one smallest
// cell; the c targets get G = floor(64/c) lanes each (the lanes of a target
// split the sources; a chunk of a full 32-dipole cell uses every lane; FP64
// plans cut a cell where that leaves fewer lanes idle, see k_chunk_fill_b), and
// blockIdx.y runs over groups of KB configurations.  Sources are staged 64 at
// a time in LDS with their moments for the group (zero for configurations
// past the batch), packed from consecutive near cells and padded with null
// sources as in k_p2p_one; the next batch is loaded while the current one is
// summed.  FP32 partial fields of a batch are added into FP64 accumulators.

// words of one staged source: position (x, y, z, unused), then m[KB][3],
// rounded up to whole 16-byte LDS reads
template <typename T, int KB>
constexpr int p2pk_words() {
  return ((4 + 3 * KB) * (int)sizeof(T) + 15) / 16 * 16 / (int)sizeof(T);
}

// a staged source in registers: whole 16-byte LDS reads (4 floats or 2
// doubles each); element i of the record is v[i / W][i % W]
template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
  typedef float type __attribute__((ext_vector_type(4)));
  static constexpr int W = 4;
};
template <>
struct Vec16<double> {
  typedef double type __attribute__((ext_vector_type(2)));
  static constexpr int W = 2;
};
template <typename T, int KB>
struct SrcRegs {
  static constexpr int W = Vec16<T>::W;
  static constexpr int NV = p2pk_words<T, KB>() / W;
  typename Vec16<T>::type v[NV];
  __device__ __forceinline__ T at(int i) const { return v[i / W][i % W]; }
};
template <typename T, int KB>
__device__ __forceinline__ SrcRegs<T, KB> load_regs(const typename Vec16<T>::type* __restrict__ p) {
  SrcRegs<T, KB> r;
#pragma unroll
  for (int i = 0; i < SrcRegs<T, KB>::NV; i++) r.v[i] = p[i];
  return r;
}

// one source on one target for KB configurations; kSelf: the pair may be at
// zero separation (target's own cell); kAcc: separations formed from the
// FP32 residuals too (own and adjacent cells, where pairs can be close)
template <typename T, int KB, bool kSelf, bool kAcc>
__device__ __forceinline__ void p2pk_pair(const SrcRegs<T, KB>& q, const P2PLo<T>& lo, const P2PTgt<T>& t,
                                          T (&f)[KB][3]) {
  T rx = t.x - q.at(0), ry = t.y - q.at(1), rz = t.z - q.at(2);
  if (kAcc) {
    rx += t.lx - lo.x;
    ry += t.ly - lo.y;
    rz += t.lz - lo.z;
  }
  const T r2 = rx * rx + ry * ry + rz * rz;
  T inv = rsqrt_t<T>(r2);
  if (kSelf) inv = (r2 > (T)0) ? inv : (T)0;
  const T inv2 = inv * inv;
  const T inv3 = inv2 * inv;
  if constexpr (std::is_same<T, double>::value) {
    // 9 operations a configuration instead of 10, after 6 more per pair:
    // k = m.u with u = 3 r / r^2, then k v - m / r^3 with v = r / r^3
    const T c3 = (T)3 * inv2;
    const T ux = c3 * rx, uy = c3 * ry, uz = c3 * rz;
    const T vx = inv3 * rx, vy = inv3 * ry, vz = inv3 * rz;
#pragma unroll
    for (int b = 0; b < KB; b++) {
      const T mx = q.at(4 + 3 * b), my = q.at(5 + 3 * b), mz = q.at(6 + 3 * b);
      const T k = mx * ux + my * uy + mz * uz;
      f[b][0] = fma(k, vx, fma(-inv3, mx, f[b][0]));
      f[b][1] = fma(k, vy, fma(-inv3, my, f[b][1]));
      f[b][2] = fma(k, vz, fma(-inv3, mz, f[b][2]));
    }
    return;
  }
  const T c3 = (T)3 * inv2;
#pragma unroll
  for (int b = 0; b < KB; b++) {
    const T mx = q.at(4 + 3 * b), my = q.at(5 + 3 * b), mz = q.at(6 + 3 * b);
    const T k = c3 * (mx * rx + my * ry + mz * rz);
    f[b][0] += inv3 * (k * rx - mx);
    f[b][1] += inv3 * (k * ry - my);
    f[b][2] += inv3 * (k * rz - mz);
  }
}

// the slots sub, sub + G, ... (K >= 1 of them) of the staged batch; the
// next slot's record is read while the current one is summed (the last
// iteration re-reads its own slot rather than pass the batch)
template <typename T, int KB, bool kSelf, bool kAcc>
__device__ __forceinline__ void p2pk_run(const T* __restrict__ src, const P2PLo<T>* __restrict__ lo, int G,
                                         int sub, int K, const P2PTgt<T>& t, T (&f)[KB][3]) {
  using V = typename Vec16<T>::type;
  constexpr int NV = SrcRegs<T, KB>::NV;
  const V* q = reinterpret_cast<const V*>(src) + sub * NV;
  const P2PLo<T>* ql = lo + sub;
  const int step = G * NV;
  SrcRegs<T, KB> cur = load_regs<T, KB>(q);
  P2PLo<T> lcur{(T)0, (T)0, (T)0, (T)0};
  if (kAcc) lcur = ql[0];
  for (int k = 0; k < K; k++) {
    const int kn = min(k + 1, K - 1);
    const SrcRegs<T, KB> nxt = load_regs<T, KB>(q + kn * step);
    P2PLo<T> lnxt{(T)0, (T)0, (T)0, (T)0};
    if (kAcc) lnxt = ql[kn * G];
    p2pk_pair<T, KB, kSelf, kAcc>(cur, lcur, t, f);
    cur = nxt;
    lcur = lnxt;
  }
}

// PL > 0: also add the smooth field of the cell's local expansion (order PL),
// the single-stream form; PL = 0: the near field alone (written, not added),
// the form that runs beside the expansion passes
// Waves per SIMD asked of the compiler: 3, except in FP64 from four
// configurations a lane (accumulators, a source record and the next one fill
// the registers of two waves, and their LDS records leave room for two blocks
// per CU) and with the smooth field at the highest order, whose registers
// would spill at 3.
template <typename T, int KB, int PL>
constexpr int multi_waves() {
  if (sizeof(T) == 8 && KB >= 4) return 2;
  if (KB >= 8 && PL >= 8) return 2;
  return 3;
}

// FP64 partial sums go straight into the accumulators; FP32 ones are added
// into FP64 after each batch of 64 sources.
template <typename T, int KB, int PL, bool kSplit = false>
__global__ void __launch_bounds__(64 * kP2PWaves, (multi_waves<T, KB, PL>())) k_p2p_multi(P2PArgs a, const T* __restrict__ y,
                                                                 const T* __restrict__ msort, const T* __restrict__ V,
                                                                 double* __restrict__ H) {
  constexpr int NW = p2pk_words<T, KB>();
  constexpr int kSlots = 64 + kP2PPad;
  __shared__ __attribute__((aligned(16))) T sS[kP2PWaves][kSlots * NW];
  constexpr bool kLo = std::is_same<T, float>::value;  // FP32 keeps residuals for close pairs
  __shared__ P2PLo<T> sL[kP2PWaves][kLo ? kSlots : 1];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t blk = xcd_run_block(gridDim.x, blockIdx.x);
  static_assert(!(kSplit && PL > 0), "the shared form leaves the smooth field to its own pass");
  const SplitItem si = split_item<kSplit>(blk, w, a.split);
  const bool live = si.item < *a.nchunks;
  if (!kSplit && !live) return;
  const int cfg0 = a.cfg0 + blockIdx.y * KB;
  const int ncfg = min(KB, a.nb - cfg0);  // configurations of this group inside the batch
  uint32_t wanted = ~0u;
  if constexpr (std::is_same<T, float>::value && PL == 0) {
    if (a.range) {
      wanted = 0;
      for (int b = 0; b < ncfg; b++) wanted |= (uint32_t)moments_wide(a.range, a.nb, cfg0 + b) << b;
      if (wanted == 0) return;
    }
  }
  const P2PChunk ch = a.chunks[live ? si.item : 0];
  const int n = (int)a.n;
  const int c = ch.count;
  const int G = 64 / c;  // lanes per target
  const int tt = lane / G, sub = lane % G;
  const bool act = tt < c;
  const int64_t it = ch.first + (act ? tt : 0);
  P2PTgt<T> tg{y[it], y[n + it], y[2 * n + it], (T)0, (T)0, (T)0};
  if constexpr (kLo) {
    tg.lx = (T)a.ylo[it];
    tg.ly = (T)a.ylo[n + it];
    tg.lz = (T)a.ylo[2 * n + it];
  }
  const int cx = a.coord[3 * ch.leaf], cy = a.coord[3 * ch.leaf + 1], cz = a.coord[3 * ch.leaf + 2];
  T* src = sS[w];
  P2PLo<T>* srclo = sL[w];
  if (lane < kP2PPad) {  // null sources past the batch (read by strides that do not divide 64)
    T* z = src + (64 + lane) * NW;
    z[0] = z[1] = z[2] = (T)1e4;
    for (int q = 3; q < NW; q++) z[q] = (T)0;
    if constexpr (kLo) {
      P2PLo<T> zl;
      zl.x = zl.y = zl.z = zl.p = (T)0;
      srclo[64 + lane] = zl;
    }
  }
  int e0 = a.near_ptr[ch.leaf], e1 = a.near_ptr[ch.leaf + 1];
  if (kSplit) {
    split_range(si.part, a.split, e0, e1);
    if (!live) e1 = e0;
  }
  // near-list metadata, 64 entries at a time (first dipole, count, own cell,
  // adjacent cell, offset in cell-relative units), read back with readlane
  int wb = e0;
  int mstart = 0, mcnt = 0, mself = 0, madj = 0;
  T mox = (T)0, moy = (T)0, moz = (T)0;
  auto load_meta = [&](int base) {
    const int e = base + lane;
    mcnt = 0;
    mself = 0;
    madj = 0;
    if (e < e1) {
      const int S = a.near_idx[e];
      mstart = a.lstart[S];
      mcnt = a.lcount[S];
      mself = S == ch.leaf;
      madj = abs(a.coord[3 * S] - cx) <= 1 && abs(a.coord[3 * S + 1] - cy) <= 1 && abs(a.coord[3 * S + 2] - cz) <= 1;
      mox = (T)((a.coord[3 * S] - cx) * a.g[0]);
      moy = (T)((a.coord[3 * S + 1] - cy) * a.g[1]);
      moz = (T)((a.coord[3 * S + 2] - cz) * a.g[2]);
    }
  };
  load_meta(wb);
  int e = e0, off = 0;
  struct Batch {
    int filled;
    bool self, adj, valid;
    int64_t j;
    T ox, oy, oz;
  };
  auto next_batch = [&]() -> Batch {
    Batch bt;
    bt.filled = 0;
    bt.self = bt.adj = bt.valid = false;
    bt.j = 0;
    bt.ox = bt.oy = bt.oz = (T)0;
    while (bt.filled < 64 && e < e1) {
      if (e - wb >= 64) {
        wb = e;
        load_meta(wb);
      }
      const int k = e - wb;
      const int cnt = __builtin_amdgcn_readlane(mcnt, k);
      const int st = __builtin_amdgcn_readlane(mstart, k);
      const int take = min(64 - bt.filled, cnt - off);
      if (lane >= bt.filled && lane < bt.filled + take) {
        bt.valid = true;
        bt.j = st + off + (lane - bt.filled);
        bt.ox = __builtin_bit_cast(T, readlane_t(mox, k));
        bt.oy = __builtin_bit_cast(T, readlane_t(moy, k));
        bt.oz = __builtin_bit_cast(T, readlane_t(moz, k));
      }
      bt.self = bt.self || __builtin_amdgcn_readlane(mself, k);
      bt.adj = bt.adj || __builtin_amdgcn_readlane(madj, k);
      bt.filled += take;
      off += take;
      if (off == cnt) {
        e++;
        off = 0;
      }
    }
    return bt;
  };
  // this lane's source of a batch: shifted position, its exact rounding
  // error joined to the stored residual (adjacent batches only), moments
  struct Src {
    T v[4 + 3 * KB];
    P2PLo<T> l;
  };
  auto load_src = [&](const Batch& bt) -> Src {
    Src q;
    q.l.x = q.l.y = q.l.z = q.l.p = (T)0;
    q.v[3] = (T)0;
    if (bt.valid) {
      const int64_t j = bt.j;
      const T hx = y[j], hy = y[n + j], hz = y[2 * n + j];
      q.v[0] = hx + bt.ox;
      q.v[1] = hy + bt.oy;
      q.v[2] = hz + bt.oz;
      if (kLo && bt.adj) {
        q.l.x = (hx - (q.v[0] - bt.ox)) + (T)a.ylo[j];
        q.l.y = (hy - (q.v[1] - bt.oy)) + (T)a.ylo[n + j];
        q.l.z = (hz - (q.v[2] - bt.oz)) + (T)a.ylo[2 * n + j];
      }
#pragma unroll
      for (int b = 0; b < KB; b++) {
        const bool in = b < ncfg;
        const T* mb = msort + (int64_t)(in ? cfg0 + b : 0) * 3 * n;
        q.v[4 + 3 * b] = in ? mb[j] : (T)0;
        q.v[5 + 3 * b] = in ? mb[n + j] : (T)0;
        q.v[6 + 3 * b] = in ? mb[2 * n + j] : (T)0;
      }
    } else {  // null source: zero moments, far from every target
      q.v[0] = q.v[1] = q.v[2] = (T)1e4;
#pragma unroll
      for (int b = 0; b < 3 * KB; b++) q.v[4 + b] = (T)0;
    }
    return q;
  };
  double h[KB][3];
#pragma unroll
  for (int b = 0; b < KB; b++) h[b][0] = h[b][1] = h[b][2] = 0.0;
  Batch cur = next_batch();
  Src qc = load_src(cur);
  while (cur.filled > 0) {
    T* slot = src + lane * NW;
#pragma unroll
    for (int q = 0; q < 4 + 3 * KB; q++) slot[q] = qc.v[q];
    if (kLo && cur.adj) srclo[lane] = qc.l;
    wave_lds_sync();
    const Batch nxt = next_batch();
    const Src qn = load_src(nxt);
    const int K = (cur.filled + G - 1) / G;
    if constexpr (!kLo) {
      if (cur.self)
        p2pk_run<T, KB, true, false>(src, srclo, G, sub, K, tg, h);
      else
        p2pk_run<T, KB, false, false>(src, srclo, G, sub, K, tg, h);
      wave_lds_sync();
    } else {
      T f[KB][3];
#pragma unroll
      for (int b = 0; b < KB; b++) f[b][0] = f[b][1] = f[b][2] = (T)0;
      if (cur.self)
        p2pk_run<T, KB, true, kLo>(src, srclo, G, sub, K, tg, f);
      else if (cur.adj)
        p2pk_run<T, KB, false, kLo>(src, srclo, G, sub, K, tg, f);
      else
        p2pk_run<T, KB, false, false>(src, srclo, G, sub, K, tg, f);
      wave_lds_sync();
#pragma unroll
      for (int b = 0; b < KB; b++) {
        h[b][0] += (double)f[b][0];
        h[b][1] += (double)f[b][1];
        h[b][2] += (double)f[b][2];
      }
    }
    cur = nxt;
    qc = qn;
  }
  // the G lanes of a target are contiguous (lane = t G + sub), G need not be
  // a power of two: a segmented tree leaves each sum in the lane with sub = 0
  for (int o = 1; o < G; o <<= 1) {
#pragma unroll
    for (int b = 0; b < KB; b++) {
      const double ox = __shfl_down(h[b][0], o), oy = __shfl_down(h[b][1], o), oz = __shfl_down(h[b][2], o);
      if (sub + o < G) {
        h[b][0] += ox;
        h[b][1] += oy;
        h[b][2] += oz;
      }
    }
  }
  if constexpr (kSplit) {
    static_assert(sizeof(sS[0]) >= 3 * 64 * sizeof(double), "the sums need the staging rows' room");
#pragma unroll
    for (int b = 0; b < KB; b++)
      split_sum(h[b], reinterpret_cast<char*>(&sS[0][0]), (int)sizeof(sS[0]), w, lane, si.part, a.split);
    if (si.part > 0 || !live) return;
  }
  if (act && sub == 0) {
    const double s3 = a.inv_s3;
    const int64_t pi = a.perm[it];
    if constexpr (PL > 0) {
      constexpr int NS = nstride(PL);
      const int pl = a.leaf_p ? a.leaf_p[ch.leaf] : PL;
#pragma unroll
      for (int b = 0; b < KB; b++)
        if (b < ncfg)
          l2p_write<T, PL>(V + a.voff + ((int64_t)ch.leaf * a.nb + cfg0 + b) * NS, pl, tg.x, tg.y, tg.z, h[b][0],
                           h[b][1], h[b][2], s3, H + ((int64_t)(cfg0 + b) * n + pi) * 3);
    } else {
      (void)V;
#pragma unroll
      for (int b = 0; b < KB; b++) {
        if (b < ncfg && (wanted >> b & 1)) {
          double* o = H + ((int64_t)(cfg0 + b) * n + pi) * 3;
          o[0] = s3 * h[b][0];
          o[1] = s3 * h[b][1];
          o[2] = s3 * h[b][2];
        }
      }
    }
  }
}

// ------------------------------------------------------------ smooth field
// The smooth field added to the near field in H (FP64, caller order): one
// configuration, one thread per dipole.
template <typename T, int P>
__global__ void k_l2p_one(int64_t n, const int32_t* __restrict__ dleaf, const int32_t* __restrict__ perm,
                          const T* __restrict__ y, const T* __restrict__ V, int64_t voff, double inv_s3,
                          const int32_t* __restrict__ leaf_p, double* __restrict__ H) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int leaf = dleaf[i];
  const SmoothMono<T, P> mono(y[i], y[n + i], y[2 * n + i]);
  T e[3];
  mono.gradient(V + voff + (int64_t)leaf * nstride(P), leaf_p ? leaf_p[leaf] : P, e);
  double* o = H + (int64_t)perm[i] * 3;
  o[0] -= inv_s3 * (double)e[0];
  o[1] -= inv_s3 * (double)e[1];
  o[2] -= inv_s3 * (double)e[2];
}

// Several configurations: one wavefront per chunk of a cell, W lanes (a power of
// two) with a dipole each and 64 / W configurations at a time, so the lanes of a
// configuration read one row of V, and H rows that are neighbours where the
// caller's dipoles are.  The monomials are formed once.  (A thread per dipole and
// configuration read a row each and wrote 24 bytes of as many arrays as there are
// configurations: 16.8 million dipoles of a film x 8 3.8 ms, now 2.7; 262,144 in a
// sphere x 64 0.97, now 0.51.)
template <typename T, int P>
__global__ void __launch_bounds__(64 * kP2PWaves) k_l2p_chunks(P2PArgs a, const T* __restrict__ y,
                                                              const T* __restrict__ V, double* __restrict__ H) {
  const int64_t item = (int64_t)blockIdx.x * kP2PWaves + (threadIdx.x >> 6);
  if (item >= *a.nchunks) return;
  const P2PChunk ch = a.chunks[item];
  const int lane = threadIdx.x & 63;
  int W = 1;
  while (W < ch.count) W <<= 1;
  const int t = lane & (W - 1);
  const bool live = t < ch.count;
  const int64_t i = ch.first + (live ? t : 0);
  const int n = (int)a.n;
  const SmoothMono<T, P> mono(y[i], y[n + i], y[2 * n + i]);
  const int pl = a.leaf_p ? a.leaf_p[ch.leaf] : P;
  const int64_t row = a.perm[i];
  const int G = 64 / W;
  for (int b = blockIdx.y * G + lane / W; b < a.nb; b += gridDim.y * G) {
    T e[3];
    mono.gradient(V + a.voff + ((int64_t)ch.leaf * a.nb + b) * nstride(P), pl, e);
    if (live) {
      double* o = H + ((int64_t)b * n + row) * 3;
      o[0] -= a.inv_s3 * (double)e[0];
      o[1] -= a.inv_s3 * (double)e[1];
      o[2] -= a.inv_s3 * (double)e[2];
    }
  }
}

P2PArgs p2p_args(Plan& P, int nb, bool fp64) {
  LevelData& D = *P.lev[P.L];
  P2PArgs a;
  a.chunks = P.chunks.as<P2PChunk>();
  a.nchunks = P.chunk_cnt.as<int32_t>() + (P.lev[P.L]->ncells + 1) + P.lev[P.L]->ncells;  // off[nl]
  a.near_ptr = D.near_ptr.as<int32_t>();
  a.near_idx = D.near_idx.as<int32_t>();
  a.coord = D.coord.as<int32_t>();
  a.lstart = P.lstart.as<int32_t>();
  a.lcount = P.lcount.as<int32_t>();
  a.perm = P.perm.as<int32_t>();
  a.n = P.n;
  a.nb = nb;
  a.cfg0 = 0;
  a.split = 1;
  for (int q = 0; q < 3; q++) a.g[q] = P.geo.lev[P.L].g[q];
  const double s = P.geo.lev[P.L].s;
  a.inv_s3 = 1.0 / (s * s * s);
  a.voff = D.qoff;
  a.leaf_p = P.has_leaf ? P.leaf_p.as<int32_t>() : nullptr;
  a.yhi = P.yf.as<float>();
  a.ylo = fp64 ? nullptr : P.yf.as<float>() + 3 * P.n;
  a.range = nullptr;
  return a;
}

// Wavefronts that share a chunk's near list, from the number of wavefronts
// that one each would give.  Sharing shortens the last wavefronts' tail and
// keeps a block's wavefronts even (they walk one list), at the price of a
// partial source batch per part: four take the clusters' 2^18 dipoles (6,300
// wavefronts) from 6.9 to 6.3 ms and a 131,072-dipole FP64 fluid from 1.01 to
// 0.94 ms; at 49,000 wavefronts (2^20 dipoles) two are the best (3.58 ms; one
// 3.70, four 3.70), as on an FP64 film window x 5 (5.42; 6.13, 5.55).  Below
// 4,096 wavefronts the near field hides beside the expansion passes, which the
// extra wavefronts only disturb (32^3 lattice: 114 us; two 117, four 122).
static int near_split(const Plan& P, int64_t waves) {
  if (P.overlap && waves <= 4096) return 1;
  return waves <= 16384 ? 4 : 2;
}

// Configurations per lane of the few-configuration near field.  FP32: the
// group size KB with the fewest vector operations, ceil(nb / KB) (13 + 10 KB)
// per pair.
static int multi_group(int nb) {
  int best = 2;
  double best_ops = 1e300;
  for (int kb : {2, 4, 8}) {
    const double ops = (double)ceil_div(nb, kb) * (13.0 + 10.0 * kb);
    if (ops < best_ops) {
      best_ops = ops;
      best = kb;
    }
  }
  return best;
}

// FP64: nb / KB full groups at 24 + 9 KB operations per pair (the reciprocal
// square root alone is worth nine) and one smaller group for the rest, in a
// launch of its own (33 configurations: four groups of 8 and one of 2).
static int group64_for(int r) {  // the smallest built group that holds r
  for (int kb : {2, 3, 4, 5, 6})
    if (r <= kb) return kb;
  return 8;
}
static int multi_group64(int nb) {
  int best = 2;
  double best_ops = 1e300;
  for (int kb : {2, 3, 4, 5, 6, 8}) {
    double ops = (double)(nb / kb) * (24.0 + 9.0 * kb);
    if (nb % kb) ops += 24.0 + 9.0 * group64_for(nb % kb);
    if (ops < best_ops) {
      best_ops = ops;
      best = kb;
    }
  }
  return best;
}

template <typename T, int KB, int PL>
static void multi_launch(Plan& P, const P2PArgs& a, const T* y, int nb, double* d_H, hipStream_t st) {
  dim3 grid(ceil_div(P.nchunks_cap, kP2PWaves), ceil_div(nb, KB));
  k_p2p_multi<T, KB, PL><<<grid, 64 * kP2PWaves, 0, st>>>(a, y, P.m_sorted.as<T>(), P.V.as<T>(), d_H);
}

// the few-configuration near field, group by group; PL > 0 adds
// the smooth field of order PL (FP32 only)
template <typename T, int PL>
static void multi_dispatch(Plan& P, P2PArgs a, const T* y, int nb, double* d_H, hipStream_t st) {
  constexpr bool fp64 = std::is_same<T, double>::value;
  static_assert(!fp64 || PL == 0, "the FP64 near field leaves the smooth field to its own pass");
  if constexpr (fp64) {
    const int nl = P.lev[P.L]->ncells;
    a.chunks = P.chunks_b.as<P2PChunk>();
    a.nchunks = P.chunk_cnt.as<int32_t>() + 3 * (nl + 1) + nl;
    const T* m = P.m_sorted.as<T>();
    constexpr int TB = 64 * kP2PWaves;
    auto launch = [&](auto kbc, int ngroups) {
      constexpr int KB = decltype(kbc)::value;
      a.split = near_split(P, (int64_t)2 * nl * ngroups);  // about two pieces a cell
      const dim3 grid(ceil_div(P.nchunks_b_cap, kP2PWaves / a.split), ngroups);
      if (a.split > 1)
        k_p2p_multi<T, KB, 0, true><<<grid, TB, 0, st>>>(a, y, m, nullptr, d_H);
      else
        k_p2p_multi<T, KB, 0><<<grid, TB, 0, st>>>(a, y, m, nullptr, d_H);
    };
    auto groups = [&](int kb, int ngroups) {
      switch (kb) {
        case 2: launch(std::integral_constant<int, 2>{}, ngroups); break;
        case 3: launch(std::integral_constant<int, 3>{}, ngroups); break;
        case 4: launch(std::integral_constant<int, 4>{}, ngroups); break;
        case 5: launch(std::integral_constant<int, 5>{}, ngroups); break;
        case 6: launch(std::integral_constant<int, 6>{}, ngroups); break;
        default: launch(std::integral_constant<int, 8>{}, ngroups); break;
      }
    };
    const int kb = multi_group64(nb);
    if (nb / kb) groups(kb, nb / kb);
    if (nb % kb) {
      a.cfg0 = nb / kb * kb;
      groups(group64_for(nb % kb), 1);
    }
  } else {
    const int kb = multi_group(nb);
    if (kb == 2)
      multi_launch<T, 2, PL>(P, a, y, nb, d_H, st);
    else if (kb == 4)
      multi_launch<T, 4, PL>(P, a, y, nb, d_H, st);
    else
      multi_launch<T, 8, PL>(P, a, y, nb, d_H, st);
  }
}

static int64_t single_waves(const Plan& P, int nb) { return ((int64_t)P.lev[P.L]->ncells + P.n / 64) * nb; }

// near field alone: written (not added) to H in the caller's order
template <typename T>
static void near_impl(Plan& P, int nb, double* d_H, hipStream_t st) {
  const bool fp64 = std::is_same<T, double>::value;
  const T* y = fp64 ? (const T*)P.yd.p : (const T*)P.yf.p;
  P2PArgs a = p2p_args(P, nb, fp64);
  if (nb >= 2 && !fp64 && P.near_f16) {
    run_near_f16(P, nb, d_H, st);
    CCFMM_HIP(hipGetLastError());
    a.range = P.gran_top.as<uint32_t>();
    multi_dispatch<T, 0>(P, a, y, nb, d_H, st);
  } else if (nb >= 2) {
    multi_dispatch<T, 0>(P, a, y, nb, d_H, st);
  } else {
    a.split = near_split(P, single_waves(P, nb));
    dim3 grid(ceil_div(P.nchunks_cap, kP2PWaves / a.split), nb);
    if (a.split > 1)
      k_p2p_one<T, true><<<grid, 64 * kP2PWaves, 0, st>>>(a, y, P.m_sorted.as<T>(), d_H);
    else
      k_p2p_one<T, false><<<grid, 64 * kP2PWaves, 0, st>>>(a, y, P.m_sorted.as<T>(), d_H);
  }
  CCFMM_HIP(hipGetLastError());
}

// smooth field of the local expansions, added to the near field in H
template <typename T, int PP>
static void l2p_impl(Plan& P, int nb, double* d_H, hipStream_t st) {
  constexpr bool fp64 = std::is_same<T, double>::value;
  const T* y = fp64 ? (const T*)P.yd.p : (const T*)P.yf.p;
  const P2PArgs a = p2p_args(P, nb, fp64);
  if (nb == 1) {
    k_l2p_one<T, PP><<<ceil_div(P.n, 256), 256, 0, st>>>(P.n, P.dleaf.as<int32_t>(), P.perm.as<int32_t>(), y,
                                                         P.V.as<T>(), a.voff, a.inv_s3, a.leaf_p, d_H);
  } else {
    // a small plan's configurations spread over as many blocks as fill the chip
    const int blocks = ceil_div(P.nchunks_cap, kP2PWaves);
    const int slices = std::max(1, std::min(ceil_div(nb, 2), 2048 / blocks));
    k_l2p_chunks<T, PP><<<dim3(blocks, slices), 64 * kP2PWaves, 0, st>>>(a, y, P.V.as<T>(), d_H);
  }
  CCFMM_HIP(hipGetLastError());
}

// near and smooth field on one stream: fused for several configurations of an
// FP32 plan on the vector units, else the smooth field in its own pass
template <typename T, int PP>
static void near_l2p_impl(Plan& P, int nb, double* d_H, hipStream_t st) {
  if constexpr (std::is_same<T, float>::value) {
    if (nb >= 2 && !P.near_f16) {
      multi_dispatch<T, PP>(P, p2p_args(P, nb, false), P.yf.as<T>(), nb, d_H, st);
      CCFMM_HIP(hipGetLastError());
      return;
    }
  }
  near_impl<T>(P, nb, d_H, st);
  l2p_impl<T, PP>(P, nb, d_H, st);
}

template <int PP>
static void l2p_d(Plan& P, int nb, double* d_H, hipStream_t st) {
  if (P.precision == CCFMM_PREC_FP64)
    l2p_impl<double, PP>(P, nb, d_H, st);
  else
    l2p_impl<float, PP>(P, nb, d_H, st);
}
template <int PP>
static void near_l2p_d(Plan& P, int nb, double* d_H, hipStream_t st) {
  if (P.precision == CCFMM_PREC_FP64)
    near_l2p_impl<double, PP>(P, nb, d_H, st);
  else
    near_l2p_impl<float, PP>(P, nb, d_H, st);
}

#define CCFMM_P2P_DISPATCH(FN)                                \
  switch (P.p) {                                              \
    case 1: FN<1>(P, nb, d_H, st); break;                     \
    case 2: FN<2>(P, nb, d_H, st); break;                     \
    case 3: FN<3>(P, nb, d_H, st); break;                     \
    case 4: FN<4>(P, nb, d_H, st); break;                     \
    case 5: FN<5>(P, nb, d_H, st); break;                     \
    case 6: FN<6>(P, nb, d_H, st); break;                     \
    case 7: FN<7>(P, nb, d_H, st); break;                     \
    case 8: FN<8>(P, nb, d_H, st); break;                     \
    default: fail(CCFMM_EINVAL, "order out of range");        \
  }

void run_near(Plan& P, int nb, double* d_H, hipStream_t st) {
  if (P.precision == CCFMM_PREC_FP64)
    near_impl<double>(P, nb, d_H, st);
  else
    near_impl<float>(P, nb, d_H, st);
}
void run_l2p(Plan& P, int nb, double* d_H, hipStream_t st) { CCFMM_P2P_DISPATCH(l2p_d) }
void run_p2p_l2p(Plan& P, int nb, double* d_H, hipStream_t st) { CCFMM_P2P_DISPATCH(near_l2p_d) }
#undef CCFMM_P2P_DISPATCH

// ------------------------------------------------------------ direct sum
// FP64 O(N) per target: the plain definition of the field at sampled targets.
// A block of 16 wavefronts takes T targets and streams every source through
// them: a source's 48 bytes are read once for T pairs, the targets sit in
// scalar registers, and the sums meet in a fixed order at the end.  Bound by
// FP64 issue (about 27 operations a pair).  1,024 targets of 2^20 dipoles:
// 9.75 ms with one wavefront per target (256 blocks of four) and IEEE square
// roots and divisions.
constexpr int kDirectThreads = 1024;

template <int T>
__global__ void __launch_bounds__(kDirectThreads) k_direct_targets(int64_t n, const double* __restrict__ pos,
                                                                   const double* __restrict__ m, int64_t nt,
                                                                   const int64_t* __restrict__ idx,
                                                                   double* __restrict__ H) {
  constexpr int NW = kDirectThreads / 64;
  __shared__ double sh[NW][3 * T];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t t0 = (int64_t)blockIdx.x * T;
  double tx[T], ty[T], tz[T], h[T][3];
  bool ok[T];
#pragma unroll
  for (int u = 0; u < T; u++) {
    int64_t i = t0 + u < nt ? idx[t0 + u] : 0;
    ok[u] = i >= 0 && i < n;
    if (!ok[u]) i = 0;  // out-of-range target: reports NaN, touches nothing
    tx[u] = pos[3 * i];
    ty[u] = pos[3 * i + 1];
    tz[u] = pos[3 * i + 2];
    h[u][0] = h[u][1] = h[u][2] = 0.0;
  }
  auto pairs = [&](double sx, double sy, double sz, double mx, double my, double mz) {
#pragma unroll
    for (int u = 0; u < T; u++) {
      const double rx = tx[u] - sx, ry = ty[u] - sy, rz = tz[u] - sz;
      const double r2 = rx * rx + ry * ry + rz * rz;
      if (r2 != 0.0) {  // the dipole itself and coincident ones are left out
        const double inv = rsqrt_t<double>(r2);
        const double inv2 = inv * inv, inv3 = inv2 * inv;
        const double k = (3.0 * inv2) * (mx * rx + my * ry + mz * rz);
        h[u][0] = fma(inv3, fma(k, rx, -mx), h[u][0]);
        h[u][1] = fma(inv3, fma(k, ry, -my), h[u][1]);
        h[u][2] = fma(inv3, fma(k, rz, -mz), h[u][2]);
      }
    }
  };
  int64_t j = threadIdx.x;
  for (; j + kDirectThreads < n; j += 2 * kDirectThreads) {  // two sources in flight
    const double* p0 = pos + 3 * j;
    const double* p1 = p0 + 3 * kDirectThreads;
    const double* m0 = m + 3 * j;
    const double* m1 = m0 + 3 * kDirectThreads;
    const double a0 = p0[0], a1 = p0[1], a2 = p0[2], b0 = m0[0], b1 = m0[1], b2 = m0[2];
    const double c0 = p1[0], c1 = p1[1], c2 = p1[2], d0 = m1[0], d1 = m1[1], d2 = m1[2];
    pairs(a0, a1, a2, b0, b1, b2);
    pairs(c0, c1, c2, d0, d1, d2);
  }
  if (j < n) pairs(pos[3 * j], pos[3 * j + 1], pos[3 * j + 2], m[3 * j], m[3 * j + 1], m[3 * j + 2]);
  // A separation whose square leaves FP64 makes the refined root inf x 0, where the
  // definition has 1 / r^3 = 0: sums that are not numbers are formed again by it
  // (tested here, once; beside every pair it took 3% of the pass).
#pragma unroll
  for (int u = 0; u < T; u++) {
    if (!__any(h[u][0] != h[u][0] || h[u][1] != h[u][1] || h[u][2] != h[u][2])) continue;
    h[u][0] = h[u][1] = h[u][2] = 0.0;
    for (int64_t k = threadIdx.x; k < n; k += kDirectThreads) {
      const double rx = tx[u] - pos[3 * k], ry = ty[u] - pos[3 * k + 1], rz = tz[u] - pos[3 * k + 2];
      const double r2 = rx * rx + ry * ry + rz * rz;
      if (r2 == 0.0) continue;
      const double inv = 1.0 / sqrt(r2), inv3 = inv * inv * inv;
      const double c = 3.0 * (m[3 * k] * rx + m[3 * k + 1] * ry + m[3 * k + 2] * rz) * inv * inv * inv3;
      h[u][0] += c * rx - inv3 * m[3 * k];
      h[u][1] += c * ry - inv3 * m[3 * k + 1];
      h[u][2] += c * rz - inv3 * m[3 * k + 2];
    }
  }
#pragma unroll
  for (int u = 0; u < T; u++)
#pragma unroll
    for (int c = 0; c < 3; c++) {
      double v = h[u][c];
      for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off);
      if (lane == 0) sh[w][3 * u + c] = v;
    }
  __syncthreads();
  if (threadIdx.x < 3 * T && t0 + threadIdx.x / 3 < nt) {
    double v = 0.0;
    for (int q = 0; q < NW; q++) v += sh[q][threadIdx.x];
    bool in = true;
#pragma unroll
    for (int u = 0; u < T; u++)
      if (u == (int)threadIdx.x / 3) in = ok[u];
    H[3 * t0 + threadIdx.x] = in ? v : __builtin_nan("");
  }
}

// ------------------------------------------------------------ energy
// E_b = -1/2 sum_i m_i . H_i (Sec. 3 with the Appendix's factor 1/2) per
// configuration, FP64.  A fixed grid of kEnergyBlocks blocks per
// configuration each sums a contiguous range of the 3n products (threads
// strided, then a tree in LDS); one block per configuration adds the partial
// sums in block order.  The order of every addition depends on n only, so
// the result is the same on every call.
constexpr int kEnergyBlocks = 256;

__global__ void __launch_bounds__(256) k_energy_part(int64_t n3, const double* __restrict__ m,
                                                     const double* __restrict__ H, double* __restrict__ part) {
  __shared__ double sh[256];
  const int b = blockIdx.y, g = blockIdx.x, t = threadIdx.x;
  const int64_t chunk = (n3 + kEnergyBlocks - 1) / kEnergyBlocks;
  const int64_t lo = (int64_t)g * chunk, hi = min(n3, lo + chunk);
  const double* mb = m + (int64_t)b * n3;
  const double* hb = H + (int64_t)b * n3;
  double s = 0.0;
  for (int64_t i = lo + t; i < hi; i += 256) s += mb[i] * hb[i];
  sh[t] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) sh[t] += sh[t + w];
    __syncthreads();
  }
  if (t == 0) part[(int64_t)b * kEnergyBlocks + g] = sh[0];
}

__global__ void __launch_bounds__(256) k_energy_final(const double* __restrict__ part, double* __restrict__ E) {
  __shared__ double sh[256];
  const int b = blockIdx.x, t = threadIdx.x;
  double s = 0.0;
  for (int g = t; g < kEnergyBlocks; g += 256) s += part[(int64_t)b * kEnergyBlocks + g];
  sh[t] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) sh[t] += sh[t + w];
    __syncthreads();
  }
  if (t == 0) E[b] = -0.5 * sh[0];
}

void run_energy(Plan& P, int nb, const double* d_m, const double* d_H, double* d_E, hipStream_t st) {
  double* part = reinterpret_cast<double*>(P.energy_part.ensure(sizeof(double) * (size_t)kEnergyBlocks * nb));
  k_energy_part<<<dim3(kEnergyBlocks, nb), 256, 0, st>>>(3 * P.n, d_m, d_H, part);
  CCFMM_HIP(hipGetLastError());
  k_energy_final<<<nb, 256, 0, st>>>(part, d_E);
  CCFMM_HIP(hipGetLastError());
}

// ------------------------------------------------------------ energy, no allocation
// The same energy with its partial sums in a fixed device array instead of a
// plan buffer, for callers that cannot allocate device memory (graph capture,
// serving loops).  Every GPU the library runs on holds its own copy of the
// array until the process ends.  Host code never passes the array's name to
// a kernel (that is a host-side stand-in); it looks up the device address
// once per device and passes that.  k_energy_part writes every slot that
// k_energy_final reads, so nothing needs clearing; overlapping calls on one
// GPU share the array and race.
static __device__ __align__(256) double scratch[kEnergyBlocks * CCFMM_NOALLOC_MAX_BATCH];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

// device address of this device's scratch array (looked up on first use)
static double* scratch_for_current_device() {
  int dev = -1;
  CCFMM_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) fail(CCFMM_EINVAL, "device ordinal beyond the supported 64");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    CCFMM_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) fail(CCFMM_EHIP, "no device address for the energy scratch array");
    g_scratch_ptr[dev] = ptr;
  }
  return static_cast<double*>(g_scratch_ptr[dev]);
}

void run_energy_noalloc(int64_t n, int nb, const double* d_m, const double* d_H, double* d_E, hipStream_t st) {
  if (nb < 1 || nb > CCFMM_NOALLOC_MAX_BATCH)
    fail(CCFMM_EINVAL, "nbatch must be in 1.." + std::to_string(CCFMM_NOALLOC_MAX_BATCH) +
                           " (the fixed partial-sum array holds that many configurations)");
  double* part = scratch_for_current_device();
  k_energy_part<<<dim3(kEnergyBlocks, nb), 256, 0, st>>>(3 * n, d_m, d_H, part);
  CCFMM_HIP(hipGetLastError());
  k_energy_final<<<nb, 256, 0, st>>>(part, d_E);
  CCFMM_HIP(hipGetLastError());
}

void run_direct_targets(int64_t n, const double* d_pos, const double* d_m, int64_t nt, const int64_t* d_idx,
                        double* d_H, hipStream_t st) {
  if (nt <= 0) return;
  // Targets per block (the sources are read once for them): one while those blocks
  // fill the compute units once, then two, then four, which beat fewer also where
  // their blocks leave units idle (2^20 dipoles, one, two and four a block: 256
  // targets 597, 617 and 1,067 us, 300 1,047, 604 and 1,064, 600 1,550, 1,219 and
  // 1,067, 1,024 2,095, 1,375 and 1,210).
  if (nt > 512)
    k_direct_targets<4><<<ceil_div(nt, 4), kDirectThreads, 0, st>>>(n, d_pos, d_m, nt, d_idx, d_H);
  else if (nt > 256)
    k_direct_targets<2><<<ceil_div(nt, 2), kDirectThreads, 0, st>>>(n, d_pos, d_m, nt, d_idx, d_H);
  else
    k_direct_targets<1><<<(unsigned)nt, kDirectThreads, 0, st>>>(n, d_pos, d_m, nt, d_idx, d_H);
  CCFMM_HIP(hipGetLastError());
}

}  // namespace ccfmm
