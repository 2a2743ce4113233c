// bse_project_blocks: H_mu = U_mu^T H U_mu and B_mu = U_mu^T B.
//
// Paper: Eq. (projection) and Eq. (transformationU), Sec. III.C.4: the
// transformation is done irrep by irrep and U is sparse (block diagonal over
// k orbits, at most |S| d_max^2 non-zeros per basis vector); the band indices
// are spectators, so
//   H_mu[(O,j,v,c),(O',j',v',c')] =
//       sum_{k in O, k' in O'} U_O[k,j] H[(k,v,c),(k',v',c')] U_O'[k',j'].
//
// Kernel k_project: one workgroup per (block, row bands (v,c), column orbit O',
// row orbit O), all blocks of a call in one launch:
//   stage 1  y_j[(k',b')] = sum_{k in O} U_O[k,j] H[(k,v,c),(k',b')]: a thread owns one
//            column (k',b') and streams the rows k straight into registers, PU
//            rows ahead; U_O comes through the scalar cache, so an element of H
//            costs one load, its conversion and 2 r FMAs, and no LDS;
//   stage 2  H_mu[j,(j',b')] = sum_{k' in O'} y_j[(k',b')] U_O'[k',j'], y staged in
//            LDS PRG vectors at a time.
// All sums in FP64.  Bound by the gathered reads of H (runs of nv nc entries).
// The earlier form staged the rows of O' in LDS and multiplied by U_O' first
// (2 r' LDS reads and conversions per element), one launch per block.  8^3 with
// 4 + 4 bands, T1u (574 MB): 312 -> 182 us (3.1 TB/s); the six blocks of
// 17 x 17 x 1 with 3 + 3 bands: 368 -> 116 us; the former block from seed
// pieces: 537 -> 240 us.
#include <hip/hip_runtime.h>

#include <vector>

#include "bse_internal.h"

namespace bse {
namespace {

constexpr int PNT = 256;     // threads per workgroup
constexpr int PMAXR = 9;     // basis vectors per orbit: d_mu m_mu(O) <= d_max^2
constexpr int PMAXL = 48;    // orbit size <= |S|
constexpr int PMAXB = 12;    // blocks per launch
// rows in flight per thread: of H in FP32 8 (182 us, 197 with 4, 205 with 12); from
// the seed pieces 4, where 8 take the registers of a wave (12 x 12 x 1, 4 + 6 bands:
// 122 us, 141 with 8)
template <typename T, bool SEEDSRC> constexpr int PU_OF = sizeof(T) == 4 && !SEEDSRC ? 8 : 4;

// One block of a launch (device pointers as in bse_block; Bmu may be NULL).
struct ProjBlk {
  const int32_t *mem_off, *members;
  const int64_t *orb_off;
  const int32_t *orb_dim;
  const int64_t *ub_off;
  const double *ub;
  void *Hmu;
  int64_t ldmu;
  double2 *Bmu;
};
struct ProjList {
  int n;
  ProjBlk b[PMAXB];
};

// Source of the H elements when projecting straight from the seed pieces
// (f1 without materialising H): every element is formed as the seed assembly
// forms it,
//   H[(k v c),(k' v' c')] = X[(o(k) v c),(o(k') v' c')] + delta (E_c - E_v)
//                           - scale D[porb(k,k')][(v c)][(v' c')],
// and rounded to T, so the projected block equals the projection of the
// assembled H exactly.
struct SeedSrc {
  const int32_t *korb, *porb;
  const double *ev, *ec;
  const void *xs, *drep;
  int64_t ldx;
  int nk;
  double scale;
};

// B_mu[(O,j,b)] = sum_{k in O} U_O[k,j] B[(k,b)] for one orbit of one block; one
// output element per thread, the members' loads four at a time.
__device__ __forceinline__ void project_vec(const ProjBlk &K, int o, int nb,
                                            const double2 *__restrict__ B) {
  const int r = K.orb_dim[o], L = K.mem_off[o + 1] - K.mem_off[o];
  const int32_t *m = K.members + K.mem_off[o];
  const double *U = K.ub + K.ub_off[o];
  for (int e = threadIdx.x; e < r * nb; e += blockDim.x) {
    const int j = e / nb, b = e % nb;
    double sr = 0, si = 0;
    for (int i = 0; i < L; i += 4) {
      double2 x[4];
      double u[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {  // members past the last read it and are dropped
        const int ii = std::min(i + q, L - 1);
        x[q] = B[int64_t(m[ii]) * nb + b];
        u[q] = U[ii * r + j];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (i + q < L) {
          sr += u[q] * x[q].x;
          si += u[q] * x[q].y;
        }
    }
    K.Bmu[K.orb_off[o] + e] = double2{sr, si};
  }
}

// A row of a basis, read through the scalar cache (the address is the same for
// every lane, the bases are never written by a kernel of this file).
typedef const __attribute__((address_space(4))) double *ConstD;
// A value that is the same for every lane, in a scalar register.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uni(int64_t x) {
  const unsigned lo = __builtin_amdgcn_readfirstlane(int(x));
  const unsigned hi = __builtin_amdgcn_readfirstlane(int(x >> 32));
  return int64_t(uint64_t(hi) << 32 | lo);
}

// One column (k',b') of the rows (k,v,c), k in O, as the kernel reads it: load()
// fetches what row i needs, value() gives the element.  From H, or formed from
// the seed pieces: the exchange entry depends on the orbits alone, so where
// every member of O has the same k orbit (ONEX, any basis of this library) it
// is loaded once per column; the diagonal term only where O is O' (diag).
template <typename T, bool SEEDSRC, bool ONEX> struct ProjSrc {
  typedef typename std::conditional<sizeof(T) == 4, float2, double2>::type C2;
  static constexpr int PU = PU_OF<T, false>;
  struct Raw {
    C2 a;
  };
  const C2 *col;
  int64_t stride;  // of k
  const int32_t *m1s;
  __device__ __forceinline__ Raw load(int i) const { return {col[int64_t(uni(m1s[i])) * stride]}; }
  __device__ __forceinline__ C2 value(const SeedSrc &, Raw r, int) const { return r.a; }
};
template <typename T, bool ONEX> struct ProjSrc<T, true, ONEX> {
  typedef typename std::conditional<sizeof(T) == 4, float2, double2>::type C2;
  static constexpr int PU = PU_OF<T, true>;
  struct Raw {
    C2 d, x;
  };
  const C2 *xcol, *dcol;  // xs of column (O', b') and drep at (band, b')
  int64_t xstride;        // xs elements of a k orbit
  int dstride;            // drep elements of a pair orbit
  C2 x0;                  // ONEX: the exchange entry
  const int32_t *m1s, *o1s, *pp;  // pair orbits (member i, this column's member)
  int L2, kdiag;          // k' where the column holds the diagonal entry of row k', else -1
  int nv, nc, band;
  __device__ __forceinline__ Raw load(int i) const {
    Raw r;
    r.d = dcol[int64_t(pp[i * L2]) * dstride];
    if constexpr (!ONEX) r.x = xcol[int64_t(o1s[i]) * xstride];
    return r;
  }
  __device__ __forceinline__ C2 value(const SeedSrc &sd, Raw r, int i) const {
    const C2 xe = ONEX ? x0 : r.x, d = r.d;
    double re = double(xe.x) - sd.scale * double(d.x), im = double(xe.y) - sd.scale * double(d.y);
    const int k = m1s[i];
    if (k == kdiag) re += sd.ec[int64_t(k) * nc + band % nc] - sd.ev[int64_t(k) * nv + band / nc];
    return C2{T(re), T(im)};
  }
};

// Stage 1 for one column: y[j] = sum_i U[i][j] h_i, PU rows in flight.  R is the
// number of basis vectors r1, or (GEN) an upper bound of it: the entries past
// r1 - 1 then read that one, and their sums are not used.
template <typename T, int R, bool GEN, typename Src>
__device__ __forceinline__ void proj_stage1(const Src &S, const SeedSrc &sd, ConstD u1, int r1,
                                            int L1, bool work, double2 (&y)[PMAXR]) {
  constexpr int PU = Src::PU;
  double ar[R], ai[R];
#pragma unroll
  for (int j = 0; j < R; ++j) ar[j] = ai[j] = 0.0;
  if (work) {
    typename Src::Raw x[PU];
#pragma unroll
    for (int u = 0; u < PU; ++u) x[u] = S.load(std::min(u, L1 - 1));
    for (int i0 = 0; i0 < L1; i0 += PU) {
      typename Src::Raw xc[PU];
#pragma unroll
      for (int u = 0; u < PU; ++u) xc[u] = x[u];
      if (i0 + PU < L1)
#pragma unroll
        for (int u = 0; u < PU; ++u) x[u] = S.load(std::min(i0 + PU + u, L1 - 1));
#pragma unroll
      for (int u = 0; u < PU; ++u) {
        if (i0 + u >= L1) break;
        const auto h = S.value(sd, xc[u], i0 + u);
        const double hr = double(h.x), hi = double(h.y);
        double w[R];
#pragma unroll
        for (int j = 0; j < R; ++j)
          w[j] = u1[GEN ? (i0 + u) * r1 + std::min(j, r1 - 1) : (i0 + u) * R + j];
#pragma unroll
        for (int j = 0; j < R; ++j) {
          ar[j] += w[j] * hr;
          ai[j] += w[j] * hi;
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < R; ++j) y[j] = double2{ar[j], ai[j]};
}
// the sizes of isotypic and partner bases, else a bound
#define BSE_PROJ_S1                                                              \
  switch (r1) {                                                                  \
    case 1: proj_stage1<T, 1, false>(S, sd, u1, r1, L1, work, y); break;         \
    case 2: proj_stage1<T, 2, false>(S, sd, u1, r1, L1, work, y); break;         \
    case 3: proj_stage1<T, 3, false>(S, sd, u1, r1, L1, work, y); break;         \
    case 4: proj_stage1<T, 4, false>(S, sd, u1, r1, L1, work, y); break;         \
    case 6: proj_stage1<T, 6, false>(S, sd, u1, r1, L1, work, y); break;         \
    case 9: proj_stage1<T, 9, false>(S, sd, u1, r1, L1, work, y); break;         \
    default: proj_stage1<T, 9, true>(S, sd, u1, r1, L1, work, y);                \
  }

// outs (dynamic LDS): [r1][r2 wb] sums over the column tiles, where there are several.
// SPLIT: the column bands b' in parts of wcol (the last may be smaller), one workgroup
// each, so that outs leaves room for the workgroups that hide the latency of a tile
// (36 bands: 47 KB of outs, two workgroups on a compute unit) and small orbits fit
// one tile.  Where: proj_parts.
constexpr int PRG = 3;  // vectors of y staged at a time (9: 271 us instead of 182)
template <typename T, bool SEEDSRC, bool SPLIT>
__global__ __launch_bounds__(PNT)
__attribute__((amdgpu_waves_per_eu(SEEDSRC && SPLIT ? 3 : 1, 8))) void k_project(
    int nv, int nc, const T *__restrict__ H, int64_t ldh, ProjList P, SeedSrc sd,
    const double2 *__restrict__ B, int bpw, int wcol) {
  typedef typename std::conditional<sizeof(T) == 4, float2, double2>::type C2;
  extern __shared__ __attribute__((aligned(16))) unsigned char plds[];
  __shared__ double2 ys[PRG * PNT];
  __shared__ double u2s[PMAXL * PMAXR];
  __shared__ int32_t m1s[PMAXL], m2s[PMAXL];
  __shared__ int32_t o1s[SEEDSRC ? PMAXL : 1], o2s[SEEDSRC ? PMAXL : 1];  // k orbits of the members
  __shared__ int32_t pps[SEEDSRC ? PMAXL * PMAXL : 1];  // pair orbits of the member pairs
  constexpr int nt = PNT;
  const int tid = threadIdx.x, nb = nv * nc;
  double2 *outs = reinterpret_cast<double2 *>(plds);
  const ProjBlk &K = P.b[blockIdx.x % P.n];
  const int ncol = SPLIT ? (nb + wcol - 1) / wcol : 1;  // parts of the column bands
  const int xp = int(blockIdx.x / P.n), c0 = SPLIT ? xp % ncol * wcol : 0;
  const int wb = SPLIT ? std::min(wcol, nb - c0) : nb;  // this part: bands c0 .. c0 + wb - 1
  const int band0 = xp / ncol * bpw;                    // first (v, c) of the output rows
  // orbit ids grow with orbit size on the simple grids, so the largest (longest)
  // orbit pairs are dispatched first and do not form a tail
  const int o2 = gridDim.y - 1 - blockIdx.y, o1 = gridDim.z - 1 - blockIdx.z;
  if (K.Bmu && xp == 0 && o1 == o2) project_vec(K, o1, nb, B);
  const int r1 = uni(K.orb_dim[o1]), r2 = uni(K.orb_dim[o2]);
  const int a1 = uni(K.mem_off[o1]), a2 = uni(K.mem_off[o2]);
  const int L1 = uni(K.mem_off[o1 + 1]) - a1, L2 = uni(K.mem_off[o2 + 1]) - a2;
  const int64_t v1 = uni(K.ub_off[o1]), v2 = uni(K.ub_off[o2]);
  const int64_t q1 = uni(K.orb_off[o1]), q2 = uni(K.orb_off[o2]);
  if (r1 == 0 || r2 == 0) return;
  // orbits have at most |S| members and bases at most d_mu^2 vectors; anything
  // else is not a valid block
  if (L1 > PMAXL || L2 > PMAXL || r1 > PMAXR || r2 > PMAXR) return;
  const int32_t *m1 = K.members + a1, *m2 = K.members + a2;
  if (tid < L2) m2s[tid] = m2[tid];
  if (tid < L1) m1s[tid] = m1[tid];
  for (int i = tid; i < L2 * r2; i += nt) u2s[i] = K.ub[v2 + i];
  bool onex = false;
  if constexpr (SEEDSRC) {
    if (tid < L2) o2s[tid] = sd.korb[m2[tid]];
    if (tid < L1) o1s[tid] = sd.korb[m1[tid]];
    for (int q = tid; q < L1 * L2; q += nt)
      pps[q] = sd.porb[int64_t(m1[q / L2]) * sd.nk + m2[q % L2]];
    onex = tid >= L1 || sd.korb[m1[tid]] == sd.korb[m1[0]];
  }
  if constexpr (SEEDSRC)
    onex = __syncthreads_and(onex);
  else
    __syncthreads();
  const ConstD u1 = (ConstD)(uintptr_t)(K.ub + v1);
  const int per = L2 * wb, oc = r2 * wb;
  // columns go to the threads in whole waves; where they take at most half of
  // them, several bands run side by side (a wave has one band)
  const int pad = std::min(nt, (per + 63) / 64 * 64), bc = nt / pad;
  const int bend = std::min(band0 + bpw, nb), bl = uni(tid / pad), ct = tid % pad;
  for (int bb = band0; bb < bend; bb += bc) {
    const int nbd = std::min(bc, bend - bb);  // bands of this round
    const int band = std::min(bb + bl, bend - 1);
    for (int t0 = 0; t0 < per; t0 += nt) {
      const int col = t0 + ct, cc = std::min(col, per - 1), i2 = cc / wb, b2 = c0 + cc % wb;
      const bool work = col < per && bl < nbd;
      double2 y[PMAXR];
      if constexpr (SEEDSRC) {
        const C2 *xcol = reinterpret_cast<const C2 *>(sd.xs) + int64_t(band) * sd.ldx +
                         int64_t(o2s[i2]) * nb + b2;
        const C2 *dcol = reinterpret_cast<const C2 *>(sd.drep) + band * nb + b2;
        const int kdiag = o1 == o2 && band == b2 ? m2s[i2] : -1;
        const C2 x0 = xcol[int64_t(o1s[0]) * nb * sd.ldx];
        if (onex) {
          const ProjSrc<T, true, true> S{xcol, dcol, nb * sd.ldx, nb * nb, x0,   m1s, o1s,
                                         pps + i2, L2, kdiag, nv, nc, band};
          BSE_PROJ_S1
        } else {
          const ProjSrc<T, true, false> S{xcol, dcol, nb * sd.ldx, nb * nb, x0,   m1s, o1s,
                                          pps + i2, L2, kdiag, nv, nc, band};
          BSE_PROJ_S1
        }
      } else {
        const ProjSrc<T, false, false> S{
            reinterpret_cast<const C2 *>(H) + band * ldh + int64_t(m2s[i2]) * nb + b2, nb * ldh, m1s};
        BSE_PROJ_S1
      }
      // ---- stage 2, PRG vectors at a time ----
      const int cn = std::min(nt, per - t0);  // columns of this tile
      const bool last = t0 + nt >= per, tiled = per > nt;  // (tiled: one band at a time)
#pragma unroll
      for (int g = 0; g < PMAXR; g += PRG) {
        if (g >= r1) break;
        __syncthreads();  // ys of the previous vectors has been read
        if (work)
#pragma unroll
          for (int q = 0; q < PRG; ++q) ys[q * nt + tid] = y[g + q];
        __syncthreads();
        const int nq = std::min(PRG, r1 - g);
        for (int e = tid; e < nbd * nq * oc; e += nt) {
          const int f = e % oc, qb = e / oc, q = qb % nq, eb = qb / nq, j2 = f / wb, bq = f % wb;
          double zr = 0, zi = 0;
          // members whose entry (k', bq) lies in this tile
          const int ia = t0 > bq ? (t0 - bq + wb - 1) / wb : 0;
          const int ib = std::min(L2, (t0 + cn - bq + wb - 1) / wb);
          const double2 *yp = ys + q * nt + eb * pad + bq - t0;
#pragma unroll 4
          for (int k2 = ia; k2 < ib; ++k2) {
            const double2 yv = yp[k2 * wb];
            const double w = u2s[k2 * r2 + j2];
            zr += w * yv.x;
            zi += w * yv.y;
          }
          if (tiled) {
            double2 &z = outs[(g + q) * oc + f];
            if (t0 > 0) {
              zr += z.x;
              zi += z.y;
            }
            z = double2{zr, zi};
          }
          if (last)
            reinterpret_cast<C2 *>(K.Hmu)[(q1 + bb + eb + int64_t(g + q) * nb) * K.ldmu + q2 +
                                          j2 * nb + c0 + bq] = C2{T(zr), T(zi)};
        }
      }
    }
  }
}

#undef BSE_PROJ_S1

// B_mu alone: one workgroup per orbit and block
__global__ __launch_bounds__(256) void k_project_vec(int nb, ProjList P,
                                                     const double2 *__restrict__ B) {
  project_vec(P.b[blockIdx.y], blockIdx.x, nb, B);
}

// |B_mu|^2 = sum over the block's orbits and basis vectors of |sum_{k in O}
// U_O[k,j] B[(k,b)]|^2, one workgroup per block (fixed summation order).
constexpr int DNT = 256;
__global__ __launch_bounds__(DNT) void k_dipole_norm(int nkorb, int nb,
                                                     const int32_t *__restrict__ mem_off,
                                                     const int32_t *__restrict__ members,
                                                     const int32_t *__restrict__ orb_dim,
                                                     const int64_t *__restrict__ ub_off,
                                                     const double *__restrict__ ub,
                                                     const double2 *__restrict__ B,
                                                     double *__restrict__ out) {
  __shared__ double sh[DNT];
  double acc = 0;
  for (int o = 0; o < nkorb; ++o) {
    const int r = orb_dim[o], L = mem_off[o + 1] - mem_off[o];
    const int32_t *m = members + mem_off[o];
    const double *U = ub + ub_off[o];
    for (int e = threadIdx.x; e < r * nb; e += DNT) {
      const int j = e / nb, b = e % nb;
      double sr = 0, si = 0;
      for (int i = 0; i < L; ++i) {
        const double2 x = B[int64_t(m[i]) * nb + b];
        sr += U[i * r + j] * x.x;
        si += U[i * r + j] * x.y;
      }
      acc += sr * sr + si * si;
    }
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int h = DNT / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

// The dipole-active block: the largest weight, if it exceeds rel times the
// total (the first such block on ties); -1 when no block carries weight.
__global__ void k_dipole_select(int nblk, const double *__restrict__ w, double rel,
                                int32_t *__restrict__ active) {
  if (threadIdx.x != 0) return;
  double tot = 0;
  for (int i = 0; i < nblk; ++i) tot += w[i];
  int best = -1;
  for (int i = 0; i < nblk; ++i)
    if (w[i] > rel * tot && (best < 0 || w[i] > w[best])) best = i;
  *active = best;
}

constexpr int PROJ_MAXCOL = 2048;  // |S| nv nc, at most

ProjBlk proj_blk(const bse_block &b, void *Hmu, int64_t ldmu, double2 *Bmu) {
  return ProjBlk{b.mem_off, b.members, b.orb_off, b.orb_dim, b.ub_off, b.ubasis, Hmu, ldmu, Bmu};
}

// Bands per workgroup: as many as leave PWGS workgroups (the tables of a
// workgroup are three dependent loads; 8^3 with 4 + 4 bands: 182 us, 196 with
// 20000 and 213 with 4096 workgroups), but few: the rows of many bands in turn keep
// workgroups side by side from reading the same stretch of H (12^3, 4 + 6 bands:
// 4.8 ms with at most 6, 5.1 with 8, 8.4 with 15, 4.9 with 1; 5.6 for a whole row
// of H at a time through LDS; 10^3: 0.76 ms, 1.07; all with the column bands whole).
constexpr int PWGS = 8192, PBPW = 6;

// Parts of the column bands (SPLIT), where the larger orbits outgrow a tile of PNT
// columns and outs takes half of the LDS: from 19 bands on two, but only where most
// orbits have more than the 12 members of a layered group (12 times 21 bands fit); from
// 22 on three (8 to 11 bands: 64 B runs at 24); from 33 on two (17 to 21: parts of 9
// or 12 read H in pieces too short).  FP32 us with one, two, three parts: 10^3, 18 bands
// 1364, 1359, 1590, 20 bands 1863, 1648, 2286; 24 x 24 x 1, 20 bands 619, 637, 807, 24
// bands 1067, 942, 850; 8^3, 30 bands 1325, 1034, 908, 36 bands 2110, 1270, 1344; 20 x
// 20 x 1, 36 bands, all blocks 4897, 3120, 4254, 3734 with four.  Calls of fewer
// workgroups than PWGS have room anyway and pay for the tables of each part (4^3, 30
// bands: 33, 29, 38).  The rule does not look at the number of blocks: a block's sums
// are the same in any company.
int proj_parts(const bse_problem *p) {
  const int nb = p->nv * p->nc;
  if (nb <= 18 || int64_t(p->nkorb) * p->nkorb * nb < PWGS) return 1;
  if (nb <= 21) return int64_t(p->grid[0]) * p->grid[1] * p->grid[2] > 12 * int64_t(p->nkorb) ? 2 : 1;
  return nb <= 32 ? 3 : 2;
}

template <typename T, bool SEEDSRC>
int32_t launch_project(const char *name, const bse_problem *p, const void *H, int64_t ldh,
                       const ProjList &L, const SeedSrc &sd, const double2 *B, hipStream_t s) {
  const int nb = p->nv * p->nc;
  const int parts = proj_parts(p), wcol = (nb + parts - 1) / parts;
  const int64_t wgs = int64_t(p->nkorb) * p->nkorb * nb * parts * L.n;
  const size_t lds = PMAXL * wcol > PNT ? sizeof(double2) * PMAXR * PMAXR * wcol : 0;
  const int bpw = int(std::max<int64_t>(1, std::min<int64_t>(std::min(nb, PBPW), wgs / PWGS)));
  const dim3 g((unsigned)((nb + bpw - 1) / bpw * parts * L.n), (unsigned)p->nkorb, (unsigned)p->nkorb);
  if (parts > 1)
    BSE_LAUNCH(name, (k_project<T, SEEDSRC, true>), g, dim3(PNT), lds, s, p->nv, p->nc,
               (const T *)H, ldh, L, sd, B, bpw, wcol);
  else
    BSE_LAUNCH(name, (k_project<T, SEEDSRC, false>), g, dim3(PNT), lds, s, p->nv, p->nc,
               (const T *)H, ldh, L, sd, B, bpw, wcol);
  BSE_HIP_CHECK(hipGetLastError());
  return BSE_OK;
}

}  // namespace
}  // namespace bse

using namespace bse;

extern "C" int32_t bse_dipole_weights(const bse_problem *p, const void *B, int32_t nblk,
                                      const bse_block *blk, double *weights, int32_t *active,
                                      bse_stream stream) {
  if (!p || !B || !weights || !active) return fail(BSE_EINVAL, "NULL pointer");
  if (nblk < 1 || !blk) return fail(BSE_EINVAL, "bad block list");
  const int n1 = p->grid[0], n2 = p->grid[1], n3 = p->grid[2];
  if (n1 < 1 || n2 < 1 || n3 < 1 || p->nv < 1 || p->nc < 1 || p->nkorb < 1)
    return fail(BSE_ESHAPE, "bad problem sizes");
  const int64_t nb = int64_t(p->nv) * p->nc, N = int64_t(n1) * n2 * n3 * nb;
  hipStream_t s = (hipStream_t)stream;
  for (int ib = 0; ib < nblk; ++ib) {
    const bse_block &b = blk[ib];
    if (b.n < 0 || !b.mem_off || !b.members || !b.orb_off || !b.orb_dim || !b.ub_off || !b.ubasis)
      return fail(BSE_EINVAL, "block %d has NULL arrays", ib);
    if (b.n > N) return fail(BSE_ESHAPE, "block %d larger than N", ib);
  }
  for (int ib = 0; ib < nblk; ++ib) {
    const bse_block &b = blk[ib];
    BSE_LAUNCH("k_dipole_norm", k_dipole_norm, dim3(1), dim3(DNT), 0, s, p->nkorb, (int)nb,
               b.mem_off, b.members, b.orb_dim, b.ub_off, b.ubasis, (const double2 *)B,
               weights + ib);
  }
  BSE_LAUNCH("k_dipole_select", k_dipole_select, dim3(1), dim3(64), 0, s, nblk,
             (const double *)weights, 1e-12, active);
  BSE_HIP_CHECK(hipGetLastError());
  return BSE_OK;
}

extern "C" int32_t bse_project_blocks(const bse_problem *p, const void *H, int64_t ldh,
                                      int32_t h_fp64, const void *B, int32_t nblk,
                                      const bse_block *blk, void *const *Hmu,
                                      const int64_t *ldmu, void *const *Bmu, bse_stream stream) {
  if (!p) return fail(BSE_EINVAL, "problem is NULL");
  if (nblk < 0 || (nblk > 0 && !blk)) return fail(BSE_EINVAL, "bad block list");
  const int n1 = p->grid[0], n2 = p->grid[1], n3 = p->grid[2];
  if (n1 < 1 || n2 < 1 || n3 < 1 || p->nv < 1 || p->nc < 1 || p->nkorb < 1)
    return fail(BSE_ESHAPE, "bad problem sizes");
  const int64_t nk = int64_t(n1) * n2 * n3, nb = int64_t(p->nv) * p->nc, N = nk * nb;
  if (int64_t(PMAXL) * nb > PROJ_MAXCOL) return fail(BSE_EUNSUPPORTED, "nv nc too large for projection");
  hipStream_t s = (hipStream_t)stream;
  for (int ib = 0; ib < nblk; ++ib) {
    const bse_block &b = blk[ib];
    if (b.n < 0 || !b.mem_off || !b.members || !b.orb_off || !b.orb_dim || !b.ub_off || !b.ubasis)
      return fail(BSE_EINVAL, "block %d has NULL arrays", ib);
    if (b.n > N) return fail(BSE_ESHAPE, "block %d larger than N", ib);
    if (Hmu && Hmu[ib]) {
      if (!H) return fail(BSE_EINVAL, "H is NULL");
      if (ldh < N) return fail(BSE_ESHAPE, "ldh < N");
      if (!ldmu || ldmu[ib] < b.n) return fail(BSE_ESHAPE, "ldmu[%d] < n", ib);
    }
    if (Bmu && Bmu[ib] && !B) return fail(BSE_EINVAL, "B is NULL");
  }
  const double2 *Bv = (const double2 *)B;
  // blocks with H_mu wanted (their B_mu comes along), then B_mu alone
  ProjList L{}, V{};
  auto flush_h = [&]() -> int32_t {
    if (L.n == 0) return BSE_OK;
    const int32_t st =
        h_fp64 ? launch_project<double, false>("k_project", p, H, ldh, L, SeedSrc{}, Bv, s)
               : launch_project<float, false>("k_project", p, H, ldh, L, SeedSrc{}, Bv, s);
    L.n = 0;
    return st;
  };
  auto flush_v = [&]() -> int32_t {
    if (V.n == 0) return BSE_OK;
    BSE_LAUNCH("k_project_vec", k_project_vec, dim3((unsigned)p->nkorb, (unsigned)V.n), dim3(256),
               0, s, (int)nb, V, Bv);
    V.n = 0;
    BSE_HIP_CHECK(hipGetLastError());
    return BSE_OK;
  };
  for (int ib = 0; ib < nblk; ++ib) {
    const bool h = Hmu && Hmu[ib], w = Bmu && Bmu[ib];
    const ProjBlk e = proj_blk(blk[ib], h ? Hmu[ib] : nullptr, h ? ldmu[ib] : 0,
                               w ? (double2 *)Bmu[ib] : nullptr);
    int32_t st = BSE_OK;
    if (h) {
      L.b[L.n++] = e;
      if (L.n == PMAXB) st = flush_h();
    } else if (w) {
      V.b[V.n++] = e;
      if (V.n == PMAXB) st = flush_v();
    }
    if (st) return st;
  }
  const int32_t st = flush_h();
  return st ? st : flush_v();
}

extern "C" int32_t bse_project_seed(int64_t plan, int32_t nblk, const bse_block *blk,
                                    void *const *Hmu, const int64_t *ldmu, bse_stream stream) {
  SeedPieces sp;
  const int32_t st = seed_pieces(plan, &sp);
  if (st) return st;
  const bse_problem *p = &sp.p;
  if (nblk < 0 || (nblk > 0 && !blk)) return fail(BSE_EINVAL, "bad block list");
  const int64_t nb = int64_t(p->nv) * p->nc, N = int64_t(sp.nk) * nb;
  if (int64_t(PMAXL) * nb > PROJ_MAXCOL) return fail(BSE_EUNSUPPORTED, "nv nc too large for projection");
  hipStream_t s = (hipStream_t)stream;
  const SeedSrc sd{p->korb, sp.porb, p->ev, p->ec, sp.xs, sp.drep, sp.ldx, sp.nk, 1.0 / sp.nk};
  for (int ib = 0; ib < nblk; ++ib) {
    if (!Hmu || !Hmu[ib]) continue;
    const bse_block &b = blk[ib];
    if (b.n < 0 || !b.mem_off || !b.members || !b.orb_off || !b.orb_dim || !b.ub_off || !b.ubasis)
      return fail(BSE_EINVAL, "block %d has NULL arrays", ib);
    if (b.n > N) return fail(BSE_ESHAPE, "block %d larger than N", ib);
    if (!ldmu || ldmu[ib] < b.n) return fail(BSE_ESHAPE, "ldmu[%d] < n", ib);
  }
  ProjList L{};
  for (int ib = 0; ib <= nblk; ++ib) {
    if (ib < nblk && Hmu && Hmu[ib]) L.b[L.n++] = proj_blk(blk[ib], Hmu[ib], ldmu[ib], nullptr);
    if (L.n == 0 || (ib < nblk && L.n < PMAXB)) continue;
    const int32_t rc =
        sp.prec == BSE_FP64
            ? launch_project<double, true>("k_project_seed", p, nullptr, 0, L, sd, nullptr, s)
            : launch_project<float, true>("k_project_seed", p, nullptr, 0, L, sd, nullptr, s);
    if (rc) return rc;
    L.n = 0;
  }
  return BSE_OK;
}
