// One panel (NBK columns) of the one-stage reduction in a single launch (FP64
// storage).
// Included by bse_eigh.hip inside its anonymous namespace.
//
// The columns of a panel depend on one another through two exchanges over all
// rows: the column itself, then the scalars that its product with the trailing
// block gives.  As launches of their own (k_colA, k_colB) each costs 2.7 us of
// launch boundary and reloads the panel: 12.2 us a column at n = 720, 16 us at
// n = 2160.  Here G workgroups stay for the panel and exchange through memory:
//   * a workgroup owns g_pan_rows(m) consecutive rows.  Their V and W entries
//     stay in LDS; A is read through the caches as before.
//   * exchanged words are written once per column at agent scope into rings of
//     four (column index mod 4) that start as XNONE, a signalling NaN that no
//     arithmetic produces; a reader polls the words it needs until none is XNONE
//     (one hop, where data + flag would be three).  Whoever has every workgroup's
//     sum of column i knows that all have finished column i - 1, and restores its
//     own words of that column.  The restore completes (wait_stores) before the
//     writer's sum of column i + 2 goes out, and nobody polls column i + 3, the
//     next user of those words, before having that sum: a reader never takes an
//     old word for a new one.  The launches before the panel (k_rank2, k_her2k)
//     leave every word XNONE.
//   * every wait ends: the workgroups of a panel count themselves in at the
//     start, and only when all have arrived does anyone wait for data.  If they
//     have not within PAN_WAIT (workgroups that no compute unit has room for, for
//     instance because several such panels from other streams wait in the same
//     way), the panel is given up as a joint effort before any data was written:
//     all leave but workgroup 0, which runs every workgroup's part in turn (the
//     same code and sums, so the same bits; a solve whose every panel is given up
//     takes 70 ms instead of 1.0 at n = 162, 634 instead of 5.4 at 720, 4.6 s
//     instead of 30 ms at 2300, of which 20 ms a panel are the wait).  A launch holds at most PAN_WGS
//     workgroups, three of which fit a compute unit: four launches fit side by
//     side on the device, and a device that holds fewer takes smaller panels
//     (g_pan_limit).
// Measured (one box, before -> now, us per column all in): n = 720 12.4 -> 6.6 (solve
// 8.73 -> 5.28 ms), n = 162 (solve with build and spectra 1.57 -> 1.07 ms), n = 1500 (solve
// 22.2 -> 14.1 ms).  Of the 16000 cycles of a column at n = 720 the two exchanges take
// about half, the product with A (through L2) a quarter, the sums over panel columns
// the rest.  PAN_M: at 2000 and 2300 rows (12 rows per workgroup) 33.5 -> 23.0 and
// 41.7 -> 29.8 ms the solve; beyond, the lower-tile product of k_colA reads half of A.
// Arithmetic and conventions are those of k_colA / k_colB: per column jn = j0 + i, with m0 = jn + 1,
//   A  v = (1, sc col), y = A22 v for the own rows, partial y^dag v; workgroups
//      g, g + G, .. of the 2 i dot products V_l^dag col, W_l^dag col sum those;
//   B  p, q, alpha, the own rows of W_i and of column jn + 1, their partial dot
//      products for the next column.

typedef unsigned long long u64;
constexpr u64 XNONE = 0x7ff1dead5eed5eedull;
constexpr long long PAN_WAIT = 2000000;  // 20 ms of the 100 MHz clock
// Polls of a committed panel (seconds).  Its waits end by themselves unless the device
// is broken; a word that never came is a NaN in every later column and so in the
// tridiagonal, where k_tri_prep turns it into a solve without finite eigenvalues.
constexpr int PAN_SPIN = 1 << 22;

__device__ __forceinline__ u64 xld(const u64 *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void xst(u64 *p, u64 v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void xput(u64 *p, double2 v) {  // complex entry: two words
  xst(p, u64(__double_as_longlong(v.x)));
  xst(p + 1, u64(__double_as_longlong(v.y)));
}
__device__ __forceinline__ double2 xval(u64 a, u64 b) {
  return double2{__longlong_as_double((long long)a), __longlong_as_double((long long)b)};
}
__device__ __forceinline__ void wait_stores() { __builtin_amdgcn_s_waitcnt(0); }

// One ring slot of the exchange words of a block (D.px); entries are complex.
typedef PanParts<u64 *> PanX;
__device__ __forceinline__ PanX pan_slot(u64 *px, int64_t n, int ring) {
  return g_pan_parts(px + 2 * g_pan_ctrl(n) + ring * g_pan_ring(n), n);
}

// Every ring word to XNONE and (ctrl) the entry counters to zero, shared by the
// nwgs workgroups of a launch in front of the panel.  Where workgroups are taken never
// to arrive, their count (the first word of each pair) starts that much below zero and
// the panels are given up.
__device__ __forceinline__ void pan_clear(const Desc &D, int64_t wg, int64_t nwgs, bool ctrl) {
  if (!D.px) return;
  const int64_t c = 2 * g_pan_ctrl(D.n), w = g_pan_words(D.n);
  u64 *px = reinterpret_cast<u64 *>(D.px);
  for (int64_t k = wg * blockDim.x + threadIdx.x; k < w; k += nwgs * blockDim.x) {
    if (k >= c) px[k] = XNONE;
    else if (ctrl) px[k] = k & 1 ? 0 : u64(-int64_t(D.pan_absent));
  }
}

template <int WR>
__device__ __forceinline__ void b_panel(const Desc &D, int j0, int g0) {
  constexpr int RWM = WR * (ENT / 64);  // rows per workgroup (WR per wave)
  extern __shared__ __attribute__((aligned(16))) unsigned char pan_lds[];
  double2 *vs = reinterpret_cast<double2 *>(pan_lds);  // the column, rows j0 .. n - 1
  __shared__ double2 VW[RWM][2 * NBK + 1];  // own rows of V_0.. | W_0..
  __shared__ double2 hs[2 * NBK], bs[2 * NBK];
  __shared__ double2 ysh[RWM], vsh[RWM], prod[RWM], ash[RWM], csh[RWM], yjs;
  __shared__ double sh[ENT / 64], sh2[2 * (ENT / 64)];
  __shared__ int mode_s;
  // 32-bit indices: at most PAN_M + 1 rows from row j0 on, and n <= 65536
  const int n = (int)D.n, lda = (int)D.lda, ldv = (int)D.ldv, m = n - j0 - 1;
  const int RW = RWM, G = g_pan_wgs(m);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const double2 *A = reinterpret_cast<const double2 *>(D.A) + int64_t(j0) * D.lda;  // from row j0
  u64 *px = reinterpret_cast<u64 *>(D.px);
  // ---- entry: count in, wait until all have, or give up ----
  {
    if (tid == 0) {
      u64 *cnt = px + 2 * (j0 / NBK), *state = cnt + 1;  // zeroed by k_rank2 of this solve
      int st = 0;
      if (__hip_atomic_fetch_add(cnt, u64(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
          u64(G - 1)) {
        u64 e = 0;
        __hip_atomic_compare_exchange_strong(state, &e, u64(1), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
      }
      const long long t0 = wall_clock64();
      while ((st = int(xld(state))) == 0) {
        if (wall_clock64() - t0 > PAN_WAIT) {
          u64 e = 0;
          __hip_atomic_compare_exchange_strong(state, &e, u64(2), __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      mode_s = st;
    }
    __syncthreads();
  }
  const bool solo = mode_s == 2;  // (uniform over the panel: the state is set once)
  if (solo && g0 != 0) return;
  const int gb = solo ? 0 : g0, ge = solo ? G : g0 + 1;
  for (int i = 0; i < NBK; ++i) {
    const int jn = j0 + i, m0 = jn + 1;
    const PanX X = pan_slot(px, n, i & (PAN_RING - 1)), XN = pan_slot(px, n, (i + 1) & (PAN_RING - 1));
    double2 tau = {0, 0}, sc = {0, 0};
    // ================= A =================
    for (int g = gb; g < ge; ++g) {
      const int rb = j0 + 1 + g * RW, nr = std::min(RW, n - rb);
      // rows of this wave: rb + wv + 4 k; the first loads of A do not wait for the column
      constexpr int HP = 2;
      double2 an[WR][HP];
      double2 a0[WR];
      int arow[WR];
#pragma unroll
      for (int k = 0; k < WR; ++k) {
        const int rr = wv + (ENT / 64) * k;
        const int r = rb + std::min(rr, nr - 1);
        arow[k] = (r - j0) * lda;
        a0[k] = A[arow[k] + m0];
#pragma unroll
        for (int u = 0; u < HP; ++u)
          an[k][u] = A[arow[k] + std::min(m0 + 1 + lane + 64 * u, n - 1)];
      }
      // ---- the column (rows jn .. n - 1) and the head rows of V, W ----
      double s1 = 0;
      auto keep = [&](int r, double2 x) {
        vs[r - j0] = x;
        if (r >= m0 + 1) s1 += x.x * x.x + x.y * x.y;
      };
      if (i == 0) {
        for (int r = jn + tid; r < n; r += ENT) keep(r, A[(r - j0) * lda + j0]);
      } else {
        constexpr int CB = 4;  // entries polled together
        const bool hd = tid < 2 * NBK && (tid & (NBK - 1)) < i;  // with the first of them
        for (int r0 = jn; r0 < n; r0 += CB * ENT) {
          u64 wa[CB], wb[CB], ha = 0, hb = 0;
          bool miss = true;
          for (int t = 0; miss && t < PAN_SPIN; ++t) {
            miss = false;
            if (hd && r0 == jn) {
              ha = xld(X.head + 2 * tid);
              hb = xld(X.head + 2 * tid + 1);
            }
#pragma unroll
            for (int u = 0; u < CB; ++u) {
              const int r = r0 + tid + ENT * u;
              wa[u] = wb[u] = 0;
              if (r < n) {
                wa[u] = xld(X.col + 2 * r);
                wb[u] = xld(X.col + 2 * r + 1);
              }
            }
#pragma unroll
            for (int u = 0; u < CB; ++u) miss |= wa[u] == XNONE || wb[u] == XNONE;
            miss |= ha == XNONE || hb == XNONE;
          }
          if (hd && r0 == jn) hs[tid] = xval(ha, hb);
#pragma unroll
          for (int u = 0; u < CB; ++u) {
            const int r = r0 + tid + ENT * u;
            if (r < n) keep(r, xval(wa[u], wb[u]));
          }
        }
      }
      s1 = sum64(s1);
      if (lane == 0) sh[wv] = s1;
      __syncthreads();  // sh, vs, hs
      double S1 = sh[0];
#pragma unroll
      for (int w = 1; w < ENT / 64; ++w) S1 += sh[w];
      double beta;
      fast_householder(vs[m0 - j0], S1, beta, tau, sc);
      // the records of this wave's first dot product (published after the column):
      // on their way during the product with A, which does not need them
      const int s0 = g + G * wv;
      u64 ra[4], rc[4];
      if (s0 < 2 * i) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const u64 *q = X.rec + (std::min(lane + 64 * u, G - 1) * 2 * NBK + s0) * 2;
          ra[u] = xld(q);
          rc[u] = xld(q + 1);
        }
      }
      // ---- y = A22 v on the own rows: sums over the columns c > m0 of A col ----
      {
        double sr[WR], si[WR];
#pragma unroll
        for (int k = 0; k < WR; ++k) sr[k] = si[k] = 0;
        // (nothing to do once every own row is above the trailing block)
        for (int c0 = rb + nr > m0 ? m0 + 1 : n; c0 < n; c0 += 64 * HP) {
          double2 ac[WR][HP];
#pragma unroll
          for (int k = 0; k < WR; ++k)
#pragma unroll
            for (int u = 0; u < HP; ++u) {
              ac[k][u] = an[k][u];
              an[k][u] = A[arow[k] + std::min(c0 + 64 * (HP + u) + lane, n - 1)];
            }
#pragma unroll
          for (int u = 0; u < HP; ++u) {
            const int c = c0 + lane + 64 * u;
            const bool ok = c < n;
            const double2 x = vs[std::min(c, n - 1) - j0];
#pragma unroll
            for (int k = 0; k < WR; ++k) {
              const double2 a = ok ? ac[k][u] : double2{0, 0};
              sr[k] += a.x * x.x - a.y * x.y;
              si[k] += a.x * x.y + a.y * x.x;
            }
          }
        }
#pragma unroll
        for (int k = 0; k < WR; ++k) {
          sr[k] = sum64(sr[k]);
          si[k] = sum64(si[k]);
          const int rr = wv + (ENT / 64) * k;
          if (lane == 0 && rr < RWM) {
            const int r = rb + rr;
            const bool on = rr < nr && r >= m0;
            const double2 y = cadd(a0[k], cmul(sc, double2{sr[k], si[k]}));
            const double2 v = !on ? double2{0, 0} : r == m0 ? double2{1, 0} : cmul(sc, vs[r - j0]);
            ysh[rr] = y;
            vsh[rr] = v;
            ash[rr] = a0[k];
            prod[rr] = on ? cmulc(y, v) : double2{0, 0};
            if (on) D.V[i * ldv + r] = v;
            if (solo && on) D.y[r] = y;
          }
        }
      }
      // ---- dot products of the previous columns: one wave per product ----
      for (int s = s0; s < 2 * i; s += G * (ENT / 64)) {
        bool miss = true;
        for (int t = 0; t < PAN_SPIN; ++t) {
          if (t > 0 || s != s0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const u64 *q = X.rec + (std::min(lane + 64 * u, G - 1) * 2 * NBK + s) * 2;
              ra[u] = xld(q);
              rc[u] = xld(q + 1);
            }
          }
          miss = false;
#pragma unroll
          for (int u = 0; u < 4; ++u) miss |= ra[u] == XNONE || rc[u] == XNONE;
          if (!miss) break;
        }
        double2 x = {0, 0};
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (lane + 64 * u < G) x = cadd(x, xval(ra[u], rc[u]));
        x.x = sum64(x.x);
        x.y = sum64(x.y);
        if (lane == 0) xput(X.bred + 2 * s, x);
      }
      __syncthreads();  // ysh, vsh, prod
      if (tid == 0) {
        double2 t = prod[0];
        for (int rr = 1; rr < nr; ++rr) t = cadd(t, prod[rr]);
        xput(X.pa + 2 * g, t);
        if (g == 0) {
          D.d[jn] = vs[jn - j0].x;
          D.e[jn] = beta;
          D.tau[m0] = tau;
          D.scl[m0] = sc;
        }
      }
      if (tid == 64 && m0 >= rb && m0 < rb + nr) xput(X.yj, ysh[m0 - rb]);
      if (solo) {
        wait_stores();
        __syncthreads();
      }
    }
    // ================= B =================
    for (int g = gb; g < ge; ++g) {
      const int rb = j0 + 1 + g * RW, nr = std::min(RW, n - rb);
      if (solo) {  // this workgroup's rows and the head entries again
        __syncthreads();
        for (int e = tid; e < RWM * 2 * NBK; e += ENT) {
          const int rr = e / (2 * NBK), s = e % (2 * NBK), l = s & (NBK - 1);
          if (rr < nr && l < i) VW[rr][s] = (s < NBK ? D.V : D.W)[l * ldv + rb + rr];
        }
        if (tid < nr) {
          const int r = rb + tid;
          vsh[tid] = r >= m0 ? D.V[i * ldv + r] : double2{0, 0};
          ysh[tid] = r >= m0 ? D.y[r] : double2{0, 0};
          ash[tid] = A[(r - j0) * lda + m0];
        }
      }
      double2 pv;
      {
        // pa[tid], and bred[tid] or yj
        const u64 *q = X.pa + 2 * tid, *e = tid < 2 * i ? X.bred + 2 * tid : X.yj;
        const bool nq = tid < G, ne = tid < 2 * i || tid == ENT - 1;
        u64 a = 0, b = 0, c = 0, d = 0;
        for (int t = 0; t < PAN_SPIN; ++t) {
          if (nq) {
            a = xld(q);
            b = xld(q + 1);
          }
          if (ne) {
            c = xld(e);
            d = xld(e + 1);
          }
          if (a != XNONE && b != XNONE && c != XNONE && d != XNONE) break;
        }
        pv = nq ? xval(a, b) : double2{0, 0};
        if (tid < 2 * i) bs[tid] = xval(c, d);
        if (tid == ENT - 1) yjs = xval(c, d);
      }
      wait_stores();  // the XNONE stores of column i - 1, before anything of column i + 1 goes out
      pv.x = sum64(pv.x);
      pv.y = sum64(pv.y);
      if (lane == 0) {
        sh2[2 * wv] = pv.x;
        sh2[2 * wv + 1] = pv.y;
      }
      __syncthreads();  // sh2, bs, yjs
      pv = double2{sh2[0], sh2[1]};  // y^dag v
#pragma unroll
      for (int w = 1; w < ENT / 64; ++w) pv = cadd(pv, double2{sh2[2 * w], sh2[2 * w + 1]});
      // half-wave hw: rows hw, hw + 8 of the workgroup; lane l: panel column l
      const int l = tid & (NBK - 1), hw = tid / NBK;
      double2 vh = {0, 0}, wh = {0, 0}, p = {0, 0}, q = {0, 0};
      if (l < i) {
        vh = hs[l];
        wh = hs[NBK + l];
        p = cadd(cconj(vh), cmul(sc, bs[2 * l]));
        q = cadd(cconj(wh), cmul(sc, bs[2 * l + 1]));
      }
      constexpr int HR = (RWM + ENT / NBK - 1) / (ENT / NBK);  // rows per half-wave
      double pq = p.x * q.x + p.y * q.y;                       // Re(p^dag q)
      double2 sj = cadd(cmul(vh, q), cmul(wh, p));
      double2 t1[HR], t2[HR];
#pragma unroll
      for (int h = 0; h < HR; ++h) {
        const int rr = hw + (ENT / NBK) * h;
        double2 vl = {0, 0}, wl = {0, 0};
        if (l < i && rr < nr) {
          vl = VW[rr][l];
          wl = VW[rr][NBK + l];
        }
        t1[h] = cadd(cmul(vl, q), cmul(wl, p));
        t2[h] = cadd(cmul(vl, cconj(wh)), cmul(wl, cconj(vh)));
      }
      pq = sum32(pq);
      sj = double2{sum32(sj.x), sum32(sj.y)};
#pragma unroll
      for (int h = 0; h < HR; ++h) {
        t1[h] = double2{sum32(t1[h].x), sum32(t1[h].y)};
        t2[h] = double2{sum32(t2[h].x), sum32(t2[h].y)};
      }
      const double2 wdv = cmulc(tau, double2{pv.x - 2 * pq, pv.y});
      const double2 al = cmul(double2{-0.5 * tau.x, -0.5 * tau.y}, wdv);
      const double2 wj = cadd(cmul(tau, csub(yjs, sj)), al);  // W_i[m0] (v = 1 there)
#pragma unroll
      for (int h = 0; h < HR; ++h) {
        const int rr = hw + (ENT / NBK) * h;
        const int r = rb + rr;
        if (l == 0 && rr < nr) {
          const bool on = r >= m0;
          const double2 v = vsh[rr];
          const double2 w = on ? cadd(cmul(tau, csub(ysh[rr], t1[h])), cmul(al, v)) : double2{0, 0};
          const double2 c = csub(csub(ash[rr], t2[h]), cadd(cmul(v, cconj(wj)), w));
          VW[rr][i] = v;
          VW[rr][NBK + i] = w;
          csh[rr] = c;
          if (on) {
            if (i + 1 < NBK) xput(XN.col + 2 * r, c);
            D.W[i * ldv + r] = w;
          }
        }
      }
      if (i + 1 < NBK) {
        __syncthreads();  // VW, csh
        {  // partial dot products of the next column, rows > m0 + 1: four lanes each
          const int sl = tid >> 2, x = (sl & 1) * NBK + (sl >> 1);
          double2 t = {0, 0};
#pragma unroll
          for (int k = 0; k < RWM / 4; ++k) {
            const int rr = (tid & 3) + 4 * k;
            if (rr < nr && rb + rr > m0 + 1 && (sl >> 1) <= i) t = cadd(t, cmulc(VW[rr][x], csh[rr]));
          }
          t.x += dppd<DPP_X1>(t.x);
          t.y += dppd<DPP_X1>(t.y);
          t.x += dppd<DPP_X2>(t.x);
          t.y += dppd<DPP_X2>(t.y);
          if ((tid & 3) == 0 && (sl >> 1) <= i) xput(XN.rec + (g * 2 * NBK + sl) * 2, t);
        }
        const int hj = m0 + 1;  // the next column's head row
        const int t = tid - ENT / 2;
        if (t >= 0 && t < 2 * NBK && (t & (NBK - 1)) <= i && hj >= rb && hj < rb + nr)
          xput(XN.head + 2 * t, VW[hj - rb][t]);
      }
      // ---- every workgroup has finished column i - 1: its words back to XNONE ----
      if (i > 0) {
        const PanX XP = pan_slot(px, n, (i + PAN_RING - 1) & (PAN_RING - 1));
        const int t = tid - ENT / 2;
        if (t >= 0) {
          if (t < 2 * nr) xst(XP.col + 2 * rb + t, XNONE);
          xst(XP.rec + g * 4 * NBK + t, XNONE);
          if (t < 2) xst(XP.pa + 2 * g + t, XNONE);
          for (int s = g; s < 2 * NBK; s += G)
            if (t < 2) xst(XP.bred + 2 * s + t, XNONE);
          if (jn >= rb && jn < rb + nr) {  // owner of the head row of column i - 1
            xst(XP.head + t, XNONE);
            if (t < 2) xst(XP.yj + t, XNONE);
          }
        }
      }
      if (solo) {
        wait_stores();
        __syncthreads();
      }
    }
  }
}

template <int WR>
__global__ __launch_bounds__(ENT, 3) void k_panel(Desc D, int64_t j0) {
  b_panel<WR>(D, int(j0), int(blockIdx.x));
}
// batched: nact blocks from Ds on.  Workgroups are dispatched in order, so the
// oldest panel with workgroups missing gets them as earlier panels end.
template <int WR>
__global__ __launch_bounds__(ENT, 3) void k_panel_b(const Desc *__restrict__ Ds,
                                                 const int *__restrict__ pre, int nact,
                                                 int64_t j0) {
  BSE_FIND_BLOCK
  b_panel<WR>(D, int(j0), wg);
}
