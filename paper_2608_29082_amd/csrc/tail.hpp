// Coarse tail of the learnable V-cycle in LDS (gfx950, wave64).
//
// Levels lt .. J-1 of one cycle (or of full multigrid) for one right-hand
// side per workgroup of 1024 work-items, with every vector of those levels in
// LDS.  Columns are independent, so workgroups never synchronise with each
// other; the sweeps inside a workgroup are separated by barriers.
//
// What bounds it: a level visit is a chain of about 25 dependent sweeps
// (V(2,2), K = 3), so the cost is latency per sweep, not bytes.  A visit
// therefore loads everything it reads from global memory once, at its start,
// into registers: 1 .. 4 rows per work-item (row r of work-item t is
// t + r * 1024) with the operator's values, the row scales and the neighbours'
// LDS addresses.  The rows' own f, u and convolution input stay in registers
// too, so a sweep is W LDS reads per row, the sums and one LDS write.  Slot
// counts are compile-time (W = 4, 6 or 8, the widest row of the level rounded
// up), so a sweep's reads are all in flight before the first is used; a slot
// that a row does not have reads the zero kept behind each vector.  Levels of
// at most 64 rows run on the first wavefront without workgroup barriers.  The
// parameters and a small coarsest inverse are copied to LDS once per launch.
//
// Measured (us a launch): 33 x 33 x 1 in FP64 26 for a whole cycle (78 with
// rows read in every sweep), 65 x 65 x 1 in FP32 52, levels of 63 x 63 and
// below with 64 columns 71, with 32 columns' own operators 113 (a value of one
// column is 4 bytes in every 128 read).
//
// Levels that do not fit this form (rows of more than 8 neighbours, or more
// rows than the register variants hold) run the generic sweeps tl_*, which
// read the operator from global memory in every sweep.
#pragma once
#include "kernels.hpp"
#include "lanes.hpp"

namespace mgl {

constexpr int kTailMaxLevels = 12;
constexpr int kTailThreads = 1024;
constexpr int kTailW = 8;        // widest row of the register variants
constexpr int kTailInv = 32;     // coarsest inverses up to this size are copied to LDS

template <class C>
struct TailLevel {
  Lvl<C> L;
  Xfer<C> P;                // n_l x n_{l+1} (levels below the coarsest)
  Xfer<C> R;                // n_{l+1} x n_l
  int off_u, off_f;         // LDS offsets in units of C
  int rpt;                  // rows per work-item of the register variant (1, 2, 3, 4), 0: generic sweeps
  int w;                    // slots its rows use (at most 8); 9: the graph is not A's pattern
};
template <class C>
struct TailArgs {
  int nl;                   // number of tail levels (the last one is the coarsest)
  TailLevel<C> lv[kTailMaxLevels];
  int off_prm, off_inv, off_vec, off_wk;  // byte offsets in LDS: parameters, inverse, f and u, work buffers
  int inv_lds;              // the coarsest inverse is copied to LDS
  int KB, KR, KP, nu_pre, nu_post, per;
  const double* prm;        // flat parameters, row `per` per level, first tail level first
  const double* Ainv;       // coarsest inverse (row-major)
  int nJ;
  int nord;                 // the first nord levels sum a residual in the order of the per-level sweeps
  C* ckf[kTailMaxLevels];   // checkpoint of the levels below the first (null: not recorded)
  C* cku[kTailMaxLevels];
};

__device__ __forceinline__ float tfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double tfma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// f - A u of one row from the off-diagonal products in slot order.  The tail
// starts the sum with the diagonal; the per-level sweeps (k_resid) end with
// it: `ord` keeps the bits of a level that moved from those into the tail.
template <int W, class C>
__device__ __forceinline__ C tail_resid(const C (&a)[W], const C (&t)[W], C dg, C u, C f, int ord) {
  C s = ord ? C(0) : dg * u;
#pragma unroll
  for (int k = 0; k < W; ++k) s = tfma(a[k], t[k], s);
  return f - (ord ? tfma(dg, u, s) : s);
}

template <bool WAVE>
__device__ __forceinline__ void tail_sync() {
  if constexpr (WAVE) {
    // one wavefront: its LDS operations complete in order; only the compiler must not reorder them
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// ------------------------------------------------------------------ register variants
// What one visit of a level does, in this order: P (prolongation and its
// convolution), the smoothing steps, R (residual or f itself, its convolution
// and the restriction).
enum { TV_PRO = 1, TV_PRO_SET = 2, TV_RES = 4, TV_RES_F = 8 };

// LDS by 32-bit address: a neighbour's address in the first work buffer is one
// register, and the other two are compile-time distances away, so reading a
// neighbour in any of them is one instruction.
typedef __attribute__((address_space(3))) char lds_char;
template <class C>
__device__ __forceinline__ C lds_get(uint32_t a) {
  return *(const __attribute__((address_space(3))) C*)(uintptr_t)a;
}
template <class C>
__device__ __forceinline__ void lds_put(uint32_t a, C v) {
  *(__attribute__((address_space(3))) C*)(uintptr_t)a = v;
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) { return (uint32_t)(uintptr_t)(const lds_char*)p; }

// bytes of one work buffer of a level with rpt rows per work-item (its rows and a zero behind them)
__host__ __device__ constexpr int tail_stride(int rpt, int n, int size) {
  return (n <= 64 ? 64 : rpt * kTailThreads) * size + 64;
}

// The rows of one work-item in a level visit.  RPT rows per work-item, W slots;
// WAVE: n <= 64, one wavefront; SAME: the graph's neighbours are A's; VC / GC: the
// operator's values / the edge weights are held in registers (else they are
// read again in every sweep, from the L2).
template <int RPT, int W, bool WAVE, bool SAME, bool VC, bool GC, bool WG, class C>
struct TailRows {
  static constexpr int nt = WAVE ? 64 : kTailThreads;
  static constexpr uint32_t ST = tail_stride(RPT, WAVE ? 64 : RPT * kTailThreads, sizeof(C));
  static constexpr uint32_t S = 0, Y = ST, V = 2 * ST;   // work buffers: two for the hops, the iterate
  static constexpr uint32_t RS = nt * sizeof(C);

  const Lvl<C>& L;
  const int n, tid, ord;
  const uint32_t wk, own;         // first work buffer; this work-item's first row in it (row r at own + r RS)
  const bool act;                 // wave-uniform: this wavefront has rows
  const int vm, vb;               // per-column operators: value (k, i) at (k ld + i) vm + vb
  int ic[RPT];
  bool ok[RPT];
  uint32_t aa[RPT][W], ga[SAME ? 1 : RPT][SAME ? 1 : W];
  C av[VC ? RPT : 1][VC ? W : 1], gw[WG && GC ? RPT : 1][WG && GC ? W : 1];
  C dg[RPT], ida[RPT], idg[RPT];

  __device__ __forceinline__ TailRows(const Lvl<C>& L_, uint32_t wk_, int ord_)
      : L(L_), n(L_.n), tid(threadIdx.x), ord(ord_), wk(wk_), own(wk_ + threadIdx.x * (uint32_t)sizeof(C)),
        act((int)(threadIdx.x & ~63u) < L_.n), vm(L_.vs ? L_.vs : 1), vb(L_.vs ? vcol(L_, (int)blockIdx.x) : 0) {
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      ok[r] = tid + r * nt < n;
      ic[r] = ok[r] ? tid + r * nt : n - 1;
    }
  }
  __device__ __forceinline__ C slotv(int k, int i) const { return L.val[(k < L.w ? k : 0) * L.ld * vm + (i * vm + vb)]; }
  __device__ __forceinline__ C slotw(int k, int i) const { return L.gval[(k < L.wg ? k : 0) * L.ld + i]; }
  __device__ __forceinline__ void load() {
    if (!act) return;
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const int i = ic[r];
      int ja[W], jg[SAME ? 1 : W];
#pragma unroll
      for (int k = 0; k < W; ++k) {
        ja[k] = L.col[(k < L.w ? k : 0) * L.ld + i];
        if constexpr (!SAME) jg[k] = L.gcol[(k < L.wg ? k : 0) * L.ld + i];
        if constexpr (VC) av[r][k] = slotv(k, i);
        if constexpr (WG && GC) gw[r][k] = slotw(k, i);
      }
      dg[r] = L.diag[i * vm + vb];
      ida[r] = L.invdiag[i * vm + vb];
      idg[r] = L.invdeg[i];
#pragma unroll
      for (int k = 0; k < W; ++k) {
        // a slot the row does not have (column == row, or past the level's width) reads the zero
        // behind the vector
        aa[r][k] = wk + (ja[k] == i || k >= L.w ? n : ja[k]) * (uint32_t)sizeof(C);
        if constexpr (!SAME) ga[r][k] = wk + (jg[k] == i || k >= L.wg ? n : jg[k]) * (uint32_t)sizeof(C);
        if constexpr (VC) av[r][k] = k < L.w ? av[r][k] : C(0);
        if constexpr (WG && GC) gw[r][k] = k < L.wg ? gw[r][k] : C(0);
      }
    }
  }
  __device__ __forceinline__ void zeros() const {
    if (tid == 0) {
      lds_put<C>(wk + S + n * (uint32_t)sizeof(C), C(0));
      lds_put<C>(wk + Y + n * (uint32_t)sizeof(C), C(0));
      lds_put<C>(wk + V + n * (uint32_t)sizeof(C), C(0));
    }
  }
  __device__ __forceinline__ uint32_t nb(int r, int k) const {
    if constexpr (SAME) return aa[r][k];
    else return ga[r][k];
  }
  __device__ __forceinline__ void store(uint32_t buf, const C (&z)[RPT]) const {
    if (act)
#pragma unroll
      for (int r = 0; r < RPT; ++r)
        if (ok[r]) lds_put<C>(own + r * RS + buf, z[r]);
  }
  // x = f - A u with u in work buffer V; no branch between the rows, so that all their reads are in
  // flight together
  __device__ __forceinline__ void resid(const C (&f)[RPT], const C (&u)[RPT], C (&x)[RPT]) const {
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      C t[W], a[W];
#pragma unroll
      for (int k = 0; k < W; ++k) {
        if constexpr (VC) {
          a[k] = av[r][k];
        } else {
          const C w = slotv(k, ic[r]);
          a[k] = k < L.w ? w : C(0);
        }
      }
#pragma unroll
      for (int k = 0; k < W; ++k) t[k] = lds_get<C>(aa[r][k] + V);
      x[r] = tail_resid<W>(a, t, dg[r], u[r], f[r], ord);
    }
  }
  // neighbour sums s of the vector in work buffer `buf`
  __device__ __forceinline__ void gsum(uint32_t buf, C (&sum)[RPT]) const {
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      C t[W], e[WG ? W : 1], s = C(0);
      if constexpr (WG) {
#pragma unroll
        for (int k = 0; k < W; ++k) {
          if constexpr (GC) {
            e[k] = gw[r][k];
          } else {
            const C w = slotw(k, ic[r]);
            e[k] = k < L.wg ? w : C(0);
          }
        }
      }
#pragma unroll
      for (int k = 0; k < W; ++k) t[k] = lds_get<C>(nb(r, k) + buf);
      if constexpr (WG) {
        if (ord) {
#pragma clang fp contract(off)
#pragma unroll
          for (int k = 0; k < W; ++k) {
            const C m = t[k] * e[k];
            s = s + m;
          }
        } else {
#pragma unroll
          for (int k = 0; k < W; ++k) s = tfma(t[k], e[k], s);
        }
      } else {
#pragma unroll
        for (int k = 0; k < W; ++k) s += t[k];
      }
      sum[r] = s;
    }
  }
  // v = a G y + c x with y in work buffer `buf`
  __device__ __forceinline__ void hop(uint32_t buf, C a, C c, const C (&x)[RPT], C (&v)[RPT]) const {
    if (!act) return;
    gsum(buf, v);
#pragma unroll
    for (int r = 0; r < RPT; ++r) v[r] = hop_value(a, idg[r], v[r], c, x[r]);
  }
  // v = sum_k c_k G^k x (Horner; K >= 1); returns the hop buffer that the last hop does not read
  __device__ __forceinline__ uint32_t conv(const C* c, int K, const C (&x)[RPT], C (&v)[RPT]) const {
    store(S, x);
    tail_sync<WAVE>();
    C a = c[K];
    int k = K - 1;
#pragma nounroll
    for (; k >= 2; k -= 2) {
      hop(S, a, c[k], x, v);
      store(Y, v);
      tail_sync<WAVE>();
      hop(Y, C(1), c[k - 1], x, v);
      store(S, v);
      tail_sync<WAVE>();
      a = C(1);
    }
    if (k == 1) {
      hop(S, a, c[1], x, v);
      store(Y, v);
      tail_sync<WAVE>();
      hop(Y, C(1), c[0], x, v);
      return S;
    }
    hop(S, a, c[0], x, v);
    return Y;
  }
  // u = (uz ? 0 : u) + scale Phi(x) (K == 0: + a0 x), to work buffer V
  __device__ __forceinline__ void add(const C* c, int K, C scale, C a0, int uz, const C (&x)[RPT], C (&u)[RPT]) const {
    C v[RPT];
    if (K == 0) {
      tail_sync<WAVE>();             // x may come from a residual: every read of u ends before it changes
      if (act)
#pragma unroll
        for (int r = 0; r < RPT; ++r) u[r] = tfma(a0, x[r], uz ? C(0) : u[r]);
    } else {
      conv(c, K, x, v);
      if (act)
#pragma unroll
        for (int r = 0; r < RPT; ++r) u[r] = hop_update(uz ? C(0) : u[r], scale, v[r]);
    }
    store(V, u);
    tail_sync<WAVE>();
  }
};

// x = (X v)_i of the rows' transfer X of two slots per row (linear interpolation on nested meshes),
// its slots loaded ahead; other widths are read in place.  v: LDS, n_c values
template <int RPT, class C>
struct TailXfer2 {
  int j[RPT][2];
  C w[RPT][2];
  __device__ __forceinline__ void load(const Xfer<C>& X, const int (&ic)[RPT]) {
    if (X.w != 2) return;
#pragma unroll
    for (int r = 0; r < RPT; ++r)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        j[r][k] = X.col[k * X.n + ic[r]];
        w[r][k] = X.val[k * X.n + ic[r]];
      }
  }
  __device__ __forceinline__ void apply(const Xfer<C>& X, const int (&ic)[RPT], const C* v, C (&x)[RPT]) const {
    if (X.w == 2) {
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        const C t0 = v[j[r][0]], t1 = v[j[r][1]];
        const C g = w[r][0] != C(0) ? tfma(w[r][0], t0, C(0)) : C(0);
        x[r] = w[r][1] != C(0) ? tfma(w[r][1], t1, g) : g;
      }
    } else {
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        C g = C(0);
        for (int k = 0; k < X.w; ++k) {
          const C a = X.val[(size_t)k * X.n + ic[r]], t = v[X.col[(size_t)k * X.n + ic[r]]];
          g = a != C(0) ? tfma(a, t, g) : g;
        }
        x[r] = g;
      }
    }
  }
};
// sum of w t over the first `cnt` slots of a restriction's row, from s on (weight 0: no term).  The per-level
// sweep (k_restrict) rounds the products, the tail's own sum does not: `ord` as in tail_resid.
template <int W, class C>
__device__ __forceinline__ C tail_rsum(C s, const C (&w)[W], const C (&t)[W], int cnt, int ord) {
  if (ord) {
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const C m = w[k] * t[k];
      s = k < cnt && w[k] != C(0) ? s + m : s;
    }
  } else {
#pragma unroll
    for (int k = 0; k < W; ++k) s = k < cnt && w[k] != C(0) ? tfma(w[k], t[k], s) : s;
  }
  return s;
}
// out[i] = (X v)_i for a transfer X to at most n_c rows; v at LDS address src.  The row's slots can be
// loaded ahead (pre)
template <bool PF, class C>
struct TailXfer8 {
  int j[PF ? kTailW : 1];
  C w[PF ? kTailW : 1];
  bool pre;
  __device__ __forceinline__ void load(const Xfer<C>& X, int nt, bool want) {
    pre = PF && want && X.n <= nt && X.w >= 1 && X.w <= kTailW;
    if constexpr (PF) {
      const int tid = threadIdx.x;
      if (pre && (tid & ~63) < X.n) {
        const int e = tid < X.n ? tid : X.n - 1;
#pragma unroll
        for (int k = 0; k < kTailW; ++k) {
          const int o = (k < X.w ? k : 0) * X.n;
          j[k] = X.col[o + e];
          w[k] = X.val[o + e];
        }
      }
    }
  }
  __device__ __forceinline__ void apply(const Xfer<C>& X, int nt, uint32_t src, C* out, int ord) const {
    const int tid = threadIdx.x;
    if (pre) {
      if constexpr (PF) {
        if ((tid & ~63) < X.n) {
          C t[kTailW];
#pragma unroll
          for (int k = 0; k < kTailW; ++k) t[k] = lds_get<C>(src + j[k] * (uint32_t)sizeof(C));
          const C g = tail_rsum(C(0), w, t, X.w, ord);
          if (tid < X.n) out[tid] = g;
        }
      }
    } else {
      for (int e = tid; e < X.n; e += nt) {
        C g = C(0);
        for (int k0 = 0; k0 < X.w; k0 += kTailW) {
          int jj[kTailW];
          C ww[kTailW], t[kTailW];
#pragma unroll
          for (int k = 0; k < kTailW; ++k) {
            const size_t o = (size_t)(k0 + k < X.w ? k0 + k : k0) * X.n + e;
            jj[k] = X.col[o];
            ww[k] = X.val[o];
          }
#pragma unroll
          for (int k = 0; k < kTailW; ++k) t[k] = lds_get<C>(src + jj[k] * (uint32_t)sizeof(C));
          g = tail_rsum(g, ww, t, X.w - k0, ord);
        }
        out[e] = g;
      }
    }
  }
};

template <int RPT, int W, bool WAVE, bool SAME, bool VC, bool GC, bool WG, class C>
__device__ __forceinline__ void tail_visit(const TailArgs<C>& T, C* sm, uint32_t wk, const C* prm, int q, int what,
                                           int nsm, int uz) {
  using Rows = TailRows<RPT, W, WAVE, SAME, VC, GC, WG, C>;
  const TailLevel<C>& tl = T.lv[q];
  if (WAVE && threadIdx.x >= 64) return;
  Rows M(tl.L, wk, q < T.nord);
  C *U = sm + tl.off_u, *F = sm + tl.off_f;
  const C* p = prm + q * T.per;
  const C *cB = p + 2, *cR = cB + T.KB + 1, *cP = cR + T.KR + 1;
  const bool pro = (what & (TV_PRO | TV_PRO_SET)) != 0;
  C f[RPT], u[RPT], x[RPT];
  TailXfer2<RPT, C> P;
  if (M.act && pro) P.load(tl.P, M.ic);
  M.load();
  if (M.act)
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      f[r] = F[M.ic[r]];
      u[r] = uz ? C(0) : U[M.ic[r]];
    }
  if (!uz) M.store(Rows::V, u);
  // the restriction's row of this work-item, loaded with the level's rows where registers allow
  TailXfer8<RPT == 1 || (sizeof(C) == 4 && RPT * W <= 24), C> R;
  R.load(tl.R, Rows::nt, (what & (TV_RES | TV_RES_F)) != 0);
  M.zeros();
  if (!uz) tail_sync<WAVE>();            // the first residual gathers u

  // x = [invdiag] (f - A u)
  auto resid = [&](int jac) __attribute__((always_inline)) {
    if (!M.act) return;
    if (uz) {
#pragma unroll
      for (int r = 0; r < RPT; ++r) x[r] = f[r];
    } else {
      M.resid(f, u, x);
    }
    if (jac)
#pragma unroll
      for (int r = 0; r < RPT; ++r) x[r] *= M.ida[r];
  };
  if (pro) {
    if (M.act) P.apply(tl.P, M.ic, sm + T.lv[q + 1].off_u, x);
    M.add(cP, T.KP, C(1), cP[0], (what & TV_PRO_SET) ? 1 : uz, x, u);
    uz = 0;
  }
#pragma nounroll
  for (int j = 0; j < nsm; ++j) {
    resid(1);
    M.add(cB, T.KB, p[0], p[1], uz, x, u);
    uz = 0;
  }
  if (M.act)   // u stays with the level (zero where nothing has been added to it yet)
#pragma unroll
    for (int r = 0; r < RPT; ++r)
      if (M.ok[r]) U[M.ic[r]] = u[r];
  if (what & (TV_RES | TV_RES_F)) {
    C v[RPT];
    if (what & TV_RES) {
      resid(0);
    } else if (M.act) {
#pragma unroll
      for (int r = 0; r < RPT; ++r) x[r] = f[r];
    }
    uint32_t out = Rows::S;
    if (T.KR == 0) {
      const C a0 = cR[0];
      if (M.act)
#pragma unroll
        for (int r = 0; r < RPT; ++r) v[r] = tfma(a0, x[r], C(0));
    } else {
      out = M.conv(cR, T.KR, x, v);
    }
    M.store(out, v);
    tail_sync<WAVE>();
    R.apply(tl.R, Rows::nt, wk + out, sm + T.lv[q + 1].off_f, M.ord);
  }
  tail_sync<WAVE>();
}

// ------------------------------------------------------------------ generic sweeps
// out = [invdiag] (f - A u); every sweep reads its rows from global memory
template <class C>
__device__ __forceinline__ void tl_resid(const Lvl<C>& L, const C* f, const C* u, int uz, int jacobi, int ord, C* out) {
  const int vs = L.vs, vb = vs ? vcol(L, (int)blockIdx.x) : 0;
  auto vi = [&](size_t o) { return vs ? o * vs + vb : o; };
  for (int i = threadIdx.x; i < L.n; i += kTailThreads) {
    C z = f[i];
    if (!uz) {
      const C dg = L.diag[vi(i)], ui = u[i];
      C s = ord ? C(0) : dg * ui;
      for (int k0 = 0; k0 < L.w; k0 += kTailW) {
        C a[kTailW], t[kTailW];
#pragma unroll
        for (int k = 0; k < kTailW; ++k) {
          const size_t o = (size_t)(k0 + k < L.w ? k0 + k : k0) * L.ld + i;
          a[k] = L.val[vi(o)];
          t[k] = u[L.col[o]];
        }
#pragma unroll
        for (int k = 0; k < kTailW; ++k) s = k0 + k < L.w ? tfma(a[k], t[k], s) : s;
      }
      z -= ord ? tfma(dg, ui, s) : s;
    }
    out[i] = jacobi ? z * L.invdiag[vi(i)] : z;
  }
  __syncthreads();
}

// out = a (G yin) + c x   (mode 0)   |   out = (oz ? 0 : out) + scale (a (G yin) + c x)   (mode 1)
template <bool WG, class C>
__device__ __forceinline__ void tl_hop(const Lvl<C>& L, const C* yin, C a, const C* x, C cc, C* out, int mode,
                                       C scale, int oz, int ord) {
  for (int i = threadIdx.x; i < L.n; i += kTailThreads) {
    C s = C(0);
    for (int k0 = 0; k0 < L.wg; k0 += kTailW) {
      C e[kTailW], t[kTailW];
      int j[kTailW];
#pragma unroll
      for (int k = 0; k < kTailW; ++k) {
        const size_t o = (size_t)(k0 + k < L.wg ? k0 + k : k0) * L.ld + i;
        j[k] = L.gcol[o];
        if constexpr (WG) e[k] = L.gval[o];
      }
#pragma unroll
      for (int k = 0; k < kTailW; ++k) t[k] = yin[j[k]];
#pragma unroll
      for (int k = 0; k < kTailW; ++k) {
        const bool on = k0 + k < L.wg && j[k] != i;
        if constexpr (WG) {
          if (ord) {
#pragma clang fp contract(off)
            const C m = t[k] * e[k];
            s = on ? s + m : s;
          } else {
            s = on ? tfma(t[k], e[k], s) : s;
          }
        } else {
          s = on ? s + t[k] : s;
        }
      }
    }
    const C h = hop_value(a, L.invdeg[i], s, cc, x[i]);
    out[i] = mode == 0 ? h : hop_update(oz ? C(0) : out[i], scale, h);
  }
  __syncthreads();
}

// out = X v  for an ELL transfer X (rows X.n)
template <class C>
__device__ __forceinline__ void tl_xfer(const Xfer<C>& X, const C* v, C* out, int ord) {
  for (int i = threadIdx.x; i < X.n; i += kTailThreads) {
    C s = C(0);
    for (int k = 0; k < X.w; ++k) {
      const C w[1] = {X.val[(size_t)k * X.n + i]}, t[1] = {v[X.col[(size_t)k * X.n + i]]};
      s = tail_rsum(s, w, t, 1, ord);
    }
    out[i] = s;
  }
  __syncthreads();
}

// u = (oz ? 0 : u) + scale * sum_k c_k G^k x  (K == 0: + a0 x)
template <bool WG, class C>
__device__ __forceinline__ void tl_conv_add(const Lvl<C>& L, const C* c, int K, const C* x, C scale, C a0, C* u,
                                            int oz, C* ya, C* yb, int ord) {
  if (K == 0) {
    for (int e = threadIdx.x; e < L.n; e += kTailThreads) u[e] = tfma(a0, x[e], oz ? C(0) : u[e]);
    __syncthreads();
    return;
  }
  const C* yin = x;
  C a = c[K];
  C* buf[2] = {ya, yb};
  int cur = 0;
  for (int k = K - 1; k >= 1; --k) {
    tl_hop<WG>(L, yin, a, x, c[k], buf[cur], 0, C(0), 0, ord);
    yin = buf[cur];
    cur ^= 1;
    a = C(1);
  }
  tl_hop<WG>(L, yin, a, x, c[0], u, 1, scale, oz, ord);
}

template <bool WG, class C>
__device__ __forceinline__ void tail_visit_generic(const TailArgs<C>& T, C* sm, C* wk, const C* prm, int q, int what,
                                                   int nsm, int uz) {
  const TailLevel<C>& tl = T.lv[q];
  const Lvl<C>& L = tl.L;
  const int ord = q < T.nord, ns = (L.n + 3) / 4 * 4;
  C *U = sm + tl.off_u, *F = sm + tl.off_f, *S = wk, *Y = S + ns, *X = Y + ns, *Z = X + ns;
  const C* p = prm + q * T.per;
  const C *cB = p + 2, *cR = cB + T.KB + 1, *cP = cR + T.KR + 1;
  if (what & (TV_PRO | TV_PRO_SET)) {
    tl_xfer(tl.P, sm + T.lv[q + 1].off_u, X, 0);
    tl_conv_add<WG>(L, cP, T.KP, X, C(1), cP[0], U, (what & TV_PRO_SET) ? 1 : uz, S, Y, ord);
    uz = 0;
  }
  for (int j = 0; j < nsm; ++j) {
    tl_resid(L, F, U, uz, 1, ord, X);
    tl_conv_add<WG>(L, cB, T.KB, X, p[0], p[1], U, uz, S, Y, ord);
    uz = 0;
  }
  if (what & (TV_RES | TV_RES_F)) {
    const C* x = F;
    if (what & TV_RES) {
      tl_resid(L, F, U, uz, 0, ord, X);
      x = X;
      if (uz) {  // u is logically zero: materialise it for the prolongation's update
        for (int e = threadIdx.x; e < L.n; e += kTailThreads) U[e] = C(0);
        __syncthreads();
      }
    }
    tl_conv_add<WG>(L, cR, T.KR, x, C(1), cR[0], Z, 1, S, Y, ord);
    tl_xfer(tl.R, Z, sm + T.lv[q + 1].off_f, ord);
  }
}

// Register variants by element size, for the 128 registers of a 1024-work-item
// workgroup: FP32 holds up to four rows of eight slots (4096 rows; the edge
// weights of more than two rows are read again in each sweep), FP64 the values
// of up to two rows (one with edge weights) and the addresses of three.  One
// kernel holds them all, and its register allocation is that of the whole: the
// compiler reports 108 spilled vector registers in FP32 (122 with edge weights)
// and 32 in FP64, where a kernel of the four-row FP32 variant alone spills 18,
// of the three-row one at most 2 and of the smaller ones none.
template <class C> constexpr int tail_max_rpt() { return sizeof(C) == 4 ? 4 : 3; }

template <bool WG, class C>
__device__ __forceinline__ void tail_level(const TailArgs<C>& T, C* sm, C* wk, const C* prm, int q, int what, int nsm,
                                           int uz) {
  const int rpt = T.lv[q].rpt, w = T.lv[q].w;
  const uint32_t wa = lds_addr(wk);
  constexpr bool F32 = sizeof(C) == 4;
#define MGL_TV(R, W_, WAVE, SAME, VC, GC) tail_visit<R, W_, WAVE, SAME, VC, GC, WG, C>(T, sm, wa, prm, q, what, nsm, uz)
#define MGL_TVW(R, VC, GC)                               \
  do {                                                   \
    if (w <= 4) MGL_TV(R, 4, false, true, VC, GC);       \
    else if (w <= 6) MGL_TV(R, 6, false, true, VC, GC);  \
    else if (w <= 8) MGL_TV(R, 8, false, true, VC, GC);  \
    else MGL_TV(R, 8, false, false, VC, GC);             \
  } while (0)
  if (rpt == 0) {
    tail_visit_generic<WG>(T, sm, wk, prm, q, what, nsm, uz);
  } else if (T.lv[q].L.n <= 64) {
    if (w <= 6) MGL_TV(1, 6, true, true, true, true);
    else MGL_TV(1, 8, true, false, true, true);
    __syncthreads();
  } else if (rpt == 1) {
    MGL_TVW(1, true, true);
  } else if (rpt == 2) {
    if constexpr (F32) MGL_TVW(2, true, true);
    else MGL_TVW(2, !WG, false);
  } else if (rpt == 3) {
    if constexpr (F32) MGL_TVW(3, true, false);
    else MGL_TVW(3, false, false);
  } else {
    if constexpr (F32) MGL_TVW(4, true, false);
  }
#undef MGL_TVW
#undef MGL_TV
}

// the coarsest tail level: u = A^{-1} f (FP64 accumulation)
template <class C>
__device__ __forceinline__ void tail_coarse(const TailArgs<C>& T, C* sm, const double* inv) {
  const TailLevel<C>& tl = T.lv[T.nl - 1];
  const C* f = sm + tl.off_f;
  C* u = sm + tl.off_u;
  const Lvl<C>& LJ = tl.L;
  const int n = T.nJ;
  // per-column operators: the inverse of this workgroup's column
  const double* Ai = T.Ainv + (LJ.vs ? (size_t)vcol(LJ, (int)blockIdx.x) * n * n : 0);
  for (int i = threadIdx.x; i < n; i += kTailThreads) {
    double acc = 0.0;
    if (T.inv_lds) {
      for (int j = 0; j < n; ++j) acc = __builtin_fma(inv[i * n + j], (double)f[j], acc);
    } else {
      for (int j = 0; j < n; ++j) acc = __builtin_fma(Ai[(size_t)i * n + j], (double)f[j], acc);
    }
    u[i] = (C)acc;
  }
  __syncthreads();
}

// The level visits of one cycle over the tail levels, u_0 <- LMG(f_0, u_0) (uz0: u_0 is logically
// zero on entry; deeper levels always start from zero), or of full multigrid: the restriction
// chain of f, the coarsest solve, then per level the prolongation (set) with one cycle.  One loop
// with one call of tail_level, so that every register variant is in the code once.
template <bool WG, class C>
__device__ __forceinline__ void tail_cycle(const TailArgs<C>& T, C* sm, C* wk, const C* prm, const double* inv,
                                           int uz0, int fmg) {
  const int last = T.nl - 1;
  int down = fmg ? 2 : 1;                 // 2: full multigrid's restriction chain, 1: down, 0: up
  int top = fmg ? last - 1 : 0, q = 0;    // the current cycle's first level
#pragma nounroll
  while (true) {
    if (down && q == last) {
      tail_coarse(T, sm, inv);
      q = down == 2 ? top : last - 1;
      --down;
    }
    if (!down && q < top) {
      if (top == 0) break;
      q = --top;
      down = 1;
    }
    int what = TV_PRO, nsm = T.nu_post, uz = 0;
    if (down == 2) {
      what = TV_RES_F;
      nsm = 0;
      uz = 1;
    } else if (down) {
      what = fmg && q == top ? TV_RES | TV_PRO_SET : TV_RES;
      nsm = T.nu_pre;
      uz = q == top && !fmg ? uz0 : 1;
    }
    tail_level<WG>(T, sm, wk, prm, q, what, nsm, uz);
    q += down ? 1 : -1;
  }
}

// The parameters in the cycle's type to LDS, a level's first two replaced by what the sweeps use: eta
// theta and (K_B = 0) eta theta c_0; and a small coarsest inverse (per-column operators: the
// workgroup's column's).
template <class C>
__device__ __forceinline__ void tail_params(const TailArgs<C>& T, C* prm, double* inv) {
  for (int e = threadIdx.x; e < (T.nl - 1) * T.per; e += kTailThreads) {
    const int k = e % T.per;
    const double* p = T.prm + (e - k);
    prm[e] = (C)(k == 0 ? p[1] * p[0] : (k == 1 ? (p[1] * p[0]) * p[2] : p[k]));
  }
  if (T.inv_lds) {
    const Lvl<C>& LJ = T.lv[T.nl - 1].L;
    const double* Ai = T.Ainv + (LJ.vs ? (size_t)vcol(LJ, (int)blockIdx.x) * T.nJ * T.nJ : 0);
    for (int e = threadIdx.x; e < T.nJ * T.nJ; e += kTailThreads) inv[e] = Ai[e];
  }
}

// fmg == 0: e = LMG(A_lt, f, e) over the tail levels lt .. J-1 (uz: e is zero on entry and not read).
// fmg == 1: e = FMG(f) over the same levels: f_{q+1} = R Phi_R(f_q), exact
//           coarsest solve, then per level u_q = Phi_P(P u_{q+1}) and one cycle.
template <bool WG, class C>
__global__ __launch_bounds__(kTailThreads) void k_tail(TailArgs<C> args, int B, const C* __restrict__ fg, C* eg,
                                                       int uz, int fmg) {
  // the arguments where the launch put them (read with scalar loads): indexing the parameter itself
  // by a level would make the compiler copy it to scratch memory first
  const TailArgs<C>& T = *(const TailArgs<C>*)__builtin_amdgcn_kernarg_segment_ptr();
  extern __shared__ __align__(16) unsigned char tail_smem[];
  C* sm = reinterpret_cast<C*>(tail_smem + T.off_vec);
  C* wk = reinterpret_cast<C*>(tail_smem + T.off_wk);
  C* prm = reinterpret_cast<C*>(tail_smem + T.off_prm);
  double* inv = reinterpret_cast<double*>(tail_smem + T.off_inv);
  const int col = blockIdx.x, tid = threadIdx.x;
  const TailLevel<C>& t0 = T.lv[0];
  // four rows at a time, so that their strided loads are in flight together
  auto load = [&](const C* src, int off) {
    for (int e = tid; e < t0.L.n; e += 4 * kTailThreads) {
      C z[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) z[r] = src[(size_t)min(e + r * kTailThreads, t0.L.n - 1) * B + col];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (e + r * kTailThreads < t0.L.n) sm[off + e + r * kTailThreads] = z[r];
    }
  };
  load(fg, t0.off_f);
  if (!uz) load(eg, t0.off_u);
  tail_params(T, prm, inv);
  __syncthreads();
  tail_cycle<WG>(T, sm, wk, prm, inv, uz, fmg);
  for (int e = tid; e < t0.L.n; e += kTailThreads) eg[(size_t)e * B + col] = sm[t0.off_u + e];
  if (T.cku[1]) {
    for (int q = 1; q < T.nl; ++q)
      for (int e = tid; e < T.lv[q].L.n; e += kTailThreads) {
        T.ckf[q][(size_t)e * B + col] = sm[T.lv[q].off_f + e];
        T.cku[q][(size_t)e * B + col] = sm[T.lv[q].off_u + e];
      }
  }
}

// ------------------------------------------------------------------ reverse sweep of the tail
// The reverse of the cycle over the tail levels for one column per workgroup,
// from the levels' checkpoint (f_l and the correction u_{l+1} of every level):
// per level the forward recomputation, the transposed post-smoothing and
// prolongation (phase 0), then, after the coarser levels, the transposed
// restriction and pre-smoothing (phase 1), in the order of operations of the
// per-level sweeps (same bits).  What bounds it is what bounds k_tail: ~45
// dependent sweeps a level, where the per-level form paid ~75 launches.  A
// transposed hop z = G^T y is the neighbour sum of the row-scaled vector, so it
// reads LDS like a forward hop.  Its merged variants spill too: 206 vector
// registers in FP32 (419 with edge weights; the four-row ones alone 13 to 48),
// none in FP64 (37); 164 us a launch from 63 x 63 x 32 down.  What a level keeps
// between its phases (S_j, the residual, P e, g and gf) is private to a row and
// lives in the level's workspace vectors, stored column by column.
template <class C>
struct TailBwdLevel {
  Xfer<C> PT, RT;           // n_{l+1} x n_l and n_l x n_{l+1}
  C* keep;                  // the level's kept vectors, `stride` apart: S_0 .. S_{nu-1}, residual, P e, g, gf
  long stride;
  const C *f, *ec;          // checkpoint: f_l [n_l][B], u_{l+1} [n_{l+1}][B]
  int slot0, slot1;         // first dot slots of the phases
};
template <class C>
struct TailBwdArgs {
  TailArgs<C> T;            // off_u / off_f: gradients of a level's output and right-hand side
  TailBwdLevel<C> b[kTailMaxLevels];
  int off_dot;              // byte offset in LDS: dot products of a visit per wavefront
  Sum2* part;               // slot s of column c at s B + c
};

template <int RPT, int W, bool WAVE, bool SAME, bool VC, bool GC, bool WG, class C>
__device__ __forceinline__ void tail_bwd_visit(const TailBwdArgs<C>& A, C* sm, uint32_t wk, Sum2* dot, const C* prm,
                                               int q, int phase, int B, const C* uin, const C* gout, C* gfo, C* gul) {
  using Rows = TailRows<RPT, W, WAVE, SAME, VC, GC, WG, C>;
  const TailArgs<C>& T = A.T;
  const TailLevel<C>& tl = T.lv[q];
  const TailBwdLevel<C>& tb = A.b[q];
  if (WAVE && threadIdx.x >= 64) return;
  Rows M(tl.L, wk, 1);
  const int n = M.n, col = blockIdx.x, nu = T.nu_pre + T.nu_post, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  C *G = sm + tl.off_u, *GF = sm + tl.off_f;
  const C* p = prm + q * T.per;
  const C *cB = p + 2, *cR = cB + T.KB + 1, *cP = cR + T.KR + 1;
  C g[RPT], gf[RPT], x[RPT], s[RPT];
  int nd = 0;                      // dot slots of this visit so far
  auto keep = [&](int k) __attribute__((always_inline)) { return tb.keep + (size_t)k * tb.stride + (size_t)col * n; };
  auto put = [&](int k, const C (&z)[RPT]) __attribute__((always_inline)) {
    C* d = keep(k);
    if (M.act)
#pragma unroll
      for (int r = 0; r < RPT; ++r)
        if (M.ok[r]) d[M.ic[r]] = z[r];
  };
  auto get = [&](int k, C (&z)[RPT]) __attribute__((always_inline)) {
    const C* d = keep(k);
    if (M.act)
#pragma unroll
      for (int r = 0; r < RPT; ++r) z[r] = d[M.ic[r]];
  };
  auto dots = [&](const C (&z)[RPT]) __attribute__((always_inline)) {
    Sum2 d{0.0, 0.0};
    if (M.act) {
#pragma unroll
      for (int r = 0; r < RPT; ++r) d = sum2_add(d, M.ok[r] ? (double)z[r] * (double)s[r] : 0.0);
      d = wave_sum(d);
    }
    if (lane == 0) dot[nd * 16 + wave] = d;
    ++nd;
  };
  // x <- acc = sum_k c_k (G^T)^k x with the dots <(G^T)^k x, s>; returns the hop buffer that the last
  // hop does not read
  auto chain = [&](const C* c, int K) __attribute__((always_inline)) -> uint32_t {
    C z[RPT];
    if (M.act)
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        z[r] = x[r];
        x[r] = tfma(c[0], z[r], C(0));
      }
    dots(z);
    auto hopT = [&](uint32_t buf, C ck) __attribute__((always_inline)) {
      C t[RPT];
      if (M.act)
#pragma unroll
        for (int r = 0; r < RPT; ++r) t[r] = z[r] * M.idg[r];
      M.store(buf, t);
      tail_sync<WAVE>();
      if (M.act) {
        M.gsum(buf, z);
#pragma unroll
        for (int r = 0; r < RPT; ++r) x[r] = tfma(ck, z[r], x[r]);
      }
      dots(z);
    };
    int k = 1;
#pragma nounroll
    for (; k + 1 <= K; k += 2) {
      hopT(Rows::S, c[k]);
      hopT(Rows::Y, c[k + 1]);
    }
    if (k > K) return Rows::S;
    hopT(Rows::S, c[k]);
    return Rows::Y;
  };
  // q = alpha acc [invdiag], gf += q, g -= A q
  auto apply = [&](C alpha, int jac, bool first) __attribute__((always_inline)) {
#pragma clang fp contract(off)
    if (M.act)
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        C v = alpha * x[r];
        if (jac) v *= M.ida[r];
        x[r] = v;
        gf[r] = first ? v : gf[r] + v;
      }
    M.store(Rows::V, x);
    tail_sync<WAVE>();
    if (M.act) {
      C t[RPT];
      M.resid(g, x, t);
#pragma unroll
      for (int r = 0; r < RPT; ++r) g[r] = t[r];
    }
  };
  auto smoothT = [&](int j, bool first) __attribute__((always_inline)) {
    if (T.KB == 0) tail_sync<WAVE>();   // (a convolution's barriers otherwise end the reads of the last A q)
    get(j, s);
    if (M.act)
#pragma unroll
      for (int r = 0; r < RPT; ++r) x[r] = g[r];
    chain(cB, T.KB);
    apply(p[0], 1, first);
  };

  if (phase == 0) {
    TailXfer2<RPT, C> P;
    if (M.act) P.load(tl.P, M.ic);
    M.load();
    C f[RPT], u[RPT];
    int uz = 1;
    if (M.act)
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        f[r] = tb.f[(size_t)M.ic[r] * B + col];
        u[r] = C(0);
      }
    if (q == 0 && uin) {
      uz = 0;
      if (M.act)
#pragma unroll
        for (int r = 0; r < RPT; ++r) u[r] = uin[(size_t)M.ic[r] * B + col];
      M.store(Rows::V, u);
    }
    // the correction e_{l+1} to LDS (the next level's gf, not in use yet)
    C* E = sm + T.lv[q + 1].off_f;
    const int nc = T.lv[q + 1].L.n;
    for (int e = threadIdx.x; e < nc; e += Rows::nt) E[e] = tb.ec[(size_t)e * B + col];
    M.zeros();
    tail_sync<WAVE>();
    auto resid = [&](int jac) __attribute__((always_inline)) {
      if (!M.act) return;
      if (uz) {
#pragma unroll
        for (int r = 0; r < RPT; ++r) x[r] = f[r];
      } else {
        M.resid(f, u, x);
      }
      if (jac)
#pragma unroll
        for (int r = 0; r < RPT; ++r) x[r] *= M.ida[r];
    };
    // forward recomputation; the iterate after the last step is not needed
#pragma nounroll
    for (int j = 0; j < T.nu_pre; ++j) {
      resid(1);
      put(j, x);
      M.add(cB, T.KB, p[0], p[1], uz, x, u);
      uz = 0;
    }
    resid(0);
    put(nu, x);
    if (M.act) P.apply(tl.P, M.ic, E, x);
    put(nu + 1, x);
    if (T.nu_post) M.add(cP, T.KP, C(1), cP[0], uz, x, u);
    uz = 0;
#pragma nounroll
    for (int j = 0; j < T.nu_post; ++j) {
      resid(1);
      put(T.nu_pre + j, x);
      if (j + 1 < T.nu_post) M.add(cB, T.KB, p[0], p[1], 0, x, u);
    }
    // reverse
    if (M.act)
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        g[r] = q == 0 ? gout[(size_t)M.ic[r] * B + col] : G[M.ic[r]];
        gf[r] = C(0);
      }
    tail_sync<WAVE>();             // the work buffers change hands
#pragma nounroll
    for (int j = T.nu_post - 1; j >= 0; --j) smoothT(T.nu_pre + j, j == T.nu_post - 1);
    get(nu + 1, s);
    if (M.act)
#pragma unroll
      for (int r = 0; r < RPT; ++r) x[r] = g[r];
    const uint32_t out = chain(cP, T.KP);
    M.store(out, x);
    put(nu + 2, g);
    put(nu + 3, gf);
    tail_sync<WAVE>();
    TailXfer8<false, C> R;
    R.load(tb.PT, Rows::nt, false);
    R.apply(tb.PT, Rows::nt, wk + out, sm + T.lv[q + 1].off_u, 0);   // (k_prolong fuses its products)
  } else {
    TailXfer2<RPT, C> P;
    if (M.act) P.load(tb.RT, M.ic);
    M.load();
    get(nu + 2, g);
    get(nu + 3, gf);
    M.zeros();
    if (M.act) P.apply(tb.RT, M.ic, sm + T.lv[q + 1].off_f, x);
    get(nu, s);
    chain(cR, T.KR);
    apply(C(1), 0, T.nu_post == 0);
#pragma nounroll
    for (int j = T.nu_pre - 1; j >= 0; --j) smoothT(j, false);
    if (M.act)
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        if (!M.ok[r]) continue;
        if (q == 0) {
          gfo[(size_t)M.ic[r] * B + col] = gf[r];
          if (gul) gul[(size_t)M.ic[r] * B + col] = g[r];
        } else {
          GF[M.ic[r]] = gf[r];
        }
      }
  }
  tail_sync<WAVE>();
  // the visit's dot products over the wavefronts, in order
  for (int t = threadIdx.x; t < nd; t += Rows::nt) {
    Sum2 d{0.0, 0.0};
    for (int w = 0; w < Rows::nt / 64; ++w) d = sum2_add(d, dot[t * 16 + w]);
    A.part[(size_t)((phase ? tb.slot1 : tb.slot0) + t) * B + col] = d;
  }
  tail_sync<WAVE>();
}

template <bool WG, class C>
__device__ __forceinline__ void tail_bwd_level(const TailBwdArgs<C>& A, C* sm, C* wk, Sum2* dot, const C* prm, int q,
                                               int phase, int B, const C* uin, const C* gout, C* gfo, C* gul) {
  const int rpt = A.T.lv[q].rpt, w = A.T.lv[q].w;
  const uint32_t wa = lds_addr(wk);
  constexpr bool F32 = sizeof(C) == 4;
#define MGL_TB(R, W_, WAVE, SAME, VC, GC) \
  tail_bwd_visit<R, W_, WAVE, SAME, VC, GC, WG, C>(A, sm, wa, dot, prm, q, phase, B, uin, gout, gfo, gul)
#define MGL_TBW(R, VC, GC)                               \
  do {                                                   \
    if (w <= 6) MGL_TB(R, 6, false, true, VC, GC);       \
    else if (w <= 8) MGL_TB(R, 8, false, true, VC, GC);  \
    else MGL_TB(R, 8, false, false, VC, GC);             \
  } while (0)
  if (A.T.lv[q].L.n <= 64) {
    if (w <= 6) MGL_TB(1, 6, true, true, true, true);
    else MGL_TB(1, 8, true, false, true, true);
    __syncthreads();
  } else if (rpt == 1) {
    MGL_TBW(1, true, true);
  } else if (rpt == 2) {
    if constexpr (F32) MGL_TBW(2, true, false);
    else MGL_TBW(2, false, false);
  } else {
    if constexpr (F32) MGL_TBW(4, true, false);
  }
#undef MGL_TBW
#undef MGL_TB
}
// rows per work-item of a level in the reverse sweep (0: not in it)
template <class C> constexpr int tail_bwd_rpt(int rpt) {
  return sizeof(C) == 4 ? (rpt == 3 ? 4 : rpt) : (rpt <= 2 ? rpt : 0);
}

template <bool WG, class C>
__global__ __launch_bounds__(kTailThreads) void k_tail_bwd(TailBwdArgs<C> args, int B, const C* __restrict__ uin,
                                                           const C* __restrict__ gout, C* __restrict__ gfo,
                                                           C* __restrict__ gul) {
  extern __shared__ __align__(16) unsigned char tail_smem[];
  const TailBwdArgs<C>& A = *(const TailBwdArgs<C>*)__builtin_amdgcn_kernarg_segment_ptr();   // (as in k_tail)
  const TailArgs<C>& T = A.T;
  C* sm = reinterpret_cast<C*>(tail_smem + T.off_vec);
  C* wk = reinterpret_cast<C*>(tail_smem + T.off_wk);
  C* prm = reinterpret_cast<C*>(tail_smem + T.off_prm);
  double* inv = reinterpret_cast<double*>(tail_smem + T.off_inv);
  Sum2* dot = reinterpret_cast<Sum2*>(tail_smem + A.off_dot);
  tail_params(T, prm, inv);
  __syncthreads();
  const int last = T.nl - 1;
  int phase = 0, q = 0;
#pragma nounroll
  while (q >= 0) {
    if (q == last) {
      // gf = A^{-T} g
      const TailLevel<C>& tl = T.lv[last];
      const double* Ai = T.inv_lds ? nullptr : T.Ainv;
      for (int i = threadIdx.x; i < T.nJ; i += kTailThreads) {
        double acc = 0.0;
        for (int j = 0; j < T.nJ; ++j)
          acc = __builtin_fma(Ai ? Ai[(size_t)j * T.nJ + i] : inv[j * T.nJ + i], (double)sm[tl.off_u + j], acc);
        sm[tl.off_f + i] = (C)acc;
      }
      __syncthreads();
      phase = 1;
      q = last - 1;
    }
    tail_bwd_level<WG>(A, sm, wk, dot, prm, q, phase, B, uin, gout, gfo, gul);
    q += phase ? -1 : 1;
  }
}

// The two kernels are the bulk of the device code: each precision is a translation unit of its own
// (tail_f32.hip, tail_f64.hip), compiled beside the engines'.
#define MGL_TAIL_KERNELS(EXTERN, C)                                                              \
  EXTERN template __global__ void k_tail<false, C>(TailArgs<C>, int, const C*, C*, int, int);    \
  EXTERN template __global__ void k_tail<true, C>(TailArgs<C>, int, const C*, C*, int, int);     \
  EXTERN template __global__ void k_tail_bwd<false, C>(TailBwdArgs<C>, int, const C*, const C*, C*, C*); \
  EXTERN template __global__ void k_tail_bwd<true, C>(TailBwdArgs<C>, int, const C*, const C*, C*, C*);

}  // namespace mgl
