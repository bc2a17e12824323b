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
// too, so a sweep is W LDS reads per row, the sums and one LDS write.  Slot counts are compile-time (W = 4, 6 or 8, the
// widest row of the level rounded up), so a sweep's reads are all in flight
// before the first is used; a slot that a row does not have reads the zero
// kept behind each vector.  Levels of at most 64 rows run on the first
// wavefront without workgroup barriers.  The parameters and a small coarsest
// inverse are copied to LDS once per launch.
//
// Levels that do not fit this form (rows of more than 8 neighbours, or more
// rows than the register variants hold) run the generic sweeps tl_*, which
// read the operator from global memory in every sweep.
#pragma once
#include "kernels.hpp"

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
  int lt;                   // global index of the first tail level
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

// RPT rows per work-item, W slots; WAVE: n <= 64, one wavefront; SAME: the
// graph's neighbours are A's; VC / GC: the operator's values / the edge weights
// are held in registers (else they are read again in every sweep, from the L2)
template <int RPT, int W, bool WAVE, bool SAME, bool VC, bool GC, bool WG, class C>
__device__ __forceinline__ void tail_visit(const TailArgs<C>& T, C* sm, uint32_t wk, const C* prm, int q, int what,
                                           int nsm, int uz) {
  const TailLevel<C>& tl = T.lv[q];
  const Lvl<C>& L = tl.L;
  const int n = L.n, tid = threadIdx.x;
  constexpr int nt = WAVE ? 64 : kTailThreads;
  constexpr uint32_t ST = tail_stride(RPT, WAVE ? 64 : RPT * kTailThreads, sizeof(C));
  constexpr uint32_t S = 0, Y = ST, V = 2 * ST;   // work buffers: two for the hops, the iterate
  if (WAVE && tid >= 64) return;
  const bool act = (tid & ~63) < n;      // wave-uniform: this wavefront has rows
  const int ord = q < T.nord;
  C *U = sm + tl.off_u, *F = sm + tl.off_f;
  const C* p = prm + q * T.per;
  const C *cB = p + 2, *cR = cB + T.KB + 1, *cP = cR + T.KR + 1;
  // per-column operators: value (k, i) of this workgroup's column at (k ld + i) vm + vb
  const int vm = L.vs ? L.vs : 1, vb = L.vs ? vcol(L, (int)blockIdx.x) : 0;
  auto slotv = [&](int k, int i) { return L.val[(k < L.w ? k : 0) * L.ld * vm + (i * vm + vb)]; };
  auto slotw = [&](int k, int i) { return L.gval[(k < L.wg ? k : 0) * L.ld + i]; };
  const bool pro = (what & (TV_PRO | TV_PRO_SET)) != 0;

  const uint32_t own = wk + tid * (uint32_t)sizeof(C);     // row r at own + r * RS
  constexpr uint32_t RS = nt * sizeof(C);
  int ic[RPT];
  bool ok[RPT];
  uint32_t aa[RPT][W], ga[SAME ? 1 : RPT][SAME ? 1 : W];
  C av[VC ? RPT : 1][VC ? W : 1], gw[WG && GC ? RPT : 1][WG && GC ? W : 1];
  C dg[RPT], ida[RPT], idg[RPT], f[RPT], u[RPT], x[RPT], v[RPT];
  // a prolongation of two slots per row (linear interpolation on nested meshes), loaded first
  const Xfer<C>& P = tl.P;
  int pj[RPT][2];
  C pw[RPT][2];
  if (act) {
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      ok[r] = tid + r * nt < n;
      ic[r] = ok[r] ? tid + r * nt : n - 1;
    }
    if (pro && P.w == 2) {
#pragma unroll
      for (int r = 0; r < RPT; ++r)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          pj[r][k] = P.col[k * P.n + ic[r]];
          pw[r][k] = P.val[k * P.n + ic[r]];
        }
    }
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
      f[r] = F[i];
      u[r] = uz ? C(0) : U[i];
      if (!uz && ok[r]) lds_put<C>(own + r * RS + V, u[r]);
    }
  }
  // the restriction's row of this work-item, loaded with the level's rows where registers allow
  constexpr bool PF = RPT == 1 || (sizeof(C) == 4 && RPT * W <= 24);
  const Xfer<C>& R = tl.R;
  const bool pre = PF && (what & (TV_RES | TV_RES_F)) && R.n <= nt && R.w >= 1 && R.w <= kTailW;
  int rj[PF ? kTailW : 1];
  C rw[PF ? kTailW : 1];
  if constexpr (PF) {
    if (pre && (tid & ~63) < R.n) {
      const int e = tid < R.n ? tid : R.n - 1;
#pragma unroll
      for (int k = 0; k < kTailW; ++k) {
        const int o = (k < R.w ? k : 0) * R.n;
        rj[k] = R.col[o + e];
        rw[k] = R.val[o + e];
      }
    }
  }
  if (tid == 0) {
    lds_put<C>(wk + S + n * (uint32_t)sizeof(C), C(0));
    lds_put<C>(wk + Y + n * (uint32_t)sizeof(C), C(0));
    lds_put<C>(wk + V + n * (uint32_t)sizeof(C), C(0));
  }
  if (!uz) tail_sync<WAVE>();            // the first residual gathers u

  auto nb = [&](int r, int k) { return SAME ? aa[r][k] : ga[SAME ? 0 : r][SAME ? 0 : k]; };
  auto store = [&](uint32_t buf, const C (&z)[RPT]) {
    if (act)
#pragma unroll
      for (int r = 0; r < RPT; ++r)
        if (ok[r]) lds_put<C>(own + r * RS + buf, z[r]);
  };
  // x = [invdiag] (f - A u); no branch between the rows, so that all their reads are in flight together
  auto resid = [&](int jac) {
    if (uz) {
#pragma unroll
      for (int r = 0; r < RPT; ++r) x[r] = f[r];
    } else {
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
    if (jac)
#pragma unroll
      for (int r = 0; r < RPT; ++r) x[r] *= ida[r];
  };
  // v = a G y + c x with y in work buffer `buf`
  auto hop = [&](uint32_t buf, C a, C c) {
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
      v[r] = hop_value(a, idg[r], s, c, x[r]);
    }
  };
  // v = sum_k c_k G^k x (Horner; K >= 1); returns the hop buffer that the last hop does not read
  auto conv = [&](const C* c, int K) -> uint32_t {
    store(S, x);
    tail_sync<WAVE>();
    C a = c[K];
    int k = K - 1;
#pragma nounroll
    for (; k >= 2; k -= 2) {
      if (act) hop(S, a, c[k]);
      store(Y, v);
      tail_sync<WAVE>();
      if (act) hop(Y, C(1), c[k - 1]);
      store(S, v);
      tail_sync<WAVE>();
      a = C(1);
    }
    if (k == 1) {
      if (act) hop(S, a, c[1]);
      store(Y, v);
      tail_sync<WAVE>();
      if (act) hop(Y, C(1), c[0]);
      return S;
    }
    if (act) hop(S, a, c[0]);
    return Y;
  };
  // u = (uz ? 0 : u) + scale Phi(x) (K == 0: + a0 x), to LDS
  auto add = [&](const C* c, int K, C scale, C a0) {
    if (K == 0) {
      tail_sync<WAVE>();             // x may come from a residual: every read of u ends before it changes
      if (act)
#pragma unroll
        for (int r = 0; r < RPT; ++r) u[r] = tfma(a0, x[r], uz ? C(0) : u[r]);
    } else {
      conv(c, K);
      if (act)
#pragma unroll
        for (int r = 0; r < RPT; ++r) u[r] = hop_update(uz ? C(0) : u[r], scale, v[r]);
    }
    uz = 0;
    store(V, u);
    tail_sync<WAVE>();
  };

  if (pro) {
    const C* E = sm + T.lv[q + 1].off_u;
    if (act) {
      if (P.w == 2) {
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          const C t0 = E[pj[r][0]], t1 = E[pj[r][1]];
          C g = pw[r][0] != C(0) ? tfma(pw[r][0], t0, C(0)) : C(0);
          x[r] = pw[r][1] != C(0) ? tfma(pw[r][1], t1, g) : g;
        }
      } else {
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          C g = C(0);
          for (int k = 0; k < P.w; ++k) {
            const C w = P.val[(size_t)k * P.n + ic[r]], t = E[P.col[(size_t)k * P.n + ic[r]]];
            g = w != C(0) ? tfma(w, t, g) : g;
          }
          x[r] = g;
        }
      }
    }
    if (what & TV_PRO_SET) uz = 1;
    add(cP, T.KP, C(1), cP[0]);
  }
#pragma nounroll
  for (int j = 0; j < nsm; ++j) {
    if (act) resid(1);
    add(cB, T.KB, p[0], p[1]);
  }
  if (act)   // u stays with the level (zero where nothing has been added to it yet)
#pragma unroll
    for (int r = 0; r < RPT; ++r)
      if (ok[r]) U[ic[r]] = u[r];
  if (what & (TV_RES | TV_RES_F)) {
    if (act) {
      if (what & TV_RES) resid(0);
      else
#pragma unroll
        for (int r = 0; r < RPT; ++r) x[r] = f[r];
    }
    uint32_t out = S;
    if (T.KR == 0) {
      const C a0 = cR[0];
      if (act)
#pragma unroll
        for (int r = 0; r < RPT; ++r) v[r] = tfma(a0, x[r], C(0));
    } else {
      out = conv(cR, T.KR);
    }
    store(out, v);
    tail_sync<WAVE>();
    const uint32_t src = wk + out;
    C* G = sm + T.lv[q + 1].off_f;
    if (pre) {
      if constexpr (PF) {
        if ((tid & ~63) < R.n) {
          C t[kTailW], g = C(0);
#pragma unroll
          for (int k = 0; k < kTailW; ++k) t[k] = lds_get<C>(src + rj[k] * (uint32_t)sizeof(C));
#pragma unroll
          for (int k = 0; k < kTailW; ++k) g = k < R.w && rw[k] != C(0) ? tfma(rw[k], t[k], g) : g;
          if (tid < R.n) G[tid] = g;
        }
      }
    } else {
      for (int e = tid; e < R.n; e += nt) {
        C g = C(0);
        for (int k0 = 0; k0 < R.w; k0 += kTailW) {
          int j[kTailW];
          C w[kTailW], t[kTailW];
#pragma unroll
          for (int k = 0; k < kTailW; ++k) {
            const size_t o = (size_t)(k0 + k < R.w ? k0 + k : k0) * R.n + e;
            j[k] = R.col[o];
            w[k] = R.val[o];
          }
#pragma unroll
          for (int k = 0; k < kTailW; ++k) t[k] = lds_get<C>(src + j[k] * (uint32_t)sizeof(C));
#pragma unroll
          for (int k = 0; k < kTailW; ++k) g = k0 + k < R.w && w[k] != C(0) ? tfma(w[k], t[k], g) : g;
        }
        G[e] = g;
      }
    }
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
__device__ __forceinline__ void tl_xfer(const Xfer<C>& X, const C* v, C* out) {
  for (int i = threadIdx.x; i < X.n; i += kTailThreads) {
    C s = C(0);
    for (int k = 0; k < X.w; ++k) {
      const C w = X.val[(size_t)k * X.n + i];
      s = w != C(0) ? tfma(w, v[X.col[(size_t)k * X.n + i]], s) : s;
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
    tl_xfer(tl.P, sm + T.lv[q + 1].off_u, X);
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
    tl_xfer(tl.R, Z, sm + T.lv[q + 1].off_f);
  }
}

// Register variants by element size, the widest that stay within the 128
// registers of a 1024-work-item workgroup: FP32 holds up to four rows of eight
// slots (4096 rows; the edge weights of more than two rows are read again in
// each sweep), FP64 the values of up to two rows (one with edge weights) and the
// addresses of three.
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
  // the parameters in the cycle's type, a level's first two replaced by what the sweeps use:
  // eta theta and (K_B = 0) eta theta c_0
  for (int e = tid; e < (T.nl - 1) * T.per; e += kTailThreads) {
    const int k = e % T.per;
    const double* p = T.prm + (e - k);
    prm[e] = (C)(k == 0 ? p[1] * p[0] : (k == 1 ? (p[1] * p[0]) * p[2] : p[k]));
  }
  if (T.inv_lds) {
    const Lvl<C>& LJ = T.lv[T.nl - 1].L;
    const double* Ai = T.Ainv + (LJ.vs ? (size_t)vcol(LJ, col) * T.nJ * T.nJ : 0);
    for (int e = tid; e < T.nJ * T.nJ; e += kTailThreads) inv[e] = Ai[e];
  }
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

}  // namespace mgl
