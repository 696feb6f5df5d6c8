// Small problems: ADMM iterations up to and including the next residual check that needs the host, or a
// whole PCG solve, in one launch of one workgroup.
//
// A problem of some hundred variables keeps the general path (one kernel per pass, 6 per PCG step
// and 5 more per ADMM iteration) at 2–3 µs per kernel on the device and 3.5–6 µs per launch on the
// host, whatever the arithmetic takes. Here the passes are phases of one kernel, separated by
// workgroup barriers; the vectors that a PCG step reads and writes, the slots and the work lists are in
// LDS, and where they fit as well, the ADMM vectors (AV) and the matrices (ML). What bounds it then is the chain of six
// phases per PCG step and, with the matrices in memory, their stream into one compute unit
// (64 bytes a clock, ≈ 150 GB/s); the problems taken end where the general path's whole chip wins
// (kSmallBytes).
//
// Every number is the one that the general path computes, bit for bit: each lane sums the segment
// that it sums there, a row's segment sums are added in the same order by the same lanes
// (combine_item), the epilogues and vector steps are the same functions, and the reductions are
// taken over the same 256-thread groups, four wavefronts of elements each, in the same trees. A check
// that neither ends the solve nor follows a stall is decided on the device too (small_decide, the host's
// arithmetic on the same norms); every other one, trials and PCG solves that fail stay with the host.
#pragma once

#include "kernels.hpp"

namespace qpg {

// Threads: 512 where the matrices are in LDS (enough for a phase's latencies, and cheaper barriers:
// control with 320 variables 27.3 ms against 31.0 with 1024), 1024 where they are streamed (the random
// QP of 200 variables 2.7 ms against 3.05).
template <bool ML>
constexpr int kSmallBlock = ML ? 512 : 1024;
constexpr int kSmallGroups = 64;     // 256-thread groups of any reduction at most: one tree's lanes
constexpr int kSmallIters = 256;     // ADMM iterations of one launch at most
constexpr int kSmallPcg = 4096;      // PCG iterations of one launch at most
constexpr int kSmallCols = 65535;    // columns and slots of a matrix at most (16-bit indices)

// Lane j's step s of a chunk is at base + 64·s + j.
struct SmallChunk {
  int32_t base, steps;
};
// Rows [r0, r1) of one 256-thread group, 2^lg lanes per row.
struct SmallItem {
  uint16_t r0, r1;
  int32_t lg;
};

// A work list for the one-workgroup kernels: the general path's segments with the slots renumbered
// in row order (row r's are [rowslot[r], rowslot[r + 1])) and 16-bit columns in value order.
template <typename T>
struct SmallMat {
  const SmallChunk* chunks;
  const SmallItem* items;
  const uint16_t *segslot, *rowslot, *col;  // segslot 65535: an empty lane
  const T* val;
  int32_t nchunk, nitem, nslot, nval, nrows;
  int32_t rows;  // segments_are_rows
};

// How the right-hand side of a launch's first iteration is formed (qpg_solver::admm): directly, by
// the recurrence in a B pass, or from a check's product B·g as it is or rescaled to a new ρ̄.
enum SmallRhs : int32_t { kRhsDirect, kRhsRec, kRhsRows, kRhsRescaled };

// Byte offsets of the LDS arrays.
struct SmallLds {
  int32_t wp, wq;  // wavefront partials of the passes, of the vector step
  int32_t pw, xt, r, kp, dinv, zt, slots;
  int32_t chunk[2], item[2], segslot[2], rowslot[2];  // Ā, B
  int32_t x, z, g, bk, qb, lb, ub, ax;                // ADMM vectors (AV): x is [x; y], g its plane 0
  int32_t val[2], col[2];                             // matrices (ML)
};

template <typename T>
struct SmallArgs {
  SmallMat<T> A, B;
  SmallLds o;
  T *x, *y, *z, *xt, *r, *p, *dinv, *bk, *zt, *g, *bg, *b, *dxy;
  const T *qb, *lb, *ub;
  double* ax;
  const double *dscale, *escale, *diagP, *colsq;
  DevState* st;
  HostRead hr;
  int32_t n, m;
  T sigma, alpha, rho, rho_inv, gamma, ratio;
  double sigma64, rho64, eps;
  int32_t maxit, rel;
  int32_t k0, k1;        // ADMM iterations of this launch
  int32_t refresh;       // the right-hand side is formed directly at multiples of it
  int32_t first_rhs;     // SmallRhs of iteration k0
  int32_t new_rho;       // ρ̄ has changed: 1: g is formed for it, 2: and the Jacobi diagonal
  int32_t check_every, max_iter;  // checks: multiples of check_every, and max_iter
  int32_t zt_every;      // every zt_every-th check recomputes z̃ by an Ā pass (0: none)
  int32_t exact_after;   // a check recomputes Āx̄ after more PCG steps than this (FP32; else a large number)
  int32_t pair, pair_after;  // a check forms the next B·g as well, unless it took more PCG steps than this
  int32_t decide;        // checks are decided on the device where they can be (small_decide)
  int32_t since, stall;  // checks since the best residual; the host decides from `stall` of them on
  int32_t rho_every, fixed_eps;
  double rho_b, bg_rho, best, tighten;
  double c, q_norm, qb_norm, eps_abs, eps_rel, lambda, eps_min, gate;
  int32_t bg_for;
  int32_t vgrid, ugrid;  // workgroups of the general path's vector kernels over n and max(n, m)
  int32_t resume;        // k_small_pcg: continue the solve in the device scalars
};

// The launch's arguments, read from the kernel's argument memory where they are used: the pointer is
// made opaque, so that a phase's scalar loads are not hoisted out of it (a hundred pointers held over
// the whole kernel spilled). Such a read takes ≈ 1 µs, so what every PCG step needs is read once, into
// the context below, and stays in scalar registers.
template <typename T>
__device__ __forceinline__ const SmallArgs<T>& small_now() {
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const SmallArgs<T>*)p;
}

template <typename T>
struct SmallCtx {
  SmallLds o;
  int32_t n, m, vgrid, maxit;
  int32_t nchunk[2], nitem[2], nslot[2];
  bool rows_A;  // each row of Ā has one segment: a slot is a row, no sums of slots to wait for
  const T* val[2];
  const uint16_t* col[2];
  T sigma, alpha, rho, rho_inv;
  double eps;
  int32_t rel;
  __device__ __forceinline__ void get() {
    const SmallArgs<T>& a = small_now<T>();
    o = a.o;
    n = a.n;
    m = a.m;
    vgrid = a.vgrid;
    maxit = a.maxit;
    nchunk[0] = a.A.nchunk;
    nchunk[1] = a.B.nchunk;
    nitem[0] = a.A.nitem;
    nitem[1] = a.B.nitem;
    nslot[0] = a.A.nslot;
    nslot[1] = a.B.nslot;
    rows_A = a.A.rows != 0;
    val[0] = a.A.val;
    val[1] = a.B.val;
    col[0] = a.A.col;
    col[1] = a.B.col;
    sigma = a.sigma;
    alpha = a.alpha;
    rho = a.rho;
    rho_inv = a.rho_inv;
    eps = a.eps;
    rel = a.rel;
  }
};

// --------------------------------------------------------------------------------- workgroup

extern __shared__ __align__(16) unsigned char small_lds[];

template <typename U>
__device__ __forceinline__ U* small_at(int off) {
  return reinterpret_cast<U*>(small_lds + off);
}
// The thread's index, opaque: the LDS addresses that a phase derives from it are then formed in the phase
// instead of being kept in registers over the whole kernel (where 1024 threads have 128 each).
__device__ __forceinline__ int small_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ int small_wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Segment sums of matrix I (0: Ā, 1: B) times the vector v in LDS, emit(slot, sum over the columns
// below nsplit, sum over the others) for each; PLANES 1: one sum. Eight steps of a lane are loaded together
// (at constant offsets: no address arithmetic per step), a chunk's last ones as 4, 2 and 1 (a serial
// remainder would pay a whole latency per step).
template <typename T, int I, bool ML, int PLANES, class E>
__device__ __forceinline__ void small_stream(const SmallCtx<T>& cx, const T* v, int nsplit, E emit) {
  const SmallChunk* chunks = small_at<const SmallChunk>(cx.o.chunk[I]);
  const uint16_t* segslot = small_at<const uint16_t>(cx.o.segslot[I]);
  const T* val = nullptr;
  const uint16_t* col = nullptr;
  if constexpr (ML) {
    val = small_at<const T>(cx.o.val[I]);
    col = small_at<const uint16_t>(cx.o.col[I]);
  } else {
    val = cx.val[I];
    col = cx.col[I];
  }
  const int lane = small_tid() & 63, nchunk = cx.nchunk[I];
  for (int ci = small_wave(); ci < nchunk; ci += (kSmallBlock<ML> / 64)) {
    const int base = __builtin_amdgcn_readfirstlane(chunks[ci].base);
    int left = __builtin_amdgcn_readfirstlane(chunks[ci].steps);
    const int slot = segslot[64 * ci + lane];
    const T* vp = val + base + lane;
    const uint16_t* cp = col + base + lane;
    T s1 = T(0), s2 = T(0);
    auto steps = [&](auto count) {
      constexpr int U = decltype(count)::value;
      T x[U], g[U];
      int c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        c[u] = cp[64 * u];
        x[u] = vp[64 * u];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) g[u] = v[c[u]];
#pragma unroll
      for (int u = 0; u < U; ++u) accumulate(x[u], g[u], PLANES == 1 || c[u] < nsplit, s1, s2);
      vp += 64 * U;
      cp += 64 * U;
    };
    for (; left >= 8; left -= 8) steps(std::integral_constant<int, 8>{});
    if (left & 4) steps(std::integral_constant<int, 4>{});
    if (left & 2) steps(std::integral_constant<int, 2>{});
    if (left & 1) steps(std::integral_constant<int, 1>{});
    if (slot != kSmallCols) emit(slot, s1, s2);
  }
}
// into the slots
template <typename T, int I, bool ML, int PLANES>
__device__ __forceinline__ void small_stream_slots(const SmallCtx<T>& cx, const T* v, int nsplit) {
  T* slots = small_at<T>(cx.o.slots);
  const int nslot = cx.nslot[I];
  small_stream<T, I, ML, PLANES>(cx, v, nsplit, [=](int slot, T s1, T s2) {
    slots[slot] = s1;
    if constexpr (PLANES == 2) slots[nslot + slot] = s2;
  });
}

// Wavefront partials of slot s, group b (a 256-thread workgroup of the general path), wavefront w
// of it: wp[(s·count + b)·4 + w], q = 4b + w.
template <int NS, unsigned MAXMASK>
__device__ __forceinline__ void small_put(double (&red)[NS], double* wp, int count, int q) {
  const double x = wave_reduce_slots<NS, MAXMASK>(red);
  const int lane = small_tid() & 63, s = lane / kSlotLanes<NS>;
  if (lane % kSlotLanes<NS> == 0 && s < NS) wp[4 * s * count + q] = x;
}

// k_combine's work, a wavefront for each quarter of an item.
template <typename T, int I, bool ML, int PLANES, class Op>
__device__ __forceinline__ void small_combine(const SmallCtx<T>& cx, const Op& op) {
  constexpr int NS = Op::NS > 0 ? Op::NS : 1;
  const int nitem = cx.nitem[I], nslot = cx.nslot[I];
  const SmallItem* items = small_at<const SmallItem>(cx.o.item[I]);
  const uint16_t* rowslot = small_at<const uint16_t>(cx.o.rowslot[I]);
  const T* slots = small_at<const T>(cx.o.slots);
  double* wp = small_at<double>(cx.o.wp);
  for (int q = small_wave(); q < 4 * nitem; q += (kSmallBlock<ML> / 64)) {
    const SmallItem c = items[q >> 2];
    const int lg = c.lg, L = 1 << lg;
    const int tid = (q & 3) * 64 + (small_tid() & 63), lane = tid & (L - 1);
    const int r = c.r0 + (tid >> lg);
    double red[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) red[s] = 0.0;
    if (r < c.r1) {
      T s1 = T(0), s2 = T(0);
      const int q1 = rowslot[r + 1];
#pragma unroll 4
      for (int k = rowslot[r] + lane; k < q1; k += L) {
        s1 += slots[k];
        if constexpr (PLANES == 2) s2 += slots[nslot + k];
      }
      if (L > 1) {
        s1 = wave_sum(s1, L);
        if constexpr (PLANES == 2) s2 = wave_sum(s2, L);
      }
      if (lane == 0) op.epilogue(r, s1, s2, red);
    }
    if constexpr (Op::NS > 0) small_put<Op::NS, Op::MAXMASK>(red, wp, nitem, q);
  }
}

// f(i, red) for the elements 0..rows−1; count groups of 256.
template <bool ML, int NS, unsigned MAXMASK, class F>
__device__ __forceinline__ void small_rows(int rows, int count, double* wp, F f) {
  for (int q = small_wave(); q < 4 * count; q += (kSmallBlock<ML> / 64)) {
    double red[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) red[s] = 0.0;
    const int i = q * 64 + (small_tid() & 63);
    if (i < rows) f(i, red);
    small_put<NS, MAXMASK>(red, wp, count, q);
  }
}

// Totals of at most 64 groups' partials, in every lane of every wavefront. reduce_partials and
// k_finalize fold them by one wavefront's tree too; their further wavefronts add zeros.
__device__ __forceinline__ double lane_value(double x, int lane) {
  int w[2];
  __builtin_memcpy(w, &x, 8);
  w[0] = __builtin_amdgcn_readlane(w[0], lane);
  w[1] = __builtin_amdgcn_readlane(w[1], lane);
  __builtin_memcpy(&x, w, 8);
  return x;
}
template <int NS, unsigned MAXMASK>
__device__ __forceinline__ void small_total(const double* wp, int count, double (&tot)[NS]) {
  const int b = small_tid() & 63;
  double v[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    v[s] = 0.0;
    if (b < count) {
      const double* p = wp + 4 * (s * count + b);
      v[s] = comb<MAXMASK>(s, 0.0, comb<MAXMASK>(s, comb<MAXMASK>(s, p[0], p[1]), comb<MAXMASK>(s, p[2], p[3])));
    }
  }
  const double x = wave_reduce_slots<NS, MAXMASK>(v);
#pragma unroll
  for (int s = 0; s < NS; ++s) tot[s] = comb<MAXMASK>(s, lane_value(x, s * kSlotLanes<NS>), 0.0);
}

template <typename T, bool ML, class Op>
__device__ __forceinline__ void small_pass_A(const SmallCtx<T>& cx, const T* v, const Op& op) {
  small_stream_slots<T, 0, ML, 1>(cx, v, 0);
  __syncthreads();
  small_combine<T, 0, ML, 1>(cx, op);
  __syncthreads();
}
template <typename T, bool ML, class Op>
__device__ __forceinline__ void small_pass_B(const SmallCtx<T>& cx, const T* v, const Op& op) {
  small_stream_slots<T, 1, ML, 2>(cx, v, cx.n);
  __syncthreads();
  small_combine<T, 1, ML, 2>(cx, op);
  __syncthreads();
}
// a check's scalar finalisation over `count` groups (k_finalize)
template <typename T, class Op>
__device__ __forceinline__ void small_finish(const SmallCtx<T>& cx, const Op& op, int count) {
  double t[Op::NS];
  small_total<Op::NS, Op::MAXMASK>(small_at<double>(cx.o.wp), count, t);
  if (threadIdx.x == 0) op((const double*)t);
  __syncthreads();
}

// The ADMM vectors, in LDS (AV) or in memory.
template <typename T>
struct SmallVecs {
  T *x, *y, *z, *g, *bk;
  const T *qb, *lb, *ub;
  double* ax;
};
template <typename T, bool AV>
__device__ __forceinline__ SmallVecs<T> small_vecs(const SmallCtx<T>& cx) {
  if constexpr (AV) {
    T* x = small_at<T>(cx.o.x);
    return {x, x + cx.n, small_at<T>(cx.o.z), small_at<T>(cx.o.g), small_at<T>(cx.o.bk), small_at<T>(cx.o.qb),
            small_at<T>(cx.o.lb), small_at<T>(cx.o.ub), small_at<double>(cx.o.ax)};
  } else {
    const SmallArgs<T>& a = small_now<T>();
    return {a.x, a.y, a.z, a.g, a.bk, a.qb, a.lb, a.ub, a.ax};
  }
}

template <typename T, bool AV, bool ML>
__device__ __forceinline__ void small_load(DevState* S, bool with_p) {
  const SmallArgs<T>& a = small_now<T>();
  constexpr unsigned kWords = offsetof(DevState, seq) / 8;
  if (threadIdx.x < kWords)
    reinterpret_cast<double*>(S)[threadIdx.x] = reinterpret_cast<const double*>(a.st)[threadIdx.x];
  auto put = [](auto* dst, const auto* src, int count) {
#pragma unroll (ML ? 8 : 2)
    for (int i = small_tid(); i < count; i += kSmallBlock<ML>) dst[i] = src[i];
  };
#pragma unroll 1
  for (int I = 0; I < 2; ++I) {
    const SmallMat<T>& M = I ? a.B : a.A;
    put(small_at<SmallChunk>(a.o.chunk[I]), M.chunks, M.nchunk);
    put(small_at<SmallItem>(a.o.item[I]), M.items, M.nitem);
    put(small_at<uint32_t>(a.o.segslot[I]), reinterpret_cast<const uint32_t*>(M.segslot), 32 * M.nchunk);
    put(small_at<uint16_t>(a.o.rowslot[I]), M.rowslot, M.nrows + 1);
    if constexpr (ML) {
      put(small_at<T>(a.o.val[I]), M.val, M.nval);
      put(small_at<uint32_t>(a.o.col[I]), reinterpret_cast<const uint32_t*>(M.col), M.nval / 2);
    }
  }
  // the vectors, those of one length together so that their loads overlap
  const int n = a.n, m = a.m;
  for (int i = small_tid(); i < n; i += kSmallBlock<ML>) {
    const T xt = a.xt[i], r = a.r[i], dinv = a.dinv[i], p = with_p ? a.p[i] : T(0);
    T x, g, bk, qb;
    if constexpr (AV) {
      x = a.x[i];
      g = a.g[i];
      bk = a.bk[i];
      qb = a.qb[i];
    }
    small_at<T>(a.o.xt)[i] = xt;
    small_at<T>(a.o.r)[i] = r;
    small_at<T>(a.o.dinv)[i] = dinv;
    if (with_p) small_at<T>(a.o.pw)[i] = p;
    if constexpr (AV) {
      small_at<T>(a.o.x)[i] = x;
      small_at<T>(a.o.g)[i] = g;
      small_at<T>(a.o.bk)[i] = bk;
      small_at<T>(a.o.qb)[i] = qb;
    }
  }
  for (int i = small_tid(); i < m; i += kSmallBlock<ML>) {
    const T zt = a.zt[i];
    T y, g, z, lb, ub;
    double ax;
    if constexpr (AV) {
      y = a.y[i];
      g = a.g[n + i];
      z = a.z[i];
      lb = a.lb[i];
      ub = a.ub[i];
      ax = a.ax[i];
    }
    small_at<T>(a.o.zt)[i] = zt;
    if constexpr (AV) {
      small_at<T>(a.o.x)[n + i] = y;
      small_at<T>(a.o.g)[n + i] = g;
      small_at<T>(a.o.z)[i] = z;
      small_at<T>(a.o.lb)[i] = lb;
      small_at<T>(a.o.ub)[i] = ub;
      small_at<double>(a.o.ax)[i] = ax;
    }
  }
  __syncthreads();
}

template <typename T, bool AV, bool ML>
__device__ __forceinline__ void small_store(const DevState* S) {
  __syncthreads();
  const SmallArgs<T>& a = small_now<T>();
  auto put = [](auto* dst, const auto* src, int count) {
    for (int i = small_tid(); i < count; i += kSmallBlock<ML>) dst[i] = src[i];
  };
  put(a.xt, small_at<T>(a.o.xt), a.n);
  put(a.r, small_at<T>(a.o.r), a.n);
  put(a.p, small_at<T>(a.o.pw), a.n);
  put(a.zt, small_at<T>(a.o.zt), a.m);
  if constexpr (AV) {
    put(a.x, small_at<T>(a.o.x), a.n + a.m);
    put(a.z, small_at<T>(a.o.z), a.m);
    put(a.g, small_at<T>(a.o.g), a.n + a.m);
    put(a.bk, small_at<T>(a.o.bk), a.n);
    put(a.ax, small_at<double>(a.o.ax), a.m);
  }
  // the scalars, for the general path's kernels and for the host
  constexpr unsigned kWords = offsetof(DevState, seq) / 8;
  if (threadIdx.x < kWords)
    reinterpret_cast<double*>(a.st)[threadIdx.x] = reinterpret_cast<const double*>(S)[threadIdx.x];
  if (a.hr.to) copy_state(S, a.hr);
}

// v (count entries) as the vector that the next pass gathers: itself if it is in LDS, or a copy there
template <typename T, bool IN_LDS, bool ML>
__device__ __forceinline__ const T* small_stage(const SmallCtx<T>& cx, const T* v, int count) {
  if constexpr (IN_LDS) return v;
  T* pw = small_at<T>(cx.o.pw);
  for (int i = small_tid(); i < count; i += kSmallBlock<ML>) pw[i] = v[i];
  __syncthreads();
  return pw;
}

// The scalars of a PCG solve, the same in every thread (DevState's of the same names).
struct SmallPcg {
  double rz, rz_prev, alpha, beta, kappa, bnorm, rnorm, thresh;
  int it, done, bad;
  int bound;  // iterations left for this launch
  __device__ __forceinline__ void get(const DevState& S) {
    it = S.iter;
    rz = S.rzp[it & 1];
    rz_prev = S.rzp[(it + 1) & 1];
    alpha = S.alpha;
    beta = S.beta;
    kappa = S.kappa;
    bnorm = S.bnorm;
    rnorm = S.rnorm;
    thresh = S.thresh;
    done = S.done;
    bad = S.breakdown;
    bound = kSmallPcg;
  }
  __device__ __forceinline__ void put(DevState& S, int maxit) const {  // one thread
    S.rzp[it & 1] = rz;
    S.rzp[(it + 1) & 1] = rz_prev;
    S.alpha = alpha;
    S.beta = beta;
    S.kappa = kappa;
    S.bnorm = bnorm;
    S.rnorm = rnorm;
    S.thresh = thresh;
    S.iter = it;
    S.done = done;
    S.breakdown = bad;
    S.maxit = maxit;
  }
  // the start of a solve from r⁰ᵀM⁻¹r⁰ and ‖r⁰‖∞ (rhs_scalars, OpR0)
  __device__ __forceinline__ void start(double rz0, double rnorm0, int maxit) {
    rz = rz0;
    rnorm = rnorm0;
    it = 0;
    bad = rz0 != rz0 ? 1 : 0;
    done = (rnorm0 <= thresh || bad || maxit <= 0) ? 1 : 0;
  }
};

// PCG iterations (pcg_iteration of the general path) until done or this launch's bound. p is in pw.
template <typename T, bool ML, bool TRACK>
__device__ __forceinline__ void small_pcg_run(const SmallCtx<T>& cx, SmallPcg& c) {
  const int n = cx.n, m = cx.m, maxit = cx.maxit, vgrid = cx.vgrid;
  const bool rows_A = cx.rows_A;
  const T rho = cx.rho, rho_inv = cx.rho_inv, sigma = cx.sigma;
  T *pw = small_at<T>(cx.o.pw), *w = pw + n, *xt = small_at<T>(cx.o.xt), *r = small_at<T>(cx.o.r);
  T *kp = small_at<T>(cx.o.kp), *dinv = small_at<T>(cx.o.dinv), *zt = small_at<T>(cx.o.zt);
  T* slots = small_at<T>(cx.o.slots);
  double *wp = small_at<double>(cx.o.wp), *wq = small_at<double>(cx.o.wq);
#pragma unroll 1
  while (!c.done && c.bound > 0) {
    const OpScaled<T> sa{pw, w, rho};
    small_stream<T, 0, ML, 1>(cx, pw, 0, [&](int slot, T s1, T s2) {
      if (rows_A)
        sa.epilogue(slot, T(0) + s1, s2, nullptr);
      else
        slots[slot] = s1;
    });
    __syncthreads();
    if (!rows_A) {
      small_combine<T, 0, ML, 1>(cx, sa);
      __syncthreads();
    }
    small_pass_B<T, ML>(cx, pw, OpKp<T>{pw, w, kp, sigma, n, nullptr});
    double kap[1];
    small_total<1, 0u>(wp, cx.nitem[1], kap);
    c.kappa = kap[0];
    c.alpha = c.kappa > 0.0 ? c.rz / c.kappa : 0.0;
    if (!(c.kappa > 0.0) && !(c.kappa == 0.0 && c.rnorm == 0.0)) c.bad = 1;
    const T al = (T)c.alpha;
    small_rows<ML, 2, 2u>(n, vgrid, wq, [&](int i, double (&red)[2]) { pcg_update_at(i, al, xt, r, pw, kp, dinv, red); });
    if constexpr (TRACK)
      for (int i = small_tid(); i < m; i += kSmallBlock<ML>) pcg_track_at(i, al, zt, w, rho_inv);
    __syncthreads();
    double t[2];
    small_total<2, 2u>(wq, vgrid, t);
    c.rz_prev = c.rz;
    c.rz = t[0];
    c.beta = c.rz / c.rz_prev;
    c.rnorm = t[1];
    const T be = (T)c.beta;
    for (int i = small_tid(); i < n; i += kSmallBlock<ML>) pcg_dir_at(i, be, pw, r, dinv);
    ++c.it;
    --c.bound;
    if (c.rz != c.rz) c.bad = 1;
    c.done = (c.rnorm <= c.thresh || c.it >= maxit || c.bad || !(c.kappa > 0.0)) ? 1 : 0;
    __syncthreads();
  }
}

// The epilogues of the right-hand side's B passes (the direct one's two, the recurrence's one): one copy
// of the pass serves all three.
template <typename T>
struct SmallRhsOp {
  static constexpr int NS = OpRhsRec<T>::NS;
  static constexpr unsigned MAXMASK = OpRhsRec<T>::MAXMASK;
  OpRhsRec<T> rec;
  OpRhsR0<T> r0;
  int kind;  // 0: OpRhsAt, 1: OpRhsR0, 2: OpRhsRec
  __device__ void epilogue(int i, T s1, T s2, double* red) const {
    if (kind == 2)
      rec.epilogue(i, s1, s2, red);
    else if (kind == 1)
      r0.epilogue(i, s1, s2, red);
    else
      rec.bk[i] = s2;
  }
};

// Right-hand side, ‖b‖∞, threshold and the warm-started residual of one ADMM iteration.
template <typename T, bool AV, bool ML>
__device__ __forceinline__ void small_rhs(const SmallCtx<T>& cx, SmallPcg& c, int mode, T gamma, T ratio) {
  const SmallVecs<T> v = small_vecs<T, AV>(cx);
  const int n = cx.n, m = cx.m;
  T *pw = small_at<T>(cx.o.pw), *xt = small_at<T>(cx.o.xt), *r = small_at<T>(cx.o.r), *dinv = small_at<T>(cx.o.dinv);
  SmallRhsOp<T> op{{v.x, xt, v.qb, v.g, dinv, r, pw, v.bk, cx.sigma, gamma, cx.maxit, cx.rel, cx.eps, nullptr},
                   {v.x, xt, v.qb, v.g, dinv, r, pw, v.bk, cx.sigma, cx.maxit, cx.rel, cx.eps, nullptr},
                   mode == kRhsDirect ? 0 : 2};
  double* wp = small_at<double>(cx.o.wp);
  double t[3];
  if (mode == kRhsDirect || mode == kRhsRec) {
    if (mode == kRhsDirect) {
      const T* zt = small_at<T>(cx.o.zt);
      T* g = small_now<T>().g;
      for (int i = small_tid(); i < n + m; i += kSmallBlock<ML>) {
        pairs_at(i, n, m, g, (const T*)xt, zt, (const T*)v.z, (const T*)v.y, cx.rho, (const uint8_t*)nullptr);
        if constexpr (AV) v.g[i] = g[i];
        pw[i] = g[(size_t)n + m + i];
      }
      __syncthreads();
    }
#pragma unroll 1
    for (; op.kind <= 2; ++op.kind) {
      const T* g = op.kind == 0 ? pw : AV ? v.g : small_stage<T, AV, ML>(cx, v.g, n + m);
      small_pass_B<T, ML>(cx, g, op);
      if (op.kind == 1) break;
    }
    small_total<3, 5u>(wp, cx.nitem[1], t);
  } else {
    const SmallArgs<T>& a = small_now<T>();
    const T *b1 = a.bg, *b2 = a.bg + n, *aty = a.bg + 2 * (size_t)n;
    small_rows<ML, 3, 5u>(n, cx.vgrid, wp, [&](int i, double (&red)[3]) {
      const T u2 = b2[i];
      op.rec.epilogue(i, b1[i], mode == kRhsRows ? u2 : rhs_rescale(u2, aty[i], ratio), red);
    });
    __syncthreads();
    small_total<3, 5u>(wp, cx.vgrid, t);
  }
  c.bnorm = t[0];
  c.thresh = cx.rel ? cx.eps * t[0] : cx.eps;
  c.start(t[1], t[2], cx.maxit);
}

template <typename T, bool AV, bool CHECK>
__device__ __forceinline__ OpUpdate<T, CHECK> small_update_op(const SmallCtx<T>& cx, DevState* S, const double* einv,
                                                                 T* zt_out, T* dxy) {
  const SmallVecs<T> v = small_vecs<T, AV>(cx);
  return OpUpdate<T, CHECK>{small_at<T>(cx.o.xt), v.x, v.z, v.y, zt_out, v.ax, v.g, v.lb, v.ub, einv,
                            cx.alpha, cx.rho, cx.rho_inv, cx.n, S, dxy, nullptr};
}

// The ADMM update.
template <typename T, bool AV, bool ML>
__device__ __forceinline__ void small_update(const SmallCtx<T>& cx) {
  const T* zt = small_at<T>(cx.o.zt);
  const OpUpdate<T, false> op = small_update_op<T, AV, false>(cx, nullptr, nullptr, nullptr, nullptr);
  for (int i = small_tid(); i < cx.m; i += kSmallBlock<ML>) op.epilogue(i, zt[i], T(0), nullptr);
  op.side();
  __syncthreads();
}

// The Ā passes of a check (the update with z̃ recomputed, the primal residual with Āx̄ recomputed) and
// its B passes (the dual residual, the next B·g), one copy of the pass for both of each.
template <typename T>
struct SmallCheckA {
  static constexpr int NS = 6;
  static constexpr unsigned MAXMASK = 0x3Fu;
  OpUpdate<T, true> up;
  OpRPrim<T> rp;
  bool update;
  __device__ void epilogue(int i, T s1, T s2, double* red) const {
    if (update)
      up.epilogue(i, s1, s2, red);
    else
      rp.epilogue(i, s1, s2, red);
  }
};
template <typename T>
struct SmallCheckB {
  static constexpr int NS = OpRDual<T>::NS;
  static constexpr unsigned MAXMASK = OpRDual<T>::MAXMASK;
  OpRDual<T> rd;
  T* bg;  // null: not formed
  bool dual;
  __device__ void epilogue(int i, T s1, T s2, double* red) const {
    if (dual) {
      rd.epilogue(i, s1, s2, red);
      if (bg) bg[2 * (size_t)rd.n + i] = s2;
    } else {
      bg[i] = s1;
      bg[rd.n + i] = s2;
    }
  }
};

// The update of a check iteration that took `it` PCG steps, and its residual norms.
template <typename T, bool AV, bool ML>
__device__ __forceinline__ bool small_check(const SmallCtx<T>& cx, DevState* S, int k, int it) {
  __syncthreads();  // the right-hand side's partials have been read
  const SmallArgs<T>& a = small_now<T>();
  const SmallVecs<T> v = small_vecs<T, AV>(cx);
  const int n = cx.n, m = cx.m, ugrid = a.ugrid;
  {
    T *zt = small_at<T>(cx.o.zt), *xt = small_at<T>(cx.o.xt);
    const int last = it > a.exact_after ? 0 : 1;
    const bool reset = a.zt_every > 0 && (k / a.check_every) % a.zt_every == 0;
    SmallCheckA<T> op{small_update_op<T, AV, true>(cx, S, a.escale, reset ? zt : nullptr, a.dxy),
                      {v.x, v.z, a.escale, S}, reset};
    if (!op.update) {
      small_rows<ML, 6, 0x3Fu>(m, ugrid, small_at<double>(cx.o.wp),
                           [&](int i, double (&red)[6]) { op.up.epilogue(i, zt[i], T(0), red); });
      op.up.side();
      __syncthreads();
      small_finish<T>(cx, op.up, ugrid);
    }
#pragma unroll 1
    for (int pass = op.update ? 1 : 0; pass >= last; --pass) {  // 1: update, 0: Āx̄ recomputed
      op.update = pass == 1;
      small_pass_A<T, ML>(cx, op.update ? xt : small_stage<T, AV, ML>(cx, v.x, n), op);
      if (op.update) {
        op.up.side();
        __syncthreads();
      }
      small_finish<T>(cx, op.up, cx.nitem[0]);
    }
  }
  const bool pair = a.pair && k < a.max_iter && it <= a.pair_after;
  SmallCheckB<T> op{{v.x, v.y, v.qb, a.dscale, n, S}, pair ? a.bg : nullptr, true};
#pragma unroll 1
  for (int pass = 0; pass < (pair ? 2 : 1); ++pass) {
    op.dual = pass == 0;
    small_pass_B<T, ML>(cx, small_stage<T, AV, ML>(cx, pass ? v.g : v.x, n + m), op);
    if (op.dual) small_finish<T>(cx, op.rd, cx.nitem[1]);
  }
  return pair;
}

// std::max and std::min, also for NaN
__device__ __forceinline__ double dmax(double a, double b) { return a < b ? b : a; }
__device__ __forceinline__ double dmin(double a, double b) { return b < a ? b : a; }

// The ADMM loop's state, the same in every thread (qpg_solver::admm's variables of these names).
struct SmallRun {
  double rho, rho_b, bg_rho, eps, best;
  int since, checks, updates, bg_for;
};

// The host's decisions after the check of iteration k (qpg_solver::admm), in its arithmetic (no
// contraction; division and square root are correctly rounded on both sides), by every thread. False
// when the check is the host's: the solve may end, or the residuals have not improved lately. True:
// ρ̄, the tolerance and the counters are those of the next iteration.
template <typename T>
__device__ __forceinline__ bool small_decide(const DevState* S, SmallRun& run, int k) {
#pragma clang fp contract(off)
  const SmallArgs<T>& a = small_now<T>();
  const double* nm = S->norms;
  if (!a.decide || a.dxy || k >= a.max_iter) return false;
  const double prim = nm[1], dual = nm[7] / a.c, nPx = nm[9] / a.c, nAty = nm[11] / a.c;
  const double eps_p = a.eps_abs + a.eps_rel * dmax(nm[3], nm[5]);
  const double eps_d = a.eps_abs + a.eps_rel * dmax(dmax(nPx, nAty), a.q_norm);
  if (!(prim == prim) || !(dual == dual) || (prim <= eps_p && dual <= eps_d)) return false;
  const double ratio = dmax(prim / dmax(eps_p, 1e-300), dual / dmax(eps_d, 1e-300));
  if (ratio < 0.99 * run.best) {
    run.best = ratio;
    run.since = 0;
  } else if (run.since + 1 >= a.stall) {
    return false;
  } else {
    ++run.since;
  }
  ++run.checks;
  if (!a.fixed_eps) {
    double eps = a.lambda * sqrt(nm[0] * nm[6]);
    if (a.rel) eps = dmin(eps, a.lambda);
    run.eps = dmax(eps * a.tighten, a.eps_min);
  }
  if (a.rho_every > 0 && k % a.rho_every == 0) {
    const double num = nm[0] / dmax(dmax(nm[2], nm[4]), 1e-10);
    const double den = nm[6] / dmax(dmax(dmax(nm[8], nm[10]), a.qb_norm), 1e-10);
    if (den > 0 && num > 0) {
      const double est = dmin(dmax(run.rho * sqrt(num / den), 1e-6), 1e6);
      if ((est >= a.gate * run.rho || est <= run.rho / a.gate) && est != run.rho) {
        run.rho = est;
        ++run.updates;
      }
    }
  }
  return true;
}

// g, and the Jacobi diagonal (unless it is the learned one), for a new ρ̄
template <typename T, bool AV, bool ML>
__device__ __forceinline__ void small_new_rho(const SmallCtx<T>& cx, double rho, bool jacobi) {
  const SmallArgs<T>& a = small_now<T>();
  const SmallVecs<T> v = small_vecs<T, AV>(cx);
  const int n = cx.n, m = cx.m;
  const T *xt = small_at<T>(cx.o.xt), *zt = small_at<T>(cx.o.zt);
  T* dinv = small_at<T>(cx.o.dinv);
  if (jacobi)
    for (int i = small_tid(); i < n; i += kSmallBlock<ML>)
      a.dinv[i] = dinv[i] = jacobi_at<T>(i, a.diagP, a.colsq, a.sigma64, rho, nullptr);
  for (int i = small_tid(); i < n + m; i += kSmallBlock<ML>) {
    pairs_at(i, n, m, a.g, xt, zt, (const T*)v.z, (const T*)v.y, cx.rho, (const uint8_t*)nullptr);
    if constexpr (AV) v.g[i] = a.g[i];
  }
  __syncthreads();
}

// ADMM iterations k0.. up to k1 or a check that is the host's, with the loop's state in S.run. An
// iteration whose PCG solve breaks down, hits the cap or is cut at this launch's bound ends the launch
// before its update, with the abort fields as k_after_pcg sets them.
template <typename T, bool AV, bool ML>
__global__ __launch_bounds__(kSmallBlock<ML>) void k_small_admm(SmallArgs<T>) {
  __shared__ DevState S;
  small_load<T, AV, ML>(&S, false);
  SmallCtx<T> cx;
  cx.get();
  const SmallArgs<T>& a = small_now<T>();
  const int k1 = a.k1, refresh = a.refresh, every = a.check_every, max_iter = a.max_iter;
  int k = a.k0, mode = a.first_rhs, at_check = 0;
  T gamma = a.gamma, ratio = a.ratio;
  SmallRun run{a.rho64, a.rho_b, a.bg_rho, a.eps, a.best, a.since, 0, 0, a.bg_for};
  if (a.new_rho) small_new_rho<T, AV, ML>(cx, run.rho, a.new_rho == 2);
  SmallPcg c;
  c.get(S);
  int sum = S.pcg_sum, most = S.pcg_max, reason = 0;
#pragma unroll 1
  for (;;) {
    small_rhs<T, AV, ML>(cx, c, mode, gamma, ratio);
    run.rho_b = run.rho;
    mode = (k + 1) % refresh == 0 ? kRhsDirect : kRhsRec;
    gamma = T(1);
    small_pcg_run<T, ML, true>(cx, c);
    // as after_pcg
    reason = c.bad ? 2 : !c.done ? 1 : (c.it >= cx.maxit && c.rnorm > c.thresh) ? 3 : 0;
    if (reason) break;
    sum += c.it;
    most = max(most, c.it);
    if (k % every == 0 || k == max_iter) {
      if (small_check<T, AV, ML>(cx, &S, k, c.it)) {
        run.bg_for = k + 1;
        run.bg_rho = run.rho;
      }
      if (!small_decide<T>(&S, run, k)) {
        at_check = 1;
        break;
      }
      cx.eps = run.eps;
      if (run.bg_for == k + 1 && mode == kRhsRec) mode = run.rho == run.bg_rho ? kRhsRows : kRhsRescaled;
      if (run.rho != run.rho_b) {
        cx.rho = (T)run.rho;
        cx.rho_inv = (T)(1.0 / run.rho);
        gamma = (T)(run.rho / run.rho_b);
        ratio = (T)(run.rho / run.bg_rho);
        small_new_rho<T, AV, ML>(cx, run.rho, true);
      }
    } else {
      small_update<T, AV, ML>(cx);
    }
    if (k == k1) break;
    ++k;
  }
  if (threadIdx.x == 0) {
    if (reason) {
      S.abort = 1;
      S.abort_k = k;
      S.abort_reason = reason;
      c.done = 1;
    }
    c.put(S, cx.maxit);
    S.pcg_sum = sum;
    S.pcg_max = most;
    S.run.rho = run.rho;
    S.run.rho_b = run.rho_b;
    S.run.bg_rho = run.bg_rho;
    S.run.eps = run.eps;
    S.run.best = run.best;
    S.run.k = k;
    S.run.since = run.since;
    S.run.checks = run.checks;
    S.run.updates = run.updates;
    S.run.at_check = at_check;
    S.run.bg_for = run.bg_for;
  }
  small_store<T, AV, ML>(&S);
}

// Algorithm 3 from x̃ with the right-hand side in b and the threshold in the device scalars (resume 0),
// or its continuation (resume 1), for at most kSmallPcg iterations.
template <typename T, bool ML>
__global__ __launch_bounds__(kSmallBlock<ML>) void k_small_pcg(SmallArgs<T>) {
  __shared__ DevState S;
  const bool resume = small_now<T>().resume != 0;
  small_load<T, false, ML>(&S, resume);
  SmallCtx<T> cx;
  cx.get();
  SmallPcg c;
  c.get(S);
  if (!resume) {
    const int n = cx.n;
    T *pw = small_at<T>(cx.o.pw), *w = pw + n, *xt = small_at<T>(cx.o.xt);
    for (int i = small_tid(); i < n; i += kSmallBlock<ML>) pw[i] = xt[i];
    small_pass_A<T, ML>(cx, xt, OpScaled<T>{xt, w, cx.rho});
    const OpR0<T> op{xt, w, small_now<T>().b, small_at<T>(cx.o.dinv), small_at<T>(cx.o.r), pw, cx.sigma, n,
                     cx.maxit, nullptr};
    small_pass_B<T, ML>(cx, pw, op);
    double t[2];
    small_total<2, 2u>(small_at<double>(cx.o.wp), cx.nitem[1], t);
    c.start(t[0], t[1], cx.maxit);
  }
  small_pcg_run<T, ML, false>(cx, c);
  if (threadIdx.x == 0) c.put(S, cx.maxit);
  small_store<T, false, ML>(&S);
}

}  // namespace qpg
