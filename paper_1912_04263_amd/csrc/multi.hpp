// Jacobi PCG on several right-hand sides at once (the Hutchinson probes). Included by learned.hip only.
//
// One solve's step reads Ā and B once and its six kernels are bound by latency at training sizes
// (1.6·10⁶ entries: 37 µs per step for 26 MB of matrix); kMulti solves that take their steps together
// read the matrices once for all and share the launches (52 µs for four steps). Vectors are interleaved: element i of
// solve v is at i·kMulti + v, so a gather takes one 32-byte piece for all solves. Each solve's numbers are
// those of the single solve, bit for bit: every lane, slot, group and tree adds the same values in the
// same order, only for kMulti vectors side by side; a solve that has ended keeps its x.
#pragma once

#include "kernels.hpp"

namespace qpg {

constexpr int kMulti = 4;  // 2·kMulti reduction slots at most (kMaxSlots)
static_assert(2 * kMulti <= kMaxSlots, "slots");

// Scalars of the kMulti solves (DevState's of the same names).
struct MultiState {
  double rzp[2][kMulti];
  double kappa[kMulti], rnorm[kMulti], thresh[kMulti];
  int32_t iter[kMulti], done[kMulti], breakdown[kMulti];
  int32_t all_done;
  int32_t maxit;
};

struct alignas(16) MultiVec {
  double v[kMulti];
};

// Segment sums of a work list times an interleaved vector (k_spmv for kMulti vectors). The window is
// staged in LDS when it fits there for all vectors (`staged`), otherwise gathered from memory.
// Bound by latency: windows of 32 bytes per column leave room for few workgroups, so these have 512
// threads and at most 64 VGPRs (2 steps unrolled). 1.6·10⁶ entries: the estimate below in 33.1 ms; with
// 1024 threads 33.9, and with 4 steps unrolled and 102 VGPRs 34.5 (512 threads) and 36.4 ms (1024).
constexpr int kMultiBlock = 512;
__global__ __launch_bounds__(kMultiBlock, 8) void k_multi_spmv(const Tile* __restrict__ tiles,
                                                       const Chunk* __restrict__ chunks,
                                                       const int32_t* __restrict__ segslot,
                                                       const uint16_t* __restrict__ col16,
                                                       const int32_t* __restrict__ col32,
                                                       const double* __restrict__ val, int nsplit,
                                                       const MultiVec* __restrict__ x,
                                                       MultiVec* __restrict__ slots, int64_t pstride, int planes,
                                                       int staged, const MultiState* __restrict__ st) {
  if (st->all_done) return;
  extern __shared__ __align__(16) unsigned char smem[];
  MultiVec* win = reinterpret_cast<MultiVec*>(smem);
  const Tile t = tiles[blockIdx.x];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (t.wlen > 0 && staged) {
#pragma unroll 4
    for (int i = threadIdx.x; i < t.wlen; i += kMultiBlock) win[i] = x[t.wlo + i];
    __syncthreads();
  }
  // a window on one side of nsplit has one sum per lane (the other stays 0): half the arithmetic
  const int lim = nsplit - t.wlo;
  const int side = planes == 1 || (t.wlen > 0 && lim >= t.wlen) ? 0 : (t.wlen > 0 && lim <= 0) ? 1 : 2;
  for (int ci = t.chunk0 + wave; ci < t.chunk0 + t.nchunk; ci += kMultiBlock / 64) {
    const Chunk ch = chunks[ci];
    const int slot = segslot[ch.seg0 + lane];
    const double* vp = val + ch.base + lane;
    MultiVec s1{}, s2{};
    // get reads LDS or memory: one walk for each, so that neither becomes a flat load
    auto walk = [&](auto both, auto get, const auto* cp, int split) {
#pragma unroll 2
      for (int s = 0; s < ch.steps; ++s) {
        const int c = cp[64 * s];
        const double a = vp[64 * s];
        const MultiVec g = get(c);
        const bool first = !decltype(both)::value || c < split;
#pragma unroll
        for (int v = 0; v < kMulti; ++v) accumulate(a, g.v[v], first, s1.v[v], s2.v[v]);
      }
    };
    auto go = [&](auto both) {
      if (t.wlen == 0)
        walk(both, [&](int c) { return x[c]; }, col32 + ch.cbase + lane, nsplit);
      else if (staged)
        walk(both, [&](int c) { return win[c]; }, col16 + ch.cbase + lane, lim);
      else
        walk(both, [&](int c) { return x[t.wlo + c]; }, col16 + ch.cbase + lane, lim);
    };
    if (side == 2)
      go(std::true_type{});
    else
      go(std::false_type{});
    if (slot >= 0) {
      MultiVec o1, o2;
#pragma unroll
      for (int v = 0; v < kMulti; ++v) {
        o1.v[v] = side == 1 ? s2.v[v] : s1.v[v];
        o2.v[v] = side == 1 ? s1.v[v] : s2.v[v];
      }
      slots[slot] = o1;
      if (planes > 1) slots[pstride + slot] = o2;
    }
  }
}

// The epilogues of k_multi_combine: w = ρ̄Āx; Kp and pᵀKp; r = Kx − b, p = −M⁻¹r, rᵀM⁻¹r, ‖r‖∞ (OpScaled,
// OpKp, OpR0). Reduction slots: one per solve (sums), then one per solve (∞-norms).
struct MultiScaled {
  static constexpr int NS = 0;
  static constexpr unsigned MAXMASK = 0;
  MultiVec* out;
  double scale;
  __device__ void epilogue(int r, const MultiVec& s1, const MultiVec& s2, double*) const {
    MultiVec o;
#pragma unroll
    for (int v = 0; v < kMulti; ++v) o.v[v] = scale * (s1.v[v] + s2.v[v]);
    out[r] = o;
  }
};
struct MultiKp {
  static constexpr int NS = kMulti;
  static constexpr unsigned MAXMASK = 0;
  const MultiVec* p;
  MultiVec* kp;
  double sigma;
  __device__ void epilogue(int i, const MultiVec& s1, const MultiVec& s2, double* red) const {
    const MultiVec pi = p[i];
    MultiVec o;
#pragma unroll
    for (int v = 0; v < kMulti; ++v) {
      const double k = s1.v[v] + s2.v[v] + sigma * pi.v[v];
      o.v[v] = k;
      red[v] += pi.v[v] * k;
    }
    kp[i] = o;
  }
};
struct MultiR0 {
  static constexpr int NS = 2 * kMulti;
  static constexpr unsigned MAXMASK = ((1u << kMulti) - 1u) << kMulti;
  const MultiVec* x;
  const int8_t* z;  // probes, n each
  const double* dinv;
  MultiVec *r, *p;
  double sigma;
  int n;
  MultiState* st;
  int maxit;
  __device__ void epilogue(int i, const MultiVec& s1, const MultiVec& s2, double* red) const {
    const MultiVec xi = x[i];
    const double d = dinv[i];
    MultiVec ro, po;
#pragma unroll
    for (int v = 0; v < kMulti; ++v) {
      const double ri = (s1.v[v] + s2.v[v] + sigma * xi.v[v]) - (double)z[(size_t)v * n + i];
      const double yi = ri * d;
      ro.v[v] = ri;
      po.v[v] = -yi;
      red[v] += ri * yi;
      red[kMulti + v] = nmax(red[kMulti + v], fabs(ri));
    }
    r[i] = ro;
    p[i] = po;
  }
  __device__ void operator()(const double* t) const {
    int all = 1;
    for (int v = 0; v < kMulti; ++v) {
      st->rzp[0][v] = t[v];
      st->rnorm[v] = t[kMulti + v];
      st->iter[v] = 0;
      st->breakdown[v] = t[v] != t[v] ? 1 : 0;
      st->done[v] = (st->rnorm[v] <= st->thresh[v] || st->breakdown[v] || maxit <= 0) ? 1 : 0;
      all &= st->done[v];
    }
    st->maxit = maxit;
    st->all_done = all;
  }
};

template <class Op>
__global__ __launch_bounds__(kBlock) void k_multi_combine(const CombItem* __restrict__ items,
                                                          const int32_t* __restrict__ rowslot,
                                                          const int32_t* __restrict__ slotidx,
                                                          const int32_t* __restrict__ tbase,
                                                          const MultiVec* __restrict__ slots, int64_t pstride,
                                                          int planes, Op op, double* __restrict__ partials,
                                                          const MultiState* __restrict__ st) {
  if (st->all_done) return;
  constexpr int NS = Op::NS > 0 ? Op::NS : 1;
  double red[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) red[s] = 0.0;
  const CombItem c = items[blockIdx.x];
  auto add = [&](MultiVec& s, const MultiVec& x) {
#pragma unroll
    for (int v = 0; v < kMulti; ++v) s.v[v] += x.v[v];
  };
  if (c.lg < 0) {
    const int r = c.r0 + threadIdx.x;
    if (r < c.r1) {
      MultiVec s1{}, s2{};
      const int32_t* tb = tbase + c.t0;
      constexpr int U = 4;
      for (int j = 0; j < -c.lg; j += U) {
        MultiVec x1[U], x2[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t q = (int64_t)tb[j + u < -c.lg ? j + u : j] + r;
          x1[u] = slots[q];
          if (planes > 1) x2[u] = slots[pstride + q];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (j + u < -c.lg) {
            add(s1, x1[u]);
            if (planes > 1) add(s2, x2[u]);
          }
      }
      op.epilogue(r, s1, s2, red);
    }
  } else {
    const int lg = c.lg, L = 1 << lg, groups = kBlock >> lg;
    const int g = threadIdx.x >> lg, lane = threadIdx.x & (L - 1);
    for (int r = c.r0 + g; r < c.r1; r += groups) {
      MultiVec s1{}, s2{};
      const int q1 = rowslot[r + 1];
#pragma unroll 2
      for (int q = rowslot[r] + lane; q < q1; q += L) {
        const int sq = slotidx[q];
        add(s1, slots[sq]);
        if (planes > 1) add(s2, slots[pstride + sq]);
      }
      if (L > 1) {
#pragma unroll
        for (int v = 0; v < kMulti; ++v) {
          s1.v[v] = wave_sum(s1.v[v], L);
          if (planes > 1) s2.v[v] = wave_sum(s2.v[v], L);
        }
      }
      if (lane == 0) op.epilogue(r, s1, s2, red);
    }
  }
  if constexpr (Op::NS > 0) publish<Op::NS, Op::MAXMASK>(red, partials);
}

// k_pcg_update for kMulti solves: those that have ended keep x and r.
__global__ __launch_bounds__(kBlock) void k_multi_update(int n, MultiVec* __restrict__ x, MultiVec* __restrict__ r,
                                                         const MultiVec* __restrict__ p,
                                                         const MultiVec* __restrict__ kp,
                                                         const double* __restrict__ dinv, MultiState* st,
                                                         const double* __restrict__ kp_partials, int kp_count,
                                                         double* __restrict__ partials, int it) {
  if (st->all_done) return;
  double kap[kMulti];
  reduce_partials<kMulti, 0u>(kp_partials, kp_count, kap);
  double alpha[kMulti];
  bool on[kMulti];
#pragma unroll
  for (int v = 0; v < kMulti; ++v) {
    on[v] = !st->done[v];
    alpha[v] = kap[v] > 0.0 ? st->rzp[it & 1][v] / kap[v] : 0.0;
    if (on[v] && blockIdx.x == 0 && threadIdx.x == 0) {
      st->kappa[v] = kap[v];
      if (!(kap[v] > 0.0) && !(kap[v] == 0.0 && st->rnorm[v] == 0.0)) st->breakdown[v] = 1;
    }
  }
  double red[2 * kMulti];
#pragma unroll
  for (int s = 0; s < 2 * kMulti; ++s) red[s] = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    MultiVec xi = x[i], ri = r[i];
    const MultiVec pi = p[i], ki = kp[i];
    const double d = dinv[i];
#pragma unroll
    for (int v = 0; v < kMulti; ++v) {
      double one[2] = {red[v], red[kMulti + v]};
      double xv = xi.v[v], rv = ri.v[v];
      pcg_update_at(0, alpha[v], &xv, &rv, &pi.v[v], &ki.v[v], &d, one);
      if (on[v]) {
        xi.v[v] = xv;
        ri.v[v] = rv;
      }
      red[v] = one[0];
      red[kMulti + v] = one[1];
    }
    x[i] = xi;
    r[i] = ri;
  }
  publish<2 * kMulti, MultiR0::MAXMASK>(red, partials);
}

// k_pcg_dir for kMulti solves. Workgroup 0 stores the scalars; the others read only the previous
// parity's rᵀM⁻¹r and, of the flags, all_done as it was when they started: a workgroup that already sees a
// solve ended skips its share of that p, which is not used any more.
__global__ __launch_bounds__(kBlock) void k_multi_dir(int n, MultiVec* __restrict__ p, const MultiVec* __restrict__ r,
                                                      const double* __restrict__ dinv, MultiState* st,
                                                      const double* __restrict__ partials, int count, int it) {
  if (st->all_done) return;
  double t[2 * kMulti];
  reduce_partials<2 * kMulti, MultiR0::MAXMASK>(partials, count, t);
  double beta[kMulti];
#pragma unroll
  for (int v = 0; v < kMulti; ++v) beta[v] = t[v] / st->rzp[it & 1][v];
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    MultiVec pi = p[i];
    const MultiVec ri = r[i];
    const double d = dinv[i];
#pragma unroll
    for (int v = 0; v < kMulti; ++v) pcg_dir_at(0, beta[v], &pi.v[v], &ri.v[v], &d);
    p[i] = pi;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    int all = 1;
    for (int v = 0; v < kMulti; ++v) {
      if (!st->done[v]) {
        st->rzp[(it + 1) & 1][v] = t[v];
        st->rnorm[v] = t[kMulti + v];
        st->iter[v] = it + 1;
        if (t[v] != t[v]) st->breakdown[v] = 1;
        st->done[v] = (t[kMulti + v] <= st->thresh[v] || it + 1 >= st->maxit || st->breakdown[v] ||
                       !(st->kappa[v] > 0.0))
                          ? 1
                          : 0;
      }
      all &= st->done[v];
    }
    st->all_done = all;
  }
}

// Start of a batch: x = 0 (also as the gathered vector of the first residual), the thresholds ε‖z‖∞ with
// ‖z‖∞ = 1, and zeros for the probes that the batch does not have (their solves end at once).
__global__ __launch_bounds__(kBlock) void k_multi_start(int n, int count, MultiVec* __restrict__ x,
                                                        MultiVec* __restrict__ p, int8_t* __restrict__ z,
                                                        MultiState* st, double eps) {
  const MultiVec zero{};
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    x[i] = zero;
    p[i] = zero;
    for (int v = count; v < kMulti; ++v) z[(size_t)v * n + i] = 0;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->all_done = 0;
    for (int v = 0; v < kMulti; ++v) st->thresh[v] = eps;
  }
}

// acc += z ∘ x of the batch's `count` solves, in their order
__global__ __launch_bounds__(kBlock) void k_multi_acc(int n, int count, const int8_t* __restrict__ z,
                                                      const MultiVec* __restrict__ x, double* __restrict__ acc) {
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const MultiVec xi = x[i];
    double a = acc[i];
    for (int v = 0; v < count; ++v) a += (double)z[(size_t)v * n + i] * xi.v[v];
    acc[i] = a;
  }
}

// The batch's progress for the host (mapped memory): whether all solves have ended, the largest iteration
// count, then the read's number.
struct MultiRead {
  int32_t all_done, iter;
  uint32_t seq, pad_;
};
__global__ void k_multi_read(const MultiState* st, MultiRead* host, uint32_t seq) {
  if (threadIdx.x != 0) return;
  int it = 0;
  for (int v = 0; v < kMulti; ++v) it = max(it, st->iter[v]);
  host->all_done = st->all_done;
  host->iter = it;
  __hip_atomic_store(&host->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace qpg
