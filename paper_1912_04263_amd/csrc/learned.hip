// Learned diagonal preconditioner: graph construction, network forward/backward, training
// objects, Hutchinson targets and the learned M⁻¹ used by the solve.
//
// The preconditioner stays diagonal and strictly positive (M⁻¹_ii = softplus(g_i)/K_ii), so the
// PCG of Algorithm 3 is unchanged; only the Jacobi diagonal of Section 6.3.1 is replaced. The
// message-passing trunk does not depend on ρ̄ and runs once per setup; the head is re-evaluated
// when ρ̄ changes (Section 6.3.2 updates ρ̄ every 10 iterations).
#include <mutex>

#include "mpnn.hpp"
#include "multi.hpp"
#include "solver_internal.hpp"

using namespace qpg;

struct qpg_net {
  int device = 0;
  int bf16 = 1;
  float* theta = nullptr;  // float32 master parameters (device)
  float* grad = nullptr;
  float* m1 = nullptr;
  float* m2 = nullptr;
  int step = 0;
  std::string err;
  ~qpg_net() {
    for (float* p : {theta, grad, m1, m2})
      if (p) (void)hipFree(p);
  }
};

namespace qpg {

struct LearnedState {
  DeviceArena arena;
  int n = 0, m = 0;
  float *fv = nullptr, *fc = nullptr;
  float *wA_hat = nullptr, *wA_chk = nullptr;  // on the Ā structure
  float *wB_hat = nullptr, *wB_chk = nullptr;  // on the B structure (Āᵀ part)
  float* hv[kRounds + 1] = {};
  float* hc[kRounds + 1] = {};
  float* av[kRounds + 1] = {};
  float* ac[kRounds + 1] = {};
  float *phi = nullptr, *u = nullptr, *g = nullptr, *dg = nullptr, *tgt = nullptr;
  double* e = nullptr;
  float *dhv = nullptr, *dhv2 = nullptr, *dav = nullptr, *dhc = nullptr, *dhc2 = nullptr,
        *dac = nullptr, *dU = nullptr;
  // work lists over the rows of Ā and over the Āᵀ parts of B's rows
  struct List {
    Piece* pieces = nullptr;
    int32_t* rows = nullptr;
    int32_t npieces = 0, packs = 0, nrows = 0, one_chain = 0;
  } list_a, list_b;
  float* part = nullptr;
  int part_groups = 0;
  NetScalars* ns = nullptr;
  NetScalars* ns_host = nullptr;
  double* acc = nullptr;    // Hutchinson accumulator (n)
  int8_t* probe = nullptr;  // one probe (n), or kMulti of them
  // kMulti solves at once (multi.hpp): vectors of up to kMultiKeep bytes stay from their first use on, larger
  // ones go at the end of the call that made them
  static constexpr size_t kMultiKeep = size_t(64) << 20;
  void* mlarge = nullptr;
  MultiVec *mx = nullptr, *mr = nullptr, *mp = nullptr, *mkp = nullptr, *mslots = nullptr;
  MultiState* mst = nullptr;
  MultiRead* mread = nullptr;  // mapped host memory
  MultiRead* mread_dev = nullptr;
  uint32_t mreads = 0;
  // inference network of the solve (settings.precond == QPG_PRECOND_LEARNED)
  float* theta_inf = nullptr;
  bool trunk_ready = false;

  template <typename T>
  T* alloc(size_t count) {
    return static_cast<T*>(arena.get(count * sizeof(T), "hipMalloc (learned preconditioner)"));
  }
  void end_multi() {
    if (!mlarge) return;
    (void)hipFree(mlarge);
    mlarge = nullptr;
    mst = nullptr;
  }
  ~LearnedState() { end_multi(); }
};

void destroy_learned(LearnedState* L) {
  if (!L) return;
  if (L->ns_host) (void)hipHostFree(L->ns_host);
  if (L->mread) (void)hipHostFree(L->mread);
  delete L;
}

}  // namespace qpg

namespace {

int div_up(long a, long b) { return (int)((a + b - 1) / b); }

// Weight gradients: rows per workgroup at least, and workgroups at most (their partials are then added
// by k_part_reduce). With 1024 rows a layer over the 20,200 variables of a training portfolio ran on 20
// of the 256 compute units and took 62 µs; with 96 it takes 8.8, and the sum of the 211 partials 3.9.
constexpr int kGradRows = 96;
constexpr int kGradGroups = 512;

// The graph data of the scaled problem: row statistics of Ā and Āᵀ, normalised
// edge weights on both CSR structures, node features; and the activations.
void build_graph(qpg_solver* h, LearnedState* L) {
  const int n = h->n, m = h->m;
  L->n = n;
  L->m = m;
  hipStream_t st = h->stream;
  const int nnzA = std::max(1, h->nnzA), nnzB = std::max(1, h->nnzB);
  // work lists from the row pointers
  {
    std::vector<int32_t> ap((size_t)m + 1), bp((size_t)n + 1), bs(n);
    auto fetch = [&](std::vector<int32_t>& v, const int32_t* d) {
      if (!v.empty())
        HIPCHK(hipMemcpyAsync(v.data(), d, v.size() * sizeof(int32_t), hipMemcpyDeviceToHost, st));
    };
    fetch(ap, h->a_ptr);
    fetch(bp, h->b_ptr);
    fetch(bs, h->b_split);
    HIPCHK(hipStreamSynchronize(st));
    auto put = [&](LearnedState::List& l, const PiecePlan& p) {
      l.npieces = (int32_t)p.pieces.size();
      l.packs = p.packs;
      l.nrows = (int32_t)p.rows.size();
      l.one_chain = p.one_chain;
      l.pieces = L->alloc<Piece>(p.pieces.size());
      l.rows = L->alloc<int32_t>(p.rows.size());
      if (l.npieces) h->copy_h2d(l.pieces, p.pieces.data(), p.pieces.size() * sizeof(Piece));
      if (l.nrows) h->copy_h2d(l.rows, p.rows.data(), p.rows.size() * sizeof(int32_t));
      HIPCHK(hipStreamSynchronize(st));  // p goes out of scope
    };
    put(L->list_a, make_pieces(ap.data(), ap.data() + 1, ap.data(), m));
    put(L->list_b, make_pieces(bs.data(), bp.data() + 1, bp.data(), n));
  }
  double *rsA = L->alloc<double>(m), *mxA = L->alloc<double>(m), *sqA = L->alloc<double>(m);
  double *rsB = L->alloc<double>(n), *mxB = L->alloc<double>(n), *sqB = L->alloc<double>(n);
  int32_t *dgA = L->alloc<int32_t>(m), *dgB = L->alloc<int32_t>(n);
  auto stats = [&](const LearnedState::List& l, int rows, const int32_t* ptr, const int32_t* start, const double* val,
                   double* rs, double* mx, double* sq, int32_t* dg) {
    if (rows == 0) return;
    if (l.packs)
      hipLaunchKernelGGL(k_rowstats, dim3(div_up(l.packs, kBlock / 64)), dim3(kBlock), 0, st, (const Piece*)l.pieces,
                         l.packs, ptr, start, val, rs, mx, sq);
    if (l.nrows)
      hipLaunchKernelGGL(k_rowstats_rows, dim3(l.nrows), dim3(64), 0, st, (const int32_t*)l.rows, ptr, start, val, rs,
                         mx, sq);
    hipLaunchKernelGGL(k_degrees, dim3(div_up(rows, kBlock)), dim3(kBlock), 0, st, rows, ptr, start, dg);
  };
  stats(L->list_a, m, h->a_ptr, nullptr, h->p64.a_val, rsA, mxA, sqA, dgA);
  stats(L->list_b, n, h->b_ptr, h->b_split, h->p64.b_val, rsB, mxB, sqB, dgB);
  L->wA_hat = L->alloc<float>(nnzA);
  L->wA_chk = L->alloc<float>(nnzA);
  L->wB_hat = L->alloc<float>(nnzB);
  L->wB_chk = L->alloc<float>(nnzB);
  auto weights = [&](const LearnedState::List& l, const int32_t* ptr, const int32_t* start, const int32_t* col,
                     const double* val, int coff, const double* rowsum, const double* colsum, float* w_row,
                     float* w_col) {
    if (l.npieces)
      hipLaunchKernelGGL(k_edge_weights, dim3(div_up(l.npieces, kBlock / 64)), dim3(kBlock), 0, st,
                         (const Piece*)l.pieces, l.npieces, ptr, start, col, val, coff, rowsum, colsum, w_row, w_col);
  };
  weights(L->list_a, h->a_ptr, nullptr, h->a_col, h->p64.a_val, 0, rsA, rsB, L->wA_hat, L->wA_chk);
  weights(L->list_b, h->b_ptr, h->b_split, h->b_col, h->p64.b_val, n, rsB, rsA, L->wB_chk, L->wB_hat);
  L->fv = L->alloc<float>((size_t)n * kH);
  L->fc = L->alloc<float>((size_t)m * kH);
  hipLaunchKernelGGL(k_features_v, dim3(div_up((long)n * kH, kBlock)), dim3(kBlock), 0, st, n,
                     (const double*)h->diagP, (const double*)h->colsq, (const int32_t*)dgB,
                     (const double*)mxB, h->s.sigma, L->fv);
  if (m > 0)
    hipLaunchKernelGGL((k_features_c<double>), dim3(div_up((long)m * kH, kBlock)), dim3(kBlock), 0, st, m,
                       (const double*)sqA, (const int32_t*)dgA, (const double*)mxA,
                       (const double*)h->p64.lb, (const double*)h->p64.ub, L->fc);
  for (int l = 0; l <= kRounds; ++l) {
    L->hv[l] = L->alloc<float>((size_t)n * kH);
    L->hc[l] = L->alloc<float>((size_t)m * kH);
    if (l > 0) {
      L->av[l] = L->alloc<float>((size_t)n * kH);
      L->ac[l] = L->alloc<float>((size_t)m * kH);
    }
  }
  L->phi = L->alloc<float>((size_t)n * kH);
  L->u = L->alloc<float>((size_t)n * kH);
  L->dU = L->alloc<float>((size_t)n * kH);
  L->g = L->alloc<float>(n);
  L->e = L->alloc<double>(n);
  L->dg = L->alloc<float>(n);
  L->tgt = L->alloc<float>(n);
  L->dhv = L->alloc<float>((size_t)n * kH);
  L->dhv2 = L->alloc<float>((size_t)n * kH);
  L->dav = L->alloc<float>((size_t)n * kH);
  L->dhc = L->alloc<float>((size_t)m * kH);
  L->dhc2 = L->alloc<float>((size_t)m * kH);
  L->dac = L->alloc<float>((size_t)m * kH);
  L->part_groups = std::max(1, std::min(kGradGroups, div_up(std::max(n, m), kGradRows)));
  L->part = L->alloc<float>((size_t)L->part_groups * (64 * kH + kH));
  L->ns = L->alloc<NetScalars>(1);
  HIPCHK(hipHostMalloc((void**)&L->ns_host, sizeof(NetScalars), hipHostMallocDefault));
  L->acc = L->alloc<double>(n);
  L->probe = L->alloc<int8_t>((size_t)kMulti * n);
  HIPCHK(hipGetLastError());
}

LearnedState* ensure_graph(qpg_solver* h) {
  return build_once(h->learned, [h](LearnedState* L) { build_graph(h, L); },
                    [h](LearnedState* L) {
                      (void)hipStreamSynchronize(h->stream);  // kernels on its arrays
                      destroy_learned(L);
                    });
}

void dense_fwd(qpg_solver* h, bool bf16, int N, const float* X1, const float* X2, const float* W,
               const float* b, float* Y) {
  if (N <= 0) return;
  if (bf16)
    hipLaunchKernelGGL(k_dense_fwd_mfma, dim3(div_up(N, 128)), dim3(kBlock), 0, h->stream, N, X1, X2, W, b, Y);
  else
    hipLaunchKernelGGL(k_dense_fwd_f32, dim3(div_up((long)N * kH, kBlock)), dim3(kBlock), 0, h->stream, N,
                       X1, X2, W, b, Y);
}

// Gradients of Y = relu([X1 X2] W + b): [W; b] written to gWb (K·32 + 32 floats, the parameter
// layout), dX1 (= or +=) and dX2 (=) when non-null.
void dense_bwd(qpg_solver* h, LearnedState* L, bool bf16, int N, const float* X1, const float* X2,
               const float* dY, const float* Y, const float* W, float* dX1, float* dX2, int acc,
               float* gWb) {
  const int K = X2 ? 64 : 32;
  const int width = K * kH + kH;
  if (N <= 0) {
    HIPCHK(hipMemsetAsync(gWb, 0, width * sizeof(float), h->stream));
    return;
  }
  const int G = std::max(1, std::min(L->part_groups, div_up(N, kGradRows)));
  if (bf16)
    hipLaunchKernelGGL(k_dense_bwd_dw_mfma, dim3(G), dim3(kBlock), 0, h->stream, N, X1, X2, dY, Y, L->part);
  else
    hipLaunchKernelGGL(k_dense_bwd_dw_f32, dim3(G), dim3(kBlock), 0, h->stream, N, X1, X2, dY, Y, L->part);
  hipLaunchKernelGGL(k_part_reduce, dim3(div_up(width, 32)), dim3(kBlock), 0, h->stream,
                     (const float*)L->part, G, width, gWb);
  if (dX1) {
    if (bf16)
      hipLaunchKernelGGL(k_dense_bwd_dx_mfma, dim3(div_up(N, 128)), dim3(kBlock), 0, h->stream, N, dY, Y, W,
                         dX1, dX2, acc);
    else
      hipLaunchKernelGGL(k_dense_bwd_dx_f32, dim3(div_up((long)N * kH, kBlock)), dim3(kBlock), 0, h->stream,
                         N, dY, Y, W, dX1, dX2, acc);
  }
}

// Y (=|+=) Â X etc.: the SpMM over the Ā structure (m rows, gather from n×32) or over the Āᵀ
// part of B (n rows, gather from m×32).
void spmm(qpg_solver* h, const LearnedState::List& l, const int32_t* ptr, const int32_t* start, const int32_t* col,
          const float* w, int coff, const float* X, float* Y, int acc) {
  if (l.packs)
    hipLaunchKernelGGL(k_spmm32, dim3(div_up(l.packs, kBlock / 64)), dim3(kBlock), 0, h->stream,
                       (const Piece*)l.pieces, l.packs, ptr, start, col, w, coff, X, Y, acc);
  if (l.one_chain)
    hipLaunchKernelGGL((k_spmm_rows<1, 32>), dim3(l.one_chain), dim3(kSpmmBlock), 0, h->stream,
                       (const int32_t*)l.rows, ptr, start, col, w, coff, X, Y, acc);
  if (l.nrows > l.one_chain)
    hipLaunchKernelGGL((k_spmm_rows<8, 16>), dim3((l.nrows - l.one_chain) * (kH / 16)), dim3(kSpmmBlock), 0, h->stream,
                       (const int32_t*)l.rows + l.one_chain, ptr, start, col, w, coff, X, Y, acc);
}
void spmm_A(qpg_solver* h, const float* w, const float* X, float* Y, int acc) {
  spmm(h, h->learned->list_a, h->a_ptr, nullptr, h->a_col, w, 0, X, Y, acc);
}
void spmm_B(qpg_solver* h, const float* w, const float* X, float* Y, int acc) {
  spmm(h, h->learned->list_b, h->b_ptr, h->b_split, h->b_col, w, h->n, X, Y, acc);
}

// Message-passing trunk: h_v^L in L->hv[kRounds].
void trunk(qpg_solver* h, LearnedState* L, const float* th, bool bf16) {
  const int n = h->n, m = h->m;
  dense_fwd(h, bf16, n, L->fv, nullptr, th + NetOff::W_v0, th + NetOff::b_v0, L->hv[0]);
  dense_fwd(h, bf16, m, L->fc, nullptr, th + NetOff::W_c0, th + NetOff::b_c0, L->hc[0]);
  for (int l = 1; l <= kRounds; ++l) {
    if (m > 0) spmm_A(h, L->wA_hat, L->hv[l - 1], L->ac[l], 0);
    dense_fwd(h, bf16, m, L->hc[l - 1], L->ac[l], th + NetOff::W_c(l), th + NetOff::b_c(l), L->hc[l]);
    spmm_B(h, L->wB_chk, L->hc[l], L->av[l], 0);
    dense_fwd(h, bf16, n, L->hv[l - 1], L->av[l], th + NetOff::W_v(l), th + NetOff::b_v(l), L->hv[l]);
  }
}

// Head for a given ρ̄: u, g; and, if dinv is given, M⁻¹ = softplus(g) / K_ii in precision T.
template <typename T>
void head(qpg_solver* h, LearnedState* L, const float* th, bool bf16, double rho, T* dinv) {
  const int n = h->n;
  hipLaunchKernelGGL(k_phi, dim3(div_up((long)n * kH, kBlock)), dim3(kBlock), 0, h->stream, n,
                     (const double*)h->diagP, (const double*)h->colsq, h->s.sigma, rho, L->phi);
  dense_fwd(h, bf16, n, L->hv[kRounds], L->phi, th + NetOff::W_h1, th + NetOff::b_h1, L->u);
  hipLaunchKernelGGL((k_head_out<T>), dim3(div_up(n, kBlock)), dim3(kBlock), 0, h->stream, n,
                     (const float*)L->u, th, L->g, dinv, (const double*)h->diagP,
                     (const double*)h->colsq, h->s.sigma, rho);
}

// Loss (mean-removed squared error of log s − target; queued into ns_host) and its gradient into `grad`.
void loss_backward(qpg_solver* h, LearnedState* L, const float* th, bool bf16, float* grad) {
  const int n = h->n, m = h->m;
  const int vg = h->vgrid;
  hipLaunchKernelGGL(k_loss_mean, dim3(vg), dim3(kBlock), 0, h->stream, n, (const float*)L->g,
                     (const float*)L->tgt, L->e, h->rb.partials);
  h->finalize_fn<1, 0u>(FinMeanE{L->ns, n}, vg);
  hipLaunchKernelGGL(k_loss_grad, dim3(vg), dim3(kBlock), 0, h->stream, n, (const double*)L->e,
                     (const float*)L->g, (const NetScalars*)L->ns, L->dg, h->rb.partials);
  h->finalize_fn<1, 0u>(FinLoss{L->ns, n}, vg);
  // head output layer
  const int G = std::max(1, std::min(L->part_groups, div_up(n, kGradRows)));
  hipLaunchKernelGGL(k_head_out_bwd, dim3(G), dim3(kBlock), 0, h->stream, n, (const float*)L->u,
                     (const float*)L->dg, th, L->dU, L->part);
  hipLaunchKernelGGL(k_part_reduce, dim3(div_up(kH + 1, 32)), dim3(kBlock), 0, h->stream, (const float*)L->part, G, kH + 1,
                     grad + NetOff::w_h2);
  // head hidden layer: input [h_v^L, φ]; only the h_v^L part of the input gradient is needed
  dense_bwd(h, L, bf16, n, L->hv[kRounds], L->phi, L->dU, L->u, th + NetOff::W_h1, L->dhv, nullptr, 0,
            grad + NetOff::W_h1);
  float *dhv = L->dhv, *dhv2 = L->dhv2, *dhc = L->dhc, *dhc2 = L->dhc2;
  for (int l = kRounds; l >= 1; --l) {
    // h_v^l = relu([h_v^{l−1}, a_v] W_vl + b_vl)
    dense_bwd(h, L, bf16, n, L->hv[l - 1], L->av[l], dhv, L->hv[l], th + NetOff::W_v(l), dhv2, L->dav, 0,
              grad + NetOff::W_v(l));
    // a_v = Ǎ h_c^l  ⇒  dh_c^l += Ǎᵀ da_v   (Ǎᵀ lives on the Ā structure)
    if (m > 0) spmm_A(h, L->wA_chk, L->dav, dhc, l < kRounds);  // dh_c^L has no other term
    // h_c^l = relu([h_c^{l−1}, a_c] W_cl + b_cl)
    dense_bwd(h, L, bf16, m, L->hc[l - 1], L->ac[l], dhc, L->hc[l], th + NetOff::W_c(l), dhc2, L->dac, 0,
              grad + NetOff::W_c(l));
    // a_c = Â h_v^{l−1}  ⇒  dh_v^{l−1} += Âᵀ da_c   (Âᵀ lives on the Āᵀ part of B)
    spmm_B(h, L->wB_hat, L->dac, dhv2, 1);
    std::swap(dhv, dhv2);
    std::swap(dhc, dhc2);
  }
  dense_bwd(h, L, bf16, n, L->fv, nullptr, dhv, L->hv[0], th + NetOff::W_v0, nullptr, nullptr, 0,
            grad + NetOff::W_v0);
  dense_bwd(h, L, bf16, m, L->fc, nullptr, dhc, L->hc[0], th + NetOff::W_c0, nullptr, nullptr, 0,
            grad + NetOff::W_c0);
  HIPCHK(hipMemcpyAsync(L->ns_host, L->ns, sizeof(NetScalars), hipMemcpyDeviceToHost, h->stream));
}

// Host-side parameter initialisation: uniform(±1/√fan_in) weights from a splitmix64 stream,
// zero biases, output layer at softplus = 1 (the Jacobi preconditioner).
void init_params(std::vector<float>& p, uint64_t seed) {
  p.assign(NetOff::total, 0.f);
  uint64_t x = seed;
  auto next = [&]() {
    x += 0x9E3779B97F4A7C15ull;
    uint64_t z = x;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (double)(z >> 11) * (1.0 / 9007199254740992.0);
  };
  auto fill = [&](int off, int fan_in, int count) {
    const double a = 1.0 / std::sqrt((double)fan_in);
    for (int i = 0; i < count; ++i) p[off + i] = (float)((2.0 * next() - 1.0) * a);
  };
  fill(NetOff::W_v0, 32, 32 * kH);
  fill(NetOff::W_c0, 32, 32 * kH);
  for (int l = 1; l <= kRounds; ++l) {
    fill(NetOff::W_c(l), 64, 64 * kH);
    fill(NetOff::W_v(l), 64, 64 * kH);
  }
  fill(NetOff::W_h1, 64, 64 * kH);
  p[NetOff::b_h2] = (float)std::log(std::exp(1.0) - 1.0);
}

int net_error(qpg_net* net, const HipError& e) {
  char buf[512];
  std::snprintf(buf, sizeof(buf), "%s failed: %s", e.what, hipGetErrorString(e.code));
  if (net) net->err = buf;
  (void)hipGetLastError();
  return e.code == hipErrorOutOfMemory ? QPG_ERR_OOM : QPG_ERR_DEVICE;
}

}  // namespace

// ------------------------------------------------------------------- learned M⁻¹ in the solve

// Prepare the inference network of the solve: graph, weights, trunk (once per setup).
void qpg_solver::learned_prepare() {
  LearnedState* L = ensure_graph(this);
  if (!L->theta_inf) {
    L->theta_inf = L->alloc<float>(NetOff::total);
    HIPCHK(hipMemcpyAsync(L->theta_inf, precond_weights.data(), NetOff::total * sizeof(float),
                          hipMemcpyHostToDevice, stream));
  }
  if (!L->trunk_ready) {
    trunk(this, L, L->theta_inf, true);
    L->trunk_ready = true;
  }
}

template <typename T>
void qpg_solver::learned_dinv(double rho) {
  learned_prepare();
  head<T>(this, learned, learned->theta_inf, true, rho, P<T>().dinv);
}
template void qpg_solver::learned_dinv<double>(double);
template void qpg_solver::learned_dinv<float>(double);

// ------------------------------------------------------------ Hutchinson targets

namespace {

// Scratch of qpg_hutchinson_noalloc: the accumulator Σ_k z_k ∘ K⁻¹z_k (n doubles, then padding
// to 256 bytes) followed by one probe (n bytes). Every device the library runs on holds one copy
// for the life of the process; calls that overlap on one device share it and race.
__device__ __align__(256) unsigned char scratch[QPG_NOALLOC_SCRATCH_BYTES];

constexpr int kScratchDevices = 64;
std::atomic<void*> g_scratch_addr[kScratchDevices];  // device address of `scratch`, per ordinal
std::mutex g_scratch_mu;

void* noalloc_scratch(int device) {
  if (device < 0 || device >= kScratchDevices) return nullptr;
  return g_scratch_addr[device].load(std::memory_order_acquire);
}

int hutchinson_check(qpg_solver* h, const int8_t* signs, int32_t nprobes, double rho, double eps,
                     int32_t max_iter, double* diag) {
  if (!h || !signs || nprobes < 1 || !diag || !(rho > 0) || !(eps >= 0) || max_iter < 1)
    return QPG_ERR_ARG;
  if (h->s.rho_vector) {
    h->err = "qpg_hutchinson: defined for R = rho*I (the handle was set up with rho_vector)";
    return QPG_ERR_STATE;
  }
  for (long k = 0; k < (long)nprobes * h->n; ++k)
    if (signs[k] != 1 && signs[k] != -1) {
      h->err = "qpg_hutchinson: probe entries must be +1 or -1";
      return QPG_ERR_ARG;
    }
  return QPG_OK;
}

// The vectors of kMulti solves, where they are not there. False when the device has no room for them: the probes
// are then solved one by one.
bool ensure_multi(qpg_solver* h, LearnedState* L) {
  if (L->mst) return true;
  const size_t n = h->n, m = h->m;
  const size_t nslot = (size_t)std::max<int64_t>(h->plan_a.nslot, 2 * h->plan_b.nslot);
  if (!L->mread) {
    HIPCHK(hipHostMalloc((void**)&L->mread, sizeof(MultiRead), hipHostMallocMapped));
    std::memset(L->mread, 0, sizeof(MultiRead));
  }
  HIPCHK(hipHostGetDevicePointer((void**)&L->mread_dev, L->mread, 0));
  void* p = nullptr;
  const size_t bytes = (4 * n + m + nslot) * sizeof(MultiVec) + sizeof(MultiState);
  const hipError_t e = hipMalloc(&p, bytes);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    return false;
  }
  HIPCHK(e);
  if (bytes <= LearnedState::kMultiKeep)
    L->arena.adopt(p, bytes);
  else
    L->mlarge = p;
  L->mx = (MultiVec*)p;
  L->mr = L->mx + n;
  L->mkp = L->mr + n;
  L->mp = L->mkp + n;
  L->mslots = L->mp + n + m;
  L->mst = (MultiState*)(L->mslots + nslot);
  return true;
}

// One pass of a work list over kMulti vectors; returns the workgroups of the combine.
template <class Op>
int multi_pass(qpg_solver* h, LearnedState* L, const DevPlan& pl, int nsplit, int planes, const MultiVec* x,
               const Op& op) {
  const size_t want = (size_t)pl.max_wlen * sizeof(MultiVec);
  const int staged = want <= (size_t)h->lds_max;
  const size_t lds = staged ? want : 0;
  static LdsLimit limit;
  allow_lds(limit, reinterpret_cast<const void*>(&k_multi_spmv), lds, h->device);
  hipLaunchKernelGGL(k_multi_spmv, dim3(pl.ntiles), dim3(kMultiBlock), lds, h->stream, (const Tile*)pl.tiles,
                     (const Chunk*)pl.chunks, (const int32_t*)pl.segslot, (const uint16_t*)pl.col16,
                     (const int32_t*)pl.col32, (const double*)pl.val64, nsplit, x, L->mslots, pl.nslot, planes, staged,
                     (const MultiState*)L->mst);
  hipLaunchKernelGGL((k_multi_combine<Op>), dim3(pl.ncomb), dim3(kBlock), 0, h->stream, (const CombItem*)pl.comb,
                     (const int32_t*)pl.rowslot, (const int32_t*)pl.slotidx, (const int32_t*)pl.tbase,
                     (const MultiVec*)L->mslots, pl.nslot, planes, op, h->rb.partials, (const MultiState*)L->mst);
  return pl.ncomb;
}

// `count` ≤ kMulti probes of hutchinson_run in one solve: bitwise the same numbers. `predicted`: PCG steps that the
// last such solve of the call took. Measured on the 20,000-asset portfolio (16 probes, about 162 PCG steps each): 97 ms
// one by one, 33 ms four at a time.
void solve_together(qpg_solver* h, LearnedState* L, const int8_t* signs, int count, double rho, double eps,
                    int32_t max_iter, double* acc, int& predicted) {
  Prec<double>& V = h->p64;
  const int n = h->n;
  MultiVec* w = L->mp + n;
  const dim3 vg(h->vgrid), vb(kBlock);
  HIPCHK(hipMemcpyAsync(L->probe, signs, (size_t)count * n, hipMemcpyHostToDevice, h->stream));
  hipLaunchKernelGGL(k_multi_start, vg, vb, 0, h->stream, n, count, L->mx, L->mp, L->probe, L->mst, eps);
  multi_pass(h, L, h->plan_a, INT32_MAX, 1, L->mx, MultiScaled{w, rho});
  const MultiR0 r0{L->mx, L->probe, V.dinv, L->mr, L->mp, h->s.sigma, n, L->mst, max_iter};
  h->finalize(r0, multi_pass(h, L, h->plan_b, n, 2, L->mp, r0));
  // iterations between host reads: first as many as the call's last four solves took, then 2, 4, 8, 8, …
  int issued = 0, batch = predicted, more = 1;
  for (;;) {
    const int b = std::min(batch, max_iter - issued);
    for (int i = 0; i < b; ++i) {
      const int it = issued + i;
      multi_pass(h, L, h->plan_a, INT32_MAX, 1, L->mp, MultiScaled{w, rho});
      const int nkp = multi_pass(h, L, h->plan_b, n, 2, L->mp, MultiKp{L->mp, L->mkp, h->s.sigma});
      hipLaunchKernelGGL(k_multi_update, vg, vb, 0, h->stream, n, L->mx, L->mr, (const MultiVec*)L->mp,
                         (const MultiVec*)L->mkp, (const double*)V.dinv, L->mst, (const double*)h->rb.partials, nkp,
                         h->rb.vpartials, it);
      hipLaunchKernelGGL(k_multi_dir, vg, vb, 0, h->stream, n, L->mp, (const MultiVec*)L->mr,
                         (const double*)V.dinv, L->mst, (const double*)h->rb.vpartials, h->vgrid, it);
    }
    issued += b;
    hipLaunchKernelGGL(k_multi_read, dim3(1), dim3(64), 0, h->stream, (const MultiState*)L->mst, L->mread_dev,
                       ++L->mreads);
    h->spin(&L->mread->seq, L->mreads);
    if (L->mread->all_done || issued >= max_iter) break;
    batch = more = std::min(2 * more, 8);
  }
  predicted = std::max(1, L->mread->iter);
  hipLaunchKernelGGL(k_multi_acc, vg, vb, 0, h->stream, n, count, (const int8_t*)L->probe, (const MultiVec*)L->mx,
                     acc);
}

// The fewest probes that are worth solving together. Four solves at a time cost this many times one alone: 1.4–2.0
// where its latencies bound it (up to 80 MB of matrices in windows of at most 2048 columns, 128 MB without windows),
// 2.2–2.9 beyond, and 2.6–4.9 where a window of 32 bytes per column does not fit in LDS, so that every gather
// goes to the caches: there it pays for four, with matrices (256 MB) and vectors (10 MB) in them. 40 steps of
// two / three / four probes, one by one → together: SVM with 2·10⁶ entries 3.0 / 4.5 / 5.9 → 2.5 / 2.6 / 2.6 ms,
// random with 2·10⁷ and no windows 23.4 / 35.0 / 46.7 → 28.4 / 28.6 / 28.9, Lasso with 10⁷ 6.2 / 9.1 / 12.1
// → 10.7 / 11.1 / 11.4, SVM with 10⁸ 44 / 66 / 88 → 105 / 108 / 111.
int together_from(const qpg_solver* h) {
  if (h->use_small<double>()) return INT32_MAX;
  const int64_t mats = ((int64_t)h->nnzA + h->nnzB) * (int64_t)(sizeof(double) + sizeof(uint16_t));
  const int64_t vecs = ((int64_t)h->n + h->m) * (int64_t)sizeof(MultiVec);
  const int wlen = std::max(h->plan_a.max_wlen, h->plan_b.max_wlen);
  if ((int64_t)wlen * (int64_t)sizeof(MultiVec) > h->lds_max)
    return mats <= qpg_solver::kStreamAll && vecs <= 10000000 ? kMulti : INT32_MAX;
  return vecs <= 20000000 && wlen <= 2048 && mats <= (wlen ? 80000000 : 128000000) ? 2 : 3;
}

// (1/s) Σ_k z_k ∘ K⁻¹z_k with K⁻¹z_k by the solver's Jacobi PCG from 0; acc (n doubles) and probe
// (n bytes) are device buffers the caller provides. ρ̄ and the Jacobi diagonal are restored. With L, groups of at
// least `from` probes are solved together.
int hutchinson_run(qpg_solver* h, const int8_t* signs, int32_t nprobes, double rho, double eps,
                   int32_t max_iter, double* diag, double* acc, int8_t* probe, LearnedState* L = nullptr,
                   int from = INT32_MAX) {
  Prec<double>& V = h->p64;
  const int n = h->n;
  const double rho_saved = h->rho_cur;
  struct Restore {  // ρ̄ of the handle is restored on every way out
    qpg_solver* h;
    double rho;
    ~Restore() { h->rho_cur = rho; }
  } restore{h, rho_saved};
  h->rho_cur = rho;
  h->jacobi<double>(rho);
  h->fill(acc, n, 0.0);
  int predicted = 1;  // nothing is carried over from an earlier call
  for (int k = 0; k < nprobes;) {
    const int8_t* z = signs + (size_t)k * n;
    const int count = std::min<int>(kMulti, nprobes - k);
    if (L && count >= from) {
      solve_together(h, L, z, count, rho, eps, max_iter, acc, predicted);
      k += count;
      continue;
    }
    HIPCHK(hipMemcpyAsync(probe, z, n, hipMemcpyHostToDevice, h->stream));
    hipLaunchKernelGGL((k_probe_load<double>), dim3(h->vgrid), dim3(kBlock), 0, h->stream, n,
                       (const int8_t*)probe, V.b);
    h->fill(V.xt, n, 0.0);
    hipLaunchKernelGGL((k_absmax<double>), dim3(h->vgrid), dim3(kBlock), 0, h->stream, n,
                       (const double*)V.b, h->rb.partials);
    h->finalize_fn<1, 1u>(FinThresh{h->st, eps, 1}, h->vgrid);
    h->last_pcg = 1;
    h->pcg_solve<double>(rho, max_iter);
    hipLaunchKernelGGL((k_probe_acc<double>), dim3(h->vgrid), dim3(kBlock), 0, h->stream, n,
                       (const int8_t*)probe, (const double*)V.xt, acc);
    ++k;
  }
  HIPCHK(hipMemcpyAsync(diag, acc, n * sizeof(double), hipMemcpyDeviceToHost, h->stream));
  HIPCHK(hipStreamSynchronize(h->stream));
  for (int i = 0; i < n; ++i) diag[i] /= nprobes;
  h->jacobi<double>(rho_saved);
  HIPCHK(hipGetLastError());
  return QPG_OK;
}

int hutchinson_device_error(qpg_solver* h, const HipError& e) {
  char buf[512];
  std::snprintf(buf, sizeof(buf), "%s failed: %s", e.what, hipGetErrorString(e.code));
  h->err = buf;
  (void)hipGetLastError();
  return QPG_ERR_DEVICE;
}

}  // namespace

namespace qpg {

// Device address of the no-alloc scratch for the current device, looked up once per device at
// setup. Ordinals beyond the table keep no address (qpg_hutchinson_noalloc then fails with
// QPG_ERR_STATE on them).
hipError_t resolve_noalloc_scratch(int device) {
  if (device < 0 || device >= kScratchDevices) return hipSuccess;
  if (g_scratch_addr[device].load(std::memory_order_acquire)) return hipSuccess;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_addr[device].load(std::memory_order_relaxed)) return hipSuccess;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e == hipSuccess) g_scratch_addr[device].store(ptr, std::memory_order_release);
  return e;
}

}  // namespace qpg

// ================================================================================== C ABI

extern "C" {

int qpg_get_kdiag(const qpg_solver* h, double rho, double* kdiag) {
  if (!h || !kdiag || !(rho > 0)) return QPG_ERR_ARG;
  if (h->s.rho_vector) return QPG_ERR_STATE;  // K is defined here with R = ρ̄I
  for (int i = 0; i < h->n; ++i) kdiag[i] = h->diagP_h[i] + h->s.sigma + rho * h->colsq_h[i];
  return QPG_OK;
}

int qpg_device_bytes(const qpg_solver* h, int64_t out[2]) {
  if (!h || !out) return QPG_ERR_ARG;
  out[0] = (int64_t)h->arena.held;
  out[1] = (int64_t)h->arena.used;
  if (h->learned) {
    out[0] += (int64_t)h->learned->arena.held;
    out[1] += (int64_t)h->learned->arena.used;
  }
  return QPG_OK;
}

int qpg_hutchinson(qpg_solver* h, const int8_t* signs, int32_t nprobes, double rho, double eps,
                   int32_t max_iter, double* diag) {
  const int rc = hutchinson_check(h, signs, nprobes, rho, eps, max_iter, diag);
  if (rc) return rc;
  try {
    HIPCHK(hipSetDevice(h->device));
    LearnedState* L = ensure_graph(h);
    const int from = together_from(h);
    if (nprobes >= from && ensure_multi(h, L)) {
      struct End {
        LearnedState* L;
        ~End() { L->end_multi(); }
      } end{L};
      return hutchinson_run(h, signs, nprobes, rho, eps, max_iter, diag, L->acc, L->probe, L, from);
    }
    return hutchinson_run(h, signs, nprobes, rho, eps, max_iter, diag, L->acc, L->probe);
  } catch (const HipError& e) {
    return hutchinson_device_error(h, e);
  } QPG_CATCH_HOST(h->err)
}

int qpg_hutchinson_noalloc(qpg_solver* h, const int8_t* signs, int32_t nprobes, double rho,
                           double eps, int32_t max_iter, double* diag) {
  const int rc = hutchinson_check(h, signs, nprobes, rho, eps, max_iter, diag);
  if (rc) return rc;
  const size_t acc_bytes = ((size_t)h->n * sizeof(double) + 255) / 256 * 256;
  if (acc_bytes + (size_t)h->n > (size_t)QPG_NOALLOC_SCRATCH_BYTES) {
    h->err = "qpg_hutchinson_noalloc: n exceeds the static scratch (QPG_NOALLOC_MAX_N)";
    return QPG_ERR_SIZE;
  }
  void* base = noalloc_scratch(h->device);
  if (!base) {
    h->err = "qpg_hutchinson_noalloc: no scratch address for this device";
    return QPG_ERR_STATE;
  }
  try {
    HIPCHK(hipSetDevice(h->device));
    unsigned char* b = static_cast<unsigned char*>(base);
    return hutchinson_run(h, signs, nprobes, rho, eps, max_iter, diag, reinterpret_cast<double*>(b),
                          reinterpret_cast<int8_t*>(b + acc_bytes));
  } catch (const HipError& e) {
    return hutchinson_device_error(h, e);
  } QPG_CATCH_HOST(h->err)
}

int qpg_net_create(qpg_net** out, const float* params, uint64_t seed, int32_t bf16, int32_t device) {
  if (!out) return QPG_ERR_ARG;
  *out = nullptr;
  qpg_net* net = new (std::nothrow) qpg_net();
  if (!net) return QPG_ERR_OOM;
  net->device = device;
  net->bf16 = bf16 ? 1 : 0;
  try {
    HIPCHK(hipSetDevice(device));
    const size_t bytes = NetOff::total * sizeof(float);
    for (float** p : {&net->theta, &net->grad, &net->m1, &net->m2}) HIPCHK(hipMalloc((void**)p, bytes));
    std::vector<float> init;
    if (params)
      init.assign(params, params + NetOff::total);
    else
      init_params(init, seed);
    HIPCHK(hipMemcpy(net->theta, init.data(), bytes, hipMemcpyHostToDevice));
    HIPCHK(hipMemset(net->grad, 0, bytes));
    HIPCHK(hipMemset(net->m1, 0, bytes));
    HIPCHK(hipMemset(net->m2, 0, bytes));
  } catch (const HipError& e) {
    int code = net_error(net, e);
    delete net;
    return code;
  } catch (const std::bad_alloc&) {
    delete net;
    return QPG_ERR_OOM;
  } catch (const std::exception&) {
    delete net;
    return QPG_ERR_HOST;
  }
  *out = net;
  return QPG_OK;
}

int qpg_net_get_params(const qpg_net* net, float* params) {
  if (!net || !params) return QPG_ERR_ARG;
  if (hipSetDevice(net->device) != hipSuccess ||
      hipMemcpy(params, net->theta, NetOff::total * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess)
    return QPG_ERR_DEVICE;
  return QPG_OK;
}

int qpg_net_set_params(qpg_net* net, const float* params) {
  if (!net || !params) return QPG_ERR_ARG;
  if (hipSetDevice(net->device) != hipSuccess ||
      hipMemcpy(net->theta, params, NetOff::total * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
    return QPG_ERR_DEVICE;
  net->step = 0;
  return QPG_OK;
}

int qpg_net_forward(qpg_net* net, qpg_solver* h, double rho, float* g) {
  if (!net || !h || !(rho > 0)) return QPG_ERR_ARG;
  if (net->device != h->device) return QPG_ERR_ARG;
  try {
    HIPCHK(hipSetDevice(h->device));
    LearnedState* L = ensure_graph(h);
    trunk(h, L, net->theta, net->bf16);
    head<double>(h, L, net->theta, net->bf16, rho, (double*)nullptr);
    if (g) HIPCHK(hipMemcpyAsync(g, L->g, h->n * sizeof(float), hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    HIPCHK(hipGetLastError());
  } catch (const HipError& e) {
    return net_error(net, e);
  } QPG_CATCH_HOST(net->err)
  return QPG_OK;
}

int qpg_net_loss_grad(qpg_net* net, qpg_solver* h, double rho, const float* target, double* loss,
                      float* grad) {
  if (!net || !h || !target || !(rho > 0)) return QPG_ERR_ARG;
  if (net->device != h->device) return QPG_ERR_ARG;
  try {
    HIPCHK(hipSetDevice(h->device));
    LearnedState* L = ensure_graph(h);
    HIPCHK(hipMemcpyAsync(L->tgt, target, h->n * sizeof(float), hipMemcpyHostToDevice, h->stream));
    trunk(h, L, net->theta, net->bf16);
    head<double>(h, L, net->theta, net->bf16, rho, (double*)nullptr);
    loss_backward(h, L, net->theta, net->bf16, net->grad);
    if (grad)
      HIPCHK(hipMemcpyAsync(grad, net->grad, NetOff::total * sizeof(float), hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    if (loss) *loss = L->ns_host->loss;
    HIPCHK(hipGetLastError());
  } catch (const HipError& e) {
    return net_error(net, e);
  } QPG_CATCH_HOST(net->err)
  return QPG_OK;
}

int qpg_net_adam_step(qpg_net* net, float lr) {
  if (!net || !(lr > 0)) return QPG_ERR_ARG;
  try {
    HIPCHK(hipSetDevice(net->device));
    net->step++;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - std::pow(b1, (float)net->step), c2 = 1.f - std::pow(b2, (float)net->step);
    hipLaunchKernelGGL(k_adam, dim3(div_up(NetOff::total, kBlock)), dim3(kBlock), 0, 0, NetOff::total,
                       net->theta, (const float*)net->grad, net->m1, net->m2, lr, b1, b2, 1e-8f, c1, c2);
    HIPCHK(hipDeviceSynchronize());
    HIPCHK(hipGetLastError());
  } catch (const HipError& e) {
    return net_error(net, e);
  } QPG_CATCH_HOST(net->err)
  return QPG_OK;
}

int qpg_net_destroy(qpg_net* net) {
  if (!net) return QPG_OK;
  (void)hipSetDevice(net->device);
  delete net;
  return QPG_OK;
}

}  // extern "C"
