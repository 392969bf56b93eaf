// Host side of Algorithm 2 (the L2 flow with replicate boundaries, driven by
// L-BFGS) and its entry points. Included once by fe_api.hip.
#pragma once

// The optimiser state lives in device vectors of the box with a margin of one voxel
// (zeros); its scalars are FP64 on the host.
struct fe_l2 {
  fe_ctx* ctx = nullptr;         // the grid with the margin, box mode
  fe::PadBox box{};
  double sigma_k = 0.0;
  int r = 0;                     // blur radius
  size_t n = 0;                  // elements with the margin
  size_t esz = 0;
  void* x = nullptr;             // the variable u (its margin is never read)
  void* g = nullptr;             // dF/du (zero margin)
  void* w0 = nullptr;            // work fields
  void* w1 = nullptr;
  void* w2 = nullptr;
  void* d = nullptr;             // search direction
  void* prev_g = nullptr;
  void* q = nullptr;             // two-loop scratch
  std::vector<void*> S, Y;       // history, oldest first (pointers rotate, memory stays)
  std::vector<double> rho;
  std::vector<double> SY, YY;    // [history][history]: s_a . y_b (a <= b) and y_a . y_b of the history
  std::vector<double> pgS, pgY;  // prev_g . s_a and prev_g . y_a for the current history
  int hist_len = 0;
  double* d_red = nullptr;       // reduction banks
  double* h_vals = nullptr;      // pinned: the values that the host reads, written by the device (null: none left)
  // settings
  double lr = 1.0, tol_grad = 1e-7, tol_change = 1e-9;
  int history = 10, max_iter = 20, max_eval = 25;
  // state
  long n_iter = 0;
  double t = 0.0, H_diag = 1.0, prev_loss = 0.0;
};

namespace {

// Copies between the box of the flow's array and a dense box field.
template <typename T>
int l2_box_copy(fe_l2* L, const void* src, void* dst, int to_padded) {
  const fe::PadBox& b = L->box;
  const int bx = b.hi[0] - b.lo[0], by = b.hi[1] - b.lo[1], bz = b.hi[2] - b.lo[2];
  hipLaunchKernelGGL(fe::box_copy<T>, dim3((unsigned)ceil_div(bx * by, 1024), (unsigned)bz), dim3(256), 0,
                     L->ctx->stream, static_cast<const T*>(src), static_cast<T*>(dst), b, to_padded);
  FE_HIP(hipGetLastError());
  return FE_OK;
}

int l2_box_copy_any(fe_l2* L, const void* src, void* dst, int to_padded) {
  return L->ctx->grid.dtype == FE_F32 ? l2_box_copy<float>(L, src, dst, to_padded)
                                      : l2_box_copy<double>(L, src, dst, to_padded);
}

// Scalars of the optimiser. Named slots: 0 energy, 1 max|g|, 2 max|d|, 3 g'd
// and 4 |g|_1 (first iteration); then the inner products of the Gram pass
// (y.y, y.s, y.g, g.g, g.s, then g.V_k for each history vector). d_red
// holds one bank of kVecBlocks partials per slot; the values go to pinned host
// memory, one per slot (the sweep's finish writes the energy there directly); where
// there was none, to the bank of kSlotE, which holds no partials, and are copied.
constexpr int kSlotE = 0, kSlotGmax = 1, kSlotDmax = 2, kSlotGtd = 3, kSlotL1 = 4, kSlotGram = 5;
constexpr int kL2MaxHistory = 64;
constexpr int kL2Banks = kSlotGram + 5 + 2 * kL2MaxHistory;
constexpr size_t kL2RedDoubles = (size_t)kL2Banks * fe::kVecBlocks;
static_assert(kL2Banks <= fe::kVecBlocks, "a value per slot in the bank of kSlotE");

double* l2_bank(fe_l2* L, int slot) { return L->d_red + (size_t)slot * fe::kVecBlocks; }
double* l2_vals(fe_l2* L) { return L->h_vals ? L->h_vals : l2_bank(L, kSlotE); }

const dim3 kVecGrid(fe::kVecBlocks), kVecBlock(fe::kVecThreads);

// Reduction of a (and b) into the bank of `slot`, stream-ordered, no sync.
template <typename T>
int l2_reduce_dev(fe_l2* L, int op, const void* a, const void* b, int slot) {
  hipStream_t s = L->ctx->stream;
  const T* pa = static_cast<const T*>(a);
  const T* pb = static_cast<const T*>(b);
  double* bank = l2_bank(L, slot);
  if (op == 0)
    hipLaunchKernelGGL((fe::vec_reduce<T, 0>), kVecGrid, kVecBlock, 0, s, pa, pb, L->n, bank);
  else if (op == 1)
    hipLaunchKernelGGL((fe::vec_reduce<T, 1>), kVecGrid, kVecBlock, 0, s, pa, pb, L->n, bank);
  else
    hipLaunchKernelGGL((fe::vec_reduce<T, 2>), kVecGrid, kVecBlock, 0, s, pa, pb, L->n, bank);
  FE_HIP(hipGetLastError());
  return FE_OK;
}

// Host copies of the values of slots [0, count), the energy's among them (one sync);
// the other slots' banks are combined on the device first, which writes them to the
// host itself.
int l2_read_slots(fe_l2* L, int count, double* out) {
  if (count > kSlotGmax) {
    hipLaunchKernelGGL(fe::vec_finish, dim3(count - kSlotGmax), dim3(64), 0, L->ctx->stream,
                       (const double*)l2_bank(L, kSlotGmax), l2_vals(L) + kSlotGmax,
                       (1u << (kSlotGmax - kSlotGmax)) | (1u << (kSlotDmax - kSlotGmax)));
    FE_HIP(hipGetLastError());
  }
  if (!L->h_vals)
    FE_HIP(hipMemcpyAsync(out, l2_vals(L), sizeof(double) * count, hipMemcpyDeviceToHost, L->ctx->stream));
  FE_HIP(hipStreamSynchronize(L->ctx->stream));
  if (L->h_vals) std::copy_n(L->h_vals, count, out);
  return FE_OK;
}

// out = sum_k c[k] v[k] (+ out when acc), in passes of up to kCombVecs vectors;
// with dmax, the last pass leaves max |out| in the bank of kSlotDmax. No sync.
template <typename T>
int l2_lincomb(fe_l2* L, const std::vector<const void*>& v, const std::vector<double>& c, bool acc, void* out,
               bool dmax, void* x = nullptr, double t = 0.0) {
  const size_t K = v.size();
  for (size_t k0 = 0; k0 < K; k0 += fe::kCombVecs) {
    fe::CombList<T> cl{};
    cl.count = (int)std::min<size_t>(fe::kCombVecs, K - k0);
    // pass widths 1, 4, 8, 16 or 24; the padding repeats the first vector with c = 0
    const int w = cl.count == 1 ? 1 : cl.count <= 4 ? 4 : cl.count <= 8 ? 8 : cl.count <= 16 ? 16 : fe::kCombVecs;
    for (int k = 0; k < w; ++k) {
      cl.v[k] = static_cast<const T*>(v[k < cl.count ? k0 + k : k0]);
      cl.c[k] = k < cl.count ? c[k0 + k] : 0.0;
    }
    const int a = (acc || k0 > 0) ? 1 : 0;
    const bool last = k0 + fe::kCombVecs >= K;
    double* dm = (dmax && last) ? l2_bank(L, kSlotDmax) : nullptr;
    T* px = last ? static_cast<T*>(x) : nullptr;
    T* po = static_cast<T*>(out);
    hipStream_t s = L->ctx->stream;
    if (w == 1)
      hipLaunchKernelGGL((fe::vec_lincomb<T, 1>), kVecGrid, kVecBlock, 0, s, cl, po, a, L->n, dm, px, t);
    else if (w == 4)
      hipLaunchKernelGGL((fe::vec_lincomb<T, 4>), kVecGrid, kVecBlock, 0, s, cl, po, a, L->n, dm, px, t);
    else if (w == 8)
      hipLaunchKernelGGL((fe::vec_lincomb<T, 8>), kVecGrid, kVecBlock, 0, s, cl, po, a, L->n, dm, px, t);
    else if (w == 16)
      hipLaunchKernelGGL((fe::vec_lincomb<T, 16>), kVecGrid, kVecBlock, 0, s, cl, po, a, L->n, dm, px, t);
    else
      hipLaunchKernelGGL((fe::vec_lincomb<T, fe::kCombVecs>), kVecGrid, kVecBlock, 0, s, cl, po, a, L->n, dm, px, t);
    FE_HIP(hipGetLastError());
  }
  return FE_OK;
}

// y = alpha x (+ y when acc) with a host coefficient
template <typename T>
int l2_scale_add(fe_l2* L, double alpha, const void* x, bool acc, void* y) {
  return l2_lincomb<T>(L, {x}, {alpha}, acc, y, false);
}

// The Gram pass: y = g - prev_g into L->q, s = t d into L->w0, and the inner
// products y.y, y.s, y.g, g.g, g.s and g.v for every history vector v (S, then Y)
// into the banks of kSlotGram on, and max |g| into kSlotGmax's; stream-ordered. Up to
// kDotVecs history vectors go through one pass; a list of 8, 16 or 24 entries, the
// unused ones pointing at g.
template <typename T>
void gram_launch(fe_l2* L, bool form, const fe::DotList<T>& dl, int bank) {
  hipStream_t s = L->ctx->stream;
  const T* g = static_cast<const T*>(L->g);
  const T* pg = static_cast<const T*>(L->prev_g);
  const T* d = static_cast<const T*>(L->d);
  T* y = static_cast<T*>(L->q);
  T* sv = static_cast<T*>(L->w0);
  double* bk = l2_bank(L, bank);
  double* gm = l2_bank(L, kSlotGmax);
  const dim3 grid = kVecGrid, blk = kVecBlock;
  const int nl = dl.count == 0 ? 0 : dl.count <= 8 ? 8 : dl.count <= 16 ? 16 : fe::kDotVecs;
  if (form) {
    if (nl == 0)
      hipLaunchKernelGGL((fe::vec_gram<T, true, 0>), grid, blk, 0, s, g, pg, d, L->t, y, sv, dl, L->n, bk, gm);
    else if (nl == 8)
      hipLaunchKernelGGL((fe::vec_gram<T, true, 8>), grid, blk, 0, s, g, pg, d, L->t, y, sv, dl, L->n, bk, gm);
    else if (nl == 16)
      hipLaunchKernelGGL((fe::vec_gram<T, true, 16>), grid, blk, 0, s, g, pg, d, L->t, y, sv, dl, L->n, bk, gm);
    else
      hipLaunchKernelGGL((fe::vec_gram<T, true, fe::kDotVecs>), grid, blk, 0, s, g, pg, d, L->t, y, sv, dl, L->n,
                         bk, gm);
  } else {
    if (nl == 8)
      hipLaunchKernelGGL((fe::vec_gram<T, false, 8>), grid, blk, 0, s, g, nullptr, nullptr, 0.0, nullptr, nullptr, dl,
                         L->n, bk, nullptr);
    else if (nl == 16)
      hipLaunchKernelGGL((fe::vec_gram<T, false, 16>), grid, blk, 0, s, g, nullptr, nullptr, 0.0, nullptr, nullptr,
                         dl, L->n, bk, nullptr);
    else
      hipLaunchKernelGGL((fe::vec_gram<T, false, fe::kDotVecs>), grid, blk, 0, s, g, nullptr, nullptr, 0.0, nullptr,
                         nullptr, dl, L->n, bk, nullptr);
  }
}

template <typename T>
int l2_gram_dev(fe_l2* L) {
  const T* g = static_cast<const T*>(L->g);
  const int m = L->hist_len, K = 2 * m;
  int bank = kSlotGram, k0 = 0;
  do {
    fe::DotList<T> dl{};
    dl.count = std::min(fe::kDotVecs, K - k0);
    for (int k = 0; k < fe::kDotVecs; ++k)
      dl.v[k] = k >= dl.count ? g : static_cast<const T*>(k0 + k < m ? L->S[k0 + k] : L->Y[k0 + k - m]);
    gram_launch<T>(L, k0 == 0, dl, bank);
    FE_HIP(hipGetLastError());
    bank += (k0 == 0 ? 5 : 0) + dl.count;
    k0 += dl.count;
  } while (k0 < K);
  return FE_OK;
}

// The box of the flow's arrays; a pass with this writes box voxels in place.
fe::EdgeBox l2_edge(const fe_l2* L) {
  const fe::PadBox& b = L->box;
  const size_t row = b.nx, plane = (size_t)b.nx * b.ny;
  return fe::EdgeBox{b.lo[0], b.hi[0] - b.lo[0], b.hi[1] - b.lo[1], b.hi[2] - b.lo[2],
                     row,     plane,             b.lo[2] * plane + b.lo[1] * row + b.lo[0]};
}

// The same box, written as a dense box field.
fe::EdgeBox l2_dense(const fe_l2* L) {
  fe::EdgeBox e = l2_edge(L);
  e.orow = e.nx;
  e.oplane = (size_t)e.nx * e.ny;
  e.ooff = 0;
  return e;
}

// The separable blur of the box (EDGE: fe::kReplicate forward, fe::kAdjoint with the
// fold of the sweep's gradient): in -> tmp1 (x) -> tmp2 (y) -> out (z), or
// in -> tmp1 (fused x-y) -> out (z) for r = 4, 8; tmp1 and tmp2 in the array's
// layout, out as `eo` says; out may be in.
template <typename T, int EDGE>
void l2_blur(fe_l2* L, const T* in, T* tmp1, T* tmp2, T* out, const fe::EdgeBox& eo) {
  const fe::FieldDims d{L->box.nx, L->box.ny, L->box.nz, 1};
  const fe::BlurTaps<T> k = blur_taps<T>(L->sigma_k);
  const fe::EdgeBox e = l2_edge(L);
  hipStream_t s = L->ctx->stream;
  if (has_xy_pass(k.r)) {
    blur_xy_pass<T, EDGE>(s, d, k, in, tmp1, e);
    blur_axis_pass<T, 2, EDGE>(s, d, k, tmp1, out, eo);
    return;
  }
  blur_x_pass<T, false, EDGE>(s, d, k, in, tmp1, nullptr, nullptr, T(0), nullptr, 0.0, 0.0, e);
  blur_axis_pass<T, 1, EDGE>(s, d, k, tmp1, tmp2, e);
  blur_axis_pass<T, 2, EDGE>(s, d, k, tmp2, out, eo);
}

// F_h(k * x) with replicate boundaries into the energy slot and its gradient into
// g, which takes box voxels only, laid out as `eo` says; stream-ordered.
template <typename T>
int l2_eval_dev(fe_l2* L, T* g, const fe::EdgeBox& eo) {
  T* x = static_cast<T*>(L->x);
  T* w0 = static_cast<T*>(L->w0);
  T* w1 = static_cast<T*>(L->w1);
  T* w2 = static_cast<T*>(L->w2);
  const T* ub = x;
  if (L->r > 0) {
    l2_blur<T, fe::kReplicate>(L, x, w0, w1, w2, l2_edge(L));   // w2 = k * x
    ub = w2;
  }
  int rc = sweep_energy(L->ctx, L->ctx->stream, fe::kGrad, ub, w0, l2_vals(L) + kSlotE);
  if (rc) return rc;
  if (L->r > 0) {
    l2_blur<T, fe::kAdjoint>(L, w0, w1, w2, g, eo);
  } else {
    const fe::FieldDims d{L->box.nx, L->box.ny, L->box.nz, 1};
    hipLaunchKernelGGL(fe::fold_shell<T>, dim3((unsigned)ceil_div(eo.nx * eo.ny, 256), (unsigned)eo.nz), dim3(256), 0,
                       L->ctx->stream, (const T*)w0, g, d, eo);
  }
  FE_HIP(hipGetLastError());
  return FE_OK;
}

// The same into the optimiser's gradient.
template <typename T>
int l2_eval_dev(fe_l2* L) {
  return l2_eval_dev<T>(L, static_cast<T*>(L->g), l2_edge(L));
}

// As l2_eval_dev, the gradient into a dense box field (null: into the optimiser's),
// with the loss copied to the host (syncs).
template <typename T>
int l2_eval(fe_l2* L, double& loss, T* g) {
  int rc = g ? l2_eval_dev<T>(L, g, l2_dense(L)) : l2_eval_dev<T>(L);
  if (rc) return rc;
  rc = l2_read_slots(L, 1, &loss);
  if (rc) return rc;
  if (!std::isfinite(loss)) return set_error(FE_ENONFINITE, "energy is not finite");
  return FE_OK;
}

// The scalars of one evaluation: the energy, max|g|, max|d| of the last direction
// and, unless the next iteration is the first ever, its Gram pass, which depends on
// nothing that the host decides in between (its vectors are scratch if the step ends
// here). One read for all of them: two reads per iteration left the device idle for
// about 85 us, one for 45 (128^3 FP64, 20 iterations: 6.16 -> 5.50 ms).
template <typename T>
int l2_eval_scalars(fe_l2* L, bool gram, std::vector<double>& sc) {
  int rc = l2_eval_dev<T>(L);
  if (!rc) rc = gram ? l2_gram_dev<T>(L) : l2_reduce_dev<T>(L, 2, L->g, nullptr, kSlotGmax);
  if (rc) return rc;
  sc.resize(gram ? kSlotGram + 5 + 2 * L->hist_len : kSlotDmax + 1);
  if ((rc = l2_read_slots(L, (int)sc.size(), sc.data()))) return rc;
  if (!std::isfinite(sc[kSlotE])) return set_error(FE_ENONFINITE, "energy is not finite");
  return FE_OK;
}

// One optimiser step of L-BFGS without line search (Nocedal and Wright, the
// two-loop recursion with H0 = s'y / y'y): up to max_iter inner iterations,
// each a fixed step t d; the first ever step is scaled by min(1, 1/|g|_1);
// a pair (s, y) enters the history only if s'y > 1e-10. Stops early on
// max|g| <= tol_grad, a non-descent direction (g'd > -tol_change), a step
// max|t d| <= tol_change, or a loss change below tol_change. `loss0` receives
// the loss at the start of the step. The host reads the scalars of an iteration
// once, after its evaluation (l2_eval_scalars).
template <typename T>
int l2_step(fe_l2* L, double& loss0) {
  std::vector<double> sc;
  int rc = l2_eval_scalars<T>(L, L->n_iter > 0, sc);
  if (rc) return rc;
  double loss = sc[kSlotE];
  loss0 = loss;
  int evals = 1;
  if (sc[kSlotGmax] <= L->tol_grad) return FE_OK;
  bool opt_cond = false;
  for (int it = 1; it <= L->max_iter; ++it) {
    ++L->n_iter;
    const bool first = L->n_iter == 1;
    double gtd = 0.0, gl1 = 0.0;
    bool moved = false;   // x already advanced by the direction pass
    if (first) {
      if ((rc = l2_lincomb<T>(L, {L->g}, {-1.0}, false, L->d, true))) return rc;   // d = -g
      L->hist_len = 0;
      L->rho.clear();
      L->pgS.clear();
      L->pgY.clear();
      L->H_diag = 1.0;
      if ((rc = l2_reduce_dev<T>(L, 0, L->g, L->d, kSlotGtd))) return rc;
      if ((rc = l2_reduce_dev<T>(L, 1, L->g, nullptr, kSlotL1))) return rc;
      double gl[kSlotL1 + 1];
      if ((rc = l2_read_slots(L, kSlotL1 + 1, gl))) return rc;
      gtd = gl[kSlotGtd];
      gl1 = gl[kSlotL1];
    } else {
      // The Gram pass came with the evaluation: y = g - prev_g (in q), s = t d (in
      // w0), the inner products of y and g with each other and with s, and g with
      // every history vector; y with a history vector is g.v - prev_g.v, the latter
      // kept from the previous pass (prev_g was that pass's g).
      int m = L->hist_len;
      const int H = L->history;
      const double* gv = sc.data() + kSlotGram;
      const double yy = gv[0], ys = gv[1], yg = gv[2], gg = gv[3], gs = gv[4];
      if ((int)L->pgS.size() != m || (int)L->pgY.size() != m)
        return set_error(FE_EINVAL, "L-BFGS state out of step with its history");
      std::vector<double> yS(m), gS(m), yY(m), gY(m);
      for (int i = 0; i < m; ++i) {
        gS[i] = gv[5 + i];
        gY[i] = gv[5 + m + i];
        yS[i] = gS[i] - L->pgS[i];
        yY[i] = gY[i] - L->pgY[i];
      }
      double* SY = L->SY.data();
      double* YY = L->YY.data();
      // accept the pair if y's > 1e-10 (the oldest leaves a full history)
      if (ys > 1e-10) {
        if (m == H) {
          std::rotate(L->S.begin(), L->S.begin() + 1, L->S.end());
          std::rotate(L->Y.begin(), L->Y.begin() + 1, L->Y.end());
          L->rho.erase(L->rho.begin());
          for (int a = 0; a + 1 < m; ++a)
            for (int b = 0; b + 1 < m; ++b) {
              SY[a * H + b] = SY[(a + 1) * H + b + 1];
              YY[a * H + b] = YY[(a + 1) * H + b + 1];
            }
          for (auto* v : {&yS, &gS, &yY, &gY}) v->erase(v->begin());
          --m;
        }
        // the new pair takes over the buffers of y and s; theirs become scratch
        std::swap(L->q, L->Y[m]);
        std::swap(L->w0, L->S[m]);
        for (int a = 0; a < m; ++a) {
          SY[a * H + m] = yS[a];                 // s_a . y_new
          YY[a * H + m] = YY[m * H + a] = yY[a];
        }
        SY[m * H + m] = ys;
        YY[m * H + m] = yy;
        gS.push_back(gs);
        gY.push_back(yg);
        L->rho.push_back(1.0 / ys);
        L->hist_len = ++m;
        L->H_diag = ys / yy;
      }
      // g becomes prev_g below: keep its products with the history as it now stands
      L->pgS = gS;
      L->pgY = gY;
      // The two-loop recursion on the inner products, newest to oldest:
      //   a_i = rho_i s_i.q with q = -g - sum_{j>i} a_j y_j,
      // then r = H q (q = -g - sum_j a_j y_j), oldest to newest:
      //   b_i = rho_i y_i.r with r = H q + sum_{j<i} (a_j - b_j) s_j,
      // and d = H q + sum_i (a_i - b_i) s_i = -H g - H sum_j a_j y_j + sum_i (a_i - b_i) s_i.
      const double Hd = L->H_diag;
      std::vector<double> al(m), be(m);
      for (int i = m - 1; i >= 0; --i) {
        double sq = -gS[i];
        for (int j = i + 1; j < m; ++j) sq -= al[j] * SY[i * H + j];
        al[i] = L->rho[i] * sq;
      }
      for (int i = 0; i < m; ++i) {
        double yq = -gY[i];
        for (int j = 0; j < m; ++j) yq -= al[j] * YY[i * H + j];
        double yr = Hd * yq;
        for (int j = 0; j < i; ++j) yr += (al[j] - be[j]) * SY[j * H + i];
        be[i] = L->rho[i] * yr;
      }
      std::vector<const void*> vv{L->g};
      std::vector<double> cc{-Hd};
      gtd = -Hd * gg;
      for (int i = 0; i < m; ++i) {
        vv.push_back(L->S[i]);
        cc.push_back(al[i] - be[i]);
        gtd += (al[i] - be[i]) * gS[i];
      }
      for (int j = 0; j < m; ++j) {
        vv.push_back(L->Y[j]);
        cc.push_back(-Hd * al[j]);
        gtd += -Hd * al[j] * gY[j];
      }
      // when the step will be taken (t = lr, g'd below -tol_change), the pass
      // that forms d also moves x
      moved = !(gtd > -L->tol_change);
      if ((rc = l2_lincomb<T>(L, vv, cc, false, L->d, true, moved ? L->x : nullptr, L->lr))) return rc;
    }
    // prev_g takes over the gradient's buffer; the next evaluation writes g anew
    std::swap(L->g, L->prev_g);
    L->prev_loss = loss;
    L->t = first ? std::min(1.0, 1.0 / gl1) * L->lr : L->lr;
    if (gtd > -L->tol_change) break;
    int ls_evals = 0;
    if (!moved && (rc = l2_scale_add<T>(L, L->t, L->d, true, L->x))) return rc;   // max |d| is in its slot already
    double dmax = 0.0;
    if (it != L->max_iter) {
      if ((rc = l2_eval_scalars<T>(L, true, sc))) return rc;
      loss = sc[kSlotE];
      opt_cond = sc[kSlotGmax] <= L->tol_grad;
      dmax = sc[kSlotDmax];
      ls_evals = 1;
    }
    evals += ls_evals;
    if (it == L->max_iter) break;
    if (evals >= L->max_eval) break;
    if (opt_cond) break;
    if (dmax * std::fabs(L->t) <= L->tol_change) break;
    if (std::fabs(loss - L->prev_loss) < L->tol_change) break;
  }
  return FE_OK;
}

int l2_free(fe_l2* L) {
  if (!L) return FE_OK;
  for (void* p : {L->x, L->g, L->w0, L->w1, L->w2, L->d, L->prev_g, L->q, (void*)L->d_red})
    if (p) (void)hipFree(p);
  pinned_give(L->h_vals, kL2Banks);
  for (void* p : L->S)
    if (p) (void)hipFree(p);
  for (void* p : L->Y)
    if (p) (void)hipFree(p);
  if (L->ctx) fe_destroy(L->ctx);
  delete L;
  return FE_OK;
}

}  // namespace

extern "C" {

int fe_l2_create(const fe_grid* grid, double eps, const double* p_coeffs, double sigma_k, void* stream,
                 fe_l2** out) {
  g_last_error.clear();
  if (!out) return set_error(FE_EINVAL, "out is NULL");
  *out = nullptr;
  int rc = check_grid(grid);
  if (rc) return rc;
  if (grid->batch != 1) return set_error(FE_EINVAL, "the L2 flow takes one field (batch 1)");
  if (!(sigma_k >= 0.0) || std::ceil(4.0 * sigma_k) > fe::kBlurMaxR)
    return set_error(FE_EINVAL, "sigma_k must lie in [0, %g]", fe::kBlurMaxR / 4.0);
  fe_l2* L = new (std::nothrow) fe_l2();
  if (!L) return set_error(FE_ENOMEM, "host allocation failed");
  L->sigma_k = sigma_k;
  L->r = sigma_k > 0.0 ? (int)std::ceil(4.0 * sigma_k) : 0;
  // the limits hold for a box with a margin as wide as the blur on every side
  const int M = std::max(1, L->r);
  fe_grid mg = *grid;
  mg.nx += 2 * M;
  mg.ny += 2 * M;
  mg.nz += 2 * M;
  if ((long)mg.nz > 65535 || (long)mg.ny > 65535 || !flow_dims_ok(mg)) {
    l2_free(L);
    return set_error(FE_EINVAL, "grid too large for the flow kernels");
  }
  if ((rc = check_grid(&mg))) {
    l2_free(L);
    return rc;
  }
  constexpr int W = 1;
  fe_grid pg = *grid;
  pg.nx += 2 * W;
  pg.ny += 2 * W;
  pg.nz += 2 * W;
  rc = fe_create(&pg, &eps, p_coeffs, stream, &L->ctx);
  if (rc) {
    l2_free(L);
    return rc;
  }
  fe_ctx* c = L->ctx;
  c->use_box = true;
  c->variant = sweep_variant(c);
  const int dims[3] = {grid->nx, grid->ny, grid->nz};
  for (int i = 0; i < 3; ++i) {
    c->box_lo[i] = W;
    c->box_hi[i] = W + dims[i];
  }
  L->box = fe::PadBox{pg.nx, pg.ny, pg.nz, {W, W, W}, {W + grid->nx, W + grid->ny, W + grid->nz}};
  L->esz = elem_size(pg);
  L->n = field_elems(pg);
  DeviceGuard dg(c->device);
  for (void** p : {&L->x, &L->g, &L->w0, &L->w1, &L->w2, &L->d, &L->prev_g, &L->q}) {
    if (hipMalloc(p, L->n * L->esz) != hipSuccess) {
      *p = nullptr;
      l2_free(L);
      return set_error(FE_ENOMEM, "L2 flow field allocation failed");
    }
    if (hipMemsetAsync(*p, 0, L->n * L->esz, c->stream) != hipSuccess) {
      l2_free(L);
      return set_error(FE_EHIP, "hipMemsetAsync failed");
    }
  }
  if (hipMalloc((void**)&L->d_red, sizeof(double) * kL2RedDoubles) != hipSuccess) {
    L->d_red = nullptr;
    l2_free(L);
    return set_error(FE_ENOMEM, "L2 flow reduction buffer allocation failed");
  }
  L->h_vals = pinned_take(kL2Banks);
  if (hipMemsetAsync(L->d_red, 0, sizeof(double) * kL2RedDoubles, c->stream) != hipSuccess) {
    l2_free(L);
    return set_error(FE_EHIP, "hipMemsetAsync failed");
  }
  rc = fe_l2_set_lbfgs(L, 1.0, 10, 20, 1e-7, 1e-9);
  if (rc) {
    l2_free(L);
    return rc;
  }
  *out = L;
  return FE_OK;
}

int fe_l2_set_lbfgs(fe_l2* L, double lr, int history, int max_iter, double tolerance_grad, double tolerance_change) {
  g_last_error.clear();
  if (!L) return set_error(FE_EINVAL, "flow is NULL");
  if (!(lr > 0.0) || !std::isfinite(lr)) return set_error(FE_EINVAL, "lr must be finite and > 0");
  if (history < 1 || history > kL2MaxHistory)
    return set_error(FE_EINVAL, "history must lie in [1, %d]", kL2MaxHistory);
  if (max_iter < 1) return set_error(FE_EINVAL, "max_iter must be >= 1");
  if (!(tolerance_grad >= 0.0) || !(tolerance_change >= 0.0))
    return set_error(FE_EINVAL, "tolerances must be >= 0");
  DeviceGuard dg(L->ctx->device);
  if (history != (int)L->S.size()) {
    // allocate the new history first, so that a failure leaves the old one intact
    std::vector<void*> S(history, nullptr), Y(history, nullptr);
    bool ok = true;
    for (int i = 0; i < history && ok; ++i)
      ok = hipMalloc(&S[i], L->n * L->esz) == hipSuccess && hipMalloc(&Y[i], L->n * L->esz) == hipSuccess;
    if (!ok) {
      for (void* p : S)
        if (p) (void)hipFree(p);
      for (void* p : Y)
        if (p) (void)hipFree(p);
      return set_error(FE_ENOMEM, "L-BFGS history allocation failed");
    }
    for (void* p : L->S)
      if (p) (void)hipFree(p);
    for (void* p : L->Y)
      if (p) (void)hipFree(p);
    L->S.swap(S);
    L->Y.swap(Y);
  }
  L->lr = lr;
  L->history = history;
  L->max_iter = max_iter;
  L->max_eval = max_iter * 5 / 4;
  L->tol_grad = tolerance_grad;
  L->tol_change = tolerance_change;
  L->n_iter = 0;
  L->hist_len = 0;
  L->rho.clear();
  L->pgS.clear();
  L->pgY.clear();
  L->SY.assign((size_t)history * history, 0.0);
  L->YY.assign((size_t)history * history, 0.0);
  return FE_OK;
}

int fe_l2_load(fe_l2* L, const void* u) {
  g_last_error.clear();
  if (!L) return set_error(FE_EINVAL, "flow is NULL");
  if (!u) return set_error(FE_EINVAL, "u is NULL");
  DeviceGuard dg(L->ctx->device);
  const int rc = l2_box_copy_any(L, u, L->x, 1);
  if (rc) return rc;
  L->n_iter = 0;
  L->hist_len = 0;
  L->rho.clear();
  L->pgS.clear();
  L->pgY.clear();
  return FE_OK;
}

int fe_l2_store(fe_l2* L, void* u) {
  g_last_error.clear();
  if (!L) return set_error(FE_EINVAL, "flow is NULL");
  if (!u) return set_error(FE_EINVAL, "u is NULL");
  DeviceGuard dg(L->ctx->device);
  return l2_box_copy_any(L, L->x, u, 0);
}

int fe_l2_energy_grad(fe_l2* L, const void* u, void* g, double* energy) {
  int rc = fe_l2_load(L, u);
  if (rc) return rc;
  DeviceGuard dg(L->ctx->device);
  double E = 0.0;
  rc = L->ctx->grid.dtype == FE_F32 ? l2_eval<float>(L, E, static_cast<float*>(g))
                                    : l2_eval<double>(L, E, static_cast<double*>(g));
  if (rc) return rc;
  if (energy) *energy = E;
  return FE_OK;
}

int fe_l2_step(fe_l2* L, int nsteps, double* energies) {
  g_last_error.clear();
  if (!L) return set_error(FE_EINVAL, "flow is NULL");
  if (nsteps < 0) return set_error(FE_EINVAL, "nsteps must be >= 0");
  DeviceGuard dg(L->ctx->device);
  for (int k = 0; k < nsteps; ++k) {
    double E = 0.0;
    const int rc = L->ctx->grid.dtype == FE_F32 ? l2_step<float>(L, E) : l2_step<double>(L, E);
    if (rc) return rc;
    if (energies) energies[k] = E;
  }
  return FE_OK;
}

int fe_l2_set_stream(fe_l2* L, void* stream) {
  g_last_error.clear();
  if (!L) return set_error(FE_EINVAL, "flow is NULL");
  return fe_set_stream(L->ctx, stream);
}

void fe_l2_destroy(fe_l2* L) { l2_free(L); }

}  // extern "C"
