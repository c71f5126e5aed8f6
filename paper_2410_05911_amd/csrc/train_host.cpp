// Host side of the quantisation-aware training step (Section 6, second phase): validation, the
// Tanner-graph lists on the device, the workspace layout and the launch sequence of one forward
// and backward pass.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include <hip/hip_runtime.h>

#include "../../include/aecct.h"
#include "aecct_internal.h"

struct aecct_trainer {
  int n, m, L, d, N, heads, hf, dff, dh;
  float ln_eps, aap_eps;
  int device, cu_count;
  size_t lds_max;
  void *blk;
  const int32_t *chk_ptr, *chk_idx, *m1_ptr, *m1_idx, *m2_ptr, *m2_idx;
};

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Workspace regions (float offsets) for `batch` words.
struct TrainWs {
  // per layer, for the backward: codes (int8) and scales alpha / 127 of every map's input, Q | K | V, the
  // attention's output and log-sum-exp, both normalised rows with their 1 / sigma, the ReLU mask
  struct Layer { size_t xq, tx, qkv, lse, o, oq, to, xn1, rho1, x1q, t1, mask, gq, tg, xn2, rho2; };
  std::vector<Layer> layer;
  size_t t, x, z, fo, df, dz, tw, tpk, gam, sc, lpart, lnpart, dx, dr2, dr1, dg, dO, dqkv, part;
  size_t part_floats, total_bytes;
};

size_t weight_floats(const aecct_trainer &T) {
  return (size_t)T.N * (4 * (size_t)T.d * T.d + 2 * (size_t)T.d * T.dff);
}

// d x d tiles of a layer's weight gradients: d_ff / d = 4 of each feed-forward map, the output map, three of Q | K | V
constexpr int kDwTiles = 12;

TrainWs train_ws(const aecct_trainer &T, int64_t batch) {
  const size_t R = (size_t)batch * T.L, d = T.d, dff = T.dff, h = T.heads;
  TrainWs w{};
  size_t off = 0;   // bytes
  auto take = [&](size_t floats) { size_t o = off; off = align_up(off + 4 * floats); return o / 4; };
  auto bytes = [&](size_t n) { return take((n + 3) / 4); };
  w.layer.resize(T.N);
  for (auto &q : w.layer) {
    q.xq = bytes(R * d);
    q.tx = take(R);
    q.qkv = take(R * 3 * d);
    q.lse = take(R * h);
    q.o = take(R * d);
    q.oq = bytes(R * d);
    q.to = take(R);
    q.xn1 = take(R * d);
    q.rho1 = take(R);
    q.x1q = bytes(R * d);
    q.t1 = take(R);
    q.mask = bytes(R * dff / 8);
    q.gq = bytes(R * dff);
    q.tg = take(R);
    q.xn2 = take(R * d);
    q.rho2 = take(R);
  }
  w.t = take(R);
  w.x = take(R * d);
  w.z = take(R);
  w.fo = take((size_t)batch * T.n);
  w.df = take((size_t)batch * T.n);
  w.dz = take(R);
  w.tw = take(weight_floats(T));
  w.tpk = take(weight_floats(T));   // every ternary matrix as int8 fragments, then T^T's
  w.gam = take((size_t)T.N * 6);
  w.sc = take((size_t)T.N * 6);
  w.lpart = take(((size_t)batch * T.n + 255) / 256 + 1);
  w.lnpart = take((size_t)aecct::train_bwd_blocks((int64_t)R, T.cu_count) * 4 * d);
  w.dx = take(R * d);
  w.dr2 = take(R * d);
  w.dr1 = take(R * d);
  w.dg = take(R * dff);
  w.dO = take(R * d);
  w.dqkv = take(R * 3 * d);
  w.part_floats = std::max<size_t>(size_t(1) << 22, 4 * std::max<size_t>((size_t)T.L * T.n, d * dff));
  w.part_floats = std::max<size_t>(
      w.part_floats, (size_t)aecct::train_dw_splits((int)d, (int64_t)R, kDwTiles, T.cu_count) * kDwTiles * d * (d + 1));
  w.part = take(w.part_floats);
  w.total_bytes = off + kAlign;   // the regions start at the workspace's first multiple of kAlign
  return w;
}

inline aecct_status st(hipError_t e) { return e == hipSuccess ? AECCT_OK : AECCT_ERR_DEVICE; }

}  // namespace

extern "C" {

aecct_status aecct_train_create(const uint8_t *H, int32_t m, int32_t n, int32_t d, int32_t n_layers, int32_t heads,
                                const aecct_options *opt, float aap_eps, aecct_trainer **out) {
  if (!out) return AECCT_ERR_INVALID_ARG;
  *out = nullptr;
  if (!H || m <= 0 || n <= 0 || d <= 0 || n_layers <= 0 || heads <= 0 || d % heads) return AECCT_ERR_INVALID_ARG;
  if (!std::isfinite(aap_eps) || aap_eps < 0.0f) return AECCT_ERR_INVALID_ARG;
  const int hf = (opt && opt->first_ring_heads >= 0) ? opt->first_ring_heads : heads / 2;
  if ((opt && opt->first_ring_heads < -1) || hf > heads) return AECCT_ERR_INVALID_ARG;
  const int dff = (opt && opt->d_ff > 0) ? opt->d_ff : 4 * d;
  if (opt && (opt->d_ff < -1 || !std::isfinite(opt->ln_eps))) return AECCT_ERR_INVALID_ARG;
  const float eps = (opt && opt->ln_eps > 0.0f) ? opt->ln_eps : 1e-5f;
  const int attention = opt ? opt->attention : AECCT_ATTN_HPSA;
  if (attention != AECCT_ATTN_HPSA && attention != AECCT_ATTN_CASA) return AECCT_ERR_INVALID_ARG;
  const int act_mode = opt ? opt->act_scale_mode : AECCT_ACT_SCALE_TOKEN;
  if (act_mode != AECCT_ACT_SCALE_TOKEN && act_mode != AECCT_ACT_SCALE_WORD) return AECCT_ERR_INVALID_ARG;
  const int64_t L64 = (int64_t)n + m;
  std::vector<int> rowdeg(m, 0), coldeg(n, 0);
  for (int j = 0; j < m; ++j)
    for (int i = 0; i < n; ++i) {
      const uint8_t v = H[(size_t)j * n + i];
      if (v > 1) return AECCT_ERR_INVALID_ARG;
      if (v) { ++rowdeg[j]; ++coldeg[i]; }
    }
  for (int j = 0; j < m; ++j) if (!rowdeg[j]) return AECCT_ERR_INVALID_ARG;
  for (int i = 0; i < n; ++i) if (!coldeg[i]) return AECCT_ERR_INVALID_ARG;
  const int dh = d / heads;
  if (!(d == 32 || d == 64 || d == 128) || !(dh == 4 || dh == 8 || dh == 16) || dff != 4 * d || L64 > 4096 ||
      n_layers > aecct::kMaxLayers || act_mode != AECCT_ACT_SCALE_TOKEN)
    return AECCT_ERR_UNSUPPORTED;
  const int L = (int)L64;

  aecct::TannerLists TL = aecct::tanner_lists(H, m, n);
  int hf_eff = hf;
  if (attention == AECCT_ATTN_CASA) {
    aecct::casa_union(TL);
    hf_eff = 0;
  }
  const std::vector<int32_t> *parts[6] = {&TL.chk_ptr, &TL.chk_idx, &TL.m1_ptr, &TL.m1_idx, &TL.m2_ptr, &TL.m2_idx};
  size_t offs[6], total = 0;
  for (int k = 0; k < 6; ++k) {
    offs[k] = total;
    total = align_up(total + 4 * std::max<size_t>(1, parts[k]->size()));
  }
  std::vector<unsigned char> img(total, 0);
  for (int k = 0; k < 6; ++k)
    if (!parts[k]->empty()) std::memcpy(img.data() + offs[k], parts[k]->data(), 4 * parts[k]->size());

  int dev = 0, cus = 0, lds = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || cus <= 0 ||
      lds <= 0 || aecct::train_set_attributes((size_t)lds) != hipSuccess)
    return AECCT_ERR_DEVICE;
  void *blk = nullptr;
  hipError_t e = hipMalloc(&blk, total);
  if (e != hipSuccess) return e == hipErrorOutOfMemory ? AECCT_ERR_OUT_OF_MEMORY : AECCT_ERR_DEVICE;
  if (hipMemcpy(blk, img.data(), total, hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipFree(blk);
    return AECCT_ERR_DEVICE;
  }
  aecct_trainer *tr = new (std::nothrow) aecct_trainer;
  if (!tr) {
    (void)hipFree(blk);
    return AECCT_ERR_OUT_OF_MEMORY;
  }
  unsigned char *b = (unsigned char *)blk;
  *tr = aecct_trainer{n, m, L, d, n_layers, heads, hf_eff, dff, dh, eps, aap_eps, dev, cus, (size_t)lds, blk,
                      (const int32_t *)(b + offs[0]), (const int32_t *)(b + offs[1]), (const int32_t *)(b + offs[2]),
                      (const int32_t *)(b + offs[3]), (const int32_t *)(b + offs[4]), (const int32_t *)(b + offs[5])};
  *out = tr;
  return AECCT_OK;
}

void aecct_train_destroy(aecct_trainer *tr) {
  if (!tr) return;
  if (tr->blk) (void)hipFree(tr->blk);
  delete tr;
}

aecct_status aecct_train_workspace_size(const aecct_trainer *tr, int64_t batch, size_t *bytes) {
  if (!tr || !bytes || batch < 0) return AECCT_ERR_INVALID_ARG;
  *bytes = batch == 0 ? 0 : train_ws(*tr, batch).total_bytes;
  return AECCT_OK;
}

aecct_status aecct_train_grad(const aecct_trainer *tr, const aecct_train_params *p, const float *y, const float *xs,
                              int64_t batch, const aecct_train_grads *g, float *loss, void *workspace,
                              size_t workspace_bytes, void *stream) {
  using namespace aecct;
  if (!tr || !p || !g || !loss || batch <= 0 || !y) return AECCT_ERR_INVALID_ARG;
  const float *pw[6] = {p->w_q, p->w_k, p->w_v, p->w_o, p->w_ff1, p->w_ff2};
  const float *pb[6] = {p->b_q, p->b_k, p->b_v, p->b_o, p->b_ff1, p->b_ff2};
  float *gw[6] = {g->w_q, g->w_k, g->w_v, g->w_o, g->w_ff1, g->w_ff2};
  float *gb[6] = {g->b_q, g->b_k, g->b_v, g->b_o, g->b_ff1, g->b_ff2};
  for (int k = 0; k < 6; ++k)
    if (!pw[k] || !pb[k] || !gw[k] || !gb[k]) return AECCT_ERR_INVALID_ARG;
  if (!p->embed || !p->delta || !p->ln1_g || !p->ln1_b || !p->ln2_g || !p->ln2_b || !p->head_w1 || !p->head_b1 ||
      !p->head_wo || !p->head_bo || !g->embed || !g->delta || !g->ln1_g || !g->ln1_b || !g->ln2_g || !g->ln2_b ||
      !g->head_w1 || !g->head_b1 || !g->head_wo || !g->head_bo)
    return AECCT_ERR_INVALID_ARG;
  int cur = -1;
  if (hipGetDevice(&cur) != hipSuccess) return AECCT_ERR_DEVICE;
  if (cur != tr->device) return AECCT_ERR_INVALID_ARG;
  const TrainWs W = train_ws(*tr, batch);
  if (workspace_bytes < W.total_bytes) return AECCT_ERR_WORKSPACE_TOO_SMALL;
  if (!workspace) return AECCT_ERR_INVALID_ARG;

  const aecct_trainer &T = *tr;
  hipStream_t s = (hipStream_t)stream;
  float *ws = (float *)align_up((size_t)(uintptr_t)workspace);
  const int64_t R = batch * T.L, B = batch;
  const int d = T.d, dff = T.dff, N = T.N;
  const int64_t K_in[6] = {d, d, d, d, d, dff}, K_out[6] = {d, d, d, d, dff, d};
  const size_t PF = W.part_floats;
  float *part = ws + W.part;
  auto wofs = [&](int l, int k) {   // float offset of matrix k of layer l inside a [N][in][out] tensor
    return (size_t)l * K_in[k] * K_out[k];
  };
  // the ternary copies: per layer the six maps back to back
  auto tmat = [&](int l, int k) {
    size_t o = W.tw;
    for (int ll = 0; ll < l; ++ll)
      for (int kk = 0; kk < 6; ++kk) o += K_in[kk] * K_out[kk];
    for (int kk = 0; kk < k; ++kk) o += K_in[kk] * K_out[kk];
    return ws + o;
  };
  float *gam = ws + W.gam, *sc = ws + W.sc;
  // a ternary matrix's packed forms: int8 fragments (the forward maps), then T^T for the input gradients,
  // as bf16 fragments (query, key, value) or selector bytes (the other three)
  auto tpk = [&](int l, int k, bool trans) {
    size_t o = 0;   // in bytes
    for (int ll = 0; ll < l; ++ll)
      for (int kk = 0; kk < 6; ++kk) o += 4 * (size_t)K_in[kk] * K_out[kk];
    for (int kk = 0; kk < k; ++kk) o += 4 * (size_t)K_in[kk] * K_out[kk];
    if (trans) o += (size_t)K_in[k] * K_out[k];
    return (void *)((unsigned char *)(ws + W.tpk) + o);
  };
  hipError_t e = hipSuccess;
#define AECCT_TRY(call)              \
  do {                               \
    e = (call);                      \
    if (e != hipSuccess) return st(e); \
  } while (0)

  // ---- forward -------------------------------------------------------------------------------
  // Eq. 1 of every layer's six matrices first (they depend on the weights only), a launch per
  // ten layers
  for (int l0 = 0; l0 < N; l0 += kTrainJobsPerLaunch / 6) {
    TrainAapJobs jobs{};
    for (int l = l0; l < std::min(N, l0 + kTrainJobsPerLaunch / 6); ++l)
      for (int k = 0; k < 6; ++k)
        jobs.j[jobs.n++] = TrainAapJob{pw[k] + wofs(l, k), tmat(l, k), K_in[k] * K_out[k], p->delta + 6 * l + k,
                                       gam + 6 * l + k, sc + 6 * l + k};
    AECCT_TRY(train_aap(jobs, T.aap_eps, s));
  }
  for (int l0 = 0; l0 < N; l0 += kTrainJobsPerLaunch / 12) {   // both layouts of every matrix, a launch per five layers
    TernPackJobs pj{};
    for (int l = l0; l < std::min(N, l0 + kTrainJobsPerLaunch / 12); ++l)
      for (int k = 0; k < 6; ++k) {
        pj.j[pj.n++] = TernPackJob{tmat(l, k), (int)K_in[k], (int)K_out[k], k < 4 ? kTernI8 : kTernI8Hidden, tpk(l, k, false)};
        pj.j[pj.n++] = TernPackJob{tmat(l, k), (int)K_in[k], (int)K_out[k], k < 3 ? kTernBf16T : kTernSelT, tpk(l, k, true)};
      }
    AECCT_TRY(train_pack_tern(pj, s));
  }
  auto i8 = [&](size_t o) { return (int8_t *)(ws + o); };
  float *X = ws + W.x, *tv = ws + W.t;
  AECCT_TRY(train_embed(y, R, T.n, T.L, d, T.chk_ptr, T.chk_idx, p->embed, p->pos, X, tv, i8(W.layer[0].xq),
                        ws + W.layer[0].tx, s));
  auto gemm = [&](bool ta, bool tb, const float *A, int64_t lda, const float *Bm, int64_t ldb, float *C, int64_t ldc,
                  int64_t M, int64_t Nn, int64_t K, const float *bias) {
    return train_gemm(ta, tb, A, lda, Bm, ldb, C, ldc, M, Nn, K, bias, part, (int64_t)PF, T.cu_count, s);
  };
  for (int l = 0; l < N; ++l) {
    const TrainWs::Layer &q = W.layer[l];
    TrainQkv qa{i8(q.xq), ws + q.tx, {}, {}, {}, ws + q.qkv, R};
    for (int k = 0; k < 3; ++k) {
      qa.f[k] = (const uint64_t *)tpk(l, k, false);
      qa.s[k] = sc + 6 * l + k;
      qa.b[k] = pb[k] + (size_t)l * d;
    }
    AECCT_TRY(train_qkv(d, qa, T.cu_count, T.lds_max, s));
    TrainAttn at{ws + q.qkv, R, T.L, d, T.heads, T.hf, T.m1_ptr, T.m1_idx, T.m2_ptr, T.m2_idx, ws + q.o, ws + q.lse,
                 nullptr, nullptr, nullptr};
    AECCT_TRY(train_attention(false, T.dh, at, T.cu_count, T.lds_max, s));
    TrainBlock tb{};
    tb.o = ws + q.o;
    tb.res = l ? ws + W.layer[l - 1].xn2 : X;
    if (l) {
      tb.res_g = p->ln2_g + (size_t)(l - 1) * d;
      tb.res_b = p->ln2_b + (size_t)(l - 1) * d;
    }
    tb.fo = (const uint64_t *)tpk(l, 3, false);
    tb.f1 = (const uint64_t *)tpk(l, 4, false);
    tb.f2 = (const uint64_t *)tpk(l, 5, false);
    tb.so = sc + 6 * l + 3;
    tb.s1 = sc + 6 * l + 4;
    tb.s2 = sc + 6 * l + 5;
    tb.bo = pb[3] + (size_t)l * d;
    tb.b1 = pb[4] + (size_t)l * dff;
    tb.b2 = pb[5] + (size_t)l * d;
    tb.g1 = p->ln1_g + (size_t)l * d;
    tb.be1 = p->ln1_b + (size_t)l * d;
    tb.g2 = p->ln2_g + (size_t)l * d;
    tb.be2 = p->ln2_b + (size_t)l * d;
    tb.eps = T.ln_eps;
    tb.rows = R;
    tb.oq = i8(q.oq);
    tb.to = ws + q.to;
    tb.xn1 = ws + q.xn1;
    tb.rho1 = ws + q.rho1;
    tb.x1q = i8(q.x1q);
    tb.t1 = ws + q.t1;
    tb.mask = (uint32_t *)(ws + q.mask);
    tb.gq = i8(q.gq);
    tb.tg = ws + q.tg;
    tb.xn2 = ws + q.xn2;
    tb.rho2 = ws + q.rho2;
    if (l + 1 < N) {
      tb.xq = i8(W.layer[l + 1].xq);
      tb.tx = ws + W.layer[l + 1].tx;
    } else {
      tb.x = X;
    }
    AECCT_TRY(train_block(d, tb, T.cu_count, T.lds_max, s));
  }
  // head and loss (Section 3, Section 6)
  float *z = ws + W.z, *fo = ws + W.fo, *df = ws + W.df, *dz = ws + W.dz;
  AECCT_TRY(train_rowdot(X, R, d, p->head_w1, p->head_b1, z, s));
  AECCT_TRY(gemm(false, false, z, T.L, p->head_wo, T.n, fo, T.n, B, T.n, T.L, p->head_bo));
  AECCT_TRY(train_loss(fo, y, xs, B * T.n, df, ws + W.lpart, loss, s));

  // ---- backward ------------------------------------------------------------------------------
  auto colsum = [&](const float *A, int64_t lda, const float *wr, int64_t rows, int C, float *o) {
    return train_colsum(A, lda, wr, rows, C, o, part, (int64_t)PF, s);
  };
  AECCT_TRY(colsum(df, T.n, nullptr, B, T.n, g->head_bo));
  AECCT_TRY(gemm(true, false, z, T.L, df, T.n, g->head_wo, T.n, T.L, T.n, B, nullptr));
  AECCT_TRY(gemm(false, true, df, T.n, p->head_wo, T.n, dz, T.L, B, T.L, T.n, nullptr));
  AECCT_TRY(colsum(dz, 1, nullptr, R, 1, g->head_b1));
  AECCT_TRY(colsum(X, d, dz, R, d, g->head_w1));
  float *dX = ws + W.dx, *dR2 = ws + W.dr2, *dR1 = ws + W.dr1, *dG = ws + W.dg, *dO = ws + W.dO,
        *dQKV = ws + W.dqkv;
  AECCT_TRY(train_outer(dz, R, p->head_w1, d, dX, s));
  for (int l = N - 1; l >= 0; --l) {
    const TrainWs::Layer &q = W.layer[l];
    const size_t ld_ = (size_t)l * d;
    // LN2, second feed-forward map, ReLU (the Eq. 2 code of the hidden row passes straight through), first
    // map, LN1, output map
    TrainBwd bw{dX, ws + q.xn2, ws + q.rho2, ws + q.xn1, ws + q.rho1, p->ln2_g + ld_, p->ln1_g + ld_,
                (const uint32_t *)(ws + q.mask), (const uint64_t *)tpk(l, 5, true), (const uint64_t *)tpk(l, 4, true),
                (const uint64_t *)tpk(l, 3, true), sc + 6 * l + 5, sc + 6 * l + 4, sc + 6 * l + 3, dR2, dG, dR1, dO,
                ws + W.lnpart, R};
    AECCT_TRY(train_bwd(d, bw, T.cu_count, s));
    // attention, then the query, key and value maps: one product over their packed gradient
    // (dX, read by train_bwd and written again by that product, lends its space to Dv)
    TrainAttn at{ws + q.qkv, R, T.L, d, T.heads, T.hf, T.m1_ptr, T.m1_idx, T.m2_ptr, T.m2_idx, ws + q.o, ws + q.lse,
                 dO, dQKV, dX};
    AECCT_TRY(train_attention(true, T.dh, at, T.cu_count, T.lds_max, s));
    const void *fq[3] = {tpk(l, 0, true), tpk(l, 1, true), tpk(l, 2, true)};
    const float *sq[3] = {sc + 6 * l, sc + 6 * l + 1, sc + 6 * l + 2};
    AECCT_TRY(train_gemm_tern(dQKV, 3 * d, fq, 3, d, sq, dR1, dX, d, R, d, s));
    // every weight and bias gradient of the layer
    TrainDwJobs dw{};
    dw.rows = R;
    dw.n = kTrainDwJobs;
    dw.lnpart = ws + W.lnpart;
    dw.ln_blocks = train_bwd_blocks(R, T.cu_count);
    float *const lng[4] = {g->ln2_g + ld_, g->ln2_b + ld_, g->ln1_g + ld_, g->ln1_b + ld_};
    for (int k = 0; k < 4; ++k) dw.ln[k] = lng[k];
    dw.j[0] = TrainDwJob{i8(q.gq), ws + q.tg, dR2, d, dff, d, d, {gw[5] + wofs(l, 5)}, {gb[5] + ld_}};
    dw.j[1] = TrainDwJob{i8(q.x1q), ws + q.t1, dG, dff, d, dff, dff, {gw[4] + wofs(l, 4)}, {gb[4] + (size_t)l * dff}};
    dw.j[2] = TrainDwJob{i8(q.oq), ws + q.to, dR1, d, d, d, d, {gw[3] + wofs(l, 3)}, {gb[3] + ld_}};
    dw.j[3] = TrainDwJob{i8(q.xq), ws + q.tx, dQKV, 3 * d, d, 3 * d, d,
                         {gw[0] + wofs(l, 0), gw[1] + wofs(l, 1), gw[2] + wofs(l, 2)}, {gb[0] + ld_, gb[1] + ld_, gb[2] + ld_}};
    AECCT_TRY(train_weight_grads(d, dw, T.cu_count, part, (int64_t)PF, s));
  }
  // the straight-through Eq. 1 gradients of every matrix from its G = Xh^T dY (nothing in the
  // backward reads G once it is formed), a launch per ten layers
  for (int l0 = 0; l0 < N; l0 += kTrainJobsPerLaunch / 6) {
    TrainDeltaJobs dj{};
    for (int l = l0; l < std::min(N, l0 + kTrainJobsPerLaunch / 6); ++l)
      for (int k = 0; k < 6; ++k)
        dj.j[dj.n++] = TrainDeltaJob{gw[k] + wofs(l, k), pw[k] + wofs(l, k), tmat(l, k), K_in[k] * K_out[k],
                                     gam + 6 * l + k, sc + 6 * l + k, g->delta + 6 * l + k};
    AECCT_TRY(train_delta_grad(dj, T.aap_eps, s));
  }
  AECCT_TRY(train_embed_grad(tv, dX, B, T.L, d, g->embed, s));
#undef AECCT_TRY
  return AECCT_OK;
}

}  // extern "C"
