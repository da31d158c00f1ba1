// libinterlock: context, routing plan, workspace layout and the C-ABI entry points.
// The step is K x (il_stage_forward, il_head_xent) followed by il_stage_backward_nwise
// for k = K..1.  Gradient streams (one per head, merged where they share their remaining
// route) live in fp32 "slots" ordered by the lowest component they reach.  Under the
// window-sum and far-head routings the streams live at any component occupy adjacent
// slots, i.e. one contiguous stack [cnt*N, d], and every backward GEMM processes all of
// them in a single launch; where the live slots are not adjacent the component's backward
// runs once per contiguous range, and the ranges' parameter gradients add up in fp32.
#include "../../include/interlock.h"
#include "../../include/interlock_test.h"

#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "common.h"
#include "gemm_tile.h"

using namespace il;

namespace {

// ------------------------------------------------------------------ routing plan ----
struct StreamDesc {
  int lo, hi;  // lowest / highest component the stream passes through (1-based)
};
struct Run {                    // a contiguous range of live slots, processed as one stack
  int s0 = 0, cnt = 0;          // slots [s0, s0+cnt)
  int off = 0;                  // streams of earlier runs: where this run's stack starts in the scratch
  float wt[kMaxStreams] = {};   // routing weight of each stream at this component
};
struct CompPlan {
  std::vector<Run> runs;        // usually one; several only when the live slots are not adjacent
  int cnt = 0;                  // live streams in total
  int inject_slot = -1;         // slot head k's fresh gradient joins, -1: head k is not used
  int inject_acc = 0;           // 1: add to the stream already in the slot
  int passes = 0;               // heads whose gradient passes through this component
};
struct Plan {
  int K = 0, nslots = 0, maxcnt = 0, maxlive = 0, maxruns = 1;
  std::vector<StreamDesc> streams;
  std::vector<CompPlan> comp;   // index k-1
};

int route_weights(int K, int n, int route, std::vector<double> &w) {
  if (K < 1 || n < 1 || n > K) return IL_E_ARG;
  w.assign((size_t)K * K, 0.0);
  for (int k = 1; k <= K; ++k) {
    const int far = std::min(k + n - 1, K);
    switch (route) {
      case IL_ROUTE_WINDOW_SUM:
        for (int j = k; j <= far; ++j) w[(k - 1) * K + j - 1] = 1.0;
        break;
      case IL_ROUTE_FAR_HEAD: w[(k - 1) * K + far - 1] = 1.0; break;
      case IL_ROUTE_MEAN_LOCAL_FAR:
        w[(k - 1) * K + k - 1] += 0.5;
        w[(k - 1) * K + far - 1] += 0.5;
        break;
      default: return IL_E_ARG;
    }
  }
  return IL_OK;
}

int build_plan(int K, int n, int route, Plan &p) {
  std::vector<double> w;
  int rc = route_weights(K, n, route, w);
  if (rc) return rc;
  auto W = [&](int k, int j) { return w[(size_t)(k - 1) * K + j - 1]; };
  p = Plan();
  p.K = K;
  p.comp.assign(K, CompPlan());
  std::vector<int> lo(K + 1, 0), group(K + 1, -1);
  for (int j = 1; j <= K; ++j)
    for (int k = 1; k <= j; ++k)
      if (W(k, j) != 0.0) { lo[j] = k; break; }
  // group heads top-down: head j joins a stream created by a higher head when both stop at
  // the same component and carry the same weights over every component they share
  struct G { int lo, hi; };
  std::vector<G> groups;
  for (int j = K; j >= 1; --j) {
    if (!lo[j]) continue;
    int found = -1;
    for (size_t g = 0; g < groups.size() && found < 0; ++g) {
      if (groups[g].lo != lo[j]) continue;
      bool same = true;
      for (int k = lo[j]; k <= j; ++k) same = same && (W(k, j) == W(k, groups[g].hi));
      if (same) found = (int)g;
    }
    if (found < 0) { groups.push_back({lo[j], j}); found = (int)groups.size() - 1; }
    group[j] = found;
  }
  // slots: ascending (lo, hi)
  std::vector<int> order(groups.size());
  for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
  for (size_t a = 0; a < order.size(); ++a)
    for (size_t b = a + 1; b < order.size(); ++b) {
      const G &x = groups[order[a]], &y = groups[order[b]];
      if (y.lo < x.lo || (y.lo == x.lo && y.hi < x.hi)) std::swap(order[a], order[b]);
    }
  std::vector<int> slot_of(groups.size());
  for (size_t s = 0; s < order.size(); ++s) {
    slot_of[order[s]] = (int)s;
    p.streams.push_back({groups[order[s]].lo, groups[order[s]].hi});
  }
  p.nslots = (int)groups.size();
  for (int k = 1; k <= K; ++k) {
    CompPlan &c = p.comp[k - 1];
    bool written = false;
    for (int s = 0; s < p.nslots; ++s) {
      if (!(p.streams[s].lo <= k && k <= p.streams[s].hi)) continue;
      if (c.runs.empty() || c.runs.back().s0 + c.runs.back().cnt != s || c.runs.back().cnt == kMaxStreams) {
        Run r;
        r.s0 = s;
        r.off = c.cnt;
        c.runs.push_back(r);
      }
      const float wt = (float)W(k, p.streams[s].hi);
      Run &q = c.runs.back();
      q.wt[q.cnt] = wt;
      written = written || wt != 0.f;
      ++q.cnt;
      ++c.cnt;
    }
    for (Run &r : c.runs) p.maxcnt = std::max(p.maxcnt, r.cnt);
    p.maxlive = std::max(p.maxlive, c.cnt);
    p.maxruns = std::max(p.maxruns, (int)c.runs.size());
    if (!written) return IL_E_ARG;  // a component no loss is credited to
    for (int j = k; j <= K; ++j)
      if (lo[j] && lo[j] <= k) ++c.passes;
    if (lo[k]) {
      c.inject_slot = slot_of[group[k]];
      c.inject_acc = (groups[group[k]].hi != k);
    }
  }
  return IL_OK;
}

// ------------------------------------------------------------------ context --------
enum KClass { KC_GEMM_FWD, KC_GEMM_DGRAD, KC_GEMM_WGRAD, KC_GEMM_HEAD, KC_ATTN_FWD, KC_ATTN_BWD, KC_LN_FWD,
              KC_LN_BWD, KC_COLSUM, KC_XENT, KC_MISC, KC_COUNT };
const char *kClassNames[KC_COUNT] = {"gemm_fwd", "gemm_dgrad", "gemm_wgrad", "gemm_head", "attn_fwd", "attn_bwd",
                                     "ln_fwd",   "ln_bwd",     "colsum",     "xent",      "misc"};

struct BlockOff {  // element offsets inside the flat parameter / gradient buffers
  size_t ln1_g, ln1_b, w_qkv, b_qkv, w_o, b_o, ln2_g, ln2_b, w_fc1, b_fc1, w_fc2, b_fc2;
};
struct BlockSave {  // workspace pointers of one block's saved activations
  float *xs, *st1, *lse, *a, *st2;
  char *h1, *qkv, *o, *h2, *u, *gl;
};
struct ProfRec { int cls; bool kernel, bracket; hipEvent_t e0, e1; KernelTimer kt; };

// The tail of a block's backward - stream sums, bias / LayerNorm column sums, weight gradients - reads what
// the data gradients leave behind, and nothing in the backward waits for it.  It is queued and launched on
// the side stream for kGroup blocks at a time: recording an event costs the recording stream about 5 us on
// this part and waiting for one about 6 us (chains of empty kernels: 1.6 us a link, 6.4 with a record,
// 12.6 with a record and a wait), which at d = 512 was a quarter of the backward when every block forked
// three times; and two blocks' eight weight gradients fill a launch better than four.  What the tails read
// lives in a ring of 2 kGroup entries, so that a group's data gradients run while the previous group's
// tails do.
constexpr int kGroup = 2, kRing = 2 * kGroup;
struct RingEntry {
  char *Ga;           // gradient stream above the MLP as a GEMM operand, [nslots][N, d]
  char *Gb;           // ... above the attention, [live streams][N, d]
  char *DU, *DQKV;    // [live streams][N, m] and [N, 3d]: gradients at the MLP's hidden layer and at Q|K|V
  float *ln[2];       // LayerNorm 2's and 1's first-stage column sums
  // What the LayerNorm that makes Ga (Gb) leaves with it: the weighted sum over the streams [N, d] (where there
  // are several) and the first stage of its column sums.
  char *sum[2]; float *sum_cols[2];
  char *sum_du; float *sum_du_cols;  // the same of DU, left by the product that makes it
};
// A block's linear outputs in the order FC2, FC1, attention output projection, QKV: the streams' weighted sum as
// an operand, and its column sums' first stage, where the kernel that made the streams has left them.
struct Summed { const void *y; const float *cols; int nblk; };
struct Tail {         // one queued tail
  const BlockOff *b; const BlockSave *s; const RingEntry *r;
  const std::vector<Run> *runs;  // (outlives the launch)
  int ln_blocks;                 // partial sums per LayerNorm
  Summed done[4];                // cols == nullptr: not summed yet
};
// The streams of a range that carry weight: how many, the first, and whether that one is their sum already.
struct Weighted { int n, first; bool plain; };
Weighted weighted(const Run &r) {
  Weighted w{0, 0, false};
  for (int i = r.cnt - 1; i >= 0; --i)
    if (r.wt[i] != 0.f) { ++w.n; w.first = i; }
  w.plain = w.n == 1 && r.wt[w.first] == 1.f;
  return w;
}
// the part-th range that carries weighted streams, nullptr beyond the last
const Run *weighted_run(const std::vector<Run> &runs, int part) {
  for (const Run &r : runs)
    if (weighted(r).n && part-- == 0) return &r;
  return nullptr;
}

}  // namespace

struct il_ctx {
  il_config cfg;
  Plan plan;
  int N, d, m, V, H, dh, L, K, eb, Lh;
  hipStream_t stream;
  std::vector<BlockOff> boff;      // K*L
  std::vector<size_t> hoff;        // K
  std::vector<BlockSave> save;     // K*L
  std::vector<BlockOff> hboff;     // K*Lh: the heads' own blocks
  std::vector<BlockSave> hsave;    // K*Lh
  float *hy = nullptr;             // output of a head's last block, fp32 [N,d]
  int accumulate = 0;              // micro-batching: add into grads instead of overwriting
  float grad_scale = 1.f;          // ... and scale every gradient (applied to dlogits)
  bool tail_inline = false;        // block_backward is running on the side stream already (inside a head)
  float *G;                        // stream slots [nslots][N,d]
  RingEntry ring[kRing];
  int pos = 0;                     // ring entry of the next block
  Summed above = {};               // what was left with the next block's Ga
  char *DH; float *dsum, *skws; size_t skws_floats;
  Tail tails[kGroup]; int ntails = 0;
  float *partials[kGroup][4];      // bias partials of the queued tails
  hipEvent_t ev_ready = nullptr, ev_tail[2] = {nullptr, nullptr};
  char tail_pending[2] = {0, 0};   // half of the ring: its tails were launched and nobody has waited for them
  int tail_last = 0;               // the half launched last
  char *xb, *Z; float *rowloss, *dxh, *hstats = nullptr, *hztgt = nullptr;
  int Nc;
  std::vector<char> fwd_done, head_done, bwd_done;
  // heads run on a side stream, concurrently with the next component's forward
  hipStream_t main_stream = nullptr, side = nullptr;
  hipEvent_t ev_fork = nullptr;
  std::vector<hipEvent_t> ev_head;   // K: head k finished (side stream)
  std::vector<char> head_pending;    // main stream has not yet waited for ev_head[k]
  // profiling
  std::vector<ProfRec> recs; size_t nrec = 0;
  double flops[KC_COUNT] = {}, bytes[KC_COUNT] = {};
};

namespace {

struct Carver {
  char *base; size_t off = 0;
  explicit Carver(void *b) : base((char *)b) {}
  void *take(size_t bytes) {
    void *p = base ? base + off : nullptr;
    off += (bytes + 255) & ~(size_t)255;
    return p;
  }
};

size_t layout_params(il_ctx *c) {
  const size_t d = c->d, m = c->m;
  size_t o = 0;
  c->boff.resize((size_t)c->K * c->L);
  for (auto &b : c->boff) {
    b.ln1_g = o; o += d; b.ln1_b = o; o += d; b.w_qkv = o; o += 3 * d * d; b.b_qkv = o; o += 3 * d;
    b.w_o = o; o += d * d; b.b_o = o; o += d; b.ln2_g = o; o += d; b.ln2_b = o; o += d;
    b.w_fc1 = o; o += d * m; b.b_fc1 = o; o += m; b.w_fc2 = o; o += m * d; b.b_fc2 = o; o += d;
  }
  auto lay = [&](BlockOff &b) {
    b.ln1_g = o; o += d; b.ln1_b = o; o += d; b.w_qkv = o; o += 3 * d * d; b.b_qkv = o; o += 3 * d;
    b.w_o = o; o += d * d; b.b_o = o; o += d; b.ln2_g = o; o += d; b.ln2_b = o; o += d;
    b.w_fc1 = o; o += d * m; b.b_fc1 = o; o += m; b.w_fc2 = o; o += m * d; b.b_fc2 = o; o += d;
  };
  c->hoff.resize(c->K);
  c->hboff.resize((size_t)c->K * c->Lh);
  for (int k = 0; k < c->K; ++k) {
    for (int l = 0; l < c->Lh; ++l) lay(c->hboff[(size_t)k * c->Lh + l]);
    c->hoff[k] = o; o += d * (size_t)c->V;
  }
  return o;
}

// bf16: (max, sum-exp) per row of the logits tile and per group of kStatGroup vocabulary columns
size_t head_stats_bytes(const il_ctx *c, int rows) {
  return c->eb == 2 ? (size_t)rows * ((c->V + kStatGroup - 1) / kStatGroup) * 2 * 4 : 0;
}

// The split of the head's dx = dz W^T (few output tiles, K = vocabulary) over `rows` token rows, within a
// scratch of `floats`, and the scratch it needs.
SplitPlan head_split(const il_ctx *c, int rows, size_t floats) {
  if (c->d % 4) return SplitPlan{1, 0};
  return gemm_split_plan(c->cfg.dtype, rows, c->d, c->V, floats);
}
size_t head_split_floats(const il_ctx *c, int rows, size_t floats) {
  const int sp = head_split(c, rows, floats).splits;
  return sp > 1 ? (size_t)sp * rows * c->d : 0;
}

// The FC2 data gradient of these ranges leaves DU's sum of streams beside it.
bool gelu_sums(const il_ctx *c, const std::vector<Run> &runs) {
  return c->eb == 2 && runs.size() == 1 && gemm_gelu_sum(runs[0].cnt, c->N, c->m);
}

size_t layout_workspace(il_ctx *c, void *base) {
  Carver cv(base);
  const size_t N = c->N, d = c->d, m = c->m, eb = c->eb, H = c->H;
  c->save.resize((size_t)c->K * c->L);
  for (auto &s : c->save) {
    s.xs = (float *)cv.take(N * d * 4); s.st1 = (float *)cv.take(N * 2 * 4);
    s.h1 = (char *)cv.take(N * d * eb); s.qkv = (char *)cv.take(N * 3 * d * eb);
    s.lse = (float *)cv.take(N * H * 4); s.o = (char *)cv.take(N * d * eb);
    s.a = (float *)cv.take(N * d * 4); s.st2 = (float *)cv.take(N * 2 * 4);
    s.h2 = (char *)cv.take(N * d * eb); s.u = (char *)cv.take(N * m * eb); s.gl = (char *)cv.take(N * m * eb);
  }
  c->hsave.resize((size_t)c->K * c->Lh);
  for (auto &s : c->hsave) {
    s.xs = (float *)cv.take(N * d * 4); s.st1 = (float *)cv.take(N * 2 * 4);
    s.h1 = (char *)cv.take(N * d * eb); s.qkv = (char *)cv.take(N * 3 * d * eb);
    s.lse = (float *)cv.take(N * H * 4); s.o = (char *)cv.take(N * d * eb);
    s.a = (float *)cv.take(N * d * 4); s.st2 = (float *)cv.take(N * 2 * 4);
    s.h2 = (char *)cv.take(N * d * eb); s.u = (char *)cv.take(N * m * eb); s.gl = (char *)cv.take(N * m * eb);
  }
  if (c->Lh) c->hy = (float *)cv.take(N * d * 4);
  // (one more stream slot carries a head's gradient through its own blocks)
  const size_t ns = c->plan.nslots + (c->Lh ? 1 : 0), S = (size_t)std::max(c->plan.maxcnt, 1) * N;
  const size_t live = (size_t)std::max(c->plan.maxlive, 1) * N;
  // What LayerNorm backward (ln_) and the FC2 data gradient (du_) leave beside the streams, by the components' ranges: column
  // sums of their sum, and the sum itself where the streams are not it already.  (A head's own blocks: one stream.)
  const bool ln = ln_backward_sums(c->N, c->d);
  bool ln_cols = ln && c->Lh, ln_sums = false, du_cols = c->Lh && c->eb == 2 && gemm_gelu_sum(1, c->N, c->m), du_sums = false;
  for (const CompPlan &k : c->plan.comp) {
    if (k.runs.size() != 1) continue;
    const bool several = !weighted(k.runs[0]).plain, gelu = gelu_sums(c, k.runs);
    ln_cols = ln_cols || ln;
    ln_sums = ln_sums || (ln && several);
    du_cols = du_cols || gelu;
    du_sums = du_sums || (gelu && several);
  }
  c->G = (float *)cv.take(ns * N * d * 4);
  for (RingEntry &r : c->ring) {
    r.Ga = (char *)cv.take(ns * N * d * eb);
    r.Gb = (char *)cv.take(live * d * eb);
    r.DU = (char *)cv.take(live * m * eb);
    r.DQKV = (char *)cv.take(live * 3 * d * eb);
    for (float *&p : r.ln) p = (float *)cv.take((size_t)c->plan.maxruns * ln_backward_max_blocks() * 2 * d * 4);
    for (int i = 0; i < 2; ++i) {
      const bool next = i || c->L > 1 || c->Lh > 1;  // (LayerNorm 1 leaves them for the next block down)
      r.sum[i] = (char *)cv.take(ln_sums && next ? N * d * eb : 0);
      r.sum_cols[i] = (float *)cv.take(ln_cols && next ? (size_t)ln_backward_max_blocks() * d * 4 : 0);
    }
    r.sum_du = (char *)cv.take(du_sums ? N * m * eb : 0);
    r.sum_du_cols = (float *)cv.take(du_cols ? (N + 63) / 64 * m * 4 : 0);
  }
  c->DH = (char *)cv.take(S * d * eb);
  c->dsum = (float *)cv.take(S * std::max(H, d / 32) * 4);
  const size_t wide[4] = {d, m, d, 3 * d};  // outputs of FC2, FC1, the attention output projection, QKV
  for (int p = 0; p < kGroup; ++p)
    for (int i = 0; i < 4; ++i) c->partials[p][i] = (float *)cv.take((size_t)colsum_max_blocks() * wide[i] * 4);
  c->skws_floats = head_split_floats(c, c->Nc, (size_t)-1);
  c->skws = (float *)cv.take(c->skws_floats * 4);
  c->xb = (char *)cv.take(N * d * eb);
  c->Z = (char *)cv.take((size_t)c->Nc * c->V * eb);
  c->rowloss = (float *)cv.take(N * 4);
  c->hstats = (float *)cv.take(head_stats_bytes(c, c->Nc));
  c->hztgt = (float *)cv.take(eb == 2 ? (size_t)c->Nc * 4 : 0);
  c->dxh = (float *)cv.take((size_t)c->K * N * d * 4);
  return cv.off;
}

// --- launch bookkeeping -----------------------------------------------------------------
struct Scope {  // brackets a group of launches with events when profiling is on
  il_ctx *c; int cls; ProfRec *r = nullptr;
  Scope(il_ctx *ctx, int cls_, double flops, double bytes) : c(ctx), cls(cls_) {
    if (!c->cfg.profile) return;
    c->flops[cls] += flops; c->bytes[cls] += bytes;
    // mode 2: the step runs as it does unprofiled (two streams); only the bf16 GEMM dispatches carry timers
    const bool in_step = c->cfg.profile == 2;
    if (in_step && !(c->cfg.dtype == IL_BF16 && cls <= KC_GEMM_HEAD)) return;
    if (c->nrec == c->recs.size()) {
      ProfRec n{};
      if (hipEventCreate(&n.e0) != hipSuccess || hipEventCreate(&n.e1) != hipSuccess ||
          hipEventCreate(&n.kt.start) != hipSuccess || hipEventCreate(&n.kt.stop) != hipSuccess)
        return;
      c->recs.push_back(n);
    }
    r = &c->recs[c->nrec++];
    r->cls = cls;
    // bf16 GEMM scopes also time their MFMA kernel launch by itself (events on the dispatch)
    r->kernel = c->cfg.dtype == IL_BF16 && cls <= KC_GEMM_HEAD;
    r->bracket = !in_step;
    if (r->kernel) gemm_time_next(&r->kt);
    if (r->bracket) hipEventRecord(r->e0, c->stream);
  }
  ~Scope() {
    if (!r) return;
    if (gemm_time_next(nullptr)) r->kernel = false;  // no MFMA GEMM was launched in this scope
    if (r->bracket) hipEventRecord(r->e1, c->stream);
  }
};

#define IL_TRY(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) return IL_E_HIP; } while (0)

hipError_t gemm(il_ctx *c, const GemmArgs &g) {
  return c->cfg.dtype == IL_F32 ? gemm_f32(g, c->stream) : gemm_bf16(g, c->stream);
}

inline const char *P(il_ctx *c, size_t off) { return (const char *)c->cfg.params + off * c->eb; }
inline float *Gr(il_ctx *c, size_t off) { return (float *)c->cfg.grads + off; }

// Algorithmic bytes of one GEMM: both operands once, the output once (and the operands the
// epilogue adds: residual, pre-activation, or the accumulated-into output).
double gemm_bytes(il_ctx *c, const GemmArgs &g) {
  const double eb = c->eb, mn = (double)g.M * g.N;
  double b = ((double)g.M * g.K + (double)g.K * g.N) * eb;
  switch (g.epi) {
    case EPI_BIAS_GELU: b += 2 * mn * eb; break;
    case EPI_BIAS_RES: b += 2 * mn * 4; break;
    case EPI_GELU_BWD:
    case EPI_STORE_DOT: b += 2 * mn * eb; break;
    case EPI_GELU_BWD_SUM: b += (1.0 + 1.0 / g.streams + (g.C2 ? 1.0 / g.streams : 0.0)) * mn * eb; break;
    case EPI_STORE_F32: b += mn * 4; break;
    case EPI_WGRAD: b += mn * 4 * (g.beta ? 2 : 1); break;
    default: b += mn * eb; break;
  }
  return b;
}

GemmArgs base_args() {
  GemmArgs g;
  memset(&g, 0, sizeof(g));
  g.scale = 1.f;
  return g;
}

// y[M,N] = x[M,K] W[K,N] (+ epilogue)
int linear_fwd(il_ctx *c, const void *x, size_t w_off, size_t b_off, int M, int Kd, int Nn, int epi, void *out,
               void *out2, const float *res) {
  GemmArgs g = base_args();
  g.A = x; g.lda = Kd; g.a_kmajor = 0;
  g.B = P(c, w_off); g.ldb = Nn; g.b_kmajor = 1;
  g.M = M; g.N = Nn; g.K = Kd; g.epi = epi; g.C = out; g.C2 = out2; g.ldc = Nn;
  g.bias = P(c, b_off); g.res = res;
  Scope sc(c, KC_GEMM_FWD, 2.0 * M * Nn * Kd, gemm_bytes(c, g));
  IL_TRY(gemm(c, g));
  return IL_OK;
}

// dx[M,Kin] = dy[M,Nout] W[Kin,Nout]^T
int linear_dgrad(il_ctx *c, const void *dy, size_t w_off, int M, int Kin, int Nout, int epi, void *out,
                 const void *aux, int aux_wrap, float *stats = nullptr, void *sum = nullptr, const Run *run = nullptr) {
  GemmArgs g = base_args();
  g.row_stats = stats; g.C2 = sum;
  if (run) {
    g.streams = run->cnt;
    for (int i = 0; i < run->cnt; ++i) g.sum_w[i] = run->wt[i];
  }
  g.A = dy; g.lda = Nout; g.a_kmajor = 0;
  g.B = P(c, w_off); g.ldb = Nout; g.b_kmajor = 0;
  g.M = M; g.N = Kin; g.K = Nout; g.epi = epi; g.C = out; g.ldc = Kin; g.aux = aux; g.aux_wrap = aux_wrap;
  Scope sc(c, KC_GEMM_DGRAD, 2.0 * M * Kin * Nout, gemm_bytes(c, g));
  IL_TRY(gemm(c, g));
  return IL_OK;
}

// The context's second stream (non-blocking, default priority) and the events that tie it to the
// caller's stream; created on first use.  The events order two streams of one device and nobody else looks at them,
// so they leave out the write-back to the host that a recorded event makes (a record 4.6 -> 3.5 us of its stream's time;
// steps 0.3 % faster at d = 1024, 1.2 % at 512, 0.7 to 2.3 % below); what the caller reads on the host is written back where the
// caller waits for its own stream.
constexpr unsigned kEventFlags = hipEventDisableTiming | hipEventDisableSystemFence;
int ensure_side(il_ctx *c) {
  if (c->side) return IL_OK;
  IL_TRY(hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking));
  IL_TRY(hipEventCreateWithFlags(&c->ev_fork, kEventFlags));
  c->ev_head.assign(c->K + 1, nullptr);
  for (int j = 1; j <= c->K; ++j) IL_TRY(hipEventCreateWithFlags(&c->ev_head[j], kEventFlags));
  IL_TRY(hipEventCreateWithFlags(&c->ev_ready, kEventFlags));
  for (int p = 0; p < 2; ++p) IL_TRY(hipEventCreateWithFlags(&c->ev_tail[p], kEventFlags));
  return IL_OK;
}

// The caller's stream waits for every tail still running on the side stream, which is in order.
int join_tails(il_ctx *c) {
  if (c->tail_pending[0] || c->tail_pending[1])
    IL_TRY(hipStreamWaitEvent(c->main_stream, c->ev_tail[c->tail_last], 0));
  c->tail_pending[0] = c->tail_pending[1] = 0;
  return IL_OK;
}

int launch_wgrads(il_ctx *c, const GemmArgs *list, int n) {
  if (n == 0) return IL_OK;
  double fl = 0, by = 0;
  for (int i = 0; i < n; ++i) {
    fl += 2.0 * list[i].M * list[i].N * list[i].K;
    by += gemm_bytes(c, list[i]);
  }
  Scope sc(c, KC_GEMM_WGRAD, fl, by);
  IL_TRY(c->cfg.dtype == IL_F32 ? gemm_f32_batch(list, n, c->stream) : gemm_bf16_batch(list, n, c->stream));
  return IL_OK;
}

int attention_fwd(il_ctx *c, const void *qkv, void *o, float *lse) {
  Scope sc(c, KC_ATTN_FWD, 2.0 * c->cfg.batch * (double)c->cfg.seq * c->cfg.seq * c->d, 0);
  IL_TRY(attention_forward(c->cfg.dtype, qkv, c->cfg.batch, c->cfg.seq, c->H, c->dh, o, lse, c->stream));
  return IL_OK;
}

int attention_bwd(il_ctx *c, const BlockSave &s, const void *d_o, int cnt, void *dqkv) {
  Scope sc(c, KC_ATTN_BWD, 5.0 * cnt * c->cfg.batch * (double)c->cfg.seq * c->cfg.seq * c->d, 0);
  IL_TRY(attention_backward(c->cfg.dtype, s.qkv, s.o, d_o, s.lse, cnt, c->cfg.batch, c->cfg.seq, c->H, c->dh,
                            dqkv, c->dsum, c->stream));
  return IL_OK;
}

// Gout: the range's rows of the updated stream as a GEMM operand.  sum, sum_cols: where the streams' weighted sum and its
// column sums may go (sum_cols nullptr: not wanted); *made: what is there afterwards.
int ln_bwd(il_ctx *c, const Run &run, const void *dy, const float *x, const float *stats, size_t g_off, void *Gout,
           float *partials, int *nblk, void *sum, float *sum_cols, Summed *made) {
  StreamWeights sw;
  memcpy(sw.w, run.wt, sizeof(sw.w));
  const int rows = run.cnt * c->N;
  const Weighted w = weighted(run);
  void *ysum = sum_cols && !w.plain ? sum : nullptr;
  Scope sc(c, KC_LN_BWD, 0, (double)rows * c->d * (c->eb + 8 + c->eb) + (double)c->N * c->d * (4 + (ysum ? c->eb : 0)));
  bool summed = false;
  IL_TRY(ln_backward_residual(c->cfg.dtype, dy, x, stats, P(c, g_off), run.cnt, c->N, c->d,
                              c->G + (size_t)run.s0 * c->N * c->d, Gout, sw, partials, nblk, ysum, sum_cols, &summed,
                              c->stream));
  if (summed)
    *made = Summed{ysum ? ysum : (const char *)Gout + (size_t)w.first * c->N * c->d * c->eb, sum_cols, *nblk};
  return IL_OK;
}

int block_forward(il_ctx *c, const BlockOff &b, const BlockSave &s, const float *x, float *xcopy, float *x_out) {
  const int N = c->N, d = c->d, m = c->m, dt = c->cfg.dtype;
  {
    Scope sc(c, KC_LN_FWD, 0, (double)N * d * (4 + c->eb));
    IL_TRY(ln_forward(dt, x, P(c, b.ln1_g), P(c, b.ln1_b), c->cfg.ln_eps, N, d, s.h1, s.st1, xcopy, c->stream));
  }
  int rc;
  if ((rc = linear_fwd(c, s.h1, b.w_qkv, b.b_qkv, N, d, 3 * d, EPI_BIAS, s.qkv, nullptr, nullptr))) return rc;
  if ((rc = attention_fwd(c, s.qkv, s.o, s.lse))) return rc;
  if ((rc = linear_fwd(c, s.o, b.w_o, b.b_o, N, d, d, EPI_BIAS_RES, s.a, nullptr, x))) return rc;
  {
    Scope sc(c, KC_LN_FWD, 0, (double)N * d * (4 + c->eb));
    IL_TRY(ln_forward(dt, s.a, P(c, b.ln2_g), P(c, b.ln2_b), c->cfg.ln_eps, N, d, s.h2, s.st2, nullptr,
                      c->stream));
  }
  if ((rc = linear_fwd(c, s.h2, b.w_fc1, b.b_fc1, N, d, m, EPI_BIAS_GELU, s.u, s.gl, nullptr))) return rc;
  if ((rc = linear_fwd(c, s.gl, b.w_fc2, b.b_fc2, N, m, d, EPI_BIAS_RES, x_out, nullptr, s.a))) return rc;
  return IL_OK;
}

// Launch the queued tails: weighted sum over the gradient streams of each of a block's four linear outputs
// (the weight gradient is linear in them, so one product over N rows serves any number of streams) with
// their column sums, the second stage of the column sums, the weight gradients.  A single stream of weight
// 1 is its own sum and is read where the data gradients left it; a sum of several takes the place of the first of
// them, which nothing else reads any more.
int launch_tails(il_ctx *c) {
  if (c->ntails == 0) return IL_OK;
  const bool async = c->cfg.profile != 1 && !c->tail_inline;
  const size_t wide[4] = {(size_t)c->d, (size_t)c->m, (size_t)c->d, 3 * (size_t)c->d};
  struct StreamSwap {
    il_ctx *c; bool on;
    ~StreamSwap() { if (on) c->stream = c->main_stream; }
  } swap{c, async};
  if (async) {
    const int rc = ensure_side(c);
    if (rc) return rc;
    IL_TRY(hipEventRecord(c->ev_ready, c->main_stream));
    IL_TRY(hipStreamWaitEvent(c->side, c->ev_ready, 0));
    c->stream = c->side;
  }
  // Ranges of slots one after the other, each for all queued tails: a range's sum of streams is stored in the
  // operands' type, but what different ranges contribute only meets in the fp32 gradients.
  for (int part = 0;; ++part) {
    SumColsumJobs sums;
    ColsumJobs finals;
    GemmArgs wg[4 * kGroup];
    int nw = 0;
    double sum_bytes = 0;
    memset(&sums, 0, sizeof(sums));
    sums.N = c->N;
    finals.count = 0;
    for (int i = 0; i < c->ntails; ++i) {
      const Tail &t = c->tails[i];
      const Run *run = weighted_run(*t.runs, part);
      if (!run) continue;
      const BlockOff &b = *t.b;
      // the weighted streams, as slots of Ga and as positions in Gb, DU and DQKV
      SumTable &by_slot = sums.table[2 * i], &by_stack = sums.table[2 * i + 1];
      for (int j = 0; j < run->cnt; ++j) {
        if (run->wt[j] == 0.f) continue;
        const int n = by_slot.ns++;
        by_stack.ns = n + 1;
        by_slot.row[n] = run->s0 + j;
        by_stack.row[n] = run->off + j;
        by_slot.w[n] = by_stack.w[n] = run->wt[j];
      }
      const int ns = by_slot.ns, acc = part > 0 || c->accumulate;
      const bool plain = ns == 1 && by_slot.w[0] == 1.f;
      char *const dy[4] = {t.r->Ga, t.r->DU, t.r->Gb, t.r->DQKV};
      const char *x[4] = {t.s->gl, t.s->h2, t.s->o, t.s->h1};
      const size_t w_off[4] = {b.w_fc2, b.w_fc1, b.w_o, b.w_qkv}, b_off[4] = {b.b_fc2, b.b_fc1, b.b_o, b.b_qkv};
      const int in[4] = {c->m, c->d, c->d, c->d};
      for (int j = 0; j < 4; ++j) {
        const void *y = t.done[j].y;
        if (t.done[j].cols) {
          finals.job[finals.count++] = ColsumJob{t.done[j].cols, t.done[j].nblk, (int)wide[j], Gr(c, b_off[j]), acc};
        } else {
          SumColsumJob &q = sums.job[sums.count++];
          q.Y = dy[j]; q.cols = (int)wide[j]; q.table = 2 * i + (j > 0);
          char *first = dy[j] + (size_t)sums.table[q.table].row[0] * c->N * wide[j] * c->eb;
          q.ysum = plain ? nullptr : first;
          q.partials = c->partials[i][j];
          y = first;
          sum_bytes += (double)(plain ? 1 : ns + 1) * c->N * wide[j] * c->eb;
          finals.job[finals.count++] = ColsumJob{q.partials, 0, q.cols, Gr(c, b_off[j]), acc};
        }
        GemmArgs g = base_args();
        g.A = x[j]; g.lda = in[j]; g.a_kmajor = 1;
        g.B = y; g.ldb = (int)wide[j]; g.b_kmajor = 1;
        g.M = in[j]; g.N = (int)wide[j]; g.K = c->N;
        g.epi = EPI_WGRAD; g.C = Gr(c, w_off[j]); g.ldc = (int)wide[j]; g.beta = acc;
        wg[nw++] = g;
      }
    }
    if (nw == 0) break;
    {
      Scope sc(c, KC_COLSUM, 0, sum_bytes);
      int nblk = 0;
      if (sums.count > 0) IL_TRY(sum_colsum_multi(c->cfg.dtype, sums, &nblk, c->stream));
      for (int i = 0; i < finals.count; ++i)
        if (finals.job[i].nblk == 0) finals.job[i].nblk = nblk;
      for (int i = 0; part == 0 && i < c->ntails; ++i) {  // (every range's LayerNorm sums at once)
        const Tail &t = c->tails[i];
        finals.job[finals.count++] = ColsumJob{t.r->ln[0], t.ln_blocks, 2 * c->d, Gr(c, t.b->ln2_g), c->accumulate};
        finals.job[finals.count++] = ColsumJob{t.r->ln[1], t.ln_blocks, 2 * c->d, Gr(c, t.b->ln1_g), c->accumulate};
      }
      IL_TRY(colsum_final_multi(finals, c->stream));
    }
    const int rc = launch_wgrads(c, wg, nw);
    if (rc) return rc;
  }
  if (async) {
    const int half = (int)(c->tails[0].r - c->ring) / kGroup;
    IL_TRY(hipEventRecord(c->ev_tail[half], c->side));
    c->tail_pending[half] = 1;
    c->tail_last = half;
  }
  c->ntails = 0;
  return IL_OK;
}

// Backward of one block for all live streams: data gradients now, its tail queued.  lowest: the streams that
// leave it are not the next block's (another component's, or nobody's).
int block_backward(il_ctx *c, const std::vector<Run> &runs, const BlockOff &b, const BlockSave &s, bool lowest) {
  const int N = c->N, d = c->d, m = c->m;
  const size_t eb = c->eb;
  const RingEntry &r = c->ring[c->pos];
  const int next = (c->pos + 1) % kRing;
  int rc, ln_blocks = 0;
  const bool sums = runs.size() == 1 && ln_backward_sums(N, d);  // (several ranges' sums only meet in the gradients)
  Tail tail{&b, &s, &r, &runs, 0, {}};
  tail.done[0] = c->above;
  c->above = Summed{};
  for (const Run &run : runs) {
    const int S = run.cnt * N;
    const size_t slot = (size_t)run.s0 * N, stack = (size_t)run.off * N;
    char *Ga = r.Ga + slot * d * eb, *Gb = r.Gb + stack * d * eb, *DU = r.DU + stack * m * eb;
    char *DQKV = r.DQKV + stack * 3 * d * eb;
    float *ln[2] = {r.ln[0] + (size_t)ln_blocks * 2 * d, r.ln[1] + (size_t)ln_blocks * 2 * d};
    int nblk = 0;
    // MLP
    if (gelu_sums(c, runs)) {
      const Weighted w = weighted(run);
      void *sum = w.plain ? nullptr : r.sum_du;
      if ((rc = linear_dgrad(c, Ga, b.w_fc2, S, m, d, EPI_GELU_BWD_SUM, DU, s.u, N, r.sum_du_cols, sum, &run))) return rc;
      tail.done[1] = Summed{sum ? sum : DU + (size_t)w.first * N * m * eb, r.sum_du_cols, (N + 63) / 64};
    } else if ((rc = linear_dgrad(c, Ga, b.w_fc2, S, m, d, EPI_GELU_BWD, DU, s.u, N))) {
      return rc;
    }
    if ((rc = linear_dgrad(c, DU, b.w_fc1, S, d, m, EPI_STORE, c->DH, nullptr, 0))) return rc;
    if ((rc = ln_bwd(c, run, c->DH, s.a, s.st2, b.ln2_g, Gb, ln[0], &nblk, r.sum[1], sums ? r.sum_cols[1] : nullptr,
                     &tail.done[2])))
      return rc;
    // attention
    const bool dots = attention_dsum_given(c->cfg.dtype, c->dh);
    if ((rc = linear_dgrad(c, Gb, b.w_o, S, d, d, dots ? EPI_STORE_DOT : EPI_STORE, c->DH, dots ? s.o : nullptr, N,
                           c->dsum)))
      return rc;
    if ((rc = attention_bwd(c, s, c->DH, run.cnt, DQKV))) return rc;
    if ((rc = linear_dgrad(c, DQKV, b.w_qkv, S, d, 3 * d, EPI_STORE, c->DH, nullptr, 0))) return rc;
    // the stream goes on to the next block's ring entry, which may still be read by an earlier group's tails
    if (!c->tail_inline && next % kGroup == 0 && c->tail_pending[next / kGroup]) {
      IL_TRY(hipStreamWaitEvent(c->main_stream, c->ev_tail[next / kGroup], 0));
      c->tail_pending[next / kGroup] = 0;
    }
    const RingEntry &n = c->ring[next];
    if ((rc = ln_bwd(c, run, c->DH, s.xs, s.st1, b.ln1_g, n.Ga + slot * d * eb, ln[1], &nblk, n.sum[0],
                     sums && !lowest ? n.sum_cols[0] : nullptr, &c->above)))
      return rc;
    ln_blocks += nblk;
  }
  tail.ln_blocks = ln_blocks;
  c->tails[c->ntails++] = tail;
  if (c->tail_inline || next % kGroup == 0)
    if ((rc = launch_tails(c))) return rc;
  c->pos = next;
  return IL_OK;
}

bool head_width_ok(int dtype, int dh) {
  return dh == 16 || dh == 32 || dh == 64 || dh == 128 || (dh == 256 && dtype == IL_BF16);
}

int validate(const il_config *cfg) {
  if (cfg->K < 1 || cfg->blocks_per_component < 1 || cfg->d_model < 1 || cfg->n_heads < 1 || cfg->d_mlp < 1 ||
      cfg->vocab < 2 || cfg->batch < 1 || cfg->seq < 1)
    return IL_E_ARG;
  if (cfg->n < 1 || cfg->n > cfg->K) return IL_E_ARG;
  if (cfg->dtype != IL_F32 && cfg->dtype != IL_BF16) return IL_E_ARG;
  if (cfg->route < 0 || cfg->route > IL_ROUTE_MEAN_LOCAL_FAR) return IL_E_ARG;
  if (!(cfg->ln_eps > 0.f)) return IL_E_ARG;
  if (cfg->profile < 0 || cfg->profile > 2) return IL_E_ARG;
  if (cfg->head_chunk < 0 || cfg->head_blocks < 0 || cfg->head_blocks > 64 || cfg->reserved != 0) return IL_E_ARG;
  if (cfg->d_model % cfg->n_heads) return IL_E_SHAPE;
  if (!head_width_ok(cfg->dtype, cfg->d_model / cfg->n_heads)) return IL_E_SHAPE;
  if (cfg->d_model > 2048) return IL_E_SHAPE;
  const long long N = (long long)cfg->batch * cfg->seq;
  if (N > (1 << 24) || (long long)cfg->vocab > (1 << 24)) return IL_E_SHAPE;
  if ((long long)cfg->batch * cfg->n_heads > 65535) return IL_E_SHAPE;  // the attention grids' y extent
  if (cfg->dtype == IL_BF16) {
    if (cfg->d_model % 8 || cfg->d_mlp % 8 || cfg->vocab % 8 || N % 64) return IL_E_SHAPE;
    if (cfg->head_chunk % 64) return IL_E_SHAPE;
  }
  return IL_OK;
}

}  // namespace

extern "C" {

const char *il_status_string(int status) {
  switch (status) {
    case IL_OK: return "IL_OK";
    case IL_E_ARG: return "IL_E_ARG: invalid argument";
    case IL_E_SHAPE: return "IL_E_SHAPE: size not supported by the kernels";
    case IL_E_STATE: return "IL_E_STATE: call order violated";
    case IL_E_WORKSPACE: return "IL_E_WORKSPACE: buffer missing or too small";
    case IL_E_HIP: return "IL_E_HIP: HIP runtime error";
    default: return "unknown status";
  }
}

int il_routing_plan(int32_t K, int32_t n, int32_t route, int32_t *live, int32_t *passes) {
  Plan p;
  int rc = build_plan(K, n, route, p);
  if (rc) return rc;
  for (int k = 0; k < K; ++k) {
    if (live) live[k] = p.comp[k].cnt;
    if (passes) passes[k] = p.comp[k].passes;
  }
  return IL_OK;
}

int il_init(il_config *cfg, il_ctx **out) {
  if (!cfg || !out) return IL_E_ARG;
  *out = nullptr;
  int rc = validate(cfg);
  if (rc) return rc;
  il_ctx *c = new (std::nothrow) il_ctx();
  if (!c) return IL_E_ARG;
  c->cfg = *cfg;
  c->K = cfg->K; c->L = cfg->blocks_per_component; c->d = cfg->d_model; c->m = cfg->d_mlp; c->V = cfg->vocab;
  c->H = cfg->n_heads; c->dh = c->d / c->H; c->N = cfg->batch * cfg->seq;
  c->eb = cfg->dtype == IL_F32 ? 4 : 2;
  c->Lh = cfg->head_blocks;
  c->stream = (hipStream_t)cfg->stream;
  c->main_stream = c->stream;
  rc = build_plan(c->K, cfg->n, cfg->route, c->plan);
  if (rc) { delete c; return rc; }
  {
    // every GEMM operand is addressed through a 32-bit buffer descriptor: below 2 GiB each
    const unsigned long long lim = 0x7FFFFFFFull, eb = c->eb, N = c->N, d = c->d, m = c->m, V = c->V;
    const unsigned long long S = (unsigned long long)std::max(c->plan.maxcnt, 1) * N;
    if (S * std::max(3 * d, m) * eb >= lim || d * V * eb >= lim || d * m * eb >= lim || 3 * d * d * eb >= lim) {
      delete c;
      return IL_E_SHAPE;
    }
  }
  int nc = cfg->head_chunk;
  if (nc == 0) {
    // default: half the rows, at most 2048, so that logits / probabilities never exist for all tokens
    // at once; halved until the tile is addressable (below 2 GiB)
    // Equal chunks, in multiples of 64 rows for bf16: a chunk of a few rows costs another pass over the
    // head matrix and its gradient (1600 rows as 768 + 768 + 64 took 1.4x the time of 832 + 768).
    int chunks = std::max(2, (c->N + 2047) / 2048);
    const int unit = cfg->dtype == IL_BF16 ? 64 : 1;
    auto rows = [&] { return ((c->N + chunks - 1) / chunks + unit - 1) / unit * unit; };
    while (rows() > unit && (unsigned long long)rows() * c->V * c->eb >= 0x7FFFFFFFull) ++chunks;
    nc = rows();
    if (nc < 1) nc = c->N;
  }
  c->Nc = std::min(nc, c->N);
  if ((unsigned long long)c->Nc * c->V * c->eb >= 0x7FFFFFFFull) {  // the logits tile is a GEMM operand too
    delete c;
    return IL_E_SHAPE;
  }
  const size_t pbytes = layout_params(c) * c->eb;
  const size_t gbytes = pbytes / c->eb * 4;
  const size_t wbytes = layout_workspace(c, cfg->workspace);
  if (!cfg->workspace) {
    cfg->params_bytes = pbytes; cfg->grads_bytes = gbytes; cfg->workspace_bytes = wbytes;
    delete c;
    return IL_E_WORKSPACE;
  }
  if (!cfg->params || !cfg->grads || cfg->params_bytes < pbytes || cfg->grads_bytes < gbytes ||
      cfg->workspace_bytes < wbytes || ((uintptr_t)cfg->workspace & 255) || ((uintptr_t)cfg->params & 15) ||
      ((uintptr_t)cfg->grads & 15)) {
    delete c;
    return IL_E_WORKSPACE;
  }
  c->fwd_done.assign(c->K + 1, 0); c->head_done.assign(c->K + 1, 0); c->bwd_done.assign(c->K + 2, 0);
  c->head_pending.assign(c->K + 1, 0);
  *out = c;
  return IL_OK;
}

int il_stage_forward(il_ctx *c, int32_t k, const float *x_in, float *x_out) {
  if (!c || !x_in || !x_out || x_in == x_out) return IL_E_ARG;
  if (k < 1 || k > c->K) return IL_E_ARG;
  if (k == 1) {
    std::fill(c->fwd_done.begin(), c->fwd_done.end(), 0);
    std::fill(c->head_done.begin(), c->head_done.end(), 0);
    std::fill(c->bwd_done.begin(), c->bwd_done.end(), 0);
    // an abandoned step may have left heads running on the side stream: they share the scratch
    // that this step's heads will use and read buffers the caller is about to overwrite
    for (int j = 1; j <= c->K; ++j)
      if (c->head_pending[j]) {
        if (hipStreamWaitEvent(c->stream, c->ev_head[j], 0) != hipSuccess) return IL_E_HIP;
        c->head_pending[j] = 0;
      }
    { const int rc = join_tails(c); if (rc) return rc; }  // ... or weight gradients of its backward
    c->ntails = 0;
    c->pos = 0;
    c->above = Summed{};
  } else if (!c->fwd_done[k - 1]) {
    return IL_E_STATE;
  }
  for (int l = 0; l < c->L; ++l) {
    const size_t bi = (size_t)(k - 1) * c->L + l;
    const BlockSave &s = c->save[bi];
    const float *xin = l == 0 ? x_in : s.xs;
    float *xout = l == c->L - 1 ? x_out : c->save[bi + 1].xs;
    int rc = block_forward(c, c->boff[bi], s, xin, l == 0 ? s.xs : nullptr, xout);
    if (rc) return rc;
  }
  c->fwd_done[k] = 1;
  c->head_done[k] = 0;
  return IL_OK;
}

// The head's scratch: the bf16 / fp32 copy of its input, one logits tile, per-row losses and the
// split-K partial products of dx.  il_head_xent takes it from the caller's workspace,
// il_head_xent_static from the library's static device array.
struct HeadScratch {
  int Nc;  // token rows per logits tile
  char *xb, *Z; float *rowloss, *skws; size_t skws_floats;
  float *stats, *ztgt;  // bf16: per-row softmax statistics of the tile ([Nc][ceil(V/64)][2]) and target logits ([Nc])
};

static int head_xent_impl(il_ctx *c, int32_t k, const float *x_k, const int32_t *targets, float *loss_out,
                          const HeadScratch &hs, bool in_line) {
  if (!c || !x_k || !targets || !loss_out) return IL_E_ARG;
  if (k < 1 || k > c->K) return IL_E_ARG;
  if (!c->fwd_done[k]) return IL_E_STATE;
  // a head with blocks of its own shares the backward scratch: it may not start once the step's
  // backward has (the backward could not order itself against it)
  if (c->Lh > 0 && c->bwd_done[c->K]) return IL_E_STATE;
  const int N = c->N, d = c->d, V = c->V, dt = c->cfg.dtype;
  const size_t eb = c->eb;
  // Head k only needs x_k; it runs on a side stream so that the next component's forward (and,
  // later, other heads' consumers) overlap with it.  il_stage_backward_nwise(k) joins.
  struct StreamSwap {
    il_ctx *c; bool on;
    ~StreamSwap() { if (on) c->stream = c->main_stream; }
  } swap{c, false};
  if (c->cfg.profile != 1 && !in_line) {
    { const int rc = ensure_side(c); if (rc) return rc; }
    IL_TRY(hipEventRecord(c->ev_fork, c->main_stream));
    IL_TRY(hipStreamWaitEvent(c->side, c->ev_fork, 0));
    c->stream = c->side;
    swap.on = true;
  }
  // the head's own blocks (App. B: the auxiliary network is Transformer blocks and an output matrix)
  const float *y = x_k;
  for (int l = 0; l < c->Lh; ++l) {
    const size_t bi = (size_t)(k - 1) * c->Lh + l;
    const BlockSave &s = c->hsave[bi];
    float *yout = l == c->Lh - 1 ? c->hy : c->hsave[bi + 1].xs;
    int rc = block_forward(c, c->hboff[bi], s, y, l == 0 ? s.xs : nullptr, yout);
    if (rc) return rc;
    y = yout;
  }
  {
    Scope sc(c, KC_MISC, 0, (double)N * d * (4 + eb));
    IL_TRY(convert_f32(dt, y, hs.xb, (size_t)N * d, c->stream));
  }
  float *dx = c->dxh + (size_t)(k - 1) * N * d;
  for (int r0 = 0, chunk = 0; r0 < N; r0 += hs.Nc, ++chunk) {
    const int rows = std::min(hs.Nc, N - r0);
    const char *xc = hs.xb + (size_t)r0 * d * eb;
    GemmArgs g = base_args();  // logits tile z = x W_h
    g.A = xc; g.lda = d; g.a_kmajor = 0;
    g.B = P(c, c->hoff[k - 1]); g.ldb = V; g.b_kmajor = 1;
    // bf16 mode: the tile holds the logits as IEEE half (three more mantissa bits for the softmax's
    // exponentials) and the GEMM's epilogue leaves the softmax statistics of every 64-column group,
    // taken from its fp32 accumulators, and the target logits beside it
    const bool fused = dt == IL_BF16;
    g.M = rows; g.N = V; g.K = d; g.epi = fused ? EPI_LOGITS : EPI_STORE; g.C = hs.Z; g.ldc = V;
    if (fused) { g.row_stats = hs.stats; g.row_targets = targets + r0; g.row_ztgt = hs.ztgt; }
    {
      Scope sc(c, KC_GEMM_HEAD, 2.0 * rows * V * d, gemm_bytes(c, g));
      IL_TRY(gemm(c, g));
    }
    {
      Scope sc(c, KC_XENT, 0, 2.0 * rows * V * eb);
      if (fused)
        IL_TRY(xent_rows_from_stats(hs.Z, hs.stats, hs.ztgt, targets + r0, rows, V, c->grad_scale / N,
                                    hs.rowloss + r0, c->stream));
      else
        IL_TRY(xent_rows(dt, hs.Z, targets + r0, rows, V, c->grad_scale / N, hs.rowloss + r0, c->stream));
    }
    g = base_args();  // dx = dz W_h^T
    g.A = hs.Z; g.lda = V; g.a_kmajor = 0;
    g.B = P(c, c->hoff[k - 1]); g.ldb = V; g.b_kmajor = 0;
    g.M = rows; g.N = d; g.K = V; g.epi = EPI_STORE_F32; g.C = dx + (size_t)r0 * d; g.ldc = d;
    {
      Scope sc(c, KC_GEMM_HEAD, 2.0 * rows * V * d, gemm_bytes(c, g));
      IL_TRY(gemm_splitk(dt, g, head_split(c, rows, hs.skws_floats), hs.skws, c->stream));
    }
    g = base_args();  // dW_h (+)= x^T dz
    g.A = xc; g.lda = d; g.a_kmajor = 1;
    g.B = hs.Z; g.ldb = V; g.b_kmajor = 1;
    g.M = d; g.N = V; g.K = rows; g.epi = EPI_WGRAD; g.C = Gr(c, c->hoff[k - 1]); g.ldc = V;
    g.beta = chunk > 0 || c->accumulate;
    {
      Scope sc(c, KC_GEMM_HEAD, 2.0 * rows * V * d, gemm_bytes(c, g));
      IL_TRY(gemm(c, g));
    }
  }
  {
    Scope sc(c, KC_MISC, 0, (double)N * 4);
    IL_TRY(sum_scalar(hs.rowloss, N, 1.f / N, loss_out, c->stream));
  }
  if (c->Lh) {
    // dL_k/dy goes back through the head's blocks as a single stream of weight 1 in a slot of its own;
    // what arrives at x_k replaces it as the head's gradient stream.
    const size_t nd = (size_t)N * d;
    const int slot = c->plan.nslots;
    float *Gh = c->G + (size_t)slot * nd;
    {
      Scope sc(c, KC_MISC, 0, (double)nd * (8 + eb));
      IL_TRY(stream_inject(dt, dx, Gh, c->ring[c->pos].Ga + (size_t)slot * nd * eb, nd, 0, c->stream));
    }
    std::vector<Run> runs(1);
    runs[0].s0 = slot; runs[0].cnt = 1; runs[0].wt[0] = 1.f;
    struct Inline { il_ctx *c; bool old; ~Inline() { c->tail_inline = old; } } guard{c, c->tail_inline};
    c->tail_inline = true;  // already off the caller's stream: the block tails run in line, block by block
    for (int l = c->Lh - 1; l >= 0; --l) {
      const size_t bi = (size_t)(k - 1) * c->Lh + l;
      int rc = block_backward(c, runs, c->hboff[bi], c->hsave[bi], l == 0);
      if (rc) return rc;
    }
    StreamWeights one;
    memset(&one, 0, sizeof(one));
    one.w[0] = 1.f;
    Scope sc(c, KC_MISC, 0, (double)nd * 8);
    IL_TRY(stream_combine(Gh, nd, 1, one, dx, nd, 0, c->stream));
  }
  if (swap.on) {
    IL_TRY(hipEventRecord(c->ev_head[k], c->side));
    c->head_pending[k] = 1;
    // The last head joins the side stream back (it is in order, so this covers every earlier head):
    // component K's backward needs this head at once anyway, and a caller that stops after the
    // heads finds every loss final on its own stream.
    if (k == c->K) {
      IL_TRY(hipStreamWaitEvent(c->main_stream, c->ev_head[k], 0));
      std::fill(c->head_pending.begin(), c->head_pending.end(), 0);
    }
  }
  c->head_done[k] = 1;
  return IL_OK;
}

int il_head_xent(il_ctx *c, int32_t k, const float *x_k, const int32_t *targets, float *loss_out) {
  if (!c) return IL_E_ARG;
  const HeadScratch hs{c->Nc, c->xb, c->Z, c->rowloss, c->skws, c->skws_floats, c->hstats, c->hztgt};
  return head_xent_impl(c, k, x_k, targets, loss_out, hs, false);
}

// ---- the head without a workspace of its own -------------------------------------------------
// The library's static scratch: every GPU the library runs on holds its own copy of this array at
// its own address until the process ends.  Host code never passes the array's name to a kernel (on
// the host it is a stand-in, not a device address): the address is looked up once per device.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// The current device's copy of `scratch` (looked up on the first call on that device).
int static_scratch(char **out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return IL_E_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return IL_E_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = (char *)g_scratch_ptr[dev];
  return IL_OK;
}
}  // namespace

int il_head_xent_static(il_ctx *c, int32_t k, const float *x_k, const int32_t *targets, float *loss_out) {
  if (!c) return IL_E_ARG;
  if (c->Lh > 0) return IL_E_SHAPE;  // heads with blocks of their own need the workspace's saved activations
  // the pieces the head's kernels use, carved from the static array (256-byte aligned pieces); where the
  // default's equal chunks do not fit, chunks rounded down to whole units may
  size_t o_xb, o_z, o_rl, o_sk, o_hs, o_zt, need, skws_floats;
  auto carve = [&](int rows, size_t floats) {
    Carver cv(nullptr);
    skws_floats = head_split_floats(c, rows, floats);
    o_xb = cv.off; cv.take((size_t)c->N * c->d * c->eb);
    o_z = cv.off; cv.take((size_t)rows * c->V * c->eb);
    o_rl = cv.off; cv.take((size_t)c->N * 4);
    o_sk = cv.off; cv.take(skws_floats * 4);
    o_hs = cv.off; cv.take(head_stats_bytes(c, rows));
    o_zt = cv.off; cv.take(c->eb == 2 ? (size_t)rows * 4 : 0);
    need = cv.off;
  };
  int rows = c->Nc;
  carve(rows, (size_t)-1);
  if (need > kStaticScratchBytes) carve(rows, (size_t)8 * rows * c->d);  // at most eight parts
  if (need > kStaticScratchBytes && c->cfg.head_chunk == 0) {
    const int unit = c->eb == 2 ? 64 : 1, down = std::min(c->N / 2, 2048) / unit * unit;
    if (down >= unit) {
      rows = std::min(rows, down);
      carve(rows, (size_t)8 * rows * c->d);
    }
  }
  // fp32 likes more parts than it did when its products were slower: fewer of them, whatever is left for them, so that no
  // size that fitted then is refused
  if (need > kStaticScratchBytes && c->cfg.dtype == IL_F32) {
    const size_t rest = need - ((skws_floats * 4 + 255) & ~(size_t)255);
    carve(rows, rest < kStaticScratchBytes ? (kStaticScratchBytes - rest) / 4 : 0);
  }
  if (need > kStaticScratchBytes) return IL_E_WORKSPACE;
  char *base = nullptr;
  { const int rc = static_scratch(&base); if (rc) return rc; }
  const HeadScratch hs{rows, base + o_xb, base + o_z, (float *)(base + o_rl), (float *)(base + o_sk), skws_floats,
                       (float *)(base + o_hs), (float *)(base + o_zt)};
  return head_xent_impl(c, k, x_k, targets, loss_out, hs, true);
}

int il_stage_backward_nwise(il_ctx *c, int32_t k, float *dx0_out) {
  if (!c) return IL_E_ARG;
  if (k < 1 || k > c->K) return IL_E_ARG;
  for (int j = 1; j <= c->K; ++j)
    if (!c->fwd_done[j]) return IL_E_STATE;
  if (c->bwd_done[k] || (k < c->K && !c->bwd_done[k + 1])) return IL_E_STATE;
  const CompPlan &cp = c->plan.comp[k - 1];
  if (cp.inject_slot >= 0 && !c->head_done[k]) return IL_E_STATE;
  // join the side stream: head k before its gradient is injected; every head before the step ends.
  // Heads with blocks of their own run a block backward there, over the scratch this call is about to
  // use: then every head still pending is joined, whatever the order the heads were enqueued in.
  const bool all_heads = k == 1 || c->Lh > 0;
  for (int j = (all_heads ? 1 : k); j <= (all_heads ? c->K : k); ++j)
    if (c->head_pending[j]) {
      IL_TRY(hipStreamWaitEvent(c->stream, c->ev_head[j], 0));
      c->head_pending[j] = 0;
    }
  const size_t nd = (size_t)c->N * c->d;
  if (cp.inject_slot >= 0) {
    Scope sc(c, KC_MISC, 0, (double)nd * (8 + c->eb));
    IL_TRY(stream_inject(c->cfg.dtype, c->dxh + (size_t)(k - 1) * nd, c->G + cp.inject_slot * nd,
                         c->ring[c->pos].Ga + cp.inject_slot * nd * c->eb, nd, cp.inject_acc, c->stream));
  }
  for (int l = c->L - 1; l >= 0; --l) {
    const size_t bi = (size_t)(k - 1) * c->L + l;
    const int rc = block_backward(c, cp.runs, c->boff[bi], c->save[bi], l == 0);
    if (rc) return rc;
  }
  // a tail that waits for a partner does not wait beyond the call: a caller that synchronises the device after
  // component k finds its gradients
  { const int rc = launch_tails(c); if (rc) return rc; }
  if (k == 1 && dx0_out) {
    Scope sc(c, KC_MISC, 0, (double)nd * 4 * (cp.cnt + 1));
    for (size_t i = 0; i < cp.runs.size(); ++i) {
      const Run &r = cp.runs[i];
      StreamWeights sw;
      memcpy(sw.w, r.wt, sizeof(sw.w));
      IL_TRY(stream_combine(c->G + r.s0 * nd, nd, r.cnt, sw, dx0_out, nd, i > 0, c->stream));
    }
  }
  c->bwd_done[k] = 1;
  // the step's last backward call joins the tails still running on the side stream
  if (k == 1) {
    const int rc = join_tails(c);
    if (rc) return rc;
    c->pos = 0;
  }
  return IL_OK;
}

int il_profile_read(il_ctx *c, int32_t cap, const char **names, int64_t *launches, double *ms, double *flops,
                    double *bytes, double *kernel_ms) {
  if (!c || cap < 0) return IL_E_ARG;
  if (hipStreamSynchronize(c->stream) != hipSuccess) return IL_E_HIP;
  if (c->side && hipStreamSynchronize(c->side) != hipSuccess) return IL_E_HIP;
  double t[KC_COUNT] = {}, tk[KC_COUNT] = {};
  int64_t n[KC_COUNT] = {};
  for (size_t i = 0; i < c->nrec; ++i) {
    float e = 0.f;
    if (c->recs[i].bracket) {
      if (hipEventElapsedTime(&e, c->recs[i].e0, c->recs[i].e1) != hipSuccess) return IL_E_HIP;
      t[c->recs[i].cls] += e;
    }
    n[c->recs[i].cls] += 1;
    if (c->recs[i].kernel) {
      if (hipEventElapsedTime(&e, c->recs[i].kt.start, c->recs[i].kt.stop) != hipSuccess) return IL_E_HIP;
      tk[c->recs[i].cls] += e;
    }
  }
  const int cnt = std::min<int>(cap, KC_COUNT);
  for (int i = 0; i < cnt; ++i) {
    if (names) names[i] = kClassNames[i];
    if (launches) launches[i] = n[i];
    if (ms) ms[i] = t[i];
    if (kernel_ms) kernel_ms[i] = tk[i];
    if (flops) flops[i] = c->flops[i];
    if (bytes) bytes[i] = c->bytes[i];
  }
  c->nrec = 0;
  memset(c->flops, 0, sizeof(c->flops));
  memset(c->bytes, 0, sizeof(c->bytes));
  return cnt;
}

int il_test_gemm(int32_t dtype, const void *A, const void *B, int32_t M, int32_t N, int32_t K, int32_t lda,
                 int32_t ldb, int32_t a_kmajor, int32_t b_kmajor, int32_t epi, void *C, void *C2, int32_t ldc,
                 const void *bias, const float *res, const void *aux, int32_t aux_wrap, float scale,
                 int32_t beta, int32_t tile, void *stream) {
  if (!A || !B || !C || M < 1 || N < 1 || K < 1) return IL_E_ARG;
  if (dtype != IL_F32 && dtype != IL_BF16) return IL_E_ARG;
  if (epi < EPI_STORE || epi > EPI_STORE_DOT + 1 || tile < 0 || tile > 8) return IL_E_ARG;
  const bool gelu_sum = epi == EPI_STORE_DOT + 1;
  if (gelu_sum && (dtype != IL_BF16 || !aux || !C2 || (beta != 1 && beta != 2) || M % (64 * beta) || ldc != N)) return IL_E_ARG;
  if (epi == EPI_STORE_DOT && (dtype != IL_BF16 || !aux || !C2 || aux_wrap < 1)) return IL_E_ARG;
  if (epi == EPI_LOGITS && (dtype != IL_BF16 || (C2 && !aux))) return IL_E_ARG;
  if ((epi == EPI_BIAS || epi == EPI_BIAS_GELU || epi == EPI_BIAS_RES) && !bias) return IL_E_ARG;
  if ((epi == EPI_BIAS_RES && !res) || (epi == EPI_BIAS_GELU && !C2)) return IL_E_ARG;
  if (epi == EPI_GELU_BWD && (!aux || aux_wrap < 1)) return IL_E_ARG;
  GemmArgs g = base_args();
  g.A = A; g.B = B; g.M = M; g.N = N; g.K = K; g.lda = lda; g.ldb = ldb;
  g.a_kmajor = a_kmajor != 0; g.b_kmajor = b_kmajor != 0; g.epi = epi; g.C = C; g.C2 = C2; g.ldc = ldc;
  g.bias = bias; g.res = res; g.aux = aux; g.aux_wrap = aux_wrap; g.scale = scale; g.beta = beta; g.tile = tile;
  if (epi == EPI_LOGITS && C2) {  // statistics and target logits share the second output buffer
    g.row_stats = (float *)C2;
    g.row_targets = (const int32_t *)aux;
    g.row_ztgt = (float *)C2 + (size_t)M * ((N + kStatGroup - 1) / kStatGroup) * 2;
    g.C2 = nullptr;
    g.aux = nullptr;
  }
  if (epi == EPI_STORE_DOT) {
    g.row_stats = (float *)C2;
    g.C2 = nullptr;
  }
  if (gelu_sum) {
    g.epi = EPI_GELU_BWD_SUM;
    g.streams = beta; g.aux_wrap = M / beta;
    g.sum_w[0] = scale; g.sum_w[1] = 1.f;
    g.row_stats = (float *)C2 + (size_t)(M / beta) * N / 2;
  }
  const hipError_t e = dtype == IL_F32 ? gemm_f32(g, (hipStream_t)stream) : gemm_bf16(g, (hipStream_t)stream);
  return e == hipSuccess ? IL_OK : (e == hipErrorInvalidValue ? IL_E_SHAPE : IL_E_HIP);
}

int il_test_gemm_splitk(int32_t dtype, const void *A, const void *B, int32_t M, int32_t N, int32_t K, int32_t splits,
                        int32_t tile, float *ws, float *C, int32_t ldc, void *stream) {
  if (!A || !B || !C || !ws || M < 1 || N < 1 || K < 1 || splits < 1 || tile < 0 || tile > 8) return IL_E_ARG;
  if (dtype != IL_F32 && dtype != IL_BF16) return IL_E_ARG;
  GemmArgs g = base_args();
  g.A = A; g.B = B; g.M = M; g.N = N; g.K = K; g.lda = K; g.ldb = K; g.epi = EPI_STORE_F32; g.C = C; g.ldc = ldc;
  const hipError_t e = gemm_splitk(dtype, g, SplitPlan{splits, tile}, ws, (hipStream_t)stream);
  return e == hipSuccess ? IL_OK : (e == hipErrorInvalidValue ? IL_E_SHAPE : IL_E_HIP);
}

int il_gemm_split_plan(int32_t dtype, int32_t M, int32_t N, int32_t K, size_t ws_floats, int32_t *tile) {
  if ((dtype != IL_F32 && dtype != IL_BF16) || M < 1 || N < 1 || K < 1) return IL_E_ARG;
  const SplitPlan p = gemm_split_plan(dtype, M, N, K, ws_floats);
  if (tile) *tile = p.tile;
  return p.splits;
}

int il_gemm_tile_of(int32_t tiles_m, int32_t tiles_n, int32_t edge_m, int32_t edge_n, int32_t K, int32_t workgroup,
                    int32_t *tile_m, int32_t *tile_n) {
  if (tiles_m < 1 || tiles_n < 1 || edge_m < 1 || edge_n < 1 || K < 1 || !tile_m || !tile_n) return IL_E_ARG;
  if ((long long)tiles_m * tiles_n > 0x7FFFFFFF || workgroup < 0 || workgroup >= tiles_m * tiles_n) return IL_E_ARG;
  const bool in_turn = tiles_in_turn({tiles_m, tiles_n, edge_m, edge_n}, K, 1);
  const TilePlace at = tile_place(tile_turn(workgroup, tiles_m * tiles_n, in_turn), tiles_m, tiles_n);
  *tile_m = at.m;
  *tile_n = at.n;
  return IL_OK;
}

int il_test_layernorm(int32_t dtype, const float *x, const void *gamma, const void *beta, float eps, int32_t rows, int32_t d,
                      void *y, float *stats, float *xcopy, void *stream) {
  if (!x || !gamma || !beta || !y || !stats || rows < 1 || d < 1) return IL_E_ARG;
  if (dtype != IL_F32 && dtype != IL_BF16) return IL_E_ARG;
  if (d > 2048 || rows > (1 << 24)) return IL_E_SHAPE;
  IL_TRY(ln_forward(dtype, x, gamma, beta, eps, rows, d, y, stats, xcopy, (hipStream_t)stream));
  return IL_OK;
}

int il_test_layernorm_backward(int32_t dtype, const void *dy, const float *x, const float *stats, const void *gamma, int32_t streams,
                               int32_t tokens, int32_t d, float *G, void *Gb, const float *weights, float *partials, void *ysum,
                               float *ypart, int32_t *blocks, int32_t *summed, void *stream) {
  if (!dy || !x || !stats || !gamma || !G || !Gb || !weights || !partials || !blocks || !summed || tokens < 1 || d < 1) return IL_E_ARG;
  if (dtype != IL_F32 && dtype != IL_BF16) return IL_E_ARG;
  if (d > 2048 || streams < 1 || streams > kMaxStreams || (long long)streams * tokens * d * 4 > 0xFFFFFFFFll) return IL_E_SHAPE;
  StreamWeights sw;
  memset(&sw, 0, sizeof(sw));
  memcpy(sw.w, weights, streams * sizeof(float));
  bool made = false;
  int nblk = 0;
  IL_TRY(ln_backward_residual(dtype, dy, x, stats, gamma, streams, tokens, d, G, Gb, sw, partials, &nblk, ysum, ypart, &made,
                              (hipStream_t)stream));
  *blocks = nblk;
  *summed = made;
  return IL_OK;
}

int il_attention_wants_dsum(int32_t dtype, int32_t width) { return attention_dsum_given(dtype, width) ? 1 : 0; }

static int attention_extents(int32_t dtype, int32_t width, int32_t batch, int32_t seq, int32_t heads, int32_t streams, bool backward) {
  if (batch < 1 || seq < 1 || heads < 1 || width < 1 || (dtype != IL_F32 && dtype != IL_BF16)) return IL_E_ARG;
  const long long N = (long long)batch * seq, rows = N * (backward ? streams : 1);
  if (!head_width_ok(dtype, width) || (long long)heads * width > 2048 || (long long)batch * heads > 65535 || N > (1 << 24) ||
      (backward && (streams < 1 || streams > kMaxStreams)) || rows * 3 * heads * width * (dtype == IL_F32 ? 4 : 2) >= 0x7FFFFFFFll)
    return IL_E_SHAPE;
  return IL_OK;
}

int il_attention_form(int32_t dtype, int32_t width, int32_t batch, int32_t seq, int32_t heads, int32_t streams, int32_t *form) {
  if (!form) return IL_E_ARG;
  const int rc = attention_extents(dtype, width, batch, seq, heads, streams, streams != 0);
  if (rc == IL_OK) *form = attention_form(dtype, width, streams, batch, seq, heads);
  return rc;
}

int il_test_attention(int32_t dtype, const void *qkv, int32_t batch, int32_t seq, int32_t heads, int32_t width,
                      void *o, float *lse, const void *d_o, int32_t streams, void *dqkv, float *dsum, void *stream) {
  if (!qkv || !o || !lse || (d_o && (!dqkv || !dsum))) return IL_E_ARG;
  if (const int rc = attention_extents(dtype, width, batch, seq, heads, streams, d_o != nullptr)) return rc;
  hipStream_t s = (hipStream_t)stream;
  IL_TRY(attention_forward(dtype, qkv, batch, seq, heads, width, o, lse, s));
  if (d_o) IL_TRY(attention_backward(dtype, qkv, o, d_o, lse, streams, batch, seq, heads, width, dqkv, dsum, s));
  return IL_OK;
}

int il_set_accumulation(il_ctx *c, int32_t accumulate, float grad_scale) {
  if (!c || !(grad_scale > 0.f) || !std::isfinite(grad_scale)) return IL_E_ARG;
  c->accumulate = accumulate ? 1 : 0;
  c->grad_scale = grad_scale;
  return IL_OK;
}

int il_free(il_ctx *c) {
  if (!c) return IL_E_ARG;
  if (c->side) hipStreamSynchronize(c->side);  // nothing of this context is left running on it
  for (auto &r : c->recs) {
    hipEventDestroy(r.e0); hipEventDestroy(r.e1);
    hipEventDestroy(r.kt.start); hipEventDestroy(r.kt.stop);
  }
  for (hipEvent_t e : c->ev_head) if (e) hipEventDestroy(e);
  if (c->ev_fork) hipEventDestroy(c->ev_fork);
  if (c->ev_ready) hipEventDestroy(c->ev_ready);
  for (hipEvent_t e : c->ev_tail) if (e) hipEventDestroy(e);
  if (c->side) hipStreamDestroy(c->side);
  delete c;
  return IL_OK;
}

}  // extern "C"
