// Lock-step execution of many reconstructions (batch and continuous serving).
//
// Every active problem advances by one outer IRLS iteration per engine step.
// Problems whose Gram matrices have the same size s share one launch sequence
// of the eigen-decomposition chain (tridiagonalisation, divide and conquer,
// back-transformation), each kernel covering all of them at once; the kernels
// treat every problem independently with the same arithmetic as for a single
// problem, so a result is bit-identical alone, in a batch and in the server.
// Within such a group the problems of one filter also share the launches of the
// images, Gram matrices, weights and masks (on the engine's stream); the others'
// run on the problem's own stream, ordered against the shared
// eigen-decomposition by events, as does the CG unless it is grouped too.
// Problems may join between steps (each keeps its own iteration index and
// epsilon schedule), which is what the server does.  Problems that use the
// library eigensolver take the single-problem path.
#include <hip/hip_runtime.h>
#include <rocprofiler-sdk-roctx/roctx.h>
#include <rocblas/rocblas.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <map>
#include <vector>

#include "engine.h"
#include "kernels.h"
#include "plan.h"
#include "tune.h"

using namespace slrx;


#define HIPCHK(expr)                                                                         \
  do {                                                                                       \
    hipError_t _e = (expr);                                                                  \
    if (_e != hipSuccess)                                                                    \
      return fail(SLRX_EDEVICE, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(_e), __FILE__, \
                  __LINE__);                                                                 \
  } while (0)

#define STCHK(expr)               \
  do {                            \
    slrx_status _s = (expr);      \
    if (_s != SLRX_OK) return _s; \
  } while (0)

slrx::EigGroup::~EigGroup() {
  if (mem) (void)hipFree(mem);
  if (tree) (void)hipFree(tree);
}

template <class T>
slrx_status slrx::DevTable<T>::upload(const std::vector<T>& h, hipStream_t s) {
  if (host.size() == h.size() && std::memcmp(host.data(), h.data(), h.size() * sizeof(T)) == 0) return SLRX_OK;
  // the new table follows, on the stream, the launches that read the old one
  if (h.size() > cap) {
    HIPCHK(hipStreamSynchronize(s));
    if (dev) HIPCHK(hipFree(dev));
    if (pinned) HIPCHK(hipHostFree(pinned));
    dev = nullptr;
    pinned = nullptr;
    cap = 0;
    pending = false;
    host.clear();
    const size_t n = std::max<size_t>(h.size(), 32);
    if (dev_malloc((void**)&dev, n * sizeof(T)) != hipSuccess) {
      (void)hipGetLastError();
      dev = nullptr;
      return fail(SLRX_ENOMEM, "table of a grouped launch (%zu entries)", n);
    }
    HIPCHK(hipHostMalloc((void**)&pinned, n * sizeof(T), hipHostMallocDefault));
    if (!copied) HIPCHK(hipEventCreateWithFlags(&copied, hipEventDisableTiming));
    cap = n;
  }
  if (pending) HIPCHK(hipEventSynchronize(copied));  // the staging copy is free again
  std::memcpy((void*)pinned, (const void*)h.data(), h.size() * sizeof(T));
  HIPCHK(hipMemcpyAsync(dev, pinned, h.size() * sizeof(T), hipMemcpyHostToDevice, s));
  HIPCHK(hipEventRecord(copied, s));
  pending = true;
  host = h;
  return SLRX_OK;
}

void slrx::engine_clear_stalls(BatchEig& be) {
  for (auto& kv : be.groups) kv.second.clear_stall = true;
}

void slrx::engine_drain(BatchEig& be) {
  if (be.stream) (void)hipStreamSynchronize(be.stream);
  if (be.cg_stream) (void)hipStreamSynchronize(be.cg_stream);
}

slrx::BatchEig::~BatchEig() {
  if (stream) (void)hipStreamSynchronize(stream);
  if (cg_stream) (void)hipStreamSynchronize(cg_stream);
  groups.clear();
  cg_tables.clear();
  weight_tables.clear();
  if (ev) (void)hipEventDestroy(ev);
  if (ev_w) (void)hipEventDestroy(ev_w);
  if (ev_free) (void)hipEventDestroy(ev_free);
  if (ev_cg) (void)hipEventDestroy(ev_cg);
  if (stream) {
    tri_resident_forget(stream);
    (void)hipStreamDestroy(stream);
  }
  if (cg_stream) (void)hipStreamDestroy(cg_stream);
}

static size_t al(size_t b) { return (b + 255) & ~(size_t)255; }

// Layout of the buffers for nb problems of size n: every matrix-sized buffer
// per problem, the vectors for all of them.
struct GroupLayout {
  size_t sA, sQ, sWi, sWd, sB, sv, sd, total;
};
static GroupLayout group_layout(int n, int nb) {
  GroupLayout L;
  const size_t nn = (size_t)n * n;
  L.sA = al(nn * sizeof(double2));
  L.sQ = al(3 * nn * sizeof(double));
  L.sWi = al(dc_ws_ints(n) * sizeof(int));
  L.sWd = al(dc_ws_doubles(n) * sizeof(double));
  L.sB = al(bt_scratch_elems(n) * sizeof(double2));
  L.sv = al((size_t)nb * n * sizeof(double2));
  L.sd = al((size_t)nb * n * sizeof(double));
  L.total = (size_t)nb * (3 * L.sA + L.sQ + L.sWi + L.sWd + L.sB) + 5 * L.sv + 2 * L.sd;
  return L;
}
// The divide-and-conquer tree, and 256 bytes for the give-up flag, which outlives the buffers
// (they are reallocated when a problem joins).
static size_t tree_ints(int n) { return std::max<size_t>((size_t)4 * n, 4); }
static size_t tree_bytes(int n) { return tree_ints(n) * sizeof(int) + 256; }

size_t slrx::engine_problem_bytes(int n) { return group_layout(n, 1).total + tree_bytes(n); }

size_t slrx::BatchEig::allocated() const {
  size_t b = 0;
  for (const auto& kv : groups) {
    if (kv.second.mem) b += group_layout(kv.first, kv.second.cap).total;
    if (kv.second.tree) b += tree_bytes(kv.first);
  }
  for (const auto& kv : cg_tables) b += kv.second.cap * sizeof(CgSlice);
  for (const auto& kv : weight_tables) b += kv.second.cap * sizeof(WeightSlice);
  return b;
}

slrx_status slrx::engine_trim(BatchEig& be, const std::map<int, int>& keep) {
  bool synced = false;
  auto sync = [&]() -> slrx_status {  // no reader of the buffers is left
    if (synced) return SLRX_OK;
    if (be.stream) HIPCHK(hipStreamSynchronize(be.stream));
    if (be.cg_stream) HIPCHK(hipStreamSynchronize(be.cg_stream));
    synced = true;
    return SLRX_OK;
  };
  auto drop_tables = [&](auto& tables) -> slrx_status {
    for (auto it = tables.begin(); it != tables.end();) {
      if (!keep.empty() && it->second.step == be.step) {
        ++it;
        continue;
      }
      STCHK(sync());
      it = tables.erase(it);
    }
    return SLRX_OK;
  };
  STCHK(drop_tables(be.cg_tables));
  STCHK(drop_tables(be.weight_tables));
  for (auto it = be.groups.begin(); it != be.groups.end();) {
    const auto k = keep.find(it->first);
    const int want = k == keep.end() ? 0 : k->second;
    if (it->second.cap <= want) {
      ++it;
      continue;
    }
    STCHK(sync());
    if (want == 0) {
      it = be.groups.erase(it);  // frees the buffers and the tree
      continue;
    }
    if (it->second.mem) HIPCHK(hipFree(it->second.mem));
    it->second.mem = nullptr;
    it->second.cap = 0;  // reserved again at the next step, for the problems present then
    ++it;
  }
  return SLRX_OK;
}

// Buffers for nb problems of size n (grown on demand; engine_trim shrinks them).
static slrx_status group_reserve(BatchEig& be, int n, int nb, EigGroup*& out) {
  if (!be.stream) {
    HIPCHK(hipStreamCreateWithFlags(&be.stream, hipStreamNonBlocking));
    HIPCHK(hipEventCreateWithFlags(&be.ev, hipEventDisableTiming));
    HIPCHK(hipEventCreateWithFlags(&be.ev_free, hipEventDisableTiming));
    HIPCHK(hipEventCreateWithFlags(&be.ev_w, hipEventDisableTiming));
  }
  EigGroup& G = be.groups[n];
  if (G.n != n) {  // first use of this size: the divide-and-conquer tree
    std::vector<int> nodes;
    dc_build_tree(n, nodes, G.level_start);
    G.node_sizes.resize(nodes.size() / 4);
    for (size_t q = 0; q < nodes.size() / 4; ++q) G.node_sizes[q] = nodes[4 * q + 1];
    if (!G.tree && dev_malloc((void**)&G.tree, tree_bytes(n)) != hipSuccess) {
      (void)hipGetLastError();
      G.tree = nullptr;
      return fail(SLRX_ENOMEM, "divide-and-conquer tree");
    }
    if (!nodes.empty())
      HIPCHK(copy_now(G.tree, nodes.data(), nodes.size() * sizeof(int), hipMemcpyHostToDevice));
    G.bufs.stall = G.tree + tree_ints(n);
    HIPCHK(hipMemsetAsync(G.bufs.stall, 0, 256, be.stream));  // in order with the launches that read it
    G.n = n;  // only once the tree is on the device
  }
  if (nb > G.cap) {
    HIPCHK(hipStreamSynchronize(be.stream));  // every reader of the old buffers has finished
    if (G.mem) (void)hipFree(G.mem);
    G.mem = nullptr;
    G.cap = 0;
    const size_t nn = (size_t)n * n;
    const GroupLayout L = group_layout(n, nb);
    const size_t sA = L.sA, sQ = L.sQ, sWi = L.sWi, sWd = L.sWd, sB = L.sB, sv = L.sv, sd = L.sd;
    const size_t total = L.total;
    if (dev_malloc(&G.mem, total) != hipSuccess) {
      (void)hipGetLastError();
      G.mem = nullptr;
      return fail(SLRX_ENOMEM, "eigen-decomposition buffers (%zu bytes)", total);
    }
    char* p = (char*)G.mem;
    auto take = [&](size_t b) {
      char* q = p;
      p += b;
      return q;
    };
    EighBufs& e = G.bufs;
    e.n = n;
    e.A = (double2*)take(nb * sA);
    e.V = (double2*)take(nb * sA);
    e.Z = (double2*)take(nb * sA);
    e.Q = (double*)take(nb * sQ);
    e.Qs = e.Q + nn;
    e.U = e.Q + 2 * nn;
    e.wsi = (int*)take(nb * sWi);
    e.wsd = (double*)take(nb * sWd);
    e.bts = (double2*)take(nb * sB);
    e.tau = (double2*)take(sv);
    e.triv[0] = (double2*)take(sv);
    e.triv[1] = (double2*)take(sv);
    e.trip[0] = (double2*)take(sv);
    e.trip[1] = (double2*)take(sv);
    e.D = (double*)take(sd);
    e.E = (double*)take(sd);
    e.sA = (long)(sA / sizeof(double2));
    e.sZ = e.sA;
    e.sQ = (long)(sQ / sizeof(double));
    e.s_wsi = (long)(sWi / sizeof(int));
    e.s_wsd = (long)(sWd / sizeof(double));
    e.s_bts = (long)(sB / sizeof(double2));
    G.cap = nb;
  }
  G.bufs.tree = G.tree;
  G.bufs.level_start = &G.level_start;
  G.bufs.node_sizes = &G.node_sizes;
  out = &G;
  return SLRX_OK;
}

slrx_status slrx::engine_begin(slrx_plan* pl, bool columns) {
  if (pl->direct() && pl->ncoils > 0) return fail(SLRX_EINVAL, "SLRX_FLAG_DIRECT is single-channel only");
  STCHK(prepare(pl));
  if (pl->direct()) STCHK(direct_setup(pl));
  pl->ktime = false;
  for (int c = 0; c < SLRX_K_NCLASS; ++c) pl->kused[c] = 0;
  HIPCHK(hipMemsetAsync(pl->info, 0, kInfoEntries * sizeof(rocblas_int), pl->stream));
  HIPCHK(hipEventRecord(pl->ev_run[0], pl->stream));
  pl->it_next = 0;
  pl->on_cg = nullptr;
  pl->tri_columns = columns;
  pl->running = true;
  pl->ran = false;
  pl->run_irls = pl->prm.n_irls;
  pl->run_timing = false;
  pl->inputs_kept = true;
  pl->gave_up = false;
  return SLRX_OK;
}

slrx_status slrx::engine_end(slrx_plan* pl) {
  HIPCHK(hipEventRecord(pl->ev_run[1], pl->stream));
  return SLRX_OK;
}

// CG strategy of the engine steps: -1 tuned online, 0 every problem on its own
// stream, 1 grouped launches (slrx_set_cg_grouping).
static std::atomic<int> g_cg_grouping{-1};

extern "C" void slrx_set_cg_grouping(int32_t mode) { g_cg_grouping.store(mode < 0 ? -1 : (mode > 0 ? 1 : 0)); }

// Plans whose CG joins a grouped launch (single-channel, FFT-based operator).
static bool cg_groupable(const slrx_plan* pl) { return pl->ncoils == 0 && !pl->direct(); }

// Problems i0 .. i0 + nb - 1 of a group.
static EighBufs sub_group(const EighBufs& e, int i0, int nb) {
  EighBufs s = e;
  const long o = (long)i0 * e.n;
  s.nb = nb;
  s.A += i0 * e.sA;
  s.V += i0 * e.sA;
  s.Z += i0 * e.sZ;
  s.Q += i0 * e.sQ;
  s.Qs += i0 * e.sQ;
  s.U += i0 * e.sQ;
  s.tau += o;
  for (int k = 0; k < 2; ++k) {
    s.triv[k] += o;
    s.trip[k] += o;
  }
  s.D += o;
  s.E += o;
  return s;
}

// One outer iteration of one problem on its own stream (the path of a plan run
// alone); with `deferred` the CG of a groupable plan is left to the grouped launch
// (its weights-done event recorded).
static slrx_status step_single(slrx_plan* pl, std::vector<slrx_plan*>* deferred = nullptr) {
  const int it = pl->it_next;
  pl->tri_stream = pl->stream;
  if (pl->direct()) {
    STCHK(step_direct_gram(pl));
    STCHK(step_eigh(pl, it));
    STCHK(step_direct_weights(pl, it, it == 0, pl->prm.gamma));
    STCHK(run_cg_direct(pl, pl->prm.n_cg, it));
    pl->it_next = it + 1;
    return SLRX_OK;
  }
  if (pl->voxel()) {
    STCHK(step_voxel(pl, it, it == 0, pl->prm.gamma));
  } else {
    STCHK(step_gram(pl));
    STCHK(step_eigh(pl, it));
    STCHK(step_weights(pl, it, it == 0, pl->prm.gamma));
  }
  if (deferred && cg_groupable(pl)) {  // deferred: the step runs its CG in grouped launches
    HIPCHK(hipEventRecord(pl->ev_step, pl->stream));
    pl->ev_weights = true;
    deferred->push_back(pl);
    return SLRX_OK;
  }
  STCHK(run_cg(pl, pl->prm.n_cg, it, false));
  pl->on_cg = nullptr;
  pl->it_next = it + 1;
  return SLRX_OK;
}

// The table entry of a plan (its buffers and its own grids).
static CgSlice cg_slice_of(const slrx_plan* pl) {
  const slrx_dims& d = pl->d;
  CgSlice c{};
  c.P = d.P; c.Q = d.Q; c.T = d.T;
  c.circ = (pl->prm.flags & SLRX_FLAG_GIRAF) ? 1 : 0;
  c.pen_scale = (float)(pl->prm.lambda / ((double)d.P * d.Q));
  c.x = pl->x; c.r = pl->r; c.p = pl->p; c.q = pl->q; c.t = pl->t;
  c.bm = pl->bm;
  c.S = pl->S;
  c.Et = pl->Et;
  c.twQ = pl->twQf;
  c.twP = pl->twPf;
  c.partA = pl->partA; c.partB = pl->partB; c.rr_hist = pl->rr_hist;
  c.flag = pl->flag;
  c.rr_out = pl->stats + 2 * SLRX_MAX_IRLS;
  cg_slice_grids(c);
  return c;
}

// The CG of one outer iteration for every plan of `g` (same M and n_cg) in grouped
// launches on the engine's CG stream, after each plan's weights (ev_step) and
// before its next work (the plans' streams wait for the CG).
static slrx_status run_cg_group(BatchEig& be, const std::vector<slrx_plan*>& g, int M, int n_cg) {
  if (!be.cg_stream) {
    HIPCHK(hipStreamCreateWithFlags(&be.cg_stream, hipStreamNonBlocking));
    HIPCHK(hipEventCreateWithFlags(&be.ev_cg, hipEventDisableTiming));
  }
  std::vector<CgSlice> host(g.size());
  int rows = 0, cols = 0, upd = 0;
  size_t pen_lds = 0;
  auto up8 = [](int n) { return (n + 7) & ~7; };
  for (size_t i = 0; i < g.size(); ++i) {
    CgSlice& c = host[i];
    c = cg_slice_of(g[i]);
    c.rows0 = rows;
    c.cols0 = cols;
    c.upd0 = upd;
    rows += up8(c.rows_gx * c.rows_gy);
    cols += up8(c.cols_gx);
    upd += up8(c.upd_gx);
    pen_lds = std::max(pen_lds, group_pen_lds(c.P, c.Q, c.T));
  }
  bool weights = false;  // some plan's weights were updated in a grouped launch
  for (slrx_plan* pl : g) {
    if (pl->ev_weights) HIPCHK(hipStreamWaitEvent(be.cg_stream, pl->ev_step, 0));
    else weights = true;
  }
  if (weights) HIPCHK(hipStreamWaitEvent(be.cg_stream, be.ev_w, 0));
  DevTable<CgSlice>& tb = be.cg_tables[std::make_pair(M, n_cg)];
  tb.step = be.step;
  STCHK(tb.upload(host, be.cg_stream));
  CgGroup G{};
  G.tab = tb.dev;
  G.ns = (int)host.size();
  G.M = M;
  G.rows_blocks = rows;
  G.cols_blocks = cols;
  G.upd_blocks = upd;
  G.pen_lds = pen_lds;
  hipStream_t s = be.cg_stream;
  // initial residual r = bm - A x, then n_cg iterations
  HIPCHK(launch_group_rows(G, ROW_PLAIN, 0, s));
  HIPCHK(launch_group_pen(G, s));
  HIPCHK(launch_group_fin(G, 1, 0, s));
  for (int k = 0; k < n_cg; ++k) {
    HIPCHK(launch_group_rows(G, k == 0 ? ROW_START : ROW_STEP, k, s));
    HIPCHK(launch_group_pen(G, s));
    HIPCHK(launch_group_fin(G, 0, k, s));
  }
  if (n_cg > 0) HIPCHK(launch_group_update(G, n_cg - 1, s));
  for (int i0 = 0; i0 < G.ns; i0 += kGroupIts) {
    const int n = std::min(kGroupIts, G.ns - i0);
    GroupIts it{};
    for (int i = 0; i < n; ++i) it.it[i] = (short)g[i0 + i]->it_next;
    HIPCHK(launch_group_store(G, i0, n, n_cg == 0, it, s));
  }
  HIPCHK(hipEventRecord(be.ev_cg, s));
  for (slrx_plan* pl : g) {
    HIPCHK(hipStreamWaitEvent(pl->stream, be.ev_cg, 0));
    pl->on_cg = &be;
    ++pl->it_next;
  }
  return SLRX_OK;
}

// A part of an eigen-decomposition group whose weight updates run as grouped launches on
// the engine's stream: problems of one filter, of which there are at least two, at most
// kGroupIts to a part (the last part may be a single problem).
struct WeightPart {
  std::vector<int> at;  // positions in the group
  WeightGroup G{};
};

// The Gram matrices of the part's problems into the group's buffers.
static slrx_status weight_part_gram(BatchEig& be, const EighBufs& e, const std::vector<slrx_plan*>& g,
                                    const std::vector<const int*>& stall, int part, WeightPart& wp) {
  bool cg = false;
  std::vector<WeightSlice> host(wp.at.size());
  WeightGroup& G = wp.G;
  const slrx_dims& d0 = g[wp.at[0]]->d;
  G.ns = (int)wp.at.size();
  G.N1 = d0.N1; G.N2 = d0.N2; G.M = d0.M;
  for (size_t k = 0; k < wp.at.size(); ++k) {
    const int i = wp.at[k];
    slrx_plan* pl = g[i];
    // after the problem's last work: the grouped CG, or what its own stream holds
    if (pl->on_cg == &be) {
      cg = true;
    } else {
      HIPCHK(hipEventRecord(pl->ev_step, pl->stream));
      HIPCHK(hipStreamWaitEvent(be.stream, pl->ev_step, 0));
    }
    const slrx_dims& d = pl->d;
    WeightSlice& c = host[k];
    std::memset((void*)&c, 0, sizeof c);
    c.x = pl->x;
    c.t = pl->t;
    c.img = pl->img;
    c.twP = pl->twPf;
    c.twQ = pl->twQf;
    c.img_scale = (float)(1.0 / std::sqrt((double)d.P * d.Q));
    c.gram = gram_args(pl, e.A + (size_t)i * e.sA, true);
    weight_args(pl, 0, false, pl->prm.gamma, e.Z + (size_t)i * e.sZ, e.D + (size_t)i * e.n, stall[i], c.w, c.spec,
                c.mask);
    G.ngroups = c.spec.ngroups;
    G.maxP = std::max(G.maxP, d.P);
    G.maxQ = std::max(G.maxQ, d.Q);
    G.maxPQ = std::max(G.maxPQ, (long)d.P * d.Q);
    G.row_blocks = std::max(G.row_blocks, image_row_blocks(d.P, d.T));
    G.col_blocks = std::max(G.col_blocks, image_col_blocks(d.Q, d.T));
  }
  if (cg) HIPCHK(hipStreamWaitEvent(be.stream, be.ev_cg, 0));
  DevTable<WeightSlice>& tb = be.weight_tables[WeightKey(d0.N1, d0.N2, d0.M, part)];
  tb.step = be.step;
  STCHK(tb.upload(host, be.stream));
  G.tab = tb.dev;
  HIPCHK(launch_group_images(G, be.stream));
  HIPCHK(launch_group_gram(G, be.stream));
  return SLRX_OK;
}

slrx_status slrx::engine_step(const std::vector<slrx_plan*>& plans, BatchEig& be) {
  roctxRangePushA("slrx engine step");  // host side: the enqueueing of one lock-step outer iteration
  struct PopRange {
    ~PopRange() { roctxRangePop(); }
  } pop;
  ++be.step;
  std::map<int, std::vector<slrx_plan*>> groups;
  std::vector<slrx_plan*> live;
  for (slrx_plan* pl : plans)
    if (pl->it_next < pl->prm.n_irls) live.push_back(pl);
  for (slrx_plan* pl : live)
    if (!(pl->lib_eigh() || pl->voxel() || pl->direct())) groups[pl->s()].push_back(pl);
  // The CG strategy of this step: each problem's CG on its own stream, or one
  // grouped launch per pass (bit-identical results).  Chosen per step shape by the
  // online tuner on whole-step times, once the tridiagonalisation's launch shape
  // for the step's groups is settled (so that one tuning does not time the other).
  int ng = 0, maxm = 0, maxcg = 0;
  long vsum = 0;
  for (slrx_plan* pl : live)
    if (cg_groupable(pl)) {
      ++ng;
      vsum += (long)pl->vol();
      maxm = std::max(maxm, pl->d.M);
      maxcg = std::max(maxcg, std::min(pl->prm.n_cg, 65535));
    }
  bool grouped = false;
  TuneTicket tk;
  const int forced = g_cg_grouping.load();
  if (forced >= 0) {
    grouped = forced == 1 && ng >= 1;
  } else if (ng >= 2) {
    bool settled = true;
    for (auto& kv : groups) {
      const int nb = (int)kv.second.size();
      if (tri_resident(kv.first)) continue;  // no launch shape to tune
      const int c = tune_choice(TUNE_TRI, kv.first, nb, 0);
      settled = settled && c >= 0 && tune_choice(TUNE_TRI_ACCESS, kv.first, nb, c) >= 0;
    }
    if (settled) {
      if (!be.cg_stream) {
        HIPCHK(hipStreamCreateWithFlags(&be.cg_stream, hipStreamNonBlocking));
        HIPCHK(hipEventCreateWithFlags(&be.ev_cg, hipEventDisableTiming));
      }
      for (slrx_plan* pl : live) {
        HIPCHK(hipEventRecord(pl->ev_begin, pl->stream));
        HIPCHK(hipStreamWaitEvent(be.cg_stream, pl->ev_begin, 0));
      }
      const int b = (int)std::min<long>(vsum >> 12, 1 << 30);
      grouped = tune_begin(TUNE_CG_GROUP, ng, b, (maxm << 16) | maxcg, 2, be.cg_stream, tk) == 1;
    }
  }
  std::vector<slrx_plan*> deferred;  // CG left to the grouped launches
  std::vector<slrx_plan*>* defer = grouped ? &deferred : nullptr;
  for (slrx_plan* pl : live)
    if (pl->lib_eigh() || pl->voxel() || pl->direct()) STCHK(step_single(pl, defer));
  bool used = false;
  for (auto& kv : groups) {
    const int n = kv.first;
    std::vector<slrx_plan*>& g = kv.second;
    const int nb = (int)g.size();
    EigGroup* G = nullptr;
    STCHK(group_reserve(be, n, nb, G));
    EighBufs e = G->bufs;
    e.nb = nb;
    // the problems whose run is repeated by column launches come last
    const bool resident = tri_resident(n) && tri_resident_on(be.stream);
    const int nres = resident ? (int)(std::stable_partition(g.begin(), g.end(),
                                                            [](const slrx_plan* pl) { return !pl->tri_columns; }) -
                                      g.begin())
                              : 0;
    // column launches neither read nor clear the group's flag: the word after its own stays 0
    std::vector<const int*> stall(nb);
    for (int i = 0; i < nb; ++i) {
      stall[i] = i < nres ? e.stall : e.stall + kStallWords;
      g[i]->tri_stream = be.stream;
    }
    // problems of one filter share launches of the weight update's kernels too (two or
    // more: one launch for all of them is never slower than their own, run at once)
    std::map<std::tuple<int, int, int>, std::vector<int>> filters;
    std::vector<int> alone;
    for (int i = 0; i < nb; ++i) {
      const slrx_dims& d = g[i]->d;
      if (spec_supported(d.N1, d.N2, d.M) && spec_groups(d.N1, d.N2, d.M, (size_t)n * n) > 0)
        filters[std::make_tuple(d.N1, d.N2, d.M)].push_back(i);
      else
        alone.push_back(i);
    }
    std::vector<WeightPart> parts;
    for (auto& f : filters) {
      const size_t m = f.second.size();
      if (m < 2) alone.push_back(f.second[0]);
      for (size_t k = 0; m >= 2 && k < m; k += kGroupIts) {
        parts.emplace_back();
        parts.back().at.assign(f.second.begin() + k, f.second.begin() + std::min(m, k + kGroupIts));
      }
    }
    // Gram matrices (row-major) into the group buffer once the previous step's readers are done
    for (size_t k = 0; k < parts.size(); ++k) STCHK(weight_part_gram(be, e, g, stall, (int)k, parts[k]));
    for (int i : alone) {
      slrx_plan* pl = g[i];
      if (be.have_free) HIPCHK(hipStreamWaitEvent(pl->stream, be.ev_free, 0));
      STCHK(step_gram(pl, false, e.A + (size_t)i * e.sA));
      HIPCHK(hipEventRecord(pl->ev_step, pl->stream));
      HIPCHK(hipStreamWaitEvent(be.stream, pl->ev_step, 0));
    }
    if (nres > 0) {
      EighBufs er = sub_group(e, 0, nres);
      er.tri_columns = false;
      er.clear_stall = G->clear_stall;
      G->clear_stall = false;
      HIPCHK(eigh_tri(er, be.stream));
    }
    if (nres < nb) {
      EighBufs ec = sub_group(e, nres, nb - nres);
      ec.tri_columns = true;
      HIPCHK(eigh_tri(ec, be.stream));
    }
    HIPCHK(eigh_tdeig(e, be.stream));
    HIPCHK(eigh_backtr(e, be.stream));
    HIPCHK(hipEventRecord(be.ev, be.stream));
    for (const WeightPart& wp : parts) {
      GroupIts its{};
      for (size_t k = 0; k < wp.at.size(); ++k) its.it[k] = (short)g[wp.at[k]]->it_next;
      HIPCHK(launch_group_weights(wp.G, its, be.stream));
      HIPCHK(hipEventRecord(be.ev_w, be.stream));
      for (int i : wp.at) {
        slrx_plan* pl = g[i];
        pl->ev_weights = false;
        if (grouped && cg_groupable(pl)) {
          deferred.push_back(pl);
        } else {
          HIPCHK(hipStreamWaitEvent(pl->stream, be.ev_w, 0));
          STCHK(run_cg(pl, pl->prm.n_cg, pl->it_next, false));
          pl->on_cg = nullptr;
          ++pl->it_next;
        }
      }
    }
    for (int i : alone) {
      slrx_plan* pl = g[i];
      const int it = pl->it_next;
      HIPCHK(hipStreamWaitEvent(pl->stream, be.ev, 0));
      STCHK(step_weights(pl, it, it == 0, pl->prm.gamma, e.Z + (size_t)i * e.sZ, e.D + (size_t)i * n, false,
                         stall[i]));
      HIPCHK(hipEventRecord(pl->ev_step, pl->stream));
      HIPCHK(hipStreamWaitEvent(be.stream, pl->ev_step, 0));
      pl->ev_weights = true;
      if (grouped && cg_groupable(pl)) {
        deferred.push_back(pl);
      } else {
        STCHK(run_cg(pl, pl->prm.n_cg, it, false));
        pl->on_cg = nullptr;
        pl->it_next = it + 1;
      }
    }
    used = true;
  }
  if (used) {
    HIPCHK(hipEventRecord(be.ev_free, be.stream));
    be.have_free = true;
  }
  // the CG of every deferred plan: one grouped launch per pass for each (M, n_cg)
  std::map<std::pair<int, int>, std::vector<slrx_plan*>> cg;
  for (slrx_plan* pl : deferred) cg[std::make_pair(pl->d.M, pl->prm.n_cg)].push_back(pl);
  for (auto& kv : cg) STCHK(run_cg_group(be, kv.second, kv.first.first, kv.first.second));
  if (tk.e1) {  // a timed step ends when every problem's CG has run
    for (slrx_plan* pl : live) {
      HIPCHK(hipEventRecord(pl->ev_step, pl->stream));
      HIPCHK(hipStreamWaitEvent(be.cg_stream, pl->ev_step, 0));
    }
    tune_end(tk, be.cg_stream);
  }
  return SLRX_OK;
}
