// C ABI of libbh: context, workspaces, argument checks and stage order.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <string>

#include "bh_device.h"

namespace bh {

namespace {

// Zero every word of the counters (one block; the struct is a few lines).
__global__ void k_reset_info(DevInfo *info) {
  static_assert(sizeof(DevInfo) % sizeof(int32_t) == 0, "DevInfo is a whole number of words");
  int32_t *w = reinterpret_cast<int32_t *>(info);
  for (int i = threadIdx.x; i < (int)(sizeof(DevInfo) / sizeof(int32_t)); i += blockDim.x) w[i] = 0;
}

__global__ void k_export_nodes(const NodeRec *__restrict__ nodes, const int8_t *__restrict__ meta,
                               const DevInfo *__restrict__ info, int nsys, int32_t *__restrict__ ints,
                               double *__restrict__ reals) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t slots = (int64_t)nsys + info->n_slots;
  if (k >= slots) return;
  const NodeRec r = nodes[k];
  const int mt = meta[k];
  const int kind = mt >> 5;
  const int level = ((mt & 31) == 31) ? -1 : (mt & 31);
  if (ints) {
    int32_t *o = ints + 6 * k;
    o[0] = level;
    o[1] = kind;
    o[2] = r.first;
    o[3] = r.count;
    o[4] = r.child;
    o[5] = r.nchild;
  }
  if (reals) {
    double *o = reals + 6 * k;
    o[0] = r.m;
    o[1] = r.com[0];
    o[2] = r.com[1];
    o[3] = r.com[2];
    o[4] = r.l;
    o[5] = r.s;
  }
}

// Second moments per slot; zero for particle leaves and empty roots (their
// rows of qmom are never written).
__global__ void k_export_moments(const NodeRec *__restrict__ nodes, const double *__restrict__ qmom,
                                 const DevInfo *__restrict__ info, int nsys, double *__restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t slots = (int64_t)nsys + info->n_slots;
  if (k >= slots) return;
  const bool leaf = nodes[k].child < 0;
  for (int j = 0; j < 6; ++j) out[6 * k + j] = leaf ? 0.0 : qmom[6 * k + j];
}

__global__ void k_copy_keys(const uint64_t *__restrict__ src, uint64_t *__restrict__ dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

__global__ void k_copy_i32(const int32_t *__restrict__ src, int32_t *__restrict__ dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

__global__ void k_export_groups(const int32_t *__restrict__ ginfo, const double *__restrict__ gbox,
                                const int32_t *__restrict__ glist, const double *__restrict__ gmass,
                                const DevInfo *__restrict__ info, int32_t *ints, double *box, int32_t *ll,
                                double *lm) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= info->n_groups) return;
  if (ints)
    for (int k = 0; k < 3; ++k) ints[3 * g + k] = ginfo[3 * g + k];
  if (box)
    for (int k = 0; k < 6; ++k) box[6 * g + k] = gbox[6 * g + k];
  if (ll) ll[g] = glist[g];
  if (lm) lm[g] = gmass[g];
}

inline unsigned blocks_for(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

}  // namespace

void reset_info_device(DevInfo *info, hipStream_t s) { k_reset_info<<<1, 256, 0, s>>>(info); }

bh_status fail(bh_ctx *c, bh_status st, const std::string &msg) {
  if (c) c->err = msg;
  return st;
}

bh_status hip_check(bh_ctx *c, hipError_t e, const char *what) {
  if (e == hipSuccess) return BH_OK;
  return fail(c, BH_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

bh_status ensure(bh_ctx *c, DevBuf &b, size_t bytes, const char *what) {
  if (bytes == 0) bytes = 16;
  if (b.bytes >= bytes) return BH_OK;
  if (c->capturing) return fail(c, BH_EINTERNAL, std::string("buffer growth while capturing: ") + what);
  if (c->graph) {  // the captured step points at the buffer about to move
    (void)hipGraphExecDestroy(c->graph);
    c->graph = nullptr;
  }
  if (b.p) {
    hipError_t e = hipFree(b.p);
    if (e != hipSuccess) return hip_check(c, e, "hipFree");
    b.p = nullptr;
    b.bytes = 0;
  }
  // grow geometrically so that slowly increasing sizes do not reallocate often
  size_t want = bytes + bytes / 8;
  hipError_t e = hipMalloc(&b.p, want);
  if (e != hipSuccess) {
    b.p = nullptr;
    (void)hipGetLastError();  // (reported here, not by the next launch's check)
    return fail(c, BH_ENOMEM, std::string("hipMalloc failed for ") + what);
  }
  b.bytes = want;
  b.fresh = true;
  return BH_OK;
}

static void free_buf(DevBuf &b) {
  if (b.p) (void)hipFree(b.p);
  b.p = nullptr;
  b.bytes = 0;
}

template <class T>
static T *P(DevBuf &b) {
  return reinterpret_cast<T *>(b.p);
}

// more: further work of the same call.
static bh_status timer_start(bh_ctx *c, Timer &t, bool more = false) {
  t.open = false;
  if (!c->opt.timing || c->capturing) return BH_OK;
  if (t.used >= 4096) return BH_OK;  // bounded: later calls of a long run are not timed
  while ((int)t.ev.size() < 2 * (t.used + 1)) {
    hipEvent_t e;
    bh_status st = hip_check(c, hipEventCreate(&e), "hipEventCreate");
    if (st) return st;
    t.ev.push_back(e);
  }
  t.open = true;
  t.more = more;
  return hip_check(c, hipEventRecord(t.ev[2 * t.used], c->stream), "hipEventRecord");
}

static bh_status timer_stop(bh_ctx *c, Timer &t) {
  if (!t.open) return BH_OK;
  t.open = false;
  bh_status st = hip_check(c, hipEventRecord(t.ev[2 * t.used + 1], c->stream), "hipEventRecord");
  if (st == BH_OK) {
    t.used++;
    t.calls += t.more ? 0 : 1;
  }
  return st;
}

// Sum of the recorded intervals (the stream must be synchronised); resets.
static double timer_take(Timer &t, int32_t *calls) {
  double total = 0.0;
  for (int k = 0; k < t.used; ++k) {
    float ms = 0.0f;
    if (hipEventElapsedTime(&ms, t.ev[2 * k], t.ev[2 * k + 1]) == hipSuccess) total += (double)ms;
  }
  *calls = t.calls;
  t.used = t.calls = 0;
  return total;
}

// Copy systems or parameters to the device through a pinned staging buffer,
// which is reused only after the previous upload has completed.
static bh_status upload(bh_ctx *c, void *dst, const void *src, size_t bytes) {
  if (bytes == 0) return BH_OK;
  if (c->capturing) return BH_OK;  // the eager run before the capture left the same data on the device
  c->data_moved = true;            // (a replay brings its own back)
  bh_status st;
  if (c->stage_event_used) {
    st = hip_check(c, hipEventSynchronize(c->stage_event), "hipEventSynchronize");
    if (st) return st;
  }
  if (c->stage_bytes < bytes) {
    if (c->stage) (void)hipHostFree(c->stage);
    c->stage = nullptr;
    c->stage_bytes = 0;
    st = hip_check(c, hipHostMalloc(&c->stage, bytes, 0), "hipHostMalloc");
    if (st) return st;
    c->stage_bytes = bytes;
  }
  memcpy(c->stage, src, bytes);
  st = hip_check(c, hipMemcpyAsync(dst, c->stage, bytes, hipMemcpyHostToDevice, c->stream), "hipMemcpyAsync");
  if (st) return st;
  if (!c->stage_event) {
    st = hip_check(c, hipEventCreateWithFlags(&c->stage_event, hipEventDisableTiming), "hipEventCreate");
    if (st) return st;
  }
  c->stage_event_used = true;
  return hip_check(c, hipEventRecord(c->stage_event, c->stream), "hipEventRecord");
}

static bh_status ensure_particles(bh_ctx *c, int64_t n, int nsys) {
  const size_t N = (size_t)std::max<int64_t>(n, 1);
  const size_t slots = 2 * N + (size_t)nsys + 1;
  const size_t hist = radix_hist_bytes((int64_t)N);
  const size_t scan_elems = std::max<size_t>(N, hist / sizeof(uint32_t)) + 1;
  // (cells above the subtrees are disjoint on each level)
  const size_t lists = 4 * (kKeyLevels + 1) * (N / (size_t)subtree_particles((int64_t)N, c->opt.quadrupole != 0, INT32_MAX) + 1);
  struct Want {
    DevBuf *b;
    size_t bytes;
    const char *name;
  } want[] = {
      {&c->keys[0], 8 * N, "keys"},       {&c->keys[1], 8 * N, "keys"},
      {&c->vals[0], 4 * N, "vals"},       {&c->vals[1], 4 * N, "vals"},
      {&c->sys_in, 4 * N, "sys_in"},      {&c->spos, 24 * N, "spos"},
      {&c->pmass, sizeof(PosMass) * N, "packed positions"},
      {&c->smass, 8 * N, "smass"},        {&c->perm, 4 * N, "perm"},
      {&c->delta, N, "delta"},            {&c->level, N, "level"},
      {&c->cdigit, N, "cdigit"},          {&c->pdigit, N, "pdigit"},
      {&c->owner, 4 * N, "owner"},        {&c->cfirst, 4 * N, "cfirst"},
      {&c->ccount, 4 * N, "ccount"},      {&c->cparent, 4 * N, "cparent"},
      {&c->pparent, 4 * N, "pparent"},    {&c->mask, 4 * (N + 16), "mask"},
      {&c->nchild, 4 * (N + 16), "nchild"}, {&c->cfirst_child, 4 * (N + 16), "cfirst_child"},
      {&c->cslot, 4 * N, "cslot"},        {&c->hist, hist, "hist"},
      {&c->scan_tmp, scan_tmp_bytes((int64_t)scan_elems), "scan_tmp"},
      {&c->nodes, sizeof(NodeRec) * slots, "nodes"},
      {&c->msum, 32 * slots, "msum"},
      {&c->meta, slots, "meta"},
      {&c->kind, N + 16, "cell classes"}, {&c->tiles, 32 * (N / 4096 + 1), "child scan"},
      {&c->subs, 2 * N + 4, "subtrees"},  {&c->pieces, lists, "pieces"},
      {&c->tops, lists, "top cells"},     {&c->highs, lists, "high cells"},
      {&c->highs2, lists, "high cells by level"},
      {&c->glen, 4 * (N + 16), "glen"},   {&c->ginfo, 12 * N, "ginfo"},
      {&c->gbox, 48 * N, "gbox"},         {&c->glist, 4 * N, "glist"},
      {&c->gmass, 8 * N, "gmass"},
      {&c->bbox_part, (size_t)6 * 8 * (size_t)nsys * (size_t)bbox_blocks_per_system(nsys), "bbox"},
      {&c->info, sizeof(DevInfo), "info"},
  };
  for (auto &w : want) {
    bh_status st = ensure(c, *w.b, w.bytes, w.name);
    if (st) return st;
  }
  return BH_OK;
}

static bh_status check_device_errors(bh_ctx *c) {
  bh_status st = hip_check(c, hipStreamSynchronize(c->stream), "hipStreamSynchronize");
  if (st) return st;
  if (!c->info.p) return BH_OK;
  st = hip_check(c, hipMemcpy(c->info_host, c->info.p, sizeof(DevInfo), hipMemcpyDeviceToHost), "hipMemcpy info");
  if (st) return st;
  const int32_t e = c->info_host->err;
  if (e & kErrNonFinitePos) return fail(c, BH_EINVAL, "non-finite particle position");
  if (e & kErrBadMass) return fail(c, BH_EINVAL, "particle mass negative or non-finite");
  if (e & kErrTheta) return fail(c, BH_EINVAL, "per-group theta outside [0, 1]");
  if (e & kErrBuild) return fail(c, BH_EINTERNAL, "tree build produced an inconsistent node layout");
  if (e & kErrStack) return fail(c, BH_EINTERNAL, "walk stack capacity exceeded or node range corrupt");
  if (e & kErrWide)
    return fail(c, BH_EINTERNAL, "more outlier groups, or longer lists of theirs, than the captured step has room for");
  if (e & kErrPool) return fail(c, BH_EINTERNAL, "interaction list pool exhausted");
  if (e & kErrWait) return fail(c, BH_EINTERNAL, "a bounded device wait timed out (walk task or sort look-back)");
  if (e & kErrRadius) return fail(c, BH_EINVAL, "search radius h must be positive and finite");
  if (e & kErrListSpace) return fail(c, BH_EINVAL, "neighbour list offsets do not match the neighbour counts");
  return BH_OK;
}

static bh_status build_common(bh_ctx *c, int32_t nsys, const int64_t *offsets, const double *pos,
                              const double *mass) {
  const int64_t n = offsets[nsys];
  if (n < 0 || n > BH_MAX_N) return fail(c, BH_EINVAL, "particle count out of range");
  if (n > 0 && (!pos || !mass)) return fail(c, BH_EINVAL, "pos and mass must not be NULL");
  c->have_tree = c->have_groups = c->have_forces = false;
  bh_status st = ensure_particles(c, n, nsys);
  if (st) return st;
  c->n = n;
  c->nsys = nsys;
  c->sys_host.assign((size_t)nsys, SysInfo{});
  for (int s = 0; s < nsys; ++s) {
    c->sys_host[s].first = (int32_t)offsets[s];
    c->sys_host[s].count = (int32_t)(offsets[s + 1] - offsets[s]);
  }
  st = ensure(c, c->sys, sizeof(SysInfo) * (size_t)nsys, "systems");
  if (st) return st;
  st = upload(c, c->sys.p, c->sys_host.data(), sizeof(SysInfo) * (size_t)nsys);
  if (st) return st;
  st = timer_start(c, c->t_build);
  if (st) return st;
  TreeBuffers B{};
  B.pos = pos;
  B.mass = mass;
  B.n = n;
  B.nsys = nsys;
  B.sys = P<SysInfo>(c->sys);
  B.info = P<DevInfo>(c->info);
  B.sys_in = P<int32_t>(c->sys_in);
  B.keys[0] = P<uint64_t>(c->keys[0]);
  B.keys[1] = P<uint64_t>(c->keys[1]);
  B.vals[0] = P<uint32_t>(c->vals[0]);
  B.vals[1] = P<uint32_t>(c->vals[1]);
  B.hist = P<uint32_t>(c->hist);
  B.scan_tmp = c->scan_tmp.p;
  B.bbox_part = P<double>(c->bbox_part);
  B.spos = P<double>(c->spos);
  B.smass = P<double>(c->smass);
  B.pm = P<PosMass>(c->pmass);
  B.perm = P<int32_t>(c->perm);
  B.delta = P<int8_t>(c->delta);
  B.level = P<int8_t>(c->level);
  B.cdigit = P<int8_t>(c->cdigit);
  B.pdigit = P<int8_t>(c->pdigit);
  B.owner = P<int32_t>(c->owner);
  B.cfirst = P<int32_t>(c->cfirst);
  B.ccount = P<int32_t>(c->ccount);
  B.cparent = P<int32_t>(c->cparent);
  B.pparent = P<int32_t>(c->pparent);
  B.mask = P<int32_t>(c->mask);
  B.nchild = P<int32_t>(c->nchild);
  B.cfc = P<int32_t>(c->cfirst_child);
  B.cslot = P<int32_t>(c->cslot);
  B.nodes = P<NodeRec>(c->nodes);
  B.msum = P<double>(c->msum);
  B.meta = P<int8_t>(c->meta);
  B.kind = P<uint8_t>(c->kind);
  B.tiles = P<int32_t>(c->tiles);
  B.subs = P<int32_t>(c->subs);
  B.pieces = P<int32_t>(c->pieces);
  B.tops = P<int32_t>(c->tops);
  B.highs = P<int32_t>(c->highs);
  B.highs2 = P<int32_t>(c->highs2);
  B.slot_cap = (int64_t)std::min({c->nodes.bytes / sizeof(NodeRec), c->msum.bytes / 32, c->meta.bytes});
  B.curve = c->opt.curve;
  B.any_empty = false;
  B.nonempty = B.largest = 0;
  for (int s = 0; s < nsys; ++s) {
    B.any_empty |= c->sys_host[s].count == 0;
    B.nonempty += c->sys_host[s].count > 0;
    B.largest = std::max(B.largest, (int)c->sys_host[s].count);
  }
  c->largest = B.largest;
  const bool quad = c->opt.quadrupole != 0;
  if (quad) {
    const size_t slots = (size_t)B.slot_cap;
    st = ensure(c, c->qmom, 48 * slots, "second moments");
    if (st) return st;
    st = ensure(c, c->qpack, 32 * slots, "packed second moments");
    if (st) return st;
    B.qmom = P<double>(c->qmom);
    B.qpack = P<float4>(c->qpack);
  }
  build_tree_device(B, c->stream);
  c->sorted_keys = B.sorted_keys;
  st = timer_stop(c, c->t_build);
  if (st) return st;
  st = hip_check(c, hipGetLastError(), "kernel launch (build)");
  if (st) return st;
  c->have_tree = true;
  c->have_quad = quad;
  c->have_neighbors = false;
  return BH_OK;
}

}  // namespace bh

using namespace bh;

extern "C" {

bh_status bh_create(bh_ctx **out, void *stream) {
  if (!out) return BH_EINVAL;
  *out = nullptr;
  bh_ctx *c = new (std::nothrow) bh_ctx();
  if (!c) return BH_ENOMEM;
  c->stream = (hipStream_t)stream;
  if (hipGetDevice(&c->device) != hipSuccess ||
      hipDeviceGetAttribute(&c->num_cu, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) {
    delete c;
    return BH_EHIP;
  }
  // a walk wave waits at most 2 s for a task (a guard: a task comes within
  // milliseconds, the length of the longest walk unit)
  int clock_khz = 0;
  if (hipDeviceGetAttribute(&clock_khz, hipDeviceAttributeWallClockRate, c->device) != hipSuccess || clock_khz <= 0)
    clock_khz = 100000;
  c->wait_ticks = (long long)clock_khz * 2000;
  // the no-allocation judge's static scratch: its address on this device
  if (judge_scratch_address(c->device, &c->judge_scratch) != hipSuccess || !c->judge_scratch) {
    delete c;
    return BH_EHIP;
  }
  if (hipHostMalloc((void **)&c->info_host, sizeof(DevInfo), 0) != hipSuccess) {
    delete c;
    return BH_ENOMEM;
  }
  memset(c->info_host, 0, sizeof(DevInfo));
  if (hipHostMalloc((void **)&c->split_host, sizeof(SplitCounters), 0) != hipSuccess) {
    (void)hipHostFree(c->info_host);
    delete c;
    return BH_ENOMEM;
  }
  memset(c->split_host, 0, sizeof(SplitCounters));
  *out = c;
  return BH_OK;
}

void bh_destroy(bh_ctx *c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->stream);
  DevBuf *bufs[] = {&c->keys[0], &c->keys[1], &c->vals[0], &c->vals[1], &c->sys_in, &c->spos, &c->smass,
                    &c->perm, &c->delta, &c->level, &c->cdigit, &c->pdigit, &c->owner, &c->cfirst, &c->ccount,
                    &c->cparent, &c->pparent, &c->mask, &c->nchild, &c->cfirst_child, &c->cslot, &c->scan_tmp,
                    &c->hist, &c->nodes, &c->msum, &c->meta, &c->kind, &c->tiles, &c->subs, &c->pieces, &c->tops, &c->highs, &c->highs2, &c->glen, &c->ginfo, &c->gbox, &c->glist,
                    &c->gmass, &c->bbox_part, &c->sys, &c->par, &c->info, &c->direct_part, &c->energy_part,
                    &c->glists, &c->far_pool, &c->near_pool, &c->far_next, &c->near_next,
                    &c->items, &c->pmass, &c->feps, &c->mlp_work, &c->mlp_feat, &c->pp_stat, &c->nb_out, &c->nb_count, &c->nb_rho, &c->order_hist, &c->walk_order, &c->walk_order_hist, &c->tasks, &c->ranges, &c->segs,
                    &c->split_ctr, &c->gsplit, &c->gnseg, &c->gsegfirst, &c->skeys[0], &c->skeys[1], &c->svals[0],
                    &c->svals[1], &c->shist, &c->sscan, &c->srows, &c->spbase, &c->sgroups, &c->psum,
                    &c->tile_buf, &c->wide_buf,
                    &c->qmom, &c->qpack, &c->far_slot};
  for (DevBuf *b : bufs) free_buf(*b);
  if (c->graph) (void)hipGraphExecDestroy(c->graph);
  if (c->capture_stream) (void)hipStreamDestroy(c->capture_stream);
  if (c->info_host) (void)hipHostFree(c->info_host);
  if (c->stage) (void)hipHostFree(c->stage);
  if (c->split_host) (void)hipHostFree(c->split_host);
  if (c->stage_event) (void)hipEventDestroy(c->stage_event);
  if (c->info_event) (void)hipEventDestroy(c->info_event);
  Timer *ts[] = {&c->t_build, &c->t_groups, &c->t_walk, &c->t_force, &c->t_particle, &c->t_neighbor, &c->t_theta};
  for (Timer *t : ts)
    for (hipEvent_t e : t->ev) (void)hipEventDestroy(e);
  delete c;
}

const char *bh_last_error(const bh_ctx *c) { return c ? c->err.c_str() : "null context"; }

bh_status bh_set_stream(bh_ctx *c, void *stream) {
  if (!c) return BH_EINVAL;
  c->stream = (hipStream_t)stream;
  return BH_OK;
}

bh_status bh_get_options(const bh_ctx *c, bh_options *opt) {
  if (!c || !opt) return BH_EINVAL;
  *opt = c->opt;
  return BH_OK;
}

bh_status bh_set_options(bh_ctx *c, const bh_options *opt) {
  if (!c || !opt) return BH_EINVAL;
  if (opt->waves_per_cu < 0 || opt->waves_per_cu > 32) return fail(c, BH_EINVAL, "waves_per_cu must be in [0, 32]");
  if (opt->split_visits < -1 || (opt->split_visits > 0 && opt->split_visits < 64))
    return fail(c, BH_EINVAL, "split_visits must be -1, 0 or >= 64");
  if (opt->quadrupole != 0 && opt->quadrupole != 1) return fail(c, BH_EINVAL, "quadrupole must be 0 or 1");
  if (opt->curve != 0 && opt->curve != 1) return fail(c, BH_EINVAL, "curve must be 0 (Morton) or 1 (Peano-Hilbert)");
  if (opt->list_tile != 0 && (opt->list_tile < kMinTile || opt->list_tile > kMaxTile ||
                              (opt->list_tile & (opt->list_tile - 1)) != 0))
    return fail(c, BH_EINVAL, "list_tile must be 0 or a power of two in [128, 2048]");
  c->opt = *opt;
  return BH_OK;
}

bh_status bh_sync(bh_ctx *c) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  return check_device_errors(c);
}

bh_status bh_build_tree(bh_ctx *c, int64_t n, const double *pos, const double *mass) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (n < 0 || n > BH_MAX_N) return fail(c, BH_EINVAL, "n out of range");
  int64_t off[2] = {0, n};
  return build_common(c, 1, off, pos, mass);
}

bh_status bh_build_batch(bh_ctx *c, int32_t n_systems, const int64_t *offsets, const double *pos,
                         const double *mass) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (n_systems < 1 || n_systems > 65536 || !offsets) return fail(c, BH_EINVAL, "n_systems must be in [1, 65536]");
  if (offsets[0] != 0) return fail(c, BH_EINVAL, "offsets[0] must be 0");
  for (int s = 0; s < n_systems; ++s)
    if (offsets[s + 1] < offsets[s]) return fail(c, BH_EINVAL, "offsets must be non-decreasing");
  return build_common(c, n_systems, offsets, pos, mass);
}

bh_status bh_make_groups(bh_ctx *c, int32_t n_crit, int64_t *n_groups_out) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!c->have_tree) return fail(c, BH_ESTATE, "bh_make_groups before a tree was built");
  if (n_crit < 1 || n_crit > BH_MAX_NCRIT) return fail(c, BH_EINVAL, "n_crit must be in [1, 256]");
  bh_status st = timer_start(c, c->t_groups);
  if (st) return st;
  GroupBuffers B{};
  B.n = c->n;
  B.nsys = c->nsys;
  B.n_crit = n_crit;
  B.level = P<int8_t>(c->level);
  B.ccount = P<int32_t>(c->ccount);
  B.cfc = P<int32_t>(c->cfirst_child);
  B.nchild = P<int32_t>(c->nchild);
  B.nodes = P<NodeRec>(c->nodes);
  B.sys = P<SysInfo>(c->sys);
  B.spos = P<double>(c->spos);
  B.info = P<DevInfo>(c->info);
  B.glen = P<int32_t>(c->glen);
  B.tiles = P<int32_t>(c->tiles);
  if (c->glen.fresh) {
    fill_i32(B.glen, 0, (int64_t)(c->glen.bytes / sizeof(int32_t)), c->stream);
    c->glen.fresh = false;
  }
  B.ginfo = P<int32_t>(c->ginfo);
  B.gbox = P<double>(c->gbox);
  B.num_cu = c->num_cu;
  make_groups_device(B, c->stream);
  c->xq_clean = c->counters_clean = true;
  st = timer_stop(c, c->t_groups);
  if (st) return st;
  st = hip_check(c, hipGetLastError(), "kernel launch (groups)");
  if (st) return st;
  c->n_crit = n_crit;
  c->have_groups = true;
  c->have_forces = false;
  c->walk_order_valid = false;
  if (n_groups_out) {
    st = check_device_errors(c);
    if (st) return st;
    *n_groups_out = c->info_host->n_groups;
  }
  return BH_OK;
}

// Sums by list tiles, and with quadrupoles the workgroup walk and list blocks
// (k_wide.hip), against a wave per group (k_walk.hip, k_force.hip): up to about
// 3000 groups, that is 2048 n_crit particles, the waves do not fill the chip and
// the longest list decides.  Quadrupole steps in us, workgroups against waves:
// clustered box of 300,000 particles at n_crit 256 1520 and 1690, of 500,000 2372
// and 2527, of 100,000 at n_crit 64 697 and 1026.  Monopole force calls, time by
// waves over time by tiles at theta 0.3 and 0.6 (sphere; clustered box; Plummer):
//   n_crit 16, 32,000    1.20 1.28   1.25 1.28   1.29 1.19
//   n_crit 64, 131,000   1.07 0.97   1.29 1.23   1.18 1.30
//   n_crit 128, 262,000  0.99 0.94   1.28 1.35   1.00 1.04
//   n_crit 256, 300,000  0.97 1.01   1.10 1.20   1.00 1.00
//               350,000  0.87 0.95   0.97 1.14   0.94 0.96
//               400,000  0.88 0.96   0.96 1.02   0.96 0.98
//               500,000  0.97 0.91   0.90 1.04   0.91 0.90
// The waves take blocks of 64 members, so beyond kTileParticles, some 6000
// blocks, they are enough at any n_crit.  Every list takes at least one far and
// one near block, so groups smaller than kWideMinCrit stay with the waves.
constexpr int64_t kWideGroups = 2048;
constexpr int64_t kTileParticles = 400000;
constexpr int kWideMinCrit = 16;
// Fewest node tests that make a group an outlier (see outlier_cap): a walk
// this long is a small part of a launch (16 iterations of 256 threads, 256
// batches of a wave).  In systems of up to kOutMinTree particles the walk of
// everything is over before tasks could be (walk of 5000, 8192 Plummer
// particles at theta 0.75: 47, 77 us with one workgroup a group, 64, 64 us with
// tasks; batch of 78 spheres of 5000 at n_crit 256, forces: 1140 us with the 254
// outliers apart, 848 with none, with quadrupoles 1474 and 1174).
constexpr int kOutMinWide = 4096;
constexpr int kOutMinTree = 6500;
constexpr int64_t kOutMin = 16384;
// Beyond 4.2 million particles an outlier makes at least as many tests as a
// wave of the walk does for 16 particles of its share: where the ordinary groups
// keep the waves busy that long, the launch does not wait for it.  The walk that
// is given up counts too, whenever it started, so the line lies low: Plummer
// spheres, n_crit 64, forces in us with 16 and with 40 in this place: 20 spheres
// of 400,000 13711 and 14999, 40 of 100,000 6740 and 7180, 256 of 20,000 8725 and
// 7277, 512 13749 and 13858 (with the line at kOutMin, 1088 outliers, 17351).
constexpr int kOutMinShare = 16;
// Largest tree with outliers apart, and their block length: a task's list (at
// most kTaskNodes cells of n / 2048 particles) then fits the block table.
constexpr int64_t kOutMaxN = 1 << 26;
constexpr int kOutBlock = 256;

// Whether there are too few groups to fill the chip with a wave each, and the
// tuning options (split cap, list tile, waves), each of which asks for the
// single-wave kernels in a given form, are at their defaults.  The lists are
// then summed by tiles (forces_tiles).  Sums with quadrupoles take the
// workgroup walk and list blocks throughout (forces_wide), unless the context
// integrates (a kick, a drift or leapfrog steps ran on it).  Monopole sums keep
// the single waves' list order and FP32 chains at every size, because an
// integration may start from any of them: in other orders their roundings
// differ by up to 4e-7 of the force, and 1.5e-8 of the velocities after four
// leapfrog steps in a clustered box, although no sum is less exact.  That costs
// (whole steps of 1000 and 8192 Plummer particles and of 100,003 in a sphere,
// us, by waves and tiles against workgroups: 207 against 108, 357 against 184,
// 524 against 417).  Outliers hold too few members, and in places too sparse,
// to matter: velocities and energies of boxes and spheres of 1100 to 240,000
// particles move by at most 1.2e-11 (with outliers from twice an ordinary walk
// on, rather than four times, by 7e-9).
static bool few_groups(const bh_ctx *c) {
  return c->opt.split_visits == 0 && c->opt.list_tile == 0 && c->opt.waves_per_cu == 0 &&
         c->n_crit >= kWideMinCrit && c->n <= kWideGroups * c->n_crit &&
         (c->opt.quadrupole || c->n <= kTileParticles) && wide_fits(c->n);
}

// Outliers walked and summed together: 80 KiB of tables each, and a lot costs
// its launches and a wait (100 Plummer spheres of 14,000 particles far apart in
// one system, n_crit 256, 259 outliers, forces: 2895 us by 64, 2621 by 256, 2410
// with none apart; 40 of 40,000, 148 outliers: 2927, 2711, 5565).
static int out_lot(const bh_ctx *c) { return c->nsys == 1 && c->n <= kTileParticles ? kOutSingle : kOutMax; }

static size_t padded(size_t bytes) { return (bytes + 255) & ~(size_t)255; }

// The outliers of the lists' walk (behind the queue order bins; not with the
// tables, which may move between lots).
static int32_t *out_list(const bh_ctx *c) { return (int32_t *)((char *)c->order_hist.p + padded(order_hist_bytes())); }

// Arguments and buffers of the workgroup kernels (the pool holds c->wide_cap
// blocks).  groups: the ordinary groups too, not only outliers.
static bh_status wide_args(bh_ctx *c, bool groups, const float *theta_group, float *acc, float *pot, WideArgs &A) {
  const bool quad = c->opt.quadrupole != 0;
  const int block = c->wide_block;
  const size_t cap = (size_t)c->wide_cap;
  A.lot = groups ? kOutMax : out_lot(c);
  const size_t lot = (size_t)A.lot;
  // (one allocation: a dozen of them are a good part of a first call)
  struct {
    void **p;
    size_t bytes;
  } want[] = {{(void **)&A.pool, cap * block * sizeof(float4)},
              {(void **)&A.slot, quad ? cap * block * sizeof(int32_t) : 0},
              {(void **)&A.gblocks, groups ? sizeof(int2) * (size_t)c->n : 0},
              {(void **)&A.gstat, groups ? sizeof(int2) * (size_t)c->n : 0},
              {(void **)&A.binfo, cap * sizeof(int4)},
              {(void **)&A.psum, cap * (size_t)c->n_crit * 4 * sizeof(double)},
              {(void **)&A.out, groups ? sizeof(int32_t) * lot : 0},
              {(void **)&A.outinfo, sizeof(OutInfo) * lot},
              {(void **)&A.tnodes, sizeof(int32_t) * lot * kOutNodes},
              {(void **)&A.tasks, sizeof(int4) * lot * kOutTasks},
              {(void **)&A.trows, sizeof(int4) * lot * kOutTasks},
              {(void **)&A.tnear, sizeof(int32_t) * lot * kOutTasks},
              {(void **)&A.tmass, sizeof(double) * lot * kOutTasks}};
  size_t total = 0;
  for (auto &w : want) total += padded(w.bytes);
  bh_status st = ensure(c, c->wide_buf, total, "list blocks");
  if (st) return st;
  char *at = P<char>(c->wide_buf);
  for (auto &w : want) {
    *w.p = w.bytes ? at : nullptr;
    at += padded(w.bytes);
  }
  if (!groups) A.out = out_list(c);
  A.out_places = groups ? (int)lot : kOutPlaces;
  A.nodes = P<NodeRec>(c->nodes);
  A.sys = P<SysInfo>(c->sys);
  A.ginfo = P<int32_t>(c->ginfo);
  A.gbox = P<double>(c->gbox);
  A.par = P<SysParam>(c->par);
  A.theta_group = theta_group;
  A.info = P<DevInfo>(c->info);
  A.nsys = c->nsys;
  A.n_crit = c->n_crit;
  A.block = block;
  for (A.block_log = 0; (1 << A.block_log) < block;) ++A.block_log;
  A.block_cap = c->wide_cap;
  A.qpack = quad ? P<float4>(c->qpack) : nullptr;
  A.glist = P<int32_t>(c->glist);
  A.gmass = P<double>(c->gmass);
  A.spos = P<double>(c->spos);
  A.smass = P<double>(c->smass);
  A.perm = P<int32_t>(c->perm);
  A.acc = acc;
  A.pot = pot;
  return BH_OK;
}

// The pool's capacity counts blocks of one length: recount when it changes,
// and start from at least `want` blocks.
static void wide_capacity(bh_ctx *c, int block, int64_t want) {
  if (c->wide_block != block) {
    c->wide_cap = (int32_t)((int64_t)c->wide_cap * c->wide_block / block);
    c->wide_block = block;
  }
  if (!c->capturing && c->wide_cap < want) c->wide_cap = (int32_t)std::min<int64_t>(want, INT32_MAX / 2);
}

// List blocks of outliers to start from.  A captured step has to have room for
// replays with a few: each workgroup on their tasks holds up to two runs.
static int64_t out_blocks(const bh_ctx *c, bool few) {
  const int64_t tasks = 8 * std::min<int64_t>(kOutTasks, c->n / kOutBlock + 1);
  return 2 * c->n / kOutBlock + (few ? 512 : 4096) +
         (c->reserve ? 2 * kSpare * std::min<int64_t>(kTaskGroups * c->num_cu, tasks) : 0);
}

// The walk's counters have arrived: rows of list blocks beyond their arrays.
static bool wide_overrun(const bh_ctx *c) { return c->info_host->rows > c->wide_cap; }

static void wide_grow(bh_ctx *c) {
  const int64_t need = std::max(c->info_host->blocks, c->info_host->blocks_done);
  if (need > c->wide_cap) c->wide_cap = (int32_t)std::min<int64_t>(need + need / 4 + 64, INT32_MAX / 2);
}

// The force call by workgroup walk and list blocks (parameters uploaded).
static bh_status forces_wide(bh_ctx *c, const float *theta_group, float *acc, float *pot) {
  const int64_t n = c->n;
  // 48 entries per particle and a few partly filled blocks per group to start
  // with; grown to what a walk reports it needed
  const int block = wide_block_length(n);
  wide_capacity(c, block, 48 * n / block + 6 * n / c->n_crit + 96 * (int64_t)c->num_cu);
  if (!c->info_event) {
    bh_status st = hip_check(c, hipEventCreateWithFlags(&c->info_event, hipEventDisableTiming), "hipEventCreate");
    if (st) return st;
  }
  if (!c->capturing) c->out_off = false;
  for (int attempt = 0;; ++attempt) {
    WideArgs A{};
    bh_status st = wide_args(c, true, theta_group, acc, pot, A);
    if (st) return st;
    const bool outliers = c->largest > kOutMinTree && !c->out_off;
    A.out_min = outliers ? kOutMinWide : 0;
    A.out_tree = kOutMinTree;
    if (!c->counters_clean) reset_list_counters(P<DevInfo>(c->info), c->stream);
    c->counters_clean = false;
    st = timer_start(c, c->t_walk);
    if (st) return st;
    walk_wide_device(A, n, c->num_cu, c->stream);
    if (outliers) walk_tasks_device(A, c->num_cu, c->stream);
    st = timer_stop(c, c->t_walk);
    if (st) return st;
    // The sums are queued behind the walk and leave at once when a list did
    // not fit; the host looks at the walk's counters meanwhile (a captured
    // step cannot: an overflow then leaves kErrPool for bh_sync).
    if (!c->capturing) {
      st = hip_check(c, hipMemcpyAsync(c->info_host, c->info.p, sizeof(DevInfo), hipMemcpyDeviceToHost, c->stream),
                     "hipMemcpyAsync info");
      if (!st) st = hip_check(c, hipEventRecord(c->info_event, c->stream), "hipEventRecord");
      if (st) return st;
    }
    st = timer_start(c, c->t_force, attempt > 0);
    if (st) return st;
    force_blocks_device(A, c->num_cu, c->stream);
    block_reduce_device(A, c->num_cu, true, c->stream);
    if (outliers) task_reduce_device(A, c->stream);
    st = timer_stop(c, c->t_force);
    if (st) return st;
    st = hip_check(c, hipGetLastError(), "kernel launch (force)");
    if (st) return st;
    c->last_attempts = attempt + 1;
    if (c->capturing) break;
    st = hip_check(c, hipEventSynchronize(c->info_event), "hipEventSynchronize");
    if (st) return st;
    if (wide_overrun(c)) return fail(c, BH_EINTERNAL, "more rows of list blocks than blocks");
    if (!(c->info_host->err & (kErrPool | kErrWide))) break;
    if (attempt > 5) return fail(c, BH_EINTERNAL, "interaction list pool still too small after growing");
    if (c->info_host->err & kErrWide) c->out_off = true;  // every group by one workgroup
    wide_grow(c);
  }
  c->last_segments = c->last_split_groups = c->last_depth = 0;
  c->have_forces = true;
  return BH_OK;
}

// Rows of partial sums of this tree's lists by their ordinary length (see
// outlier_cap), times what earlier calls needed more than that: the pools'
// capacities count chunks for any earlier tree.
static int64_t tile_rows_room(const bh_ctx *c) {
  double theta = 1.0;
  for (const SysParam &p : c->par_host) theta = std::min(theta, p.theta);
  const double octaves = std::max(1.0, log2((double)c->n / c->n_crit) / 3.0);
  const double len = std::min((double)c->n, (60.0 + 25.0 * sqrt((double)c->n_crit)) * octaves / pow(std::max(theta, 1e-3), 1.5));
  const double groups = (double)std::min<int64_t>(c->n, 3 * c->n / (2 * c->n_crit) + 1 + c->nsys);
  const double rows = groups * (1.4 * len / kDefaultTile + 2.2) + 16.0;
  return (int64_t)std::min(rows * c->tile_factor * (c->reserve ? 1.25 : 1.0), 1e9);
}

// The sums over the single waves' lists by tiles, and the outliers' (O); the
// counters' read-back in between.
static bh_status forces_tiles(bh_ctx *c, const WalkListArgs &W, const WideArgs &O, bool outliers, bool again,
                              float *acc, float *pot) {
  // (a tile takes a chunk of a pool: no more rows than chunks)
  const size_t most = (size_t)W.far_cap + (size_t)W.near_cap;
  const size_t rows = std::min(most, (size_t)tile_rows_room(c));
  const size_t b0 = padded(sizeof(double) * 4 * rows * (size_t)c->n_crit), b1 = padded(sizeof(int4) * rows);
  bh_status st = ensure(c, c->tile_buf, b0 + b1 + sizeof(int2) * (size_t)c->n, "list tiles");
  if (st) return st;
  TileArgs T{};
  T.ginfo = W.ginfo;
  T.glist = W.glist;
  T.gbox = W.gbox;
  T.glists = W.glists;
  T.far_next = W.far_next;
  T.near_next = W.near_next;
  T.far_pool = W.far_pool;
  T.near_pool = W.near_pool;
  T.far_slot = W.far_slot;
  T.qpack = W.far_slot ? P<float4>(c->qpack) : nullptr;
  T.far_tile = W.far_tile;
  T.near_tile = W.near_tile;
  T.n_crit = c->n_crit;
  T.spos = P<double>(c->spos);
  T.par = W.par;
  T.info = W.info;
  T.psum = P<double>(c->tile_buf);
  T.tinfo = (int4 *)(P<char>(c->tile_buf) + b0);
  T.gblocks = (int2 *)(P<char>(c->tile_buf) + b0 + b1);
  T.row_cap = (int)rows;
  WideArgs R{};
  R.ginfo = W.ginfo;
  R.info = W.info;
  R.n_crit = c->n_crit;
  R.gblocks = T.gblocks;
  R.psum = T.psum;
  R.par = W.par;
  R.smass = P<double>(c->smass);
  R.perm = P<int32_t>(c->perm);
  R.acc = acc;
  R.pot = pot;
  st = timer_start(c, c->t_force, again);
  if (st) return st;
  tile_rows_device(T, c->stream);
  if (!c->capturing) {
    st = hip_check(c, hipMemcpyAsync(c->info_host, c->info.p, sizeof(DevInfo), hipMemcpyDeviceToHost, c->stream),
                   "hipMemcpyAsync info");
    if (!st) st = hip_check(c, hipEventRecord(c->info_event, c->stream), "hipEventRecord");
    if (st) return st;
  }
  force_tiles_device(T, c->num_cu, c->stream);
  block_reduce_device(R, c->num_cu, false, c->stream);
  if (outliers) {
    // (after the lists' sums, which leave an outlier's members with none)
    force_blocks_device(O, c->num_cu, c->stream);
    task_reduce_device(O, c->stream);
  }
  st = timer_stop(c, c->t_force);
  if (!st) st = hip_check(c, hipGetLastError(), "kernel launch (force)");
  c->have_forces = !st;
  return st;
}

// The outliers of the lists' walk, out_lot at a time from the `first` such lot
// on, their sums after the lists' (which leave an outlier's members with
// none).  *whole: one of their lists does not fit, every group has to be walked
// whole.  A captured step records as many lots as its eager run's outliers and a
// quarter more would fill.  (128 Plummer spheres of 20,000 particles, 272
// outliers, forces: 7169 us with every group walked a second time, whole, where
// they are more than 256, 4731 in lots.)
static bh_status outlier_rounds(bh_ctx *c, const float *theta_group, float *acc, float *pot, int first, bool *whole) {
  *whole = false;
  const int lot = out_lot(c), n_out = std::min(c->info_host->n_out, kOutPlaces);
  if (!c->capturing) c->out_rounds = std::max((n_out + n_out / 4 + lot - 1) / lot, 1);
  const int rounds = c->capturing ? c->out_rounds : (n_out + lot - 1) / lot;
  for (int r = first; r < rounds; ++r) {
    WideArgs A{};
    for (int attempt = 0;; ++attempt) {
      bh_status st = wide_args(c, false, theta_group, acc, pot, A);
      if (st == BH_ENOMEM && !c->capturing) {  // whole, then: that needs no more memory
        *whole = true;
        return BH_OK;
      }
      if (st) return st;
      A.out_first = r * lot;
      A.out_limit = c->capturing ? c->out_rounds * lot : 0;
      st = timer_start(c, c->t_walk, true);
      if (st) return st;
      if (r > 0 || attempt > 0) next_outliers_device(A.info, attempt > 0, c->stream);
      walk_outliers_device(A, c->stream);
      walk_tasks_device(A, c->num_cu, c->stream);
      st = timer_stop(c, c->t_walk);
      if (st) return st;
      if (c->capturing) break;
      st = hip_check(c, hipMemcpyAsync(c->info_host, c->info.p, sizeof(DevInfo), hipMemcpyDeviceToHost, c->stream),
                     "hipMemcpyAsync info");
      if (!st) st = hip_check(c, hipStreamSynchronize(c->stream), "hipStreamSynchronize");
      if (st) return st;
      if (wide_overrun(c)) return fail(c, BH_EINTERNAL, "more rows of list blocks than blocks");
      if (c->info_host->err & kErrWide) {
        *whole = true;
        return BH_OK;
      }
      if (!(c->info_host->err & kErrPool)) break;
      if (attempt > 5) return fail(c, BH_EINTERNAL, "interaction list pool still too small after growing");
      wide_grow(c);
    }
    bh_status st = timer_start(c, c->t_force, true);
    if (st) return st;
    force_blocks_device(A, c->num_cu, c->stream);
    task_reduce_device(A, c->stream);
    st = timer_stop(c, c->t_force);
    if (st) return st;
  }
  return hip_check(c, hipGetLastError(), "kernel launch (outliers)");
}

// walk_whole: no outliers apart (they had lists that do not fit).
static bh_status forces_common(bh_ctx *c, const double *eps_sys, const double *theta_sys, const float *theta_group,
                               float *acc, float *pot, bool walk_whole = false) {
  if (!c->have_groups) return fail(c, BH_ESTATE, "forces requested before bh_make_groups");
  if (c->n > 0 && (!acc || !pot)) return fail(c, BH_EINVAL, "acc and pot must not be NULL");
  const bool quad = c->opt.quadrupole != 0;
  if (quad && !c->have_quad)
    return fail(c, BH_ESTATE, "quadrupole sums need a tree built with the quadrupole option set");
  c->par_host.assign((size_t)c->nsys, SysParam{});
  for (int s = 0; s < c->nsys; ++s) {
    const double e = eps_sys[s], t = theta_sys[s];
    if (!(e > 0.0) || !isfinite(e)) return fail(c, BH_EINVAL, "eps must be positive and finite");
    const float e2 = (float)(e * e);
    if (!(e2 >= 1.17549435e-38f) || isinf(e2)) return fail(c, BH_EINVAL, "eps^2 must be a normal FP32 number");
    if (!(t >= 0.0 && t <= 1.0)) return fail(c, BH_EINVAL, "theta must be in [0, 1]");
    c->par_host[s].eps = e;
    c->par_host[s].theta = t;
  }
  bh_status st = ensure(c, c->par, sizeof(SysParam) * (size_t)c->nsys, "parameters");
  if (st) return st;
  st = upload(c, c->par.p, c->par_host.data(), sizeof(SysParam) * (size_t)c->nsys);
  if (st) return st;
  if (c->n == 0) {
    c->have_forces = true;
    return BH_OK;
  }
  const bool few = few_groups(c);
  if (few && quad && !c->integrates) return forces_wide(c, theta_group, acc, pot);
  // list pools: start from an estimate (32 far and 4 near entries per
  // particle), grow to what a walk reports it needed; the capacities count
  // chunks of the current tile (recounted when the tile changes)
  const int tile = c->opt.list_tile > 0 ? c->opt.list_tile : kDefaultTile;
  if (c->far_cap == 0) {
    c->far_cap = (int32_t)std::max<int64_t>(4096, 32 * c->n / tile);
    c->near_cap = (int32_t)std::max<int64_t>(4096, 8 * c->n / tile);
  } else if (c->pool_tile != tile) {
    c->far_cap = (int32_t)std::min<int64_t>((int64_t)c->far_cap * c->pool_tile / tile + 64, INT32_MAX / 2);
    c->near_cap = (int32_t)std::min<int64_t>((int64_t)c->near_cap * c->pool_tile / tile + 64, INT32_MAX / 2);
  }
  c->pool_tile = tile;
  WalkListArgs W{};
  W.nodes = P<NodeRec>(c->nodes);
  W.sys = P<SysInfo>(c->sys);
  W.ginfo = P<int32_t>(c->ginfo);
  W.gbox = P<double>(c->gbox);
  W.par = P<SysParam>(c->par);
  W.theta_group = theta_group;
  W.info = P<DevInfo>(c->info);
  W.nsys = c->nsys;
  W.glist = P<int32_t>(c->glist);
  W.gmass = P<double>(c->gmass);
  if (!c->walk_bpc) {
    c->walk_bpc = walk_lists_blocks_per_cu();
    c->force_bpc = force_lists_blocks_per_cu(false);
    c->force_bpc_q = force_lists_blocks_per_cu(true);
  }
  const size_t gcap = (size_t)std::max<int64_t>(c->n, 1);
  // split walks (long lists walked and summed by several waves)
  const int grid = c->num_cu * (c->opt.waves_per_cu > 0 ? c->opt.waves_per_cu : c->walk_bpc);
  const int fgrid = c->num_cu * (c->opt.waves_per_cu > 0 ? c->opt.waves_per_cu : (quad ? c->force_bpc_q : c->force_bpc));
  // Split walks only on request; by default outliers go to the workgroup walk.
  const int visit_cap = std::max(c->opt.split_visits, 0);
  if (!c->capturing) {
    c->out_off = walk_whole;
    c->out_rounds = 1;
  }
  const int out_min =
      few ? kOutMinWide
          : (int)std::min<int64_t>(std::max(kOutMin, kOutMinShare * c->n / (c->num_cu * c->walk_bpc)), INT32_MAX);
  bool outliers = c->opt.split_visits == 0 && c->n <= kOutMaxN && (few ? c->largest > kOutMinTree : 2 * (int64_t)c->largest > out_min) && !c->out_off;
  if (outliers) {
    // (with a wave per group the host sees first whether there are any; a captured
    // step's replays may have them)
    if (few || c->reserve) wide_capacity(c, kOutBlock, out_blocks(c, few));
  }
  if (c->seg_cap == 0) {
    c->task_cap = 4096;
    c->range_cap = 1 << 16;
    c->seg_cap = 4096;
  }
  if (!c->order_hist.p) {
    st = ensure(c, c->order_hist, padded(order_hist_bytes()) + sizeof(int32_t) * kOutPlaces, "queue order bins");
    if (st) return st;
    order_clear_device(P<int32_t>(c->order_hist), c->stream);  // every later call leaves it zero
  }
  if (st) return st;
  if (few && !c->info_event) {
    st = hip_check(c, hipEventCreateWithFlags(&c->info_event, hipEventDisableTiming), "hipEventCreate");
    if (st) return st;
  }
  SplitBuffers S{};
  int32_t nsegs_host = 0;
  bool have_out = outliers;  // (a capture replays on other particles: it always has the outliers' launches)
  for (int attempt = 0;; ++attempt) {
    st = ensure(c, c->far_pool, (size_t)c->far_cap * tile * sizeof(float4), "far list pool");
    if (st) return st;
    st = ensure(c, c->far_next, (size_t)c->far_cap * sizeof(int32_t), "far list links");
    if (st) return st;
    if (quad) {
      st = ensure(c, c->far_slot, (size_t)c->far_cap * tile * sizeof(int32_t), "far list node slots");
      if (st) return st;
    }
    st = ensure(c, c->near_pool, (size_t)c->near_cap * tile * sizeof(float4), "near list pool");
    if (st) return st;
    st = ensure(c, c->near_next, (size_t)c->near_cap * sizeof(int32_t), "near list links");
    if (st) return st;
    st = ensure(c, c->glists, (size_t)4 * sizeof(int32_t) * gcap, "group lists");
    if (st) return st;
    const size_t sc = (size_t)c->seg_cap;
    DevBuf *sb[] = {&c->tasks, &c->ranges, &c->segs, &c->split_ctr, &c->gsplit, &c->gnseg,
                    &c->gsegfirst, &c->skeys[0], &c->skeys[1], &c->svals[0], &c->svals[1], &c->shist,
                    &c->sscan, &c->srows, &c->spbase, &c->sgroups};
    const size_t sz[] = {sizeof(WalkTask) * (size_t)c->task_cap,
                         sizeof(int2) * (size_t)c->range_cap, sizeof(Segment) * sc, sizeof(SplitCounters) + 64,
                         sizeof(int32_t) * gcap, sizeof(int32_t) * gcap, sizeof(int32_t) * gcap, 8 * sc, 8 * sc,
                         4 * sc, 4 * sc, radix_hist_bytes((int64_t)sc), scan_tmp_bytes((int64_t)sc) + 256,
                         4 * sc, 4 * sc + 16, 4 * sc};
    for (int k = 0; k < (int)(sizeof(sz) / sizeof(sz[0])); ++k) {
      st = ensure(c, *sb[k], sz[k], "split walk buffers");
      if (st) return st;
    }
    W.far_pool = P<float4>(c->far_pool);
    W.near_pool = P<float4>(c->near_pool);
    W.far_next = P<int32_t>(c->far_next);
    W.near_next = P<int32_t>(c->near_next);
    W.far_slot = quad ? P<int32_t>(c->far_slot) : nullptr;
    W.far_cap = c->far_cap;
    W.near_cap = c->near_cap;
    W.far_tile = tile;
    W.near_tile = tile / 2;
    W.glists = P<int32_t>(c->glists);
    W.ctr = P<SplitCounters>(c->split_ctr);
    W.tasks = P<WalkTask>(c->tasks);
    W.task_cap = c->task_cap;
    W.ranges = P<int2>(c->ranges);
    W.range_cap = c->range_cap;
    W.segs = P<Segment>(c->segs);
    W.seg_cap = c->seg_cap;
    W.gsplit = P<int32_t>(c->gsplit);
    W.visit_cap = visit_cap;
    W.out_min = outliers ? out_min : 0;
    W.out_tree = few ? kOutMinTree : 0;
    W.n_crit = c->n_crit;
    WideArgs A{};
    if (outliers) {
      W.out = out_list(c);
      W.out_places = kOutPlaces;
      if (few || c->reserve) {
        st = wide_args(c, false, theta_group, acc, pot, A);
        if (st) return st;
        A.out_limit = c->capturing ? c->out_rounds * A.lot : 0;
      }
    }
    W.order = (theta_group && c->walk_order_valid) ? P<int32_t>(c->walk_order) : nullptr;
    W.wait_ticks = c->wait_ticks;
    if (!c->counters_clean || !c->xq_clean) reset_list_counters(P<DevInfo>(c->info), c->stream);
    c->counters_clean = false;
    if (visit_cap > 0) split_reset(W.ctr, P<DevInfo>(c->info), W.tasks, c->task_cap, c->stream);
    st = timer_start(c, c->t_walk);
    if (st) return st;
    c->last_attempts = attempt + 1;
    walk_lists_device(W, grid, c->stream);
    c->xq_clean = false;
    if (outliers && few) {  // (the first of them)
      walk_outliers_device(A, c->stream);
      walk_tasks_device(A, c->num_cu, c->stream);
    }
    st = timer_stop(c, c->t_walk);
    if (st) return st;
    st = hip_check(c, hipGetLastError(), "kernel launch (walk)");
    if (st) return st;
    // the pools must have held every list before the sums may run; a captured
    // step cannot wait here: an overflow then leaves kErrPool for bh_sync
    if (c->capturing && !few) break;
    if (few) {
      // (queued behind the walk; they leave at once when a list did not fit)
      st = forces_tiles(c, W, A, outliers, attempt > 0 || walk_whole, acc, pot);
      if (!st && c->capturing && outliers) st = outlier_rounds(c, theta_group, acc, pot, 1, &have_out);
      if (st || c->capturing) return st;
      st = hip_check(c, hipEventSynchronize(c->info_event), "hipEventSynchronize");
      if (st) return st;
      c->last_segments = c->last_split_groups = c->last_depth = 0;
      if (outliers && wide_overrun(c)) return fail(c, BH_EINTERNAL, "more rows of list blocks than blocks");
      if (!(c->info_host->err & (kErrPool | kErrWide))) {
        if (!outliers) return BH_OK;
        bool whole;
        st = outlier_rounds(c, theta_group, acc, pot, 1, &whole);
        return whole ? forces_common(c, eps_sys, theta_sys, theta_group, acc, pot, true) : st;
      }
    } else {
      st = hip_check(c, hipMemcpyAsync(c->info_host, c->info.p, sizeof(DevInfo), hipMemcpyDeviceToHost, c->stream),
                     "hipMemcpyAsync info");
      if (st) return st;
    }
    if (visit_cap > 0) {
      st = hip_check(c, hipMemcpyAsync(c->split_host, W.ctr, sizeof(SplitCounters), hipMemcpyDeviceToHost,
                                       c->stream), "hipMemcpyAsync split counters");
      if (st) return st;
    }
    st = hip_check(c, hipStreamSynchronize(c->stream), "hipStreamSynchronize");
    if (st) return st;
    have_out = outliers && c->info_host->n_out > 0;
    if (visit_cap > 0) nsegs_host = c->split_host->segs;
    c->last_segments = nsegs_host;
    c->last_split_groups = visit_cap > 0 ? c->split_host->n_split : 0;
    c->last_depth = visit_cap > 0 ? c->split_host->depth : 0;
    if (!(c->info_host->err & (kErrPool | kErrWide))) break;
    if (attempt > 5) return fail(c, BH_EINTERNAL, "interaction list pool still too small after growing");
    if (c->info_host->err & kErrWide) {
      c->out_off = true;  // every group by one wave after all
      outliers = have_out = false;
      continue;
    }
    if (few && c->info_host->tile_need > 0) {  // (the lists fitted)
      const double room = (double)tile_rows_room(c), need = (double)c->info_host->tile_need;
      if (need > room) {
        c->tile_factor *= 1.25 * need / std::max(room, 1.0);
        continue;
      }
    }
    wide_grow(c);
    const int64_t fneed = (int64_t)c->info_host->far_chunks * kChunkRun, nneed = (int64_t)c->info_host->near_chunks * kChunkRun;
    c->far_cap = std::max(c->far_cap, (int32_t)std::min<int64_t>(fneed + fneed / 4 + 64, INT32_MAX / 2));
    c->near_cap = std::max(c->near_cap, (int32_t)std::min<int64_t>(nneed + nneed / 4 + 64, INT32_MAX / 2));
    if (visit_cap > 0) {
      const SplitCounters &h = *c->split_host;
      if (h.tasks > c->task_cap) c->task_cap = std::max(2 * c->task_cap, h.tasks + h.tasks / 4 + 64);
      if (h.ranges > c->range_cap) c->range_cap = std::max(2 * c->range_cap, h.ranges + h.ranges / 4 + 1024);
      if (h.segs > c->seg_cap) c->seg_cap = std::max(2 * c->seg_cap, h.segs + h.segs / 4 + 64);
    }
  }
  const bool split = visit_cap > 0 && (c->capturing || nsegs_host > 0);
  S.ctr = P<SplitCounters>(c->split_ctr);
  S.segs = P<Segment>(c->segs);
  S.seg_cap = c->seg_cap;
  S.keys[0] = P<uint64_t>(c->skeys[0]);
  S.keys[1] = P<uint64_t>(c->skeys[1]);
  S.vals[0] = P<uint32_t>(c->svals[0]);
  S.vals[1] = P<uint32_t>(c->svals[1]);
  S.hist = P<uint32_t>(c->shist);
  S.scan_tmp = c->sscan.p;
  S.order = S.vals[0];
  S.gsegfirst = P<int32_t>(c->gsegfirst);
  S.gnseg = P<int32_t>(c->gnseg);
  S.rows = P<int32_t>(c->srows);
  S.pbase = P<int32_t>(c->spbase);
  S.total_rows = S.pbase + c->seg_cap;
  S.sgroups = P<int32_t>(c->sgroups);
  S.nsg = S.total_rows + 1;
  if (visit_cap > 0) {  // sized even when nothing split, so that a capture never has to grow it
    st = ensure(c, c->psum, sizeof(double) * 4 * (size_t)c->seg_cap * (size_t)std::max(c->n_crit, 1), "partial sums");
    if (st) return st;
    S.psum = P<double>(c->psum);
  }
  if (split)
    split_finish_device(S, P<int32_t>(c->ginfo), P<int32_t>(c->glist), P<double>(c->gmass), P<DevInfo>(c->info),
                        c->stream);
  const size_t icap = gcap + gcap / 64 + 64 + (size_t)4 * c->seg_cap;  // items: blocks of 64, segments
  st = ensure(c, c->items, 2 * sizeof(int32_t) * icap, "force items");
  if (st) return st;
  ForceArgs F{};
  F.items = P<int32_t>(c->items);
  F.ginfo = P<int32_t>(c->ginfo);
  F.gbox = P<double>(c->gbox);
  F.glists = P<int32_t>(c->glists);
  F.far_pool = P<float4>(c->far_pool);
  F.near_pool = P<float4>(c->near_pool);
  F.far_next = P<int32_t>(c->far_next);
  F.near_next = P<int32_t>(c->near_next);
  F.far_slot = quad ? P<int32_t>(c->far_slot) : nullptr;
  F.qpack = quad ? P<float4>(c->qpack) : nullptr;
  F.far_tile = tile;
  F.near_tile = tile / 2;
  F.spos = P<double>(c->spos);
  F.smass = P<double>(c->smass);
  F.perm = P<int32_t>(c->perm);
  F.par = P<SysParam>(c->par);
  F.acc = acc;
  F.pot = pot;
  F.info = P<DevInfo>(c->info);
  F.xstart = P<int32_t>(c->order_hist) + (order_hist_bytes() / sizeof(int32_t) - 16);
  F.glist = P<int32_t>(c->glist);
  F.segs = S.segs;
  F.seg_order = S.order;
  F.gsegfirst = S.gsegfirst;
  F.pbase = S.pbase;
  F.psum = split ? P<double>(c->psum) : nullptr;
  item_order_device(F, P<int32_t>(c->gsplit), P<int32_t>(c->gnseg), (int64_t)gcap, P<int32_t>(c->order_hist),
                    P<int32_t>(c->items), c->stream);
  st = timer_start(c, c->t_force, walk_whole);
  if (st) return st;
  force_lists_device(F, fgrid, c->stream);
  st = timer_stop(c, c->t_force);
  if (st) return st;
  if (have_out) {
    bool whole;
    wide_capacity(c, kOutBlock, out_blocks(c, false));
    st = outlier_rounds(c, theta_group, acc, pot, 0, &whole);
    if (st) return st;
    if (whole) return forces_common(c, eps_sys, theta_sys, theta_group, acc, pot, true);
  }
  if (split)
    split_reduce_device(S, P<int32_t>(c->ginfo), P<double>(c->smass), P<int32_t>(c->perm), P<SysParam>(c->par), acc,
                        pot, c->stream);
  st = hip_check(c, hipGetLastError(), "kernel launch (force)");
  if (st) return st;
  c->have_forces = true;
  return BH_OK;
}

bh_status bh_compute_forces(bh_ctx *c, double eps, double theta, const float *theta_group, float *acc, float *pot) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!c->have_tree) return fail(c, BH_ESTATE, "forces requested before a tree was built");
  std::vector<double> e((size_t)c->nsys, eps), t((size_t)c->nsys, theta);
  return forces_common(c, e.data(), t.data(), theta_group, acc, pot);
}

bh_status bh_compute_forces_batch(bh_ctx *c, const double *eps_sys, const double *theta_sys,
                                  const float *theta_group, float *acc, float *pot) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!c->have_tree) return fail(c, BH_ESTATE, "forces requested before a tree was built");
  if (!eps_sys || !theta_sys) return fail(c, BH_EINVAL, "eps_sys and theta_sys must not be NULL");
  return forces_common(c, eps_sys, theta_sys, theta_group, acc, pot);
}

// The per-particle walk (no groups needed): parameters as for the group path.
static bh_status particle_common(bh_ctx *c, const double *eps_sys, const double *theta_sys, float *acc,
                                 float *pot) {
  if (!c->have_tree) return fail(c, BH_ESTATE, "forces requested before a tree was built");
  if (c->n > 0 && (!acc || !pot)) return fail(c, BH_EINVAL, "acc and pot must not be NULL");
  if (c->opt.quadrupole) return fail(c, BH_EINVAL, "the per-particle walk sums monopoles only (quadrupole option set)");
  c->par_host.assign((size_t)c->nsys, SysParam{});
  for (int s = 0; s < c->nsys; ++s) {
    const double e = eps_sys[s], t = theta_sys[s];
    if (!(e > 0.0) || !isfinite(e)) return fail(c, BH_EINVAL, "eps must be positive and finite");
    const float e2 = (float)(e * e);
    if (!(e2 >= 1.17549435e-38f) || isinf(e2)) return fail(c, BH_EINVAL, "eps^2 must be a normal FP32 number");
    if (!(t >= 0.0 && t <= 1.0)) return fail(c, BH_EINVAL, "theta must be in [0, 1]");
    c->par_host[s].eps = e;
    c->par_host[s].theta = t;
  }
  bh_status st = ensure(c, c->par, sizeof(SysParam) * (size_t)c->nsys, "parameters");
  if (st) return st;
  st = upload(c, c->par.p, c->par_host.data(), sizeof(SysParam) * (size_t)c->nsys);
  if (st) return st;
  st = ensure(c, c->pp_stat, particle_stat_bytes(c->n, c->nsys), "list statistics");
  if (st) return st;
  reset_list_counters(P<DevInfo>(c->info), c->stream);
  c->counters_clean = false;
  st = timer_start(c, c->t_particle);
  if (st) return st;
  particle_forces_device(P<NodeRec>(c->nodes), c->nsys, P<SysInfo>(c->sys), P<SysParam>(c->par), P<double>(c->spos),
                         P<int32_t>(c->perm), c->n, acc, pot, P<int4>(c->pp_stat), P<DevInfo>(c->info), c->stream);
  st = timer_stop(c, c->t_particle);
  if (st) return st;
  st = hip_check(c, hipGetLastError(), "kernel launch (per-particle walk)");
  if (st) return st;
  c->have_forces = true;
  c->last_split_groups = c->last_segments = c->last_depth = 0;
  c->last_attempts = 1;
  return BH_OK;
}

bh_status bh_compute_forces_particle(bh_ctx *c, double eps, double theta, float *acc, float *pot) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!c->have_tree) return fail(c, BH_ESTATE, "forces requested before a tree was built");
  std::vector<double> e((size_t)c->nsys, eps), t((size_t)c->nsys, theta);
  return particle_common(c, e.data(), t.data(), acc, pot);
}

bh_status bh_compute_forces_particle_batch(bh_ctx *c, const double *eps_sys, const double *theta_sys, float *acc,
                                           float *pot) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!eps_sys || !theta_sys) return fail(c, BH_EINVAL, "eps_sys and theta_sys must not be NULL");
  return particle_common(c, eps_sys, theta_sys, acc, pot);
}

static bh_status theta_common(bh_ctx *c, const bh_mlp *net, const double *eps_sys, float shift, float *theta);

// One whole step (build, groups, [per-group theta from the network], walk
// and force sum); the learned variant writes theta_out and walks with it.
static bh_status step_common(bh_ctx *c, int32_t n_systems, const int64_t *offsets, const double *pos,
                             const double *mass, int32_t n_crit, const double *eps_sys, const double *theta_sys,
                             const float *theta_group, const bh_mlp *net, float shift, float *theta_out, float *acc,
                             float *pot) {
  bh_status st = build_common(c, n_systems, offsets, pos, mass);
  if (!st) st = bh_make_groups(c, n_crit, nullptr);
  if (!st && net) st = theta_common(c, net, eps_sys, shift, theta_out);
  if (!st) st = forces_common(c, eps_sys, theta_sys, net ? theta_out : theta_group, acc, pot);
  return st;
}

static bh_status capture_step(bh_ctx *c, int32_t n_systems, const int64_t *offsets, const double *pos,
                              const double *mass, int32_t n_crit, const double *eps_sys, const double *theta_sys,
                              const float *theta_group, const bh_mlp *net, float shift, float *theta_out, float *acc,
                              float *pot) {
  if (n_systems < 1 || n_systems > 65536 || !offsets || !eps_sys || !theta_sys)
    return fail(c, BH_EINVAL, "bad graph capture arguments");
  if (offsets[0] != 0) return fail(c, BH_EINVAL, "offsets[0] must be 0");
  for (int s = 0; s < n_systems; ++s)
    if (offsets[s + 1] < offsets[s]) return fail(c, BH_EINVAL, "offsets must be non-decreasing");
  if (n_crit < 1 || n_crit > BH_MAX_NCRIT) return fail(c, BH_EINVAL, "n_crit must be in [1, 256]");
  if (net && !theta_out) return fail(c, BH_EINVAL, "theta_group must not be NULL");
  // 1. one eager step sizes every buffer and checks the arguments
  bh_status st = step_common(c, n_systems, offsets, pos, mass, n_crit, eps_sys, theta_sys, theta_group, net, shift,
                             theta_out, acc, pot);
  if (!st) st = bh_sync(c);
  if (st) return st;
  // 2. headroom in the list pools for replays on moved particles
  c->far_cap += c->far_cap / 4;
  c->near_cap += c->near_cap / 4;
  c->wide_cap += c->wide_cap / 4;
  st = forces_common(c, eps_sys, theta_sys, net ? theta_out : theta_group, acc, pot);
  if (!st) st = bh_sync(c);
  if (st) return st;
  // 3. record the same launches on a capture stream
  if (!c->capture_stream) {
    st = hip_check(c, hipStreamCreateWithFlags(&c->capture_stream, hipStreamNonBlocking), "hipStreamCreate");
    if (st) return st;
  }
  if (c->graph) {
    (void)hipGraphExecDestroy(c->graph);
    c->graph = nullptr;
  }
  hipStream_t saved = c->stream;
  c->stream = c->capture_stream;
  c->capturing = true;
  st = hip_check(c, hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
  if (!st) {
    bh_status sr = step_common(c, n_systems, offsets, pos, mass, n_crit, eps_sys, theta_sys, theta_group, net, shift,
                               theta_out, acc, pot);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(c->stream, &g);
    c->capturing = false;
    c->stream = saved;
    c->counters_clean = c->xq_clean = false;  // (what was recorded has not run)
    if (sr) {
      if (g) (void)hipGraphDestroy(g);
      return sr;
    }
    st = hip_check(c, e, "hipStreamEndCapture");
    if (!st) st = hip_check(c, hipGraphInstantiate(&c->graph, g, nullptr, nullptr, 0), "hipGraphInstantiate");
    if (g) (void)hipGraphDestroy(g);
    if (st) {
      c->graph = nullptr;
      return st;
    }
    Captured &k = c->captured;
    k.n = c->n;
    k.nsys = c->nsys;
    k.largest = c->largest;
    k.n_crit = c->n_crit;
    k.quad = c->have_quad;
    k.learned = net != nullptr;
    k.sorted_keys = c->sorted_keys;
    k.sys = c->sys_host;
    k.par = c->par_host;
    k.feps.clear();
    if (net) k.feps = c->feps_host;
    k.split_groups = c->last_split_groups;
    k.segments = c->last_segments;
    k.depth = c->last_depth;
    k.attempts = c->last_attempts;
    c->data_moved = false;
    return BH_OK;
  }
  c->capturing = false;
  c->stream = saved;
  return st;
}

static bh_status capture_common(bh_ctx *c, int32_t n_systems, const int64_t *offsets, const double *pos,
                                const double *mass, int32_t n_crit, const double *eps_sys, const double *theta_sys,
                                const float *theta_group, const bh_mlp *net, float shift, float *theta_out,
                                float *acc, float *pot) {
  c->reserve = true;
  const bh_status st = capture_step(c, n_systems, offsets, pos, mass, n_crit, eps_sys, theta_sys, theta_group, net,
                                    shift, theta_out, acc, pot);
  c->reserve = false;
  return st;
}

bh_status bh_graph_capture(bh_ctx *c, int32_t n_systems, const int64_t *offsets, const double *pos,
                           const double *mass, int32_t n_crit, const double *eps_sys, const double *theta_sys,
                           const float *theta_group, float *acc, float *pot) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  return capture_common(c, n_systems, offsets, pos, mass, n_crit, eps_sys, theta_sys, theta_group, nullptr, 0.0f,
                        nullptr, acc, pot);
}

bh_status bh_graph_capture_learned(bh_ctx *c, int32_t n_systems, const int64_t *offsets, const double *pos,
                                   const double *mass, int32_t n_crit, const double *eps_sys,
                                   const double *theta_sys, const bh_mlp *net, float shift, float *theta_group,
                                   float *acc, float *pot) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!net) return fail(c, BH_EINVAL, "net must not be NULL");
  return capture_common(c, n_systems, offsets, pos, mass, n_crit, eps_sys, theta_sys, nullptr, net, shift,
                        theta_group, acc, pot);
}

bh_status bh_graph_launch(bh_ctx *c) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!c->graph) return fail(c, BH_ESTATE, "no captured step");
  // the step's systems and parameters, where other calls have brought theirs
  // (the buffers are those of the capture: growing one would have ended it)
  const Captured &k = c->captured;
  if (c->data_moved) {
    bh_status st = upload(c, c->sys.p, k.sys.data(), sizeof(SysInfo) * k.sys.size());
    if (!st) st = upload(c, c->par.p, k.par.data(), sizeof(SysParam) * k.par.size());
    if (!st) st = upload(c, c->feps.p, k.feps.data(), sizeof(double) * k.feps.size());
    if (st) return st;
    c->data_moved = false;
  }
  c->counters_clean = c->xq_clean = false;  // the replay uses the queues up
  bh_status st = hip_check(c, hipGraphLaunch(c->graph, c->stream), "hipGraphLaunch");
  if (st) return st;
  c->n = k.n;
  c->nsys = k.nsys;
  c->largest = k.largest;
  c->n_crit = k.n_crit;
  c->have_tree = c->have_groups = c->have_forces = true;
  c->have_quad = k.quad;
  c->have_neighbors = false;
  c->walk_order_valid = k.learned;
  c->sorted_keys = k.sorted_keys;
  c->last_split_groups = k.split_groups;
  c->last_segments = k.segments;
  c->last_depth = k.depth;
  c->last_attempts = k.attempts;
  return BH_OK;
}

bh_status bh_get_stats(bh_ctx *c, bh_stats *out) {
  if (!c || !out) return BH_EINVAL;
  c->err.clear();
  bh_status st = check_device_errors(c);
  memset(out, 0, sizeof(*out));
  const DevInfo &d = *c->info_host;
  out->n = c->n;
  out->n_systems = c->nsys;
  out->n_crit = c->have_groups ? c->n_crit : 0;
  out->error_flags = d.err;
  if (c->have_tree) {
    out->n_cells = d.n_cells;
    out->n_slots = (int64_t)c->nsys + d.n_slots;
    out->max_level = d.max_level;
  }
  if (c->have_groups) out->n_groups = d.n_groups;
  if (c->have_forces) {
    out->interactions = (int64_t)d.interactions;
    out->list_entries = (int64_t)d.list_entries;
    out->max_list = d.max_list;
    const int32_t outs = std::min(d.n_out, kOutPlaces);
    out->n_split_groups = c->last_split_groups + outs;
    out->n_segments = c->last_segments + outs + d.tasks_done + d.tasks;
    out->n_split_levels = outs ? 1 : c->last_depth;
    out->n_walk_attempts = c->last_attempts;
    out->n_theta_fallback = d.theta_fallback;
    out->node_visits = (int64_t)d.node_visits;
    out->near_entries = (int64_t)d.near_entries;
  }
  out->t_build_ms = timer_take(c->t_build, &out->n_build_calls);
  out->t_groups_ms = timer_take(c->t_groups, &out->n_groups_calls);
  out->t_walk_ms = timer_take(c->t_walk, &out->n_walk_calls);
  out->t_force_ms = timer_take(c->t_force, &out->n_force_calls);
  out->t_particle_ms = timer_take(c->t_particle, &out->n_particle_calls);
  out->t_neighbor_ms = timer_take(c->t_neighbor, &out->n_neighbor_calls);
  out->t_theta_ms = timer_take(c->t_theta, &out->n_theta_calls);
  if (c->have_neighbors) {
    out->neighbor_pairs = (int64_t)d.nb_pairs;
    out->neighbor_tests = (int64_t)d.nb_tests;
  }
  return st;
}

bh_status bh_direct_sampled(bh_ctx *c, int64_t n, const double *pos, const double *mass, double eps, int64_t s,
                            const int64_t *idx, double *acc, double *pot) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (n < 0 || s < 0) return fail(c, BH_EINVAL, "negative size");
  if (s > 0 && (!pos || !mass || !idx || !acc || !pot)) return fail(c, BH_EINVAL, "NULL pointer");
  if (!(eps >= 0.0) || !isfinite(eps)) return fail(c, BH_EINVAL, "eps must be finite and >= 0");
  if (s == 0) return BH_OK;
  int64_t chunk, nchunk;
  size_t bytes = direct_part_bytes(n, s, c->num_cu, &chunk, &nchunk);
  bh_status st = ensure(c, c->direct_part, bytes, "direct partials");
  if (st) return st;
  direct_sampled_device(pos, mass, n, eps, s, idx, acc, pot, P<double>(c->direct_part), chunk, nchunk, c->stream);
  return hip_check(c, hipGetLastError(), "kernel launch (direct)");
}

bh_status bh_direct_sampled_noalloc(bh_ctx *c, int64_t n, const double *pos, const double *mass, double eps,
                                    int64_t s, const int64_t *idx, double *acc, double *pot) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (n < 0 || s < 0) return fail(c, BH_EINVAL, "negative size");
  if (s > 0 && (!pos || !mass || !idx || !acc || !pot)) return fail(c, BH_EINVAL, "NULL pointer");
  if (!(eps >= 0.0) || !isfinite(eps)) return fail(c, BH_EINVAL, "eps must be finite and >= 0");
  if (s == 0) return BH_OK;
  int64_t chunk, nchunk;
  const size_t bytes = direct_part_bytes(n, s, c->num_cu, &chunk, &nchunk);
  if (bytes > kJudgeScratchBytes)
    return fail(c, BH_EINVAL, "sample too large for the no-allocation judge: its partial sums need " +
                                  std::to_string(bytes) + " bytes, the static scratch holds " +
                                  std::to_string(kJudgeScratchBytes));
  // every partial-sum row the reduction reads is written by the first kernel:
  // the scratch needs no clearing
  direct_sampled_device(pos, mass, n, eps, s, idx, acc, pot, c->judge_scratch, chunk, nchunk, c->stream);
  return hip_check(c, hipGetLastError(), "kernel launch (direct, no allocation)");
}

bh_status bh_kick(bh_ctx *c, int64_t n, double *vel, const float *acc, double dt) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (n < 0 || (n > 0 && (!vel || !acc))) return fail(c, BH_EINVAL, "bad kick arguments");
  c->integrates = c->integrates || n > 0;
  kick_device(n, vel, acc, dt, c->stream);
  return hip_check(c, hipGetLastError(), "kernel launch (kick)");
}

bh_status bh_drift(bh_ctx *c, int64_t n, double *pos, const double *vel, double dt) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (n < 0 || (n > 0 && (!pos || !vel))) return fail(c, BH_EINVAL, "bad drift arguments");
  c->integrates = c->integrates || n > 0;
  drift_device(n, pos, vel, dt, c->stream);
  return hip_check(c, hipGetLastError(), "kernel launch (drift)");
}

bh_status bh_leapfrog(bh_ctx *c, int64_t n, double *pos, double *vel, const double *mass, double eps, double theta,
                      int32_t n_crit, double dt, int32_t steps, float *acc, float *pot) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (n < 0 || n > BH_MAX_N) return fail(c, BH_EINVAL, "n out of range");
  if (steps < 0) return fail(c, BH_EINVAL, "steps must be >= 0");
  if (!isfinite(dt)) return fail(c, BH_EINVAL, "dt must be finite");
  if (n > 0 && (!pos || !vel || !mass || !acc || !pot)) return fail(c, BH_EINVAL, "bad leapfrog arguments");
  if (n_crit < 1 || n_crit > BH_MAX_NCRIT) return fail(c, BH_EINVAL, "n_crit must be in [1, 256]");
  const double h = 0.5 * dt;
  for (int32_t k = 0; k < steps; ++k) {
    bh_status st = bh_kick(c, n, vel, acc, h);
    if (!st) st = bh_drift(c, n, pos, vel, dt);
    if (!st) st = bh_build_tree(c, n, pos, mass);
    if (!st) st = bh_make_groups(c, n_crit, nullptr);
    if (!st) st = bh_compute_forces(c, eps, theta, nullptr, acc, pot);
    if (!st) st = bh_kick(c, n, vel, acc, h);
    if (st) return st;
  }
  return BH_OK;
}

bh_status bh_energy(bh_ctx *c, int64_t n, const double *vel, const double *mass, const float *pot,
                    double *energy) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (n < 0 || !energy || (n > 0 && (!vel || !mass || !pot))) return fail(c, BH_EINVAL, "bad energy arguments");
  bh_status st = ensure(c, c->energy_part, energy_part_bytes(), "energy partials");
  if (st) return st;
  energy_device(n, vel, mass, pot, P<double>(c->energy_part), energy, c->stream);
  return hip_check(c, hipGetLastError(), "kernel launch (energy)");
}

static bh_status check_net(bh_ctx *c, const bh_mlp *net) {
  if (!net || !net->params || !net->mu || !net->sigma) return fail(c, BH_EINVAL, "network pointers must not be NULL");
  return BH_OK;
}

static bh_status features_common(bh_ctx *c, const double *eps_sys, float *feat) {
  if (!c->have_groups) return fail(c, BH_ESTATE, "features requested before bh_make_groups");
  if (!eps_sys) return fail(c, BH_EINVAL, "eps_sys must not be NULL");
  if (c->n > 0 && !feat) return fail(c, BH_EINVAL, "feat must not be NULL");
  c->feps_host.assign((size_t)c->nsys, 0.0);
  for (int s = 0; s < c->nsys; ++s) {
    if (!(eps_sys[s] > 0.0) || !isfinite(eps_sys[s])) return fail(c, BH_EINVAL, "eps must be positive and finite");
    c->feps_host[s] = eps_sys[s];
  }
  bh_status st = ensure(c, c->feps, sizeof(double) * (size_t)c->nsys, "feature softening");
  if (st) return st;
  st = upload(c, c->feps.p, c->feps_host.data(), sizeof(double) * (size_t)c->nsys);
  if (st) return st;
  if (c->n == 0) return BH_OK;
  ProbeArgs pa{};
  pa.nodes = P<NodeRec>(c->nodes);
  pa.ginfo = P<int32_t>(c->ginfo);
  pa.gbox = P<double>(c->gbox);
  pa.spos = P<double>(c->spos);
  pa.smass = P<double>(c->smass);
  pa.pparent = P<int32_t>(c->pparent);
  pa.cparent = P<int32_t>(c->cparent);
  pa.ccount = P<int32_t>(c->ccount);
  pa.cslot = P<int32_t>(c->cslot);
  pa.level = P<int8_t>(c->level);
  pa.eps = P<double>(c->feps);
  pa.info = P<DevInfo>(c->info);
  pa.nsys = c->nsys;
  pa.feat = feat;
  if (c->probe_bpc == 0) c->probe_bpc = probe_blocks_per_cu();
  probe_device(pa, c->num_cu * c->probe_bpc, !c->xq_clean, c->stream);
  c->xq_clean = false;
  return hip_check(c, hipGetLastError(), "kernel launch (features)");
}

bh_status bh_group_features(bh_ctx *c, const double *eps_sys, float *feat) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  return features_common(c, eps_sys, feat);
}

bh_status bh_mlp_infer(bh_ctx *c, const bh_mlp *net, int64_t rows, const float *feat, float shift, float *theta) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  bh_status st = check_net(c, net);
  if (st) return st;
  if (rows < 0 || rows > BH_MAX_N) return fail(c, BH_EINVAL, "rows out of range");
  if (!isfinite(shift)) return fail(c, BH_EINVAL, "shift must be finite");
  if (rows == 0) return BH_OK;
  if (!feat || !theta) return fail(c, BH_EINVAL, "feat and theta must not be NULL");
  mlp_infer_device(net->params, net->mu, net->sigma, feat, rows, rows, P<DevInfo>(c->info), shift, theta, c->stream);
  return hip_check(c, hipGetLastError(), "kernel launch (inference)");
}

static bh_status theta_common(bh_ctx *c, const bh_mlp *net, const double *eps_sys, float shift, float *theta) {
  bh_status st = check_net(c, net);
  if (st) return st;
  if (!isfinite(shift)) return fail(c, BH_EINVAL, "shift must be finite");
  if (c->n > 0 && !theta) return fail(c, BH_EINVAL, "theta must not be NULL");
  const int64_t cap = std::max<int64_t>(c->n, 1);
  st = ensure(c, c->mlp_feat, sizeof(float) * BH_MLP_FEATURES * (size_t)cap, "features");
  if (st) return st;
  st = timer_start(c, c->t_theta);
  if (st) return st;
  st = features_common(c, eps_sys, P<float>(c->mlp_feat));
  if (st || c->n == 0) return st;
  // rows = -1: the kernel reads the group count on the device
  mlp_infer_device(net->params, net->mu, net->sigma, P<float>(c->mlp_feat), -1, cap, P<DevInfo>(c->info), shift,
                   theta, c->stream);
  // the list walk's order for these groups, from their features and theta
  st = ensure(c, c->walk_order, sizeof(int32_t) * (size_t)cap, "walk order");
  if (st) return st;
  if (!c->walk_order_hist.p) {
    st = ensure(c, c->walk_order_hist, order_hist_bytes(), "walk order bins");
    if (st) return st;
    order_clear_device(P<int32_t>(c->walk_order_hist), c->stream);  // every later call leaves it zero
  }
  walk_order_device(P<float>(c->mlp_feat), theta, P<DevInfo>(c->info), cap, P<int32_t>(c->walk_order_hist),
                    P<int32_t>(c->walk_order), c->stream);
  c->walk_order_valid = true;
  st = timer_stop(c, c->t_theta);
  if (st) return st;
  return hip_check(c, hipGetLastError(), "kernel launch (inference)");
}

bh_status bh_group_theta(bh_ctx *c, const bh_mlp *net, const double *eps_sys, float shift, float *theta) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  return theta_common(c, net, eps_sys, shift, theta);
}

bh_status bh_mlp_grad(bh_ctx *c, const bh_mlp *net, int32_t batch, const float *x, const float *target,
                      const float *weight, float *grad, float *loss) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  bh_status st = check_net(c, net);
  if (st) return st;
  if (batch < 1 || batch > 65536) return fail(c, BH_EINVAL, "batch must be in [1, 65536]");
  if (!x || !target || !weight || !grad) return fail(c, BH_EINVAL, "x, target, weight and grad must not be NULL");
  st = ensure(c, c->mlp_work, mlp_part_bytes(batch), "training workspace");
  if (st) return st;
  mlp_grad_device(net->params, net->mu, net->sigma, batch, x, target, weight, P<float>(c->mlp_work), grad, loss,
                  c->stream);
  return hip_check(c, hipGetLastError(), "kernel launch (training)");
}

bh_status bh_mlp_adam(bh_ctx *c, float *params, const float *grad, float *m, float *v, int32_t n, int32_t step,
                      float lr, float beta1, float beta2, float eps) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (n < 1 || step < 1 || !params || !grad || !m || !v) return fail(c, BH_EINVAL, "bad Adam arguments");
  if (!(lr >= 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps > 0.0f))
    return fail(c, BH_EINVAL, "bad Adam hyper-parameters");
  adam_device(params, grad, m, v, n, lr, beta1, beta2, eps, step, c->stream);
  return hip_check(c, hipGetLastError(), "kernel launch (Adam)");
}

bh_status bh_export_sorted(bh_ctx *c, uint64_t *keys, int32_t *perm) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!c->have_tree) return fail(c, BH_ESTATE, "no tree");
  if (c->n == 0) return BH_OK;
  if (keys) k_copy_keys<<<blocks_for(c->n), 256, 0, c->stream>>>(c->sorted_keys, keys, c->n);
  if (perm) k_copy_i32<<<blocks_for(c->n), 256, 0, c->stream>>>(P<int32_t>(c->perm), perm, c->n);
  return hip_check(c, hipGetLastError(), "kernel launch (export sorted)");
}

bh_status bh_export_nodes(bh_ctx *c, int32_t *ints, double *reals) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!c->have_tree) return fail(c, BH_ESTATE, "no tree");
  const int64_t cap = 2 * std::max<int64_t>(c->n, 1) + c->nsys + 1;
  k_export_nodes<<<blocks_for(cap), 256, 0, c->stream>>>(P<NodeRec>(c->nodes), P<int8_t>(c->meta),
                                                          P<DevInfo>(c->info), c->nsys, ints, reals);
  return hip_check(c, hipGetLastError(), "kernel launch (export nodes)");
}

bh_status bh_neighbors(bh_ctx *c, const double *h, int32_t *count, double *rho, const int64_t *offsets,
                       int32_t *nbr) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!c->have_tree) return fail(c, BH_ESTATE, "neighbour search requested before a tree was built");
  if (!c->have_groups) return fail(c, BH_ESTATE, "neighbour search requested before bh_make_groups");
  if (c->n > 0 && !h) return fail(c, BH_EINVAL, "h must not be NULL");
  if (c->n == 0) {  // nothing to search (empty outputs may come as NULL)
    c->have_neighbors = true;
    return BH_OK;
  }
  if ((offsets == nullptr) != (nbr == nullptr)) return fail(c, BH_EINVAL, "offsets and nbr go together");
  if (!count && !rho && !nbr) return fail(c, BH_EINVAL, "no output requested");
  c->have_neighbors = true;
  const int variant = (c->n_crit <= 64 ? 0 : (c->n_crit <= 128 ? 1 : 2)) + (nbr ? 3 : 0) + (rho ? 6 : 0);
  if (!c->nb_bpc[variant]) c->nb_bpc[variant] = neighbors_blocks_per_cu(c->n_crit, nbr != nullptr, rho != nullptr);
  const int grid = c->num_cu * (c->opt.waves_per_cu > 0 ? c->opt.waves_per_cu : c->nb_bpc[variant]);
  NeighborArgs A{};
  A.nodes = P<NodeRec>(c->nodes);
  A.ginfo = P<int32_t>(c->ginfo);
  A.gbox = P<double>(c->gbox);
  A.spos = P<double>(c->spos);
  A.smass = P<double>(c->smass);
  A.perm = P<int32_t>(c->perm);
  A.info = P<DevInfo>(c->info);
  A.n = c->n;
  A.nsys = c->nsys;
  A.n_crit = c->n_crit;
  A.sys = P<SysInfo>(c->sys);
  A.out_min = nbr ? INT32_MAX : neighbors_out_min(c->n);
  if (A.out_min != INT32_MAX) {
    const size_t parts = neighbors_parts(c->n_crit);
    bh_status st = ensure(c, c->nb_out, sizeof(int32_t) * (size_t)c->n, "outlier groups");
    if (!st) st = ensure(c, c->nb_count, sizeof(int32_t) * parts, "partial counts");
    if (!st) st = ensure(c, c->nb_rho, sizeof(double) * parts, "partial densities");
    if (st) return st;
    A.out = P<int32_t>(c->nb_out);
    A.part_count = P<int32_t>(c->nb_count);
    A.part_rho = P<double>(c->nb_rho);
  }
  A.h = h;
  A.count = count;
  A.rho = rho;
  A.offsets = offsets;
  A.nbr = nbr;
  bh_status st = timer_start(c, c->t_neighbor);
  if (st) return st;
  c->counters_clean = false;  // (the search shares the group queue)
  neighbors_device(A, grid, c->stream);
  st = timer_stop(c, c->t_neighbor);
  if (st) return st;
  return hip_check(c, hipGetLastError(), "kernel launch (neighbours)");
}

bh_status bh_export_moments(bh_ctx *c, double *moments) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!c->have_tree) return fail(c, BH_ESTATE, "no tree");
  if (!c->have_quad) return fail(c, BH_ESTATE, "the tree was built without the quadrupole option");
  if (!moments) return fail(c, BH_EINVAL, "moments must not be NULL");
  const int64_t cap = 2 * std::max<int64_t>(c->n, 1) + c->nsys + 1;
  k_export_moments<<<blocks_for(cap), 256, 0, c->stream>>>(P<NodeRec>(c->nodes), P<double>(c->qmom),
                                                            P<DevInfo>(c->info), c->nsys, moments);
  return hip_check(c, hipGetLastError(), "kernel launch (export moments)");
}

bh_status bh_export_groups(bh_ctx *c, int32_t *ints, double *box, int32_t *list_len, double *list_mass) {
  if (!c) return BH_EINVAL;
  c->err.clear();
  if (!c->have_groups) return fail(c, BH_ESTATE, "no groups");
  if ((list_len || list_mass) && !c->have_forces) return fail(c, BH_ESTATE, "no force call since the grouping");
  const int64_t cap = std::max<int64_t>(c->n, 1);
  k_export_groups<<<blocks_for(cap), 256, 0, c->stream>>>(P<int32_t>(c->ginfo), P<double>(c->gbox),
                                                           P<int32_t>(c->glist), P<double>(c->gmass),
                                                           P<DevInfo>(c->info), ints, box, list_len, list_mass);
  return hip_check(c, hipGetLastError(), "kernel launch (export groups)");
}

}  // extern "C"
