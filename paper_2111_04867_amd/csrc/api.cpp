// C ABI: plan upload and batched evaluation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "kernels.h"
#include "plan.h"

namespace taccl {
namespace {

struct Packer {
  std::vector<unsigned char> bytes;
  template <class T>
  size_t add(const std::vector<T> &v) {
    size_t off = (bytes.size() + 255) & ~size_t(255);
    bytes.resize(off + std::max<size_t>(v.size() * sizeof(T), 1), 0);
    if (!v.empty()) std::memcpy(bytes.data() + off, v.data(), v.size() * sizeof(T));
    return off;
  }
};

taccl_status_t hip_fail(hipError_t e, const char *what) {
  return fail(TACCL_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

// Upload the read-only tables of `p` to the current device (once).
taccl_status_t ensure_device(taccl_plan *p, DeviceTables **out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> lock(p->mu);
  auto it = p->dev.find(dev);
  if (it != p->dev.end()) {
    *out = &it->second;
    return TACCL_OK;
  }
  hipDeviceProp_t prop;
  e = hipGetDeviceProperties(&prop, dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDeviceProperties");
  Packer pk;
  size_t o_cost = pk.add(p->cost), o_lsrc = pk.add(p->lsrc), o_ldst = pk.add(p->ldst),
         o_pb = pk.add(p->pair_base), o_np = pk.add(p->npaths), o_po = pk.add(p->path_off),
         o_pl = pk.add(p->path_links), o_own = pk.add(p->coll.owner),
         o_pm = pk.add(p->post_mask), o_hc = pk.add(p->hop_class),
         o_plh = pk.add(p->path_lvl_hop), o_lcb = pk.add(p->lvl_cls_begin),
         o_llc = pk.add(p->llc), o_trec = pk.add(p->tree_rec), o_own8 = pk.add(p->owner8),
         o_arec = pk.add(p->arec), o_cpath = pk.add(p->cpath), o_cinfo = pk.add(p->cinfo),
         o_cbkt = pk.add(p->cbkt), o_topt = pk.add(p->topt), o_trec4 = pk.add(p->tree_rec4),
         o_lal = pk.add(p->lalpha), o_lbs = pk.add(p->lbs), o_lmg = pk.add(p->lmerge),
         o_lrev = pk.add(p->lrev), o_hc2 = pk.add(p->hop_class2),
         o_lcb2 = pk.add(p->lvl_cls2_begin), o_llc2 = pk.add(p->llc2),
         o_gkr = pk.add(p->gkrank), o_rimg = pk.add(p->rank_img), o_tent = pk.add(p->tent), o_c2l = pk.add(p->cls2_link),
         o_cnr = pk.add(p->cn_rec), o_cnc = pk.add(p->cn_chunk),
         o_plfb = pk.add(p->ports_lfb), o_pwalk = pk.add(p->pwalk), o_pport = pk.add(p->pport),
         o_cml = pk.add(p->cml), o_cwalk = pk.add(p->cwalk);
  void *blk = nullptr;
  e = hipMalloc(&blk, pk.bytes.size());
  if (e != hipSuccess) return fail(TACCL_ERR_NO_MEMORY, "hipMalloc of plan tables failed");
  e = hipMemcpy(blk, pk.bytes.data(), pk.bytes.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(blk);
    return hip_fail(e, "hipMemcpy of plan tables");
  }
  DeviceTables t;
  auto at = [&](size_t off) { return (const unsigned char *)blk + off; };
  t.block = blk;
  t.cost = (const uint32_t *)at(o_cost);
  t.lsrc = (const uint16_t *)at(o_lsrc);
  t.ldst = (const uint16_t *)at(o_ldst);
  t.pair_base = (const uint32_t *)at(o_pb);
  t.npaths = (const uint8_t *)at(o_np);
  t.path_off = (const uint32_t *)at(o_po);
  t.path_links = (const uint16_t *)at(o_pl);
  t.owner = (const int32_t *)at(o_own);
  t.post_mask = (const uint64_t *)at(o_pm);
  t.hop_class = (const uint16_t *)at(o_hc);
  t.path_lvl_hop = (const int8_t *)at(o_plh);
  t.lvl_cls_begin = (const uint32_t *)at(o_lcb);
  t.llc = (const uint32_t *)at(o_llc);
  t.tree_rec = (const uint32_t *)at(o_trec);
  t.owner8 = (const uint8_t *)at(o_own8);
  t.topt = p->topt.empty() ? nullptr : (const uint8_t *)at(o_topt);
  t.tree_rec4 = p->tree_rec4.empty() ? nullptr : (const uint32_t *)at(o_trec4);
  t.lalpha = (const uint32_t *)at(o_lal);
  t.lbs = (const uint64_t *)at(o_lbs);
  t.lmerge = (const uint8_t *)at(o_lmg);
  t.lrev = (const uint16_t *)at(o_lrev);
  t.hop_class2 = (const uint16_t *)at(o_hc2);
  t.lvl_cls2_begin = (const uint32_t *)at(o_lcb2);
  t.llc2 = (const uint32_t *)at(o_llc2);
  t.cls2_link = (const uint16_t *)at(o_c2l);
  t.arec = (const uint32_t *)at(o_arec);
  t.cpath = (const uint32_t *)at(o_cpath);
  t.cinfo = (const uint32_t *)at(o_cinfo);
  t.cbkt = (const uint32_t *)at(o_cbkt);
  t.gkrank = (const uint32_t *)at(o_gkr);
  t.tent = (const uint8_t *)at(o_tent);
  t.rank_img = p->rank_img.empty() ? nullptr : at(o_rimg);
  t.ports_lfb = (const uint32_t *)at(o_plfb);
  t.pwalk = (const uint32_t *)at(o_pwalk);
  t.pport = (const uint16_t *)at(o_pport);
  t.cml = (const uint32_t *)at(o_cml);
  t.cwalk = (const uint32_t *)at(o_cwalk);
  t.cn_rec = p->cn_rec.empty() ? nullptr : (const uint32_t *)at(o_cnr);
  t.cn_chunk = (const uint32_t *)at(o_cnc);
  t.max_lds = (int)prop.sharedMemPerBlock;
  t.lds_per_cu = (int)std::max<size_t>(prop.maxSharedMemoryPerMultiProcessor, prop.sharedMemPerBlock);
  t.num_cus = prop.multiProcessorCount;
  *out = &(p->dev[dev] = t);
  return TACCL_OK;
}

// Resident blocks of `threads` threads per CU by registers, `otherwise` if the
// query fails
int blocks_by_registers(const void *fn, int threads, int otherwise) {
  int nb = 0;
  if (!fn || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, threads, 0) != hipSuccess ||
      nb < 1)
    return otherwise;
  return nb;
}

// The launch shape of a kernel whose blocks hold wavefronts of `wave` bytes
// of LDS beside `shared` bytes, up to max_waves of them.
LaunchShape wave_shape(taccl_plan *p, DeviceTables *t, Kernel kernel, bool reduce, const void *fn,
                       int shared, int wave, int max_waves) {
  std::lock_guard<std::mutex> lock(p->mu);
  LaunchShape &s = t->shape[kernel][reduce];
  if (!s.waves)
    // a block of four wavefronts has one on every SIMD
    s = resident_shape(shared, wave, max_waves, std::min(blocks_by_registers(fn, 256, 8), 8),
                       kernel == kTreeRank || kernel == kTree, t->max_lds, t->lds_per_cu);
  return s;
}

// The same for one block size of a kernel: its resident blocks per CU.
LaunchShape block_shape(taccl_plan *p, DeviceTables *t, Kernel kernel, int variant, const void *fn,
                        int threads, int bytes) {
  std::lock_guard<std::mutex> lock(p->mu);
  LaunchShape &s = t->shape[kernel][variant];
  if (!s.waves)
    s = LaunchShape{1, std::max(1, std::min(blocks_by_lds(bytes, t->lds_per_cu),
                                            blocks_by_registers(fn, threads, 1)))};
  return s;
}

}  // namespace
}  // namespace taccl

using namespace taccl;

extern "C" {

void taccl_plan_destroy(taccl_plan_t p) {
  if (!p) return;
  int cur = -1;
  (void)hipGetDevice(&cur);
  for (auto &kv : p->dev) {
    if (hipSetDevice(kv.first) == hipSuccess) (void)hipFree(kv.second.block);
  }
  if (cur >= 0) (void)hipSetDevice(cur);
  delete p;
}

taccl_status_t taccl_plan_upload(taccl_plan_t p) {
  if (!p) return fail(TACCL_ERR_INVALID_ARGUMENT, "null plan");
  DeviceTables *t = nullptr;
  return ensure_device(p, &t);
}

taccl_status_t taccl_eval_batch(taccl_plan_t p, int64_t n, const uint8_t *d_routes,
                                const uint32_t *d_prio, uint32_t *d_makespan, uint8_t *d_valid,
                                taccl_stream_t stream) {
  if (!p) return fail(TACCL_ERR_INVALID_ARGUMENT, "null plan");
  if (n < 0) return fail(TACCL_ERR_INVALID_ARGUMENT, "negative candidate count");
  if (n == 0) return TACCL_OK;
  if (!d_routes || !d_prio || !d_makespan || !d_valid)
    return fail(TACCL_ERR_INVALID_ARGUMENT, "null device pointer");
  if (((uintptr_t)d_prio & 3) || ((uintptr_t)d_makespan & 3))
    return fail(TACCL_ERR_INVALID_ARGUMENT, "d_prio and d_makespan must be 4-byte aligned");
  DeviceTables *t = nullptr;
  taccl_status_t st = ensure_device(p, &t);
  if (st) return st;
  hipStream_t s = (hipStream_t)stream;
  // enough blocks to fill every CU several times over; each block loops
  const int64_t cap = (int64_t)std::max(t->num_cus, 1) * 64;
  const int grid = (int)std::min<int64_t>(n, cap);
  hipError_t e;
  const bool route_words = (p->route_stride % 4 == 0) && (((uintptr_t)d_routes & 3) == 0);
  PathArgs a{};
  PathGreedyArgs g{};
  PortsArgs pa{};
  const Kernel kernel =
      p->coll.kind == TACCL_ALLTOALL ? path_select(*p, t->max_lds, a, g, pa) : kNoKernel;
  if (p->coll.kind == TACCL_ALLTOALL && p->greedy) {
    if (kernel == kNoKernel)
      return fail(TACCL_ERR_UNSUPPORTED,
                  "time-aware greedy orders for Alltoall need at most 65535 send slots "
                  "(chunks x longest path), 4096 chunks and no zero-cost link");
    g.mirror = p->greedy == 2;
    g.gkrank = t->gkrank;
    g.C = p->coll.C;
    g.P = p->topo.P;
    g.E = p->topo.E;
    g.H = std::max(p->H, 1);
    g.cpr = std::max(p->coll.cpr, 1);
    g.route_stride = p->route_stride;
    g.prio_stride = p->prio_stride;
    g.cost = t->cost;
    g.pair_base = t->pair_base;
    g.npaths = t->npaths;
    g.path_off = t->path_off;
    g.path_links = t->path_links;
    g.routes = d_routes;
    g.prio = d_prio;
    g.makespan = d_makespan;
    g.valid = d_valid;
    g.n = n;
    if (kernel == kPathGreedyBlock) {
      // the block kernel has one size: only its resident blocks are asked for
      const LaunchShape sh = block_shape(p, t, kernel, 0, path_greedy_block_fn(g),
                                         kGreedyBlockThreads, g.block_bytes);
      const int bgrid = (int)std::min<int64_t>(n, (int64_t)std::max(t->num_cus, 1) * sh.per_cu);
      e = launch_path_greedy_block(g, bgrid, s);
      if (e != hipSuccess) return hip_fail(e, "kernel launch");
      return TACCL_OK;
    }
    // wavefronts per block: most resident wavefronts per CU
    const LaunchShape sh = wave_shape(p, t, kernel, false, path_greedy_fn(), g.o_wave, g.wave_bytes,
                                      kTreeMaxThreads / 64);
    g.waves_per_block = sh.waves;
    e = launch_path_greedy(g, wave_grid(sh, n, t->num_cus, false), s);
    if (e != hipSuccess) return hip_fail(e, "kernel launch");
    return TACCL_OK;
  }
  if (kernel == kPathPorts) {
    pa.C = p->coll.C;
    pa.H = std::max(p->H, 1);
    pa.nlev = p->nlev;
    pa.route_stride = p->route_stride;
    pa.prio_stride = p->prio_stride;
    pa.routes_words = route_words;
    pa.cost = t->cost;
    pa.arec = t->arec;
    pa.cpath = t->cpath;
    pa.cinfo = t->cinfo;
    pa.cbkt = t->cbkt;
    pa.lfb = t->ports_lfb;
    pa.pwalk = t->pwalk;
    pa.pport = t->pport;
    pa.routes = d_routes;
    pa.prio = d_prio;
    pa.makespan = d_makespan;
    pa.valid = d_valid;
    pa.n = n;
    path_ports_block(pa, n, t->num_cus);
    const LaunchShape sh =
        block_shape(p, t, kernel, pa.nt / 512, path_ports_fn(pa), pa.nt, pa.lds_bytes);
    const int pgrid = (int)std::min<int64_t>(n, (int64_t)std::max(t->num_cus, 1) * sh.per_cu);
    e = launch_path_ports(pa, pgrid, s);
  } else if (p->coll.kind == TACCL_ALLTOALL) {
    if (kernel == kNoKernel)
      return fail(TACCL_ERR_UNSUPPORTED,
                  a.lds_bytes > t->max_lds ? "Alltoall plan needs more LDS than a block has"
                                           : "switch ports take at most four links per thread");
    a.C = p->coll.C;
    a.P = p->topo.P;
    a.E = p->topo.E;
    a.H = std::max(p->H, 1);
    a.cpr = p->coll.cpr;
    a.nlev = p->nlev;
    a.route_stride = p->route_stride;
    a.prio_stride = p->prio_stride;
    a.cost = t->cost;
    a.pair_base = t->pair_base;
    a.npaths = t->npaths;
    a.path_off = t->path_off;
    a.hop_class = t->hop_class;
    a.path_lvl_hop = t->path_lvl_hop;
    a.lvl_cls_begin = t->lvl_cls_begin;
    a.llc = t->llc;
    a.routes = d_routes;
    a.prio = d_prio;
    a.makespan = d_makespan;
    a.valid = d_valid;
    a.n = n;
    a.contig = p->contig;
    a.lalpha = t->lalpha;
    a.lbs = t->lbs;
    a.lmerge = t->lmerge;
    a.cml = (const uint4 *)t->cml;
    a.cwalk = t->cwalk;
    a.nmerge = (int32_t)p->cml.size() / 4;
    a.ports = p->ports;
    a.hop_class2 = t->hop_class2;
    a.lvl_cls2_begin = t->lvl_cls2_begin;
    a.llc2 = t->llc2;
    a.cls2_link = t->cls2_link;
    a.arec = t->arec;
    a.cpath = t->cpath;
    a.routes_words = route_words;
    a.cinfo = t->cinfo;
    a.cbkt = t->cbkt;
    if (kernel == kPathFast) {
      const int cpt = path_fast_cpt(*p), nt = path_fast_threads(*p);
      const LaunchShape sh =
          block_shape(p, t, kernel, 0, path_fast_fn(a, cpt, nt), nt, a.lds_bytes);
      const int fgrid = (int)std::min<int64_t>(n, (int64_t)std::max(t->num_cus, 1) * sh.per_cu);
      e = launch_path_fast(a, cpt, nt, fgrid, s);
    } else {
      e = launch_path(a, grid, s);
    }
  } else {
    TreeArgs x{};
    x.C = p->coll.C;
    x.P = p->topo.P;
    x.V = p->topo.V;
    x.E = p->topo.E;
    x.route_stride = p->route_stride;
    x.prio_stride = p->prio_stride;
    x.routes_word_aligned = route_words;
    x.cost = t->cost;
    x.lsrc = t->lsrc;
    x.ldst = t->ldst;
    x.lrev = t->lrev;
    x.rec = t->tree_rec;
    x.npaths = t->npaths;
    x.owner8 = t->owner8;
    x.topt = t->topt;
    x.ent = t->tent;
    x.rank_img = (const uint4 *)t->rank_img;
    x.contig = p->contig;
    x.greedy = p->greedy;
    x.lalpha = t->lalpha;
    x.lbs = t->lbs;
    x.lmerge = t->lmerge;
    x.rec4 = (const uint4 *)t->tree_rec4;
    x.post_mask = t->post_mask;
    x.routes = d_routes;
    x.makespan = d_makespan;
    x.valid = d_valid;
    x.n = n;
    // An Allreduce is a ReduceScatter on the first priority row, then an
    // Allgather on the second, adding its makespan (same stream, so in order);
    // both kernels are chosen before the first is launched
    TreeArgs phase[2];
    Kernel kernels[2];
    int phases = 0;
    const int kind = p->coll.kind;
    for (int reduce = 1; reduce >= 0; reduce--) {
      if (reduce ? kind != TACCL_REDUCESCATTER && kind != TACCL_ALLREDUCE
                 : kind == TACCL_REDUCESCATTER)
        continue;
      TreeArgs &y = phase[phases] = x;
      y.reduce = reduce;
      y.accumulate = phases;
      y.prio = d_prio + (size_t)phases * p->coll.C * p->topo.V;
      kernels[phases] = tree_select(*p, reduce, route_words, t->max_lds, y);
      if (kernels[phases++] == kNoKernel)
        return fail(TACCL_ERR_UNSUPPORTED, "multicast plan needs more LDS than a block has");
    }
    e = hipSuccess;
    for (int i = 0; i < phases && e == hipSuccess; i++) {
      TreeArgs &y = phase[i];
      const Kernel k = kernels[i];
      const void *fn = k == kTreeRank     ? tree_rank_fn(y)
                       : k == kTreeGreedy ? tree_greedy_fn(y)
                       : k == kTreeLayers ? tree_layers_fn(y)
                                          : tree_fn(y);
      const LaunchShape sh =
          wave_shape(p, t, k, y.reduce != 0, fn, y.o_wave, y.wave_bytes,
                     k == kTreeRank ? tree_rank_max_waves(y) : kTreeMaxThreads / 64);
      y.waves_per_block = sh.waves;
      // The ranked and the general kernel deal candidates out over the blocks
      // where a CU holds one of them, so that a batch which is no multiple of
      // the resident wavefronts leaves every CU with as few as it can (20000
      // Allgathers on two 8-rank meshes 144 -> 129 us, 44 Allreduces on two
      // nodes of 7 ranks 41.1 -> 30.4 us), and where there is a CU for each
      // candidate. Else several blocks per CU fill up block by block: dealt
      // out, the last candidates would all be on the SIMDs of the blocks' first
      // wavefronts (20000 Allgathers on 10 ranks 35.1 -> 38.2 us).
      const bool spread =
          (k == kTreeRank || k == kTree) && (sh.per_cu == 1 || n <= t->num_cus);
      const int tgrid = wave_grid(sh, n, t->num_cus, spread);
      y.first_block = spread ? 1 : sh.waves;
      y.first_wave = spread ? tgrid : 1;
      e = k == kTreeRank     ? launch_tree_rank(y, tgrid, s)
          : k == kTreeGreedy ? launch_tree_greedy(y, tgrid, s)
          : k == kTreeLayers ? launch_tree_layers(y, tgrid, s)
                             : launch_tree(y, tgrid, s);
    }
  }
  if (e != hipSuccess) return hip_fail(e, "kernel launch");
  return TACCL_OK;
}

taccl_status_t taccl_count_faults(int64_t n, const uint32_t *makespan, int64_t *faults) {
  if (!faults) return fail(TACCL_ERR_INVALID_ARGUMENT, "null output");
  if (n < 0) return fail(TACCL_ERR_INVALID_ARGUMENT, "negative candidate count");
  if (n > 0 && !makespan) return fail(TACCL_ERR_INVALID_ARGUMENT, "null makespan array");
  int64_t k = 0;
  for (int64_t i = 0; i < n; i++) k += makespan[i] == TACCL_MAKESPAN_FAULT;
  *faults = k;
  return TACCL_OK;
}

// the seeded input generator shared with the tests (workloads/candgen.c)
extern "C" int candgen_fill(uint64_t seed, int64_t first, int64_t count, int route_stride,
                            const int32_t *options, int prio_stride, uint8_t *routes,
                            uint32_t *prio);

taccl_status_t taccl_generate_host(taccl_plan_t p, uint64_t seed, int64_t first, int64_t count,
                                   uint8_t *routes, uint32_t *prio) {
  if (!p) return fail(TACCL_ERR_INVALID_ARGUMENT, "null plan");
  if (first < 0 || count < 0)
    return fail(TACCL_ERR_INVALID_ARGUMENT, "negative first candidate or count");
  if (count == 0) return TACCL_OK;
  if (!routes || !prio) return fail(TACCL_ERR_INVALID_ARGUMENT, "null output buffer");
  if (candgen_fill(seed, first, count, p->route_stride, p->route_options.data(), p->prio_stride,
                   routes, prio) != 0)
    return fail(TACCL_ERR_INVALID_ARGUMENT, "candidate range beyond 2^32");
  return TACCL_OK;
}

taccl_status_t taccl_connections_batch(taccl_plan_t p, int64_t n, const uint8_t *d_routes,
                                       uint32_t *d_connections, taccl_stream_t stream) {
  if (!p) return fail(TACCL_ERR_INVALID_ARGUMENT, "null plan");
  if (n < 0) return fail(TACCL_ERR_INVALID_ARGUMENT, "negative candidate count");
  if (n == 0) return TACCL_OK;
  if (!d_routes || !d_connections) return fail(TACCL_ERR_INVALID_ARGUMENT, "null device pointer");
  if ((uintptr_t)d_connections & 3)
    return fail(TACCL_ERR_INVALID_ARGUMENT, "d_connections must be 4-byte aligned");
  const int32_t P = p->topo.P, V = p->topo.V;
  const bool tree = p->coll.kind != TACCL_ALLTOALL;
  if (P > 256 || (tree && (P > 64 || V > 255)))
    return fail(TACCL_ERR_UNSUPPORTED, "connection counts need at most 256 ranks (multicast: "
                                       "64 ranks and 255 vertices)");
  DeviceTables *t = nullptr;
  taccl_status_t st = ensure_device(p, &t);
  if (st) return st;
  ConnArgs a{};
  a.C = p->coll.C;
  a.P = P;
  a.V = V;
  a.cpr = std::max(p->coll.cpr, 1);
  a.kind = p->coll.kind;
  a.tree = tree ? 1 : 0;
  a.mask_words = (P * P + 31) / 32;
  a.route_stride = p->route_stride;
  a.ldst = t->ldst;
  a.pair_base = t->pair_base;
  a.npaths = t->npaths;
  a.path_off = t->path_off;
  a.path_links = t->path_links;
  a.owner = t->owner;
  a.post_mask = t->post_mask;
  a.routes = d_routes;
  a.out = d_connections;
  a.n = n;
  if (t->cn_rec) {
    a.rec = t->cn_rec;
    a.chunk = (const uint4 *)t->cn_chunk;
    a.nrec = (int32_t)p->cn_rec.size();
    a.cells = p->conn_cells;
    a.nwords = (a.C + 3) / 4;
    a.lanes = 4;
    while (a.lanes < 64 && a.lanes < a.nwords) a.lanes *= 2;
    a.routes_words = (p->route_stride % 4 == 0) && (((uintptr_t)d_routes & 3) == 0);
    const int64_t cus = std::max(t->num_cus, 1), per_wave = 64 / a.lanes;
    // The record table is copied to LDS when a CU makes half as many lookups as
    // it has records or more, or it is small; else it is read from the L2. 24
    // ranks on a switch (12697 records, 576 lookups a candidate): 64 candidates 8.3
    // us with the copy and 4.3 us without, 2000 (4500 lookups per CU) 7.0 and
    // 5.3 us, 4000 7.1 and 7.9 us, 20000 12.2 and 18.8 us; 8 ranks (393
    // records) 4.4 and 4.6 us at any batch.
    a.rec_lds = 4 * a.nrec <= kConnRecLdsMax &&
                (a.nrec <= kConnRecSmall || n * a.C / cus >= a.nrec / 2);
    // as many wavefronts per block as spread the batch over every CU, 4 at
    // least (they share the record table), 16 at most
    const int64_t want = (n + per_wave - 1) / per_wave;
    int waves = (int)std::min<int64_t>(kConnWaveThreads / 64, std::max<int64_t>(4, want / cus));
    while (waves > 1 && connections_wave_lds_bytes(a, waves) > t->max_lds) waves--;
    const int bytes = connections_wave_lds_bytes(a, waves);
    if (bytes <= t->max_lds) {
      const int bpc = std::max(1, std::min(t->lds_per_cu / bytes, 32 / waves));
      const int wgrid = (int)std::min<int64_t>((want + waves - 1) / waves, cus * bpc);
      hipError_t e = launch_connections_wave(a, waves, wgrid, (hipStream_t)stream);
      if (e != hipSuccess) return hip_fail(e, "kernel launch");
      return TACCL_OK;
    }
  }
  // one chunk per thread at a time; multicast blocks keep a parent byte per
  // vertex and thread in LDS
  int threads = std::min(kConnMaxThreads, std::max(64, (a.C + 63) / 64 * 64));
  while (threads > 64 && connections_lds_bytes(a, threads) > t->max_lds) threads -= 64;
  if (connections_lds_bytes(a, threads) > t->max_lds)
    return fail(TACCL_ERR_UNSUPPORTED, "connection count needs more LDS than a block has");
  const int per_cu = std::max(1, std::min(t->lds_per_cu / std::max(connections_lds_bytes(a, threads), 1),
                                          2048 / threads));
  const int grid = (int)std::min<int64_t>(n, (int64_t)std::max(t->num_cus, 1) * per_cu);
  hipError_t e = launch_connections(a, threads, grid, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "kernel launch");
  return TACCL_OK;
}

}  // extern "C"
