// Alltoall with switch ports (App. B.3) for gfx950: plans whose tables and
// level buffers fit one block's LDS (routes of at most 6 hops, 8 levels,
// 4096 chunks); eval_path.hip's general kernel takes the rest.
//
// One block evaluates one candidate at a time. A send is one hop, or a hop
// pair rank -> switch -> rank that holds the sender's send port (uplink) and
// the receiver's receive port (downlink) together. Sends of equal remaining
// cost form a level, and no send depends on another one of its level except
// through a port. Each port serves its sends of a level in one key order
// (travelled, priority, chunk), so per level:
//   A. the level's switched sends are ordered by receive port, which gives
//      every send its place on its receive port;
//   B. all its sends are ordered by send port;
//   C. every send port walks its run: a switched send goes once its receive
//      port has served as many sends as its place says, a plain one at once.
// The chosen routes' records and the priorities of their hops are in
// registers, loaded while the previous candidate's last level is walked.
// Both orders of every level are counted once per candidate and scanned
// together; each is a counting sort into (class, top priority bits) buckets
// and a rank inside the bucket.
//
// What bounds it: the walk, a chain of about 1.5 sends per send of the
// busiest port and level, each one LDS round trip. A receive port is one
// 8-byte word, {sends served, busy until}: a waiting send reads that word
// alone, and the send that serves it writes it, so a step costs one read and
// one write. The send ports into one switch lie in one wavefront where they
// fit (their receive ports are shared with no others), so a step seen by
// the next iteration costs no polling across wavefronts. fournode64 (four
// 16-rank switches, 8192 candidates): 7.69 ms on the general kernel, 2.42 ms
// here (177 K cycles per candidate, one block per CU: 103 K in the walk, 17 K
// set-up and counting, 50 K in the two orders). The general kernel looks
// every hop up through three dependent global loads in each pass and polls
// a chunk's predecessor across wavefronts, about 870 cycles a step.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "path_sort.h"
#include "wave.h"

namespace taccl {

namespace {

constexpr uint32_t kNoClass = 0xFFFFu;
// the place a send port waits for once its run is served: no receive port's
// count reaches it
constexpr uint32_t kThrough = 0xFFFFFFFFu;
// the receive ports' words lie at the start of the block's LDS and the
// chunks' arrivals behind them, so that both have constant bases
constexpr int kPortsMaxRecv = 256;
constexpr int kPortsCtime = 8 * kPortsMaxRecv;

__device__ __forceinline__ uint64_t lds_get64(uint64_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_put64(uint64_t *p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Hop h of a chunk (7: none) out of its six classes and priorities.
__device__ __forceinline__ uint32_t pick_class(const uint32_t (&w)[3], uint32_t h) {
  const uint32_t w0 = w[0], w1 = w[1], w2 = w[2];  // values: no array address is selected
  const uint32_t x = h >= 4 ? w2 : h >= 2 ? w1 : w0;
  return (h & 1) ? x >> 16 : x & 0xFFFFu;
}
__device__ __forceinline__ uint32_t pick_prio(const uint32_t (&p)[kFastMaxHops], uint32_t h) {
  const bool c2 = h >= 2, c4 = h >= 4;
  const uint32_t p0 = p[0], p1 = p[1], p2 = p[2], p3 = p[3], p4 = p[4], p5 = p[5];
  const uint32_t e = c4 ? p4 : c2 ? p2 : p0, o = c4 ? p5 : c2 ? p3 : p1;
  return (h & 1) ? o : e;
}

template <int CPT, int NT>
__global__ __launch_bounds__(NT) void path_eval_ports(PortsArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int C = a.C, H = a.H, nlev = a.nlev;
  const uint32_t NB = (uint32_t)(a.nb1 + a.nb2);
  // per class first bucket | bits << 24, the receive-port classes after the
  // send-port ones (and their buckets too); per receive-port class port |
  // first bucket of the port's run << 16
  uint32_t *s_cbkt = (uint32_t *)(lds + a.o_cbkt), *s_cbkt2 = s_cbkt + a.ncls;
  uint32_t *s_cinfo2 = (uint32_t *)(lds + a.o_cinfo);
  uint32_t *s_lfb = (uint32_t *)(lds + a.o_lfb);    // [nlev+1] first send-port bucket
  uint32_t *s_lfb2 = s_lfb + nlev + 1;              // [nlev+1] first receive-port bucket
  // a receive port: sends served at this level << 32 | busy until
  uint64_t *rp = (uint64_t *)lds;
  uint32_t *ctime = (uint32_t *)(lds + kPortsCtime);  // a chunk's arrival so far
  // bucket cursors as in the register-resident kernel: bst[b + 1] holds
  // bucket b's count, then its start, then its end; a dummy counter per lane
  // follows
  uint32_t *bst = (uint32_t *)(lds + a.o_bst) + 3;
  uint64_t *e64 = (uint64_t *)(lds + a.o_e64);  // priority << 32 | link << cb | chunk
  uint32_t *aux = (uint32_t *)(lds + a.o_aux);  // bucket | first bucket of the port's run << 16
  uint32_t *pinfo = (uint32_t *)(lds + a.o_pinfo);  // link << cb | chunk by send-port position
  // per chunk: place on its receive port << 8 | that port
  uint32_t *rk = (uint32_t *)(lds + a.o_rk);
  // the walk's view of a position (over e64): chunk << 20 | place on the
  // receive port << 8 | that port, and the ready time
  uint2 *wcr = (uint2 *)e64;
  auto place_of = [](const uint2 &w) -> uint32_t { return (w.x >> 8) & 0xFFFu; };
  uint32_t *red = (uint32_t *)(lds + a.o_red);
  const uint32_t cb = (uint32_t)a.cbits, cmask = (1u << cb) - 1;

  for (int j = tid; j < a.ncls + a.ncls2; j += NT) s_cbkt[j] = a.cbkt[j];
  for (int j = tid; j < a.ncls2; j += NT) s_cinfo2[j] = a.cinfo[j];
  for (int j = tid; j < 2 * (nlev + 1); j += NT) s_lfb[j] = a.lfb[j];
  for (uint32_t j = tid; j < NB + 2; j += NT) bst[j] = 0;
  // every word of the receive ports' region, also those of no port: a send
  // port that is through reads one by whatever lies behind its run
  for (int l = tid; l < kPortsMaxRecv; l += NT) rp[l] = 0;
  // this thread's send port (0xFFFF: none) and its latency; wavefronts hold
  // either ports into switches, on which every send is switched, or plain
  // links
  const uint32_t port = tid < a.nports ? a.pport[tid] : 0xFFFFu;
  const uint32_t pcost = port != 0xFFFFu ? a.cost[port] : 0u;
  const bool wave_switched = __builtin_amdgcn_readfirstlane(tid) < a.nswitched;
  __syncthreads();

  uint32_t pr[CPT][kFastMaxHops], kk[CPT], cp[CPT];
#pragma unroll
  for (int j = 0; j < CPT; j++)
#pragma unroll
    for (int h = 0; h < kFastMaxHops; h++) pr[j][h] = 0;
  // the candidate's route choices, chunk table entries and priorities, one
  // batch of branch-free loads (past the batch: the last candidate again,
  // past the chunks: the last chunk, never used)
  auto load_inputs = [&](int64_t i) {
    const int64_t ii = i < a.n ? i : a.n - 1;
    const uint8_t *grt = a.routes + (size_t)ii * a.route_stride;
    const uint32_t *grw = (const uint32_t *)grt;
    const uint32_t *gpr = a.prio + (size_t)ii * a.prio_stride;
    int tv = tid;
    asm volatile("" : "+v"(tv));  // addresses recomputed, not kept in registers
#pragma unroll
    for (int j = 0; j < CPT; j++) {
      const uint32_t cc = (uint32_t)min(tv + NT * j, C - 1);
      if (a.routes_words)
        kk[j] = grw[cc >> 2];
      else
        kk[j] = (uint32_t)grt[cc] << (8 * (cc & 3));
      cp[j] = a.cpath[cc];
      const uint32_t *row = gpr + __umul24(cc, (uint32_t)H);
#pragma unroll
      for (int h = 0; h < kFastMaxHops; h++)
        if (h < H) pr[j][h] = row[h];
    }
  };
  load_inputs(blockIdx.x);
  for (int64_t i = blockIdx.x; i < a.n; i += gridDim.x) {
    int tv = tid;
    asm volatile("" : "+v"(tv));
    // route records: hop at each level (3 bits per level, 7: none), send-port
    // and receive-port class of every hop (kNoClass: no send starts there)
    uint32_t lv[CPT], rc1[CPT][3], rc2[CPT][3];
    bool unrouted = false;
#pragma unroll
    for (int j = 0; j < CPT; j++) {
      const int c = tv + NT * j;
      const uint32_t np = cp[j] >> 24;
      const bool live = c < C;
      const uint32_t k = (kk[j] >> (8 * ((uint32_t)c & 3u))) & 0xFFu;
      if (live && (cp[j] == kNoRoute || (np && k >= np))) unrouted = true;
      const uint32_t rec = (live && k < np) ? (cp[j] & 0xFFFFFFu) + k : 0u;
      const uint4 r = ((const uint4 *)a.arec)[2 * rec];
      const uint4 r2 = ((const uint4 *)a.arec)[2 * rec + 1];
      lv[j] = r.x;
      rc1[j][0] = r.y;
      rc1[j][1] = r.z;
      rc1[j][2] = r.w;
      rc2[j][0] = r2.x;
      rc2[j][1] = r2.y;
      rc2[j][2] = r2.z;
      if (live) ctime[c] = 0;
    }
    for (int l = tid; l < a.nrecv; l += NT) lds_put64(&rp[l], 0);
    // count both orders of every level
#pragma unroll
    for (int j = 0; j < CPT; j++)
#pragma unroll
      for (int h = 0; h < kFastMaxHops; h++) {
        if (h >= H) break;
        const uint32_t c1 = (rc1[j][h >> 1] >> (16 * (h & 1))) & 0xFFFFu;
        const uint32_t c2 = (rc2[j][h >> 1] >> (16 * (h & 1))) & 0xFFFFu;
        const uint32_t k1 = s_cbkt[c1 != kNoClass ? c1 : 0u];
        const uint32_t k2 = s_cbkt2[c2 != kNoClass ? c2 : 0u];
        const uint32_t b1 = (k1 & 0xFFFFFFu) + top_bits(pr[j][h], k1 >> 24);
        const uint32_t b2 = (k2 & 0xFFFFFFu) + top_bits(pr[j][h], k2 >> 24);
        atomicAdd(&bst[c1 != kNoClass ? b1 + 1 : NB + 2 + lane], 1u);
        atomicAdd(&bst[c2 != kNoClass ? b2 + 1 : NB + 2 + lane], 1u);
      }
    const bool any_unrouted = __syncthreads_or(unrouted);
    block_excl_scan4(bst + 1, (int)NB, red);

    uint32_t mk = 0, F = 0;  // F: this thread's send port is busy until then
    bool fault = false;
    for (int L = 0; L < nlev; L++) {
      // the level's run of this thread's port: first and end bucket
      const uint32_t pb = tid < a.nports ? a.pwalk[(size_t)L * a.nports + tid] : 0u;
      // ---- A. places on the receive ports -----------------------------------
      const uint32_t q0 = bst[s_lfb2[L]];
#pragma unroll
      for (int j = 0; j < CPT; j++) {
        const uint32_t h = (lv[j] >> (3 * L)) & 7;
        const uint32_t c2 = h < (uint32_t)kFastMaxHops ? pick_class(rc2[j], h) : kNoClass;
        const bool act = c2 != kNoClass;
        const uint32_t pv = pick_prio(pr[j], h);
        const uint32_t ck = act ? c2 : 0u;
        const uint32_t kb = s_cbkt2[ck], ci = s_cinfo2[ck];
        const uint32_t b = (kb & 0xFFFFFFu) + top_bits(pv, kb >> 24);
        const uint32_t gp = atomicAdd(&bst[act ? b + 1 : NB + 2 + lane], 1u);
        if (act) {
          e64[gp - q0] = ((uint64_t)pv << 32) | (uint32_t)(tid + NT * j) | ((ci & 0xFFFFu) << cb);
          aux[gp - q0] = b | (ci & 0xFFFF0000u);
        }
      }
      __syncthreads();
      const uint32_t tot2 = bst[s_lfb2[L + 1]] - q0;
      for (uint32_t x = tid; x < tot2; x += NT) {
        const uint64_t me = e64[x];
        const uint32_t ax = aux[x], b = ax & 0xFFFFu;
        const uint32_t b0 = bst[b] - q0, b1 = bst[b + 1] - q0, rs = bst[ax >> 16] - q0;
        const uint32_t place = b0 + rank_in_bucket(e64, b0, b1, me) - rs;
        rk[(uint32_t)me & cmask] = (place << 8) | ((uint32_t)me >> cb);
      }
      __syncthreads();
      // ---- B. send-port order -----------------------------------------------
      const uint32_t p0 = bst[s_lfb[L]];
#pragma unroll
      for (int j = 0; j < CPT; j++) {
        const uint32_t h = (lv[j] >> (3 * L)) & 7;
        const uint32_t c1 = h < (uint32_t)kFastMaxHops ? pick_class(rc1[j], h) : kNoClass;
        const bool act = c1 != kNoClass;
        const uint32_t pv = pick_prio(pr[j], h);
        const uint32_t ck = act ? c1 : 0u;
        const uint32_t kb = s_cbkt[ck];
        const uint32_t b = (kb & 0xFFFFFFu) + top_bits(pv, kb >> 24);
        const uint32_t gp = atomicAdd(&bst[act ? b + 1 : NB + 2 + lane], 1u);
        if (act) {
          // the receive port's class says whether the send is switched
          const bool sw = pick_class(rc2[j], h) != kNoClass;
          e64[gp - p0] = ((uint64_t)pv << 32) | (uint32_t)(tid + NT * j) |
                         (sw ? 0x80000000u : 0u);
          aux[gp - p0] = b;
        }
      }
      if (L == nlev - 1) load_inputs(i + gridDim.x);  // this candidate's inputs are dead
      __syncthreads();
      const uint32_t tot = bst[s_lfb[L + 1]] - p0;
      for (uint32_t x = tid; x < tot; x += NT) {
        const uint64_t me = e64[x];
        const uint32_t b = aux[x];
        const uint32_t b0 = bst[b] - p0, b1 = bst[b + 1] - p0;
        pinfo[b0 + rank_in_bucket(e64, b0, b1, me)] = (uint32_t)me;
      }
      __syncthreads();
      // ---- C. the walk -------------------------------------------------------
      for (uint32_t x = tid; x < tot; x += NT) {
        const uint32_t pi = pinfo[x], c = pi & cmask, k = (pi >> 31) ? rk[c] : 0u;
        wcr[x] = make_uint2((c << 20) | k, ctime[c]);
      }
      // a receive port has served none of this level's sends yet
      for (int l = tid; l < a.nrecv; l += NT) ((uint32_t *)&rp[l])[1] = 0;
      uint32_t p = 0, e = 0;
      if (pb != 0) {
        p = bst[pb & 0xFFFFu] - p0;
        e = bst[pb >> 16] - p0;
      }
      __syncthreads();
      if (!wave_switched) {  // plain links only (or no ports)
        uint2 w = wcr[p];
        asm volatile("" : "+v"(w.x), "+v"(w.y));
        while (__ballot(p < e)) {
          uint2 n = wcr[p + 1];
          asm volatile("" : "+v"(n.x), "+v"(n.y));
          if (p < e) {
            F = max(w.y, F) + pcost;
            ((uint32_t *)(lds + kPortsCtime))[w.x >> 20] = F;
            p++;
            w = n;
          }
        }
      } else {
        // want: the place this lane's front send waits for on its receive
        // port (a lane that is through waits for one no port's word holds). A
        // step reads the port's word and, with it, the send behind, so it
        // is one LDS round trip whether the send goes or not; the empty asm
        // keeps the second read out of the branch, where the compiler moves
        // it and makes that two (2.81 ms). One wavefront has the CU to itself here, so
        // every instruction of the step counts: constant LDS bases, and the
        // end is looked for every fourth step (2.74 ms with a test per step).
        const uint2 *at = wcr + p, *end = wcr + e;
        uint2 w = *at;
        uint32_t want = at < end ? place_of(w) : kThrough;
        // (their loads end here, not at the loop's head, where the wait would
        // also cover every step's stores)
        asm volatile("" : "+v"(w.x), "+v"(w.y), "+v"(want));
        const int limit = 16 * (__builtin_amdgcn_readfirstlane((int)tot) + 64);
        for (int step = 0; __ballot(want != kThrough); step++) {
#pragma unroll
          for (int u = 0; u < 4; u++) {
            uint64_t *port_word = (uint64_t *)lds + (w.x & 0xFFu);
            const uint64_t rv = lds_get64(port_word);
            const uint2 n = at[1];
            asm volatile("" ::: "memory");
            if ((uint32_t)(rv >> 32) == want) {
              F = max(max(w.y, F), (uint32_t)rv) + pcost;
              lds_put64(port_word, ((uint64_t)(want + 1) << 32) | F);
              ((uint32_t *)(lds + kPortsCtime))[w.x >> 20] = F;
              at++;
              w = n;
              want = at < end ? place_of(w) : kThrough;
            }
          }
          if (step > limit) {  // unreachable: both ports serve one key order
            fault = true;
            break;
          }
        }
      }
      mk = max(mk, F);
      __syncthreads();
    }
    if (nlev == 0) load_inputs(i + gridDim.x);
    // a send port's finishes ascend, so the makespan is the latest busy time
    mk = wave_reduce_max(mk);
    if (lane == 0) red[wave] = mk;
    const bool failed = __syncthreads_or(fault);
    if (tid == 0) {
      uint32_t m = 0;
      for (int v = 0; v < NT / 64; v++) m = max(m, red[v]);
      a.makespan[i] = failed ? 0xFFFFFFFFu : m;
      a.valid[i] = (uint8_t)(!any_unrouted && !failed);
    }
    for (uint32_t j = tid; j < (NB + 4) / 4; j += NT)
      ((uint4 *)(bst + 1))[j] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
  }
}

const void *ports_fn(int cpt, int nt) {
  switch (nt * 8 + cpt) {
    case 256 * 8 + 1: return (const void *)path_eval_ports<1, 256>;
    case 256 * 8 + 4: return (const void *)path_eval_ports<4, 256>;
    case 512 * 8 + 1: return (const void *)path_eval_ports<1, 512>;
    case 512 * 8 + 2: return (const void *)path_eval_ports<2, 512>;
    case 1024 * 8 + 1: return (const void *)path_eval_ports<1, 1024>;
    case 1024 * 8 + 2: return (const void *)path_eval_ports<2, 1024>;
    case 1024 * 8 + 4: return (const void *)path_eval_ports<4, 1024>;
  }
  return nullptr;
}

}  // namespace

int32_t path_ports_layout(const taccl_plan &p, PortsArgs &a) {
  const int32_t C = p.coll.C, M = std::max(p.max_lvl_sends, 1);
  if (!p.ports_fast || C < 1) return 0;
  a.nt = C <= 256 ? 256 : C <= 512 ? 512 : 1024;
  const int32_t per = (C + a.nt - 1) / a.nt;
  a.cpt = per <= 1 ? 1 : per <= 2 ? 2 : 4;
  a.nports = (int32_t)p.pport.size();
  a.nswitched = p.nswitched;
  a.nrecv = p.nrecv;
  // one send port per thread; a position's word holds 12 bits of chunk, 12 of
  // place and 8 of receive port
  if (per > 4 || a.nports > a.nt || a.nrecv > kPortsMaxRecv || C > 4096 || M > 4096) return 0;
  a.nb1 = p.nb_total;
  a.nb2 = p.nb2_total;
  a.ncls = p.ncls;
  a.ncls2 = (int32_t)p.cls2_link.size();
  a.cbits = 0;
  while ((1 << a.cbits) < C) a.cbits++;
  int32_t off = (kPortsCtime + 4 * C + 15) & ~15;
  auto take = [&](int32_t bytes) {
    const int32_t o = off;
    off = (off + bytes + 15) & ~15;
    return o;
  };
  a.o_cinfo = take(4 * (a.ncls2 + 1));
  a.o_cbkt = take(4 * (a.ncls + a.ncls2 + 1));
  a.o_lfb = take(4 * 2 * (p.nlev + 1));
  // three words of padding, a zero, the cursors, the total, a dummy per lane
  a.o_bst = take(4 * (3 + a.nb1 + a.nb2 + 2 + 64));
  // three spare entries past the end (the rank pass reads four at a time, the
  // walk one ahead)
  a.o_e64 = take(8 * (M + 3));
  a.o_aux = take(4 * M);
  a.o_pinfo = take(4 * M);
  a.o_rk = take(4 * C);
  a.o_red = take(4 * 2 * (1024 / 64));
  a.lds_bytes = off;
  return off;
}

// One candidate per block, and its walk keeps a few wavefronts busy, so with
// 513 to 1024 chunks a batch that fills the CUs takes smaller blocks, of which
// a CU holds more (registers admit one of 1024 threads, two of 512, four of
// 256), as far as a thread per send port goes. 24 ranks on two switches: 3000
// candidates 281 us in blocks of 1024 (261 on the general kernel, whose
// blocks have 256), 165 of 512, 111 of 256; 300 candidates 49.8, 30.7 and
// 34.9 us; one 24.7, 25.7 and 30.3 us.
void path_ports_block(PortsArgs &a, int64_t n, int cus) {
  if (a.C <= 512 || a.C > 1024) return;
  a.nt = n <= cus ? 1024 : n <= 2 * (int64_t)cus ? 512 : 256;
  while (a.nt < a.nports) a.nt *= 2;
  a.cpt = 1024 / a.nt;
}

const void *path_ports_fn(const PortsArgs &a) { return ports_fn(a.cpt, a.nt); }

hipError_t launch_path_ports(const PortsArgs &a, int grid, hipStream_t stream) {
  const void *fn = ports_fn(a.cpt, a.nt);
  if (!fn) return hipErrorInvalidValue;
  void *args[] = {(void *)&a};
  return hipLaunchKernel(fn, dim3(grid), dim3(a.nt), args, a.lds_bytes, stream);
}

}  // namespace taccl
