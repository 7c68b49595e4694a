// Switch-hyperedge connection count for gfx950 (Sec. 3.2 and the
// switch-hyperedge policy of Sec. 5.1; App. B.3: is_util[src, r] is 1 when
// some chunk travels from GPU src to GPU r over a switched link, and the
// uc-max / uc-min policies add gamma * sum(is_util) to the objective, gamma
// negative for uc-max and positive for uc-min).
//
// A connection is an ordered rank pair (a, b) that exchanges a chunk
// through switch vertices only. Alltoall: two ranks of a chunk's routed
// path with only switch vertices between them. Multicast: the routed paths
// of a chunk merge into its tree by first reach (destinations ascending, as
// in the evaluation kernels); a rank whose tree parent is a switch forms a
// pair with the nearest rank above it. ReduceScatter runs the trees
// backwards, so its pairs are reversed; Allreduce has both directions.
//
// One block per candidate at a time (grid-stride). The candidate's pairs
// are set in a P x P bit matrix in LDS, which is then counted.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"

namespace taccl {

namespace {

__device__ __forceinline__ void set_pair(uint32_t *bits, uint32_t a, uint32_t b, uint32_t P) {
  const uint32_t x = a * P + b;
  atomicOr(&bits[x >> 5], 1u << (x & 31));
}

template <bool kTree>
__global__ __launch_bounds__(kConnMaxThreads) void connections_kernel(ConnArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ uint32_t total;
  const uint32_t P = (uint32_t)a.P, V = (uint32_t)a.V;
  const int C = a.C, MW = a.mask_words;
  uint32_t *bits = (uint32_t *)lds;
  // multicast: tree parent of every vertex of this thread's chunk (0xFF: not
  // reached); vertex ids are below 255
  uint8_t *par = lds + 4 * MW + threadIdx.x * V;
  for (int64_t i = blockIdx.x; i < a.n; i += gridDim.x) {
    for (int w = threadIdx.x; w < MW; w += blockDim.x) bits[w] = 0;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    const uint8_t *rt = a.routes + (size_t)i * a.route_stride;
    for (int c = threadIdx.x; c < C; c += blockDim.x) {
      if (!kTree) {
        // chunk c = (s*P + d)*cpr + j
        const uint32_t sd = (uint32_t)c / (uint32_t)a.cpr;
        const uint32_t s = sd / P, d = sd - s * P;
        if (s == d) continue;
        const uint32_t k = rt[c];
        if (k >= a.npaths[sd]) continue;  // unrouted
        const uint32_t q = a.pair_base[sd] + k;
        uint32_t last = s;
        bool through_switch = false;
        for (uint32_t j = a.path_off[q]; j < a.path_off[q + 1]; j++) {
          const uint32_t v = a.ldst[a.path_links[j]];
          if (v >= P) {
            through_switch = true;
            continue;
          }
          if (through_switch) set_pair(bits, last, v, P);
          last = v;
          through_switch = false;
        }
      } else {
        const uint32_t o = (uint32_t)a.owner[c];
        const uint64_t pm = a.post_mask[c];
        for (uint32_t v = 0; v < V; v++) par[v] = 0xFF;
        par[o] = (uint8_t)o;
        for (uint32_t d = 0; d < P; d++) {
          if (d == o || !((pm >> d) & 1)) continue;
          const uint32_t k = rt[(size_t)c * P + d];
          const uint32_t pp = o * P + d;
          if (k >= a.npaths[pp]) continue;  // unrouted
          const uint32_t q = a.pair_base[pp] + k;
          uint32_t u = o;
          for (uint32_t j = a.path_off[q]; j < a.path_off[q + 1]; j++) {
            const uint32_t v = a.ldst[a.path_links[j]];
            if (par[v] == 0xFF) par[v] = (uint8_t)u;  // first reach
            u = v;
          }
        }
        for (uint32_t b = 0; b < P; b++) {
          if (b == o || par[b] == 0xFF) continue;
          uint32_t x = par[b];
          if (x < P) continue;
          while (x >= P) x = par[x];  // the owner is a rank, so this ends
          if (a.kind != TACCL_REDUCESCATTER) set_pair(bits, x, b, P);
          if (a.kind == TACCL_REDUCESCATTER || a.kind == TACCL_ALLREDUCE)
            set_pair(bits, b, x, P);
        }
      }
    }
    __syncthreads();
    uint32_t cnt = 0;
    for (int w = threadIdx.x; w < MW; w += blockDim.x) cnt += __popc(bits[w]);
    for (int o = 32; o > 0; o >>= 1) cnt += (uint32_t)__shfl_xor((int)cnt, o);
    if ((threadIdx.x & 63) == 0 && cnt) atomicAdd(&total, cnt);
    __syncthreads();
    if (threadIdx.x == 0) a.out[i] = total;
    __syncthreads();
  }
}

// Alltoall plans whose routes form at most two switched pairs each (every
// one-switch-per-machine sketch): a.lanes lanes per candidate, no block
// barrier after the tables are in place. The walk along the path is done at
// plan time: a route choice gives one word with its pairs' cells of the
// candidate's P x P byte matrix, so a chunk costs one table read and two
// byte stores (plain stores of 1: a cell needs no atomic), and a route
// option without a second pair stores to a cell past the matrix. Bound by
// LDS: 12 accesses per lane and route word. switch16 (240 pairs, 65536
// candidates): 143 us on the block kernel above, 18 us here.
// kOne: one route word per lane, so the chunk table stays in registers.
template <bool kOne, bool kRecLds, bool kWords>
__global__ __launch_bounds__(kConnWaveThreads) void connections_wave_kernel(ConnArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const uint32_t *rec = a.rec;
  uint32_t off = 0;
  if (kRecLds) {
    uint32_t *r = (uint32_t *)lds;
    for (int j = threadIdx.x; j < a.nrec; j += blockDim.x) r[j] = a.rec[j];
    rec = r;
    off = (4u * (uint32_t)a.nrec + 15u) & ~15u;
  }
  const int G = a.lanes, gl = lane & (G - 1), per_wave = 64 / G;
  const uint32_t fs = (uint32_t)a.cells + 16u;  // the matrix and the cell past it
  uint8_t *flag = lds + off + fs * (uint32_t)(wave * per_wave + lane / G);
  uint4 *flag4 = (uint4 *)flag;
  const int nf = a.cells / 16;
  for (int w = gl; w < nf; w += G) flag4[w] = make_uint4(0u, 0u, 0u, 0u);
  const int64_t stride = (int64_t)gridDim.x * nw * per_wave;
  const int64_t first = ((int64_t)blockIdx.x * nw + wave) * per_wave + lane / G;
  // route word w of candidate i (past the batch: the last candidate again,
  // past the row: the last chunks, both unused)
  auto route_word = [&](int64_t i, int w) -> uint32_t {
    const uint8_t *row = a.routes + (size_t)min(i, a.n - 1) * a.route_stride;
    if (kWords) return ((const uint32_t *)row)[min(w, a.nwords - 1)];
    uint32_t x = 0;
#pragma unroll
    for (int b = 0; b < 4; b++) x |= (uint32_t)row[min(4 * w + b, a.C - 1)] << (8 * b);
    return x;
  };
  auto mark = [&](uint32_t word, const uint4 &ci) {
    const uint32_t cs[4] = {ci.x, ci.y, ci.z, ci.w};
    uint32_t r[4];
#pragma unroll
    for (int b = 0; b < 4; b++) {
      const uint32_t k = (word >> (8 * b)) & 0xFFu;
      r[b] = rec[k < (cs[b] >> 24) ? (cs[b] & 0xFFFFFFu) + k : 0u];
    }
#pragma unroll
    for (int b = 0; b < 4; b++) {
      flag[r[b] & 0xFFFFu] = 1;
      flag[r[b] >> 16] = 1;
    }
  };
  const uint4 none = make_uint4(0u, 0u, 0u, 0u);
  const uint4 own = kOne && gl < a.nwords ? a.chunk[gl] : none;
  uint32_t next = kOne ? route_word(first, gl) : 0u;
  if (kRecLds) __syncthreads();
  // every lane of a wavefront takes the same number of rounds; a group past
  // the batch works on the last candidate and writes nothing
  const int64_t wfirst = ((int64_t)blockIdx.x * nw + wave) * per_wave;
  for (int64_t w0 = wfirst; w0 < a.n; w0 += stride) {
    const int64_t i = w0 + lane / G;
    if (kOne) {
      const uint32_t word = next;
      next = route_word(i + stride, gl);
      mark(word, own);
    } else {
      for (int w = gl; w < a.nwords; w += G) mark(route_word(i, w), a.chunk[w]);
    }
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");  // one wavefront's LDS accesses are in order
    uint32_t cnt = 0;
    for (int w = gl; w < nf; w += G) {
      const uint4 x = flag4[w];
      flag4[w] = none;
      cnt += __popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w);
    }
    for (int o = G >> 1; o > 0; o >>= 1) cnt += (uint32_t)__shfl_xor((int)cnt, o);
    if (gl == 0 && i < a.n) a.out[i] = cnt;
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
  }
}

template <bool kOne, bool kRecLds>
const void *conn_wave_fn_or(bool words) {
  return words ? (const void *)connections_wave_kernel<kOne, kRecLds, true>
               : (const void *)connections_wave_kernel<kOne, kRecLds, false>;
}

}  // namespace

int32_t connections_wave_lds_bytes(const ConnArgs &a, int waves) {
  const int64_t b = (a.rec_lds ? (4 * (int64_t)a.nrec + 15) / 16 * 16 : 0) +
                    (int64_t)waves * (64 / a.lanes) * (a.cells + 16);
  return (int32_t)std::min<int64_t>(b, INT32_MAX);
}

hipError_t launch_connections_wave(const ConnArgs &a, int waves, int grid, hipStream_t stream) {
  if (waves < 1 || waves > kConnWaveThreads / 64 || a.cells % 16 || a.lanes < 1 || a.lanes > 64 ||
      (a.lanes & (a.lanes - 1)))
    return hipErrorInvalidValue;
  const bool one = a.nwords <= a.lanes, words = a.routes_words != 0;
  const void *fn = one ? (a.rec_lds ? conn_wave_fn_or<true, true>(words)
                                    : conn_wave_fn_or<true, false>(words))
                       : (a.rec_lds ? conn_wave_fn_or<false, true>(words)
                                    : conn_wave_fn_or<false, false>(words));
  void *args[] = {(void *)&a};
  return hipLaunchKernel(fn, dim3(grid), dim3(64 * waves), args,
                         connections_wave_lds_bytes(a, waves), stream);
}

int32_t connections_lds_bytes(const ConnArgs &a, int threads) {
  return 4 * a.mask_words + (a.tree ? threads * a.V : 0);
}

hipError_t launch_connections(const ConnArgs &a, int threads, int grid, hipStream_t stream) {
  if (threads < 64 || threads > kConnMaxThreads || threads % 64) return hipErrorInvalidValue;
  const void *fn = a.tree ? (const void *)connections_kernel<true>
                          : (const void *)connections_kernel<false>;
  void *args[] = {(void *)&a};
  return hipLaunchKernel(fn, dim3(grid), dim3(threads), args, connections_lds_bytes(a, threads),
                         stream);
}

}  // namespace taccl
