// Flat proximity graph on the GPU: the k nearest other points of every
// point (the exact kNN kernels with k + 1 and the point itself dropped),
// symmetrization by two stable radix sorts of the 2nk directed edges (by
// target, then by (source, distance)), HNSW's neighbour-selection heuristic
// for rows longer than the degree cap (one wavefront per row), and the
// pieces of the reachability repair.
//
// The repair visits the unreached nodes in id order; what each step reaches
// depends on the pruned graph only (the edges it adds lead to nodes already
// reached), so all steps are known at once: a node is first reached from the
// smallest id that leads to it (the entry counting as smallest), and the
// steps' start nodes are the nodes that no smaller id leads to.  That label
// comes from propagating minima along the edges; the nearest reached nodes
// of all start nodes then come from one kNN call restricted to smaller
// labels, and the host only walks the short lists to keep track of the free
// slots.  Where a list does not settle which node is nearest (candidate
// scores or distances too close for their rounding, or no free slot left in
// it) all nodes are searched for that step.  Step by step on the host (a
// search of the whole set and a breadth-first walk each, several round trips)
// took 42 ms for the 100 components of a 100,000 x 128 mixture; this takes
// 1.2 ms.
//
// Edge e of the 2nk directed edges: e < nk is the kNN edge (e / k -> ids[e])
// and e >= nk the reverse of kNN edge e - nk.  Both carry the kNN list's
// distance, a float32 sum of squared differences whose value does not depend
// on the direction, so a pair listed from both ends sorts into adjacent
// equal entries and the duplicate is dropped.
#include <hipcub/hipcub.hpp>

#include <algorithm>

#include "device_common.h"
#include "internal.h"

namespace finger {
namespace {

struct Edge {
  uint32_t src, dst;
  float d;
};

__device__ __forceinline__ Edge edge_of(uint32_t e, int64_t nk, int k, const int32_t* ids,
                                        const float* dk) {
  Edge r;
  if ((int64_t)e < nk) {
    r.src = e / (uint32_t)k;
    r.dst = (uint32_t)ids[e];
    r.d = dk[e];
  } else {
    const uint32_t f = e - (uint32_t)nk;
    r.src = (uint32_t)ids[f];
    r.dst = f / (uint32_t)k;
    r.d = dk[f];
  }
  return r;
}

// row i of a query batch starting at point `first`
__global__ void k_drop_self(const int32_t* ids1, const float* d1, int64_t n, int k1, int k,
                            int32_t* ids, float* dk, int64_t first, int64_t id_offset) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int o = 0;
  for (int t = 0; t < k1 && o < k; ++t) {
    const int32_t v = ids1[i * k1 + t];
    if (v == (int32_t)(first + i)) continue;
    ids[i * k + o] = (int32_t)(v + id_offset);
    dk[i * k + o] = d1[i * k1 + t];
    ++o;
  }
}

__global__ void k_keys_dst(int64_t ne, int64_t nk, int k, const int32_t* ids, const float* dk,
                           uint32_t* keys, uint32_t* vals) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= ne) return;
  keys[e] = edge_of((uint32_t)e, nk, k, ids, dk).dst;
  vals[e] = (uint32_t)e;
}

__global__ void k_keys_src_d(int64_t ne, int64_t nk, int k, const int32_t* ids, const float* dk,
                             const uint32_t* perm, uint64_t* keys) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= ne) return;
  const Edge g = edge_of(perm[x], nk, k, ids, dk);
  keys[x] = ((uint64_t)g.src << 32) | order_bits(g.d);
}

// flag[x] = 1 unless sorted edge x repeats the (source, target) of x - 1;
// cnt[source] counts the kept edges of each row
__global__ void k_dedupe(int64_t ne, int64_t nk, int k, const int32_t* ids, const float* dk,
                         const uint32_t* perm, uint32_t* flag, uint32_t* cnt) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= ne) return;
  const Edge g = edge_of(perm[x], nk, k, ids, dk);
  uint32_t f = 1;
  if (x > 0) {
    const Edge p = edge_of(perm[x - 1], nk, k, ids, dk);
    f = (p.src != g.src || p.dst != g.dst) ? 1u : 0u;
  }
  flag[x] = f;
  if (f) atomicAdd(&cnt[g.src], 1u);
}

__global__ void k_fill_rows(int64_t ne, int64_t nk, int k, const int32_t* ids, const float* dk,
                            const uint32_t* perm, const uint32_t* flag, const uint32_t* pos,
                            int32_t* nbr, float* nd) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= ne || flag[x] == 0) return;
  const Edge g = edge_of(perm[x], nk, k, ids, dk);
  nbr[pos[x]] = (int32_t)g.dst;
  nd[pos[x]] = g.d;
}

template <int G, int T4>
__device__ __forceinline__ void load_vec(const float4* data, int m4, int id, int lg, bool valid,
                                         float4 (&v)[T4]) {
  const float4* row = data + (int64_t)(valid ? id : 0) * m4;
#pragma unroll
  for (int t = 0; t < T4; ++t) {
    const int j = lg + G * t;
    v[t] = (valid && j < m4) ? row[j] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// (fused multiply-adds written out: the same bits in every kernel)
template <int G, int T4>
__device__ __forceinline__ float sq_dist(const float4 (&a)[T4], const float4 (&b)[T4]) {
  float acc = 0.f;
#pragma unroll
  for (int t = 0; t < T4; ++t) {
    const float dx = a[t].x - b[t].x, dy = a[t].y - b[t].y;
    const float dz = a[t].z - b[t].z, dw = a[t].w - b[t].w;
    const float s = __builtin_fmaf(dw, dw, __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx)));
    acc = t == 0 ? s : acc + s;
  }
  return group_sum<G>(acc);
}

// One wavefront per row.  Short rows are copied; a long row is scanned in
// (distance, id) order and a candidate kept iff fewer than W are kept and it
// is strictly closer to the base than to every kept neighbour.  Lane t holds
// the t-th kept id.
template <int G, int T4>
__global__ __launch_bounds__(256) void k_prune(const float4* data, int64_t n, int m4,
                                               const uint32_t* indptr, const int32_t* nbr,
                                               const float* nd, int W, int32_t* out) {
  constexpr int NPAR = 64 / G;
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
  if (i >= n) return;
  const int lg = lane % G, grp = lane / G;
  const uint32_t off = indptr[i];
  const int deg = (int)(indptr[i + 1] - off);
  int32_t* row = out + i * W;
  if (deg <= W) {
    for (int t = lane; t < W; t += 64) row[t] = t < deg ? nbr[off + t] : -1;
    return;
  }
  int kept = -1;
  int kc = 0;
  for (int c = 0; c < deg && kc < W; ++c) {
    const int id = uniform_i(nbr[off + c]);
    const float dc = uniform_f(nd[off + c]);
    float4 xc[T4];
    load_vec<G, T4>(data, m4, id, lg, true, xc);
    bool reject = false;
    for (int p0 = 0; p0 < kc && !reject; p0 += NPAR) {
      const int t = p0 + grp;
      const bool valid = t < kc;
      const int kid = shfl_i(kept, valid ? t : 0);
      float4 xt[T4];
      load_vec<G, T4>(data, m4, kid, lg, valid, xt);
      const float dd = sq_dist<G, T4>(xc, xt);
      reject = ballot(valid && !(dc < dd)) != 0;
    }
    if (!reject) {
      if (lane == kc) kept = id;
      ++kc;
    }
  }
  for (int t = lane; t < W; t += 64) row[t] = t < kc ? kept : -1;
}

__global__ void k_degrees(const int32_t* G, int64_t n, int W, int32_t* deg) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int d = 0;
  for (int t = 0; t < W; ++t) d += G[i * W + t] >= 0 ? 1 : 0;
  deg[i] = d;
}

// label[v]: 0 for the entry, else v + 1 (before propagation)
__global__ void k_label_init(int64_t n, int entry, uint32_t* label, uint32_t* stamp) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  label[i] = i == entry ? 0u : (uint32_t)i + 1u;
  stamp[i] = 0u;
}

// One sweep: every node of the frontier (NULL: all nodes) hands its label to
// its out-neighbours; those it lowers form the next frontier.  counts[sweep]
// is this frontier's size, counts[sweep + 1] (zeroed by the host) the next
// one's; an empty frontier ends the kernel at once.  One thread per edge slot;
// the grid is fixed, the size being known on the device only.  Labels above
// `limit` stay where they are.
__global__ void k_label_sweep(const int32_t* G, int64_t n, int W, const int32_t* frontier, uint32_t* counts, int sweep,
                              uint32_t epoch, uint32_t limit, uint32_t* label, uint32_t* stamp, int32_t* next) {
  const int64_t items = (frontier == nullptr ? n : (int64_t)counts[sweep]) * W;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < items;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t f = frontier == nullptr ? i / W : frontier[i / W];
    const int32_t v = G[f * W + i % W];
    if (v < 0) continue;
    const uint32_t lf = __hip_atomic_load(&label[f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lf > limit || lf >= __hip_atomic_load(&label[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) continue;
    if (atomicMin(&label[v], lf) > lf && atomicExch(&stamp[v], epoch) != epoch)
      next[atomicAdd(&counts[sweep + 1], 1u)] = v;
  }
}

// lowest label of the listed nodes
__global__ void __launch_bounds__(256) k_lowest_label(const int32_t* nodes, int64_t cnt, const uint32_t* label,
                                                      uint32_t* lowest) {
  uint32_t lo = ~0u;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < cnt; i += (int64_t)gridDim.x * 256)
    lo = min(lo, label[nodes[i]]);
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
  if ((threadIdx.x & 63) == 0) atomicMin(lowest, lo);
}

__global__ void k_root_flags(int64_t n, const uint32_t* label, const int32_t* deg, int W, uint32_t* flag,
                             uint32_t* free_label) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  flag[i] = label[i] == (uint32_t)i + 1u ? 1u : 0u;
  free_label[i] = deg[i] < W ? label[i] : ~0u;  // ~0: no free slot, below no label
}

__global__ void k_root_list(int64_t n, const uint32_t* flag, const uint32_t* pos, int32_t* roots) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && flag[i] != 0u) roots[pos[i]] = (int32_t)i;
}

// dist[r][c]: the distance of candidate c to start node r as k_nearest_free
// has it (one wave per start node; infinity where the list has ended)
template <int G, int T4>
__global__ __launch_bounds__(256) void k_repair_dists(const float4* data, int m4, const int32_t* roots, int64_t cnt,
                                                      const int32_t* cand, int J, float* dist) {
  constexpr int NPAR = 64 / G;
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= cnt) return;
  const int lg = lane % G, grp = lane / G;
  float4 xu[T4];
  load_vec<G, T4>(data, m4, roots[r], lg, true, xu);
  for (int c0 = 0; c0 < J; c0 += NPAR) {
    const int c = c0 + grp;
    const int id = c < J ? cand[r * J + c] : -1;
    float4 xv[T4];
    load_vec<G, T4>(data, m4, id, lg, id >= 0, xv);
    const float d = sq_dist<G, T4>(xu, xv);
    if (c < J && lg == 0) dist[r * J + c] = id >= 0 ? d : __int_as_float(0x7f800000);
  }
}

// per start node: its row, its degree, the candidates, their degrees and
// distances, the kNN's last distance, its score bound and |q|^2 (floats as
// bits)
__global__ void k_repair_gather(const int32_t* G, int W, const int32_t* deg, const int32_t* roots, int64_t cnt,
                                const int32_t* cand, const float* dist, const float* knn_dist, const float2* bound,
                                int J, int32_t* out) {
  const int per = W + 4 + 3 * J;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= cnt * per) return;
  const int64_t r = i / per;
  int c = (int)(i % per);
  const int32_t u = roots[r];
  int32_t v;
  if (c < W) v = G[(int64_t)u * W + c];
  else if (c == W) v = deg[u];
  else if ((c -= W + 1) < J) v = cand[r * J + c];
  else if ((c -= J) < J) {
    const int32_t id = cand[r * J + c];
    v = id >= 0 ? deg[id] : 0;
  } else if ((c -= J) < J) v = __float_as_int(dist[r * J + c]);
  else v = __float_as_int(c == J ? knn_dist[r * J + J - 1] : c == J + 1 ? bound[r].x : bound[r].y);
  out[i] = v;
}

__global__ void k_scatter_i32(const int64_t* at, const int32_t* val, int64_t cnt, int32_t* dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) dst[at[i]] = val[i];
}

// smallest (squared distance to u, id) over the nodes with a smaller label
// and a free slot (when a start node's short list holds none any more, or
// does not settle which is nearest)
template <int G, int T4>
__global__ __launch_bounds__(256) void k_nearest_free(const float4* data, int64_t n, int m4, int u,
                                                      const uint32_t* label, const int32_t* deg,
                                                      int W, unsigned long long* best) {
  constexpr int NPAR = 64 / G;
  __shared__ uint64_t red[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lg = lane % G, grp = lane / G;
  float4 xu[T4];
  load_vec<G, T4>(data, m4, u, lg, true, xu);
  uint64_t mine = ~0ull;
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x / 64);
  for (int64_t b = ((int64_t)blockIdx.x * (blockDim.x / 64) + w) * NPAR; b < n; b += waves * NPAR) {
    const int64_t v = b + grp;
    const bool ok = v < n && label[v] < (uint32_t)u + 1u && deg[v] < W;
    float4 xv[T4];
    load_vec<G, T4>(data, m4, (int)v, lg, ok, xv);
    const float d = sq_dist<G, T4>(xu, xv);
    if (ok) {
      const uint64_t key = make_key(d, (int)v);
      mine = key < mine ? key : mine;
    }
  }
  if constexpr (G < 64) { const uint64_t o = shfl_xor_u64(mine, G); mine = o < mine ? o : mine; }
  if constexpr (G < 32) { const uint64_t o = shfl_xor_u64(mine, 2 * G); mine = o < mine ? o : mine; }
  if (lane == 0) red[w] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t b = red[0];
    for (int t = 1; t < (int)(blockDim.x / 64); ++t) b = red[t] < b ? red[t] : b;
    if (b != ~0ull) atomicMin(best, (unsigned long long)b);
  }
}

// lanes per vector and float4 per lane by vector length (the shape fixes the
// order of a distance's sum)
#define FINGER_BY_LENGTH(m4, LAUNCH)  \
  if (m4 <= 16) LAUNCH(16, 1);        \
  else if (m4 <= 32) LAUNCH(16, 2);   \
  else if (m4 <= 64) LAUNCH(16, 4);   \
  else if (m4 <= 128) LAUNCH(16, 8);  \
  else if (m4 <= 256) LAUNCH(64, 4);  \
  else LAUNCH(64, 8);

inline unsigned blocks_for(int64_t n, int per = 256) { return (unsigned)((n + per - 1) / per); }

}  // namespace

hipError_t launch_drop_self(const int32_t* ids1, const float* d1, int64_t n, int k1, int k,
                            int32_t* ids, float* dk, int64_t first, int64_t id_offset, hipStream_t s) {
  hipLaunchKernelGGL(k_drop_self, dim3(blocks_for(n)), dim3(256), 0, s, ids1, d1, n, k1, k, ids, dk,
                     first, id_offset);
  return hipGetLastError();
}

hipError_t launch_sym_keys_dst(int64_t n, int k, const int32_t* ids, const float* dk, uint32_t* keys,
                               uint32_t* vals, hipStream_t s) {
  const int64_t nk = n * k, ne = 2 * nk;
  hipLaunchKernelGGL(k_keys_dst, dim3(blocks_for(ne)), dim3(256), 0, s, ne, nk, k, ids, dk, keys, vals);
  return hipGetLastError();
}

hipError_t launch_sym_keys_src_d(int64_t n, int k, const int32_t* ids, const float* dk,
                                 const uint32_t* perm, uint64_t* keys, hipStream_t s) {
  const int64_t nk = n * k, ne = 2 * nk;
  hipLaunchKernelGGL(k_keys_src_d, dim3(blocks_for(ne)), dim3(256), 0, s, ne, nk, k, ids, dk, perm, keys);
  return hipGetLastError();
}

hipError_t launch_sym_dedupe(int64_t n, int k, const int32_t* ids, const float* dk,
                             const uint32_t* perm, uint32_t* flag, uint32_t* cnt, hipStream_t s) {
  const int64_t nk = n * k, ne = 2 * nk;
  hipLaunchKernelGGL(k_dedupe, dim3(blocks_for(ne)), dim3(256), 0, s, ne, nk, k, ids, dk, perm, flag, cnt);
  return hipGetLastError();
}

hipError_t launch_sym_fill(int64_t n, int k, const int32_t* ids, const float* dk, const uint32_t* perm,
                           const uint32_t* flag, const uint32_t* pos, int32_t* nbr, float* nd,
                           hipStream_t s) {
  const int64_t nk = n * k, ne = 2 * nk;
  hipLaunchKernelGGL(k_fill_rows, dim3(blocks_for(ne)), dim3(256), 0, s, ne, nk, k, ids, dk, perm,
                     flag, pos, nbr, nd);
  return hipGetLastError();
}

hipError_t radix_sort_u32(void* tmp, size_t& tmp_bytes, const uint32_t* kin, uint32_t* kout,
                          const uint32_t* vin, uint32_t* vout, int64_t count, int end_bit, hipStream_t s) {
  return hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, kin, kout, vin, vout, (int)count, 0,
                                            end_bit, s);
}

hipError_t radix_sort_u64(void* tmp, size_t& tmp_bytes, const uint64_t* kin, uint64_t* kout,
                          const uint32_t* vin, uint32_t* vout, int64_t count, int end_bit, hipStream_t s) {
  return hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, kin, kout, vin, vout, (int)count, 0,
                                            end_bit, s);
}

hipError_t exclusive_sum_u32(void* tmp, size_t& tmp_bytes, const uint32_t* in, uint32_t* out,
                             int64_t count, hipStream_t s) {
  return hipcub::DeviceScan::ExclusiveSum(tmp, tmp_bytes, in, out, (int)count, s);
}

hipError_t launch_prune(const float* data, int64_t n, int m, const uint32_t* indptr,
                        const int32_t* nbr, const float* nd, int W, int32_t* out, hipStream_t s) {
  const float4* d4 = reinterpret_cast<const float4*>(data);
  const int m4 = m / 4;
  const dim3 grid(blocks_for(n, 4)), block(256);
#define FINGER_PRUNE(G_, T_) hipLaunchKernelGGL((k_prune<G_, T_>), grid, block, 0, s, d4, n, m4, indptr, nbr, nd, W, out)
  FINGER_BY_LENGTH(m4, FINGER_PRUNE)
#undef FINGER_PRUNE
  return hipGetLastError();
}

hipError_t launch_degrees(const int32_t* G, int64_t n, int W, int32_t* deg, hipStream_t s) {
  hipLaunchKernelGGL(k_degrees, dim3(blocks_for(n)), dim3(256), 0, s, G, n, W, deg);
  return hipGetLastError();
}

hipError_t launch_label_init(int64_t n, int entry, uint32_t* label, uint32_t* stamp, hipStream_t s) {
  hipLaunchKernelGGL(k_label_init, dim3(blocks_for(n)), dim3(256), 0, s, n, entry, label, stamp);
  return hipGetLastError();
}

hipError_t launch_label_sweep(const int32_t* G, int64_t n, int W, const int32_t* frontier, uint32_t* counts, int sweep,
                              uint32_t epoch, uint32_t limit, uint32_t* label, uint32_t* stamp, int32_t* next,
                              hipStream_t s) {
  const unsigned grid = std::min(blocks_for(n * W), 4096u);
  hipLaunchKernelGGL(k_label_sweep, dim3(grid), dim3(256), 0, s, G, n, W, frontier, counts, sweep, epoch, limit, label,
                     stamp, next);
  return hipGetLastError();
}

hipError_t launch_lowest_label(const int32_t* nodes, int64_t cnt, const uint32_t* label, uint32_t* lowest,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_lowest_label, dim3(std::min(blocks_for(cnt), 1024u)), dim3(256), 0, s, nodes, cnt, label, lowest);
  return hipGetLastError();
}

hipError_t launch_root_flags(int64_t n, const uint32_t* label, const int32_t* deg, int W, uint32_t* flag,
                             uint32_t* free_label, hipStream_t s) {
  hipLaunchKernelGGL(k_root_flags, dim3(blocks_for(n)), dim3(256), 0, s, n, label, deg, W, flag, free_label);
  return hipGetLastError();
}

hipError_t launch_root_list(int64_t n, const uint32_t* flag, const uint32_t* pos, int32_t* roots, hipStream_t s) {
  hipLaunchKernelGGL(k_root_list, dim3(blocks_for(n)), dim3(256), 0, s, n, flag, pos, roots);
  return hipGetLastError();
}

hipError_t launch_repair_gather(const float* data, int m, const int32_t* G, int W, const int32_t* deg,
                                const int32_t* roots, int64_t cnt, const int32_t* cand, const float* knn_dist,
                                const float2* bound, int J, float* dist, int32_t* out, hipStream_t s) {
  if (cnt == 0) return hipSuccess;
  const float4* d4 = reinterpret_cast<const float4*>(data);
  const int m4 = m / 4;
  const dim3 grid(blocks_for(cnt, 4)), block(256);
#define FINGER_RDIST(G_, T_) hipLaunchKernelGGL((k_repair_dists<G_, T_>), grid, block, 0, s, d4, m4, roots, cnt, cand, J, dist)
  FINGER_BY_LENGTH(m4, FINGER_RDIST)
#undef FINGER_RDIST
  hipLaunchKernelGGL(k_repair_gather, dim3(blocks_for(cnt * (W + 4 + 3 * J))), dim3(256), 0, s, G, W, deg, roots, cnt,
                     cand, dist, knn_dist, bound, J, out);
  return hipGetLastError();
}

hipError_t launch_scatter_i32(const int64_t* at, const int32_t* val, int64_t cnt, int32_t* dst, hipStream_t s) {
  if (cnt == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_i32, dim3(blocks_for(cnt)), dim3(256), 0, s, at, val, cnt, dst);
  return hipGetLastError();
}

hipError_t launch_nearest_free(const float* data, int64_t n, int m, int u, const uint32_t* label,
                               const int32_t* deg, int W, unsigned long long* best, hipStream_t s) {
  const float4* d4 = reinterpret_cast<const float4*>(data);
  const int m4 = m / 4;
  const dim3 grid((unsigned)std::min<int64_t>(4096, (n + 15) / 16)), block(256);
#define FINGER_NEAR(G_, T_) hipLaunchKernelGGL((k_nearest_free<G_, T_>), grid, block, 0, s, d4, n, m4, u, label, deg, W, best)
  FINGER_BY_LENGTH(m4, FINGER_NEAR)
#undef FINGER_NEAR
  return hipGetLastError();
}

}  // namespace finger
