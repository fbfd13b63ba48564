// Launch rules of the graph search (the kernel is in search_kernel.h), the ef
// classes of a search with per-query K and ef, and the estimate of single
// edges.
#include "search_kernel.h"

namespace finger {

namespace {

int wave_bytes(int ef_max, int vis_cap, int r, int m, int gate_in) {
  const int rpad = rpad_of(r);
  int b = ((8 * ef_max + 15) & ~15) + 4 * vis_cap + 64 * 4 * 2 + 8 * rpad + (r > 0 ? 4 * m : 0);
  if (gate_in > 0) {
    // edge features [32][k1] and hidden activations [32][k2] in bf16, outputs [32]
    const GateLayout GL = gate_layout(r, 64);
    b += 2 * 32 * (GL.k1 + GL.k2) + 4 * 32;
  }
  return (b + 15) & ~15;
}

void fill_common(KArgs& a, const Tables& t) {
  a.ip = t.metric == FINGER_IP ? 1 : 0;
  a.data = t.data;
  a.graph = t.graph;
  a.n = t.n;
  a.m = t.m;
  a.m4 = t.m / 4;
  a.deg = t.deg;
  a.r = t.r;
  a.rpad = rpad_of(t.r);
  a.cpr = a.rpad > 0 ? a.rpad / chunk_elems_rt(t.code_type) : 1;
  a.spp = 64 / a.cpr;
  a.cc = t.cc;
  a.pc = t.pc;
  a.alpha = t.alpha;
  a.rho = t.rho;
  a.codes = t.codes;
  a.scale = t.scale;
  a.mu = (float)t.mu;
  a.dm_scale = (float)(t.sigma_hat > 0 ? t.sigma / t.sigma_hat : 1.0);
  a.mu_hat = (float)t.mu_hat;
  a.eps = (float)t.eps;
}

}  // namespace

int search_lds_bytes(int ef_max, int vis_cap, int r, int m, int gate_in) {
  return wave_bytes(ef_max, vis_cap, r, m, gate_in);
}

bool search_prefetch_supported(const Tables& t) {
  // the first screening pass covers every slot, so all codes can be issued
  // with the adjacency row
  return t.r > 0 && t.deg <= 64 / (rpad_of(t.r) / chunk_elems_rt(t.code_type));
}

hipError_t launch_search(const Tables& t, const SearchLaunch& L, hipStream_t s) {
  KArgs a{};
  fill_common(a, t);
  a.queries = L.queries;
  a.nq = L.nq;
  a.qq = L.qq;
  a.pq = L.pq;
  a.entries = L.entries;
  a.entry = L.entry;
  a.kq = L.kq;
  a.efq = L.efq;
  a.k_all = L.k_all;
  a.ef_all = L.ef_all;
  a.k_max = L.k_max;
  a.ef_max = L.ef_max;
  a.warmup = L.warmup;
  a.out_ids = L.out_ids;
  a.out_dist = L.out_dist;
  a.counters = L.counters;
  a.queue = L.queue;
  a.persistent = L.persistent;
  a.qlist = L.qlist;
  a.qcount = L.qcount;
  a.nclass = L.nclass;
  a.list_stride = L.list_stride;
  a.spill = L.spill;
  a.spill_slots = L.spill_slots_per_wave;
  a.vis_cap = L.vis_cap;
  a.vis_buckets = L.vis_probe / 4;
  // the tag table where an id's bits past the bucket's fit sixteen: up to
  // 2^16 ids per bucket of 32 bytes (16M points with the default 8 KB)
  {
    int id_bits = 1, bucket_bits = 0;
    while (((int64_t)1 << id_bits) < t.n) ++id_bits;
    while ((kTagBucketWords << (bucket_bits + 1)) <= L.vis_cap) ++bucket_bits;
    const int tag_bits = id_bits > bucket_bits ? id_bits - bucket_bits : 0;
    a.vis_id_mask = id_bits >= 32 ? ~0u : (1u << id_bits) - 1u;
    a.vis_mul = (uint32_t)(0.6180339887498949 * (double)((uint64_t)1 << id_bits)) | 1u;
    a.vis_tag_bits = tag_bits <= 16 ? tag_bits : -1;
  }
  a.log_x = L.log_x;
  a.log_y = L.log_y;
  a.log_cap = L.log_cap;
  a.log_count = L.log_count;
  const bool gated = L.mode == FINGER_MODE_GATED;
  a.gate_w = gated ? t.gate_w : nullptr;
  a.gate_b = gated ? t.gate_b : nullptr;
  a.gate_in = gated ? t.gate_in : 0;
  a.gate_h = gated ? t.gate_h : 0;
  a.eps_gate = (float)t.eps_gate;
  a.gate_band = L.gate_band;
  // one query wave per workgroup keeps LDS allocation fine grained
  a.waves_per_block = 1;
  a.cus = L.cus;
  a.fit_grid = L.fit_grid;
  a.coalesced = L.coalesced;
  a.lds_shared_bytes = 0;
  a.lds_wave_bytes = wave_bytes(L.ef_max, L.vis_cap, L.mode == FINGER_MODE_PLAIN ? 0 : t.r, t.m,
                                gated ? a.gate_in : 0);
  const int lds = a.lds_shared_bytes + a.waves_per_block * a.lds_wave_bytes;
  const int blocks = (L.waves + a.waves_per_block - 1) / a.waves_per_block;
  const bool pf = L.prefetch && search_prefetch_supported(t);
  if (L.mode == FINGER_MODE_PLAIN) return search_plain(a, blocks, lds, s);
  if (L.mode == FINGER_MODE_GATED) return search_gated(a, t.code_type, blocks, lds, s);
  if (L.log_x != nullptr) return search_log(a, t.code_type, pf, blocks, lds, s);
  if (t.code_type == FINGER_CODE_BF16) return search_bf16(a, pf, blocks, lds, s);
  if (t.code_type == FINGER_CODE_FP8E4M3) return search_fp8(a, pf, blocks, lds, s);
  return search_f32(a, pf, blocks, lds, s);
}

// ------------------------------------------------------ ef classes

namespace {

// One block: every query's class (the first bound >= its ef_eff = max(ef,
// K), the last class for anything above), appended to that class's list
// lists[c nq ..] (order inside a class is not fixed: a query's search does
// not depend on the others); counts[c] and the lists drive the per-class
// launches.
__global__ void __launch_bounds__(1024) k_ef_classes(const int32_t* __restrict__ kq,
                                                     const int32_t* __restrict__ efq, int64_t nq,
                                                     int k_all, int ef_all, ClassBounds cb,
                                                     int32_t* __restrict__ counts,
                                                     int32_t* __restrict__ lists) {
  __shared__ int cnt[kMaxEfClasses];
  const int t = threadIdx.x;
  if (t < kMaxEfClasses) cnt[t] = 0;
  __syncthreads();
  for (int64_t i = t; i < nq; i += blockDim.x) {
    const int k = kq ? kq[i] : k_all;
    const int ef = efq ? efq[i] : ef_all;
    const int e = ef > k ? ef : k;
    int c = 0;
    while (c + 1 < cb.n && e > cb.bound[c]) ++c;
    lists[(int64_t)c * nq + atomicAdd(&cnt[c], 1)] = (int32_t)i;
  }
  __syncthreads();
  if (t < cb.n) counts[t] = cnt[t];
}

}  // namespace

hipError_t launch_ef_classes(const int32_t* kq, const int32_t* efq, int64_t nq, int k_all, int ef_all,
                             const ClassBounds& cb, int32_t* counts, int32_t* lists, hipStream_t s) {
  hipLaunchKernelGGL(k_ef_classes, dim3(1), dim3(1024), 0, s, kq, efq, nq, k_all, ef_all, cb, counts, lists);
  return hipGetLastError();
}

// ------------------------------------------------- estimate test kernel

namespace {
// One wave per (query, centre, slot) item, computing exactly what the
// search's screening step computes for that edge.
template <int CODE>
__global__ void k_estimate_edges(KArgs a, const int32_t* qi, const int32_t* ci,
                                 const int32_t* si, int64_t items, float* est, float* that) {
  extern __shared__ __align__(16) float wsm[];
  const int64_t item = (int64_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
  float* wv = wsm + (threadIdx.x / 64) * a.rpad;
  if (item >= items) return;
  const int l = lane_id();
  const int q = qi[item], c = ci[item], slot = si[item];
  // the exact d2(q, c) the search has in T
  const float4* q4 = reinterpret_cast<const float4*>(a.queries + (int64_t)q * a.m);
  const float4* c4 = reinterpret_cast<const float4*>(a.data + (int64_t)c * a.m);
  float acc = 0.f;
  for (int j = l; j < a.m4; j += 64) {
    const float4 x = q4[j], y = c4[j];
    if (a.ip) {
      acc -= x.x * y.x + x.y * y.y + x.z * y.z + x.w * y.w;
    } else {
      const float dx = x.x - y.x, dy = x.y - y.y, dz = x.z - y.z, dw = x.w - y.w;
      acc += dx * dx + dy * dy + dz * dz + dw * dw;
    }
  }
  const float dcur = wave_sum(acc);
  const float qq = a.qq[q];
  const float ccv = a.cc[c];
  const float qc = a.ip ? -dcur : 0.5f * (qq + ccv - dcur);
  const float aq = ccv > 0.f ? qc / ccv : 0.f;
  const float rq2 = fmaxf(qq - aq * qc, 0.f);
  const float rq = sqrtf(rq2);
  float w2 = 0.f;
  for (int e = l; e < a.rpad; e += 64) {
    const float w = a.pq[(int64_t)q * a.rpad + e] - aq * a.pc[(int64_t)c * a.rpad + e];
    wv[e] = w;
    w2 += w * w;
  }
  w2 = wave_sum(w2);
  wave_lds_sync();
  const float inv_w = w2 > 0.f ? 1.0f / sqrtf(w2) : 0.f;
  float dot = 0.f;
  constexpr int kChunk = chunk_elems<CODE>();
  if (l < a.cpr) {
    Chunk<CODE> code;
    code.load(a.codes, ((int64_t)c * a.deg + slot) * a.rpad + l * kChunk);
    dot = code.dot(wv + l * kChunk);
  }
  dot = wave_sum(dot);
  const float scl = (CODE == FINGER_CODE_FP8E4M3) ? a.scale[c] : 1.f;
  const float t_hat = dot * scl * inv_w;
  const float ad = a.alpha[(int64_t)c * a.deg + slot];
  const float rd = a.rho[(int64_t)c * a.deg + slot];
  const float t = (t_hat - a.mu_hat) * a.dm_scale + a.mu + a.eps;
  const float da = aq - ad;
  if (l == 0) {
    est[item] = a.ip ? -(aq * ad * ccv + rq * rd * t) : da * da * ccv + rq2 + rd * rd - 2.f * rq * rd * t;
    that[item] = t_hat;
  }
}
}  // namespace

hipError_t launch_estimate_edges(const Tables& t, const float* Q, const float* qq,
                                 const float* Pq, const int32_t* qi, const int32_t* ci,
                                 const int32_t* si, int64_t items, float* est, float* that,
                                 hipStream_t s) {
  if (items == 0) return hipSuccess;
  KArgs a{};
  fill_common(a, t);
  a.queries = Q;
  a.qq = qq;
  a.pq = Pq;
  const int wpb = 4;
  const int blocks = (int)((items + wpb - 1) / wpb);
  const int lds = wpb * a.rpad * 4;
  if (t.code_type == FINGER_CODE_BF16)
    hipLaunchKernelGGL(k_estimate_edges<FINGER_CODE_BF16>, dim3(blocks), dim3(64 * wpb), lds, s, a,
                       qi, ci, si, items, est, that);
  else if (t.code_type == FINGER_CODE_FP8E4M3)
    hipLaunchKernelGGL(k_estimate_edges<FINGER_CODE_FP8E4M3>, dim3(blocks), dim3(64 * wpb), lds, s,
                       a, qi, ci, si, items, est, that);
  else
    hipLaunchKernelGGL(k_estimate_edges<FINGER_CODE_F32>, dim3(blocks), dim3(64 * wpb), lds, s, a,
                       qi, ci, si, items, est, that);
  return hipGetLastError();
}

}  // namespace finger
