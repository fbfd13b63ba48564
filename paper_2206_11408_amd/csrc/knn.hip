// Brute-force kNN (the recall ground truth of Section 1, and the graph
// build's self-join): candidate scores on the bf16 matrix cores in split
// precision, then an exact float32 re-rank.
//
// Scores.  Each float x is split once per call as hi = bf16(x) and lo =
// bf16(x - hi) (k_knn_split), and q.x ~ hi.hi' + hi.lo' + lo.hi' (the dropped
// lo.lo' term is below 2^-16 of |q||x|), accumulated in float32 by
// v_mfma_f32_16x16x32_bf16.  When every lo of both sides is zero (integers up
// to 256), the two products with lo add nothing and are left out.  The scores
// only choose the KK = k + kKnnSlack candidates that k_knn_final re-ranks by
// exact float32 differences: a true neighbour is lost only if kKnnSlack others
// sit within the score error of it (about 1e-5 of |q||x|).  Integers up to 256
// score exactly while |x|^2 and |q|^2 are below 2^24 (the sums start at
// -|x|^2 / 2 in float32): for any such data up to 256 dimensions; beyond, sums
// of that size are rounded.
//
// Selection.  The points are scanned in phases over growing prefixes of a
// pseudo-random order (position p holds point p a mod n, a near 0.618 n and
// prime to n, so that any run of ids is spread evenly over the order).  The
// first phase keeps every score of a short prefix; each later phase appends
// only scores below the row's bound, the KK-th smallest key so far, and
// k_knn_select then tightens the bound.  Growing by at most kKnnGrowth, a
// phase appends about (kKnnGrowth - 1) KK keys per row, whatever the data's
// distribution, because the rank of a sample's KK-th smallest key depends on
// the order only; a row whose space runs out all the same (an order the data
// was built against) is flagged and searched exactly by k_knn_final.
//
// Measured (integer points, one product): 10,000 queries x 300,000 x 128 in
// 1.48 ms, of which k_knn_scan 1.27 ms at 0.61 PFLOP/s, where sorted lists kept
// in the tile loop, with the split redone for every tile, took 19.5 ms (the
// per-row merges bound it); continuous points 2.55 ms (three products, 0.9
// PFLOP/s); 77 angular queries x 100,003 x 100 with k = 100 in 0.20 ms against
// 5.0 ms (32 blocks, and the candidates re-ranked one after another).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <numeric>

#include "device_common.h"
#include "internal.h"

namespace finger {

namespace {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 b8v __attribute__((ext_vector_type(8)));

constexpr int kKnnSlack = 16;
constexpr int kKnnGrowth = 5;
constexpr int kTileQ = 128;                // query rows of a block's tile
constexpr int kPadX = 128;                 // points are padded to a multiple of this
constexpr int kBK = 32;                    // k extent of one staged slab
constexpr int64_t kRowBatch = 65536;       // query rows whose candidates are held at a time, at most
constexpr int kMaxChunks = 512;

// ------------------------------------------------------------- operands

// Positions first .. first + rows_pad of `src` in split precision, 16 lanes
// per row: hi/lo [rows_pad][kpad] (zero past the data), half the squared norm
// (norm_scale 0.5; 1 for queries, 0 for the inner product) and, with stride
// a > 0, position p taken from point p a mod n, whose id goes to perm[p].  inv != NULL: unit-normalized rows, the
// reciprocal norms written there.  flag (may be NULL) is set if any lo is not
// zero.
__global__ void __launch_bounds__(256) k_knn_split(const float* __restrict__ src, int64_t n, int m, int64_t first,
                                                   int64_t rows_pad, int kpad, int64_t a, float norm_scale, float pad_norm,
                                                   __bf16* __restrict__ hi, __bf16* __restrict__ lo,
                                                   float* __restrict__ norm, int32_t* __restrict__ perm,
                                                   double* __restrict__ inv, uint32_t* __restrict__ flag) {
  const int lg = threadIdx.x & 15;
  const int64_t p = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  if (p >= rows_pad) return;  // (rows_pad is a multiple of 16: whole blocks)
  const int64_t pos = first + p;
  const bool live = pos < n;
  const int64_t id = !live ? 0 : (a > 0 ? (int64_t)(((uint64_t)pos * (uint64_t)a) % (uint64_t)n) : pos);
  const float* x = src + id * m;
  double s = 1.0;
  if (inv != nullptr) {
    // summed in the order of k_normalize_rows (64 partial sums, halved pairwise;
    // a lane here holds four of them), so that a row is scaled by the same
    // bits wherever it is normalized
    double qp[4] = {0.0, 0.0, 0.0, 0.0};
    if (live)
      for (int j = lg; j < m; j += 64)
#pragma unroll
        for (int h = 0; h < 4; ++h)
          if (j + 16 * h < m) {
            const double v = x[j + 16 * h];
            qp[h] += v * v;
          }
    double q = (qp[0] + qp[2]) + (qp[1] + qp[3]);
    for (int o = 8; o >= 1; o >>= 1) q += __shfl_xor(q, o, 64);
    s = q > 0 ? 1.0 / sqrt(q) : 0.0;
    if (lg == 0 && live) inv[id] = s;
  }
  float nrm = 0.f;
  bool any_lo = false;
  for (int j = 8 * lg; j < kpad; j += 128) {
    float v[8];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
      if (live && j + 4 * h < m) t = *reinterpret_cast<const float4*>(x + j + 4 * h);
      v[4 * h] = t.x; v[4 * h + 1] = t.y; v[4 * h + 2] = t.z; v[4 * h + 3] = t.w;
    }
    b8v vh, vl;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float y = inv != nullptr ? (float)(v[e] * s) : v[e];
      nrm += y * y;
      vh[e] = (__bf16)y;
      const float r = y - (float)vh[e];
      any_lo |= !(r == 0.f);
      vl[e] = (__bf16)r;
    }
    *reinterpret_cast<b8v*>(hi + p * kpad + j) = vh;
    *reinterpret_cast<b8v*>(lo + p * kpad + j) = vl;
  }
  nrm = group_sum<16>(nrm);
  if (lg == 0) {
    norm[p] = live ? norm_scale * nrm : pad_norm;
    if (perm != nullptr) perm[pos] = live ? (int32_t)id : -1;
  }
  if (flag != nullptr && ballot(any_lo) != 0ull && (threadIdx.x & 63) == 0 && *flag == 0u) *flag = 1u;
}

// ---------------------------------------------------------------- scores

struct ScanArgs {
  // indexed by query row and position; only this batch's rows and this
  // window's positions are there
  const __bf16 *qh, *ql;    // [q_pad][kpad]
  const __bf16 *xh, *xl;    // [n_pad][kpad]
  const float* qn;          // [q_pad] |q|^2 (0 for the inner product)
  const float* hx;          // [n_pad] |x|^2 / 2 (0; +inf past n)
  const int32_t* perm;      // [n_pad] point of each position
  const uint32_t* flag;     // nonzero: the lo planes matter (NULL: taken to)
  const uint64_t* tauk;     // [rows] bound: keys below it are kept
  const float* ht;          // [rows] the bound in accumulator space (never above it)
  uint64_t* cand;           // [rows][stride] (distance bits, position)
  int32_t* counts;          // [rows][nch]
  int64_t n, nq, row0;      // points; queries; first query row of this batch
  int64_t tile0;            // first tile of points of this phase
  int tiles, rowtiles, nch, per, region;
  int64_t stride;
  int kpad, ip, base;
  KnnFilter f;              // point_label == NULL: every point counts
};

__device__ __forceinline__ bool knn_allowed(const KnnFilter& f, int64_t row, int32_t id) {
  return f.point_label == nullptr || f.point_label[id] < (uint32_t)f.row_id[row] + 1u;
}

// One (row tile, chunk of point tiles) per block of four waves; wave w owns
// query rows 32 w .. 32 w + 31 of the tile's 128 against all points of a point
// tile.  The points' slabs (32 or 64 coordinates of hi and lo) go through LDS,
// two buffers deep, one slab ahead in registers; the query fragments stay in
// registers for kpad = 32 KS <= 128 (KS = 0: they go through LDS as well).
// Chunks are dealt so that the blocks of one XCD (every eighth block) walk the
// same points at the same time with different query rows: a tile is fetched
// once per XCD and its L2 serves the rest.
// An LDS row's 16-byte pieces are placed at piece ^ (row / 2) % 4 (rows of 64
// bytes) or piece ^ row % 8 (of 128), so that eight consecutive rows cover
// every bank once.
// Accumulators start at -|x|^2 / 2, so d2 = |q|^2 - 2 acc and one comparison
// with ht decides; a wave whose comparisons of a tile all fail (most of them
// after the first phases) goes on to the next tile.
// Points of a tile for kpad = 32 ks <= 128 (ks = 0: longer vectors): 64, so that
// three waves fit a SIMD and one wave's comparisons and waits overlap another's
// products (128 points with two waves take 1.67 ms where 64 with three take
// 1.53 ms for 10,000 x 300,000 x 128, one product); longer vectors spend their
// time on the products and take 128, which halves their query traffic.
constexpr int tile_x(int ks) { return ks > 0 ? 64 : 128; }
// 32-wide k steps per slab
constexpr int slab_steps(int ks, bool lo) { return ks > 0 && !lo && ks % 2 == 0 ? 2 : 1; }

template <int KS, bool LO>
__device__ __forceinline__ void scan_body(const ScanArgs& a, __bf16* sm, uint64_t* s_tau, float* s_qn, int* s_cnt) {
  constexpr int kTileX = tile_x(KS), kCols = kTileX / 16;
  constexpr int KB = slab_steps(KS, LO);
  constexpr int kRow = kBK * KB;                       // elements of an LDS row
  constexpr int kPlane = kTileX * kRow;                // elements of one plane of one slab
  constexpr int kSide = (LO ? 2 : 1) * kPlane;         // hi (and lo) of one side
  constexpr int kPlaneQ = kTileQ * kRow;               // the same of the queries (KS = 0)
  constexpr int kBuf = kSide + (KS == 0 ? (LO ? 2 : 1) * kPlaneQ : 0);
  constexpr int kPieces = 4 * KB;                      // 16-byte pieces per LDS row
  constexpr int kPer = kTileX * kPieces / 256;         // pieces per thread and plane
  static_assert(KS > 0 || kTileX == kTileQ, "one staging loop for both sides");
  const int t = threadIdx.x, w = uniform_i(t >> 6), l = t & 63;
  const int lr = l & 15, g = l >> 4;
  const int b = blockIdx.x;
  int chunk, rt;
  if (a.nch % 8 == 0) {
    const int i = b >> 3;
    rt = i % a.rowtiles;
    chunk = (i / a.rowtiles) * 8 + (b & 7);
  } else {
    rt = b % a.rowtiles;
    chunk = b / a.rowtiles;
  }
  const int t_beg = chunk * a.per, t_end = min(a.tiles, t_beg + a.per);
  const int64_t lrow0 = (int64_t)rt * kTileQ;          // first row of the tile in the batch
  const int64_t qrow0 = a.row0 + lrow0;
  for (int i = t; i < kTileQ; i += 256) {
    s_cnt[i] = 0;
    s_qn[i] = a.qn[qrow0 + i];
    if (!a.base) s_tau[i] = a.tauk[lrow0 + i];
  }
  float ht[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) ht[i][v] = a.base ? 0.f : a.ht[lrow0 + 32 * w + 16 * i + 4 * g + v];
  __syncthreads();
  if (t_beg < t_end) {
    const int slabs = KS > 0 ? KS / KB : a.kpad / kBK;
    constexpr int KA = KS > 0 ? KS : 1;
    b8v ah[2][KA], al[2][KA];
    if constexpr (KS > 0) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const int64_t o = (qrow0 + 32 * w + 16 * i + lr) * a.kpad + kBK * ks + 8 * g;
          ah[i][ks] = *reinterpret_cast<const b8v*>(a.qh + o);
          if constexpr (LO) al[i][ks] = *reinterpret_cast<const b8v*>(a.ql + o);
        }
    }
    // staging: 16-byte pieces t, t + 256, ... of the slab
    auto swz = [](int piece, int row) {
      return KB % 2 == 0 ? piece ^ (row & 7) : piece ^ ((row >> 1) & 3);
    };
    b8v rh[kPer], rl[kPer], rqh[kPer], rql[kPer];
    auto load = [&](int tile, int slab) {
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int row = (t + 256 * u) / kPieces, pc = (t + 256 * u) % kPieces;
        const int64_t o = ((a.tile0 + tile) * kTileX + row) * a.kpad + kRow * slab + 8 * pc;
        rh[u] = *reinterpret_cast<const b8v*>(a.xh + o);
        if constexpr (LO) rl[u] = *reinterpret_cast<const b8v*>(a.xl + o);
        if constexpr (KS == 0) {
          const int64_t p = (qrow0 + row) * a.kpad + kRow * slab + 8 * pc;
          rqh[u] = *reinterpret_cast<const b8v*>(a.qh + p);
          if constexpr (LO) rql[u] = *reinterpret_cast<const b8v*>(a.ql + p);
        }
      }
    };
    auto put = [&](__bf16* buf) {
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int row = (t + 256 * u) / kPieces, pc = (t + 256 * u) % kPieces;
        const int so = row * kRow + swz(pc, row) * 8;
        *reinterpret_cast<b8v*>(buf + so) = rh[u];
        if constexpr (LO) *reinterpret_cast<b8v*>(buf + kPlane + so) = rl[u];
        if constexpr (KS == 0) {
          *reinterpret_cast<b8v*>(buf + kSide + so) = rqh[u];
          if constexpr (LO) *reinterpret_cast<b8v*>(buf + kSide + kPlaneQ + so) = rql[u];
        }
      }
    };
    // slab s + 2 of the walk (tile-major), the last slab again past the end
    int ltile = t_beg, lslab = 0;
    auto advance = [&]() {
      if (lslab + 1 < slabs) {
        ++lslab;
      } else if (ltile + 1 < t_end) {
        ++ltile;
        lslab = 0;
      }
    };
    load(ltile, lslab);
    advance();
    put(sm);
    load(ltile, lslab);
    advance();
    int cur = 0;
    float hxn[kCols];
#pragma unroll
    for (int j = 0; j < kCols; ++j) hxn[j] = a.hx[(a.tile0 + t_beg) * kTileX + 16 * j + lr];
    for (int tile = t_beg; tile < t_end; ++tile) {
      const int64_t c0 = (a.tile0 + tile) * kTileX;
      f4v acc[2][kCols];
#pragma unroll
      for (int j = 0; j < kCols; ++j) {
        acc[0][j] = f4v{-hxn[j], -hxn[j], -hxn[j], -hxn[j]};
        acc[1][j] = acc[0][j];
      }
      {
        const int64_t cn = (a.tile0 + min(tile + 1, t_end - 1)) * kTileX;
#pragma unroll
        for (int j = 0; j < kCols; ++j) hxn[j] = a.hx[cn + 16 * j + lr];
      }
      auto step = [&](int slab) {
        // LDS only: the loads in flight stay in flight over the barrier
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        const __bf16* rd = sm + cur * kBuf;
        put(sm + (cur ^ 1) * kBuf);
        load(ltile, lslab);
        advance();
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const int fo = lr * kRow + swz(4 * kb + g, lr) * 8;  // this lane's fragment in 16 rows
          b8v qh[2], ql[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            if constexpr (KS > 0) {
              qh[i] = ah[i][slab * KB + kb];
              if constexpr (LO) ql[i] = al[i][slab * KB + kb];
            } else {
              qh[i] = *reinterpret_cast<const b8v*>(rd + kSide + (32 * w + 16 * i) * kRow + fo);
              if constexpr (LO) ql[i] = *reinterpret_cast<const b8v*>(rd + kSide + kPlaneQ + (32 * w + 16 * i) * kRow + fo);
            }
          }
#pragma unroll
          for (int j = 0; j < kCols; ++j) {
            const b8v xh = *reinterpret_cast<const b8v*>(rd + 16 * j * kRow + fo);
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qh[i], xh, acc[i][j], 0, 0, 0);
            if constexpr (LO) {
              const b8v xl = *reinterpret_cast<const b8v*>(rd + kPlane + 16 * j * kRow + fo);
#pragma unroll
              for (int i = 0; i < 2; ++i) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qh[i], xl, acc[i][j], 0, 0, 0);
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ql[i], xh, acc[i][j], 0, 0, 0);
              }
            }
          }
        }
        cur ^= 1;
      };
      if constexpr (KS > 0) {
#pragma unroll
        for (int sl = 0; sl < KS / KB; ++sl) step(sl);
      } else {
        for (int sl = 0; sl < slabs; ++sl) step(sl);
      }
      if (a.base) {
        // every score of the prefix, at its own place
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int rr = 32 * w + 16 * i + 4 * g + v;
            uint64_t* row = a.cand + (lrow0 + rr) * a.stride;
            const float qn = s_qn[rr];
#pragma unroll
            for (int j = 0; j < kCols; ++j) {
              const int64_t col = c0 + 16 * j + lr;
              const float d = a.ip ? -acc[i][j][v] : fmaxf(qn - 2.f * acc[i][j][v], 0.f);
              bool in = col < a.n && d < __int_as_float(0x7f800000);
              if (a.f.point_label != nullptr && in) in = qrow0 + rr < a.nq && knn_allowed(a.f, qrow0 + rr, a.perm[col]);
              row[col] = in ? make_key(d, (int)col) : ~0ull;
            }
          }
        continue;
      }
      // lanes with a score to look at, by accumulator row, as scalar masks, so
      // that only the rows concerned are gone through (a NaN passes the
      // comparison, and scores 0 below)
      uint64_t rows[2][4], any = 0ull;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          uint64_t r = 0ull;
#pragma unroll
          for (int j = 0; j < kCols; ++j) r |= ballot(!(acc[i][j][v] < ht[i][v]));
          rows[i][v] = r;
          any |= r;
        }
      if (any == 0ull) continue;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (rows[i][v] == 0ull) continue;
          uint32_t todo = 0u;
#pragma unroll
          for (int j = 0; j < kCols; ++j) todo |= !(acc[i][j][v] < ht[i][v]) ? 1u << j : 0u;
          const int rr = 32 * w + 16 * i + 4 * g + v;
          const uint64_t tk = s_tau[rr];
          const float qn = s_qn[rr];
          while (todo != 0u) {
            const int j = __ffs(todo) - 1;
            todo &= todo - 1u;
            float s = acc[i][0][v];
#pragma unroll
            for (int e = 1; e < kCols; ++e) s = j == e ? acc[i][e][v] : s;
            const int64_t col = c0 + 16 * j + lr;
            const float d = a.ip ? -s : fmaxf(qn - 2.f * s, 0.f);
            if (!(col < a.n && d < __int_as_float(0x7f800000))) continue;
            const uint32_t db = order_bits(d), tb = (uint32_t)(tk >> 32);
            bool in = db < tb;
            if (db == tb) in = (uint32_t)a.perm[col] < (uint32_t)tk;
            if (!in || (a.f.point_label != nullptr && !knn_allowed(a.f, qrow0 + rr, a.perm[col]))) continue;
            const int pos = atomicAdd(&s_cnt[rr], 1);
            if (pos < a.region)
              a.cand[(lrow0 + rr) * a.stride + (int64_t)chunk * a.region + pos] = ((uint64_t)db << 32) | (uint32_t)col;
          }
        }
    }
  }
  if (a.base) return;
  __syncthreads();
  for (int i = t; i < kTileQ; i += 256) a.counts[(lrow0 + i) * a.nch + chunk] = s_cnt[i];
}

// The instance without the lo products needs fewer registers; both are launched
// and the flag decides on the device which of them works.  Waves per SIMD: as
// many as the registers allow without spilling in the products' loop (at 96
// coordinates with lo, two addresses are kept in scratch and reread where a key
// is kept: 10,000 x 300,000 x 96 2.0 ms with three waves, 2.2 with two).
constexpr int scan_waves(int ks, bool lo) { return ks == 0 || (lo && ks == 4) ? 2 : 3; }

template <int KS, bool LO>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(scan_waves(KS, LO), 4))) k_knn_scan(ScanArgs a) {
  extern __shared__ __align__(16) char smem[];
  if (a.flag != nullptr && (*a.flag != 0u) != LO) return;
  uint64_t* s_tau = reinterpret_cast<uint64_t*>(smem);
  float* s_qn = reinterpret_cast<float*>(s_tau + kTileQ);
  int* s_cnt = reinterpret_cast<int*>(s_qn + kTileQ);
  __bf16* sm = reinterpret_cast<__bf16*>(s_cnt + kTileQ);
  scan_body<KS, LO>(a, sm, s_tau, s_qn, s_cnt);
}

// two buffers of a slab (of the queries too for KS = 0)
constexpr int scan_lds(int ks, bool lo) {
  return kTileQ * 16 + 2 * (tile_x(ks) + (ks == 0 ? kTileQ : 0)) * (lo ? 2 : 1) * kBK * slab_steps(ks, lo) * 2;
}

// ------------------------------------------------------------- selection

// Per row: the KK smallest keys (distance, id) of the row's list so far and the
// keys appended by the last phase, found without a sort: the KK-th smallest
// distance bit by bit (counting the keys below a trial value by ballots over
// registers), then, where equal distances straddle the cut, the id the same
// way.  Leaves the list (in no order), the bound and its accumulator form; a
// row that ran out of space is flagged and its list left as it is.
// W waves share a row's gather (one where rows fill the GPU, four where few
// rows have many short regions); the first selects.
struct SelectArgs {
  const uint64_t* cand;
  const int32_t* counts;
  const int32_t* perm;
  const float* qn;
  uint64_t* best;   // [rows][KK]
  uint64_t* tauk;
  float* ht;
  int32_t* over;    // [rows]
  int64_t rows, rows_pad, row0, stride;
  int KK, nch, region, cap, base, prefix, ip;
};

constexpr int kSelRegs = 10;  // keys per lane held in registers (640 keys); more are read from LDS

template <int W>
__global__ void __launch_bounds__(256) k_knn_select(SelectArgs a) {
  extern __shared__ __align__(16) char smem[];
  __shared__ int s_n[4];
  const int wv = uniform_i(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int slot = W == 1 ? wv : 0;               // row of the block
  const int tid = W == 1 ? l : threadIdx.x;       // thread of the row
  const int64_t row = (int64_t)blockIdx.x * (4 / W) + slot;
  auto sync = [] {
    if constexpr (W == 1) wave_lds_sync();
    else __syncthreads();
  };
  if (row >= a.rows_pad) return;
  if (row >= a.rows) {  // padding rows of the last tile keep nothing
    if (tid == 0) {
      a.tauk[row] = 0ull;
      a.ht[row] = __int_as_float(0x7f800000);
    }
    return;
  }
  if (!a.base && uniform_i(a.over[row]) != 0) return;
  uint32_t* D = reinterpret_cast<uint32_t*>(smem) + (size_t)slot * 2 * a.cap;
  uint32_t* I = D + a.cap;
  uint64_t* best = a.best + row * a.KK;
  const uint64_t* cand = a.cand + row * a.stride;
  if (tid == 0) s_n[slot] = 0;
  sync();
  // place the existing ones of 64 keys; a wave's lanes share one claim
  auto place = [&](uint64_t k, uint32_t id) {
    const uint64_t bm = ballot(k != ~0ull);
    if (bm == 0ull) return;
    const int first = __ffsll((unsigned long long)bm) - 1;
    int at = 0;
    if (l == first) at = atomicAdd(&s_n[slot], popc64(bm));
    at = __shfl(at, first, 64) + mask_rank(bm);
    if (k != ~0ull && at < a.cap) {
      D[at] = (uint32_t)(k >> 32);
      I[at] = id;
    }
  };
  // U keys per thread together, so that their loads (and those of the ids
  // behind the positions) overlap
  constexpr int U = 4;
  auto take = [&](const uint64_t (&k)[U]) {
    uint32_t id[U];
#pragma unroll
    for (int u = 0; u < U; ++u) id[u] = k[u] != ~0ull ? (uint32_t)a.perm[(uint32_t)k[u]] : 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) place(k[u], id[u]);
  };
  constexpr int P = 64 * W;
  bool over = false;
  if (a.base) {
    for (int i0 = 0; i0 < a.prefix; i0 += U * P) {
      uint64_t k[U];
#pragma unroll
      for (int u = 0; u < U; ++u) k[u] = i0 + u * P + tid < a.prefix ? cand[i0 + u * P + tid] : ~0ull;
      take(k);
    }
    if (tid == 0) a.over[row] = 0;
  } else {
    for (int i0 = 0; i0 < a.KK; i0 += P) {
      const uint64_t k = i0 + tid < a.KK ? best[i0 + tid] : ~0ull;
      place(k, (uint32_t)k);
    }
    // G threads per region (a power of two), so that few regions of many keys
    // are read as wide as many of few
    int G = 1;
    while (2 * G * a.nch <= P) G *= 2;
    const int sub = tid & (G - 1);
    for (int c0 = 0; c0 < a.nch; c0 += P / G) {
      const int c = c0 + tid / G;
      const int cnt = c < a.nch ? a.counts[row * a.nch + c] : 0;
      over |= cnt > a.region;
      const int have = min(cnt, a.region);
      for (int i = sub; ballot(i < have) != 0ull; i += U * G) {
        uint64_t k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = i + u * G < have ? cand[(int64_t)c * a.region + i + u * G] : ~0ull;
        take(k);
      }
    }
  }
  if (over) s_n[slot] = a.cap + 1;  // (after every claim of this thread; a later claim only adds)
  sync();
  const int N = uniform_i(s_n[slot]);
  if (W > 1 && wv != 0) return;
  if (N > a.cap) {
    if (l == 0) {
      a.over[row] = 1;
      a.tauk[row] = 0ull;
      a.ht[row] = __int_as_float(0x7f800000);  // nothing more is appended
    }
    return;
  }
  // Too few points so far: any further one is kept.  (Not with KK: a phase that
  // appends nothing leaves the bound, or the next one would append everything.)
  if (N < a.KK) {
    for (int i = l; i < a.KK; i += 64) best[i] = i < N ? (((uint64_t)D[i] << 32) | I[i]) : ~0ull;
    if (l == 0) {
      a.tauk[row] = ~0ull;
      a.ht[row] = -__int_as_float(0x7f800000);
    }
    return;
  }
  // distances: the first 64 kSelRegs in registers (past N: all ones, below no
  // trial), the rest from LDS
  uint32_t dv[kSelRegs];
#pragma unroll
  for (int r = 0; r < kSelRegs; ++r) dv[r] = 64 * r + l < N ? D[64 * r + l] : ~0u;
  const int regs = min(kSelRegs, (N + 63) / 64);
  auto count_below = [&](uint32_t trial) {
    int c = 0;
#pragma unroll
    for (int r = 0; r < kSelRegs; ++r)
      if (r < regs) c += popc64(ballot(dv[r] < trial));
    for (int i = 64 * kSelRegs + l; i - l < N; i += 64) c += popc64(ballot(i < N && D[i] < trial));
    return c;
  };
  // the KK-th smallest distance: the common leading bits, then bit by bit
  uint32_t mn = ~0u, mx = 0u;
  for (int i = l; i < N; i += 64) {
    mn = min(mn, D[i]);
    mx = max(mx, D[i]);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    mn = min(mn, (uint32_t)__shfl_xor((int)mn, o, 64));
    mx = max(mx, (uint32_t)__shfl_xor((int)mx, o, 64));
  }
  mx = (uint32_t)uniform_i((int)mx);
  const uint32_t x = (uint32_t)uniform_i((int)mn) ^ mx;
  const int top = x ? 31 - __clz(x) : -1;
  uint32_t v = top == 31 ? 0u : mx >> (top + 1) << (top + 1);
  int below = 0;  // keys below v: none shares fewer leading bits
  for (int bit = top; bit >= 0; --bit) {
    const uint32_t trial = v | (1u << bit);
    const int c = count_below(trial);
    if (c < a.KK) {
      v = trial;
      below = c;
    }
  }
  const int need = a.KK - below;
  // ids among the equal distances
  int eq = 0;
  uint32_t idmax = 0u;
  for (int i = l; i - l < N; i += 64) {
    const bool same = i < N && D[i] == v;
    eq += popc64(ballot(same));
    if (same) idmax = max(idmax, I[i]);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) idmax = max(idmax, (uint32_t)__shfl_xor((int)idmax, o, 64));
  uint32_t lim = (uint32_t)uniform_i((int)idmax);
  if (eq > need) {
    uint32_t id = 0u;
    for (int bit = 30; bit >= 0; --bit) {
      const uint32_t trial = id | (1u << bit);
      int c = 0;
      for (int i = l; i - l < N; i += 64) c += popc64(ballot(i < N && D[i] == v && I[i] < trial));
      if (c < need) id = trial;
    }
    lim = id;
  }
  int out = 0;
  for (int i0 = 0; i0 < N; i0 += 64) {
    const int i = i0 + l;
    const bool in = i < N && (D[i] < v || (D[i] == v && I[i] <= lim));
    const uint64_t bm = ballot(in);
    if (in) best[out + mask_rank(bm)] = ((uint64_t)D[i] << 32) | I[i];
    out += popc64(bm);
  }
  if (l == 0) {
    a.tauk[row] = ((uint64_t)v << 32) | lim;
    // accumulators below ht score above the bound for certain (d2 is rounded
    // once from |q|^2 - 2 acc)
    const float td = order_bits_inv(v), qn = a.qn[a.row0 + row];
    a.ht[row] = a.ip ? -td : 0.5f * (qn - td) - 2.4e-7f * (fabsf(qn) + fabsf(td));
  }
}

// ------------------------------------------------------------- final list

// Per query one block of four waves: the candidates' exact distances by
// direct float32 differences (four candidates in flight per wave), then the
// best k by (d2, id).  A flagged row then scans every point, eight in flight
// per wave, and ranks those below the k-th distance known so far (rare: see
// the top of the file).  Ten such rows x 300,000 x 128 take 15 ms (97 with the
// points one after another and every slab ranked whole), bounded by the
// latency of one workgroup's loads.
struct FinalArgs {
  const float *q, *x;
  const double *qinv, *xinv;  // angular: reciprocal norms
  const uint64_t* best;
  const int32_t* over;
  int64_t row0, n;
  int m, k, KK, ip;
  KnnFilter f;
  int32_t* ids;
  float* dist;
};

__device__ __forceinline__ float knn_term(const FinalArgs& a, float q, float x, double qi, double xi, float d) {
  if (a.qinv != nullptr) {
    q = (float)(q * qi);
    x = (float)(x * xi);
  }
  // fused multiply-adds written out: left to the compiler, the two branches
  // merge into a select of products and a plain add, one rounding more
  if (a.ip) return __builtin_fmaf(-q, x, d);
  const float u = q - x;
  return __builtin_fmaf(u, u, d);
}

// Eight wave sums at once: lane l gets that of v[sum8_index(l)], by the
// additions of wave_sum (each step adds the same two partial sums, and splits
// the values between the two lanes that did).
__device__ __forceinline__ int sum8_index(int l) { return ((l & 1) << 2) | (l & 2) | ((l >> 2) & 1); }
__device__ __forceinline__ float sum8(float (&v)[8]) {
  constexpr int kDppXor3 = 0x1B, kDppRor8 = 0x128;
  const int l = lane_id();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool up = (l & 1) != 0;
    v[j] = (up ? v[j + 4] : v[j]) + dpp_f<kDppXor1>(up ? v[j] : v[j + 4]);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const bool up = (l & 2) != 0;
    v[j] = (up ? v[j + 2] : v[j]) + dpp_f<kDppXor2>(up ? v[j] : v[j + 2]);
  }
  const bool up = (l & 4) != 0;
  // (half mirror, then reversed quads: lane l ^ 4)
  float s = (up ? v[1] : v[0]) + dpp_f<kDppXor3>(dpp_f<kDppHalfMirror>(up ? v[0] : v[1]));
  s += dpp_f<kDppRor8>(s);
  s += shfl_xor_f(s, 16);
  return s + shfl_xor_f(s, 32);
}

// A flagged row: the k smallest keys of all points to ex[0 .. k).  ex holds the
// candidates' KK exact keys, which only give the first bound (they are met
// again among the points); room for 2 k + 256 keys.
__device__ __forceinline__ void search_all(const FinalArgs& a, int64_t q, uint64_t* ex) {
  const int t = threadIdx.x, w = uniform_i(t >> 6), l = t & 63;
  const float* qv = a.q + q * a.m;
  const double qi = a.qinv != nullptr ? a.qinv[q] : 1.0;
  __shared__ uint64_t s_bound;
  __shared__ int s_cnt;
  for (int i = t; i < a.KK; i += 256) {
    const uint64_t v = ex[i];
    int rk = 0;
    for (int o = 0; o < a.KK; ++o) rk += (ex[o] < v || (ex[o] == v && o < i)) ? 1 : 0;
    if (rk == a.k - 1) s_bound = v;
  }
  if (t == 0) s_cnt = 0;
  __syncthreads();
  uint64_t bound = s_bound;
  uint64_t* list = ex;        // [k] ascending
  uint64_t* slab = ex + a.k;  // [256] keys up to the bound among 256 points
  uint64_t* next = slab + 256;  // [k]
  for (int i = t; i < a.k; i += 256) list[i] = ~0ull;
  for (int64_t b0 = 0; b0 < a.n; b0 += 256) {
    for (int e0 = 0; e0 < 64; e0 += 8) {
      const int64_t first = b0 + 64 * w + e0;
      if (first >= a.n) break;
      const int last = (int)min(a.n - 1 - first, (int64_t)7);
      const float* x0 = a.x + first * a.m;
      float d[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      for (int j = l; j < a.m; j += 64) {
        const float qj = qv[j];
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = x0[min(e, last) * a.m + j];
#pragma unroll
        for (int e = 0; e < 8; ++e)
          d[e] = knn_term(a, qj, x[e], qi, a.xinv != nullptr ? a.xinv[first + min(e, last)] : 1.0, d[e]);
      }
      const float mine = sum8(d);
      const int64_t id = first + sum8_index(l);
      if (l < 8 && id < a.n) {
        const uint64_t key = make_key(mine, (int)id);
        if (key <= bound && knn_allowed(a.f, q, (int32_t)id)) slab[atomicAdd(&s_cnt, 1)] = key;
      }
    }
    __syncthreads();
    const int total = a.k + s_cnt;
    if (total > a.k) {
      for (int i = t; i < total; i += 256) {
        const uint64_t key = list[i];
        int rk = 0;
        for (int o = 0; o < total; ++o) rk += (list[o] < key || (list[o] == key && o < i)) ? 1 : 0;
        if (rk < a.k) next[rk] = key;
      }
      __syncthreads();
      for (int i = t; i < a.k; i += 256) list[i] = next[i];
      bound = min(bound, next[a.k - 1]);
      if (t == 0) s_cnt = 0;
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(256) k_knn_final(FinalArgs a) {
  extern __shared__ __align__(16) char smem[];
  uint64_t* ex = reinterpret_cast<uint64_t*>(smem);  // [KK], or [2 k + 256] for a flagged row
  const int t = threadIdx.x, w = uniform_i(t >> 6), l = t & 63;
  const int64_t row = blockIdx.x, q = a.row0 + row;
  const float* qv = a.q + q * a.m;
  const double qi = a.qinv != nullptr ? a.qinv[q] : 1.0;
  const bool flagged = a.over[row] != 0;
  const uint64_t* best = a.best + row * a.KK;
  for (int c0 = 4 * w; c0 < a.KK; c0 += 16) {
    const float* xv[4];
    double xi[4] = {1.0, 1.0, 1.0, 1.0};
    int id[4];
    float d[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint64_t key = c0 + e < a.KK ? best[c0 + e] : ~0ull;
      id[e] = uniform_i(key == ~0ull ? -1 : key_id(key));
      xv[e] = a.x + (int64_t)(id[e] < 0 ? 0 : id[e]) * a.m;
      if (a.xinv != nullptr) xi[e] = a.xinv[id[e] < 0 ? 0 : id[e]];
    }
    for (int j = l; j < a.m; j += 64) {
      const float qj = qv[j];
#pragma unroll
      for (int e = 0; e < 4; ++e) d[e] = knn_term(a, qj, xv[e][j], qi, xi[e], d[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float s = wave_sum(d[e]);
      if (l == 0 && c0 + e < a.KK) ex[c0 + e] = id[e] < 0 ? ~0ull : make_key(s, id[e]);
    }
  }
  __syncthreads();
  int keep = a.KK;
  if (flagged) {
    search_all(a, q, ex);
    keep = a.k;
  }
  for (int i = t; i < keep; i += 256) {
    const uint64_t v = ex[i];
    int rk = 0;
    for (int o = 0; o < keep; ++o) rk += (ex[o] < v || (ex[o] == v && o < i)) ? 1 : 0;
    if (rk < a.k) {
      a.ids[q * a.k + rk] = v == ~0ull ? -1 : key_id(v);
      a.dist[q * a.k + rk] = v == ~0ull ? __int_as_float(0x7f800000) : key_d2(v);
    }
  }
}

// bound[i]: see launch_exact_knn.  (In k_knn_final it cost that 9 us of 43.)
__global__ void k_knn_bounds(const uint64_t* tauk, const int32_t* over, const float* qn, int64_t rows, float2* bound) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows) return;
  const uint64_t tk = over[i] == 0 ? tauk[i] : ~0ull;
  bound[i] = make_float2(tk == ~0ull ? __int_as_float(0x7f800000) : order_bits_inv((uint32_t)(tk >> 32)), qn[i]);
}

// ------------------------------------------------------------------ plan

size_t up256(size_t b) { return (b + 255) / 256 * 256; }

struct KnnPlan {
  int KK, kpad, prefix, cap, nch;
  int64_t n_pad, q_pad, rows, window, stride;
  size_t off_xh, off_xl, off_qh, off_ql, off_hx, off_qn, off_perm, off_xinv, off_qinv, off_flag, off_best, off_tauk,
      off_ht, off_over, off_counts, off_cand, total;
};

// Keys a phase may append per (row, chunk): the expected (kKnnGrowth - 1) KK
// keys of a row are shared evenly by the chunks; four times that, and 16 for
// the spread of small shares.
int knn_region(int cap, int nch) { return nch == 1 ? cap : (cap + nch - 1) / nch + 16; }

// Memory: the planes hold a window of positions at a time (kKnnPlanes bytes
// at most; with several windows they are split again for every batch of rows:
// 12 bytes moved per element against 2 x 65,536 operations), and the keys those
// of kRowBatch rows.  Both are 1/16 of that where the caller asks for a small
// workspace.  Neither changes a result: the KK smallest keys do not depend on
// where a phase ends.  Several windows cost calls of few queries up to 8% (one
// query x 400,000 x 2,048: 3.0 ms, 2.8 with all points held; 5,000 the same).
constexpr size_t kKnnPlanes = (size_t)1 << 30;

KnnPlan knn_plan(int64_t n, int m, int64_t nq, int k, const KnnSpace& space) {
  const int shrink = space.small ? 16 : 1;
  KnnPlan p{};
  p.KK = k + kKnnSlack;
  p.kpad = (m + kBK - 1) / kBK * kBK;
  p.n_pad = (n + kPadX - 1) / kPadX * kPadX;
  p.q_pad = (nq + kTileQ - 1) / kTileQ * kTileQ;
  p.cap = std::max(512, 16 * p.KK);
  p.rows = std::min(p.q_pad, kRowBatch / shrink);
  // prefix scored whole: a few times KK, or everything when little is left
  int64_t prefix = p.KK <= 64 ? 512 : 1024;
  if (n <= 1024) prefix = 1024;
  p.prefix = (int)std::min(prefix, p.n_pad);
  p.window = std::min(p.n_pad, std::max<int64_t>(1024, (int64_t)(kKnnPlanes / shrink) / (4 * p.kpad) / kPadX * kPadX));
  // chunks of points per row tile: enough blocks (two or three fit a CU) for
  // several rounds, in whole multiples of the eight XCDs
  const int64_t rowtiles = p.rows / kTileQ, tiles = p.n_pad / kPadX;
  int64_t nch = (2048 + rowtiles - 1) / rowtiles;
  nch = std::min<int64_t>({(nch + 7) / 8 * 8, tiles, kMaxChunks});
  if (nch > 8) nch = nch / 8 * 8;
  p.nch = (int)std::max<int64_t>(nch, 1);
  p.stride = p.prefix;
  // fewer chunks in an early phase have larger regions
  for (int c = 1; c <= p.nch; ++c) p.stride = std::max<int64_t>(p.stride, (int64_t)c * knn_region(p.cap, c));
  // Space for the keys and counts: bounds that never fall as n or nq grows,
  // so that a workspace taken for the largest call holds every smaller one
  // (c regions hold at most cap + 17 c keys; chunks <= rowtiles nch).
  const int64_t chunks = std::min<int64_t>({rowtiles * kMaxChunks, 2048 + 8 * rowtiles, rowtiles * tiles});
  const size_t cand_keys = (size_t)p.rows * std::max(1024, p.cap) + (size_t)17 * kTileQ * chunks;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += up256(bytes);
    return at;
  };
  p.off_xh = take((size_t)p.window * p.kpad * 2);
  p.off_xl = take((size_t)p.window * p.kpad * 2);
  p.off_qh = take((size_t)p.rows * p.kpad * 2);
  p.off_ql = take((size_t)p.rows * p.kpad * 2);
  p.off_hx = take((size_t)p.window * 4);
  p.off_qn = take((size_t)p.rows * 4);
  p.off_perm = take((size_t)p.n_pad * 4);
  p.off_xinv = take(space.angular ? (size_t)n * 8 : 0);
  p.off_qinv = take(space.angular ? (size_t)nq * 8 : 0);
  p.off_flag = take(4);
  p.off_best = take((size_t)p.rows * p.KK * 8);
  p.off_tauk = take((size_t)p.rows * 8);
  p.off_ht = take((size_t)p.rows * 4);
  p.off_over = take((size_t)p.rows * 4);
  p.off_counts = take((size_t)kTileQ * chunks * 4);
  p.off_cand = take(cand_keys * 8);
  p.total = o;
  return p;
}

template <int KS, bool LO>
hipError_t launch_scan_lo(const ScanArgs& a, hipStream_t s) {
  constexpr int lds = scan_lds(KS, LO);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_knn_scan<KS, LO>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_knn_scan<KS, LO>), dim3((unsigned)(a.rowtiles * a.nch)), dim3(256), lds, s, a);
  return hipGetLastError();
}

template <int KS>
hipError_t launch_scan(const ScanArgs& a, hipStream_t s) {
  const hipError_t e = a.flag != nullptr ? launch_scan_lo<KS, false>(a, s) : hipSuccess;
  return e != hipSuccess ? e : launch_scan_lo<KS, true>(a, s);
}

}  // namespace

size_t exact_knn_ws_bytes(int64_t n, int m, int64_t nq, int k, const KnnSpace& space) {
  return knn_plan(n, m, nq, k, space).total;
}

bool knn_certain(float d, float last, float score, float qq, int m) {
  // A float32 distance is a sum of squares with at most 64 roundings on any
  // path (m <= 2048), so two of them order as the exact ones do when they
  // differ by more than 2^-16 of themselves, whatever their order of sums.
  constexpr double rel = 1.0 / 65536;
  if (!(d < last * (1.0 - rel))) return false;
  // Scores: with Q = |q| and X = |x| the products left out by the split are
  // below 3 2^-18 Q X, and 3 m products, the norms' 2 m and the start value are
  // added with an error of 2^-23 of the largest partial sum each.  Points with
  // X > Q + sqrt(d) are further away than d in any case.
  const double e = m / 8388608.0, Q = std::sqrt((double)qq) * (1.0 + e);
  const double X = (Q + std::sqrt((double)d)) * (1.0 + rel);
  const double err = Q * X * (1.0 / 32768 + 6.2 * e) + X * X * 4.0 * e + Q * Q * e + 1e-30;
  return (double)d * (1.0 + rel) < (double)score - err && err < 1e37;
}

hipError_t launch_exact_knn(const float* data, int64_t n, int m, const float* Q, int64_t nq, int k, int metric,
                            int32_t* ids, float* dist, void* ws, size_t ws_bytes, hipStream_t s, const KnnFilter* filter,
                            float2* bound, const KnnSpace& space) {
  if (nq == 0) return hipSuccess;
  const KnnPlan p = knn_plan(n, m, nq, k, space);
  if (ws_bytes < p.total || (metric == FINGER_ANGULAR && !space.angular)) return hipErrorInvalidValue;
  char* b = static_cast<char*>(ws);
  auto at = [&](size_t off) { return static_cast<void*>(b + off); };
  const bool ang = metric == FINGER_ANGULAR, ip = metric == FINGER_IP;
  __bf16 *xh = (__bf16*)at(p.off_xh), *xl = (__bf16*)at(p.off_xl), *qh = (__bf16*)at(p.off_qh), *ql = (__bf16*)at(p.off_ql);
  float *hx = (float*)at(p.off_hx), *qn = (float*)at(p.off_qn);
  int32_t* perm = (int32_t*)at(p.off_perm);
  double *xinv = ang ? (double*)at(p.off_xinv) : nullptr, *qinv = ang ? (double*)at(p.off_qinv) : nullptr;
  // A call of one short scan takes the products with lo without asking whether
  // they matter (zeros add nothing): two launches fewer (one query x 100 points
  // x 32: 49 us, now 44).
  const bool ask = p.n_pad > p.prefix || nq > 2048;
  uint32_t* flag = ask ? (uint32_t*)at(p.off_flag) : nullptr;
  hipError_t e = ask ? launch_fill_u32(flag, 0u, 1, s) : hipSuccess;
  if (e != hipSuccess) return e;
  // stride of the scan order: near the golden section of n, prime to n
  int64_t a = std::max<int64_t>(1, (int64_t)(0.6180339887498949 * (double)n));
  while (std::gcd(a, n) != 1) ++a;
  auto split_points = [&](int64_t first) {
    const int64_t rows = std::min(p.window, p.n_pad - first);
    hipLaunchKernelGGL(k_knn_split, dim3((unsigned)(rows / 16)), dim3(256), 0, s, data, n, m, first, rows, p.kpad, a,
                       ip ? 0.f : 0.5f, __builtin_inff(), xh, xl, hx, perm, xinv, flag);
    return hipGetLastError();
  };
  auto split_queries = [&](int64_t first, int64_t rows_pad) {
    hipLaunchKernelGGL(k_knn_split, dim3((unsigned)(rows_pad / 16)), dim3(256), 0, s, Q, nq, m, first, rows_pad, p.kpad,
                       (int64_t)0, ip ? 0.f : 1.f, 0.f, qh, ql, qn, (int32_t*)nullptr, qinv, flag);
    return hipGetLastError();
  };

  ScanArgs c{};
  c.perm = perm;
  c.flag = flag;
  c.tauk = (uint64_t*)at(p.off_tauk);
  c.ht = (float*)at(p.off_ht);
  c.cand = (uint64_t*)at(p.off_cand);
  c.counts = (int32_t*)at(p.off_counts);
  c.n = n;
  c.nq = nq;
  if (filter != nullptr) c.f = *filter;
  c.stride = p.stride;
  c.kpad = p.kpad;
  c.ip = ip ? 1 : 0;
  auto scan = [&]() {
    // query fragments stay in registers up to 128 dimensions
    switch (p.kpad / kBK) {
      case 1: return launch_scan<1>(c, s);
      case 2: return launch_scan<2>(c, s);
      case 3: return launch_scan<3>(c, s);
      case 4: return launch_scan<4>(c, s);
      default: return launch_scan<0>(c, s);
    }
  };
  SelectArgs v{};
  v.cand = c.cand;
  v.counts = c.counts;
  v.perm = perm;
  v.best = (uint64_t*)at(p.off_best);
  v.tauk = (uint64_t*)at(p.off_tauk);
  v.ht = (float*)at(p.off_ht);
  v.over = (int32_t*)at(p.off_over);
  v.stride = p.stride;
  v.KK = p.KK;
  v.cap = std::max(p.prefix, p.cap) + p.KK;
  v.prefix = p.prefix;
  v.ip = c.ip;
  // four waves per row while one per row leaves the GPU under two waves a SIMD
  const bool wide = std::min(nq, p.rows) <= 2048;
  const int sel_lds = (wide ? 1 : 4) * 2 * v.cap * 4;
  const void* sel = wide ? reinterpret_cast<const void*>(k_knn_select<4>) : reinterpret_cast<const void*>(k_knn_select<1>);
  e = hipFuncSetAttribute(sel, hipFuncAttributeMaxDynamicSharedMemorySize, sel_lds);
  if (e != hipSuccess) return e;
  auto select = [&]() {
    if (wide)
      hipLaunchKernelGGL(k_knn_select<4>, dim3((unsigned)v.rows_pad), dim3(256), sel_lds, s, v);
    else
      hipLaunchKernelGGL(k_knn_select<1>, dim3((unsigned)(v.rows_pad / 4)), dim3(256), sel_lds, s, v);
    return hipGetLastError();
  };
  const int fin_lds = std::max(p.KK, 2 * k + 256) * 8;
  const int tx = tile_x(p.kpad <= 128 ? p.kpad / kBK : 0);
  const int64_t all_tiles = p.n_pad / tx, first = p.prefix / tx;
  // phases after the prefix, each growing it by the same factor
  int phases = 0;
  double grow = 1.0;
  if (all_tiles > first) {
    const double f = (double)all_tiles / (double)first;
    while (grow < f) {
      grow *= kKnnGrowth;
      ++phases;
    }
    grow = std::pow(f, 1.0 / phases);
  }
  const int64_t wtiles = p.window / tx;
  // arrays of which a part is held, as if from index zero
  auto from = [](auto* held, int64_t index) {
    return reinterpret_cast<decltype(held)>(reinterpret_cast<uintptr_t>(held) - (uintptr_t)index * sizeof(*held));
  };
  int64_t held = -1;  // first position that the planes hold
  auto hold = [&](int64_t first_pos) {
    if (held == first_pos) return hipSuccess;
    held = first_pos;
    c.xh = from(xh, first_pos * p.kpad);
    c.xl = from(xl, first_pos * p.kpad);
    c.hx = from(hx, first_pos);
    return split_points(first_pos);
  };
  for (int64_t r0 = 0; r0 < nq; r0 += p.rows) {
    const int64_t rows = std::min(nq - r0, p.rows);
    c.row0 = v.row0 = r0;
    c.qh = from(qh, r0 * p.kpad);
    c.ql = from(ql, r0 * p.kpad);
    c.qn = v.qn = from(qn, r0);
    c.rowtiles = (int)((rows + kTileQ - 1) / kTileQ);
    v.rows = rows;
    v.rows_pad = (int64_t)c.rowtiles * kTileQ;
    if ((e = hold(0)) != hipSuccess) return e;
    if ((e = split_queries(r0, v.rows_pad)) != hipSuccess) return e;
    c.base = v.base = 1;
    c.tile0 = 0;
    c.tiles = (int)first;
    c.nch = c.tiles;
    c.per = 1;
    c.region = 0;
    if ((e = scan()) != hipSuccess) return e;
    v.nch = 0;
    v.region = 0;
    if ((e = select()) != hipSuccess) return e;
    c.base = v.base = 0;
    int64_t done = first;
    for (int ph = 1; ph <= phases;) {
      int64_t next = ph == phases ? all_tiles : (int64_t)std::llround((double)first * std::pow(grow, ph));
      next = std::min(std::max(next, done), all_tiles);
      if (next == done) {
        ++ph;
        continue;
      }
      // a phase ends with the window
      const int64_t wfirst = done / wtiles * wtiles;
      if ((e = hold(wfirst * tx)) != hipSuccess) return e;
      next = std::min(next, wfirst + wtiles);
      c.tile0 = done;
      c.tiles = (int)(next - done);
      int64_t nch = std::min<int64_t>(p.nch, c.tiles);
      if (nch > 8) nch = nch / 8 * 8;
      c.nch = v.nch = (int)nch;
      c.per = (int)((c.tiles + nch - 1) / nch);
      c.region = v.region = knn_region(p.cap, c.nch);
      if ((e = scan()) != hipSuccess) return e;
      if ((e = select()) != hipSuccess) return e;
      done = next;
    }
    FinalArgs f{};
    f.q = Q;
    f.x = data;
    f.qinv = qinv;
    f.xinv = xinv;
    f.best = v.best;
    f.over = v.over;
    f.row0 = r0;
    f.n = n;
    f.m = m;
    f.k = k;
    f.KK = p.KK;
    f.ip = c.ip;
    f.f = c.f;
    f.ids = ids;
    f.dist = dist;
    hipLaunchKernelGGL(k_knn_final, dim3((unsigned)rows), dim3(256), fin_lds, s, f);
    if (bound != nullptr)
      hipLaunchKernelGGL(k_knn_bounds, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, s, v.tauk, v.over, qn, rows,
                         bound + r0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace finger
