// Batched solver: one workgroup runs the complete search of one instance
// (Algorithm 1's cost loop, Algorithm 2's constructors, uniqueness, ordered
// append, precision) with barriers as the only synchronisation, so many small
// instances progress side by side in one launch and no host round trip is
// needed per level or chunk.  Results are bit-identical to the per-chunk grid
// path: the same enumeration order, the same deterministic winner rule
// (smallest enumeration index), the same ordered append.
#include <algorithm>
#include <mutex>

#include "device_common.h"

namespace rei {

// Arenas of the allocation-free batched entry point.  In host code this name
// stands for the array only through hipGetSymbolAddress (static_scratch);
// kernels receive the address that call returns.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr uint32_t kWords = kBatchChunk / 32;  // winner bitmap words per chunk
constexpr int kMaxBlocks = 2 + 2 * (int)kBatchMaxCost;
constexpr uint32_t kTreeMax = kBatchTreeNodes;  // nodes of the answer tree written back

struct BlockD {
  uint32_t op, L, R, same;
  uint64_t count;
};

// The rows of a level that a block takes as one operand: [0, a) and [b, n).
// The others give candidates that equal an earlier one by an identity (see
// the per-chunk path: concatenations as left operands of concatenations,
// unions and r? as left operands and r? as right operands of unions, r? and
// r* as operands of ? and *).
struct Kept {
  uint32_t a, b, n;
  __device__ uint32_t count() const { return a + (n - b); }
  __device__ uint32_t below(uint32_t r) const {
    r = min(r, n);
    return r <= a ? r : (r > b ? r - (b - a) : a);
  }
  __device__ uint32_t row(uint32_t k) const { return k < a ? k : b + (k - a); }
  __device__ bool has(uint32_t r) const { return r < a || (r >= b && r < n); }
};

// A level's rows by constructor: characters below q, r? below s, r* below k,
// concatenations below u, then unions.
struct Marks {
  uint32_t q, s, k, u;
};

__device__ inline Kept left_kept(uint32_t op, const Marks& m, uint32_t n) {
  if (op == OP_CONCAT) return Kept{m.k, m.u, n};
  if (op == OP_UNION) return Kept{m.q, m.s, m.u};
  if (op == OP_CHAR) return Kept{n, n, n};
  return Kept{m.q, m.k, n};
}

// Work of block b's candidates [e0, e1): the first kept index and the items.
// Concatenations: an item is a 64-candidate tile, 64 right operands of one
// left operand (`a` kept left row, `b` tile), or 64 left operands of one right
// operand when the right level is small and shorter than the left (`a` tile
// of kept left rows); others: 64 consecutive kept candidates from `k`
// (unions of two levels: kept left row `a`, kept right row `b`).
struct Span {
  uint64_t k;
  uint32_t a, b, items;
};

__device__ __forceinline__ bool right_lanes(uint32_t nL, uint32_t nR) { return nR >= 64 || nR >= nL; }

__device__ inline Span block_span(const BlockD& blk, uint64_t e0, uint64_t e1, uint32_t nL, uint32_t nR, const Kept& kl,
                                  const Kept& kr) {
  Span sp{0, 0, 0, 0};
  if (blk.op == OP_CONCAT) {
    const uint64_t i0 = e0 / nR, i1 = (e1 - 1) / nR;
    if (right_lanes(nL, nR)) {
      const uint32_t nT = (nR + 63) / 64;
      const uint32_t r0 = kl.below((uint32_t)i0), r1 = kl.below((uint32_t)i1);
      sp.a = r0;
      sp.b = kl.has((uint32_t)i0) ? (uint32_t)((e0 - i0 * nR) / 64) : 0u;
      const uint32_t last = kl.has((uint32_t)i1) ? (uint32_t)((e1 - 1 - i1 * nR) / 64) + 1 : 0u;
      sp.items = (r1 - r0) * nT + last - sp.b;
    } else {
      const uint32_t r0 = kl.below((uint32_t)i0), r1 = kl.below((uint32_t)i1 + 1);
      sp.a = r0 / 64;
      sp.items = r1 > r0 ? ((r1 - 1) / 64 - sp.a + 1) * nR : 0u;
    }
    return sp;
  }
  uint64_t k1;
  if (blk.op != OP_UNION) {
    sp.k = kl.below((uint32_t)e0);
    k1 = kl.below((uint32_t)e1);
  } else if (!blk.same) {
    const uint32_t cols = kr.count();
    const uint64_t i0 = e0 / nR, i1 = e1 / nR;
    sp.a = kl.below((uint32_t)i0);
    sp.b = kl.has((uint32_t)i0) ? kr.below((uint32_t)(e0 - i0 * nR)) : 0u;
    const uint32_t a1 = kl.below((uint32_t)i1);
    const uint32_t b1 = kl.has((uint32_t)i1) ? kr.below((uint32_t)(e1 - i1 * nR)) : 0u;
    sp.k = 0;
    k1 = (uint64_t)(a1 - sp.a) * cols + b1 - sp.b;
  } else {
    // pairs of kept rows before pair e of all rows
    const uint64_t m = kl.count();
    auto before = [&](uint64_t e) -> uint64_t {
      if (e >= blk.count) return m ? m * (m - 1) / 2 : 0;
      uint64_t i, j;
      tri_decode(e, nL, &i, &j);
      const uint64_t a = kl.below((uint32_t)i);
      if (a + 1 >= m) return m ? m * (m - 1) / 2 : 0;
      const uint64_t first = a * m - a * (a + 1) / 2;
      if (!kl.has((uint32_t)i)) return first;
      const uint64_t b = kl.below((uint32_t)j);
      return first + (b > a + 1 ? b - (a + 1) : 0);
    };
    sp.k = before(e0);
    k1 = before(e1);
  }
  sp.items = (uint32_t)((k1 - sp.k + 63) / 64);
  return sp;
}

// Barrier between phases whose global-memory effects later phases read.  An
// instance's buffers are touched by its own workgroup only, and all waves of
// a workgroup run on one CU, so workgroup scope suffices: the barrier makes
// every store and atomic issued before it visible to every wave after it.
// (Agent scope would write back and invalidate the whole L2 at each phase.)
__device__ __forceinline__ void phase_barrier() { __syncthreads(); }


// Concatenation of 64 candidates that share one operand ("uniform") while the
// other operand varies over the 64 bit positions of the transposed tile T.
// left = false: tile = right rows, out_t(w) = OR over cuts (u, v) of w with
//                uniform(u) of T[v];
// left = true:  tile = left rows,  out_t(w) = OR over cuts (u, v) with
//                uniform(v) of T[u].
// Lane t receives the W words of candidate t.
// The guide table (gto, gtp) is the workgroup's LDS copy.
// qn: most cuts of any word (the longest word's length + 1).  From 8 words
// on, cut position q is the outer loop and the lane's W words the inner one
// (each word's read clamped to its last cut and masked after), so 24
// independent LDS reads are in flight per round of eight words instead of a
// chain of three per cut; below that the per-word loop keeps the register
// count of the 1024-thread instantiations down.
template <int W>
__device__ __forceinline__ void concat_tile(const uint64_t* T, const uint64_t* uni, const uint32_t* gto,
                                            const uint32_t* gtp, uint32_t n, uint32_t qn, bool left, uint64_t (&key)[W]) {
  const uint32_t lane = lane_id();
  if constexpr (W >= 8) {
    // eight words at a time keeps the registers of the 16- and 32-word
    // instantiations within their launch bounds
#pragma unroll
    for (int k0 = 0; k0 < W; k0 += 8) {
      uint32_t first[8], last[8], cnt[8];
      uint64_t acc[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t w = 64u * (k0 + k) + lane;
        first[k] = w < n ? gto[w] : 0u;
        cnt[k] = w < n ? gto[w + 1] - first[k] : 0u;
        last[k] = first[k] + (cnt[k] ? cnt[k] - 1 : 0u);
        acc[k] = 0;
      }
      for (uint32_t q = 0; q < qn; ++q) {
        uint32_t p[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) p[k] = gtp[min(first[k] + q, last[k])];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint32_t ui = left ? (p[k] & 0xFFFFu) : (p[k] >> 16);
          const uint32_t si = left ? (p[k] >> 16) : (p[k] & 0xFFFFu);
          const uint64_t t = T[si];
          const bool on = q < cnt[k] && ((uni[ui >> 6] >> (ui & 63)) & 1ull);
          acc[k] |= on ? t : 0ull;
        }
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) key[k0 + k] = transpose64(acc[k]);
    }
  } else {
    // four cuts of a word at a time: their reads overlap (one by one, the
    // three reads of a cut and the next cut's are a chain)
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const uint32_t w = 64u * k + lane;
      const uint32_t q0 = w < n ? gto[w] : 0u, q1 = w < n ? gto[w + 1] : 0u;
      uint64_t acc = 0;
      for (uint32_t q = q0; q < q1; q += 4) {
        uint32_t p[4];
        uint64_t t[4], u[4];
#pragma unroll
        for (int z = 0; z < 4; ++z) p[z] = gtp[min(q + z, q1 - 1)];
#pragma unroll
        for (int z = 0; z < 4; ++z) {
          const uint32_t ui = left ? (p[z] & 0xFFFFu) : (p[z] >> 16);
          t[z] = T[left ? (p[z] >> 16) : (p[z] & 0xFFFFu)];
          u[z] = uni[ui >> 6] >> (ui & 63);  // (the last cut again is harmless)
        }
#pragma unroll
        for (int z = 0; z < 4; ++z) acc |= (u[z] & 1ull) ? t[z] : 0ull;
      }
      key[k] = transpose64(acc);
    }
  }
}

// The same for output words k0 .. k0 + kN - 1 only, left in the tile out (word
// k of lane t at 64 k + t): a wave's share of a tile that several build.
template <int kN>
__device__ __forceinline__ void concat_words(const uint64_t* T, const uint64_t* uni, const uint32_t* gto,
                                             const uint32_t* gtp, uint32_t n, uint32_t qn, bool left, uint32_t k0,
                                             uint64_t* out) {
  const uint32_t lane = lane_id();
  uint32_t first[kN], last[kN], cnt[kN];
  uint64_t acc[kN];
#pragma unroll
  for (int k = 0; k < kN; ++k) {
    const uint32_t w = 64u * (k0 + k) + lane;
    first[k] = w < n ? gto[w] : 0u;
    cnt[k] = w < n ? gto[w + 1] - first[k] : 0u;
    last[k] = first[k] + (cnt[k] ? cnt[k] - 1 : 0u);
    acc[k] = 0;
  }
  for (uint32_t q = 0; q < qn; ++q) {
    uint32_t p[kN];
#pragma unroll
    for (int k = 0; k < kN; ++k) p[k] = gtp[min(first[k] + q, last[k])];
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      const uint32_t ui = left ? (p[k] & 0xFFFFu) : (p[k] >> 16);
      const uint64_t t = T[left ? (p[k] >> 16) : (p[k] & 0xFFFFu)];
      const bool on = q < cnt[k] && ((uni[ui >> 6] >> (ui & 63)) & 1ull);
      acc[k] |= on ? t : 0ull;
    }
  }
#pragma unroll
  for (int k = 0; k < kN; ++k) out[64 * (k0 + k) + lane] = transpose64(acc[k]);
}

// Words k0 .. k0 + kN - 1 of each lane's row (zeros when !have), transposed
// into the tile T.
template <int W, int kN>
__device__ __forceinline__ void stage_words(uint64_t* T, const uint64_t* rows, uint64_t row, bool have, uint32_t k0) {
  const uint32_t lane = lane_id();
  uint64_t v[kN];
#pragma unroll
  for (int k = 0; k < kN; ++k) v[k] = have ? rows[row * W + k0 + k] : 0ull;
#pragma unroll
  for (int k = 0; k < kN; ++k) T[64 * (k0 + k) + lane] = transpose64(v[k]);
}

// Constructor block k of level c, blocks in enumeration order: the characters
// at c1; else r?, r*, r.s by left cost, r+s by left cost (blocks may be
// empty).  The counts of the levels below c are final.
struct BlockList {
  const BatchDesc& d;
  const uint64_t* lcount;
  uint32_t c;
  int32_t n_cat, n_uni;
  __device__ BlockList(const BatchDesc& d_, const uint64_t* lcount_, uint32_t c_) : d(d_), lcount(lcount_), c(c_) {
    const int64_t cc = c, c1 = d.c1;
    n_cat = c == d.c1 ? 0 : (int32_t)max((int64_t)0, cc - (int64_t)d.c4 - 2 * c1 + 1);
    n_uni = c == d.c1 ? 0 : (int32_t)max((int64_t)0, (cc >= (int64_t)d.c5 ? (cc - (int64_t)d.c5) / 2 : -1) - c1 + 1);
  }
  __device__ int32_t count() const { return c == d.c1 ? 1 : 2 + n_cat + n_uni; }
  __device__ BlockD get(int32_t k) const {
    const int64_t cc = c, c1 = d.c1;
    auto lc = [&](int64_t q) -> uint64_t { return (q >= c1 && q < cc) ? lcount[q] : 0ull; };
    if (k >= count()) return BlockD{0, 0, 0, 0, 0};
    if (c == d.c1) return BlockD{OP_CHAR, 0, 0, 0, (uint64_t)d.nsigma};
    if (k == 0) return BlockD{OP_QUESTION, (uint32_t)(cc - d.c2), 0, 0, lc(cc - d.c2)};
    if (k == 1) return BlockD{OP_STAR, (uint32_t)(cc - d.c3), 0, 0, lc(cc - d.c3)};
    if (k < 2 + n_cat) {
      const int64_t L = c1 + (k - 2), R = cc - d.c4 - L;
      return BlockD{OP_CONCAT, (uint32_t)L, (uint32_t)R, 0, lc(L) * lc(R)};
    }
    const int64_t L = c1 + (k - 2 - n_cat), R = cc - d.c5 - L;
    const uint64_t x = lc(L), y = lc(R);
    return BlockD{OP_UNION, (uint32_t)L, (uint32_t)R, L == R ? 1u : 0u, L < R ? x * y : (x ? x * (x - 1) / 2 : 0)};
  }
};

// The inclusive prefix sum of v over the wave's lanes.
__device__ __forceinline__ uint64_t wave_scan(uint64_t v) {
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint64_t o = __shfl_up((unsigned long long)v, off, kWave);
    if ((int)lane_id() >= off) v += o;
  }
  return v;
}

// Decodes level index e of level c into its constructor and operands (rows),
// the level's blocks a lane each.  Called by a whole wave, every lane gets the
// answer.  lstart and lcount are the workgroup's level tables in LDS.
__device__ __forceinline__ bool decode_index(const BatchDesc& d, const uint64_t* lstart, const uint64_t* lcount,
                                             uint32_t c, uint64_t e, uint32_t* op, uint64_t* a, uint64_t* b) {
  const BlockList bl(d, lcount, c);
  const int32_t n = bl.count();
  uint64_t run = 0;
  for (int32_t k0 = 0; k0 < n; k0 += 64) {
    const BlockD blk = bl.get(k0 + (int32_t)lane_id());
    const uint64_t end = run + wave_scan(blk.count), first = end - blk.count;
    const uint64_t hit = __ballot(e >= first && e < end);
    if (hit) {
      const int at = __ffsll((unsigned long long)hit) - 1;
      const uint64_t r = e - __shfl((unsigned long long)first, at, kWave);
      const uint32_t L = (uint32_t)__shfl((int)blk.L, at, kWave), R = (uint32_t)__shfl((int)blk.R, at, kWave);
      *op = (uint32_t)__shfl((int)blk.op, at, kWave);
      const uint64_t rc = lcount[R];
      uint64_t i = r, j = 0;
      if (*op == OP_UNION && L == R)
        tri_decode(r, lcount[L], &i, &j);
      else if (*op == OP_CONCAT || *op == OP_UNION) {
        i = r / rc;
        j = r - i * rc;
      }
      *a = *op == OP_CHAR ? r : lstart[L] + i;
      *b = *op == OP_CONCAT || *op == OP_UNION ? lstart[R] + j : 0;
      return true;
    }
    run = __shfl((unsigned long long)end, kWave - 1, kWave);
  }
  return false;
}

constexpr int solver_waves(int W, uint32_t threads) { return W > 4 ? 1 : threads == 256 && W > 1 ? 3 : 4; }

// kT threads per instance (256, 512 or 1024; at most batch_max_threads(W),
// so that the per-wave operand tiles and the guide table fit the LDS):
// many waves shorten one instance's search, few let more instances share a
// CU.  The host picks kT per launch (tuned or from the batch size).
// Two launch forms.  next == nullptr: workgroup b solves instance b.
// Persistent (next != nullptr): a grid of at most the resident workgroups;
// each takes the next item from the device counter *next (zero at launch)
// and solves instance order[item] (or item itself when order is null),
// until the items run out, so the longest instances can start first
// whatever the grid size.
// Queue (qc != nullptr, with next): descs is a ring the host fills while the
// launch runs (n_inst slots, published up to qc->tail); a workgroup claims
// the next published slot by compare-and-swap on *next (zero at launch), so
// a slot is taken only once it exists and exactly once.  Every workgroup
// leaves once it has waited qc->idle_ticks without finding a slot, or when
// the host sets qc->closing; slots published after the last one left are
// found unsolved by the host and published again in its next launch.
// Registers: up to four words per language at most 128 (168 for 256 threads
// beside a full guide table, where the LDS holds three workgroups), so that
// two workgroups of 512 threads or three to four of 256 fit a compute unit
// (left alone the compiler takes 180-220, and one or two fit).
template <int W, bool kInl, uint32_t kT>
__global__ __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(solver_waves(W, kT)))) void solve_batch(const BatchDesc* descs, uint32_t n_inst, const uint32_t* order,
                                                  uint32_t* next, const QueueCtl* qc) {
  static_assert(kT >= kBatchChunk / 32 && kT <= batch_max_threads(W) && kT % 64 == 0, "one scan value per thread");
  constexpr uint32_t kIc = batch_max_ic(W), kPairs = batch_max_pairs(W);
  constexpr uint32_t kWaves = kT / 64;
  __shared__ uint64_t s_lstart[kBatchMaxCost + 2], s_lcount[kBatchMaxCost + 2];
  __shared__ uint64_t s_uniq[kBatchMaxCost + 2], s_cand[kBatchMaxCost + 2];
  __shared__ BlockD s_blk[kMaxBlocks];
  __shared__ uint64_t s_bstart[kMaxBlocks + 1];  // level index of each block's first candidate
  __shared__ uint32_t s_item0[kMaxBlocks + 1];   // each block's first work item in the current chunk
  __shared__ Span s_span[kMaxBlocks];            // and its work there
  __shared__ Marks s_mk[kBatchMaxCost + 2];      // each level's rows by constructor
  __shared__ uint64_t s_thr[4];                  // this level's first index after its characters, r?, r*, r.s
  __shared__ uint32_t s_nblk;
  __shared__ uint32_t s_nsurv, s_ans, s_rank, s_over, s_stop, s_resume, s_leave;
  __shared__ uint64_t s_total;
  __shared__ uint32_t s_bm[kWords], s_pre[kWords];
  __shared__ uint32_t s_winners;
  // a star item needs two tiles: up to two words per language each wave has
  // its own two, from four on waves pair up for the star blocks (more tiles
  // would leave room for fewer workgroups on a compute unit)
  constexpr bool kStarItems = W <= 2;
  __shared__ uint64_t s_tile[kWaves][(kStarItems ? 2 : 1) * 64 * W];
  static_assert(W < 8 || sizeof(s_tile) >= kBatchChunk * sizeof(uint16_t), "ranks of a chunk fit the tiles");
  static_assert(kBatchChunk <= 0xFFFFu, "ranks of a chunk fit 16 bits");
  __shared__ uint64_t s_uni[kWaves][W];
  __shared__ uint32_t s_gto[kIc + 1], s_gtp[kPairs], s_lo[kIc + 2];
  // From eight words on concatenation tiles are dealt apart from the other
  // items: a tile keeps its wave 20-30 us, and a small level has few.
  constexpr bool kSplitItems = W >= 8;
  __shared__ uint32_t s_cat0[kSplitItems ? kMaxBlocks + 1 : 1];  // each block's first tile in the chunk
  __shared__ uint32_t s_item;
  __shared__ uint32_t s_desc[sizeof(BatchDesc) / 4];

  for (uint32_t pass = 0;; ++pass) {
  uint32_t item;
  if (!next) {
    if (pass || blockIdx.x >= n_inst) return;
    item = blockIdx.x;
  } else if (qc) {
    if (threadIdx.x == 0) {
      uint32_t got = ~0u;
      const long long t_wait = wall_clock64();
      for (;;) {
        const uint32_t tail = __hip_atomic_load(&qc->tail, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
        const uint32_t h = __hip_atomic_load(next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (h < tail && h < n_inst) {
          if (atomicCAS(next, h, h + 1) == h) {
            got = h;
            break;
          }
          continue;  // another workgroup took it: look again
        }
        const uint32_t closing = __hip_atomic_load(&qc->closing, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        if (closing || (uint64_t)(wall_clock64() - t_wait) > qc->idle_ticks) break;
        __builtin_amdgcn_s_sleep(16);
      }
      s_item = got;
    }
    __syncthreads();
    item = s_item;
    __syncthreads();
    if (item >= n_inst) return;
  } else {
    if (threadIdx.x == 0) s_item = atomicAdd(next, 1u);
    __syncthreads();
    item = s_item;
    __syncthreads();  // read by every wave before thread 0 writes the next one
    if (item >= n_inst) return;
    if (order) item = order[item];
  }
  // The descriptor goes through LDS into scalar registers: its 90-odd words
  // are the same for every lane, but loaded as a struct by an index the
  // compiler cannot prove uniform they took that many vector registers (200 in
  // all, 100 of them spilled in the 1024-thread forms: one workgroup per
  // compute unit).
  static_assert(sizeof(BatchDesc) % 4 == 0 && sizeof(BatchDesc) / 4 <= kT, "one word per thread");
  if (threadIdx.x < sizeof(BatchDesc) / 4)
    s_desc[threadIdx.x] = reinterpret_cast<const uint32_t*>(descs + item)[threadIdx.x];
  __syncthreads();
  BatchDesc d;
  {
    uint32_t w[sizeof(BatchDesc) / 4];
#pragma unroll
    for (uint32_t i = 0; i < sizeof(BatchDesc) / 4; ++i) w[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_desc[i]);
    __builtin_memcpy(&d, w, sizeof(d));
  }
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // The dedup table starts small and grows (cleared and rebuilt from the
  // stored rows) while rows accumulate, up to the arena's slot_mask: a
  // small instance clears a few KB instead of its whole arena.
  uint64_t tmask = min(d.slot_mask, (uint64_t)1023);
  Probe probe{d.rows, d.slots, tmask, d.pmask, d.nmask, d.max_err};
  const Sink sink{d.skey, d.se, d.spos, &s_nsurv, &s_ans};

  // start: empty table, zero counters
  for (uint64_t i = tid; i < (tmask + 1) * kSlotWords<kInl>; i += kT) d.slots[i] = kEmpty;
  // guide table and words-by-length offsets into LDS (batchable instances
  // have at most batch_max_ic(W) words and batch_max_pairs(W) cuts)
  for (uint32_t i = tid; i <= d.n; i += kT) s_gto[i] = d.gt_off[i];
  for (uint32_t i = tid; i < d.n_pairs; i += kT) s_gtp[i] = d.gt_pair[i];
  for (uint32_t i = tid; i < d.max_len + 2; i += kT) s_lo[i] = d.len_off[i];
  for (uint32_t c = tid; c < kBatchMaxCost + 2; c += kT) {
    s_lstart[c] = 0;
    s_lcount[c] = 0;
    s_uniq[c] = 0;
    s_cand[c] = 0;
  }
  if (tid == 0) {
    s_total = 0;
    s_stop = STOP_NONE;
    s_resume = 0;
  }
  phase_barrier();

  uint32_t ans_cost = 0;
  uint64_t ans_e = 0;
  uint64_t ref_gen = (1ull << 36) - 2;  // inline-key references: one lower each chunk, so older ones need no reset
  const long long t_start = wall_clock64();
  for (uint32_t c = d.c1; c <= d.max_cost && s_stop == STOP_NONE; ++c) {
    if (wave == 0) {
      // constructor blocks of level c, in enumeration order, one per lane
      const BlockList bl(d, s_lcount, c);
      const int32_t n_all = bl.count();
      uint32_t nb = 0;
      uint64_t run = 0, thr[4] = {0, 0, 0, 0};
      for (int32_t k0 = 0; k0 < n_all; k0 += 64) {
        const BlockD b = bl.get(k0 + (int32_t)lane);
        const uint64_t incl = wave_scan(b.count);
        const uint64_t some = __ballot(b.count != 0);
        if (b.count) {
          const uint32_t at = nb + (uint32_t)__popcll(some & ((1ull << lane) - 1));
          s_blk[at] = b;
          s_bstart[at] = run + incl - b.count;
        }
        // ends of the constructors' index ranges
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const uint64_t mine = __ballot(b.count != 0 && (int)b.op <= t);
          if (mine) {
            const int last = 63 - __clzll((long long)mine);
            thr[t] = run + __shfl((unsigned long long)incl, last, kWave);
          }
        }
        nb += (uint32_t)__popcll(some);
        run += __shfl((unsigned long long)incl, kWave - 1, kWave);
      }
      if (lane == 0) {
        s_lstart[c] = s_total;
        s_nblk = nb;
        s_bstart[nb] = run;
        uint64_t t = 0;
        for (int q = 0; q < 4; ++q) s_thr[q] = t = thr[q] > t ? thr[q] : t;
        s_mk[c] = Marks{~0u, ~0u, ~0u, ~0u};
        // a level this large is work for the whole device: hand the instance,
        // with its lower levels stored, to the per-chunk path; so is a
        // mid-sized level of an instance that has kept its workgroup long
        // (the deep searches of a batch), while the device has room beside it
        const bool late = d.time_ticks && run > kBatchTimeMinLevel &&
                          (uint64_t)(wall_clock64() - t_start) > d.time_ticks;
        s_leave = run > d.level_max || late ? 1u : 0u;
      }
    }
    __syncthreads();
    // (s_stop is written where no wave reads it: other waves may still be at
    // the loop's condition while the blocks are built)
    if (s_leave) {
      if (tid == 0) {
        s_stop = STOP_HANDOFF;
        s_resume = c;
      }
      break;
    }
    const uint32_t nblk = s_nblk;
    const uint64_t level_total = s_bstart[nblk];
    // Chunks cover consecutive level indices [E0, E1) and may span several
    // constructor blocks, so small blocks share one round of phases.
    for (uint64_t E0 = 0; E0 < level_total && s_stop == STOP_NONE; E0 += kBatchChunk) {
      const uint64_t E1 = min(level_total, E0 + (uint64_t)kBatchChunk);
      const uint32_t len = (uint32_t)(E1 - E0);
      {
        // keep the load at most 1/2 with this chunk's survivors inserted
        const uint64_t total = s_total;
        if (2 * (total + len) > tmask + 1) {
          uint64_t cap = tmask + 1;
          while (cap < 4 * (total + len) && cap <= d.slot_mask) cap *= 2;
          tmask = min(d.slot_mask, cap - 1);
          for (uint64_t i = tid; i < (tmask + 1) * kSlotWords<kInl>; i += kT) d.slots[i] = kEmpty;
          __syncthreads();
          for (uint64_t row = tid; row < total; row += kT) {
            uint64_t key[W];
#pragma unroll
            for (int k = 0; k < W; ++k) key[k] = d.rows[row * W + k];
            table_rebuild_one<W, kInl>(d.slots, tmask, key, row);
          }
          probe.slot_mask = tmask;
          __syncthreads();
        }
      }
      --ref_gen;
      for (uint32_t i = tid; i < (len + 31) / 32; i += kT) s_bm[i] = 0;
      if (wave == 0) {
        if (lane == 0) {
          s_nsurv = 0;
          s_ans = ~0u;
          s_rank = ~0u;
          s_over = ~0u;
        }
        // each block's work in this chunk, a block per lane
        uint32_t run = 0, run_cat = 0;
        for (uint32_t b0 = 0; b0 < nblk; b0 += 64) {
          const uint32_t bi = b0 + lane;
          Span sp{0, 0, 0, 0};
          if (bi < nblk) {
            const uint64_t bs = s_bstart[bi], be = s_bstart[bi + 1];
            const BlockD blk = s_blk[bi];
            if (be > E0 && bs < E1) {
              const uint32_t nL = blk.op == OP_CHAR ? d.nsigma : (uint32_t)s_lcount[blk.L], nR = (uint32_t)s_lcount[blk.R];
              const Marks mr = s_mk[blk.R];
              sp = block_span(blk, max(E0, bs) - bs, min(E1, be) - bs, nL, nR, left_kept(blk.op, s_mk[blk.L], nL),
                              Kept{mr.q, mr.s, nR});
            }
            s_span[bi] = sp;
          }
          const bool apart = bi < nblk && ((!kStarItems && s_blk[bi].op == OP_STAR) ||
                                           (kSplitItems && s_blk[bi].op == OP_CONCAT));
          // (both prefixes in one scan: items in the low half, tiles above;
          // a chunk has fewer than 2^31 of either)
          const uint64_t dealt = apart ? (s_blk[bi].op == OP_CONCAT ? (uint64_t)sp.items << 32 : 0ull) : sp.items;
          const uint64_t incl = wave_scan(dealt);
          if (bi < nblk) {
            s_item0[bi] = run + (uint32_t)(incl - dealt);
            if constexpr (kSplitItems) s_cat0[bi] = run_cat + (uint32_t)((incl - dealt) >> 32);
          }
          const uint64_t all = __shfl((unsigned long long)incl, kWave - 1, kWave);
          run += (uint32_t)all;
          run_cat += (uint32_t)(all >> 32);
        }
        if (lane == 0) {
          s_item0[nblk] = run;
          if constexpr (kSplitItems) s_cat0[nblk] = run_cat;
        }
      }
      __syncthreads();
      // Star blocks first, one at a time, where they pair the waves: they
      // need the workgroup barriers around them.
      if constexpr (!kStarItems)
      for (uint32_t bi = 0; bi < nblk; ++bi) {
        const uint64_t bs = s_bstart[bi], be = s_bstart[bi + 1];
        if (be <= E0) continue;
        if (bs >= E1) break;
        const BlockD blk = s_blk[bi];
        if (blk.op != OP_STAR) continue;
        const uint64_t lst = s_lstart[blk.L];
        // block-local candidate range of this chunk; candidate e of the block
        // has chunk-relative index bs + e - E0
        const uint64_t e0 = max(E0, bs) - bs, e1 = min(E1, be) - bs;
        const uint64_t rel0 = bs - E0;  // modulo 2^64: rel0 + e >= 0 for e >= e0
        // r* for 64 rows per wave pair: the even wave of each pair owns
        // the pair's two tiles (Xt = its own, Yt = its partner's), so
        // kWaves/2 groups of rows run at once with wave-level syncs only.
        // The workgroup barriers around the block keep the partner's tile
        // out of the neighbouring blocks' per-wave use.
        __syncthreads();
        if constexpr (kSplitItems) {
          // few groups: four waves share each, every wave staging its words
          // and taking its share of the words of each length
          constexpr uint32_t kGroups = kWaves / 4;
          const Span sp = s_span[bi];
          if (sp.items <= kGroups) {
            constexpr int kPart = W / 4;
            const uint32_t slot = wave / 4, part = wave % 4;
            const uint32_t k_lo = part * kPart;
            uint64_t* Xt = s_tile[4 * slot];
            uint64_t* Yt = s_tile[4 * slot + 1];
            uint64_t* K = s_tile[4 * slot + 2];
            const Kept kl = left_kept(OP_STAR, s_mk[blk.L], (uint32_t)s_lcount[blk.L]);
            const bool have = slot < sp.items;
            const uint32_t kk = (uint32_t)sp.k + 64 * slot + lane;
            const uint64_t e = have && kk < kl.count() ? kl.row(kk) : e1;
            if (have) {
              stage_words<W, kPart>(Xt, d.rows, lst + e, e < e1, k_lo);
#pragma unroll
              for (int k = 0; k < kPart; ++k) Yt[64 * (k_lo + k) + lane] = (k_lo + k == 0 && lane == 0) ? ~0ull : 0ull;
            }
            __syncthreads();
            for (uint32_t l = 1; l <= d.max_len; ++l) {
              if (have) {
                const uint32_t lo = s_lo[l], hi = s_lo[l + 1];
                for (uint32_t w = lo + lane + 64 * part; w < hi; w += 256)
                  Yt[w] = star_fold(Xt, Yt, s_gtp, s_gto[w], l);
              }
              __syncthreads();
            }
            if (have) {
#pragma unroll
              for (int k = 0; k < kPart; ++k) K[64 * (k_lo + k) + lane] = transpose64(Yt[64 * (k_lo + k) + lane]);
            }
            __syncthreads();
            if (have && part == 0) {
              uint64_t key[W];
#pragma unroll
              for (int k = 0; k < W; ++k) key[k] = K[64 * k + lane];
              filter_emit<W, kInl>(probe, sink, e >= e0 && e < e1, false, key, (uint32_t)(rel0 + e));
            }
            __syncthreads();
            continue;
          }
        }
        if ((wave & 1u) == 0) {
          uint64_t* Xt = s_tile[wave];
          uint64_t* Yt = s_tile[wave + 1];
          constexpr uint32_t kPairs = kWaves / 2;
          const Kept kl = left_kept(OP_STAR, s_mk[blk.L], (uint32_t)s_lcount[blk.L]);
          const Span sp = s_span[bi];
          for (uint32_t g = wave >> 1; g < sp.items; g += kPairs) {
            const uint32_t kk = (uint32_t)sp.k + 64 * g + lane;
            const uint64_t e = kk < kl.count() ? kl.row(kk) : e1;
#pragma unroll
            for (int k = 0; k < W; ++k) {
              const uint64_t v = (e < e1) ? d.rows[(lst + e) * W + k] : 0ull;
              Xt[64 * k + lane] = transpose64(v);
            }
            for (uint32_t w = lane; w < 64u * W; w += 64) Yt[w] = (w == 0) ? ~0ull : 0ull;
            wave_sync_lds();
            // Y(eps) = 1; by increasing length, Y(w) = OR over cuts w = u v
            // with u non-empty of X(u) & Y(v) (v is shorter)
            for (uint32_t l = 1; l <= d.max_len; ++l) {
              const uint32_t lo = s_lo[l], hi = s_lo[l + 1];
              for (uint32_t w = lo + lane; w < hi; w += 64) {
                // a word of length l has cuts 0..l; cut 0 has u = eps
                Yt[w] = star_fold(Xt, Yt, s_gtp, s_gto[w], l);
              }
              wave_sync_lds();
            }
            uint64_t key[W];
#pragma unroll
            for (int k = 0; k < W; ++k) key[k] = transpose64(Yt[64 * k + lane]);
            filter_emit<W, kInl>(probe, sink, e >= e0 && e < e1, false, key, (uint32_t)(rel0 + e));
            wave_sync_lds();  // the tiles are rewritten by the next group
          }
        }
        __syncthreads();
      }
      // Every other block's work items (64 consecutive candidates, or one
      // concatenation tile) are dealt to the waves together, so a chunk that
      // spans many small blocks keeps every wave busy.
      if constexpr (kSplitItems) {
        constexpr uint32_t kGroups = kWaves / 4;
        const uint32_t n_cat = s_cat0[nblk];
        // four waves share a tile where that takes less time: a shared round
        // is about a third of a wave's own (16 words: 9 against 28 us)
        const bool shared = (n_cat + kGroups - 1) / kGroups < 3 * ((n_cat + kWaves - 1) / kWaves);
        const uint32_t step = shared ? kGroups : kWaves, slot = shared ? wave / 4 : wave, part = shared ? wave % 4 : 0;
        constexpr int kPart = W / 4;
        uint64_t* T = s_tile[shared ? 4 * slot : wave];
        uint64_t* K = s_tile[shared ? 4 * slot + 1 : wave];  // the tile's candidates, word by word
        uint64_t* U = s_uni[shared ? 4 * slot : wave];
        uint32_t bi = 0;
        // (every wave takes every round: workgroup barriers inside when shared)
        for (uint32_t base = 0; base < n_cat; base += step) {
          const uint32_t it = base + slot;
          const bool have = it < n_cat;
          uint64_t e = 0;
          bool valid = false, left = false;
          uint32_t rel = 0;
          if (have) {
            while (s_cat0[bi + 1] <= it) ++bi;
            const uint32_t li = it - s_cat0[bi];
            const uint64_t bs = s_bstart[bi], be = s_bstart[bi + 1];
            const BlockD blk = s_blk[bi];
            const uint64_t lst = s_lstart[blk.L], rst = s_lstart[blk.R];
            const uint32_t nL = (uint32_t)s_lcount[blk.L], nR = (uint32_t)s_lcount[blk.R];
            const uint64_t e0 = max(E0, bs) - bs, e1 = min(E1, be) - bs;
            const Span sp = s_span[bi];
            const Kept kl = left_kept(OP_CONCAT, s_mk[blk.L], nL);
            uint64_t row, urow;  // this lane's row of the tile, the uniform row
            if (right_lanes(nL, nR)) {
              const uint32_t nT = (nR + 63) / 64, f = sp.b + li;
              const uint64_t i = kl.row(sp.a + f / nT), j = 64 * (f % nT) + lane;
              valid = j < nR;
              row = rst + j;
              urow = lst + i;
              e = i * nR + j;
            } else {
              left = true;
              const uint32_t kk = 64 * (sp.a + li / nR) + lane, j = li % nR;
              valid = kk < kl.count();
              const uint64_t i = valid ? kl.row(kk) : 0ull;
              row = lst + i;
              urow = rst + j;
              e = i * nR + j;
            }
            for (uint32_t k0 = shared ? part * kPart : 0; k0 < (shared ? (part + 1) * kPart : (uint32_t)W); k0 += kPart)
              stage_words<W, kPart>(T, d.rows, row, valid, k0);
            if (part == 0 && lane < (uint32_t)W) U[lane] = d.rows[urow * W + lane];
            valid = valid && e >= e0 && e < e1;
            rel = (uint32_t)(bs - E0 + e);
          }
          if (shared)
            __syncthreads();
          else
            wave_sync_lds();
          if (shared) {
            if (have) concat_words<kPart>(T, U, s_gto, s_gtp, d.n, d.max_len + 1, left, part * kPart, K);
            __syncthreads();
          }
          if (have && part == 0) {
            uint64_t key[W];
            if (shared) {
#pragma unroll
              for (int k = 0; k < W; ++k) key[k] = K[64 * k + lane];
            } else {
              concat_tile<W>(T, U, s_gto, s_gtp, d.n, d.max_len + 1, left, key);
            }
            filter_emit<W, kInl>(probe, sink, valid, false, key, rel);
          }
          if (!shared) wave_sync_lds();  // the tile is rewritten in the next round
        }
      }
      {
        const uint32_t n_items = s_item0[nblk];
        uint32_t bi = 0;
        for (uint32_t it = wave; it < n_items; it += kWaves) {
          while (s_item0[bi + 1] <= it) ++bi;  // blocks with no items here are skipped
          const uint32_t li = it - s_item0[bi];
          const uint64_t bs = s_bstart[bi], be = s_bstart[bi + 1];
          const BlockD blk = s_blk[bi];
          const uint64_t lst = s_lstart[blk.L], lct = s_lcount[blk.L];
          const uint64_t rst = s_lstart[blk.R], rct = s_lcount[blk.R];
          const uint64_t e0 = max(E0, bs) - bs, e1 = min(E1, be) - bs;
          const uint64_t rel0 = bs - E0;
          const Span sp = s_span[bi];
          const Kept kl = left_kept(blk.op, s_mk[blk.L], blk.op == OP_CHAR ? d.nsigma : (uint32_t)lct);
          if (blk.op != OP_CONCAT) {
            // kept candidate 64 li + lane of the block's in this chunk
            uint64_t e = ~0ull, i = 0, j = 0;
            if (blk.op != OP_UNION) {
              const uint32_t kk = (uint32_t)sp.k + 64 * li + lane;
              if (kk < kl.count()) e = kl.row(kk);
            } else if (blk.same) {
              const uint64_t m = kl.count(), kk = sp.k + 64 * li + lane;
              if (kk < m * (m - 1) / 2) {
                tri_decode(kk, m, &i, &j);
                i = kl.row((uint32_t)i);
                j = kl.row((uint32_t)j);
                e = i * lct - i * (i + 1) / 2 + (j - i - 1);
              }
            } else {
              const Marks mr = s_mk[blk.R];
              const Kept kr{mr.q, mr.s, (uint32_t)rct};
              const uint32_t cols = kr.count(), t = sp.b + 64 * li + lane;
              const uint32_t ai = sp.a + t / cols;
              if (ai < kl.count()) {
                i = kl.row(ai);
                j = kr.row(t - (ai - sp.a) * cols);
                e = i * rct + j;
              }
            }
            const bool valid = e >= e0 && e < e1;
            uint64_t key[W];
            bool dup = false;
            if (kStarItems && blk.op == OP_STAR) {
              // r* of 64 rows (as for the paired waves above)
              uint64_t* Xt = s_tile[wave];
              uint64_t* Yt = s_tile[wave] + 64 * W;
#pragma unroll
              for (int k = 0; k < W; ++k) {
                Xt[64 * k + lane] = transpose64(valid ? d.rows[(lst + e) * W + k] : 0ull);
                Yt[64 * k + lane] = (k == 0 && lane == 0) ? ~0ull : 0ull;
              }
              wave_sync_lds();
              for (uint32_t l = 1; l <= d.max_len; ++l) {
                const uint32_t lo = s_lo[l], hi = s_lo[l + 1];
                for (uint32_t w = lo + lane; w < hi; w += 64) Yt[w] = star_fold(Xt, Yt, s_gtp, s_gto[w], l);
                wave_sync_lds();
              }
#pragma unroll
              for (int k = 0; k < W; ++k) key[k] = transpose64(Yt[64 * k + lane]);
              wave_sync_lds();  // the tiles are rewritten by the next item
            } else if (blk.op == OP_CHAR) {
              const int idx = valid ? d.char_index[e] : -1;
#pragma unroll
              for (int k = 0; k < W; ++k) key[k] = (idx >= 0 && (idx >> 6) == k) ? (1ull << (idx & 63)) : 0ull;
            } else if (blk.op == OP_QUESTION) {
              const uint64_t* src = d.rows + (lst + (valid ? e : 0)) * W;
#pragma unroll
              for (int k = 0; k < W; ++k) key[k] = valid ? src[k] : 0ull;
              dup = (key[0] & 1ull) != 0;
              key[0] |= 1ull;
            } else {
              const uint64_t* x = d.rows + (lst + i) * W;
              const uint64_t* y = d.rows + (rst + j) * W;
              bool eqx = true, eqy = true;
#pragma unroll
              for (int k = 0; k < W; ++k) {
                const uint64_t xv = valid ? x[k] : 0ull, yv = valid ? y[k] : 0ull;
                key[k] = xv | yv;
                eqx = eqx && key[k] == xv;
                eqy = eqy && key[k] == yv;
              }
              dup = eqx || eqy;
            }
            filter_emit<W, kInl>(probe, sink, valid, dup, key, (uint32_t)(rel0 + e));
            continue;
          }
          if constexpr (!kSplitItems) {
          uint64_t* T = s_tile[wave];
          uint64_t* U = s_uni[wave];
          const uint32_t nL = (uint32_t)lct, nR = (uint32_t)rct;
          if (right_lanes(nL, nR)) {
            // right operands across the lanes: the block's tiles, row by kept
            // left row, from the one at (sp.a, sp.b)
            const uint32_t nT = (nR + 63) / 64, f = sp.b + li;
            const uint64_t i = kl.row(sp.a + f / nT);
            const uint32_t jt = f % nT;
            const uint64_t jr = 64 * jt + lane;
#pragma unroll
            for (int k = 0; k < W; ++k)
              T[64 * k + lane] = transpose64(jr < nR ? d.rows[(rst + jr) * W + k] : 0ull);
            if (lane < (uint32_t)W) U[lane] = d.rows[(lst + i) * W + lane];
            wave_sync_lds();
            uint64_t key[W];
            concat_tile<W>(T, U, s_gto, s_gtp, d.n, d.max_len + 1, false, key);
            const uint64_t e = i * nR + jr;
            filter_emit<W, kInl>(probe, sink, jr < nR && e >= e0 && e < e1, false, key, (uint32_t)(rel0 + e));
            wave_sync_lds();
          } else {
            // left operands across the lanes (the right level is small):
            // item li is (tile of kept left rows, right operand j)
            const uint32_t kk = 64 * (sp.a + li / nR) + lane, j = li % nR;
            const uint64_t ir = kk < kl.count() ? kl.row(kk) : nL;
            const uint64_t ec = ir * nR + j;
            if (!__any(ir < nL && ec >= e0 && ec < e1)) continue;
#pragma unroll
            for (int k = 0; k < W; ++k)
              T[64 * k + lane] = transpose64(ir < nL ? d.rows[(lst + ir) * W + k] : 0ull);
            if (lane < (uint32_t)W) U[lane] = d.rows[(rst + j) * W + lane];
            wave_sync_lds();
            uint64_t key[W];
            concat_tile<W>(T, U, s_gto, s_gtp, d.n, d.max_len + 1, true, key);
            const uint64_t e = ir * nR + j;
            filter_emit<W, kInl>(probe, sink, ir < nL && e >= e0 && e < e1, false, key, (uint32_t)(rel0 + e));
            wave_sync_lds();
          }
          }
        }
      }
      phase_barrier();

        // ---- insert survivors; winners' bits end up set (a survivor that
        // takes its slot toggles its bit on, one that is displaced has its
        // bit toggled off)
        const uint32_t ns = s_nsurv;
        for (uint32_t sid = tid; sid < ns; sid += kT) {
          const uint64_t h = d.spos[sid];
          const uint32_t e = d.se[sid];
          const uint64_t mine = kInl ? chunk_ref(ref_gen, e) : new_ref(e, sid);
          uint64_t old;
          const uint64_t pos = table_insert<W, kInl>(d.slots, tmask, d.rows, d.skey, sid, h, mine, &old);
          if constexpr (!kInl) d.spos[sid] = spos_pack(pos, h);
          if (mine < old) {
            atomicXor(&s_bm[e >> 5], 1u << (e & 31));
            uint32_t oe;
            if (displaced_survivor<kInl>(old, ref_gen, &oe)) atomicXor(&s_bm[oe >> 5], 1u << (oe & 31));
          }
        }
        phase_barrier();

        // ---- ranks, ordered append, accounting
        const uint32_t words = (len + 31) / 32;
        if (wave == 0) {
          const uint32_t t = wave_popc_scan<kWords / 64>(s_bm, s_pre, words);
          if (lane == 0) s_winners = t;
        }
        __syncthreads();
        const uint32_t winners = s_winners;
        const uint64_t total = s_total;
        const uint64_t room = d.row_cap > total ? d.row_cap - total : 0;
        const uint64_t alloc_room = d.rows_alloc > total ? d.rows_alloc - total : 0;
        const uint32_t ans = s_ans;
        // constructor boundaries of the level that lie in this chunk
        if (tid < 4 && s_thr[tid] >= E0 && s_thr[tid] < E1) {
          const uint32_t r = (uint32_t)(s_thr[tid] - E0);
          (&s_mk[c].q)[tid] = (uint32_t)s_lcount[c] + s_pre[r >> 5] + (uint32_t)__popc(s_bm[r >> 5] & ((1u << (r & 31)) - 1));
        }
        // each survivor's rank among the stored rows (kNotStored: not stored)
        constexpr uint32_t kNotStored = 0xFFFFu;  // ranks are below kBatchChunk
        auto place = [&](uint32_t sid, uint32_t e) -> uint32_t {
          const uint32_t word = s_bm[e >> 5];
          const uint32_t bit = 1u << (e & 31);
          if (!(word & bit)) return kNotStored;
          const uint32_t rank = s_pre[e >> 5] + (uint32_t)__popc(word & (bit - 1));
          if (e == ans) s_rank = rank;
          if (ans != ~0u && e >= ans) return kNotStored;
          if (rank < room && rank < alloc_room) return rank;
          if (rank == room) s_over = e;
          return kNotStored;
        };
        if constexpr (W < 8) {
          for (uint32_t sid = tid; sid < ns; sid += kT) {
            const uint32_t e = d.se[sid];
            const uint32_t rank = place(sid, e);
            if (rank == kNotStored) continue;
            const uint64_t row = total + rank;
#pragma unroll
            for (int k = 0; k < W; ++k) d.rows[row * W + k] = d.skey[(uint64_t)sid * W + k];
            d.aux[row] = E0 + e;
            if constexpr (!kInl) table_publish(d.slots, d.spos[sid], row);
          }
        } else {
          // wide rows: ranks into LDS (over the tiles, idle in this phase),
          // then W consecutive lanes copy one row, whole rows per wave
          uint16_t* s_dst = reinterpret_cast<uint16_t*>(&s_tile[0][0]);
          for (uint32_t sid = tid; sid < ns; sid += kT) s_dst[sid] = (uint16_t)place(sid, d.se[sid]);
          __syncthreads();
          constexpr uint32_t kPer = kT / W;  // rows per round
          const uint32_t k = tid % W;
          for (uint32_t q = tid / W; q < ns; q += kPer) {
            const uint32_t rank = s_dst[q];
            if (rank == kNotStored) continue;
            const uint64_t row = total + rank;
            d.rows[row * W + k] = d.skey[(uint64_t)q * W + k];
            if (k == 0) {
              d.aux[row] = E0 + d.se[q];
              table_publish(d.slots, d.spos[q], row);
            }
          }
        }
        __syncthreads();
        if (tid == 0) {
          uint64_t stored, du, dc;
          uint32_t stop = STOP_NONE;
          if (ans != ~0u) {
            if ((uint64_t)s_rank > room) {
              stored = room;
              dc = (uint64_t)s_over + 1;
              du = room;
              stop = STOP_OOM;
            } else {
              stored = s_rank;
              dc = (uint64_t)ans + 1;
              du = (uint64_t)s_rank + 1;
              stop = STOP_ANSWER;
              ans_cost = c;
              ans_e = E0 + ans;
            }
          } else if ((uint64_t)winners > room) {
            stored = room;
            dc = (uint64_t)s_over + 1;
            du = room;
            stop = STOP_OOM;
          } else {
            stored = winners;
            dc = len;
            du = winners;
          }
          if (stored > alloc_room) {
            stop = STOP_CAPACITY;
          } else {
            s_total = total + stored;
            s_lcount[c] += stored;
            s_uniq[c] += du;
            s_cand[c] += dc;
          }
          s_stop = stop;
        }
        phase_barrier();
    }
    // boundaries at the level's end
    if (tid < 4 && (&s_mk[c].q)[tid] == ~0u) (&s_mk[c].q)[tid] = (uint32_t)s_lcount[c];
    __syncthreads();  // every wave is done with this level's blocks
  }

  // ---- results, written straight to the instance's host-visible buffers
  if (wave == 0) {
    // The answer's expression tree (A12): the answer candidate, then every
    // stored row below it, each decoded from its back-pointer (level index)
    // with the block structure of its level, by one wave.  Trees have at most
    // one node per unit of cost; a count of 0 tells the host to decode from
    // the back-pointers itself.
    uint32_t k = 0;
    if (s_stop == STOP_ANSWER) {
      uint64_t* stk = s_tile[0];  // free after the search
      uint32_t sp = 0;
      bool ok = true;
      auto node = [&](uint64_t row, uint32_t c, uint64_t e) {
        uint32_t op = 0;
        uint64_t a = 0, b = 0;
        if (k >= kTreeMax || sp + 2 > 64 || !decode_index(d, s_lstart, s_lcount, c, e, &op, &a, &b)) {
          ok = false;
          return;
        }
        if (lane == 0) {
          uint64_t* o = d.htree + 1 + 4 * k;
          o[0] = row;
          o[1] = op;
          o[2] = a;
          o[3] = b;
          if (op != OP_CHAR) stk[sp] = a;
          if (op == OP_CONCAT || op == OP_UNION) stk[sp + 1] = b;
        }
        ++k;
        if (op != OP_CHAR) ++sp;
        if (op == OP_CONCAT || op == OP_UNION) ++sp;
        wave_sync_lds();
      };
      node(~0ull, (uint32_t)__shfl((int)ans_cost, 0, kWave), __shfl((unsigned long long)ans_e, 0, kWave));
      while (ok && sp) {
        const uint64_t row = stk[--sp];
        const bool mine = lane >= d.c1 && lane <= d.max_cost && row >= s_lstart[lane] &&
                          row < s_lstart[lane] + s_lcount[lane];
        const uint64_t at = __ballot(mine);
        if (!at) {
          ok = false;
          break;
        }
        node(row, (uint32_t)__ffsll((unsigned long long)at) - 1, d.aux[row]);
      }
      if (!ok) k = 0;
    }
    if (lane == 0) {
      d.htree[0] = k;
      d.hst->total_rows = s_total;
      d.hst->row_cap = d.row_cap;
      d.hst->stop = s_stop;
      d.hst->answer_cost = ans_cost;
      d.hst->answer_e = ans_e;
      d.hst->resume_level = s_resume;
    }
  }
  const uint32_t L = d.max_cost + 2;
  for (uint32_t i = tid; i < L; i += kT) {
    d.hlev[i] = s_lcount[i];
    d.hlev[L + i] = s_uniq[i];
    d.hlev[2 * L + i] = s_cand[i];
  }
  // Publish: every result above, and the rows and table in device memory,
  // become visible to the host and to other kernels before the flag does,
  // so the host may hand the instance to the per-chunk path while the rest
  // of the launch still runs.
  __threadfence_system();
  __syncthreads();
  if (tid == 0) __hip_atomic_store(&d.hst->done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }  // next instance
}

// Writes up to kDescPack descriptors, passed by value, to device memory (the
// allocation-free entry point sets its descriptors up with no copy API).
struct DescPack {
  BatchDesc d[kDescPack];
  uint32_t n;
};
__global__ void put_descs(BatchDesc* dst, DescPack p) {
  static_assert(sizeof(BatchDesc) % 8 == 0, "descriptors copy as 64-bit words");
  const uint32_t words = p.n * (uint32_t)(sizeof(BatchDesc) / 8);
  const uint64_t* src = reinterpret_cast<const uint64_t*>(p.d);
  for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) reinterpret_cast<uint64_t*>(dst)[i] = src[i];
}

// Puts the work counters of the persistent launches back to zero (a kernel,
// so that it can sit in a captured graph).
__global__ void reset_counters(uint32_t* c, uint32_t n) {
  if (threadIdx.x < n) c[threadIdx.x] = 0;
}

}  // namespace

hipError_t set_hash_mask_batch(uint64_t mask) {
  return hipMemcpyToSymbol(HIP_SYMBOL(g_hash_mask), &mask, sizeof(mask));
}

hipError_t launch_solve_batch(int W, bool inl, uint32_t threads, const BatchDesc* d_descs, uint32_t n,
                              hipStream_t s, const uint32_t* order, uint32_t* next, uint32_t grid,
                              const QueueCtl* qc) {
  if (n == 0) return hipSuccess;
  if (!next) grid = n;
  if (qc && !next) return hipErrorInvalidValue;
  if (grid == 0 || (grid > n && !qc)) return hipErrorInvalidValue;
#define REI_BATCH_L(WW, II, TT)                                                                          \
  launch_timed(solve_batch<WW, II, std::min(TT, batch_max_threads(WW))>, dim3(grid), dim3(TT), 0, s, d_descs, n, \
               order, next, qc)
#define REI_BATCH_T(WW, II)                                              \
  if (threads > batch_max_threads(WW)) return hipErrorInvalidValue;      \
  switch (threads) {                                                     \
    case 256: REI_BATCH_L(WW, II, 256u); break;                          \
    case 512: REI_BATCH_L(WW, II, 512u); break;                          \
    case 1024: REI_BATCH_L(WW, II, 1024u); break;                        \
    default: return hipErrorInvalidValue;                                \
  }
  switch (W) {
    case 1:
      if (inl) {
        REI_BATCH_T(1, true)
      } else {
        REI_BATCH_T(1, false)
      }
      break;
    case 2: REI_BATCH_T(2, false) break;
    case 4: REI_BATCH_T(4, false) break;
    case 8: REI_BATCH_T(8, false) break;
    case 16: REI_BATCH_T(16, false) break;
    case 32: REI_BATCH_T(32, false) break;
    default: return hipErrorInvalidValue;
  }
#undef REI_BATCH_L
#undef REI_BATCH_T
  return hipGetLastError();
}

hipError_t batch_resident(int W, bool inl, uint32_t threads, uint32_t* per_cu) {
  int nb = 0;
  hipError_t e = hipErrorInvalidValue;
#define REI_OCC_L(WW, II, TT)                                                                          \
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, solve_batch<WW, II, std::min(TT, batch_max_threads(WW))>, \
                                                   (int)TT, 0)
#define REI_OCC(WW, II)                                              \
  if (threads > batch_max_threads(WW)) return hipErrorInvalidValue;  \
  switch (threads) {                                                 \
    case 256: REI_OCC_L(WW, II, 256u); break;                        \
    case 512: REI_OCC_L(WW, II, 512u); break;                        \
    case 1024: REI_OCC_L(WW, II, 1024u); break;                      \
    default: return hipErrorInvalidValue;                            \
  }
  switch (W) {
    case 1:
      if (inl) {
        REI_OCC(1, true)
      } else {
        REI_OCC(1, false)
      }
      break;
    case 2: REI_OCC(2, false) break;
    case 4: REI_OCC(4, false) break;
    case 8: REI_OCC(8, false) break;
    case 16: REI_OCC(16, false) break;
    case 32: REI_OCC(32, false) break;
    default: return hipErrorInvalidValue;
  }
#undef REI_OCC_L
#undef REI_OCC
  if (e == hipSuccess) *per_cu = (uint32_t)std::max(nb, 1);
  return e;
}

hipError_t launch_put_descs(BatchDesc* dst, const BatchDesc* src, uint32_t n, hipStream_t s) {
  for (uint32_t k = 0; k < n; k += kDescPack) {
    DescPack p;
    p.n = std::min<uint32_t>(kDescPack, n - k);
    for (uint32_t i = 0; i < p.n; ++i) p.d[i] = src[k + i];
    hipLaunchKernelGGL(put_descs, dim3(1), dim3(256), 0, s, dst + k, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t static_scratch(void** out) {
  constexpr int kDevices = 64;
  static std::mutex mu;
  static void* addr[kDevices] = {nullptr};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *out = addr[dev];
  return hipSuccess;
}

hipError_t launch_reset_counters(uint32_t* c, uint32_t n, hipStream_t s) {
  if (n == 0 || n > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(reset_counters, dim3(1), dim3(64), 0, s, c, n);
  return hipGetLastError();
}

}  // namespace rei
