// Device kernels of the REI search for CDNA4 (gfx950), wave64.
//
// One chunk of candidates (a contiguous range of level indices, spanning one
// or more constructor blocks of a cost level) goes through:
//   gen_*     build each candidate's language (characteristic sequence over
//             ic, W 64-bit words) and probe the dedup table read-only; a
//             candidate whose language is not yet stored is a survivor and
//             is appended with its chunk-relative index; precise survivors
//             lower ctrl->answer_e (Algorithm 2: uniqueness, then precision);
//   insert    survivors claim table slots; equal languages meet in one slot
//             and keep the smallest enumeration index (deterministic
//             atomicMin), so the first occurrence wins; winners' bits end up
//             set in a per-chunk bitmap indexed by enumeration index;
//   scan      exclusive prefix of the bitmap popcounts = rank of each winner
//             in enumeration order;
//   compact   winners before the answer are appended to the level in rank
//             order (new languages wait in temporary storage and only the
//             unique ones enter the cache: Sec. 3, GPU language cache).
#include <algorithm>

#include <cstdlib>

#include "device_common.h"

namespace rei {

namespace {

// Probe the table and append survivors (see filter_emit in device_common.h).
// In OnTheFly mode (Sec. 3) the cache is full: no probe and no survivors,
// only the precision test (a known duplicate equals a stored language, which
// is not precise, or the search would have stopped there).
template <int W, bool kInl>
__device__ __forceinline__ void filter_emit(const GenArgs& a, bool valid, bool known_dup,
                                            const uint64_t (&key)[W], uint32_t e_rel) {
  if (a.st->otf) {
    if (valid && !known_dup && misclassified<W>(a.pmask, a.nmask, key) <= (int)a.max_err)
      atomicMin(&a.ctrl->answer_e, e_rel);
    return;
  }
  const Probe p{a.rows, a.slots, a.slot_mask, a.pmask, a.nmask, a.max_err};
  const Sink k{a.skey, a.se, a.spos, &a.ctrl->n_surv, &a.ctrl->answer_e};
  filter_emit<W, kInl>(p, k, valid, known_dup, key, e_rel);
}

// One wave's own range of survivor slots: the large generators append there,
// so that no counter is shared.  (One counter for the whole launch cost a
// returning atomic on one address per wave iteration with a survivor, 4-7 ns
// each one after the other: 835 us per 16.7 M-candidate gen_concat launch
// and 545 us per gen_union launch of one-word languages, 58 infixes.)
struct Region {
  uint32_t base, n;
};

template <int W, bool kInl>
__device__ __forceinline__ void region_emit(const GenArgs& a, Region& r, bool valid, bool known_dup,
                                            const uint64_t (&key)[W], uint32_t e_rel) {
  if (a.st->otf) {
    if (valid && !known_dup && misclassified<W>(a.pmask, a.nmask, key) <= (int)a.max_err)
      atomicMin(&a.ctrl->answer_e, e_rel);
    return;
  }
  bool surv = false;
  uint64_t h = 0;
  if (valid && !known_dup) {
    h = hash_key<W>(key);
    surv = !table_find<W, kInl>(a.slots, a.slot_mask, a.rows, key, h);
  }
  const uint64_t m = __ballot(surv);
  if (surv) {
    const uint32_t sid = r.base + r.n + (uint32_t)__popcll(m & ((1ull << lane_id()) - 1));
    uint64_t* dst = a.skey + (uint64_t)sid * W;
#pragma unroll
    for (int k = 0; k < W; ++k) dst[k] = key[k];
    a.se[sid] = e_rel;
    a.spos[sid] = h;
    if (misclassified<W>(a.pmask, a.nmask, key) <= (int)a.max_err) atomicMin(&a.ctrl->answer_e, e_rel);
  }
  r.n += (uint32_t)__popcll(m);
}

// Records the wave's range (every wave of a launch with ranges does).
__device__ __forceinline__ void region_close(const GenArgs& a, uint32_t id, const Region& r) {
  if (lane_id() == 0) a.reg[id] = make_uint2(r.base, r.n);
}

// ---- generators -----------------------------------------------------------

// A wave of the one-candidate-per-lane generators takes a.per_wave * 64
// consecutive candidates.
template <int W, bool kInl>
__global__ __launch_bounds__(256) void gen_char(GenArgs a) {
  if (a.st->stop) return;
  const uint32_t wave = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  Region rg{a.slot0 + wave * a.per_wave * 64, 0};
  const uint64_t w0 = a.e0 + (uint64_t)wave * a.per_wave * 64;
  for (uint32_t it = 0; it < a.per_wave && w0 + 64 * it < a.e1; ++it) {
    const uint64_t e = w0 + 64 * it + lane;
    const bool valid = e < a.e1;
    uint64_t key[W];
    const int idx = valid ? a.char_index[e] : -1;
#pragma unroll
    for (int k = 0; k < W; ++k) key[k] = (idx >= 0 && (idx >> 6) == k) ? (1ull << (idx & 63)) : 0ull;
    region_emit<W, kInl>(a, rg, valid, false, key, (uint32_t)(e - a.e0) + a.rel0);
  }
  region_close(a, a.reg0 + wave, rg);
}

// r? = eps + r; eps is word 0 of ic (shortlex puts the empty word first).
template <int W, bool kInl>
__global__ __launch_bounds__(256) void gen_question(GenArgs a) {
  if (a.st->stop) return;
  const uint32_t wave = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  Region rg{a.slot0 + wave * a.per_wave * 64, 0};
  const uint64_t w0 = a.e0 + (uint64_t)wave * a.per_wave * 64;
  for (uint32_t it = 0; it < a.per_wave && w0 + 64 * it < a.e1; ++it) {
    const uint64_t e = w0 + 64 * it + lane;
    const bool valid = e < a.e1;
    uint64_t key[W];
    load_row<W>(a.rows, a.lstart + e, valid, key);
    const bool dup = (key[0] & 1ull) != 0;  // already contains eps: r? = r
    key[0] |= 1ull;
    region_emit<W, kInl>(a, rg, valid, dup, key, (uint32_t)(e - a.e0) + a.rel0);
  }
  region_close(a, a.reg0 + wave, rg);
}

// r* for a.per_wave groups of 64 rows per workgroup, bit-sliced: Xt[w] / Yt[w] hold bit t = row t's
// membership of word w.  Y(eps) = 1 and, by increasing length,
// Y(w) = OR over cuts w = u v with u non-empty of X(u) & Y(v) (v is shorter).
template <int W, bool kInl>
__global__ __launch_bounds__(256) void gen_star(GenArgs a) {
  __shared__ uint64_t Xt[64 * W];
  __shared__ uint64_t Yt[64 * W];
  if (a.st->stop) return;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Region rg{a.slot0 + blockIdx.x * a.per_wave * 64, 0};
  for (uint32_t it = 0; it < a.per_wave; ++it) {
    const uint64_t base = a.e0 + ((uint64_t)blockIdx.x * a.per_wave + it) * 64;
    if (base >= a.e1) break;
    for (int k = wave; k < W; k += 4) {
      const uint64_t e = base + lane;
      const uint64_t v = (e < a.e1) ? a.rows[(a.lstart + e) * W + k] : 0ull;
      Xt[64 * k + lane] = transpose64(v);
    }
    for (uint32_t w = threadIdx.x; w < 64u * W; w += 256) Yt[w] = (w == 0) ? ~0ull : 0ull;
    __syncthreads();
    for (uint32_t l = 1; l <= a.max_len; ++l) {
      const uint32_t lo = a.len_off[l], hi = a.len_off[l + 1];
      for (uint32_t w = lo + threadIdx.x; w < hi; w += 256)
        Yt[w] = star_fold(Xt, Yt, a.gt_pair, a.gt_off[w], l);  // cuts 1..l (cut 0 has u = eps)
      __syncthreads();
    }
    if (wave == 0) {
      uint64_t key[W];
#pragma unroll
      for (int k = 0; k < W; ++k) key[k] = transpose64(Yt[64 * k + lane]);
      const uint64_t e = base + lane;
      region_emit<W, kInl>(a, rg, e < a.e1, false, key, (uint32_t)(e - a.e0) + a.rel0);
    }
    __syncthreads();  // the tiles are rewritten by the next group
  }
  if (wave == 0) region_close(a, a.reg0 + blockIdx.x, rg);
}

// The same with a wave per group: its own tiles, no workgroup barrier per word
// length, and the guide table in LDS.  A workgroup per group spends its time
// in those barriers, each for a handful of words (237 us per launch of one-
// word languages with 58 infixes; a wave per group: 65 us, of which its probes
// are most; four words: 58 -> 27 us); taken where the tiles of four waves and
// the table fit (star_by_wave).
constexpr uint32_t kStarPairs = 3072;
constexpr uint32_t kStarMaxLen = 62;
template <int W, bool kInl>
__global__ __launch_bounds__(256) void gen_star_wave(GenArgs a) {
  __shared__ uint64_t tiles[4][2 * 64 * W];
  __shared__ uint32_t gp[kStarPairs], go[64 * W + 1], lo[kStarMaxLen + 2];
  if (a.st->stop) return;
  stage_u32(gp, a.gt_pair, a.n_pairs, threadIdx.x, 256);
  for (uint32_t i = threadIdx.x; i <= a.n; i += 256) go[i] = a.gt_off[i];
  for (uint32_t i = threadIdx.x; i < a.max_len + 2; i += 256) lo[i] = a.len_off[i];
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63, wave = blockIdx.x * 4 + (threadIdx.x >> 6);
  uint64_t* Xt = tiles[threadIdx.x >> 6];
  uint64_t* Yt = Xt + 64 * W;
  Region rg{a.slot0 + wave * a.per_wave * 64, 0};
  const uint64_t w0 = a.e0 + (uint64_t)wave * a.per_wave * 64;
  for (uint32_t it = 0; it < a.per_wave && w0 + 64 * it < a.e1; ++it) {
    const uint64_t e = w0 + 64 * it + lane;
    uint64_t key[W];
    load_row<W>(a.rows, a.lstart + e, e < a.e1, key);
#pragma unroll
    for (int k = 0; k < W; ++k) {
      Xt[64 * k + lane] = transpose64(key[k]);
      Yt[64 * k + lane] = (k == 0 && lane == 0) ? ~0ull : 0ull;
    }
    wave_sync_lds();
    for (uint32_t l = 1; l <= a.max_len; ++l) {
      for (uint32_t w = lo[l] + lane; w < lo[l + 1]; w += 64) Yt[w] = star_fold(Xt, Yt, gp, go[w], l);
      wave_sync_lds();
    }
#pragma unroll
    for (int k = 0; k < W; ++k) key[k] = transpose64(Yt[64 * k + lane]);
    region_emit<W, kInl>(a, rg, e < a.e1, false, key, (uint32_t)(e - a.e0) + a.rel0);
    wave_sync_lds();  // the tiles are rewritten by the next group
  }
  region_close(a, a.reg0 + wave, rg);
}

bool star_by_wave(int W, const GenArgs& a) {
  return W <= 4 && a.n_pairs <= kStarPairs && a.max_len <= kStarMaxLen && a.n <= 64u * W;
}

// x.y, bit-sliced over 64 values of one operand.  A workgroup owns up to YT
// tiles of 64 rows of the operand across the lanes (transposed into LDS:
// Yt[tile][w], bit t = row t contains word w) and a group of rows of the
// other, uniform, operand.  Right rows across the lanes (kLeft = false): for
// a left row x, lane l of a wave owns word w = 64k + l of output word k; the
// cuts (u, v) of w with u in x select which Yt[v] are or-ed:
//   out_t(w) = OR_{(u,v) cut of w, x(u)=1} y_t(v)
// (Algorithm 2, the fold over the guide table, done for 64 candidates at once).
// Left rows across the lanes (kLeft = true): the mirror image, the uniform
// right row y selects by v and Yt[u] are or-ed.
// A wave transpose then gives lane t the W words of its candidate.
// Half of a level's blocks pair a huge left level with a right level of 2, 4,
// 5, ... rows: with right rows across the lanes only, those filled 2 to 24 of
// 64 lanes and took most of the launch.  With the left form for them, searches
// of 0.5-3.5 G candidates went 175.6 -> 99.6 ms (one word per language, 58
// infixes), 88.7 -> 31.3 ms (two words, 95), 22.1 -> 9.2 ms (four words, 130).
constexpr int kConcatYT = 8;

// kShort: every word has at most 32 cuts (length <= 31), so the cuts whose
// factor is in the uniform row fit one 32-bit mask per output word; otherwise
// that bit is tested inside the fold.
// kGtLds: the guide table is staged in LDS.  The choice is made at compile
// time so that every access has a fixed address space: reading LDS through a
// generic pointer (chosen at run time between LDS and global memory) gave
// wrong prefix bits now and then on gfx950.
template <int W, bool kShort, bool kInl, bool kGtLds, bool kLeft>
__device__ __forceinline__ void concat_part(const GenArgs& a, const ConcatPart& cp, uint32_t bid, uint64_t* lds) {
  const uint32_t yt_per_wg = cp.yt, xi_per_wg = cp.xi;
  uint64_t* Yt = lds;                                        // [yt_per_wg][64W]
  uint64_t* Xs = Yt + (size_t)yt_per_wg * 64 * W;            // [xi_per_wg][W]
  uint32_t* G = (uint32_t*)(Xs + (size_t)xi_per_wg * W);     // guide pairs (if gt_lds)
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t nR = cp.rcount;
  // rows [l0, l1) of the lane operand, [u0, u1) of the uniform one
  const uint64_t l0 = kLeft ? cp.i_lo : 0, l1 = kLeft ? cp.i_hi + 1 : nR;
  const uint64_t u0 = kLeft ? 0 : cp.i_lo, u1 = kLeft ? nR : cp.i_hi + 1;
  const uint64_t lane_start = kLeft ? cp.lstart : cp.rstart, uni_start = kLeft ? cp.rstart : cp.lstart;
  const uint64_t nT = (l1 - l0 + 63) / 64;
  // flat grid: workgroup -> (group of tiles, group of uniform rows)
  const uint64_t t0 = (uint64_t)(bid % cp.gx) * yt_per_wg;
  const uint32_t nt = (uint32_t)min<uint64_t>(yt_per_wg, nT - t0);
  const uint64_t x0 = u0 + (uint64_t)(bid / cp.gx) * xi_per_wg;
  const uint32_t nx = (uint32_t)min<uint64_t>(xi_per_wg, u1 - x0);

  // stage tiles (transposed), uniform rows and guide table; every load of a
  // thread is issued before the first is used
  for (uint32_t tq = wave; tq < nt; tq += 4) {
    const uint64_t r = l0 + (t0 + tq) * 64 + lane;
    uint64_t v[W];
    load_row<W>(a.rows, lane_start + r, r < l1, v);
#pragma unroll
    for (int k = 0; k < W; ++k) Yt[(size_t)tq * 64 * W + 64 * k + lane] = transpose64(v[k]);
  }
  {
    const uint64_t* src = a.rows + (uni_start + x0) * W;
    const uint32_t total = nx * W;
    uint32_t q = threadIdx.x;
    for (; q + 3 * 256 < total; q += 4 * 256) {
      const uint64_t v0 = src[q], v1 = src[q + 256], v2 = src[q + 512], v3 = src[q + 768];
      Xs[q] = v0;
      Xs[q + 256] = v1;
      Xs[q + 512] = v2;
      Xs[q + 768] = v3;
    }
    for (; q < total; q += 256) Xs[q] = src[q];
  }
  if constexpr (kGtLds) stage_u32(G, a.gt_pair, a.n_pairs, threadIdx.x, 256);
  __syncthreads();
  const uint32_t* gp;
  if constexpr (kGtLds)
    gp = G;
  else
    gp = a.gt_pair;
  // a cut's factor in the uniform row, and the one in the tile
  auto uni_of = [](uint32_t p) -> uint32_t { return kLeft ? (p & 0xFFFFu) : (p >> 16); };
  auto tile_of = [](uint32_t p) -> uint32_t { return kLeft ? (p >> 16) : (p & 0xFFFFu); };

  // cut ranges of this lane's words
  uint32_t off[W], cnt[W];
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const uint32_t w = 64u * k + lane;
    off[k] = (w < a.n) ? a.gt_off[w] : 0u;
    cnt[k] = (w < a.n) ? a.gt_off[w + 1] - off[k] : 0u;
  }

  // a wave takes whole uniform rows, or every 2nd or 4th tile of one when
  // there are only two rows or one
  const uint32_t per_row = nx >= 3 ? 1u : 4u / nx;
  // this wave's slots: the workgroup's tiles and rows are a dense range of
  // the part's nT x (u1 - u0) tiles of 64, its waves' shares lie in order
  uint32_t before = 0;  // wave iterations of this workgroup's lower waves
  for (uint32_t v = 0; v < wave; ++v)
    before += ((nx + 4 / per_row - 1 - v / per_row) / (4 / per_row)) * ((nt + per_row - 1 - v % per_row) / per_row);
  Region rg{cp.slot0 + (uint32_t)(((x0 - u0) * nT + nx * t0 + before) * 64), 0};
  for (uint32_t xi = wave / per_row; xi < nx; xi += 4 / per_row) {
    const uint64_t* xr = Xs + (size_t)xi * W;
    // bit q of m[k]: the uniform row contains its factor of cut q of word 64k+lane
    uint32_t m[W];
    if constexpr (kShort) {
#pragma unroll
      for (int k = 0; k < W; ++k) {
        uint32_t mm = 0;
        for (uint32_t q0 = 0; q0 < cnt[k]; q0 += 4) {
          // four cuts at a time: their reads overlap
          uint32_t u[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) u[t] = (q0 + t < cnt[k]) ? uni_of(gp[off[k] + q0 + t]) : 0u;
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (q0 + t < cnt[k]) mm |= (uint32_t)((xr[u[t] >> 6] >> (u[t] & 63)) & 1ull) << (q0 + t);
        }
        m[k] = mm;
      }
    }
    for (uint32_t tq = wave % per_row; tq < nt; tq += per_row) {
      const uint64_t* Y = Yt + (size_t)tq * 64 * W;
      uint64_t key[W];
#pragma unroll
      for (int k = 0; k < W; ++k) {
        uint64_t acc = 0;
        if constexpr (kShort) {
          for (uint32_t mm = m[k]; mm; mm &= mm - 1) {
            const uint32_t q = __ffs(mm) - 1;
            acc |= Y[tile_of(gp[off[k] + q])];
          }
        } else {
          for (uint32_t q = 0; q < cnt[k]; ++q) {
            const uint32_t p = gp[off[k] + q];
            const uint32_t u = uni_of(p);
            if ((xr[u >> 6] >> (u & 63)) & 1ull) acc |= Y[tile_of(p)];
          }
        }
        key[k] = transpose64(acc);
      }
      const uint64_t r = l0 + (t0 + tq) * 64 + lane;  // this lane's row
      const uint64_t e = kLeft ? r * nR + (x0 + xi) : (x0 + xi) * nR + r;
      const bool valid = r < l1 && e >= cp.e0 && e < cp.e1;
      region_emit<W, kInl>(a, rg, valid, false, key, (uint32_t)(e - cp.e0) + cp.rel0);
    }
  }
  region_close(a, cp.reg0 + bid * 4 + wave, rg);
}

template <int W, bool kShort, bool kInl, bool kGtLds>
__global__ __launch_bounds__(256) void gen_concat(GenArgs a, ConcatSet cs) {
  extern __shared__ uint64_t lds[];
  if (a.st->stop) return;
  // this workgroup's part (block) and its place in the part's grid
  uint32_t part = 0;
  while (part + 1 < cs.n && cs.p[part + 1].wg0 <= blockIdx.x) ++part;
  const ConcatPart& cp = cs.p[part];
  if (cp.left)
    concat_part<W, kShort, kInl, kGtLds, true>(a, cp, blockIdx.x - cp.wg0, lds);
  else
    concat_part<W, kShort, kInl, kGtLds, false>(a, cp, blockIdx.x - cp.wg0, lds);
}

// Row of a level from its position among the rows that are left (UnionPart).
__device__ __forceinline__ uint64_t kept_row(const UnionPart& p, uint64_t c) {
  if (c < p.n0) return c;
  c -= p.n0;
  return c < p.n1 ? p.s0 + c : p.us + (c - p.n1);
}

// One lane per pair x + y of the rows left (UnionPart), us.per_wave * 64
// consecutive ones per wave; several union blocks of a chunk share a launch,
// each workgroup in one block.
template <int W, bool kInl>
__global__ __launch_bounds__(256) void gen_union(GenArgs a, UnionSet us) {
  if (a.st->stop) return;
  uint32_t part = 0;
  while (part + 1 < us.n && us.p[part + 1].wg0 <= blockIdx.x) ++part;
  const UnionPart& up = us.p[part];
  const uint32_t wave = (blockIdx.x - up.wg0) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  Region rg{up.slot0 + wave * us.per_wave * 64, 0};
  const uint64_t w0 = (uint64_t)wave * us.per_wave * 64;
  const uint64_t i0 = up.same ? 0 : up.e0 / up.rcount;          // first left row
  const uint64_t cols = up.n0 + up.n1 + (up.rcount - up.us);    // right rows left
  const bool narrow = up.k0 + up.lanes <= 0xFFFFFFFFull && cols <= 0xFFFFFFFFull;
  for (uint32_t it = 0; it < us.per_wave && w0 + 64 * it < up.lanes; ++it) {
    const uint64_t q = w0 + 64 * it + lane, k = up.k0 + q;
    bool valid = q < up.lanes;
    uint64_t i = 0, j = 0, e = 0;
    if (valid) {
      if (up.same) {
        tri_decode(k, up.n0 + up.n1, &i, &j);
        i = kept_row(up, i);
        j = kept_row(up, j);
        e = i * up.rcount - i * (i + 1) / 2 + (j - i - 1);
      } else {
        uint64_t c;
        if (narrow) {
          i = (uint32_t)k / (uint32_t)cols;
          c = (uint32_t)k - (uint32_t)i * (uint32_t)cols;
        } else {
          i = k / cols;
          c = k - i * cols;
        }
        i += i0;
        j = kept_row(up, c);
        e = i * up.rcount + j;
        if (j >= up.us && j < up.ue) {
          const uint64_t r = a.aux[up.rstart + j] - up.eq_base;
          const uint64_t first = up.eq_tri ? (i + 1) * up.eq_n - (i + 1) * (i + 2) / 2 : (i + 1) * up.eq_n;
          valid = r >= first;
        }
      }
      valid = valid && e >= up.e0 && e < up.e1;
    }
    if (!__any(valid)) continue;
    uint64_t x[W], y[W], key[W];
    load_row<W>(a.rows, up.lstart + i, valid, x);
    load_row<W>(a.rows, up.rstart + j, valid, y);
    bool eqx = true, eqy = true;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      key[w] = x[w] | y[w];
      eqx = eqx && key[w] == x[w];
      eqy = eqy && key[w] == y[w];
    }
    // x+y equals x or y (one contains the other): that language is stored
    region_emit<W, kInl>(a, rg, valid, eqx || eqy, key, (uint32_t)(e - up.e0) + up.rel0);
  }
  region_close(a, up.reg0 + wave, rg);
}

// Many small pieces of one chunk (see PieceArgs): one wave per item of 64
// candidates, so a level's small constructor blocks cost one launch.  The
// constructors are those of the kernels above, at wave scale; the guide
// table is read through the caches.

// An item of 64 candidates of a CHAR, QUESTION, UNION or STAR piece (the
// star with the wave's tiles X and Y): lane t's candidate key.
template <int W>
__device__ __forceinline__ void piece_simple(const GenArgs& a, const PieceD& p, uint64_t li, uint32_t lane,
                                             uint64_t* X, uint64_t* Y, uint64_t (&key)[W], bool* valid,
                                             bool* dup, uint64_t* e_out) {
  const uint64_t e = p.e0 + 64 * li + lane;
  *valid = e < p.e1;
  *dup = false;
  *e_out = e;
  if (p.op == OP_CHAR) {
    const int idx = *valid ? a.char_index[p.char_off + e] : -1;
#pragma unroll
    for (int q = 0; q < W; ++q) key[q] = (idx >= 0 && (idx >> 6) == q) ? (1ull << (idx & 63)) : 0ull;
  } else if (p.op == OP_QUESTION) {
    const uint64_t* src = a.rows + (p.lstart + (*valid ? e : 0)) * W;
#pragma unroll
    for (int q = 0; q < W; ++q) key[q] = *valid ? src[q] : 0ull;
    *dup = (key[0] & 1ull) != 0;
    key[0] |= 1ull;
  } else if (p.op == OP_UNION) {
    uint64_t i = 0, j = 0;
    if (*valid) {
      if (p.same) {
        tri_decode(e, p.lcount, &i, &j);
      } else {
        i = e / p.rcount;
        j = e - i * p.rcount;
      }
    }
    const uint64_t* x = a.rows + (p.lstart + i) * W;
    const uint64_t* y = a.rows + (p.rstart + j) * W;
    bool eqx = true, eqy = true;
#pragma unroll
    for (int q = 0; q < W; ++q) {
      const uint64_t xv = *valid ? x[q] : 0ull, yv = *valid ? y[q] : 0ull;
      key[q] = xv | yv;
      eqx = eqx && key[q] == xv;
      eqy = eqy && key[q] == yv;
    }
    *dup = eqx || eqy;
  } else {  // OP_STAR: Y(eps) = 1; by increasing length, Y(w) = OR over
            // cuts with a non-empty first factor of X(u) & Y(v)
#pragma unroll
    for (int q = 0; q < W; ++q) {
      X[64 * q + lane] = transpose64(*valid ? a.rows[(p.lstart + e) * W + q] : 0ull);
      Y[64 * q + lane] = (q == 0 && lane == 0) ? ~0ull : 0ull;
    }
    wave_sync_lds();
    for (uint32_t l = 1; l <= a.max_len; ++l) {
      const uint32_t lo = a.len_off[l], hi = a.len_off[l + 1];
      for (uint32_t w = lo + lane; w < hi; w += 64) Y[w] = star_fold(X, Y, a.gt_pair, a.gt_off[w], l);
      wave_sync_lds();
    }
#pragma unroll
    for (int q = 0; q < W; ++q) key[q] = transpose64(Y[64 * q + lane]);
  }
}

// A CONCAT item: its varying operand's rows across the lanes (right rows
// with one left row, or left rows with one right row when the right level
// is small), staged transposed in X for words [q_lo, q_hi), the uniform
// operand's row in U (when stage_u).  Returns lane t's candidate index and
// whether it is one.
template <int W>
__device__ __forceinline__ void concat_stage(const GenArgs& a, const PieceD& p, uint64_t li, uint32_t lane,
                                             uint64_t* X, uint64_t* U, int q_lo, int q_hi, bool stage_u,
                                             uint64_t* e_out, bool* valid) {
  const uint64_t nR = p.rcount, nL = p.lcount;
  uint64_t i, j, row, urow;
  bool have;
  if (!p.left_lanes) {
    i = p.t0 + li / p.nt;
    j = 64 * (li % p.nt) + lane;
    have = j < nR;
    row = p.rstart + j;
    urow = p.lstart + i;
  } else {
    i = 64 * (p.t0 + li / p.nt) + lane;
    j = li % p.nt;
    have = i < nL;
    row = p.lstart + i;
    urow = p.rstart + j;
  }
#pragma unroll
  for (int q = 0; q < W; ++q)
    if (q >= q_lo && q < q_hi) X[64 * q + lane] = transpose64(have ? a.rows[row * W + q] : 0ull);
  if (stage_u && lane < (uint32_t)W) U[lane] = a.rows[urow * W + lane];
  const uint64_t e = i * nR + j;
  *e_out = e;
  *valid = have && e >= p.e0 && e < p.e1;
}

// The fold of a CONCAT item for output words [q_lo, q_hi) (X and U staged;
// q_lo and q_hi multiples of kG): key[q] for those q.  From 8 words, cut
// position outer over kG of the lane's words at a time, 3 kG independent
// reads per round (each word's read clamped to its last cut, masked
// after); below, per word.
template <int W, int kG = 8>
__device__ __forceinline__ void concat_fold(const GenArgs& a, const PieceD& p, uint32_t lane, const uint64_t* X,
                                            const uint64_t* U, int q_lo, int q_hi, uint64_t (&key)[W]) {
  if constexpr (W >= 8) {
#pragma unroll
    for (int q0 = 0; q0 < W; q0 += kG) {
      if (q0 < q_lo || q0 >= q_hi) continue;
      uint32_t first[kG], last[kG], cnt[kG];
      uint64_t acc[kG];
#pragma unroll
      for (int q = 0; q < kG; ++q) {
        const uint32_t w = 64u * (q0 + q) + lane;
        first[q] = w < a.n ? a.gt_off[w] : 0u;
        cnt[q] = w < a.n ? a.gt_off[w + 1] - first[q] : 0u;
        last[q] = first[q] + (cnt[q] ? cnt[q] - 1 : 0u);
        acc[q] = 0;
      }
      for (uint32_t c = 0; c <= a.max_len; ++c) {
        uint32_t pr[kG];
#pragma unroll
        for (int q = 0; q < kG; ++q) pr[q] = a.gt_pair[min(first[q] + c, last[q])];
#pragma unroll
        for (int q = 0; q < kG; ++q) {
          const uint32_t uu = p.left_lanes ? (pr[q] & 0xFFFFu) : (pr[q] >> 16);  // index into the uniform row
          const uint32_t tt = p.left_lanes ? (pr[q] >> 16) : (pr[q] & 0xFFFFu);  // index into the tile
          const uint64_t xv = X[tt];
          const bool on = c < cnt[q] && ((U[uu >> 6] >> (uu & 63)) & 1ull);
          acc[q] |= on ? xv : 0ull;
        }
      }
#pragma unroll
      for (int q = 0; q < kG; ++q) key[q0 + q] = transpose64(acc[q]);
    }
  } else {
#pragma unroll
    for (int q = 0; q < W; ++q) {
      if (q < q_lo || q >= q_hi) continue;
      const uint32_t w = 64u * q + lane;
      const uint32_t c0 = w < a.n ? a.gt_off[w] : 0u, c1 = w < a.n ? a.gt_off[w + 1] : 0u;
      uint64_t acc = 0;
      // four cuts at a time: their reads overlap
      for (uint32_t c = c0; c < c1; c += 4) {
        uint32_t pr[4];
        uint64_t xv[4], uv[4];
#pragma unroll
        for (int z = 0; z < 4; ++z) pr[z] = a.gt_pair[min(c + z, c1 - 1)];
#pragma unroll
        for (int z = 0; z < 4; ++z) {
          const uint32_t uu = p.left_lanes ? (pr[z] & 0xFFFFu) : (pr[z] >> 16);  // index into the uniform row
          xv[z] = X[p.left_lanes ? (pr[z] >> 16) : (pr[z] & 0xFFFFu)];           // of the tile
          uv[z] = U[uu >> 6] >> (uu & 63);
        }
#pragma unroll
        for (int z = 0; z < 4; ++z) acc |= (uv[z] & 1ull) ? xv[z] : 0ull;  // (the last cut again is harmless)
      }
      key[q] = transpose64(acc);
    }
  }
}

__device__ __forceinline__ uint32_t piece_of(const PieceArgs& pa, uint64_t it) {
  uint32_t k = 0;
  while (k + 1 < pa.n && pa.p[k + 1].item0 <= it) ++k;
  return k;
}

// kSplit (from 16 words, launches of few items, where one item's latency
// is the launch's): kSplit waves (2 or 4) share each CONCAT item, each
// staging and folding W / kSplit of the words, and each STAR item (each
// stages its words; the words of each length are dealt to all of them);
// the others hand their key words to the first through LDS, which probes.
// Other items are the first wave's.
template <int W, bool kInl, int kSplit>
__global__ __launch_bounds__(256) void gen_pieces(GenArgs a, PieceArgs pa) {
  __shared__ uint64_t lds[4][2 * 64 * W + W];
  if (a.st->stop) return;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if constexpr (kSplit == 1) {
    uint64_t* X = lds[wave];       // star: X tile; concat: operand tile
    uint64_t* Y = X + 64 * W;      // star: Y tile
    uint64_t* U = Y + 64 * W;      // concat: the uniform operand
    for (uint64_t it = (uint64_t)blockIdx.x * 4 + wave; it < pa.items; it += (uint64_t)gridDim.x * 4) {
      const PieceD& p = pa.p[piece_of(pa, it)];
      const uint64_t li = it - p.item0;
      uint64_t key[W];
      bool valid = false, dup = false;
      uint64_t e = 0;
      if (p.op != OP_CONCAT) {
        piece_simple<W>(a, p, li, lane, X, Y, key, &valid, &dup, &e);
      } else {
        concat_stage<W>(a, p, li, lane, X, U, 0, W, true, &e, &valid);
        wave_sync_lds();
        concat_fold<W>(a, p, lane, X, U, 0, W, key);
      }
      filter_emit<W, kInl>(a, valid, dup, key, valid ? (uint32_t)(e - p.e0) + p.rel0 : 0u);
      wave_sync_lds();  // the tiles are rewritten by the next item
    }
  } else {
    constexpr int kPart = W / kSplit;          // words per wave
    constexpr int kG = kPart < 8 ? kPart : 8;  // fold group
    constexpr uint32_t kItems = 4 / kSplit;    // items per workgroup round
    static_assert((kSplit == 2 || kSplit == 4) && kPart >= 4 && kPart % kG == 0, "whole fold groups per wave");
    const uint32_t slot = wave / kSplit, part = wave % kSplit;
    uint64_t* X = lds[kSplit * slot];
    uint64_t* Y = X + 64 * W;
    uint64_t* U = Y + 64 * W;
    uint64_t* K = lds[kSplit * slot + 1];  // the other waves' key words, [q - kPart][lane]
    const int q_lo = (int)part * kPart, q_hi = q_lo + kPart;  // this wave's words
    // every wave takes the same number of rounds (workgroup barriers inside)
    for (uint64_t base = (uint64_t)blockIdx.x * kItems; base < pa.items; base += (uint64_t)gridDim.x * kItems) {
      const uint64_t it = base + slot;
      const bool have = it < pa.items;
      const PieceD& p = pa.p[have ? piece_of(pa, it) : 0];
      const uint64_t li = have ? it - p.item0 : 0;
      const bool cat = have && p.op == OP_CONCAT;
      const bool star = have && p.op == OP_STAR;
      uint64_t key[W];
      bool valid = false, dup = false;
      uint64_t e = 0;
      if (cat) concat_stage<W>(a, p, li, lane, X, U, q_lo, q_hi, part == 0, &e, &valid);
      if (star) {
        // r* of 64 rows: each wave stages its words of X and Y
        e = p.e0 + 64 * li + lane;
        valid = e < p.e1;
#pragma unroll
        for (int q = 0; q < W; ++q)
          if (q >= q_lo && q < q_hi) {
            X[64 * q + lane] = transpose64(valid ? a.rows[(p.lstart + e) * W + q] : 0ull);
            Y[64 * q + lane] = (q == 0 && lane == 0) ? ~0ull : 0ull;
          }
      }
      // (uniform over the workgroup: the star's barriers below are taken by
      // all of its waves or by none)
      const bool any_star = __syncthreads_or(star);
      if (any_star) {
        // Y(w) by increasing length from shorter words' Y: the words of one
        // length dealt to the item's waves, a barrier per length
        for (uint32_t l = 1; l <= a.max_len; ++l) {
          if (star) {
            const uint32_t lo = a.len_off[l], hi = a.len_off[l + 1];
            for (uint32_t w = lo + lane + 64 * part; w < hi; w += 64 * kSplit)
              Y[w] = star_fold(X, Y, a.gt_pair, a.gt_off[w], l);
          }
          __syncthreads();
        }
      }
      if (cat) concat_fold<W, kG>(a, p, lane, X, U, q_lo, q_hi, key);
      if (star) {
#pragma unroll
        for (int q = 0; q < W; ++q)
          if (q >= q_lo && q < q_hi) key[q] = transpose64(Y[64 * q + lane]);
      }
      if ((cat || star) && part != 0) {
#pragma unroll
        for (int q = 0; q < W; ++q)
          if (q >= q_lo && q < q_hi) K[64 * (q - kPart) + lane] = key[q];
      }
      __syncthreads();
      if (part == 0 && have) {
        if (cat || star) {
#pragma unroll
          for (int q = kPart; q < W; ++q) key[q] = K[64 * (q - kPart) + lane];
        } else {
          piece_simple<W>(a, p, li, lane, X, Y, key, &valid, &dup, &e);
        }
        filter_emit<W, kInl>(a, valid, dup, key, valid ? (uint32_t)(e - p.e0) + p.rel0 : 0u);
      }
      __syncthreads();  // the tiles are rewritten in the next round
    }
  }
}

// ---- chunk pipeline ------------------------------------------------------

__global__ void fill_u64(uint64_t* p, uint64_t n, uint64_t v) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

__device__ __forceinline__ void ctrl_clear(Ctrl* c) {
  c->n_surv = 0;
  c->answer_e = ~0u;
  c->append = 0;
}

__global__ __launch_bounds__(256) void search_reset(ResetArgs a) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, n = (uint64_t)gridDim.x * blockDim.x;
  if (t == 0) {
    ctrl_clear(a.ctrl);
    ctrl_clear(a.ctrl + 1);
    DevState* st = a.st;
    st->total_rows = a.total_rows;
    st->row_cap = a.row_cap;
    st->stop = STOP_NONE;
    st->answer_cost = 0;
    st->answer_e = 0;
    st->resume_level = 0;
    st->otf_on = a.otf_on;
    st->otf = 0;
    st->chunks = 0;
  }
  for (uint64_t i = t; i < a.n_levels; i += n) a.levels[i] = a.levels_src ? a.levels_src[i] : 0;
  for (uint64_t i = t; i < a.n_slot_words; i += n) a.slots[i] = kEmpty;
  for (int b = 0; b < 2; ++b)
    for (uint64_t i = t; i < a.bitmap_words[b]; i += n) a.bitmap[b][i] = 0;
}

template <int W, bool kInl>
__global__ __launch_bounds__(256) void rehash_rows(const uint64_t* rows, uint64_t nrows, uint64_t* slots,
                                                   uint64_t mask) {
  for (uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; r < nrows;
       r += (uint64_t)gridDim.x * blockDim.x) {
    uint64_t key[W];
#pragma unroll
    for (int k = 0; k < W; ++k) key[k] = rows[r * W + k];
    table_rebuild_one<W, kInl>(slots, mask, key, r);
  }
}

// Every survivor of the chunk once, over the grid: the pieces' (slots 0 ..
// n_surv - 1), then those in the large generators' per-wave ranges, a wave
// per range.  f(sid, have) is called by whole waves; lanes without a survivor
// get have = false.
template <typename F>
__device__ __forceinline__ void for_survivors(const ChunkArgs& a, F f) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, waves = (gridDim.x * blockDim.x) >> 6;
  const uint32_t ns = a.ctrl->n_surv;
  for (uint32_t k = 64 * wave; k < ns; k += 64 * waves) f(k + lane, k + lane < ns);
  for (uint32_t r = wave; r < a.n_reg; r += waves) {
    const uint2 g = a.reg[r];
    for (uint32_t k = 0; k < g.y; k += 64) f(g.x + k + lane, k + lane < g.y);
  }
}

// Toggles bit e of the bitmap for every lane with `on`, lanes next to each
// other that share a word in one atomic (survivors lie in enumeration order
// along a wave, mostly several to a word).  Called by the whole wave.
__device__ __forceinline__ void toggle_bits(uint32_t* bitmap, uint32_t e, bool on) {
  const uint32_t lane = lane_id();
  const uint32_t w = on ? e >> 5 : ~0u;
  uint32_t m = on ? 1u << (e & 31) : 0u;
  const uint32_t w_before = (uint32_t)__shfl_up((int)w, 1, kWave);
  const bool head = lane == 0 || w_before != w;
  const uint64_t heads = __ballot(head);
  // first lane after this lane's run of equal words
  const uint64_t above = lane == 63 ? 0ull : heads >> (lane + 1);
  const uint32_t end = above ? lane + (uint32_t)__ffsll((unsigned long long)above) : 64u;
#pragma unroll
  for (uint32_t d = 1; d < 64; d <<= 1) {
    const uint32_t o = (uint32_t)__shfl_down((int)m, d, kWave);
    if (lane + d < end) m |= o;
  }
  if (head && on) atomicXor(&bitmap[w], m);
}

// Insertion, and the winners' bits: a survivor that takes its slot toggles
// its bit on, one that is displaced has its bit toggled off by the displacing
// survivor.  Toggles commute, so each winner's bit ends up set and every
// other clear, whatever the order.  Bound by the table's random atomics
// (probe and atomicMin reach 14-16 G/s on this card): 169 us a launch, mean of
// the 89 of a one-word search, 58 infixes, that stores 130 M languages, i.e.
// 116 ps each for the two atomics on a slot's line; the ordered append 25 us.
// (Marking the winners in a pass of its own, over the survivors of every
// candidate, took 75 us per chunk beside an insertion of 121 us and an append
// of 48 us that reset each reference: 122, none and 20 us on the same chunks
// with toggles, 166 us with one toggle per lane instead of one per run.)
template <int W, bool kInl>
__global__ __launch_bounds__(256) void insert_survivors(ChunkArgs a) {
  if (a.st->stop) return;
  for (uint32_t w = blockIdx.x * blockDim.x + threadIdx.x; w < a.clear_words; w += gridDim.x * blockDim.x)
    a.bitmap_next[w] = 0;
  for_survivors(a, [&](uint32_t sid, bool have) {
    uint32_t e = 0;
    bool won = false;
    if (have) {
      const uint64_t h = a.spos[sid];
      e = a.se[sid];
      const uint64_t mine = kInl ? chunk_ref(a.ref_gen, e) : new_ref(e, sid);
      uint64_t old;
      const uint64_t pos = table_insert<W, kInl>(a.slots, a.slot_mask, a.rows, a.skey, sid, h, mine, &old);
      if constexpr (!kInl) a.spos[sid] = spos_pack(pos, h);
      won = mine < old;  // else an earlier candidate has it
      uint32_t oe;
      if (won && displaced_survivor<kInl>(old, a.ref_gen, &oe)) atomicXor(&a.bitmap[oe >> 5], 1u << (oe & 31));
    }
    toggle_bits(a.bitmap, e, won);
  });
}

// Outcome of a chunk, in enumeration order: the answer (first precise
// candidate) if its winners before it fit the row cap, else out of memory at
// the first winner that does not fit; otherwise all winners are stored.
// With OnTheFly allowed, the first winner that does not fit switches the
// search to OnTheFly mode instead: the winners that fit are stored, and the
// rest of the chunk (and of the search) is tested for precision only.
__device__ void account_chunk(const ChunkArgs& a, uint32_t ans, uint32_t answer_rank, uint32_t winners,
                              uint32_t overflow_e) {
  DevState* st = a.st;
  const uint64_t room = st->row_cap > st->total_rows ? st->row_cap - st->total_rows : 0;
  const uint32_t c = a.cost;
  a.ctrl->append = a.chunk_id;
  a.ctrl->row_base = st->total_rows;
  a.ctrl->room = room;
  uint64_t stored;
  if (st->otf) {
    stored = 0;
    if (ans != ~0u) {
      a.cand[c] += (uint64_t)ans + 1;
      st->stop = STOP_ANSWER;
      st->answer_cost = c;
      st->answer_e = a.chunk_e0 + ans;
    } else {
      a.cand[c] += a.len;
    }
  } else if (ans != ~0u) {
    if ((uint64_t)answer_rank > room && st->otf_on) {
      // the cache filled before the answer, which is found on the fly
      stored = room;
      a.cand[c] += (uint64_t)ans + 1;
      a.uniq[c] += room;
      st->stop = STOP_ANSWER;
      st->answer_cost = c;
      st->answer_e = a.chunk_e0 + ans;
    } else if ((uint64_t)answer_rank > room) {
      stored = room;
      a.cand[c] += (uint64_t)overflow_e + 1;
      a.uniq[c] += room;
      st->stop = STOP_OOM;
    } else {
      stored = answer_rank;
      a.cand[c] += (uint64_t)ans + 1;
      a.uniq[c] += (uint64_t)answer_rank + 1;
      st->stop = STOP_ANSWER;
      st->answer_cost = c;
      st->answer_e = a.chunk_e0 + ans;
    }
  } else if ((uint64_t)winners > room && st->otf_on) {
    stored = room;
    a.cand[c] += a.len;
    a.uniq[c] += room;
    st->otf = 1;
  } else if ((uint64_t)winners > room) {
    stored = room;
    a.cand[c] += (uint64_t)overflow_e + 1;
    a.uniq[c] += room;
    st->stop = STOP_OOM;
  } else {
    stored = winners;
    a.cand[c] += a.len;
    a.uniq[c] += winners;
  }
  st->total_rows += stored;
  a.lcount[c] += stored;
  ctrl_clear(a.ctrl_next);
  // the host reads these at level boundaries without a copy
  DevState* h = a.hst;
  h->total_rows = st->total_rows;
  h->row_cap = st->row_cap;
  h->stop = st->stop;
  h->answer_cost = st->answer_cost;
  h->answer_e = st->answer_e;
  h->resume_level = st->resume_level;
  h->otf_on = st->otf_on;
  h->otf = st->otf;
  a.hlev[c] = a.lcount[c];
  a.hlev[a.nlev + c] = a.uniq[c];
  a.hlev[2 * a.nlev + c] = a.cand[c];
  // the count last: a host that sees it sees everything above
  st->chunks += 1;
  __hip_atomic_store(&h->chunks, st->chunks, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <int W, bool kInl>
__device__ __forceinline__ void store_winner(const ChunkArgs& a, uint32_t sid, uint32_t e, uint64_t row) {
  uint64_t key[W];
  load_row<W>(a.skey, sid, true, key);
  uint64_t rec = 0;
  if constexpr (!kInl) rec = a.spos[sid];
#pragma unroll
  for (int k = 0; k < W; ++k) a.rows_w[row * W + k] = key[k];
  a.aux[row] = a.chunk_e0 + e;
  if constexpr (!kInl) table_publish(a.slots, rec, row);
}

constexpr uint32_t kSmallWords = (uint32_t)(kSmallChunk / 32);
constexpr uint64_t kSmallCopyWords = 1ull << 16;
static_assert(kSmallChunk <= 0xFFFFu, "survivor ranks of a small chunk fit 16 bits");

// Whole finalization of a small chunk in one workgroup: winner bitmap copied
// to LDS, its prefix scan, ordered append, accounting.
template <int W, bool kInl>
__global__ __launch_bounds__(1024) void finalize_small(ChunkArgs a) {
  __shared__ uint32_t bm[kSmallWords];
  __shared__ uint32_t pre[kSmallWords];
  __shared__ uint32_t s_rank, s_over, s_total;
  __shared__ uint16_t dst[W <= 2 ? 1 : kSmallChunk];  // wide rows: each survivor's rank
  constexpr uint32_t kNotStored = 0xFFFFu;             // ranks are below kSmallChunk
  if (a.st->stop) return;
  const uint32_t t = threadIdx.x;
  const uint32_t ns = a.ctrl->n_surv, ans = a.ctrl->answer_e;
  const uint32_t words = (uint32_t)((a.len + 31) / 32);
  for (uint32_t i = t; i < words; i += 1024) bm[i] = a.bitmap[i];
  if (t == 0) {
    s_rank = ~0u;
    s_over = ~0u;
  }
  __syncthreads();
  if (t < 64) {
    const uint32_t tot = wave_popc_scan<kSmallWords / 64>(bm, pre, words);
    if (t == 0) s_total = tot;
  }
  __syncthreads();
  const uint32_t total = s_total;
  const uint64_t row_base = a.st->total_rows;
  const uint64_t room = a.st->row_cap > row_base ? a.st->row_cap - row_base : 0;
  // each survivor's rank among the stored rows (kNotStored: not stored)
  auto place = [&](uint32_t sid, uint32_t e) -> uint32_t {
    const uint32_t word = bm[e >> 5];
    const uint32_t bit = 1u << (e & 31);
    if (!(word & bit)) return kNotStored;  // e is unique per survivor: the bit marks this one
    const uint32_t rank = pre[e >> 5] + (uint32_t)__popc(word & (bit - 1));
    if (e == ans) s_rank = rank;
    if (ans != ~0u && e >= ans) return kNotStored;  // the answer and later ones are not stored
    if (rank < room) return rank;
    if (rank == room) s_over = e;
    return kNotStored;
  };
  if constexpr (W <= 2) {
    // four survivors per thread and round, their reads issued together
    uint32_t sid = t;
    for (; sid + 3 * 1024 < ns; sid += 4 * 1024) {
      const uint32_t e0 = a.se[sid], e1 = a.se[sid + 1024], e2 = a.se[sid + 2048], e3 = a.se[sid + 3072];
      const uint32_t r0 = place(sid, e0), r1 = place(sid + 1024, e1), r2 = place(sid + 2048, e2),
                     r3 = place(sid + 3072, e3);
      if (r0 != kNotStored) store_winner<W, kInl>(a, sid, e0, row_base + r0);
      if (r1 != kNotStored) store_winner<W, kInl>(a, sid + 1024, e1, row_base + r1);
      if (r2 != kNotStored) store_winner<W, kInl>(a, sid + 2048, e2, row_base + r2);
      if (r3 != kNotStored) store_winner<W, kInl>(a, sid + 3072, e3, row_base + r3);
    }
    for (; sid < ns; sid += 1024) {
      const uint32_t e = a.se[sid];
      const uint32_t r = place(sid, e);
      if (r != kNotStored) store_winner<W, kInl>(a, sid, e, row_base + r);
    }
  } else {
    // wide rows: ranks first, then W consecutive lanes copy one row, so
    // that each wave reads and writes whole rows (coalesced)
    uint32_t sid = t;
    for (; sid + 3 * 1024 < ns; sid += 4 * 1024) {
      const uint32_t e0 = a.se[sid], e1 = a.se[sid + 1024], e2 = a.se[sid + 2048], e3 = a.se[sid + 3072];
      dst[sid] = (uint16_t)place(sid, e0);
      dst[sid + 1024] = (uint16_t)place(sid + 1024, e1);
      dst[sid + 2048] = (uint16_t)place(sid + 2048, e2);
      dst[sid + 3072] = (uint16_t)place(sid + 3072, e3);
    }
    for (; sid < ns; sid += 1024) dst[sid] = (uint16_t)place(sid, a.se[sid]);
    __syncthreads();
    constexpr uint32_t kPer = 1024 / W;  // rows per round
    const uint32_t k = t % W;
    for (uint32_t q = t / W; q < ns; q += kPer) {
      const uint32_t r = dst[q];
      if (r == kNotStored) continue;
      const uint64_t row = row_base + r;
      a.rows_w[row * W + k] = a.skey[(uint64_t)q * W + k];
      if (k == 0) {
        a.aux[row] = a.chunk_e0 + a.se[q];
        table_publish(a.slots, a.spos[q], row);
      }
    }
  }
  __syncthreads();
  if (t == 0) account_chunk(a, ans, s_rank, total, s_over);
}

// ---- grid path for large chunks ----

constexpr uint32_t kScanBlock = 1024;  // bitmap words per scan block (256 threads x 4)

__global__ __launch_bounds__(256) void scan_reduce(ChunkArgs a) {
  __shared__ uint32_t red[256];
  if (a.st->stop) return;
  const uint32_t b = blockIdx.x, t = threadIdx.x;
  uint32_t s = 0;
  for (uint32_t q = 0; q < 4; ++q) {
    const uint32_t w = b * kScanBlock + t * 4 + q;
    if (w < a.n_bitmap_words) s += __popc(a.bitmap[w]);
  }
  red[t] = s;
  __syncthreads();
  for (uint32_t st = 128; st > 0; st >>= 1) {
    if (t < st) red[t] += red[t + st];
    __syncthreads();
  }
  if (t == 0) a.block_sums[b] = red[0];
}

// The chunk's accounting by the workgroup that knows the total: before[w] is
// the number of winners below bitmap word w.  Called by one thread.
template <typename Before>
__device__ void account_scanned(const ChunkArgs& a, uint32_t winners, Before before) {
  const uint32_t ans = a.ctrl->answer_e;
  const uint64_t total = a.st->total_rows;
  const uint64_t room = a.st->row_cap > total ? a.st->row_cap - total : 0;
  uint32_t answer_rank = ~0u, overflow_e = ~0u;
  if (ans != ~0u) answer_rank = before(ans >> 5) + (uint32_t)__popc(a.bitmap[ans >> 5] & ((1u << (ans & 31)) - 1));
  if (winners > room) {
    // the first winner that does not fit: bisect the words, then the bits
    uint32_t lo = 0, hi = a.n_bitmap_words;
    while (hi - lo > 1) {
      const uint32_t mid = lo + (hi - lo) / 2;
      if (before(mid) <= room)
        lo = mid;
      else
        hi = mid;
    }
    uint32_t m = a.bitmap[lo];
    for (uint32_t k = (uint32_t)room - before(lo); k; --k) m &= m - 1;
    overflow_e = 32 * lo + (uint32_t)__ffs(m) - 1;
  }
  account_chunk(a, ans, answer_rank, winners, overflow_e);
}

// Chunks whose bitmap has at most kScanSingleWords words (2^18 candidates,
// eight words per thread): the whole exclusive scan of the winner bitmap in
// one workgroup (each thread a contiguous run of words), and the accounting,
// one launch of 7 us where scan_reduce and scan_down, which account too, take
// 5 + 7 us and a gap; larger bitmaps scan faster spread out.
constexpr uint32_t kScanSingleWords = 8192;
__global__ __launch_bounds__(1024) void scan_single(ChunkArgs a) {
  __shared__ uint32_t part[1024];
  if (a.st->stop) return;
  const uint32_t t = threadIdx.x;
  const uint32_t words = a.n_bitmap_words;
  const uint32_t per = (words + 1023) / 1024;
  const uint32_t lo = min(words, t * per), hi = min(words, lo + per);
  uint32_t s = 0;
  for (uint32_t w = lo; w < hi; ++w) s += __popc(a.bitmap[w]);
  part[t] = s;
  __syncthreads();
  for (uint32_t st = 1; st < 1024; st <<= 1) {
    const uint32_t v = (t >= st) ? part[t - st] : 0u;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  uint32_t run = part[t] - s;  // exclusive
  for (uint32_t w = lo; w < hi; ++w) {
    a.word_prefix[w] = run;
    run += __popc(a.bitmap[w]);
  }
  __syncthreads();
  if (t == 0) account_scanned(a, part[1023], [&](uint32_t w) { return a.word_prefix[w]; });
}

// Each block adds the sums of the blocks before it by itself (a launch of one
// workgroup in between cost 4.4 us and its gap per chunk); the last one also
// accounts the chunk (a launch of its own at the end cost 4 us).
__global__ __launch_bounds__(256) void scan_down(ChunkArgs a, uint32_t nb) {
  __shared__ uint32_t part[256];
  __shared__ uint32_t s_base, s_ans, s_stopped;
  __shared__ uint64_t s_room;
  // (no look at the stop code before the last block's accounting, which may
  // set it while others have not started: a chunk after a stop writes prefixes
  // that nobody reads)
  const uint32_t b = blockIdx.x, t = threadIdx.x;
  uint32_t before = 0;
  for (uint32_t i = t; i < b; i += 256) before += a.block_sums[i];
  part[t] = before;
  __syncthreads();
  for (uint32_t st = 128; st > 0; st >>= 1) {
    if (t < st) part[t] += part[t + st];
    __syncthreads();
  }
  if (t == 0) {
    s_base = part[0];
    if (b + 1 == nb) {
      // what the accounting starts from, read once: thread 0 changes the state
      // below while the other waves still decide by these
      const uint64_t total = a.st->total_rows;
      s_room = a.st->row_cap > total ? a.st->row_cap - total : 0;
      s_ans = a.ctrl->answer_e;
      s_stopped = a.st->stop;
    }
  }
  __syncthreads();
  uint32_t c[4], s = 0;
  for (uint32_t q = 0; q < 4; ++q) {
    const uint32_t w = b * kScanBlock + t * 4 + q;
    c[q] = (w < a.n_bitmap_words) ? __popc(a.bitmap[w]) : 0u;
    s += c[q];
  }
  part[t] = s;
  __syncthreads();
  for (uint32_t st = 1; st < 256; st <<= 1) {
    const uint32_t v = (t >= st) ? part[t - st] : 0u;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  uint32_t run = s_base + part[t] - s;
  for (uint32_t q = 0; q < 4; ++q) {
    const uint32_t w = b * kScanBlock + t * 4 + q;
    if (w < a.n_bitmap_words) a.word_prefix[w] = run;
    run += c[q];
  }
  if (b + 1 == nb && !s_stopped) {
    const uint32_t winners = s_base + part[255];
    // winners below a word: the other blocks' prefixes may not be written
    // yet, so the sums and the words of its block are added up (one word for
    // the answer; some twenty more when the cache overflows)
    auto sum_below = [&](uint32_t w) -> uint32_t {  // by the whole block
      uint32_t v = 0;
      const uint32_t wb = w / kScanBlock;
      for (uint32_t i = t; i < wb; i += 256) v += a.block_sums[i];
      for (uint32_t i = wb * kScanBlock + t; i < w; i += 256) v += __popc(a.bitmap[i]);
      __syncthreads();
      part[t] = v;
      __syncthreads();
      for (uint32_t st = 128; st > 0; st >>= 1) {
        if (t < st) part[t] += part[t + st];
        __syncthreads();
      }
      return part[0];
    };
    const uint32_t ans = s_ans;
    const uint64_t room = s_room;
    uint32_t answer_rank = ~0u, overflow_e = ~0u;
    if (ans != ~0u)
      answer_rank = sum_below(ans >> 5) + (uint32_t)__popc(a.bitmap[ans >> 5] & ((1u << (ans & 31)) - 1));
    if (winners > room) {
      uint32_t lo = 0, hi = a.n_bitmap_words;
      while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (sum_below(mid) <= room)
          lo = mid;
        else
          hi = mid;
      }
      const uint32_t first = sum_below(lo);
      if (t == 0) {
        uint32_t m = a.bitmap[lo];
        for (uint32_t k = (uint32_t)room - first; k; --k) m &= m - 1;
        overflow_e = 32 * lo + (uint32_t)__ffs(m) - 1;
      }
    }
    if (t == 0) account_chunk(a, ans, answer_rank, winners, overflow_e);
  }
}

template <int W, bool kInl>
__global__ __launch_bounds__(256) void compact_winners(ChunkArgs a) {
  // (the chunk is accounted already, the stop code may be its own; a block left
  // by an earlier chunk, when a stop kept this one from being accounted, has
  // that chunk's number)
  if (a.ctrl->append != a.chunk_id) return;
  const uint32_t ans = a.ctrl->answer_e;
  const uint64_t row_base = a.ctrl->row_base, room = a.ctrl->room;
  for_survivors(a, [&](uint32_t sid, bool have) {
    if (!have) return;
    const uint32_t e = a.se[sid];
    const uint32_t word = a.bitmap[e >> 5];
    const uint32_t bit = 1u << (e & 31);
    if (!(word & bit)) return;
    const uint32_t rank = a.word_prefix[e >> 5] + (uint32_t)__popc(word & (bit - 1));
    if (ans != ~0u && e >= ans) return;
    if (rank < room) store_winner<W, kInl>(a, sid, e, row_base + rank);
  });
}

__global__ void account_large(ChunkArgs a) {
  if (a.st->stop) return;
  account_chunk(a, a.ctrl->answer_e, ~0u, 0, ~0u);  // (no winners: nothing is stored)
}

inline uint32_t grid_for(uint64_t n, uint64_t block, uint32_t cap = 0x7fffffffu) {
  uint64_t g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (uint32_t)g;
}

// Candidates (times 64) per wave of the one-candidate-per-lane generators:
// one iteration while the launch would leave waves idle (8192 fill the
// device at 32 per compute unit), up to 16.
uint32_t iterations_per_wave(uint64_t candidates) {
  return (uint32_t)std::min<uint64_t>(16, std::max<uint64_t>(1, candidates / (64 * 8192)));
}

size_t concat_lds(int W, const ConcatPart& p) { return (size_t)p.yt * 64 * W * 8 + (size_t)p.xi * W * 8; }

template <int W, bool kInl>
hipError_t launch_concat_w(const GenArgs& a, const ConcatSet& cs, hipStream_t s) {
  size_t lds = 0;
  for (uint32_t k = 0; k < cs.n; ++k) lds = std::max(lds, concat_lds(W, cs.p[k]));
  const uint32_t gt_lds = (lds + (size_t)a.n_pairs * 4 <= 60 * 1024) ? 1u : 0u;
  if (gt_lds) lds += (size_t)a.n_pairs * 4;
  const dim3 grid(cs.wgs);
  const bool shrt = a.max_len < 32;
  if (shrt && gt_lds)
    launch_timed(gen_concat<W, true, kInl, true>, grid, dim3(256), lds, s, a, cs);
  else if (shrt)
    launch_timed(gen_concat<W, true, kInl, false>, grid, dim3(256), lds, s, a, cs);
  else if (gt_lds)
    launch_timed(gen_concat<W, false, kInl, true>, grid, dim3(256), lds, s, a, cs);
  else
    launch_timed(gen_concat<W, false, kInl, false>, grid, dim3(256), lds, s, a, cs);
  return hipGetLastError();
}

template <int W, bool kInl>
hipError_t launch_gen_w(int op, const GenArgs& a, hipStream_t s) {
  const uint64_t per = (uint64_t)a.per_wave * 64;
  const uint64_t cnt = a.e1 - a.e0;
  switch (op) {
    case OP_CHAR:
      launch_timed(gen_char<W, kInl>, dim3(grid_for(cnt, 4 * per)), dim3(256), 0, s, a);
      break;
    case OP_QUESTION:
      launch_timed(gen_question<W, kInl>, dim3(grid_for(cnt, 4 * per)), dim3(256), 0, s, a);
      break;
    case OP_STAR:
      if constexpr (W <= 4) {
        if (star_by_wave(W, a)) {
          launch_timed(gen_star_wave<W, kInl>, dim3(grid_for(cnt, 4 * per)), dim3(256), 0, s, a);
          break;
        }
      }
      launch_timed(gen_star<W, kInl>, dim3(grid_for(cnt, per)), dim3(256), 0, s, a);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

// W words per language; inl selects the inline-key table (only with W = 1).
#define REI_DISPATCH_WI(W, INL, CALL)                                        \
  switch (W) {                                                               \
    case 1:                                                                  \
      if (INL) {                                                             \
        constexpr int kW = 1;                                                \
        constexpr bool kI = true;                                            \
        CALL;                                                                \
      } else {                                                               \
        constexpr int kW = 1;                                                \
        constexpr bool kI = false;                                           \
        CALL;                                                                \
      }                                                                      \
      break;                                                                 \
    case 2: { constexpr int kW = 2; constexpr bool kI = false; CALL; } break;   \
    case 4: { constexpr int kW = 4; constexpr bool kI = false; CALL; } break;   \
    case 8: { constexpr int kW = 8; constexpr bool kI = false; CALL; } break;   \
    case 16: { constexpr int kW = 16; constexpr bool kI = false; CALL; } break; \
    case 32: { constexpr int kW = 32; constexpr bool kI = false; CALL; } break; \
    default: return hipErrorInvalidValue;                                    \
  }

hipError_t launch_fill(uint64_t* p, uint64_t n, uint64_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u64, dim3(grid_for(n, 256, 65536)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_search_reset(const ResetArgs& a, hipStream_t s) {
  if (!a.ctrl || !a.st || (a.n_levels && !a.levels) || (a.n_slot_words && !a.slots)) return hipErrorInvalidValue;
  for (int b = 0; b < 2; ++b)
    if (a.bitmap_words[b] && !a.bitmap[b]) return hipErrorInvalidValue;
  const uint64_t most = std::max<uint64_t>({a.n_levels, a.n_slot_words, a.bitmap_words[0], a.bitmap_words[1], 1});
  hipLaunchKernelGGL(search_reset, dim3(grid_for(most, 1024, 65536)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_rehash(int W, bool inl, const uint64_t* rows, uint64_t nrows, uint64_t* slots,
                         uint64_t slot_mask, hipStream_t s) {
  if (nrows == 0) return hipSuccess;
  REI_DISPATCH_WI(W, inl, hipLaunchKernelGGL((rehash_rows<kW, kI>), dim3(grid_for(nrows, 256, 65536)),
                                             dim3(256), 0, s, rows, nrows, slots, slot_mask));
  return hipGetLastError();
}

// Adds a launch's survivor slots and ranges to the chunk's; false when they
// do not fit 32-bit indices.
bool take_slots(SlotPlan* sp, uint64_t slots, uint64_t regions) {
  if (sp->slots + slots > kMaxSlots || sp->regions + regions > kMaxSlots) return false;
  sp->slots += slots;
  sp->regions += regions;
  return true;
}

hipError_t plan_gen(int W, int op, GenArgs* a, SlotPlan* sp) {
  const uint64_t cnt = a->e1 - a->e0;
  if (a->e1 <= a->e0) return hipErrorInvalidValue;
  // (a workgroup per group of a star is one wave of candidates)
  const bool by_group = op == OP_STAR && !star_by_wave(W, *a);
  a->per_wave = by_group ? (uint32_t)std::min<uint64_t>(16, std::max<uint64_t>(1, cnt / (64 * 4096)))
                              : iterations_per_wave(cnt);
  const uint64_t per = (uint64_t)a->per_wave * 64;
  const uint64_t waves = by_group ? (cnt + per - 1) / per : 4 * ((cnt + 4 * per - 1) / (4 * per));
  a->slot0 = (uint32_t)sp->slots;
  a->reg0 = (uint32_t)sp->regions;
  return take_slots(sp, waves * per, waves) ? hipSuccess : hipErrorInvalidConfiguration;
}

hipError_t plan_concat_set(int W, const GenArgs& a, ConcatSet* cs, SlotPlan* sp) {
  if (cs->n == 0 || cs->n > (uint32_t)kMaxConcatParts) return hipErrorInvalidValue;
  // tiles in LDS: at most 32 KB
  const uint32_t yt_cap = (uint32_t)std::max(1, std::min(kConcatYT, 32768 / (512 * W)));
  // per part: uniform rows per workgroup at most concat_xi (16 by default),
  // fewer (down to 4), then fewer tiles, while its grid has under concat_wg
  // workgroups (2048 by default)
  const uint64_t target = a.concat_wg ? a.concat_wg : 2048;
  const uint32_t xi_max = a.concat_xi ? std::min<uint32_t>(a.concat_xi, 64) : 16;
  uint64_t wgs_total = 0;
  for (uint32_t k = 0; k < cs->n; ++k) {
    ConcatPart& p = cs->p[k];
    const uint64_t nR = p.rcount;
    if (nR == 0 || p.e1 <= p.e0) return hipErrorInvalidValue;
    p.i_lo = p.e0 / nR;
    p.i_hi = (p.e1 - 1) / nR;
    const uint64_t rowsx = p.i_hi - p.i_lo + 1;
    // the operand across the lanes: the one whose tiles of 64 fill better
    // (fewer wave iterations; left rows when the right level is small)
    p.left = ((rowsx + 63) / 64) * nR < rowsx * ((nR + 63) / 64) ? 1u : 0u;
    const uint64_t nT = ((p.left ? rowsx : nR) + 63) / 64, nU = p.left ? nR : rowsx;
    uint32_t yt = (uint32_t)std::min<uint64_t>(yt_cap, nT);
    uint32_t xi = xi_max;
    auto wgs = [&](uint32_t y, uint32_t x) { return ((nT + y - 1) / y) * ((nU + x - 1) / x); };
    while (xi > 4 && (wgs(yt, xi) < target || xi >= 2 * nU)) xi /= 2;
    while (yt > 1 && wgs(yt, xi) < target) yt /= 2;
    const uint64_t gx = (nT + yt - 1) / yt, gy = (nU + xi - 1) / xi;
    p.yt = yt;
    p.xi = xi;
    p.gx = (uint32_t)gx;
    p.wg0 = (uint32_t)wgs_total;
    p.slot0 = (uint32_t)sp->slots;
    p.reg0 = (uint32_t)sp->regions;
    wgs_total += gx * gy;
    if (wgs_total > 0x7fffffffull || !take_slots(sp, nT * nU * 64, gx * gy * 4)) return hipErrorInvalidConfiguration;
  }
  cs->wgs = (uint32_t)wgs_total;
  return hipSuccess;
}

// Pairs (i, j), i < j, of m rows before row i's first.
uint64_t pairs_before(uint64_t i, uint64_t m) { return i * m - i * (i + 1) / 2; }

// Pairs of a part's kept rows that come before candidate e of the block.
uint64_t kept_before(const UnionPart& p, uint64_t e) {
  // kept rows below row r
  auto below = [&](uint64_t r) -> uint64_t {
    uint64_t n = std::min(r, p.n0);
    if (r > p.s0) n += std::min(r - p.s0, p.n1);
    if (!p.same && r > p.us) n += r - p.us;
    return n;
  };
  if (!p.same) {
    const uint64_t cols = p.n0 + p.n1 + (p.rcount - p.us), i = e / p.rcount, i0 = p.e0 / p.rcount;
    return (i - i0) * cols + below(e - i * p.rcount);
  }
  const uint64_t m = p.n0 + p.n1, n = p.rcount;
  if (e >= pairs_before(n, n)) return m ? pairs_before(m - 1, m) : 0;
  uint64_t lo = 0, hi = n;  // row of e: the last whose first pair is at or before it
  while (hi - lo > 1) {
    const uint64_t mid = lo + (hi - lo) / 2;
    (pairs_before(mid, n) <= e ? lo : hi) = mid;
  }
  const uint64_t i = lo, j = i + 1 + (e - pairs_before(i, n));
  const uint64_t a = below(i);
  if (a + 1 >= m) return m ? pairs_before(m - 1, m) : 0;
  if (below(i + 1) == a) return pairs_before(a, m);  // row i is not kept
  return pairs_before(a, m) + (std::max(below(j), a + 1) - (a + 1));
}

hipError_t plan_union_set(UnionSet* us, SlotPlan* sp) {
  if (us->n == 0 || us->n > (uint32_t)kMaxUnionParts) return hipErrorInvalidValue;
  uint64_t total = 0, wgs = 0;
  for (uint32_t k = 0; k < us->n; ++k) {
    UnionPart& p = us->p[k];
    if (p.e1 <= p.e0 || p.lcount == 0 || p.rcount == 0 || p.n0 + p.n1 > p.rcount || p.us > p.rcount)
      return hipErrorInvalidValue;
    p.k0 = kept_before(p, p.e0);
    p.lanes = kept_before(p, p.e1) - p.k0;
    total += p.lanes;
  }
  us->per_wave = iterations_per_wave(total);
  const uint64_t per = 4ull * 64 * us->per_wave;  // candidates per workgroup
  for (uint32_t k = 0; k < us->n; ++k) {
    UnionPart& p = us->p[k];
    const uint64_t g = (p.lanes + per - 1) / per;
    p.wg0 = (uint32_t)wgs;
    p.slot0 = (uint32_t)sp->slots;
    p.reg0 = (uint32_t)sp->regions;
    wgs += g;
    if (wgs > 0x7fffffffull || !take_slots(sp, g * per, 4 * g)) return hipErrorInvalidConfiguration;
  }
  us->wgs = (uint32_t)wgs;
  return hipSuccess;
}

hipError_t launch_gen(int W, int op, const GenArgs& a, hipStream_t s) {
  if (a.e1 <= a.e0 || a.per_wave == 0 || !a.reg) return hipErrorInvalidValue;
  REI_DISPATCH_WI(W, a.inl, return (launch_gen_w<kW, kI>(op, a, s)));
  return hipGetLastError();
}

hipError_t launch_union_set(int W, const GenArgs& a, const UnionSet& us, hipStream_t s) {
  if (us.wgs == 0) return hipSuccess;  // no pair is left
  if (!a.rows || !a.aux || !a.st || !a.ctrl || !a.reg) return hipErrorInvalidValue;
  REI_DISPATCH_WI(W, a.inl,
                  launch_timed(gen_union<kW, kI>, dim3(us.wgs), dim3(256), 0, s, a, us));
  return hipGetLastError();
}

hipError_t launch_concat_set(int W, const GenArgs& a, const ConcatSet& cs, hipStream_t s) {
  if (!a.rows || !a.gt_off || !a.gt_pair || !a.st || !a.ctrl || !a.reg || cs.wgs == 0) return hipErrorInvalidValue;
  REI_DISPATCH_WI(W, a.inl, return (launch_concat_w<kW, kI>(a, cs, s)));
  return hipGetLastError();
}

constexpr uint64_t kPairItemsMax = 1024;  // gen_pieces items up to which a wide item takes two waves
constexpr uint64_t kQuadItemsMax = 256;   // ... and up to which four

hipError_t launch_gen_pieces(int W, const GenArgs& a, const PieceArgs& p, hipStream_t s) {
  if (p.items == 0) return hipSuccess;
  if (W > kPiecesMaxW || p.n > (uint32_t)kMaxPieces) return hipErrorInvalidValue;
  // every table a piece reads must be there, and every range non-empty
  if (!a.char_index || !a.gt_off || !a.gt_pair || !a.len_off || !a.st || !a.ctrl) return hipErrorInvalidValue;
  for (uint32_t k = 0; k < p.n; ++k) {
    const PieceD& d = p.p[k];
    if (d.op != OP_CHAR && !a.rows) return hipErrorInvalidValue;  // (no rows yet: only characters)
    if (d.e1 <= d.e0 || (k && d.item0 < p.p[k - 1].item0) || d.item0 >= p.items) return hipErrorInvalidValue;
    if (d.op == OP_CONCAT && (d.rcount == 0 || d.lcount == 0 || d.nt == 0)) return hipErrorInvalidValue;
    if ((d.op == OP_UNION && !d.same && d.rcount == 0) || (d.op != OP_CHAR && d.lcount == 0))
      return hipErrorInvalidValue;
  }
  // few items (one item's latency is the launch's): from 16 words, two or
  // four waves per concatenation or star item
  const int split = W < 16 ? 1 : p.items <= kQuadItemsMax ? 4 : p.items <= kPairItemsMax ? 2 : 1;
  const uint32_t grid = (uint32_t)std::min<uint64_t>((p.items * split + 3) / 4, 4096);
#define REI_PIECES_SPLIT(WW)                                                                   \
  do {                                                                                         \
    if (split == 4)                                                                            \
      launch_timed(gen_pieces<WW, false, 4>, dim3(grid), dim3(256), 0, s, a, p);                \
    else if (split == 2)                                                                       \
      launch_timed(gen_pieces<WW, false, 2>, dim3(grid), dim3(256), 0, s, a, p);                \
    else                                                                                       \
      launch_timed(gen_pieces<WW, false, 1>, dim3(grid), dim3(256), 0, s, a, p);                \
  } while (0)
  switch (W) {
    case 1:
      if (a.inl)
        launch_timed(gen_pieces<1, true, 1>, dim3(grid), dim3(256), 0, s, a, p);
      else
        launch_timed(gen_pieces<1, false, 1>, dim3(grid), dim3(256), 0, s, a, p);
      break;
    case 2: launch_timed(gen_pieces<2, false, 1>, dim3(grid), dim3(256), 0, s, a, p); break;
    case 4: launch_timed(gen_pieces<4, false, 1>, dim3(grid), dim3(256), 0, s, a, p); break;
    case 8: launch_timed(gen_pieces<8, false, 1>, dim3(grid), dim3(256), 0, s, a, p); break;
    case 16: REI_PIECES_SPLIT(16); break;
    case 32: REI_PIECES_SPLIT(32); break;
    default: return hipErrorInvalidValue;
  }
#undef REI_PIECES_SPLIT
  return hipGetLastError();
}

// Workgroups that walk a chunk's survivors: a thread per possible survivor of
// the pieces, a wave per range, 8192 workgroups at most.
uint32_t survivor_grid(const ChunkArgs& a) {
  return grid_for(std::max<uint64_t>(a.dense_cap, 64ull * a.n_reg), 256, 8192);
}

hipError_t launch_insert(int W, const ChunkArgs& a, hipStream_t s) {
  if (!a.bitmap || (a.clear_words && !a.bitmap_next) || (a.n_reg && !a.reg)) return hipErrorInvalidValue;
  REI_DISPATCH_WI(W, a.inl, hipLaunchKernelGGL((insert_survivors<kW, kI>), dim3(survivor_grid(a)), dim3(256), 0, s,
                                               a));
  return hipGetLastError();
}

bool finalize_in_one_workgroup(int W, uint64_t len) {
  // one workgroup moves at most kSmallCopyWords words of rows: a chunk
  // with more is finalized by the grid kernels, spread over the device
  return len <= kSmallChunk && len * (uint64_t)W <= kSmallCopyWords;
}

hipError_t launch_finalize(int W, const ChunkArgs& a, hipStream_t s) {
  if (finalize_in_one_workgroup(W, a.len)) {
    if (a.n_reg) return hipErrorInvalidValue;  // (reads the pieces' survivors only)
    REI_DISPATCH_WI(W, a.inl, hipLaunchKernelGGL((finalize_small<kW, kI>), dim3(1), dim3(1024), 0, s, a));
    return hipGetLastError();
  }
  const uint32_t g = survivor_grid(a);
  if (a.n_bitmap_words <= kScanSingleWords) {
    hipLaunchKernelGGL(scan_single, dim3(1), dim3(1024), 0, s, a);
  } else {
    const uint32_t nb = (a.n_bitmap_words + kScanBlock - 1) / kScanBlock;
    hipLaunchKernelGGL(scan_reduce, dim3(nb), dim3(256), 0, s, a);
    hipLaunchKernelGGL(scan_down, dim3(nb), dim3(256), 0, s, a, nb);
  }
  REI_DISPATCH_WI(W, a.inl, hipLaunchKernelGGL((compact_winners<kW, kI>), dim3(g), dim3(256), 0, s, a));
  return hipGetLastError();
}

namespace {
__global__ void noop_kernel() {}

__global__ __launch_bounds__(kMaxMarks) void level_marks(MarksArgs a) {
  const uint32_t k = threadIdx.x;
  if (k < a.n) {
    const MarksArgs::Entry& m = a.m[k];
    const uint64_t* aux = a.aux + m.lstart;
    uint64_t lo = 0, hi = a.levels[m.level];
    while (lo < hi) {
      const uint64_t mid = lo + (hi - lo) / 2;
      if (aux[mid] < m.thr)
        lo = mid + 1;
      else
        hi = mid;
    }
    a.out[k] = lo;
  }
  __threadfence_system();
  __syncthreads();
  if (k == 0) __hip_atomic_store(a.seq_out, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
}

hipError_t launch_level_marks(const MarksArgs& a, hipStream_t s) {
  if (!a.aux || !a.levels || !a.out || !a.seq_out || a.n > kMaxMarks) return hipErrorInvalidValue;
  hipLaunchKernelGGL(level_marks, dim3(1), dim3(kMaxMarks), 0, s, a);
  return hipGetLastError();
}

namespace {
// Decodes level index e of level c: the characters of cost c, then r? over
// c - c2, r* over c - c3, concatenations by left cost and unions by left cost
// (Sec. 3 enumeration order; the counts of the levels below c are final).
__device__ bool tree_decode_index(const TreeArgs& t, const uint64_t* lstart, const uint64_t* lcount, uint32_t c,
                                  uint64_t e, uint32_t* op, uint64_t* a, uint64_t* b) {
  const int64_t c1 = t.c1, cc = c;
  auto lc = [&](int64_t k) -> uint64_t { return (k >= c1 && k < cc) ? lcount[k] : 0ull; };
  *b = 0;
  uint32_t first = 0, cnt = 0;
  for (uint32_t k = 0; k < t.nsigma; ++k) {
    first += t.ccost[k] < c;
    cnt += t.ccost[k] == c;
  }
  if (e < cnt) {
    *op = OP_CHAR;
    *a = first + e;
    return true;
  }
  e -= cnt;
  uint64_t n = lc(cc - t.c2);
  if (e < n) {
    *op = OP_QUESTION;
    *a = lstart[cc - t.c2] + e;
    return true;
  }
  e -= n;
  n = lc(cc - t.c3);
  if (e < n) {
    *op = OP_STAR;
    *a = lstart[cc - t.c3] + e;
    return true;
  }
  e -= n;
  for (int64_t L = c1; cc - (int64_t)t.c4 - L >= c1; ++L) {
    const int64_t R = cc - t.c4 - L;
    n = lc(L) * lc(R);
    if (e < n) {
      *op = OP_CONCAT;
      *a = lstart[L] + e / lc(R);
      *b = lstart[R] + e % lc(R);
      return true;
    }
    e -= n;
  }
  for (int64_t L = c1; L <= cc - (int64_t)t.c5 - L; ++L) {
    const int64_t R = cc - t.c5 - L;
    const uint64_t x = lc(L), y = lc(R);
    n = (L < R) ? x * y : (x ? x * (x - 1) / 2 : 0);
    if (e < n) {
      *op = OP_UNION;
      if (L == R) {
        uint64_t i = 0, j = 0;
        tri_decode(e, x, &i, &j);
        *a = lstart[L] + i;
        *b = lstart[L] + j;
      } else {
        *a = lstart[L] + e / y;
        *b = lstart[R] + e % y;
      }
      return true;
    }
    e -= n;
  }
  return false;
}

__global__ __launch_bounds__(64) void decode_tree(TreeArgs t) {
  __shared__ uint64_t lstart[kTreeMaxLevels], lcount[kTreeMaxLevels];
  __shared__ uint64_t stk[64];
  const uint32_t ans_c = t.st->answer_cost;
  const uint64_t ans_e = t.st->answer_e;
  const bool have = t.st->stop == STOP_ANSWER && ans_c < kTreeMaxLevels && ans_c >= t.c1;
  // level sizes loaded by the whole wave, prefix sums by lane 0
  if (have)
    for (uint32_t c = threadIdx.x; c <= ans_c; c += blockDim.x) lcount[c] = c >= t.c1 ? t.levels[c] : 0ull;
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (!have) {
    t.out[0] = 0;
    return;
  }
  uint64_t start = 0;
  for (uint32_t c = 0; c <= ans_c; ++c) {
    lstart[c] = start;
    start += lcount[c];
  }
  uint32_t k = 0, sp = 0;
  bool ok = true;
  auto node = [&](uint64_t row, uint32_t c, uint64_t e) {
    uint32_t op = 0;
    uint64_t a = 0, b = 0;
    if (k >= t.max_nodes || sp + 2 > 64 || !tree_decode_index(t, lstart, lcount, c, e, &op, &a, &b)) {
      ok = false;
      return;
    }
    uint64_t* o = t.out + 1 + 4 * k++;
    o[0] = row;
    o[1] = op;
    o[2] = a;
    o[3] = b;
    if (op != OP_CHAR) stk[sp++] = a;
    if (op == OP_CONCAT || op == OP_UNION) stk[sp++] = b;
  };
  node(~0ull, ans_c, ans_e);
  while (ok && sp) {
    const uint64_t row = stk[--sp];
    uint32_t rc = 0;
    for (uint32_t c = t.c1; c < ans_c; ++c)
      if (row >= lstart[c] && row < lstart[c] + lcount[c]) rc = c;
    if (!rc) {
      ok = false;
      break;
    }
    node(row, rc, t.aux[row]);
  }
  t.out[0] = ok ? k : 0;
}
}  // namespace

hipError_t launch_decode_tree(const TreeArgs& t, hipStream_t s) {
  if (!t.levels || !t.aux || !t.st || !t.out || t.nsigma > kTreeMaxChars || t.max_nodes == 0)
    return hipErrorInvalidValue;
  launch_timed(decode_tree, dim3(1), dim3(64), 0, s, t);
  return hipGetLastError();
}

hipError_t set_hash_mask_kernels(uint64_t mask) {
  return hipMemcpyToSymbol(HIP_SYMBOL(g_hash_mask), &mask, sizeof(mask));
}

hipError_t launch_noop_timed(hipStream_t s) {
  launch_timed(noop_kernel, dim3(1), dim3(64), 0, s);
  return hipGetLastError();
}

hipError_t launch_account(const ChunkArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(account_large, dim3(1), dim3(1), 0, s, a);
  return hipGetLastError();
}


}  // namespace rei
