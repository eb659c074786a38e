// Beam search on lists of valid candidates (gfx950), for the bf16 MLPs that the list scorer takes.
//
// Secs. 3.1 and 4.1 search with a beam guided by V.  A layer is three launches: the scores of all
// slots' candidates (the LAYER form of k_whole: compact scores by list position and the first
// minimum of every 64 entries), the choice of the B smallest of them (k_beam_select), and per
// survivor its commit and the opening of its next decision (k_beam_advance).
#include <type_traits>
#include <utility>

#include "vf_internal.h"

namespace {

#include "vf_sched_dev.h"

#include "vf_score_dev.h"

#include "vf_layer_dev.h"

constexpr unsigned long long NO_KEY = ~0ull;
constexpr int SEL_THREADS = 1024;
constexpr int SEL_CAP = 2048;  // keys that the final sort takes

// Sorts `size` keys (a power of two from 128 on); complete for all threads.
__device__ __forceinline__ void sort_keys(unsigned long long *sorted, int size) {
  const int tid = threadIdx.x;
  // bitonic sort; a wave's 64 pairs of a step of stride 64 or less lie in the same 128 keys, so
  // that only the wider steps need the whole workgroup
  for (int len = 2; len <= size; len <<= 1)
    for (int stride = len >> 1; stride > 0; stride >>= 1) {
      if (stride >= 64 && len > 128) __syncthreads();
      if (tid < size / 2) {
        const int a = 2 * tid - (tid & (stride - 1)), b = a + stride;
        const unsigned long long x = sorted[a], y = sorted[b];
        if ((x > y) == ((a & len) == 0)) { sorted[a] = y; sorted[b] = x; }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  __syncthreads();
}

// The smallest keys of key(0) .. key(n - 1) (NO_KEY = none, all others different), sorted, in
// sorted[0..return value): the `want` smallest ones and possibly more, at most SEL_CAP.  A threshold
// is bisected over the 64-bit keys until at least `want` and at most 4 * want keys lie below it
// (the keys are all different, so there is such a threshold), and only those are sorted.
// R: keys a thread keeps in registers (n <= 1024 R), 0 = they are evaluated again in every pass.
// key(i) is called for i >= n too and must then only be safe to evaluate.
template <int R, typename KEY>
__device__ int block_select(KEY key, uint32_t n, int want, unsigned long long *sorted) {
  __shared__ unsigned int cnt[3][3];
  __shared__ unsigned long long range[2];
  const int tid = threadIdx.x, lane = tid & 63;
  unsigned long long reg[R > 0 ? R : 1];
  __syncthreads();  // (the shared words may still be in use by a call before)
  if (tid < 9) cnt[tid / 3][tid % 3] = 0u;
  if (tid == 0) { range[0] = NO_KEY; range[1] = 0ull; }
  // (no branch around a load: all of them are under way at once)
  if (R > 0) {
#pragma unroll
    for (int e = 0; e < R; ++e) reg[e] = key((uint32_t)e * SEL_THREADS + tid);
#pragma unroll
    for (int e = 0; e < R; ++e)
      if ((uint32_t)e * SEL_THREADS + tid >= n) reg[e] = NO_KEY;
  }
  auto each = [&](auto f) __attribute__((always_inline)) {
    if (R > 0) {
#pragma unroll
      for (int e = 0; e < R; ++e) f(reg[e]);
    } else {
      for (uint32_t i0 = 0; i0 < n; i0 += SEL_THREADS) {
        const unsigned long long k = key(i0 + tid);
        f(i0 + tid < n ? k : NO_KEY);
      }
    }
  };
  // (counts by ballots: one scalar sum per wave, in every lane)
  auto count_upto = [&](unsigned long long mid) __attribute__((always_inline)) {
    unsigned int c = 0u;
    each([&](unsigned long long k) { c += (unsigned int)__popcll(__ballot(k <= mid)); });
    return c;
  };
  unsigned long long mn = NO_KEY, mx = 0ull;
  each([&](unsigned long long k) {
    mn = k < mn ? k : mn;
    if (k != NO_KEY) mx = k > mx ? k : mx;
  });
  const unsigned int have = count_upto(NO_KEY - 1ull);
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long a = __shfl_down(mn, off), b = __shfl_down(mx, off);
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
  }
  __syncthreads();
  if (lane == 0 && have) {
    atomicMin(&range[0], mn);
    atomicMax(&range[1], mx);
    atomicAdd(&cnt[0][0], have);
  }
  __syncthreads();
  unsigned int below = cnt[0][0];  // keys <= hi
  const unsigned int most = 4 * want < 256 ? 256u : 4 * want > SEL_CAP ? (unsigned int)SEL_CAP : 4u * want;
  unsigned long long lo = range[0], hi = range[1];
  // (three thresholds a round: what a round costs is the meeting of the sixteen waves)
  for (int r = 1; below > most; ++r) {  // (the same in every thread)
    const unsigned long long step = (hi - lo) / 4 + 1ull;  // lo + 3 step may pass hi: it then counts all
    unsigned int c[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) c[q] = count_upto(lo + (unsigned long long)q * step);
    unsigned int *const slot = cnt[r % 3];
    if (lane == 0) {
#pragma unroll
      for (int q = 0; q < 3; ++q)
        if (c[q]) atomicAdd(&slot[q], c[q]);
    }
    if (tid < 3) cnt[(r + 1) % 3][tid] = 0u;
    __syncthreads();
    bool found = false;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const unsigned int got = slot[q];
      if (!found && got >= (unsigned int)want) {
        found = true;
        below = got;
        hi = lo + (unsigned long long)q * step;
        if (q > 0) lo = lo + (unsigned long long)(q - 1) * step + 1ull;
      }
    }
    if (!found) lo = lo + 2ull * step + 1ull;
  }
  __syncthreads();
  if (tid == 0) cnt[0][0] = 0u;
  int size = 128;
  while (size < (int)below) size <<= 1;
  for (int i = tid; i < size; i += SEL_THREADS) sorted[i] = NO_KEY;
  __syncthreads();
  if (below)
    each([&](unsigned long long k) {
      if (k <= hi && k != NO_KEY) sorted[atomicAdd(&cnt[0][0], 1u)] = k;
    });
  __syncthreads();
  sort_keys(sorted, size);
  return (int)below;
}

// One pass of the selection for scorers that leave masked scores [slot][Mpad] by id: every block of 1024 R
// pairs is reduced to its `want` smallest, ordered by (value, index).  First pass (idx_in null): the
// values are the scores, index = slot * Mpad + candidate id, columns from M on are skipped; later ones
// read the pairs of the pass before.  sel_n (nullable, the last pass: one block) receives the count.  +inf and
// NaN never survive.  A layer of 4096 ids and 16 slots: 25 + 25 us with 16 rounds of block-wide minima,
// 10 + 7 now; 6000 ids and 64 slots: 3 x 25 us of sorting, 11 + 14 now.
template <int R>
__global__ __launch_bounds__(SEL_THREADS) void k_select_pass(const float *val_in, const int32_t *idx_in, uint32_t n, uint32_t M,
                                                             uint32_t Mpad, int want, float *val_out, int32_t *idx_out, int32_t *sel_n) {
  __shared__ unsigned long long sorted[SEL_CAP];
  const uint32_t base = blockIdx.x * (uint32_t)(SEL_THREADS * R);
  const uint32_t here = n - base < (uint32_t)(SEL_THREADS * R) ? n - base : (uint32_t)(SEL_THREADS * R);
  auto key = [&](uint32_t i) {
    const uint32_t at = base + (i < here ? i : 0u);
    const float v = val_in[at];
    if (idx_in) return idx_in[at] >= 0 ? topk_key(v, idx_in[at]) : NO_KEY;
    return v < __builtin_inff() && at % Mpad < M ? topk_key(v, (int32_t)at) : NO_KEY;
  };
  int found = block_select<R>(key, here, want, sorted);
  if (found > want) found = want;
  for (int r = threadIdx.x; r < want; r += SEL_THREADS) {
    const bool is = r < found;
    val_out[(size_t)blockIdx.x * want + r] = is ? topk_value(sorted[r]) : __builtin_inff();
    idx_out[(size_t)blockIdx.x * want + r] = is ? (int32_t)(uint32_t)sorted[r] : -1;
  }
  if (sel_n && threadIdx.x == 0) {
    sel_n[0] = found;
    if (found > 0) sel_n[1] = found;
  }
}

// block-wide first minimum of (v, c); every thread gets the result
__device__ void block_min(float &v, int32_t &c, float *sv, int32_t *sc) {
  for (int off = 32; off > 0; off >>= 1) {
    float ov = __shfl_down(v, off);
    int32_t oc = __shfl_down(c, off);
    take_min(v, c, ov, oc);
  }
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { sv[w] = v; sc[w] = c; }
  __syncthreads();
  v = sv[0]; c = sc[0];
  for (int k = 1; k < nw; ++k) take_min(v, c, sv[k], sc[k]);
}

// The same pass for up to four survivors, 2048 pairs per block: k rounds of a block-wide first minimum (one
// 4 us, four 8 us per pass).
__global__ __launch_bounds__(256) void k_topk_pass_few(const float *val_in, const int32_t *idx_in, uint32_t n,
                                                   uint32_t M, uint32_t Mpad, int k, float *val_out,
                                                   int32_t *idx_out, int32_t *sel_n) {
  __shared__ float sv[4];
  __shared__ int32_t sc[4];
  const uint32_t base = blockIdx.x * 2048u;
  float v[8];
  int32_t id[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t i = base + threadIdx.x + e * 256u;
    float s = __builtin_inff();
    int32_t ix = -1;
    if (i < n) {
      if (idx_in) {
        ix = idx_in[i];
        if (ix >= 0) s = val_in[i];
      } else if ((i % Mpad) < M) {
        const float t = val_in[i];
        if (t < s) { s = t; ix = (int32_t)i; }  // NaN and +inf never survive
      }
    }
    v[e] = s;
    id[e] = ix;
  }
  int found = 0;
  for (int r = 0; r < k; ++r) {
    float bv = __builtin_inff();
    int32_t bi = -1;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (id[e] >= 0 && (v[e] < bv || (v[e] == bv && (bi < 0 || id[e] < bi)))) { bv = v[e]; bi = id[e]; }
    block_min(bv, bi, sv, sc);
    if (threadIdx.x == 0) {
      val_out[(size_t)blockIdx.x * k + r] = bv;
      idx_out[(size_t)blockIdx.x * k + r] = bi;
    }
    if (bi >= 0) {
      ++found;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (id[e] == bi) id[e] = -1;  // indices are unique: only the owner retires it
    }
  }
  if (sel_n && threadIdx.x == 0) {
    sel_n[0] = found;
    if (found > 0) sel_n[1] = found;
  }
}

// The survivors of a layer: the `want` smallest of all scores, ordered by (score, slot, candidate
// id); +inf and NaN never survive.  The lists are in ascending id order, so list positions order
// as the ids do.  No part of 64 entries outside the `want` parts with the smallest minima can hold
// a survivor, so first those parts are chosen by their minima, then the survivors among their
// entries: one workgroup reads the parts' minima and at most 64 * want scores instead of sorting
// all of them (64 slots of the 100-layer network, 16384 ids each: 83 us in three launches before).
//
// One workgroup, so what counts is the number of rounds.  The minima are counted in SEL_BINS bins of equal width
// over their range; up to the bin in which the count reaches `want` (cut) a score can survive, behind it
// none can: the parts up to it already have that many smaller ones.  (A bin's number never falls as the value
// grows, whatever the rounding.)  The scores of those parts that lie up to the cut - a few more than `want` - are ranked
// by counting the smaller ones.  The bisection above (20 us for the same layers, 8.2 now) is left for what does
// not fit: more parts than threads, or more scores up to the cut than are sorted at once (equal scores, ranges that
// overflow).
constexpr int SEL_BINS = SEL_THREADS;
constexpr int SEL_RANK = 256;  // keys that are ranked by counting; more of them are sorted
struct SelBins { float lo, scale; };
__device__ __forceinline__ int sel_bin(const SelBins &b, float v) {
  const float f = (v - b.lo) * b.scale;  // (not a number only where the range is 0 or overflows: bin 0)
  return f >= (float)(SEL_BINS - 1) ? SEL_BINS - 1 : f > 0.0f ? (int)f : 0;
}
// The keys up to the cut, unordered, in keys[0..return value); -1: not chosen this way.  R: part minima per thread.
template <int R>
__device__ int beam_cut(const float *scores, const float *pval, const int32_t *pidx, uint32_t nmin, int nparts, const uint32_t *pub,
                        int64_t Mpad, int want, unsigned long long *keys, uint32_t *parts) {
  __shared__ unsigned int bins[SEL_BINS], wave_sum[SEL_THREADS / 64];
  __shared__ float wave_lo[SEL_THREADS / 64], wave_hi[SEL_THREADS / 64];
  __shared__ unsigned int nchosen, nkeys;
  __shared__ int cut_bin;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  float v[R];
  int32_t part[R];
#pragma unroll
  for (int e = 0; e < R; ++e) {
    const uint32_t i = (uint32_t)e * SEL_THREADS + tid, at = i < nmin ? i : 0u;
    v[e] = pval[at];  // (+inf where a part has no minimum)
    part[e] = pidx[at];
  }
  bins[tid] = 0u;
  if (tid == 0) { nchosen = nkeys = 0u; cut_bin = SEL_BINS - 1; }
  float lo = __builtin_inff(), hi = -__builtin_inff();
#pragma unroll
  for (int e = 0; e < R; ++e) {
    if ((uint32_t)e * SEL_THREADS + tid >= nmin || !(v[e] < __builtin_inff())) part[e] = -1;
    if (part[e] >= 0) { lo = fminf(lo, v[e]); hi = fmaxf(hi, v[e]); }
  }
  for (int off = 32; off > 0; off >>= 1) { lo = fminf(lo, __shfl_xor(lo, off)); hi = fmaxf(hi, __shfl_xor(hi, off)); }
  if (lane == 0) { wave_lo[w] = lo; wave_hi[w] = hi; }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < SEL_THREADS / 64; ++k) { lo = fminf(lo, wave_lo[k]); hi = fmaxf(hi, wave_hi[k]); }
  SelBins b;
  b.lo = lo;
  b.scale = (float)(SEL_BINS - 1) / (hi - lo);
#pragma unroll
  for (int e = 0; e < R; ++e)
    if (part[e] >= 0) atomicAdd(&bins[sel_bin(b, v[e])], 1u);
  __syncthreads();
  const unsigned int mine = bins[tid];
  unsigned int upto = mine;
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned int o = __shfl_up(upto, off);
    if (lane >= off) upto += o;
  }
  if (lane == 63) wave_sum[w] = upto;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < SEL_THREADS / 64; ++k)
    if (k < w) upto += wave_sum[k];
  if (upto >= (unsigned int)want && upto - mine < (unsigned int)want) cut_bin = tid;
  __syncthreads();
  const int cut = cut_bin;
#pragma unroll
  for (int e = 0; e < R; ++e)
    if (part[e] >= 0 && sel_bin(b, v[e]) <= cut) {
      const unsigned int at = atomicAdd(&nchosen, 1u);
      if (at < SEL_THREADS) parts[at] = (uint32_t)part[e];
    }
  __syncthreads();
  const int np = (int)nchosen;
  if (np > SEL_THREADS) return -1;
  // (a wave takes a part, a lane an entry; four parts' loads under way at once)
  for (int q0 = w; q0 < np; q0 += 4 * (SEL_THREADS / 64)) {
    float s[4];
    uint32_t at[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int q = q0 + e * (SEL_THREADS / 64);
      const uint32_t p = parts[q < np ? q : q0], slot = p / (uint32_t)nparts, entry = (p - slot * (uint32_t)nparts) * 64u + lane;
      const uint32_t count = pub[(size_t)slot * VF_PUB_WORDS + VF_PUB_COUNT];
      at[e] = slot * (uint32_t)Mpad + (entry < (uint32_t)Mpad ? entry : 0u);
      s[e] = scores[at[e]];
      if (q >= np || entry >= count) s[e] = __builtin_inff();
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (s[e] < __builtin_inff() && sel_bin(b, s[e]) <= cut) {
        const unsigned int k = atomicAdd(&nkeys, 1u);
        if (k < SEL_CAP) keys[k] = topk_key(s[e], (int32_t)at[e]);
      }
  }
  __syncthreads();
  return nkeys <= SEL_CAP ? (int)nkeys : -1;
}
// keys[0..n) in order (n <= SEL_CAP, all different): up to SEL_RANK four threads count the keys below one.
__device__ void order_keys(unsigned long long *keys, int n) {
  const int tid = threadIdx.x;
  if (n <= SEL_RANK) {
    const bool on = (tid >> 2) < n;
    const unsigned long long mine = keys[on ? tid >> 2 : 0];
    int below = 0;
#pragma unroll 4
    for (int i = tid & 3; i < n; i += 4) below += keys[i] < mine ? 1 : 0;
    below += __shfl_xor(below, 1);
    below += __shfl_xor(below, 2);
    __syncthreads();
    if (on && (tid & 3) == 0) keys[below] = mine;
    __syncthreads();
  } else {
    int size = 128;
    while (size < n) size <<= 1;
    for (int i = n + tid; i < size; i += SEL_THREADS) keys[i] = NO_KEY;
    __syncthreads();
    sort_keys(keys, size);
  }
}

__global__ __launch_bounds__(SEL_THREADS) void k_beam_select(const float *scores, const float *pval, const int32_t *pidx,
                                                             const uint32_t *n_minima, int nparts, const uint32_t *list, const uint32_t *pub,
                                                             const int32_t *space, int64_t Mpad, int want, float *sel_val,
                                                             int32_t *sel_idx, int32_t *sel_n) {
  __shared__ unsigned long long sorted[SEL_CAP];
  __shared__ uint32_t parts[SEL_THREADS];
  __shared__ vf_space sp;
  const int tid = threadIdx.x;
  for (int i = tid; i < (int)(sizeof(vf_space) / 4); i += SEL_THREADS) reinterpret_cast<int32_t *>(&sp)[i] = space[i];
  const uint32_t nmin = n_minima[0];
  int found = nmin <= 2 * SEL_THREADS    ? beam_cut<2>(scores, pval, pidx, nmin, nparts, pub, Mpad, want, sorted, parts)
              : nmin <= 8 * SEL_THREADS  ? beam_cut<8>(scores, pval, pidx, nmin, nparts, pub, Mpad, want, sorted, parts)
              : nmin <= 32 * SEL_THREADS ? beam_cut<32>(scores, pval, pidx, nmin, nparts, pub, Mpad, want, sorted, parts)
                                         : -1;
  if (found >= 0) {
    order_keys(sorted, found);
  } else {
    auto part_key = [&](uint32_t i) {
      const uint32_t at = i < nmin ? i : 0u;
      const float v = pval[at];  // (+inf where a part has no minimum)
      const int32_t part = pidx[at];
      return v < __builtin_inff() ? topk_key(v, part) : NO_KEY;
    };
    int np = nmin <= 4 * SEL_THREADS    ? block_select<4>(part_key, nmin, want, sorted)
             : nmin <= 16 * SEL_THREADS ? block_select<16>(part_key, nmin, want, sorted)
                                        : block_select<0>(part_key, nmin, want, sorted);
    if (np > want) np = want;
    if (tid < np) parts[tid] = (uint32_t)sorted[tid];
    if (tid == 0 && np == 0) parts[0] = 0u;
    __syncthreads();
    const uint32_t nent = (uint32_t)np * 64u;
    auto entry_key = [&](uint32_t i) {
      const uint32_t part = parts[i < nent ? i >> 6 : 0u], slot = part / (uint32_t)nparts;
      const uint32_t entry = (part - slot * (uint32_t)nparts) * 64u + (i & 63u);
      const uint32_t at = slot * (uint32_t)Mpad + (entry < (uint32_t)Mpad ? entry : 0u);
      const uint32_t count = pub[(size_t)slot * VF_PUB_WORDS + VF_PUB_COUNT];
      const float s = scores[at];
      return entry < count && s < __builtin_inff() ? topk_key(s, (int32_t)at) : NO_KEY;
    };
    found = nent <= 4 * SEL_THREADS    ? block_select<4>(entry_key, nent, want, sorted)
            : nent <= 16 * SEL_THREADS ? block_select<16>(entry_key, nent, want, sorted)
                                       : block_select<0>(entry_key, nent, want, sorted);
  }
  if (found > want) found = want;
  for (int r = tid; r < want; r += SEL_THREADS) {
    const bool is = r < found;
    const uint32_t at = is ? (uint32_t)sorted[r] : 0u, slot = at / (uint32_t)Mpad;
    sel_val[r] = is ? topk_value(sorted[r]) : __builtin_inff();
    sel_idx[r] = is ? (int32_t)(slot * (uint32_t)Mpad + id_of(sp, unpack_digits(list[at]))) : -1;
  }
  if (tid == 0) {
    sel_n[0] = found;
    if (found > 0) sel_n[1] = found;
  }
}

// Survivor j of a layer: its parent's schedule is copied into slot j of the other table set, its
// candidate becomes the decision of the layer, and (open) the next decision is opened for the
// scorer.  The next context comes from the parent's rows in the old tables and the winner's rows in
// LDS, so nothing waits for the copies.  A slot without a survivor is cleared; if the layer has none
// at all the schedules end: every slot is carried over unchanged and marked dead.
// Two workgroups per slot: one goes on to the next decision, the other carries the parent's rows over.
template <int RT, int AHEAD>
__global__ __launch_bounds__(512) void k_beam_advance(Tables t, AltTables nw, int stage, int open, int64_t Mpad,
                                                      const float *sel_val, const int32_t *sel_idx, const int32_t *sel_n,
                                                      vf_fast_dev md, const uint32_t *pub_cur, uint32_t *pub, uint32_t *list) {
  __shared__ AdvanceShared sh;
  const int tid = threadIdx.x, lane = tid & 63, width = (int)gridDim.x / 2, S = t.S;
  const bool carries = (int)blockIdx.x >= width;
  const int j = (int)blockIdx.x - (carries ? width : 0);
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nsel = sel_n[0];
  const size_t dst = (size_t)j * S;
  int src_slot = -1;
  int32_t cid = -1;
  if (nsel == 0) src_slot = j;
  else if (j < nsel) { src_slot = sel_idx[j] / (int32_t)Mpad; cid = sel_idx[j] % (int32_t)Mpad; }
  if (carries) {
    const int rows = nsel == 0 ? S : stage;  // committed rows to carry over
    const size_t src = (size_t)(src_slot < 0 ? 0 : src_slot) * S;
    const int32_t *const cf = t.cf + src * 64, *const states = t.states + src * 16, *const cids = t.cids + src;
    const int32_t *const prefix = t.prefix + (size_t)(src_slot < 0 ? 0 : src_slot) * (S + 1) * 2;
    const float *const vals = t.vals + src;
    int32_t *const ncf = nw.cf + dst * 64, *const nst = nw.states + dst * 16, *const nci = nw.cids + dst;
    int32_t *const npre = nw.prefix + (size_t)j * (S + 1) * 2;
    float *const nva = nw.vals + dst;
    if (src_slot >= 0) {
#pragma unroll 4
      for (int i = tid; i < rows * 16; i += 512) reinterpret_cast<int4 *>(ncf)[i] = reinterpret_cast<const int4 *>(cf)[i];
      for (int i = tid; i < rows * 4; i += 512) reinterpret_cast<int4 *>(nst)[i] = reinterpret_cast<const int4 *>(states)[i];
      for (int i = tid; i < rows; i += 512) { nci[i] = cids[i]; nva[i] = vals[i]; }
      // (the entries behind the layer's own are the commit's)
      for (int i = tid; i < (S + 1) * 2; i += 512)
        if (nsel == 0 || i < (stage + 1) * 2) npre[i] = prefix[i];
        else if (i >= (stage + 2) * 2) npre[i] = 0;
    } else {
      for (int i = tid; i < (stage + 1) * 64; i += 512) ncf[i] = 0;
      for (int i = tid; i < (stage + 1) * 16; i += 512) nst[i] = 0;
      for (int i = tid; i <= stage; i += 512) { nci[i] = -1; nva[i] = __builtin_inff(); }
      for (int i = tid; i < (S + 1) * 2; i += 512) npre[i] = 0;
    }
    return;
  }
  if (cid >= 0) {
    fetch_opened(sh, pub_cur + (size_t)src_slot * VF_PUB_WORDS, tid);
    if (tid == 0) { sh.cid = cid; sh.val = sel_val[j]; }
    Tables tn = t;
    tn.states = nw.states; tn.cf = nw.cf; tn.prefix = nw.prefix; tn.cids = nw.cids; tn.alive = nw.alive; tn.vals = nw.vals;
    advance_layer<RT, AHEAD>(sh, t, tn, src_slot, j, stage, open, md, pub + (size_t)j * VF_PUB_WORDS, list + (size_t)j * Mpad,
                             tid, w, lane);
    if (tid == 256) {  // (the thread that advance_layer has mark the dead)
      nw.alive[j] = sh.sums[2] ? 1 : 0;
      if (!sh.sums[2]) t.err[0] = 1;  // cannot happen: only valid candidates have finite scores
    }
  } else if (tid == 0) {
    nw.alive[j] = 0;
    if (open) pub[(size_t)j * VF_PUB_WORDS + VF_PUB_COUNT] = 0u;
  }
}

}  // namespace

// The survivors of the masked scores in d_scores: d_sel_val / d_sel_idx / d_sel_n.
int vfk_beam_select(vf_ctx *c) {
  // (3 slots of 6000 ids, two layers: 88 us with k_topk_pass_few, 96 without; 8 slots: 145 against 107)
  const int k = c->B;
  const bool few = k <= 4;
  // pairs of one block: the last pass, the others
  const uint32_t MOST = few ? 2048 : 16 * SEL_THREADS, BLOCK = few ? 2048 : 4 * SEL_THREADS;
  uint32_t n = (uint32_t)((size_t)c->B * c->Mpad);
  const size_t want = n > MOST ? (size_t)((n + BLOCK - 1) / BLOCK) * k : 0;
  if (want > c->tk_elems) {
    if (c->d_tk_val) { VF_HIP(c, hipStreamSynchronize(c->stream)); (void)hipFree(c->d_tk_val); (void)hipFree(c->d_tk_idx); }
    c->d_tk_val = nullptr; c->d_tk_idx = nullptr; c->tk_elems = 0;
    if (hipMalloc((void **)&c->d_tk_val, want * 8) != hipSuccess || hipMalloc((void **)&c->d_tk_idx, want * 8) != hipSuccess) {
      (void)hipGetLastError();
      return VF_ENOMEM;
    }
    c->tk_elems = want;
  }
  // (buffers alternate between the two halves; a pass leaves at most a quarter of its pairs: k <= 1024)
  float *va = c->d_tk_val, *vb = va ? va + want : nullptr;
  int32_t *ia = c->d_tk_idx, *ib = ia ? ia + want : nullptr;
  const float *vin = c->d_scores;
  const int32_t *iin = nullptr;
  while (n > MOST) {
    const uint32_t blocks = (n + BLOCK - 1) / BLOCK;
    hipLaunchKernelGGL(few ? k_topk_pass_few : k_select_pass<4>, dim3(blocks), dim3(few ? 256 : SEL_THREADS), 0, c->stream, vin, iin, n,
                       (uint32_t)c->M, (uint32_t)c->Mpad, k, va, ia, (int32_t *)nullptr);
    VF_HIP(c, hipGetLastError());
    vin = va; iin = ia;
    n = blocks * (uint32_t)k;
    std::swap(va, vb);
    std::swap(ia, ib);
  }
  hipLaunchKernelGGL(few               ? k_topk_pass_few
                     : n <= SEL_THREADS ? k_select_pass<1>
                     : n <= BLOCK       ? k_select_pass<4>
                                        : k_select_pass<16>,
                     dim3(1), dim3(few ? 256 : SEL_THREADS), 0, c->stream, vin, iin, n, (uint32_t)c->M, (uint32_t)c->Mpad, k, c->d_sel_val, c->d_sel_idx, c->d_sel_n);
  VF_HIP(c, hipGetLastError());
  return VF_OK;
}

// All but single slots with short decisions, whose selection on id ranges is one pass of block minima
// (256-512-512-1, whole search, on id ranges / lists: 20 layers, one slot, 63 ids 559 / 603 us, 405: 588 / 603, 768:
// 552 / 530, 4096: 688 / 617; two slots, 63 ids 619 / 619, 405: 640 / 620, 768: 618 / 540, 4096: 779 / 637; four slots,
// 63 ids 692 / 625; 256-1024-1024-1, one slot, 4096 ids 1017 / 911; 100 layers of 16384 ids, one slot 3203 / 3196).
bool vfk_beam_lists(const vf_ctx *c) { return (c->B > 1 || c->M > 512) && vfk_layer_fits(c); }

int vfk_beam_layers(vf_ctx *c, int first, int last) {
  int rc = vfk_scores_buffer(c);
  if (rc == VF_OK) rc = vfk_layer_open(c, first);
  if (rc != VF_OK) return rc;
  vf_fast_dev fd;
  vfk_fast_dev(c, true, &fd, nullptr, nullptr);
  int ncu = 256;
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device);
  const bool ahead = c->B <= ncu;  // (as in vfk_greedy_layers)
  for (int i = first; i <= last; ++i) {
    int nparts = 0;
    rc = vfk_layer_score(c, -1, c->d_scores, &nparts);
    if (rc != VF_OK) return rc;
    const uint32_t *list = reinterpret_cast<const uint32_t *>(c->d_wlist);
    uint32_t *const pub = c->d_pub + (size_t)c->pub_set * c->B * VF_PUB_WORDS;
    c->pub_set ^= 1;
    hipLaunchKernelGGL(k_beam_select, dim3(1), dim3(SEL_THREADS), 0, c->stream, c->d_scores, c->d_pval, c->d_pidx,
                       (const uint32_t *)(c->d_pub + (size_t)2 * c->B * VF_PUB_WORDS), nparts, list, pub, c->d_space, (int64_t)c->Mpad, c->B, c->d_sel_val, c->d_sel_idx, c->d_sel_n);
    VF_HIP(c, hipGetLastError());
    {
      vf_prof_scope prof(c, VF_PROF_COMMIT);
      hipLaunchKernelGGL((c->pm.fast_rt == 4 ? ahead ? k_beam_advance<4, 4> : k_beam_advance<4, 0> : ahead ? k_beam_advance<2, 14> : k_beam_advance<2, 0>),
                         dim3((unsigned)c->B * 2), dim3(512), 0,
                         c->stream, tables_of(c), alt_of(c), i, (int)(i < last), (int64_t)c->Mpad,
                         c->d_sel_val, c->d_sel_idx, c->d_sel_n, fd, pub, c->d_pub + (size_t)c->pub_set * c->B * VF_PUB_WORDS,
                         reinterpret_cast<uint32_t *>(c->d_wlist));
      VF_HIP(c, hipGetLastError());
    }
    c->dec_stage = -1;  // (the context of the next layer is among the opened decisions)
    vfk_beam_swap(c);
    c->n_sched = i + 1;
  }
  return VF_OK;
}
