// What the kernels that work on lists of valid candidates share: opening a decision (quotient
// tables, folded first-layer bias, the ordered list of valid candidates) and the form in which an
// opened decision is left in memory for other workgroups.  Included inside the anonymous namespace
// of each .hip file that needs it, after vf_sched_dev.h and vf_score_dev.h.
#ifndef VF_LAYER_DEV_H
#define VF_LAYER_DEV_H

// words of a published layer: DecPack, EvalTabs, first-layer bias (up to 1024 rows), count
constexpr int VF_PUB_TABS = VF_DECPACK_DWORDS;
constexpr int VF_PUB_BIAS = VF_PUB_TABS + (int)(sizeof(EvalTabs) / 4);
constexpr int VF_PUB_COUNT = VF_PUB_BIAS + 1024;
static_assert(VF_PUB_COUNT + 4 == VF_PUB_WORDS, "published layer size");

struct OpenScratch {
  int pos[13], cat[12], dec[12];  // per open (store_at, compute_at) pair: first list position, level, digits
  int nok[3][3], ok[3][3][8];     // per level and dimension: the split factors that fit
  float rcp[3][3];                // 1 / nok, for div_small
  int npairs, ncand;
};

// Ordered list of a decision's valid ids, written down directly from the validity rules: per
// (compute_at, store_at) digit pair that is open - the level is offered and the hoist does not exceed
// it - the valid ids are the products of the split factors that fit the level's region with every
// loop order / vectorize / parallel choice; an inlining pair has the single id with every other digit
// zero.  In three parts with a workgroup barrier behind each of the first two.
// First: the split factors that fit (nine threads, i = 0..8).
[[maybe_unused]] __device__ __forceinline__ void list_factors(const DecPack &pk, OpenScratch &os, int i) {
  const int lvl = i / 3, dd = i % 3;
  int cnt = 0;
  for (int k = 0; k < pk.sp.nf[dd]; ++k)
    if ((uint32_t)pk.sp.fac[dd][k] <= pk.d.E[lvl][dd]) os.ok[lvl][dd][cnt++] = k;
  os.nok[lvl][dd] = cnt;
  os.rcp[lvl][dd] = 1.0f / (float)(cnt > 0 ? cnt : 1);
}
// Second: the open pairs numbered and given their first list position in order (one wave; lane j
// looks at pair j = (store_at digit, compute_at digit)).
[[maybe_unused]] __device__ __forceinline__ void list_pairs(const DecPack &pk, OpenScratch &os, int lane) {
  const int rest_n = pk.sp.nperm * pk.sp.nvec * pk.sp.npar;
  const int npairs_all = pk.sp.nsat * pk.sp.ncat;
  int cnt = 0, cat = 0, dec = 0;
  if (lane < npairs_all && lane < 12) {
    const int isat = lane / pk.sp.ncat, icat = lane % pk.sp.ncat;
    cat = pk.sp.cat[icat];
    dec = (int)((uint32_t)icat << 24 | (uint32_t)isat << 28);
    if (pk.d.lvl_ok[cat] != 0) {
      if (cat == VF_INLINE) cnt = isat == 0 ? 1 : 0;
      else if (isat <= cat) cnt = os.nok[cat][0] * os.nok[cat][1] * os.nok[cat][2] * rest_n;
    }
  }
  int np = 0, pos = 0;
#pragma unroll
  for (int j = 0; j < 12; ++j) {
    const int cj = __builtin_amdgcn_readlane(cnt, j);
    if (cj == 0) continue;
    const int catj = __builtin_amdgcn_readlane(cat, j), decj = __builtin_amdgcn_readlane(dec, j);
    if (lane == 0) {
      os.pos[np] = pos;
      os.cat[np] = catj;
      os.dec[np] = decj;
    }
    pos += cj;
    ++np;
  }
  if (lane == 0) {
    os.pos[np] = pos;
    os.npairs = np;
    os.ncand = pos;
  }
}
// Third: the packed digits of entry k (pos_r: the pairs' first positions in registers, 0x7fffffff
// behind the last pair, so that an entry's pair is found without a chain of dependent reads).
[[maybe_unused]] __device__ __forceinline__ uint32_t list_entry(const DecPack &pk, const OpenScratch &os, const int (&pos_r)[12], int k,
                                               float rcp_perm, float rcp_vec) {
  int q = 0;
#pragma unroll
  for (int j = 1; j < 12; ++j) q += k >= pos_r[j] ? 1 : 0;
  const int cat = os.cat[q];
  uint32_t dec = (uint32_t)os.dec[q];
  if (cat != VF_INLINE) {
    uint32_t r = (uint32_t)(k - os.pos[q]), nxt;
    const uint32_t nx = os.nok[cat][0], ny = os.nok[cat][1], nc = os.nok[cat][2];
    nxt = div_small(r, nx, os.rcp[cat][0]); const uint32_t jx = r - nxt * nx; r = nxt;
    nxt = div_small(r, ny, os.rcp[cat][1]); const uint32_t jy = r - nxt * ny; r = nxt;
    nxt = div_small(r, nc, os.rcp[cat][2]); const uint32_t jc = r - nxt * nc; r = nxt;
    const int ix = os.ok[cat][0][jx], iy = os.ok[cat][1][jy], ic = os.ok[cat][2][jc];
    nxt = div_small(r, (uint32_t)pk.sp.nperm, rcp_perm); const uint32_t ip = r - nxt * (uint32_t)pk.sp.nperm; r = nxt;
    const uint32_t par = div_small(r, (uint32_t)pk.sp.nvec, rcp_vec), vec = r - par * (uint32_t)pk.sp.nvec;
    dec |= (uint32_t)ix | (uint32_t)iy << 4 | (uint32_t)ic << 8 | (uint32_t)ip << 12 | (uint32_t)vec << 16 |
           (uint32_t)par << 20;
  }
  return dec;
}

// Opens a decision whose context (pk.d, pk.sp) is in LDS: quotient tables, the shared input rows
// as the first layer wants them, the folded bias, the ordered list of the valid candidates with
// its length (os.ncand).  Every thread of a workgroup of 512 calls it; the list is complete for
// other threads behind the caller's next barrier, everything else behind this function's own.
template <int RT>
__device__ __forceinline__ void open_layer(DecPack &pk, EvalTabs &tabs, OpenScratch &os, const vf_fast_dev &md,
                                           __amdgpu_buffer_rsrc_t wf, int tid, int w, int lane, float *bias_out,
                                           uint32_t *idlist) {
  // three small jobs side by side, on different waves: the quotient tables (waves 0, 1), the
  // shared input rows as the first layer wants them (waves 2, 3), the split factors that fit
  // (wave 4)
  fill_evaltabs(tabs, pk.d, pk.sp);
  if (tid >= 128 && tid < 128 + VF_STAT_WORDS) pk.stat[tid - 128] = stat_word(pk.d, tid - 128);
  // (the list holds the digits, packed, rather than the id: the evaluation works on digits, and putting
  // an id together takes a few multiplications where taking it apart takes as many divisions)
  if (tid >= 256 && tid < 265) list_factors(pk, os, tid - 256);
  __syncthreads();
  const float rcp_perm = 1.0f / (float)pk.sp.nperm, rcp_vec = 1.0f / (float)pk.sp.nvec;
  if (w == 0) list_pairs(pk, os, lane);
  fold_bias<RT>(wf, pk.stat, md.dims[0] == 256, w, lane, md.aux + md.bias_off[0], bias_out);
  __syncthreads();  // the pairs are numbered, the bias is complete
  int pos_r[12];
#pragma unroll
  for (int j = 0; j < 12; ++j) pos_r[j] = j < os.npairs ? os.pos[j] : 0x7fffffff;
  for (int k = tid; k < os.ncand; k += 512) idlist[k] = list_entry(pk, os, pos_r, k, rcp_perm, rcp_vec);
}

// Leaves an opened decision in memory (every thread of a workgroup of 512; bias: the folded one).
__device__ __forceinline__ void publish_layer(uint32_t *pub, const DecPack &pk, const EvalTabs &tabs, const float *bias,
                                              int nbias, int ncand, int tid) {
  for (int i = tid; i < VF_DECPACK_DWORDS; i += 512) pub[i] = reinterpret_cast<const uint32_t *>(&pk)[i];
  for (int i = tid; i < (int)(sizeof(EvalTabs) / 4); i += 512) pub[VF_PUB_TABS + i] = reinterpret_cast<const uint32_t *>(&tabs)[i];
  for (int i = tid; i < nbias; i += 512) pub[VF_PUB_BIAS + i] = __float_as_uint(bias[i]);
  if (tid == 0) pub[VF_PUB_COUNT] = (uint32_t)ncand;
}

// The parts of 64 list entries behind the ones that the scorer will write have no minimum.  (A
// tile of 128 entries writes both its parts, one of 64 the one it has: the last part of a count that
// ends in the first half of 128 entries is written here as well as there, by launches in order.)
__device__ __forceinline__ void no_minima(float *pval, int32_t *pidx, int ncand, int nparts, int tid) {
  for (int i = (ncand + 63) / 64 + tid; i < nparts; i += 512) {
    pval[i] = __builtin_inff();
    pidx[i] = -1;
  }
}

// LDS of a workgroup that goes on from one decision to the next.
struct AdvanceShared {
  DecPack pk, next;  // the decision's context, the next one's
  DecScratch ds;
  EvalTabs tabs;
  OpenScratch os;
  float bias[1024];
  int32_t cf64[64], st16[16], sums[3];
  int32_t cid;       // the decision: a candidate id, -1 = none
  float val;
};

// Algorithm 1's s_i := s and, with `open`, the next decision opened for the scorer: problem `src`
// of the tables `from` goes on as problem `dst` of the tables `to` (the same one in a greedy
// schedule).  The next context comes from the rows of `from` and the winner's rows in LDS.  Every
// thread of a workgroup of 512 calls it, without a barrier behind its writes to s.pk, s.cid, s.val.
template <int RT>
__device__ __forceinline__ void advance_layer(AdvanceShared &s, const Tables &from, const Tables &to, int src, int dst,
                                              int stage, int open, uint32_t M, const vf_fast_dev &md, uint32_t *pub,
                                              uint32_t *idlist, uint32_t *decpack_next, int tid, int w, int lane) {
  if (open) dec_fetch_rows(s.next.d, s.next.sp, s.ds, from, src, stage + 1, stage);
  __syncthreads();  // the decision and its context have arrived
  fill_evaltabs(s.tabs, s.pk.d, s.pk.sp, 64);
  if (open) dec_fetch_anchor(s.next.d, s.ds, from, src, stage + 1, stage);
  __syncthreads();
  if (tid == 0) commit_winner_fresh(to, s.pk.d, s.pk.sp, dst, stage, s.cid, s.val, M, s.tabs, true, s.cf64, s.st16, s.sums);
  __syncthreads();
  if (!open) return;
  FreshRows fr;
  fr.stage = stage; fr.cf = s.cf64; fr.st = s.st16;
  fr.pm = s.sums[0]; fr.pb = s.sums[1]; fr.alive = s.sums[2];
  dec_finish(s.next.d, s.next.sp, s.ds, stage + 1, fr);
  open_layer<RT>(s.next, s.tabs, s.os, md, stream_rsrc(md.w_full + (size_t)w * md.wave_stride_full), tid, w, lane, s.bias,
                 idlist);
  publish_layer(pub, s.next, s.tabs, s.bias, md.dims[1], s.os.ncand, tid);
  if (tid < VF_DECPACK_DWORDS) decpack_next[tid] = reinterpret_cast<const uint32_t *>(&s.next)[tid];
}

#endif  // VF_LAYER_DEV_H
