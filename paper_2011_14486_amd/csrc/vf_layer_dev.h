// What the kernels that work on lists of valid candidates share: opening a decision (quotient
// tables, folded first-layer bias, the ordered list of valid candidates) and the form in which an
// opened decision is left in memory for other workgroups.  Included inside the anonymous namespace
// of each .hip file that needs it, after vf_sched_dev.h and vf_score_dev.h.
#ifndef VF_LAYER_DEV_H
#define VF_LAYER_DEV_H

// words of a published layer: DecPack, EvalTabs, first-layer bias (up to 1024 rows; from a multiple of 16 bytes on), count
constexpr int VF_PUB_TABS = VF_DECPACK_DWORDS;
constexpr int VF_PUB_BIAS = (VF_PUB_TABS + (int)(sizeof(EvalTabs) / 4) + 3) & ~3;
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
// Third: entry k's place in the list (pos_r: the pairs' first positions in registers, 0x7fffffff
// behind the last pair, so that an entry's pair is found without a chain of dependent reads), and the
// packed digits there.
struct ListPlace {
  int q, cat;                      // the pair, its level
  uint32_t dec;                    // the pair's digits
  uint32_t nx, ny, nc;             // factors that fit
  uint32_t jx, jy, jc, ip, vec, par;
};
[[maybe_unused]] __device__ __forceinline__ void list_pair(const OpenScratch &os, ListPlace &at) {
  at.cat = os.cat[at.q];
  at.dec = (uint32_t)os.dec[at.q];
  at.nx = at.ny = at.nc = 1u;
  at.jx = at.jy = at.jc = at.ip = at.vec = at.par = 0u;
  if (at.cat != VF_INLINE) { at.nx = os.nok[at.cat][0]; at.ny = os.nok[at.cat][1]; at.nc = os.nok[at.cat][2]; }
}
[[maybe_unused]] __device__ __forceinline__ ListPlace list_place(const DecPack &pk, const OpenScratch &os, const int (&pos_r)[12], int k,
                                                                 float rcp_perm, float rcp_vec) {
  ListPlace at;
  at.q = 0;
#pragma unroll
  for (int j = 1; j < 12; ++j) at.q += k >= pos_r[j] ? 1 : 0;
  list_pair(os, at);
  if (at.cat != VF_INLINE) {
    uint32_t r = (uint32_t)(k - os.pos[at.q]), nxt;
    nxt = div_small(r, at.nx, os.rcp[at.cat][0]); at.jx = r - nxt * at.nx; r = nxt;
    nxt = div_small(r, at.ny, os.rcp[at.cat][1]); at.jy = r - nxt * at.ny; r = nxt;
    nxt = div_small(r, at.nc, os.rcp[at.cat][2]); at.jc = r - nxt * at.nc; r = nxt;
    nxt = div_small(r, (uint32_t)pk.sp.nperm, rcp_perm); at.ip = r - nxt * (uint32_t)pk.sp.nperm; r = nxt;
    at.par = div_small(r, (uint32_t)pk.sp.nvec, rcp_vec); at.vec = r - at.par * (uint32_t)pk.sp.nvec;
  }
  return at;
}
[[maybe_unused]] __device__ __forceinline__ uint32_t list_digits(const OpenScratch &os, const ListPlace &at) {
  if (at.cat == VF_INLINE) return at.dec;
  return at.dec | (uint32_t)os.ok[at.cat][0][at.jx] | (uint32_t)os.ok[at.cat][1][at.jy] << 4 | (uint32_t)os.ok[at.cat][2][at.jc] << 8 |
         at.ip << 12 | at.vec << 16 | at.par << 20;
}
[[maybe_unused]] __device__ __forceinline__ uint32_t list_entry(const DecPack &pk, const OpenScratch &os, const int (&pos_r)[12], int k,
                                                                float rcp_perm, float rcp_vec) {
  return list_digits(os, list_place(pk, os, pos_r, k, rcp_perm, rcp_vec));
}
// The list, by `threads` threads (of them tid): a thread takes four entries in a row and goes on from the first to the
// others by carrying (the divisions of an entry are most of its work).  The list is 16-byte aligned and has room for a
// multiple of four.  Where there is a thread for every entry it takes just that one: the carrying would be three more
// steps behind the divisions (fours / this, 20 layers, 256-512-512-1: 24 problems of 768 ids 899 / 874 us, 200: 1000 / 992,
// 22: 497 / 487; 256-1024-1024-1, 200 of 768: 2382 / 2360).  k_whole with 1024 units spills 20 registers with both
// forms, 11 with single entries alone, and takes as long: 256 problems of 4096 ids 12.63 ms / 12.64.
__device__ __forceinline__ void write_list(const DecPack &pk, const OpenScratch &os, uint32_t *idlist, int tid, int threads = 512) {
  const float rcp_perm = 1.0f / (float)pk.sp.nperm, rcp_vec = 1.0f / (float)pk.sp.nvec;
  const int n = os.ncand, last = os.npairs - 1;
  int pos_r[12];
#pragma unroll
  for (int j = 0; j < 12; ++j) pos_r[j] = j <= last ? os.pos[j] : 0x7fffffff;
  if (n <= threads) {
    if (tid < n) idlist[tid] = list_entry(pk, os, pos_r, tid, rcp_perm, rcp_vec);
    return;
  }
  for (int k = 4 * tid; k < n; k += 4 * threads) {
    ListPlace at = list_place(pk, os, pos_r, k, rcp_perm, rcp_vec);
    int next = os.pos[at.q + 1];  // (behind the last pair: n)
    uint32_t e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      e[i] = k + i < n ? list_digits(os, at) : 0u;
      if (i == 3) break;
      if (k + i + 1 == next) {
        if (at.q < last) {
          ++at.q;
          list_pair(os, at);
          next = os.pos[at.q + 1];
        }
      } else if (++at.jx == at.nx) {
        at.jx = 0u;
        if (++at.jy == at.ny) {
          at.jy = 0u;
          if (++at.jc == at.nc) {
            at.jc = 0u;
            if (++at.ip == (uint32_t)pk.sp.nperm) {
              at.ip = 0u;
              if (++at.vec == (uint32_t)pk.sp.nvec) { at.vec = 0u; ++at.par; }
            }
          }
        }
      }
    }
    *reinterpret_cast<uint4 *>(idlist + k) = make_uint4(e[0], e[1], e[2], e[3]);
  }
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
  if (w == 0) list_pairs(pk, os, lane);
  fold_bias<RT>(wf, pk.stat, md.dims[0] == 256, w, lane, md.aux + md.bias_off[0], bias_out);
  __syncthreads();  // the pairs are numbered, the bias is complete
  write_list(pk, os, idlist, tid);
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
struct __attribute__((aligned(16))) AdvanceShared {
  DecPack pk;        // the decision, as it was published
  EvalTabs tabs;
  uint32_t pad[VF_PUB_BIAS - VF_PUB_TABS - (int)(sizeof(EvalTabs) / 4)];
  struct __attribute__((aligned(16))) {  // the next one, as it is published
    DecPack pk;
    EvalTabs tabs;
    uint32_t pad[VF_PUB_BIAS - VF_PUB_TABS - (int)(sizeof(EvalTabs) / 4)];
    float bias[1024];  // of the first layer; folded
  } next;
  DecScratch ds;
  OpenScratch os;
  int32_t cf64[64], st16[16], sums[3];
  int32_t cid;       // the decision: a candidate id, -1 = none
  float val;
};
static_assert(offsetof(AdvanceShared, next) % 16 == 0 && sizeof(DecPack) + sizeof(EvalTabs) + sizeof(AdvanceShared::pad) == VF_PUB_BIAS * 4,
              "a decision in LDS lies as it is published");
// The published decision (one 16-byte piece by each of the threads from 256 on).
__device__ __forceinline__ void fetch_opened(AdvanceShared &s, const uint32_t *pub, int tid) {
  if (tid >= 256 && tid < 256 + VF_PUB_BIAS / 4) reinterpret_cast<uint4 *>(&s.pk)[tid - 256] = reinterpret_cast<const uint4 *>(pub)[tid - 256];
}

// Algorithm 1's s_i := s and, with `open`, the next decision opened for the scorer: problem `src`
// of the tables `from` goes on as problem `dst` of the tables `to` (the same one in a greedy
// schedule).  The next context comes from the rows of `from` and the winner's rows in LDS.  Every
// thread of a workgroup of 512 calls it, without a barrier behind its writes to s.pk, s.tabs, s.cid, s.val.
//
// A chain of small steps, so what does not depend on the winner runs beside them: the shared input rows
// that only move on by a stage, and AHEAD k-steps of the folded layer's weights, in flight while the winner
// is worked out (a compute unit takes 2.5 us to fetch the 229 KB of 512 units; 0: none, for a caller that runs
// several workgroups per compute unit and would lose them to the registers).  Nothing is stored to memory
// before the weights have been used: their use would wait for the stores too.
template <int RT, int AHEAD>
__device__ __forceinline__ void advance_layer(AdvanceShared &s, const Tables &from, const Tables &to, int src, int dst,
                                              int stage, int open, const vf_fast_dev &md, uint32_t *pub,
                                              uint32_t *idlist, int tid, int w, int lane) {
  const __amdgpu_buffer_rsrc_t wf = stream_rsrc(md.w_full + (size_t)w * md.wave_stride_full);
  const bool wide = md.dims[0] == 256;
  DecPack &nk = s.next.pk;
  if (open) {
    dec_fetch_rows(nk.d, nk.sp, s.ds, from, src, stage + 1, stage);
    for (int i = tid; AHEAD > 0 && i < md.dims[1]; i += 512) s.next.bias[i] = md.aux[md.bias_off[0] + i];
  }
  __syncthreads();  // the decision and what is known of the next one have arrived
  if (open && w == 4) dec_fetch_anchor(nk.d, s.ds, from, src, stage + 1, stage, tid - 256);
  // (fold_bias's k-steps in its order: 0, 3, 4, 5, ...; with 64 inputs only the first two)
  uint4 ahead[AHEAD > 0 ? AHEAD : 1][RT];
  if (AHEAD > 0 && open) {
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) fold_load<RT>(ahead[i], wf, i == 0 || (i > 1 && !wide) ? 0 : i + 2, lane);
  }
  winner_rows(s, s.pk, s.cid >= 0 ? (int32_t)pack_digits(digits_small(s.pk.sp, (uint32_t)s.cid)) : -1, lane, w);
  if (AHEAD > 0 && open && tid >= 320 && tid < 404) {
    const int q = tid - 320 < 72 ? 40 + tid - 320 : tid - 392;
    nk.stat[q] = stat_word(nk.d, q);
  }
  __syncthreads();
  next_shared_rows(s, nk, true, stage, tid);
  __syncthreads();
  if (open) {
    if constexpr (AHEAD == 0) {
      if (tid == 0) next_derive(s, nk, true, stage);
      __syncthreads();
      open_layer<RT>(nk, s.next.tabs, s.os, md, wf, tid, w, lane, s.next.bias, idlist);
    } else {
      // the folded layer: first by all waves but wave 0, which derives the rest of the context meanwhile, then by
      // wave 0, while the others make the quotient tables and number the open pairs
      for (int ph = 0; ph < 2; ++ph) {
        if ((ph == 0) == (w != 0)) {
          floatx16 fa[RT];
          fold_zero<RT>(fa);
          auto products = [&](auto n) __attribute__((always_inline)) {
            constexpr int N = decltype(n)::value;
  #pragma unroll
            for (int i = 0; i < N; ++i) {
              fold_step<RT>(fa, ahead[i % AHEAD], nk.stat, i == 0 ? 0 : i + 2, lane);
              if (i + AHEAD < N) fold_load<RT>(ahead[i % AHEAD], wf, i + AHEAD + 2, lane);
            }
          };
          if (wide) products(std::integral_constant<int, 14>{});
          else products(std::integral_constant<int, 2>{});
          if ((lane & 31) == 0) {
  #pragma unroll
            for (int r = 0; r < RT; ++r)
  #pragma unroll
              for (int g = 0; g < 4; ++g) {
                float4 *const b = reinterpret_cast<float4 *>(s.next.bias + (w + r * 8) * 32 + 4 * (lane >> 5) + 8 * g);
                float4 v = *b;
                v.x += fa[r][4 * g]; v.y += fa[r][4 * g + 1]; v.z += fa[r][4 * g + 2]; v.w += fa[r][4 * g + 3];
                *b = v;
              }
          }
        } else if (ph == 0) {
          if (lane == 0) next_derive(s, nk, true, stage);
        } else {
          fill_evaltabs(s.next.tabs, nk.d, nk.sp, 64);
          if (w == 7) {
            if (lane < 9) list_factors(nk, s.os, lane);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            list_pairs(nk, s.os, lane);
          }
        }
        __syncthreads();
      }
      write_list(nk, s.os, idlist, tid);
    }
    if (tid < (VF_PUB_BIAS + md.dims[1]) / 4) reinterpret_cast<uint4 *>(pub)[tid] = reinterpret_cast<const uint4 *>(&s.next)[tid];
    if (tid == 448) pub[VF_PUB_COUNT] = (uint32_t)s.os.ncand;
  }
  // the winner to the tables
  const bool ok = s.st16[15] != 0;
  const size_t at = (size_t)dst * to.S + stage;
  if (tid >= 128 && tid < 192 && ok) to.cf[at * 64 + tid - 128] = s.cf64[tid - 128];
  if (tid >= 192 && tid < 208 && ok) to.states[at * 16 + tid - 192] = s.st16[tid - 192];
  if (tid == 256) {
    to.cids[at] = ok ? s.cid : -1;
    to.vals[at] = ok ? s.val : __builtin_inff();
    if (!ok) to.alive[dst] = 0;
  }
  if (tid == 257 || tid == 258) to.prefix[((size_t)dst * (to.S + 1) + stage + 1) * 2 + tid - 257] = s.sums[tid - 257];
}

#endif  // VF_LAYER_DEV_H
