// What the kernels that follow a whole schedule with several workgroups per problem share (vf_chain.hip,
// vf_small.hip): between two decisions the tiles' minima are exchanged, the winner committed and the next context
// built by every workgroup for itself.  Workgroups of 512.  Included inside the anonymous namespace of each
// .hip file that needs it, after vf_sched_dev.h and vf_score_dev.h.
#ifndef VF_CHAIN_DEV_H
#define VF_CHAIN_DEV_H

struct ChainArgs {
  Tables t;
  int first, last;
  int64_t M;
  int nprob, ntiles;           // tiles of a decision, as many workgroups per problem; grid = nprob * ntiles
  unsigned long long *slots;   // [nprob][S][ntiles] first minimum of every tile, 0 = not there yet
  unsigned int *claims;        // [nprob][S + 1] tiles claimed per stage; workgroups that have left
  unsigned int wait_rounds;
  uint32_t *decpack;           // [nprob] receives the context of stage last + 1, if there is one
  int32_t *out_states, *out_cids;  // nullable: the caller's tables
  float *out_vals;
  unsigned long long *stat;    // nullable: [0] += ids pushed through the network, [1] += valid ones
};

struct ChainShared {
  DecPack pks[2];     // the open decision's context and the next one's, in turn
  EvalTabs tabs;      // the open decision's quotient tables
  DecScratch ds;
  int32_t cf64[64], st16[16], sums[3];  // the last winner's rows, the sums behind it, alive
  int claim;          // a tile of the next decision
  int missing;        // >= 0: a tile whose minimum did not come
  int32_t win_c;      // the winner's digits, packed (they order like the ids); -1: none
  float win_v;
};
constexpr int CLAIMER = 448;  // the thread that claims tiles (first of the wave that polls)
constexpr unsigned int NO_CLAIM = 0xffffffffu;

// A first minimum as a word that is not zero.
__device__ __forceinline__ unsigned long long word_of(float v, int32_t c) {
  return (unsigned long long)__float_as_uint(v) << 32 | (c >= 0 ? (uint32_t)c + 1u : 0xffffffffu);
}

// Once per workgroup: the space; the layers that this call does not decide to the caller's tables, as they
// are (the others follow one by one).
__device__ __forceinline__ void chain_begin(ChainShared &sh, const ChainArgs &ca, size_t row, int member, int tid) {
  const int S = ca.t.S;
  for (int i = tid; i < (int)(sizeof(vf_space) / 4); i += 512)
    reinterpret_cast<int32_t *>(&sh.pks[0].sp)[i] = reinterpret_cast<int32_t *>(&sh.pks[1].sp)[i] = ca.t.space[i];
  if (member == 0 && (ca.out_states || ca.out_cids || ca.out_vals)) {
    for (int i = tid; i < S * 16; i += 512) {
      const int j = i / 16;
      if (j >= ca.first && j <= ca.last) continue;
      if (ca.out_states) ca.out_states[row * 16 + i] = ca.t.states[row * 16 + i];
      if ((i & 15) == 0 && ca.out_cids) ca.out_cids[row + j] = ca.t.cids[row + j];
      if ((i & 15) == 0 && ca.out_vals) ca.out_vals[row + j] = ca.t.vals[row + j];
    }
  }
}

// What is known of the next stage's context (nk) before the open decision is (pk; stage < ca.first: there is none
// yet and everything is).  pre: what the thread fetched for it (chain_prefetch).  With barriers inside if there
// is a next stage.
__device__ __forceinline__ void chain_rows(ChainShared &sh, DecPack &nk, const DecPack &pk, const ChainArgs &ca, int p, size_t row,
                                           int stage, unsigned int c_next, int32_t pre, int tid, int lane, int w) {
  const int next = stage + 1;
  DecScratch &ds = sh.ds;
  if (stage < ca.first) {
    // the call's first stage, from the tables
    dec_fetch_rows(nk.d, nk.sp, ds, ca.t, p, next, -1);
    __syncthreads();
    dec_fetch_anchor(nk.d, ds, ca.t, p, next, -1, tid);
    if (tid >= 128 && tid < 128 + VF_STAT_WORDS) nk.stat[tid - 128] = stat_word(nk.d, tid - 128);
    if (tid < 3) sh.sums[tid] = ds.sc[tid < 2 ? 1 + tid : 0];
    if (tid == CLAIMER) sh.claim = (int)c_next;
    __syncthreads();
  } else if (next < ca.t.S) {
    // from the open context where it has them (its neighbour rows move on by one), else fetched before
    if (tid < 128) {
      nk.d.nb[48 + tid] = pk.d.nb[tid < 96 ? tid : tid + 64];
    } else if (tid < 192) {
      const int q = tid - 128;  // the same as pairs, normalised
      nk.stat[40 + q] = pk.stat[q < 48 ? 16 + q : 48 + q];
    } else if (tid < 208) {
      nk.d.intr[tid - 192] = pk.d.nb[144 + tid - 192];
    } else if (tid < 216) {
      nk.stat[tid - 208] = pk.stat[88 + tid - 208];
    } else if (tid < 220) {
      nk.stat[tid - 208] = 0u;
    } else if (w == 6) {
      if (lane < 16) {
        nk.d.nb[176 + lane] = pre;
        const int32_t odd = __shfl_down(pre, 1);
        if ((lane & 1) == 0) nk.stat[104 + lane / 2] = pack_bf16(plog2_dev(pre), plog2_dev(odd));
      } else if (lane < 32) {
        nk.d.srec[lane - 16] = pre;
      } else if (lane < 34) {
        ds.sc[lane - 29] = pre;
      }
    }
    __syncthreads();
    if (w == 5) {  // the anchor's rows (as dec_fetch_anchor)
      const int a = nk.d.srec[8];
      int32_t v = 0;
      if (a >= 0 && a < next) {
        const size_t ar = row + a;
        if (lane < 16) v = a != stage ? ca.t.states[ar * 16 + lane] : 0;
        else if (lane < 32) v = ca.t.stages[ar * 16 + lane - 16];
        else if (lane < 36) v = a != stage ? ca.t.cf[ar * 64 + (lane == 32 ? 42 : lane == 33 ? 54 : lane == 34 ? 32 : 23)] : 0;
      }
      if (lane < 16) ds.ast[lane] = v;
      else if (lane < 32) ds.arec[lane - 16] = v;
      else if (lane < 36) ds.acf[lane - 32] = v;
    }
  }
}

// One wave: the first minimum of a decision's tiles, once all are there; or a tile to score (missing).
__device__ __forceinline__ void chain_poll(ChainShared &sh, const ChainArgs &ca, unsigned long long *slots, unsigned int *claims, int ntiles,
                                           int stage, unsigned int c_next, int lane) {
  float v = __builtin_inff();
  int32_t c = -1;
  int miss = -1;
  unsigned int rounds = 0;
  bool drained = false;  // no unclaimed tile
  for (int q0 = 0; q0 < ntiles && miss < 0; q0 += 256) {
    unsigned long long word[4] = {0ull, 0ull, 0ull, 0ull};
    for (;;) {
      bool lack = false;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int q = q0 + 64 * k + lane;
        if (q < ntiles && word[k] == 0ull)
          word[k] = __hip_atomic_load(&slots[(size_t)stage * ntiles + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) lack = lack || (q0 + 64 * k + lane < ntiles && word[k] == 0ull);
      if (__ballot(lack) == 0ull) break;
      // a tile that nobody has claimed: one for this workgroup (some are not running yet)
      if (!drained && (rounds & 7u) == 7u) {
        int q = 0;
        if (lane == 0) q = (int)atomicAdd(&claims[stage], 1u);
        q = __builtin_amdgcn_readfirstlane(q);
        if (q < ntiles) { miss = q; break; }
        drained = true;
      }
      if (rounds++ >= ca.wait_rounds) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const unsigned long long m = __ballot(q0 + 64 * k + lane < ntiles && word[k] == 0ull);
          if (m != 0ull && miss < 0) miss = q0 + 64 * k + (int)__builtin_ctzll(m);
        }
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t dg = (uint32_t)word[k];
      take_min(v, c, __uint_as_float((uint32_t)(word[k] >> 32)), dg == 0xffffffffu ? -1 : (int32_t)dg - 1);
    }
  }
  wave_min(v, c);
  if (lane == 0) { sh.win_v = v; sh.win_c = c; sh.missing = miss; sh.claim = (int)c_next; }
}

// The winner to the tables: every workgroup writes them (it reads its anchors from there), one the caller's.
__device__ __forceinline__ void chain_tables(const ChainShared &sh, const DecPack &pk, const ChainArgs &ca, int p, size_t row, int stage,
                                             int member, int tid) {
  const bool ok = sh.st16[15] != 0;
  const size_t at = row + stage;
  if (tid >= 128 && tid < 192 && ok) ca.t.cf[at * 64 + tid - 128] = sh.cf64[tid - 128];
  if (tid >= 192 && tid < 208) {
    const int i = tid - 192;
    const int32_t v = i < 15 ? sh.cf64[state_feature(i)] : sh.st16[15];
    if (ok) ca.t.states[at * 16 + i] = v;
    if (member == 0 && ca.out_states) ca.out_states[at * 16 + i] = ok ? v : 0;
  }
  if (tid == 256) {
    const int32_t id = ok ? (int32_t)id_of(pk.sp, unpack_digits((uint32_t)sh.win_c)) : -1;
    const float v = ok ? sh.win_v : __builtin_inff();
    ca.t.cids[at] = id;
    ca.t.vals[at] = v;
    if (member == 0 && ca.out_cids) ca.out_cids[at] = id;
    if (member == 0 && ca.out_vals) ca.out_vals[at] = v;
  }
  if (tid == 257 || tid == 258) ca.t.prefix[((size_t)p * (ca.t.S + 1) + stage + 1) * 2 + tid - 257] = sh.sums[tid - 257];
}

// One wave: what the context behind the open one takes from memory, for the end of this decision.
__device__ __forceinline__ int32_t chain_prefetch(const ChainArgs &ca, size_t row, int stage, int lane) {
  const int S = ca.t.S;
  int32_t pre = 0;
  if (stage + 1 < S) {
    if (lane < 16) pre = stage + 4 < S ? ca.t.intr[(row + stage + 4) * 16 + lane] : 0;
    else if (lane < 32) pre = ca.t.stages[(row + stage + 1) * 16 + lane - 16];
    else if (lane < 34) pre = ca.t.suffix[(row + stage + 1) * 2 + lane - 32];
  }
  return pre;
}

// The last workgroup of the problem to leave clears its words, and marks a problem that found no winner: one
// that only starts when others have gone on still needs the mark that the call began with.
__device__ __forceinline__ void chain_leave(ChainShared &sh, const ChainArgs &ca, unsigned long long *slots, unsigned int *claims,
                                            int p, int ntiles, int tid) {
  const int S = ca.t.S;
  __syncthreads();
  if (tid == 0) sh.missing = (int)(atomicAdd(&claims[S], 1u) + 1u);
  __syncthreads();
  if (sh.missing == ntiles) {
    for (size_t i = (size_t)ca.first * ntiles + tid; i < (size_t)(ca.last + 1) * ntiles; i += 512) slots[i] = 0ull;
    for (int i = tid; i <= S; i += 512) claims[i] = 0u;
    if (tid == 0 && sh.st16[15] == 0) ca.t.alive[p] = 0;
  }
}

// Everything between two decisions, for a kernel without anything of its own to do meanwhile: on to tile t of the
// open decision or of the next one; false behind the last one.  Every thread calls it when no tile is left to score.
[[maybe_unused]] __device__ __forceinline__ bool chain_between(ChainShared &sh, const ChainArgs &ca, unsigned long long *slots,
                                                               unsigned int *claims, int p, size_t row, int member, int &cur,
                                                               int &stage, int &t, unsigned int &c_next, int32_t &pre, int tid) {
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), next = stage + 1;
  DecPack &nk = sh.pks[cur ^ 1];
  const DecPack &pk = sh.pks[cur];
  const bool opens = next < ca.t.S, decides = next <= ca.last;
  if (tid == CLAIMER && decides && c_next == NO_CLAIM) c_next = atomicAdd(&claims[next], 1u);
  chain_rows(sh, nk, pk, ca, p, row, stage, c_next, pre, tid, lane, w);
  if (stage >= ca.first) {
    if (w == 7) chain_poll(sh, ca, slots, claims, ca.ntiles, stage, c_next, lane);
    __syncthreads();
    if (sh.missing >= 0) {
      t = __builtin_amdgcn_readfirstlane(sh.missing);
      __syncthreads();  // (before the word is written again)
      return true;
    }
    winner_rows(sh, pk, sh.win_c, lane, w);
    __syncthreads();
    chain_tables(sh, pk, ca, p, row, stage, member, tid);
  }
  if (!opens) return false;
  next_shared_rows(sh, nk, stage >= ca.first, stage, tid);
  __syncthreads();
  if (tid == 0) next_derive(sh, nk, stage >= ca.first, stage);
  __syncthreads();
  if (!decides) {
    // (a schedule in pieces: the context is left for the call that goes on)
    if (member == 0)
      for (int i = tid; i < VF_DECPACK_DWORDS; i += 512)
        ca.decpack[(size_t)p * VF_DECPACK_DWORDS + i] = reinterpret_cast<const uint32_t *>(&nk)[i];
    return false;
  }
  fill_evaltabs(sh.tabs, nk.d, nk.sp);
  t = __builtin_amdgcn_readfirstlane(sh.claim);
  c_next = NO_CLAIM;
  cur ^= 1;
  stage = next;
  if (w == 6) pre = chain_prefetch(ca, row, stage, lane);
  __syncthreads();
  return true;
}

// The arguments of a launch over stages first..last; VF_ENOMEM without memory for its words.
[[maybe_unused]] static int chain_args(vf_ctx *c, int first, int last, int ntiles, int32_t *out_states, int32_t *out_cids,
                                       float *out_vals, ChainArgs *ca) {
  const size_t nslots = (size_t)c->B * c->S * ntiles, nclaims = (size_t)c->B * (c->S + 1);
  const int rc = vfk_chain_words(c, (nslots * 8 + nclaims * 4 + 15) / 16);
  if (rc != VF_OK) return rc;
  ca->t = tables_of(c);
  ca->first = first; ca->last = last;
  ca->M = c->M;
  ca->nprob = c->B;
  ca->ntiles = ntiles;
  ca->slots = c->d_chain;
  ca->claims = reinterpret_cast<unsigned int *>(c->d_chain + nslots);
  ca->wait_rounds = c->wait_rounds;
  ca->decpack = c->d_decpack;
  ca->out_states = out_states; ca->out_cids = out_cids; ca->out_vals = out_vals;
  ca->stat = c->profiling ? c->d_stat : nullptr;
  return VF_OK;
}

#endif  // VF_CHAIN_DEV_H
