// The recurrent value network of Sec. 3.2 wired to the search (gfx950).
//
// V reads a state as a sequence with one timestep per stage of the pipeline, in
// scheduling order: a stage that is scheduled in the state gives its 64 core features,
// a stage that is not gives its intrinsic block and zeros; every timestep's hidden
// state goes through the linear head and the predictions are summed.  For the
// candidates of decision i all timesteps before i are the same, so the recurrence over
// the committed prefix is kept per problem (cell state, the fed-back h folded into the
// gate pre-activations of the next step, the head's sum so far) and advanced by one
// step at every commit.  A candidate then costs one cell step on its own features plus
// one step per stage still unscheduled; for those the input part of the gates does not
// depend on the candidate either and comes from a per-problem table.
#include "vf_internal.h"

namespace {

#include "vf_sched_dev.h"
#include "vf_score_dev.h"

// fp32 blob of the model: W_ih[4H][64], W_hh[4H][H], b_ih[4H], b_hh[4H], w_head[H], b_head
struct SeqWeights {
  const float *Wih, *Whh, *bih, *bhh, *wh, *bh;
  int H;
};

__device__ __forceinline__ float wave_sum(float v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// G[b][t][r] = b_ih[r] + b_hh[r] + sum_{k<16} W_ih[r][k] x_k, x = the normalised intrinsic
// block of stage t: the input part of the gates of a stage that is not scheduled yet.
__global__ __launch_bounds__(256) void k_seq_tables(const int32_t *intr, SeqWeights sw, size_t n_bt, float *G) {
  const int H4 = 4 * sw.H;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_bt * (size_t)H4) return;
  const size_t bt = i / H4;
  const int r = (int)(i % H4);
  float acc = 0.0f;
#pragma unroll
  for (int k = 0; k < 16; ++k)
    acc = fmaf(bf16_val(sw.Wih[(size_t)r * 64 + k]), bf16_val(plog2_dev(intr[bt * 16 + k])), acc);
  G[i] = acc + sw.bih[r] + sw.bhh[r];
}

// the recurrence before the first stage: h = c = 0, so the gates start from the biases
__global__ __launch_bounds__(256) void k_seq_reset(SeqWeights sw, int B, float *hfb, float *cpre, float *P,
                                                   float *hsum) {
  const int H = sw.H;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < (size_t)B * H) { hfb[i] = 0.0f; cpre[i] = 0.0f; }
  if (i < (size_t)B * 4 * H) P[i] = sw.bih[i % (4 * H)] + sw.bhh[i % (4 * H)];
  if (i < (size_t)B) hsum[i] = 0.0f;
}

// One cell step per problem on the vector committed for `stage`; then the part of the
// next step's gates that comes from the new h.  A problem whose schedule has ended
// keeps its state (it has no candidates any more).  With sel_idx (beam search) slot b
// of the dst set continues the recurrence of its parent slot sel_idx[b] / Mpad of the
// src set; slots past the sel_n[0] survivors are dead and left alone.
struct SeqState {
  float *hfb, *cpre, *P, *hsum;  // [B][H] (bf16 values), [B][H], [B][4H], [B]
};

constexpr int SEQ_PB = 4;  // problems per workgroup of k_seq_advance: they share the weight reads

// [W_ih | W_hh] transposed and rounded: WT[k][r], k over the 64 inputs then the H hidden
// units, r over the 4H gate rows, so that thread r of a block reads its row coalesced.
__global__ __launch_bounds__(256) void k_pack_seqT(SeqWeights sw, float *WT) {
  const int H = sw.H, H4 = 4 * H;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)(64 + H) * H4) return;
  const int k = (int)(i / H4), r = (int)(i % H4);
  WT[i] = bf16_val(k < 64 ? sw.Wih[(size_t)r * 64 + k] : sw.Whh[(size_t)r * H + (k - 64)]);
}

__global__ __launch_bounds__(1024) void k_seq_advance(Tables t, int stage, SeqWeights sw, const float *WT, SeqState src,
                                                      SeqState dst, const int32_t *sel_idx, const int32_t *sel_n,
                                                      int64_t Mpad, int B) {
  __shared__ float x[SEQ_PB][64], z[SEQ_PB][1024], hn[SEQ_PB][256], hraw[SEQ_PB][256];
  __shared__ int from_s[SEQ_PB], mode_s[SEQ_PB];  // 0: leave alone, 1: carry the state over, 2: one cell step
  const int tid = threadIdx.x, lane = tid & 63;
  const int H = sw.H, H4 = 4 * H, S = t.S;
  const int b0 = blockIdx.x * SEQ_PB;
  if (tid < SEQ_PB) {
    const int b = b0 + tid;
    int mode = 0, from = b;
    if (b < B) {
      const bool survivor = !sel_idx || b < sel_n[0];  // beam search: slots past the survivors are dead
      if (survivor) {
        if (sel_idx) from = (int)((int64_t)sel_idx[b] / Mpad);
        const bool live = t.cids[(size_t)b * S + stage] >= 0;
        mode = live ? 2 : (src.cpre != dst.cpre ? 1 : 0);
      }
    }
    from_s[tid] = from;
    mode_s[tid] = mode;
  }
  __syncthreads();
  for (int i = tid; i < SEQ_PB * 64; i += 1024) {
    const int pb = i / 64, k = i % 64;
    x[pb][k] = mode_s[pb] == 2 ? bf16_val(plog2_dev(t.cf[((size_t)(b0 + pb) * S + stage) * 64 + k])) : 0.0f;
  }
  __syncthreads();
  // gate pre-activations: thread r owns row r for the block's problems
  if (tid < H4) {
    float acc[SEQ_PB];
#pragma unroll
    for (int pb = 0; pb < SEQ_PB; ++pb) acc[pb] = 0.0f;
#pragma unroll 16
    for (int k = 0; k < 64; ++k) {
      const float wv = WT[(size_t)k * H4 + tid];
#pragma unroll
      for (int pb = 0; pb < SEQ_PB; ++pb) acc[pb] = fmaf(wv, x[pb][k], acc[pb]);
    }
#pragma unroll
    for (int pb = 0; pb < SEQ_PB; ++pb)
      if (mode_s[pb] == 2) z[pb][tid] = src.P[(size_t)from_s[pb] * H4 + tid] + acc[pb];
  }
  __syncthreads();
  for (int i = tid; i < SEQ_PB * H; i += 1024) {
    const int pb = i / H, u = i % H, b = b0 + pb, from = from_s[pb];
    if (mode_s[pb] == 2) {
      float cn = src.cpre[(size_t)from * H + u];
      const float h = lstm_cell(z[pb][u], z[pb][H + u], z[pb][2 * H + u], z[pb][3 * H + u], cn);
      dst.cpre[(size_t)b * H + u] = cn;
      hraw[pb][u] = h;
      hn[pb][u] = bf16_val(h);
      dst.hfb[(size_t)b * H + u] = hn[pb][u];
    } else if (mode_s[pb] == 1) {
      dst.cpre[(size_t)b * H + u] = src.cpre[(size_t)from * H + u];
      dst.hfb[(size_t)b * H + u] = src.hfb[(size_t)from * H + u];
    }
  }
  __syncthreads();
  // the head's prediction for this timestep: one wave per problem, fixed order
  if (tid < SEQ_PB * 64) {
    const int pb = tid / 64;
    if (mode_s[pb] == 2) {
      float v = 0.0f;
      for (int u = lane; u < H; u += 64) v = fmaf(bf16_val(sw.wh[u]), hraw[pb][u], v);
      v = wave_sum(v);
      if (lane == 0) dst.hsum[b0 + pb] = src.hsum[from_s[pb]] + v + sw.bh[0];
    } else if (mode_s[pb] == 1 && lane == 0) {
      dst.hsum[b0 + pb] = src.hsum[from_s[pb]];
    }
  }
  // the h part of the next step's gates
  if (tid < H4) {
    float acc[SEQ_PB];
#pragma unroll
    for (int pb = 0; pb < SEQ_PB; ++pb) acc[pb] = 0.0f;
#pragma unroll 16
    for (int k = 0; k < H; ++k) {
      const float wv = WT[(size_t)(64 + k) * H4 + tid];
#pragma unroll
      for (int pb = 0; pb < SEQ_PB; ++pb) acc[pb] = fmaf(wv, hn[pb][k], acc[pb]);
    }
    const float bias = sw.bih[tid] + sw.bhh[tid];
#pragma unroll
    for (int pb = 0; pb < SEQ_PB; ++pb) {
      if (mode_s[pb] == 2) dst.P[(size_t)(b0 + pb) * H4 + tid] = bias + acc[pb];
      else if (mode_s[pb] == 1) dst.P[(size_t)(b0 + pb) * H4 + tid] = src.P[(size_t)from_s[pb] * H4 + tid];
    }
  }
}

// The valid candidates of decision (problem b, stage), in ascending id order:
// list[b][0..count[b]).  The recurrent network costs one cell step per remaining stage and
// candidate, so the scoring kernel works on this dense list instead of the id range, where
// valid and invalid ids are interleaved.  Also fills the masked score array (nullable)
// with +inf: the scorer then only writes the candidates' entries.
__global__ __launch_bounds__(1024) void k_seq_compact(const uint32_t *decpack, uint32_t M, int64_t Mpad, int32_t *list,
                                                      int32_t *count, float *scores) {
  __shared__ DecPack pk;
  __shared__ int wsum[16];
  __shared__ int base;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid < VF_DECPACK_DWORDS) reinterpret_cast<uint32_t *>(&pk)[tid] = decpack[(size_t)b * VF_DECPACK_DWORDS + tid];
  if (tid == 0) base = 0;
  __syncthreads();
  for (uint32_t c0 = 0; c0 < (uint32_t)Mpad; c0 += 1024u) {
    const uint32_t cid = c0 + tid;
    bool ok = false;
    if (cid < M && !range_closed(pk.d, pk.sp, c0, c0 + 1024u < M ? c0 + 1024u : M)) {
      uint32_t dec;
      ok = eval_candidate<false>(pk.d, pk.sp, cid, dec, nullptr);
    }
    if (scores && cid < (uint32_t)Mpad) scores[(size_t)b * Mpad + cid] = __builtin_inff();
    const unsigned long long m = __ballot(ok);
    if (lane == 0) wsum[w] = __popcll(m);
    __syncthreads();
    int off = base;
    for (int k = 0; k < w; ++k) off += wsum[k];
    if (ok) list[(size_t)b * Mpad + off + __popcll(m & ((1ull << lane) - 1ull))] = (int32_t)cid;
    __syncthreads();
    if (tid == 0) {
      int tot = 0;
      for (int k = 0; k < 16; ++k) tot += wsum[k];
      base += tot;
    }
    __syncthreads();
  }
  if (tid == 0) count[b] = base;
}

struct SeqDev {
  int H, S;
  const uint16_t *w_pack;  // [unit tile][k step][gate][lane][8]; 4 k-steps of x, then H/16 of h
  const float *aux;        // b_ih + b_hh [4H], head vector [H] (bf16 values), head bias
  const float *G;          // [B][S][4H]
  const float *P;          // [B][4H]
  const float *cpre;       // [B][H]
  const float *hsum;       // [B]
  const uint32_t *decpack; // [B][VF_DECPACK_DWORDS]
  const int32_t *list;     // [B][Mpad] valid candidate ids of the decision, ascending
  const int32_t *count;    // [B]
  int64_t Mpad;
  unsigned long long *stat;
};

// Workgroup = NC consecutive entries of the valid-candidate list of decision `stage` of
// problem blockIdx.y: featurize them, one cell step on their features from the problem's prefix state, one
// step per later stage, the head's sum, the tile's first minimum.  Wave w owns hidden
// units 32w..32w+31 (their four gate row tiles); c lives in registers, h goes through
// LDS as bf16, double-buffered; the weight fragments of a step are one contiguous stream
// per wave, kept PD k-steps ahead in a register ring that wraps at the end of the step;
// the per-step gate biases of the problem are staged through LDS one step ahead.
template <int NC, int PD>
__global__ __launch_bounds__(512) void k_seq_step(SeqDev md, int stage, int64_t M, float *scores, int64_t ld_scores,
                                                  float *pval, int32_t *pidx, NoiseArgs na) {
  constexpr int CT = NC / 32;
  constexpr int XLD = 72;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int H = md.H, S = md.S, H4 = 4 * H, hld = H + 8;
  uint16_t *xs = reinterpret_cast<uint16_t *>(smem);                    // [NC][XLD]
  uint16_t *hs = xs + (size_t)NC * XLD;                                 // [2][NC][hld]
  float *gls = reinterpret_cast<float *>(hs + (size_t)2 * NC * hld);    // [2][4H]
  float *red = gls + 2 * H4;                                            // [8][NC]
  float *whs = red + 8 * NC;                                            // [H]
  int32_t *okf = reinterpret_cast<int32_t *>(whs + H);                  // [NC]
  int32_t *cids = okf + NC;                                             // [NC] candidate id of each column
  __shared__ DecPack pk;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.y, nparts = gridDim.x;
  const int64_t n0 = (int64_t)blockIdx.x * NC;
  const size_t slot = (size_t)b * nparts + blockIdx.x;

  if (tid < VF_DECPACK_DWORDS)
    reinterpret_cast<uint32_t *>(&pk)[tid] = md.decpack[(size_t)b * VF_DECPACK_DWORDS + tid];
  __syncthreads();

  const int nvalid = md.count[b];
  if (n0 >= nvalid) {
    // past the end of the list: nothing for the network to do
    if (tid == 0) {
      pval[slot] = __builtin_inff();
      pidx[slot] = -1;
    }
    return;
  }
  // four threads per candidate, each producing 16 of the 64 core rows
  if (tid < NC) cids[tid] = (n0 + tid) < nvalid ? md.list[(size_t)b * md.Mpad + n0 + tid] : -1;
  if (tid < 4 * NC) {
    const int n = tid % NC, part = tid / NC;
    const bool inb = (n0 + n) < nvalid;
    const uint32_t cid = inb ? (uint32_t)md.list[(size_t)b * md.Mpad + n0 + n] : 0u;
    int32_t core[64];
    uint32_t dec;
    // the parts a thread does not store are dead code in its copy of the evaluation
    auto put = [&](const int32_t *v, int row0) {
      uint4 q0, q1;
      q0.x = pack_bf16(plog2_dev(v[0]), plog2_dev(v[1]));
      q0.y = pack_bf16(plog2_dev(v[2]), plog2_dev(v[3]));
      q0.z = pack_bf16(plog2_dev(v[4]), plog2_dev(v[5]));
      q0.w = pack_bf16(plog2_dev(v[6]), plog2_dev(v[7]));
      q1.x = pack_bf16(plog2_dev(v[8]), plog2_dev(v[9]));
      q1.y = pack_bf16(plog2_dev(v[10]), plog2_dev(v[11]));
      q1.z = pack_bf16(plog2_dev(v[12]), plog2_dev(v[13]));
      q1.w = pack_bf16(plog2_dev(v[14]), plog2_dev(v[15]));
      if (!inb) q0 = q1 = make_uint4(0u, 0u, 0u, 0u);
      uint4 *dst = reinterpret_cast<uint4 *>(xs + (size_t)n * XLD + row0);
      dst[0] = q0;
      dst[1] = q1;
    };
    if (part == 0) {
      // evaluated for padding columns too: core must be defined before put reads it
      const bool okc = eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      okf[n] = inb && okc;
      put(core, 0);
    } else if (part == 1) {
      eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      put(core + 16, 16);
    } else if (part == 2) {
      eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      put(core + 32, 32);
    } else {
      eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      put(core + 48, 48);
    }
  }

  const bool active = w < H / 32;
  const int wu = active ? w : 0;  // idle waves shadow tile 0 but never store
  const int ksh = H / 16, ksteps = 4 + ksh;
  // the wave's weight stream (4 k-steps of x part, then the h part): base in scalar registers,
  // 16 bytes per lane, fragment i at byte 1024 i
  const __amdgpu_buffer_rsrc_t ws = stream_rsrc(reinterpret_cast<const uint4 *>(md.w_pack) + (size_t)wu * ksteps * 4 * 64);
  const int voff = 16 * lane;
  int wstep = PD;  // the k-step of the stream that refills the next slot
  uint4 ring[PD][4];
#pragma unroll
  for (int j = 0; j < PD; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g) ring[j][g] = stream_load(ws, voff, j * 4 + g);

  for (int i = tid; i < H4; i += 512) gls[i] = md.P[(size_t)b * H4 + i];
  for (int i = tid; i < H; i += 512) whs[i] = md.aux[H4 + i];
  floatx16 cst[CT];
  float vsum[CT];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 cv = *reinterpret_cast<const float4 *>(md.cpre + (size_t)b * H + wu * 32 + 4 * (lane >> 5) + 8 * q);
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      cst[c][4 * q + 0] = cv.x; cst[c][4 * q + 1] = cv.y;
      cst[c][4 * q + 2] = cv.z; cst[c][4 * q + 3] = cv.w;
    }
  }
#pragma unroll
  for (int c = 0; c < CT; ++c) vsum[c] = 0.0f;
  __syncthreads();

  const int rowoff = (lane & 31), koff = 8 * (lane >> 5);
  for (int t = stage; t < S; ++t) {
    const int k = t - stage;
    // the next step's biases, fetched now, parked in LDS after this step's contraction
    const bool fetch_g = (t + 1 < S) && tid < H;
    float4 gnext = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (fetch_g) gnext = reinterpret_cast<const float4 *>(md.G + ((size_t)b * S + t + 1) * H4)[tid];

    // the step's gate biases (staged in LDS one step ahead) are the addends of the first k-step:
    // gate by gate, so that one bias vector is in registers at a time
    const float *bias = gls + (size_t)(k & 1) * H4;
    floatx16 acc[4][CT];

    if (active) {  // (waves without units of their own only keep the barriers company)
    const uint16_t *src = (k == 0) ? xs : hs + (size_t)(k & 1) * NC * hld;
    const int ld = (k == 0) ? XLD : hld;
    const int nsteps = (k == 0) ? 4 : ksh;
    {
      const uint16_t *brow = src + (size_t)rowoff * ld + koff;
      uint4 bcur[CT];
#pragma unroll
      for (int c = 0; c < CT; ++c) bcur[c] = *reinterpret_cast<const uint4 *>(brow + (size_t)c * 32 * ld);
      auto round = [&](int s0, auto startc) __attribute__((always_inline)) {
        constexpr bool starts = decltype(startc)::value;
        if (s0 + PD >= nsteps) wstep = 4;  // the next step's first fragments (always an h step)
#pragma unroll
        for (int j = 0; j < PD; ++j) {
          if constexpr (starts) {
            if (j == 0) {
              int boff = wu * 32 + 4 * (lane >> 5);
              asm volatile("" : "+v"(boff));  // (read afresh every step, not kept across them)
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                floatx16 bg;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  const float4 bv = *reinterpret_cast<const float4 *>(bias + g * H + boff + 8 * q);
                  bg[4 * q + 0] = bv.x; bg[4 * q + 1] = bv.y; bg[4 * q + 2] = bv.z; bg[4 * q + 3] = bv.w;
                }
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                  acc[g][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                      __builtin_bit_cast(bf16x8, ring[0][g]), __builtin_bit_cast(bf16x8, bcur[c]), bg, 0, 0, 0);
                  if (g == 3) bcur[c] = *reinterpret_cast<const uint4 *>(brow + (size_t)c * 32 * ld + 16);
                }
                ring[0][g] = stream_load(ws, voff, wstep * 4 + g);
              }
              continue;
            }
          }
          // column by column; every operand register is refilled in place behind the last product
          // that reads it: a column's activation fragment with the next k-step's (one k-step
          // past the end stays inside the row's padding or the next row), a weight fragment
          // with the one PD k-steps ahead
#pragma unroll
          for (int i = 0; i < 4 * CT; ++i) {
            const int c = i / 4, g = i % 4;
            acc[g][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, ring[j][g]), __builtin_bit_cast(bf16x8, bcur[c]), acc[g][c], 0, 0, 0);
            if (g == 3) bcur[c] = *reinterpret_cast<const uint4 *>(brow + (size_t)c * 32 * ld + (s0 + j + 1) * 16);
            if (c == CT - 1) ring[j][g] = stream_load(ws, voff, (wstep + j) * 4 + g);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        wstep += PD;
      };
      round(0, vf_tag<true>{});
      for (int s0 = PD; s0 < nsteps; s0 += PD) round(s0, vf_tag<false>{});
    }
    uint16_t *hout = hs + (size_t)((k + 1) & 1) * NC * hld;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int u0 = wu * 32 + 4 * (lane >> 5) + 8 * q;
      const float4 whv = *reinterpret_cast<const float4 *>(whs + u0);
      const float whq[4] = {whv.x, whv.y, whv.z, whv.w};
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        float hv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int j = 4 * q + e;
          float cn = cst[c][j];
          hv[e] = lstm_cell(acc[0][c][j], acc[1][c][j], acc[2][c][j], acc[3][c][j], cn);
          cst[c][j] = cn;
          vsum[c] = fmaf(whq[e], hv[e], vsum[c]);
        }
        uint2 pkd;
        pkd.x = pack_bf16(hv[0], hv[1]);
        pkd.y = pack_bf16(hv[2], hv[3]);
        *reinterpret_cast<uint2 *>(hout + (size_t)(c * 32 + (lane & 31)) * hld + u0) = pkd;
      }
    }
    }
    if (fetch_g) reinterpret_cast<float4 *>(gls + (size_t)((k + 1) & 1) * H4)[tid] = gnext;
    __syncthreads();  // h_t and the next step's biases are in place
  }

#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const float v = vsum[c] + __shfl_xor(vsum[c], 32);
    if (lane < 32) red[w * NC + c * 32 + lane] = active ? v : 0.0f;
  }
  __syncthreads();
  if (tid < NC) {
    float s = md.hsum[b] + (float)(S - stage) * md.aux[H4 + H];
#pragma unroll
    for (int g = 0; g < 8; ++g) s += red[g * NC + tid];
    const bool ok = okf[tid] != 0;
    const int32_t cid = cids[tid];
    if (scores && ok) scores[(size_t)b * ld_scores + cid] = s;
    if (na.eps != 0.0f) s = add_noise(na, s, b, cid);
    float v = __builtin_inff();
    int32_t c = -1;
    if (ok && s < v) { v = s; c = cid; }
    wave_min(v, c);
    if (md.stat) {
      const int nok = __popcll(__ballot(ok));
      if (lane == 0) {
        atomicAdd(&md.stat[0], (unsigned long long)nok);
        atomicAdd(&md.stat[1], (unsigned long long)nok);
      }
    }
    if (tid == 0) {
      pval[slot] = v;
      pidx[slot] = c;
    }
  }
}

// The same for tiles of 96 entries.  What bounds k_seq_step is that its two phases alternate: the
// contraction of a tile of 64 waits for the weight stream (512 KB per step out of L2 at H = 256, 1.5
// times what its products take), then the gates keep the vector ALUs busy for as long with the matrix
// cores idle.  Here the stream serves 96 entries, so that the products take as long as the stream, and
// a wave does its 32 hidden units in two passes of 16 (all four gates: two row tiles, three column
// tiles, 96 accumulators), with the waves 0..3 ahead of the waves 4..7 by wave priority: on every SIMD
// one wave's gates run under the other wave's products.  A step of 96 takes about 22k cycles, 20k of
// them vector work of the gates (210 cycles per cell and wave, 128 of those in 5 exp and 3 rcp).
// 64 problems of 20 layers, H = 256: 19.4 -> 17.0 ms per schedule, H = 128 8.7 -> 7.5, 12 layers of other
// shapes 5.4 -> 3.1.  (128 entries: the accumulators and cell states leave no registers, and what is
// spilled in the gates comes back behind the weight fragments under way: 28.6 ms.)
// The weights are one stream per wave (k_pack_seq_wide): per pass the k-steps of h, then those of x;
// row tile 0 of a pass holds gate i of its units in rows 0..15 and gate f in rows 16..31, row tile 1
// the gates g and o.  The first step's x lies in the h buffer that the second step writes.
constexpr int SEQ_WIDE = 96;
template <int PD>
__global__ __launch_bounds__(512) void k_seq_step_wide(SeqDev md, const uint16_t *w_wide, int stage, float *scores,
                                                       int64_t ld_scores, float *pval, int32_t *pidx, NoiseArgs na) {
  constexpr int NC = SEQ_WIDE, CT = NC / 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int H = md.H, S = md.S, H4 = 4 * H, hld = H + 8;
  uint16_t *hs = reinterpret_cast<uint16_t *>(smem);                    // [2][NC][max(hld, 72)]
  const int hcol = hld < 72 ? 72 : hld;
  float *gls = reinterpret_cast<float *>(hs + (size_t)2 * NC * hcol);   // [2][4H]
  float *red = gls + 2 * H4;                                            // [8][NC]
  float *whs = red + 8 * NC;                                            // [H]
  int32_t *okf = reinterpret_cast<int32_t *>(whs + H);                  // [NC] candidate id + 1, 0 = none
  __shared__ DecPack pk;
  __shared__ float sv[2];
  __shared__ int32_t sc[2];

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.y, nparts = gridDim.x;
  const int64_t n0 = (int64_t)blockIdx.x * NC;
  const size_t slot = (size_t)b * nparts + blockIdx.x;

  const int nvalid = md.count[b];
  if (n0 >= nvalid) {
    if (tid == 0) {
      pval[slot] = __builtin_inff();
      pidx[slot] = -1;
    }
    return;
  }
  if (tid < VF_DECPACK_DWORDS)
    reinterpret_cast<uint32_t *>(&pk)[tid] = md.decpack[(size_t)b * VF_DECPACK_DWORDS + tid];
  const bool active = w < H / 32;
  const int wu = active ? w : 0;  // idle waves shadow the first units but never store
  const int ksh = H / 16;
  const __amdgpu_buffer_rsrc_t ws = stream_rsrc(reinterpret_cast<const uint4 *>(w_wide) + (size_t)wu * (2 * ksh + 8) * 2 * 64);
  const int voff = 16 * lane;
  // (the first step's x part sits behind the passes' h parts)
  int wstep = 2 * ksh + PD;
  uint4 ring[PD][2];
#pragma unroll
  for (int j = 0; j < PD; ++j)
#pragma unroll
    for (int r = 0; r < 2; ++r) ring[j][r] = stream_load(ws, voff, (2 * ksh + j) * 2 + r);
  for (int i = tid; i < H4; i += 512) gls[i] = md.P[(size_t)b * H4 + i];
  for (int i = tid; i < H; i += 512) whs[i] = md.aux[H4 + i];
  __syncthreads();
  if (tid < 4 * NC) {
    // four threads per candidate, each producing 16 of the 64 core rows (what a thread does not
    // store is dead code in its copy); padding columns are evaluated too and store zeros
    const int n = tid % NC, part = tid / NC;
    const bool inb = (n0 + n) < nvalid;
    const uint32_t cid = inb ? (uint32_t)md.list[(size_t)b * md.Mpad + n0 + n] : 0u;
    int32_t core[64];
    uint32_t dec;
    auto put = [&](const int32_t *v, int row0) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        uint4 q;
        q.x = pack_bf16(plog2_dev(v[8 * k + 0]), plog2_dev(v[8 * k + 1]));
        q.y = pack_bf16(plog2_dev(v[8 * k + 2]), plog2_dev(v[8 * k + 3]));
        q.z = pack_bf16(plog2_dev(v[8 * k + 4]), plog2_dev(v[8 * k + 5]));
        q.w = pack_bf16(plog2_dev(v[8 * k + 6]), plog2_dev(v[8 * k + 7]));
        if (!inb) q = make_uint4(0u, 0u, 0u, 0u);
        reinterpret_cast<uint4 *>(hs + (size_t)n * hcol + row0)[k] = q;
      }
    };
    if (part == 0) {
      const bool okc = eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      okf[n] = inb && okc ? (int32_t)cid + 1 : 0;
      put(core, 0);
    } else if (part == 1) {
      eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      put(core + 16, 16);
    } else if (part == 2) {
      eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      put(core + 32, 32);
    } else {
      eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      put(core + 48, 48);
    }
  }
  // cell state: per pass and column tile a lane's eight units 8 q + 4 (lane / 32) + e of the pass's 16
  float cst[2][CT][8];
  float vsum[CT];
#pragma unroll
  for (int ps = 0; ps < 2; ++ps)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float4 cv = *reinterpret_cast<const float4 *>(md.cpre + (size_t)b * H + wu * 32 + 16 * ps + 8 * q + 4 * (lane >> 5));
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        cst[ps][c][4 * q + 0] = cv.x; cst[ps][c][4 * q + 1] = cv.y;
        cst[ps][c][4 * q + 2] = cv.z; cst[ps][c][4 * q + 3] = cv.w;
      }
    }
#pragma unroll
  for (int c = 0; c < CT; ++c) vsum[c] = 0.0f;
  __syncthreads();

  for (int t = stage; t < S; ++t) {
    const int k = t - stage;
    // the next step's biases, fetched now, parked in LDS after this step's passes
    const bool fetch_g = (t + 1 < S) && tid < H;
    float4 gnext = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (fetch_g) gnext = reinterpret_cast<const float4 *>(md.G + ((size_t)b * S + t + 1) * H4)[tid];
    const uint16_t *src = hs + (size_t)(k & 1) * NC * hcol;
    uint16_t *hout = hs + (size_t)((k + 1) & 1) * NC * hcol;
    if (active) {
#pragma unroll
    for (int ps = 0; ps < 2; ++ps) {
      int u0 = wu * 32 + 16 * ps + 4 * (lane >> 5);  // the lane's units: u0 + 8 q + e
      asm volatile("" : "+v"(u0));                   // (biases read afresh every step, not kept across them)
      floatx16 acc[2][CT];
      const uint16_t *bb = src + (size_t)(lane & 31) * hcol + 8 * (lane >> 5);
      const int nsteps = k == 0 ? 4 : ksh;
      if (w < 4) __builtin_amdgcn_s_setprio(3);
      else __builtin_amdgcn_s_setprio(1);
      {
        uint4 bcur[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) bcur[c] = *reinterpret_cast<const uint4 *>(bb + (size_t)c * 32 * hcol);
        __builtin_amdgcn_s_waitcnt(0x0070);  // (see contract_layer)
        auto round = [&](int s0, auto startc) __attribute__((always_inline)) {
          constexpr bool starts = decltype(startc)::value;
          if (ps == 1 && s0 + PD >= nsteps) wstep = 0;  // the next step's first fragments
#pragma unroll
          for (int j = 0; j < PD; ++j) {
            if constexpr (starts) {
              if (j == 0) {
                // the first k-step takes the step's gate biases as its addend, row tile by row tile,
                // so that one of the two bias vectors is in registers at a time
                const float *bias = gls + (size_t)(k & 1) * H4 + u0;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                  floatx16 bg;
#pragma unroll
                  for (int g = 0; g < 4; ++g) {
                    const float4 v = *reinterpret_cast<const float4 *>(bias + (2 * r + (g >> 1)) * H + 8 * (g & 1));
                    bg[4 * g + 0] = v.x; bg[4 * g + 1] = v.y; bg[4 * g + 2] = v.z; bg[4 * g + 3] = v.w;
                  }
#pragma unroll
                  for (int c = 0; c < CT; ++c) {
                    acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[0][r]),
                                                                       __builtin_bit_cast(bf16x8, bcur[c]), bg, 0, 0, 0);
                    if (r == 1) bcur[c] = *reinterpret_cast<const uint4 *>(bb + (size_t)c * 32 * hcol + 16);
                  }
                  ring[0][r] = stream_load(ws, voff, wstep * 2 + r);
                  __builtin_amdgcn_sched_barrier(0);
                }
                continue;
              }
            }
#pragma unroll
            for (int i = 0; i < 2 * CT; ++i) {
              const int c = i / 2, r = i % 2;
              acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[j][r]),
                                                                 __builtin_bit_cast(bf16x8, bcur[c]), acc[r][c], 0, 0, 0);
              if (r == 1) bcur[c] = *reinterpret_cast<const uint4 *>(bb + (size_t)c * 32 * hcol + (s0 + j + 1) * 16);
              if (c == CT - 1) ring[j][r] = stream_load(ws, voff, (wstep + j) * 2 + r);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
          wstep += PD;
        };
        round(0, vf_tag<true>{});
        for (int s0 = PD; s0 < nsteps; s0 += PD) round(s0, vf_tag<false>{});
      }
      __builtin_amdgcn_s_setprio(0);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float4 whv = *reinterpret_cast<const float4 *>(whs + u0 + 8 * q);
        const float whq[4] = {whv.x, whv.y, whv.z, whv.w};
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          float hv[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float cn = cst[ps][c][4 * q + e];
            hv[e] = lstm_cell(acc[0][c][4 * q + e], acc[0][c][8 + 4 * q + e], acc[1][c][4 * q + e], acc[1][c][8 + 4 * q + e], cn);
            cst[ps][c][4 * q + e] = cn;
            vsum[c] = fmaf(whq[e], hv[e], vsum[c]);
          }
          uint2 pkd;
          pkd.x = pack_bf16(hv[0], hv[1]);
          pkd.y = pack_bf16(hv[2], hv[3]);
          *reinterpret_cast<uint2 *>(hout + (size_t)(c * 32 + (lane & 31)) * hcol + u0 + 8 * q) = pkd;
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    }
    if (fetch_g) reinterpret_cast<float4 *>(gls + (size_t)((k + 1) & 1) * H4)[tid] = gnext;
    __syncthreads();  // h_t and the next step's biases are in place
  }

#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const float v = vsum[c] + __shfl_xor(vsum[c], 32);
    if (lane < 32) red[w * NC + c * 32 + lane] = active ? v : 0.0f;
  }
  __syncthreads();
  if (tid < (NC + 63) / 64 * 64) {
    const bool col = tid < NC;
    float s = md.hsum[b] + (float)(S - stage) * md.aux[H4 + H];
#pragma unroll
    for (int g = 0; g < 8; ++g) s += col ? red[g * NC + tid] : 0.0f;
    const int32_t cid = col ? okf[tid] - 1 : -1;
    const bool ok = cid >= 0;
    if (scores && ok) scores[(size_t)b * ld_scores + cid] = s;
    if (na.eps != 0.0f) s = add_noise(na, s, b, cid);
    float v = __builtin_inff();
    int32_t c = -1;
    if (ok && s < v) { v = s; c = cid; }
    wave_min(v, c);
    if (md.stat) {
      const int nok = __popcll(__ballot(ok));
      if (lane == 0) {
        atomicAdd(&md.stat[0], (unsigned long long)nok);
        atomicAdd(&md.stat[1], (unsigned long long)nok);
      }
    }
    if (lane == 0) { sv[w] = v; sc[w] = c; }
  }
  __syncthreads();
  if (tid == 0) {
    float v = sv[0];
    int32_t c = sc[0];
    take_min(v, c, sv[1], sc[1]);
    pval[slot] = v;
    pidx[slot] = c;
  }
}

// The weights of k_seq_step_wide: out[wave][step][row tile][lane][8], steps = k-steps of h of pass 0,
// of pass 1, then the four k-steps of x of either pass.
__global__ __launch_bounds__(256) void k_pack_seq_wide(SeqWeights sw, uint16_t *out) {
  const int H = sw.H, ksh = H / 16, steps = 2 * ksh + 8;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= H / 32 * steps * 1024) return;
  const int e = i & 7, lane = (i >> 3) & 63, r = (i >> 9) & 1, step = (i >> 10) % steps, w = (i >> 10) / steps;
  const bool of_x = step >= 2 * ksh;
  const int at = of_x ? step - 2 * ksh : step, per = of_x ? 4 : ksh, ps = at / per, s = at % per;
  const int row = lane & 31, gate = 2 * r + (row >> 4), unit = w * 32 + 16 * ps + (row & 15);
  const int k = s * 16 + 8 * (lane >> 5) + e;
  const float v = of_x ? sw.Wih[(size_t)(gate * H + unit) * 64 + k] : sw.Whh[(size_t)(gate * H + unit) * H + k];
  out[i] = (uint16_t)bf16_bits(v);
}

SeqWeights weights_of(const vf_ctx *c) {
  const int H = c->model.dims[1];
  SeqWeights sw;
  sw.H = H;
  sw.Wih = c->pm.w_f32;
  sw.Whh = sw.Wih + (size_t)4 * H * 64;
  sw.bih = sw.Whh + (size_t)4 * H * H;
  sw.bhh = sw.bih + 4 * H;
  sw.wh = sw.bhh + 4 * H;
  sw.bh = sw.wh + H;
  return sw;
}

SeqState state_of(const vf_ctx *c, int set) {
  SeqState s;
  s.hfb = c->d_seq_h[set]; s.cpre = c->d_seq_c[set]; s.P = c->d_seq_P[set]; s.hsum = c->d_seq_hs[set];
  return s;
}

}  // namespace

bool vfk_seq_model(const vf_ctx *c) {
  return c->has_model && c->model.kind == VF_LSTM && c->model.dtype == VF_BF16 && c->model.dims[0] == 64 &&
         c->pm.w_f32 != nullptr;
}

void vfk_seq_free(vf_ctx *c) {
  void *ps[] = {c->d_seq_G, c->d_seq_h[0], c->d_seq_h[1], c->d_seq_c[0], c->d_seq_c[1],
                c->d_seq_P[0], c->d_seq_P[1], c->d_seq_hs[0], c->d_seq_hs[1], c->d_seq_list, c->d_seq_count};
  for (void *p : ps)
    if (p) (void)hipFree(p);
  c->d_seq_G = nullptr;
  c->d_seq_list = nullptr;
  c->d_seq_count = nullptr;
  for (int k = 0; k < 2; ++k) c->d_seq_h[k] = c->d_seq_c[k] = c->d_seq_P[k] = c->d_seq_hs[k] = nullptr;
  c->seq_stage = -1;
  c->seq_cur = 0;
}

// Tables and prefix state of the recurrence for the context's pipeline, model and
// committed prefix: built on first use, rebuilt after anything but a commit changed them.
int vfk_seq_sync(vf_ctx *c, int stage) {
  const int H = c->model.dims[1], B = c->B, S = c->S;
  const SeqWeights sw = weights_of(c);
  hipStream_t st = c->stream;
  if (!c->d_seq_G) {
    struct { float **p; size_t n; } want[] = {
        {&c->d_seq_G, (size_t)B * S * 4 * H},
        {&c->d_seq_h[0], (size_t)B * H}, {&c->d_seq_h[1], (size_t)B * H},
        {&c->d_seq_c[0], (size_t)B * H}, {&c->d_seq_c[1], (size_t)B * H},
        {&c->d_seq_P[0], (size_t)B * 4 * H}, {&c->d_seq_P[1], (size_t)B * 4 * H},
        {&c->d_seq_hs[0], (size_t)B}, {&c->d_seq_hs[1], (size_t)B}};
    bool ok = true;
    for (auto &wt : want) ok = ok && hipMalloc((void **)wt.p, wt.n * sizeof(float)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->d_seq_list, (size_t)B * c->Mpad * 4) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->d_seq_count, (size_t)B * 4) == hipSuccess;
    if (!ok) {
      (void)hipGetLastError();
      vfk_seq_free(c);
      return VF_ENOMEM;
    }
    const size_t n = (size_t)B * S * 4 * H;
    hipLaunchKernelGGL(k_seq_tables, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, c->d_intr, sw,
                       (size_t)B * S, c->d_seq_G);
    VF_HIP(c, hipGetLastError());
    if (!c->pm.w_seqT) {
      const size_t nw = (size_t)(64 + H) * 4 * H;
      if (hipMalloc((void **)&c->pm.w_seqT, nw * sizeof(float)) != hipSuccess) {
        (void)hipGetLastError();
        vfk_seq_free(c);
        return VF_ENOMEM;
      }
      hipLaunchKernelGGL(k_pack_seqT, dim3((unsigned)((nw + 255) / 256)), dim3(256), 0, st, sw, c->pm.w_seqT);
      VF_HIP(c, hipGetLastError());
    }
    if (!c->pm.w_seq_wide) {
      // (without memory for this second form every step runs in tiles of 64, see vfk_seq_step)
      const size_t nv = (size_t)H / 32 * (2 * (H / 16) + 8) * 1024;
      if (hipMalloc((void **)&c->pm.w_seq_wide, nv * sizeof(uint16_t)) != hipSuccess) {
        (void)hipGetLastError();
        c->pm.w_seq_wide = nullptr;
      } else {
        hipLaunchKernelGGL(k_pack_seq_wide, dim3((unsigned)((nv + 255) / 256)), dim3(256), 0, st, sw, c->pm.w_seq_wide);
        VF_HIP(c, hipGetLastError());
      }
    }
    c->seq_stage = -1;
  }
  if (c->seq_stage == stage) return VF_OK;
  c->seq_cur = 0;
  const size_t n = (size_t)B * 4 * H;
  const SeqState s0 = state_of(c, 0);
  hipLaunchKernelGGL(k_seq_reset, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, sw, B, s0.hfb, s0.cpre, s0.P,
                     s0.hsum);
  VF_HIP(c, hipGetLastError());
  for (int t = 0; t < stage; ++t) {
    hipLaunchKernelGGL(k_seq_advance, dim3((unsigned)((B + SEQ_PB - 1) / SEQ_PB)), dim3(1024), 0, st, tables_of(c), t, sw,
                       (const float *)c->pm.w_seqT, s0, s0, (const int32_t *)nullptr, (const int32_t *)nullptr,
                       (int64_t)c->Mpad, B);
    VF_HIP(c, hipGetLastError());
  }
  c->seq_stage = stage;
  return VF_OK;
}

// after the commit of `stage`: one more step of every problem's prefix recurrence
int vfk_seq_advance(vf_ctx *c, int stage) {
  if (c->seq_stage != stage) return VF_OK;  // not in step: rebuilt at the next use
  const SeqState s = state_of(c, c->seq_cur);
  hipLaunchKernelGGL(k_seq_advance, dim3((unsigned)((c->B + SEQ_PB - 1) / SEQ_PB)), dim3(1024), 0, c->stream,
                     tables_of(c), stage, weights_of(c), (const float *)c->pm.w_seqT, s, s, (const int32_t *)nullptr,
                     (const int32_t *)nullptr, (int64_t)c->Mpad, c->B);
  VF_HIP(c, hipGetLastError());
  c->seq_stage = stage + 1;
  return VF_OK;
}

// beam search: slot j of the new layer continues the recurrence of its parent slot
int vfk_seq_advance_beam(vf_ctx *c, int stage) {
  if (c->seq_stage != stage) return VF_OK;
  const SeqState src = state_of(c, c->seq_cur), dst = state_of(c, c->seq_cur ^ 1);
  hipLaunchKernelGGL(k_seq_advance, dim3((unsigned)((c->B + SEQ_PB - 1) / SEQ_PB)), dim3(1024), 0, c->stream,
                     tables_of(c), stage, weights_of(c), (const float *)c->pm.w_seqT, src, dst,
                     (const int32_t *)c->d_sel_idx, (const int32_t *)c->d_sel_n, (int64_t)c->Mpad, c->B);
  VF_HIP(c, hipGetLastError());
  c->seq_cur ^= 1;
  c->seq_stage = stage + 1;
  return VF_OK;
}

// V of every candidate state of decision `stage` of every problem: per-tile minima into
// the partial arrays, optionally the masked scores [B][ld_scores].
int vfk_seq_step(vf_ctx *c, int stage, float *scores, int64_t ld_scores, int noise_stage, int *nparts_out) {
  int rc = vfk_seq_sync(c, stage);
  if (rc != VF_OK) return rc;
  rc = vfk_prepare(c, stage);
  if (rc != VF_OK) return rc;
  const int H = c->model.dims[1];
  // Tiles of 96 where tiles of 64 would be more than about one round of the compute units (a third
  // of the ids is valid, as a rule): 8 problems of 4096 ids 3.1 against 3.4 ms or 1.3 against 1.1, 12: 4.7
  // against 4.4 or 1.3 against 1.6, 16: 5.0 against 5.6, 64: 17.0 against 19.4; 1 problem: 2.9 against 2.2.
  int ncu = 256;
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device);
  const bool wide = c->pm.w_seq_wide && (c->M + 63) / 64 * c->B >= 3 * (int64_t)ncu;
  const int NC = wide ? SEQ_WIDE : 64;
  const int nparts = (int)((c->M + NC - 1) / NC);
  rc = vfk_ensure_parts(c, (size_t)nparts * c->B);
  if (rc != VF_OK) return rc;
  const SeqState s = state_of(c, c->seq_cur);
  SeqDev md;
  md.H = H; md.S = c->S; md.w_pack = c->pm.w_pack; md.aux = c->pm.aux;
  md.G = c->d_seq_G; md.P = s.P; md.cpre = s.cpre; md.hsum = s.hsum;
  md.decpack = c->d_decpack;
  md.list = c->d_seq_list; md.count = c->d_seq_count; md.Mpad = c->Mpad;
  md.stat = c->profiling ? c->d_stat : nullptr;
  hipLaunchKernelGGL(k_seq_compact, dim3((unsigned)c->B), dim3(1024), 0, c->stream, c->d_decpack, (uint32_t)c->M,
                     (int64_t)c->Mpad, c->d_seq_list, c->d_seq_count, scores);
  VF_HIP(c, hipGetLastError());
  NoiseArgs na;
  na.eps = noise_stage >= 0 ? c->noise_eps : 0.0f;
  na.k0 = (uint32_t)c->noise_seed; na.k1 = (uint32_t)(c->noise_seed >> 32);
  na.stage = noise_stage; na.first_rollout = c->noise_first;
  const int hld = H + 8;
  const size_t smem = (size_t)NC * 72 * 2 + (size_t)2 * NC * hld * 2 + (size_t)2 * 4 * H * 4 + (size_t)8 * NC * 4 +
                      (size_t)H * 4 + (size_t)2 * NC * 4;
  {
    vf_prof_scope prof(c, VF_PROF_SCORE);
    if (wide) {
      const int hcol = hld < 72 ? 72 : hld;
      const size_t lds = (size_t)2 * NC * hcol * 2 + (size_t)2 * 4 * H * 4 + (size_t)8 * NC * 4 + (size_t)H * 4 + (size_t)NC * 4;
      VF_HIP(c, hipFuncSetAttribute((const void *)k_seq_step_wide<2>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      hipLaunchKernelGGL(k_seq_step_wide<2>, dim3((unsigned)nparts, (unsigned)c->B), dim3(512), lds, c->stream, md,
                         (const uint16_t *)c->pm.w_seq_wide, stage, scores, ld_scores, c->d_pval, c->d_pidx, na);
      VF_HIP(c, hipGetLastError());
      *nparts_out = nparts;
      return VF_OK;
    }
    void (*kern)(SeqDev, int, int64_t, float *, int64_t, float *, int32_t *, NoiseArgs) = k_seq_step<64, 2>;
    VF_HIP(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    hipLaunchKernelGGL(kern, dim3((unsigned)nparts, (unsigned)c->B), dim3(512), smem, c->stream, md, stage, c->M,
                       scores, ld_scores, c->d_pval, c->d_pidx, na);
    VF_HIP(c, hipGetLastError());
  }
  *nparts_out = nparts;
  return VF_OK;
}
