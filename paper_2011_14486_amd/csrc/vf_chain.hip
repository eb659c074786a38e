// Algorithm 1 for a few problems in one launch (gfx950): as many workgroups as a decision has tiles of
// ids share a problem, and every one of them follows the whole schedule.
//
// With one round of tiles per decision a schedule is a chain: the winner's loop structure makes the next
// decision's context, the context the candidates' features and the folded first layer, those the scores,
// their minimum the winner.  A launch per layer spends a third of that chain on leaving the chip and
// coming back (the last store, the kernel boundary, the tables and contexts out of memory).  Here the only
// thing that travels between workgroups is a tile's first minimum: value and id in one 64-bit word of its own
// (slots), stored and polled past the caches, so that no fence and no flag is needed - a word that is not
// zero is complete.  The rest every workgroup works out for itself, identically: the winner, its rows (which
// all of them write to the tables, the same values), the next context.
//
// What does not depend on the winner is done while the minima are on their way: the next stage's
// records and the neighbour rows that only move on by one, the weights of the folded first layer (for tiles of 32
// four k-steps in registers and six in LDS for good), the ids of the next tile.
//
// What bounds it: the chain of small steps.  256-512-512-1, 20 layers of 4096 ids, one problem: 437 us with a launch
// per layer, 287 here (two problems 438 -> 293, four, with tiles of 64, 443 -> 304; 100 layers of 16384 ids 2342 ->
// 1599).  A decision takes 13 us: the tile 6 (features 0.8, first layer 0.5, hidden layer 4 with 512 KB of weights
// per compute unit at 55 bytes a cycle, output and scan 0.7), the minima 1.5, the winner 1.1, the context and the fold 2.6.  Tiles of
// 32 ids as long as there are compute units for them: the products of a tile of 64 take as long as its weights.
// Slower or the same: the winner's and the candidates' arithmetic in doubles, the context derived by several
// lanes, eight k-steps of weights in flight instead of four (spills), 1024 units per layer (spills; 988 against 807 us).
// Every store to the tables is waited for by the next use of a register that a load in flight may still fill: loads
// that are used behind them are waited for in front (the empty asm statements).
//
// Tiles are claimed (a counter per decision), and a claim is only made by a workgroup that is running: one
// for every decision, and those that are left over while it waits.  So every wait ends whether or not all workgroups
// are resident at once; the waits are bounded all the same,
// and a workgroup whose wait runs out scores the missing tile itself, with the same result.  The last
// workgroup of a problem to leave clears the problem's words for the next launch.
#include <type_traits>

#include "vf_internal.h"

namespace {

#include "vf_sched_dev.h"

#include "vf_score_dev.h"

#include "vf_chain_dev.h"

__global__ __launch_bounds__(256) void k_chain_clear(uint4 *p, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

constexpr int CHAIN_XS = 56;  // elements between the columns of the input buffer (48 used)

// NC ids per tile; hidden layers of 512 units (RT row tiles per wave), PD k-steps of weight fragments in
// flight.  ONE: the network has a single hidden layer.
template <int NC, bool ONE>
__global__ __launch_bounds__(512, 2) void k_chain(vf_fast_dev md, int ks, NoiseArgs na, ChainArgs ca) {
  constexpr int CT = NC / 32, RT = 2, PD = 4;
  constexpr int XS = CHAIN_XS;
  // the weights of the folded first layer's last four k-steps: in registers for good, where there are enough
  constexpr bool LATE = CT == 1;
  // of the k-steps from HELD0 on HELD in LDS, as many as there is room for
  constexpr int HELD0 = LATE ? 7 : 3, HELD = LATE ? 6 : 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t *act = reinterpret_cast<uint16_t *>(smem);             // [NC][ks] hidden activations
  uint16_t *xin = act + (size_t)NC * ks;                          // [NC][XS] rows 16..63 of the tile's candidates
  float *red = reinterpret_cast<float *>(xin + (size_t)NC * XS);  // [8][NC] partial output dots
  int32_t *okf = reinterpret_cast<int32_t *>(red + 8 * NC);       // [NC]
  float *auxs = reinterpret_cast<float *>(okf + NC);              // [wl_off] biases
  uint32_t *wls = reinterpret_cast<uint32_t *>(auxs + ((md.wl_off + 3) & ~3));  // [dims[NH] / 2] output vector, bfloat16 pairs
  uint4 *heldw = reinterpret_cast<uint4 *>(wls + md.dims[1] / 2);  // [8][HELD][RT][64] weights of the folded first layer
  __shared__ ChainShared sh;
  __shared__ uint32_t digs[NC];  // the next tile's ids, taken apart
  __shared__ int shut;           // none of them can be valid

  int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NH = md.L - 1;
  const int p = (int)blockIdx.x % ca.nprob, member = (int)blockIdx.x / ca.nprob;
  const int S = ca.t.S, ntiles = ca.ntiles;
  const bool wide = md.dims[0] == 256;
  const size_t row = (size_t)p * S;
  unsigned long long *const slots = ca.slots + row * ntiles;
  unsigned int *const claims = ca.claims + (size_t)p * (S + 1);

  // ---- once per workgroup
  unsigned int c_next = NO_CLAIM;  // (the claimer's) a tile of the next decision
  for (int i = tid; i < (int)md.wl_off; i += 512) auxs[i] = md.aux[i];
  for (int i = tid; i < md.dims[NH] / 2; i += 512) wls[i] = pack_bf16(md.aux[md.wl_off + 2 * i], md.aux[md.wl_off + 2 * i + 1]);
  const __amdgpu_buffer_rsrc_t ws = stream_rsrc(md.w_stream + (size_t)w * md.wave_stride);
  const __amdgpu_buffer_rsrc_t wf = stream_rsrc(md.w_full + (size_t)w * md.wave_stride_full);
  int wstep = PD;
  uint4 ring[PD][RT];
#pragma unroll
  for (int j = 0; j < PD; ++j)
#pragma unroll
    for (int r = 0; r < RT; ++r) ring[j][r] = stream_load(ws, 16 * lane, j * RT + r);
  chain_begin(sh, ca, row, member, tid);

  int stage = ca.first - 1;  // the open decision's (none yet)
  int t = ntiles;
  int cur = 1;               // pks[cur]: its context
  bool ready = false;        // digs and shut are tile t's
  int32_t pre = 0;           // what a thread has fetched for the next context
  floatx16 fa[RT];           // the folded first layer
  // the weights of k-steps 3..6 of the folded layer: in registers for good, where there are enough
  uint4 late[LATE ? 4 : 1][RT];
  if constexpr (LATE) {
#pragma unroll
    for (int i = 0; i < 4; ++i) fold_load<RT>(late[i], wf, wide || i == 0 ? 3 + i : 0, lane);
    // (arrived: a use must not wait for what was sent for or stored since)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < RT; ++r)
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(late[i][r].x), "+v"(late[i][r].y), "+v"(late[i][r].z), "+v"(late[i][r].w));
  }
  // those of HELD others in LDS
#pragma unroll
  for (int i = 0; i < HELD; ++i)
    if (wide || HELD0 + i == 3) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
        heldw[((w * HELD + i) * RT + r) * 64 + lane] = stream_load(wf, 16 * lane, (HELD0 + i) * RT + r);
    }
  // by one wave: the digits of a tile's ids; whether none of them is valid
  auto take_apart = [&](int tile, const vf_space &sp) __attribute__((always_inline)) {
    const int64_t id = (int64_t)tile * NC + lane;
    if (lane < NC) digs[lane] = pack_digits(digits_small(sp, id < ca.M ? (uint32_t)id : 0u));
  };
  auto look_shut = [&](int tile, const DecPack &k) __attribute__((always_inline)) {
    const bool in = lane < NC && (int64_t)tile * NC + lane < ca.M;
    const unsigned long long m = __ballot(in && eval_digits<false>(k.d, k.sp, unpack_digits(digs[lane < NC ? lane : 0]), nullptr, nullptr));
    if (lane == 0) shut = m == 0ull;
  };
  for (;;) {
    // (what is worked out from the thread's number is worked out afresh: kept over the loop it would spill)
    asm volatile("" : "+v"(tid));
    lane = tid & 63;
    if (t < ntiles) {
      // ---- a tile of the open decision
      const DecPack &pk = sh.pks[cur];
      const int64_t n0 = (int64_t)t * NC, nend = n0 + NC < ca.M ? n0 + NC : ca.M;
      if (!ready) {
        if (w == 4) {
          take_apart(t, pk.sp);
          look_shut(t, pk);
        }
        __syncthreads();
      }
      ready = false;
      const bool closed = shut != 0;
      float dot[CT];
      if (!closed) {
        // wave w < 6 produces eight input rows of every candidate (as in the other scorers: rows 16..55, and of
        // 56..63 the candidate's own row 59)
        if (lane < NC && w < 6) {
          const bool inb = n0 + lane < ca.M;
          const Digits dg = unpack_digits(digs[lane]);
          int32_t core[64];
          auto put8 = [&](const int32_t *v) __attribute__((always_inline)) {
            uint4 o;
            o.x = pack_bf16(plog2_dev(v[0]), plog2_dev(v[1]));
            o.y = pack_bf16(plog2_dev(v[2]), plog2_dev(v[3]));
            o.z = pack_bf16(plog2_dev(v[4]), plog2_dev(v[5]));
            o.w = pack_bf16(plog2_dev(v[6]), plog2_dev(v[7]));
            if (!inb) o = make_uint4(0u, 0u, 0u, 0u);
            *reinterpret_cast<uint4 *>(xin + (size_t)lane * XS + 8 * w) = o;
          };
          if (w == 0) {
            const bool valid = eval_digits<true>(pk.d, pk.sp, dg, &sh.tabs, core);
            okf[lane] = inb && valid;
            put8(core + 16);
          } else if (w == 1) {
            eval_digits<true>(pk.d, pk.sp, dg, &sh.tabs, core);
            put8(core + 24);
          } else if (w == 2) {
            eval_digits<true>(pk.d, pk.sp, dg, &sh.tabs, core);
            put8(core + 32);
          } else if (w == 3) {
            eval_digits<true>(pk.d, pk.sp, dg, &sh.tabs, core);
            put8(core + 40);
          } else if (w == 4) {
            eval_digits<true>(pk.d, pk.sp, dg, &sh.tabs, core);
            put8(core + 48);
          } else {
            eval_digits<true>(pk.d, pk.sp, dg, &sh.tabs, core);
            *reinterpret_cast<uint4 *>(xin + (size_t)lane * XS + 40) =
                make_uint4(0u, inb ? pack_bf16(0.0f, plog2_dev(core[59])) : 0u, 0u, 0u);
          }
        }
        __syncthreads();  // the inputs are complete
        const uint16_t *const bx = xin + (size_t)(lane & 31) * XS + 8 * (lane >> 5);
        const uint16_t *const ba = act + (size_t)(lane & 31) * ks + 8 * (lane >> 5);
        const int voff = 16 * lane;
        floatx16 acc[RT][CT], bv[RT];
        contract_own_rows<RT, CT, PD, ONE>(acc, fa, ring, ws, voff, bx, 32 * XS);
        wstep = VF_K0_OWN + PD;
        auto write_back = [&]() __attribute__((always_inline)) {
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            const int m0 = (w + r * 8) * 32 + 8 * (lane >> 5);
#pragma unroll
            for (int g = 0; g < 4; g += 2) {
#pragma unroll
              for (int c = 0; c < CT; ++c) {
                uint32_t x0 = relu_bf16x2(pack_bf16(acc[r][c][4 * g + 0], acc[r][c][4 * g + 1]));
                uint32_t x1 = relu_bf16x2(pack_bf16(acc[r][c][4 * g + 2], acc[r][c][4 * g + 3]));
                uint32_t y0 = relu_bf16x2(pack_bf16(acc[r][c][4 * g + 4], acc[r][c][4 * g + 5]));
                uint32_t y1 = relu_bf16x2(pack_bf16(acc[r][c][4 * g + 6], acc[r][c][4 * g + 7]));
                swap_halves(x0, y0);
                swap_halves(x1, y1);
                *reinterpret_cast<uint4 *>(act + (size_t)(c * 32 + (lane & 31)) * ks + m0 + 8 * g) = make_uint4(x0, x1, y0, y1);
              }
            }
          }
        };
        if constexpr (!ONE) {
          // (nobody reads the activations of the tile before any more)
          write_back();
          __syncthreads();
          for (int l = 1;; ++l) {
            load_bias<RT>(bv, auxs + md.bias_off[l], w, lane);
            contract_layer<RT, CT, PD, VF_K0_OWN % PD>(acc, bv, ring, ws, wstep, voff, l == NH - 1, md.dims[l] / 16, ba, 32 * ks);
            if (l == NH - 1) break;
            __syncthreads();  // every wave has read the layer's input
            write_back();
            __syncthreads();
          }
        }
        output_dots_mfma<RT, CT>(acc, dot, [&](int u) { return wls[u >> 1]; }, w, lane);
#pragma unroll
        for (int c = 0; c < CT; ++c)
          if (lane < 32) red[w * NC + c * 32 + lane] = dot[c];
      }
      __syncthreads();
      if (w == 0) {
        float v = __builtin_inff();
        int32_t c = -1;
        if (!closed) {
          if (lane < NC) {
            float s = auxs[md.bias_off[md.L - 1]];
#pragma unroll
            for (int g = 0; g < 8; ++g) s += red[g * NC + lane];
            const int32_t id = (int32_t)(n0 + lane);
            if (na.eps != 0.0f) {
              na.stage = stage;
              s = add_noise(na, s, p, id);
            }
            if (okf[lane] != 0 && s < v) { v = s; c = (int32_t)digs[lane]; }
          }
          wave_min(v, c);
          if (ca.stat) {
            const int nvalid = __popcll(__ballot(lane < NC && okf[lane < NC ? lane : 0] != 0));
            if (lane == 0) {
              atomicAdd(&ca.stat[0], (unsigned long long)(nend - n0));
              atomicAdd(&ca.stat[1], (unsigned long long)nvalid);
            }
          }
        }
        if (lane == 0)
          __hip_atomic_store(&slots[(size_t)stage * ntiles + t], word_of(v, c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      t = ntiles;
    }

    // ---- no tile left to claim: what is known of the next stage
    const int next = stage + 1;
    DecPack &nk = sh.pks[cur ^ 1];
    const DecPack &pk = sh.pks[cur];
    const bool opens = next < S;         // (behind the last stage there is no context to make)
    const bool decides = next <= ca.last;
    if (tid == CLAIMER && decides && c_next == NO_CLAIM) c_next = atomicAdd(&claims[next], 1u);
    uint4 ends[LATE ? 4 : 1][RT];  // k-steps 0 and 13..15 of the folded layer
    if (decides) {
#pragma unroll
      for (int i = 0; i < (LATE ? 4 : 1); ++i) fold_load<RT>(ends[i], wf, i == 0 || !wide ? 0 : 12 + i, lane);
    }
    chain_rows(sh, nk, pk, ca, p, row, stage, c_next, pre, tid, lane, w);

    if (stage >= ca.first) {
      // ---- the open decision's minima
      if (w == 7) chain_poll(sh, ca, slots, claims, ntiles, stage, c_next, lane);
      __syncthreads();
      if (sh.missing >= 0) {
        t = __builtin_amdgcn_readfirstlane(sh.missing);
        __syncthreads();  // (before the word is written again)
        continue;
      }
      // (the weights have arrived: waited for here, they are not waited for behind the stores below)
      if (decides) {
#pragma unroll
        for (int i = 0; i < (LATE ? 4 : 1); ++i)
#pragma unroll
          for (int r = 0; r < RT; ++r) asm volatile("" : "+v"(ends[i][r].x), "+v"(ends[i][r].y), "+v"(ends[i][r].z), "+v"(ends[i][r].w));
      }
      // ---- s_i := the winner: its rows, a share each by threads of four waves; the ids of the next tile
      winner_rows(sh, pk, sh.win_c, lane, w);
      if (w == 4 && decides && sh.claim < ntiles) take_apart(sh.claim, pk.sp);
      __syncthreads();
      chain_tables(sh, pk, ca, p, row, stage, member, tid);
    }
    if (!opens) break;

    // ---- the next decision's context: the shared rows, so that the folded layer can begin
    next_shared_rows(sh, nk, stage >= ca.first, stage, tid);
    __syncthreads();
    if (!decides) {
      // (a schedule in pieces: the context is left for the call that goes on)
      if (tid == 0) next_derive(sh, nk, stage >= ca.first, stage);
      __syncthreads();
      if (member == 0)
        for (int i = tid; i < VF_DECPACK_DWORDS; i += 512)
          ca.decpack[(size_t)p * VF_DECPACK_DWORDS + i] = reinterpret_cast<const uint32_t *>(&nk)[i];
      break;
    }
    t = __builtin_amdgcn_readfirstlane(sh.claim);
    if (stage < ca.first && w == 4 && t < ntiles) take_apart(t, nk.sp);
    ready = t < ntiles;
    c_next = NO_CLAIM;
    // the folded layer; first by all waves but wave 0, which derives the rest of the context meanwhile, then by
    // wave 0, while the others make the quotient tables of it
    for (int ph = 0; ph < 2; ++ph) {
      if ((ph == 0) == (w != 0)) {
        fold_zero<RT>(fa);
        fold_step<RT>(fa, ends[0], nk.stat, 0, lane);
        // (one straight run of products: with a condition in front of each they would not be read ahead)
        auto products = [&](auto from, auto to) __attribute__((always_inline)) {
#pragma unroll
          for (int i = decltype(from)::value; i < decltype(to)::value; ++i) {
            uint4 a[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r)
              a[r] = LATE && i >= 13                     ? ends[LATE && i >= 13 ? i - 12 : 0][r]
                     : LATE && i < 7                     ? late[LATE && i < 7 ? i - 3 : 0][r]
                     : i >= HELD0 && i < HELD0 + HELD ? heldw[((w * HELD + i - HELD0) * RT + r) * 64 + lane]
                                                       : stream_load(wf, 16 * lane, i * RT + r);
            fold_step<RT>(fa, a, nk.stat, i, lane);
          }
        };
        if (wide) products(std::integral_constant<int, 3>{}, std::integral_constant<int, 16>{});
        else products(std::integral_constant<int, 3>{}, std::integral_constant<int, 4>{});
        floatx16 bv[RT];
        load_bias<RT>(bv, auxs + md.bias_off[0], w, lane);
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int q = 0; q < 16; ++q) fa[r][q] = bv[r][q] + fa[r][q];
      } else if (ph == 0) {
        if (lane == 0) next_derive(sh, nk, stage >= ca.first, stage);
      } else {
        fill_evaltabs(sh.tabs, nk.d, nk.sp, 64);
        if (w == 4 && t < ntiles) look_shut(t, nk);
      }
      __syncthreads();
    }
    cur ^= 1;
    stage = next;
    if (w == 6) pre = chain_prefetch(ca, row, stage, lane);
  }
  chain_leave(sh, ca, slots, claims, p, ntiles, tid);
}

}  // namespace

// The words of a launch with `units` 16-byte units, zero; VF_ENOMEM without memory for them.
int vfk_chain_words(vf_ctx *c, size_t units) {
  if (units <= c->chain_units) return VF_OK;
  // (not while the stream is captured: they would be cleared when the graph runs, and a call may come before)
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(c->stream, &capture) != hipSuccess) (void)hipGetLastError();
  if (capture != hipStreamCaptureStatusNone) return VF_ENOMEM;
  if (c->d_chain) { VF_HIP(c, hipStreamSynchronize(c->stream)); (void)hipFree(c->d_chain); c->d_chain = nullptr; }
  c->chain_units = 0;
  if (hipMalloc((void **)&c->d_chain, units * 16) != hipSuccess) { (void)hipGetLastError(); c->d_chain = nullptr; return VF_ENOMEM; }
  hipLaunchKernelGGL(k_chain_clear, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, c->stream,
                     reinterpret_cast<uint4 *>(c->d_chain), units);
  VF_HIP(c, hipGetLastError());
  c->chain_units = units;
  return VF_OK;
}

typedef void (*chain_kernel)(vf_fast_dev, int, NoiseArgs, ChainArgs);

// The launch for a context's model and batch: kernel, candidates per tile, dynamic LDS; null if there is none.
static chain_kernel chain_shape(const vf_ctx *c, vf_fast_dev *fd, int *ks, int *NC, size_t *smem) {
  if (!vfk_can_fuse_step(c) || c->M < 1) return nullptr;
  vfk_fast_dev(c, true, fd, ks, nullptr);
  if (fd->k0 != VF_K0_OWN || !fd->w_full) return nullptr;
  int ncu = 256, lds_max = 0;
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device);
  (void)hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, c->device);
  if (c->pm.fast_rt != 2 || (c->M + 63) / 64 * c->B > ncu) return nullptr;
  const bool one = fd->L == 2;
  *NC = (c->M + 31) / 32 * c->B <= ncu ? 32 : 64;
  *smem = (size_t)*NC * *ks * 2 + (size_t)*NC * CHAIN_XS * 2 + (size_t)9 * *NC * 4 + (size_t)((fd->wl_off + 3) & ~3) * 4 +
          (size_t)fd->dims[1] * 2 +
          (size_t)(*NC == 32 ? 6 : 4) * 16 * 1024;  // (HELD k-steps of weights)
  chain_kernel kern;
  if (*NC == 32) kern = one ? k_chain<32, true> : k_chain<32, false>;
  else kern = one ? k_chain<64, true> : k_chain<64, false>;
  hipFuncAttributes attr;
  if (hipFuncGetAttributes(&attr, (const void *)kern) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
  return *smem + attr.sharedSizeBytes <= (size_t)lds_max ? kern : nullptr;
}

bool vfk_can_chain(const vf_ctx *c) {
  vf_fast_dev fd;
  int ks = 0, NC = 0;
  size_t smem = 0;
  return chain_shape(c, &fd, &ks, &NC, &smem) != nullptr;
}

int vfk_greedy_chain(vf_ctx *c, int first, int last, int32_t *out_states, int32_t *out_cids, float *out_vals) {
  vf_fast_dev fd;
  int ks = 0, NC = 0;
  size_t smem = 0;
  const chain_kernel kern = chain_shape(c, &fd, &ks, &NC, &smem);
  if (!kern || first > last) return VF_ESTATE;
  ChainArgs ca;
  const int rc = chain_args(c, first, last, (int)((c->M + NC - 1) / NC), out_states, out_cids, out_vals, &ca);
  if (rc != VF_OK) return rc;
  NoiseArgs na;
  na.eps = c->noise_eps;
  na.k0 = (uint32_t)c->noise_seed; na.k1 = (uint32_t)(c->noise_seed >> 32);
  na.stage = first; na.first_rollout = c->noise_first;
  vf_prof_scope prof(c, VF_PROF_SCORE);
  VF_HIP(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  hipLaunchKernelGGL(kern, dim3((unsigned)(c->B * ca.ntiles)), dim3(512), smem, c->stream, fd, ks, na, ca);
  VF_HIP(c, hipGetLastError());
  c->dec_stage = last + 1 < c->S ? last + 1 : -1;
  return VF_OK;
}
