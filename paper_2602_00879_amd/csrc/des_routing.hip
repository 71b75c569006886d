// Routing half of the DES layer for gfx950, in ONE launch:
//   router scores G(x)                      (Background, definition of G)
//   coreset election  Phi                   (Alg. 1 stage 1; Eq. 5 / Alg. 2, Eq. 6 / Alg. 3)
//   constrained re-routing + gates          (Alg. 1 stage 2)
//   token permutation by expert, cnt_i      (Eq. 2)
//
// The paper fuses its selection into two kernels that add votes into a global
// vector with float atomics (Sec. 4.3).  Here the whole routing step is one
// kernel whose workgroups take one of three roles, chained through per-producer
// flags in device memory instead of kernel boundaries:
//   role R (one per 16x16 logits tile)  router GEMM tile, then flag[tile] = epoch
//   role S (one per sequence, or one    waits for the R flags, elects the coreset,
//           per group of its tokens)    re-routes, then flag[seq] = epoch
//   role P (one, merged into S if B==1) waits for the S flags, builds counts,
//                                       offsets, the slot table and the permutation
// A flag is a 64-bit word that a producer sets to the call's epoch (a host
// counter that never repeats), so the workspace needs no clearing, stale
// contents can never satisfy a wait, and no two workgroups ever write the same
// word (no atomic read-modify-write at all).  Waiting is safe because the launch
// is only used in this fused form when every workgroup fits on the chip at once
// (one 1024-thread workgroup per compute unit), so a producer can always run;
// every wait is also bounded and gives up, reporting n_unique = -1.
// Larger problems run the same three roles as three launches.
//
// Votes are accumulated without floating-point atomics: a 16-lane row of a
// wavefront owns one token, each lane owns a contiguous slice of the experts,
// votes stay in the owning lane's registers, and rows / waves are combined in a
// fixed order.  Every ranking compares order-preserving integer keys of the
// fp32 logits with ties to the lowest expert index.
#include <atomic>

#include "des_common.h"
#include "des_select.h"
#include "des_stream_gemm.h"

namespace des {

constexpr int kRtWaves = 16;
constexpr int kRtThreads = kRtWaves * kWave;  // 1024
constexpr int kMaxWaitIters = 1 << 22;        // bounded waits (~ seconds), then give up
int g_test_max_wait = 0;     // test hooks (des_test_hooks): a tiny wait bound, and a fused
int g_test_skip_router = 0;  // routing launch without its router tiles, so that a wait expires
int g_test_compute_units = -1;  // (des_test_compute_units) answer to the next question for their number

#ifdef DES_ROUTING_TIMESTAMPS  // development aid: 100 MHz timestamps into meta[16..]
#define DES_STAMP(a, i) do { if (threadIdx.x == 0 && (a).meta != nullptr) reinterpret_cast<long long*>((a).meta + 16)[i] = wall_clock64(); } while (0)
#else
#define DES_STAMP(a, i) do { } while (0)
#endif

struct RoutingArgs {
  // router
  const void* x;
  const void* w_router;
  const float* bias;
  float* logits;          // [B][N][M]
  // selection
  int32_t* coreset_idx;   // [B][cap]
  int32_t* coreset_size;  // [B]
  float* votes;           // [B][M] or null
  int32_t* k_seq_used;    // [B] or null
  int32_t* topk_idx;      // [B][N][K] or null (then stage 2 and permutation are skipped)
  float* topk_w;
  // permutation
  int32_t* expert_counts; // [M]
  int32_t* n_unique;      // [1]
  int32_t* offsets;       // [M+1]
  int4* slots;            // [n_slots] {expert, first sorted pair, pairs, 0}; expert -1 = unused
  int32_t* meta;          // [8]: [0] live experts, [1] routed pairs, [2] live units
  int32_t* units;         // [max units] slot | split << 16 | splits of the slot << 24
  int rows_shift;         // log2 of the token rows per unit (blocks of more than 32 tokens)
  int32_t* pair_tok;      // [T*K] token of each sorted pair
  int32_t* pos;           // [T*K] sorted position of pair (t*K+j), -1 = unused slot
  unsigned long long* flags;  // [n_tiles + 2*B*groups] epoch flags: router tiles, selector
                              // partials published, selectors done
  uint32_t* sel_part;         // [B*groups][3][kSelPartStride] per-group election partials
  unsigned long long epoch;
  int32_t* slot_of;       // [M] slot of each live expert, -1 otherwise
  int B, N, M, K, C, k_seq, mode, cap, D, n_slots;
  int groups;             // selector workgroups per sequence (each takes every groups-th pass)
  int k_route;            // experts per token in stage 2 (<= K)
  float skip_beta;        // > 0: cumulative-probability skipping of a token's weakest experts
  int sigmoid;            // router weights are sigmoid(logit) instead of softmax over M
  int vote_renorm;        // a token's K votes are divided by their sum
  int n_group;            // > 1: group-limited router over this many groups of experts
  int group_lanes;        // selector lanes per group (group size / 8)
  int topk_group;         // groups a token keeps
  int group_top2;         // group score: sum of the two best router weights (else the best logit)
  int vote_atomic;        // votes meet in floating-point LDS atomics (arrival order) instead of
                          // the fixed-order reduction
  int perm_parts;         // workgroups of the permutation (1, or more in a launch of its own)
  int tiles_m, tiles_t;   // router tiles along experts / tokens
  int max_wait;           // polls before a wait gives up
  const int32_t* prev_n_unique;  // the previous layer's n_unique (a stack), or null: a negative
                                 // value there is carried into this layer's n_unique
  int do_router, do_select, do_permute, use_flags, bf16;
  int solo;               // one router tile and one selector workgroup: it computes the tile itself
  int skip_router_tiles;  // test hook: the fused launch runs without its router tiles
  int small_perm;         // one selector workgroup, at most 32 tokens, no skipping: the permutation
                          // is built from per-expert token bitmaps recorded during stage 2
  int dense;              // dense short block (LayerForm): the launch ends with the election
                          // and the slot table of the coreset; stage 2 runs beside the gate/up
                          // projection, there is no permutation
  uint32_t* tokmask;      // [n_slots] cleared here for that stage 2
  uint16_t* xo;           // [D / 8][T][8] x in operand order (LayerForm), by the workgroups from x_first on, or null
  int x_first;
};

// ------------------------------------------------------------------ flags
// Two hand-off styles.  `fenced`: the data was written with ordinary stores, so
// a device-scope fence (an L2 write-back on this chip, ~1 us) precedes the flag
// and the waiter ends with one too.  Unfenced: the data itself is written and
// read with device-scope accesses (the logits), which reach the level all
// compute units share on their own, so the flag only has to follow them.
// A workgroup barrier does not wait for outstanding stores: every thread that
// stored data the flag stands for must have waited for its own stores
// (stores_done()) BEFORE the barrier that precedes the publishing thread's call.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void flag_publish(unsigned long long* f, unsigned long long epoch,
                                             bool fenced) {
  if (fenced) __threadfence();
  __hip_atomic_store(f, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Every thread polls a subset of the flags; returns false if a wait ran out.
__device__ __forceinline__ bool flags_wait(const unsigned long long* f, int n,
                                           unsigned long long epoch, bool fenced, int max_wait) {
  bool ok = true;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    int it = 0;
    // relaxed polls; the fence after the barrier below is the acquire
    while (__hip_atomic_load(f + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != epoch) {
      __builtin_amdgcn_s_sleep(4);
      if (++it > max_wait) { ok = false; break; }
    }
  }
  const int all = __syncthreads_and(ok ? 1 : 0);
  if (fenced) __threadfence();
  return all != 0;
}

// Four floats that other workgroups of this launch may have stored with device-scope stores, in one
// load with the same scope (sc1; the flags order it, it need not be atomic).  base + byte_off is 16-byte
// aligned.  The selection's lanes are 32 bytes apart, so every load takes as long as any, and 16 wavefronts
// queue up on one compute unit: with a load per float the routing of 32 tokens took 12.6 us, of 128 26.3
// (128 experts), of 32 on 256 experts 15.4; with two of four floats 11.8, 25.3 and 13.8.
__device__ __forceinline__ f32x4 load_device_quad(const float* base, uint32_t byte_off) {
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0x7fffffff, 0x00027000);
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, byte_off, 0, 16));
}

// ------------------------------------------------------------ role R: router
// experts [i0, i0+16) x tokens [t0, t0+16); wave w takes k-steps w, w+16, ...
// MFMA 16x16x32: lane l supplies row (l%16), reduction elements 8*(l/16)..+7;
// the accumulator of lane l holds column (l%16), rows 4*(l/16)..+3.  Both operands go through
// operand_write / operand_read (128 experts of width 2048, 32 tokens: routing 14.6 -> 12.5 us).
__device__ __forceinline__ void router_tile_bf16(const RoutingArgs& a, int tile_m, int tile_t,
                                                 char* lds /* [16][2 KB] */) {
  const int lane = threadIdx.x & 63;
  const int wave = uniform_int(threadIdx.x >> 6);  // (it guards matrix instructions, see stream_pipeline)
  const int T = a.B * a.N, D = a.D, M = a.M;
  const int i0 = tile_m * 16, t0 = tile_t * 16;
  const int r = lane & 15, kq = (lane & 3) * 8;
  const int ei = min(i0 + (lane >> 2), M - 1);  // clamped rows are computed and dropped
  const int ti = min(t0 + (lane >> 2), T - 1);
  // of this wavefront: the operands of a k-step, then its partial tile
  char* mine = lds + wave * (2 * kOperandBytes);
  const uint16_t* ap = static_cast<const uint16_t*>(a.w_router) + static_cast<size_t>(ei) * D + kq;
  const uint16_t* bp = static_cast<const uint16_t*>(a.x) + static_cast<size_t>(ti) * D + kq;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int nks = D / 32;
  // the bias of the expert this thread will finish (below), fetched now so that its
  // latency is not added after the reduction
  const int er_fin = threadIdx.x & 15;
  const float bias_fin = (threadIdx.x < 256 && a.bias && i0 + er_fin < M) ? a.bias[i0 + er_fin] : 0.f;
  // four k-steps per trip, all eight loads in flight before the first MFMA
  for (int ks = wave; ks < nks; ks += 4 * kRtWaves) {
    bf16x8 av[4], bv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = min(ks + u * kRtWaves, nks - 1);  // clamped steps are skipped below
      av[u] = *reinterpret_cast<const bf16x8*>(ap + k * 32);
      bv[u] = *reinterpret_cast<const bf16x8*>(bp + k * 32);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      turn_fence();
      operand_write(av[u], mine, lane);
      operand_write(bv[u], mine + kOperandBytes, lane);
      turn_fence();
      av[u] = operand_read(mine, lane);
      bv[u] = operand_read(mine + kOperandBytes, lane);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (ks + u * kRtWaves < nks)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[u], bv[u], acc, 0, 0, 0);
  }
  turn_fence();
  float* part = reinterpret_cast<float*>(lds);  // [16][512]
  *reinterpret_cast<f32x4*>(part + wave * 512 + r * 16 + 4 * (lane >> 4)) = acc;  // [token][expert]
  __syncthreads();
  if (threadIdx.x < 256) {
    const int er = er_fin, tc = threadIdx.x >> 4;
    float s = 0.f;
    const float bias_e = bias_fin;
#pragma unroll
    for (int w = 0; w < kRtWaves; ++w) s += part[w * 512 + tc * 16 + er];  // fixed order
    const int e = i0 + er, t = t0 + tc;
    if (e < M && t < T)  // device-scope store: the selector reads it without a fence
      __hip_atomic_store(a.logits + static_cast<size_t>(t) * M + e, s + bias_e, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  }
}

// fp32 inputs: wavefront w has expert w of the tile, lanes stride the reduction dimension with
// 16-byte loads, several tokens at a time so that their loads are in flight together: eight
// (one dot product after the other: routing of 30 tokens, 16 experts of width 1024, 28.0 us, so
// 20.6), fewer where fewer are left (one token as eight copies of it: 15.2 us, alone 12.1).
template <int TOK>
__device__ __forceinline__ void router_tokens_f32(const RoutingArgs& a, int e, int t0, int t1, float bias) {
  const int lane = threadIdx.x & 63, D = a.D;
  const float4* wp = reinterpret_cast<const float4*>(static_cast<const float*>(a.w_router) + static_cast<size_t>(e) * D);
  const float4* xp[TOK];
  float s[TOK];
#pragma unroll
  for (int i = 0; i < TOK; ++i) {
    xp[i] = reinterpret_cast<const float4*>(static_cast<const float*>(a.x) + static_cast<size_t>(min(t0 + i, t1 - 1)) * D);
    s[i] = 0.f;
  }
  for (int v = lane; v < D / 4; v += 64) {
    const float4 q4 = wp[v];
    float4 p4[TOK];
#pragma unroll
    for (int i = 0; i < TOK; ++i) p4[i] = xp[i][v];
#pragma unroll
    for (int i = 0; i < TOK; ++i) {
      s[i] = fmaf(p4[i].x, q4.x, s[i]);
      s[i] = fmaf(p4[i].y, q4.y, s[i]);
      s[i] = fmaf(p4[i].z, q4.z, s[i]);
      s[i] = fmaf(p4[i].w, q4.w, s[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < TOK; ++i) {
    const float sum = wave_sum_f32(s[i]);
    if (lane == 0 && t0 + i < t1)
      __hip_atomic_store(a.logits + static_cast<size_t>(t0 + i) * a.M + e, sum + bias, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  }
}
__device__ __forceinline__ void router_tile_f32(const RoutingArgs& a, int tile_m, int tile_t) {
  static_assert(kRtWaves == 16, "one wavefront per expert of the tile");
  const int e = tile_m * 16 + uniform_int(threadIdx.x >> 6);
  if (e >= a.M) return;  // uniform per wave; no barrier below
  const float bias = a.bias ? a.bias[e] : 0.f;
  const int t1 = min(tile_t * 16 + 16, a.B * a.N);
  for (int t = tile_t * 16; t < t1;) {
    const int left = t1 - t;
    if (left > 4) { router_tokens_f32<8>(a, e, t, t1, bias); t += 8; }
    else if (left > 2) { router_tokens_f32<4>(a, e, t, t1, bias); t += 4; }
    else if (left > 1) { router_tokens_f32<2>(a, e, t, t1, bias); t += 2; }
    else { router_tokens_f32<1>(a, e, t, t1, bias); t += 1; }
  }
}

// LDS carve-up of the selection (bytes).  MP = padded expert count = 8 * LPT.
template <int LPT>
struct SelLds {
  static constexpr int MP = kEpl * LPT;
  static constexpr int sorted = 0;                               // u32 [16 waves][8][64 lanes]
  static constexpr int vpart = sorted + 4 * kRtWaves * kEpl * 64; // float [16 waves][MP]
  static constexpr int level = vpart + 4 * kRtWaves * MP;        // int [MP]
  static constexpr int cnt1 = level + 4 * MP;                    // int [MP]
  static constexpr int key = cnt1 + 4 * MP;                      // u32 [MP]
  static constexpr int rank = key + 4 * MP;                      // int [MP]
  static constexpr int core = rank + 4 * MP;                     // int [MP]
  static constexpr int hist = core + 4 * MP;                     // int [36]
  static constexpr int mask = hist + 4 * 36;                     // u32 [MP] tokens routed to an expert (T <= 32)
  static constexpr int vsum = mask + 4 * MP;                     // float [MP] the votes, all waves added
  static constexpr int off = vsum + 4 * MP;                      // int [MP + 1] first pair of an expert
  static constexpr int liv = off + 4 * (MP + 1);                 // int [MP + 1] live experts before it
  static constexpr int total = liv + 4 * (MP + 1);
};

// ------------------------------------------------------- role S: selection
// `dry` runs the same instructions on whatever the logits buffer holds and
// stores nothing to global memory: the selector workgroup uses it to pull its
// code into the instruction cache while it waits for the router tiles (every
// index below derives from lane and slot numbers, never from the data read).
// EXT = the variants few callers use (group-limited router, votes added with
// floating-point atomics) are compiled in; the plain instantiation leaves them
// out, so the common path pays nothing for them.
template <int LPT, bool EXT>
__device__ bool select_sequence(const RoutingArgs& a, int b, int g, char* smem, bool dry,
                                bool wait_router) {
  using L = SelLds<LPT>;
  constexpr int MP = L::MP;
  constexpr int RPW = 64 / LPT;          // rows (tokens) per wave
  constexpr int TPP = kRtWaves * RPW;    // tokens per pass
  constexpr int NW = (32 + LPT - 1) / LPT;  // gate slots a lane keeps (K <= 32)
  uint32_t* s_sorted = reinterpret_cast<uint32_t*>(smem + L::sorted);
  float* s_vpart = reinterpret_cast<float*>(smem + L::vpart);
  int* s_level = reinterpret_cast<int*>(smem + L::level);
  int* s_cnt1 = reinterpret_cast<int*>(smem + L::cnt1);
  uint32_t* s_key = reinterpret_cast<uint32_t*>(smem + L::key);
  int* s_rank = reinterpret_cast<int*>(smem + L::rank);
  int* s_core = reinterpret_cast<int*>(smem + L::core);
  int* s_hist = reinterpret_cast<int*>(smem + L::hist);  // [0..32] histogram, [33] k used, [34] size
  uint32_t* s_mask = reinterpret_cast<uint32_t*>(smem + L::mask);
  float* s_vsum = reinterpret_cast<float*>(smem + L::vsum);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane / LPT, rl = lane % LPT;
  const int slot = wave * RPW + row;  // fill a wave's rows first: idle waves issue nothing
  const int N = a.N, M = a.M, K = a.K;
  const float* Lg = a.logits + static_cast<size_t>(b) * N * M;
  uint32_t* my_sorted = s_sorted + wave * (kEpl * 64) + lane;  // [s * 64]
  const int G = a.groups;
  const bool single_pass = N <= G * TPP;  // this workgroup sees each of its tokens once
  const bool quads = M % 4 == 0 && (reinterpret_cast<size_t>(a.logits) & 15) == 0;  // rows of whole, aligned fours

  for (int e = threadIdx.x; e < MP; e += kRtThreads) {
    s_level[e] = K;
    s_cnt1[e] = 0;
    s_rank[e] = 0;
    s_key[e] = 0u;
    s_core[e] = (a.mode == DES_VANILLA && e < M) ? 1 : 0;
    s_vpart[e] = 0.f;  // the accumulator of the atomic vote variant
    s_mask[e] = 0u;
  }
  if (threadIdx.x < 36) s_hist[threadIdx.x] = 0;
  // the LDS set-up above does not need the logits: only now wait for the router
  // tiles (the wait ends with a barrier of its own)
  if (wait_router) {
    if (!flags_wait(a.flags, a.tiles_m * a.tiles_t, a.epoch, false, a.max_wait)) return false;
  } else {
    __syncthreads();
  }
  DES_STAMP(a, 14);

  uint32_t sidx = 0;     // packed original slots of the sorted positions
  uint32_t nvalid = 0;   // sorted positions [0, nvalid) hold real experts

  // Loads token n's logits, sorts this lane's 8 keys into LDS, returns the
  // unsorted values (for the softmax).
  auto load_sort = [&](int n, float (&val)[kEpl], uint32_t (&key)[kEpl]) {
    const bool live = n < N;
    const float* rowp = Lg + static_cast<size_t>(live ? n : 0) * M;
    nvalid = 0;
    if (quads) {
#pragma unroll
      for (int j = 0; j < kEpl; j += 4) {
        const int idx = rl * kEpl + j;
        // (the row once more: named or left out, 256 experts need scratch and routing takes 2 % longer)
        const f32x4 v = live && idx < M
                            ? load_device_quad(Lg, static_cast<uint32_t>((live ? n : 0) * M + idx) * 4u)
                            : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 4; ++q) val[j + q] = v[q];
      }
    } else {
#pragma unroll
      for (int j = 0; j < kEpl; ++j) {
        const int idx = rl * kEpl + j;
        val[j] = live && idx < M ? __hip_atomic_load(rowp + idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.f;
      }
    }
#pragma unroll
    for (int j = 0; j < kEpl; ++j) {
      const bool ok = live && rl * kEpl + j < M;
      key[j] = ok ? order_key(val[j]) : 0u;
      nvalid += ok ? 1u : 0u;
    }
    uint32_t sk[kEpl];
#pragma unroll
    for (int j = 0; j < kEpl; ++j) sk[j] = key[j];
    sort8_desc(sk, sidx);
#pragma unroll
    for (int j = 0; j < kEpl; ++j) my_sorted[j * 64] = sk[j];
    if (EXT && a.n_group > 1) {
      // Group-limited router (a sigma of Sec. 4.1): a group is GL adjacent lanes
      // of the row.  Its two best keys are merged from the lanes' sorted heads,
      // its score is ranked against the other groups' (ties to the lowest group),
      // and the lanes of a group that is not kept offer no candidate from here on.
      const int GL = a.group_lanes, rowbase = lane - rl;
      const int gidx = rl / GL, gsrc = min(gidx, a.n_group - 1);  // padding lanes read a real group
      uint32_t b1 = 0u, b2 = 0u;
      for (int i = 0; i < GL; ++i) {
        const int src = rowbase + gsrc * GL + i;
        const uint32_t k0 = static_cast<uint32_t>(__shfl(static_cast<int>(sk[0]), src));
        const uint32_t k1 = static_cast<uint32_t>(__shfl(static_cast<int>(sk[1]), src));
        if (k0 > b1) { b2 = max(b1, k1); b1 = k0; } else { b2 = max(b2, k0); }
      }
      uint32_t gs = b1;  // "max": the best logit's key, an exact integer comparison
      if (a.group_top2) {
        // sum of the two best router weights, fp32; positive floats order like their
        // bit patterns.  The softmax denominator is the same for every group of a
        // token, so the numerators suffice.
        const float mx = a.sigmoid ? 0.f : key_to_f32(row_max_u32<LPT>(sk[0]));
        const float s1 = !b1 ? 0.f : a.sigmoid ? sigmoid_f(key_to_f32(b1)) : exp_neg(key_to_f32(b1) - mx);
        const float s2 = !b2 ? 0.f : a.sigmoid ? sigmoid_f(key_to_f32(b2)) : exp_neg(key_to_f32(b2) - mx);
        gs = __float_as_uint(s1 + s2);
      }
      int grank = 0;
      for (int j = 0; j < a.n_group; ++j) {
        const uint32_t o = static_cast<uint32_t>(__shfl(static_cast<int>(gs), rowbase + j * GL));
        grank += (o > gs || (o == gs && j < gidx)) ? 1 : 0;
      }
      if (gidx >= a.n_group || grank >= a.topk_group) nvalid = 0;
    }
  };

  // ---------------------------------------------------------- stage 1: Phi
  if (a.mode != DES_VANILLA) {
    const bool vote = a.mode == DES_VOTE;
    const int kk = (!vote && a.k_seq > 0) ? a.k_seq : K;
    float vacc[kEpl];
#pragma unroll
    for (int j = 0; j < kEpl; ++j) vacc[j] = 0.f;

    for (int n0 = g * TPP; n0 + wave * RPW < N; n0 += G * TPP) {  // fixed token order per row
      float val[kEpl], p[kEpl];
      uint32_t key[kEpl];
      load_sort(n0 + slot, val, key);
      DES_STAMP(a, 15);
      if (vote && a.sigmoid) {  // router weights of a sigmoid router
#pragma unroll
        for (int j = 0; j < kEpl; ++j) p[j] = key[j] ? sigmoid_f(val[j]) : 0.f;
      } else if (vote) {  // softmax over all M experts (Sec. 4.3), fp32
        const float mx = key_to_f32(row_max_u32<LPT>(my_sorted[0]));
        float se = 0.f;
#pragma unroll
        for (int j = 0; j < kEpl; ++j) {
          p[j] = key[j] ? exp_neg(val[j] - mx) : 0.f;
          se += p[j];
        }
        const float den = row_sum_f32<LPT>(se);
        const float inv = den > 0.f ? 1.0f / den : 0.f;
#pragma unroll
        for (int j = 0; j < kEpl; ++j) p[j] *= inv;
      }
      DES_STAMP(a, 16);
      Head hd;
      head_set(hd, (1u << nvalid) - 1u, my_sorted);
      uint32_t taken = 0;  // original slots this token nominated
      for (int it = 0; it < kk; ++it) {  // Mask(I, K): the token's own top-K
        bool mine;
        row_draw<LPT>(hd, mine);
        if (mine) {
          const uint32_t j = (sidx >> (3 * hd.h)) & 7u;
          taken |= 1u << j;
          const int e = rl * kEpl + static_cast<int>(j);
          if (vote) {
            s_level[e] = 0;  // "nominated": only < K matters for votes
          } else {
            atomicMin(&s_level[e], it);
            if (it == 0) atomicAdd(&s_cnt1[e], 1);
          }
          head_set(hd, hd.mask & (hd.mask - 1u), my_sorted);
        }
      }
      if (vote) {
        float scale = 1.0f;
        if (a.vote_renorm) {  // the token's K weights sum to one
          float mine_sum = 0.f;
#pragma unroll
          for (int j = 0; j < kEpl; ++j) mine_sum += ((taken >> j) & 1u) ? p[j] : 0.f;
          const float tot = row_sum_f32<LPT>(mine_sum);
          scale = tot > 0.f ? 1.0f / tot : 0.f;
        }
        if (EXT && a.vote_atomic) {
          // the variant Sec. 4.3 describes: every vote is an atomic add into the
          // shared vector, in whatever order the lanes arrive
#pragma unroll
          for (int j = 0; j < kEpl; ++j)
            if ((taken >> j) & 1u) atomicAdd(&s_vpart[rl * kEpl + j], p[j] * scale);
        } else {
#pragma unroll
          for (int j = 0; j < kEpl; ++j) vacc[j] += ((taken >> j) & 1u) ? p[j] * scale : 0.f;  // Eq. 6
        }
      }
    }
    DES_STAMP(a, 2);
    if (vote && !(EXT && a.vote_atomic)) {
      // rows of a wave in a fixed pairwise order, then waves in order
#pragma unroll
      for (int j = 0; j < kEpl; ++j) {
        float v = vacc[j];
        if (RPW >= 2) v += __shfl_xor(v, LPT);
        if (RPW >= 4) v += __shfl_xor(v, 2 * LPT);
        if (RPW >= 8) v += __shfl_xor(v, 4 * LPT);
        if (RPW >= 16) v += __shfl_xor(v, 8 * LPT);
        if (row == 0) s_vpart[wave * MP + rl * kEpl + j] = v;
      }
    }
    __syncthreads();
    DES_STAMP(a, 11);

    // this workgroup's votes: waves in order (into an array of their own, so that no
    // barrier is needed between reading the partials and writing the sums)
    for (int e = threadIdx.x; e < MP; e += kRtThreads) {
      float v = 0.f;
      if (vote && !(EXT && a.vote_atomic)) {
#pragma unroll
        for (int w = 0; w < kRtWaves; ++w) v += s_vpart[w * MP + e];
      } else if (vote) {
        v = s_vpart[e];
      }
      s_vsum[e] = v;
    }
    if (G > 1) __syncthreads();
    if (G > 1) {
      // The sequence's tokens are spread over G workgroups: each publishes what
      // its tokens contributed (votes, best nomination rank, top-1 nominations),
      // waits for the others and combines all G records in group order, so every
      // workgroup of the sequence elects the same coreset from the same numbers.
      // The records travel with device-scope accesses, like the logits.
      uint32_t* mine = a.sel_part + static_cast<size_t>(b * G + g) * 3 * kSelPartStride;
      for (int e = threadIdx.x; e < MP; e += kRtThreads) {
        __hip_atomic_store(mine + e, __float_as_uint(vote ? s_vsum[e] : 0.f), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(mine + kSelPartStride + e, static_cast<uint32_t>(s_level[e]),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(mine + 2 * kSelPartStride + e, static_cast<uint32_t>(s_cnt1[e]),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      stores_done();
      __syncthreads();
      unsigned long long* pf = a.flags + a.tiles_m * a.tiles_t + b * G;
      if (threadIdx.x == 0) flag_publish(pf + g, a.epoch, false);
      if (!flags_wait(pf, G, a.epoch, false, a.max_wait)) return false;
      for (int e = threadIdx.x; e < MP; e += kRtThreads) {
        float v = 0.f;
        int lvl = K, c1 = 0;
        for (int gg = 0; gg < G; ++gg) {
          const uint32_t* rec = a.sel_part + static_cast<size_t>(b * G + gg) * 3 * kSelPartStride;
          v += __uint_as_float(__hip_atomic_load(rec + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
          lvl = min(lvl, static_cast<int>(__hip_atomic_load(rec + kSelPartStride + e, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT)));
          c1 += static_cast<int>(__hip_atomic_load(rec + 2 * kSelPartStride + e, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT));
        }
        s_vsum[e] = v;
        s_level[e] = lvl;
        s_cnt1[e] = c1;
      }
      __syncthreads();
    }

    // (without an exchange every thread reads back only the s_vsum entry it wrote itself)
    if (vote) {
      for (int e = threadIdx.x; e < MP; e += kRtThreads) {
        const float v = s_vsum[e];
        const bool nominated = e < M && s_level[e] < K;
        s_key[e] = nominated ? order_key(v) : 0u;
        if (a.votes && e < M && !dry && g == 0) a.votes[static_cast<size_t>(b) * M + e] = v;
      }
      if (threadIdx.x == 0) s_hist[33] = 0;
    } else if (a.k_seq > 0) {  // Eq. 5 with the caller's k
      for (int e = threadIdx.x; e < MP; e += kRtThreads) s_core[e] = s_level[e] < a.k_seq;
      if (threadIdx.x == 0) s_hist[33] = a.k_seq;
    } else {  // largest k' whose union fits in C
      for (int e = threadIdx.x; e < M; e += kRtThreads)
        if (s_level[e] < K) atomicAdd(&s_hist[s_level[e]], 1);
      __syncthreads();
      if (threadIdx.x == 0) {
        int size = 0, ku = 0;
        for (int k1 = 1; k1 <= K; ++k1) {
          size += s_hist[k1 - 1];
          if (size <= a.C) ku = k1; else break;
        }
        s_hist[33] = ku;
      }
      __syncthreads();
      const int ku = s_hist[33];
      for (int e = threadIdx.x; e < MP; e += kRtThreads) {
        if (ku > 0) s_core[e] = s_level[e] < ku;
        else s_key[e] = (s_level[e] == 0) ? static_cast<uint32_t>(s_cnt1[e]) : 0u;
      }
    }
    __syncthreads();
    DES_STAMP(a, 12);

    if (vote || s_hist[33] == 0) {  // top-C by key, ties to the lowest index
      // rank[e] = #{j : key[j] beats key[e]}; the j range is split over the
      // threads that share an expert, partial counts meet in an integer LDS add
      constexpr int P = kRtThreads / MP;
      constexpr int CH = MP / P;  // keys per thread: a compile-time count (padding keys are 0
                                  // and never beat a candidate), so the reads batch up
      for (int t = threadIdx.x; t < MP * P; t += kRtThreads) {
        const int e = t % MP, part = t / MP;
        const uint32_t ke = s_key[e];
        if (ke == 0u) continue;
        const int j0 = part * CH;
        // key j beats key e if it is larger, or equal with j < e: kj >= ke for j < e,
        // kj >= ke + 1 for j >= e (a candidate's key is never the largest integer).
        // A chunk that lies wholly on one side of e needs one threshold.
        const int d = e - j0;
        int rank = 0;
        if (d <= 0 || d >= CH) {
          const uint32_t thr = ke + (d <= 0 ? 1u : 0u);
#pragma unroll
          for (int jj = 0; jj < CH; ++jj) rank += s_key[j0 + jj] >= thr ? 1 : 0;
        } else {
#pragma unroll
          for (int jj = 0; jj < CH; ++jj) rank += s_key[j0 + jj] >= ke + (jj >= d ? 1u : 0u) ? 1 : 0;
        }
        if (rank) atomicAdd(&s_rank[e], rank);
      }
    }
    __syncthreads();
  }

  DES_STAMP(a, 3);
  // ------------------------------------- coreset as an ascending index list
  // (where the election ranked keys, membership = "rank below C": the first wavefront
  // derives it here and records it for stage 2, which saves a pass and a barrier)
  const bool from_rank = a.mode != DES_VANILLA && (a.mode == DES_VOTE || s_hist[33] == 0);
  if (wave == 0) {
    int base = 0;
    int32_t* out = a.coreset_idx + static_cast<size_t>(b) * a.cap;
    for (int c = 0; c < MP; c += 64) {
      const int e = c + lane;
      const bool f = e < MP && (from_rank ? (s_key[e] != 0u && s_rank[e] < a.C) : (s_core[e] != 0));
      if (from_rank && e < MP) s_core[e] = f ? 1 : 0;
      const unsigned long long bal = __ballot(f);
      const int pre = __popcll(bal & ((1ull << lane) - 1ull));
      if (a.dense && e < MP) s_level[e] = f ? base + pre : -1;  // the expert's slot (stage 1 is done with s_level)
      if (f && base + pre < a.cap && !dry && g == 0) out[base + pre] = e;
      base += __popcll(bal);
    }
    if (!dry && g == 0)
      for (int i = base + lane; i < a.cap; i += 64) out[i] = -1;
    if (lane == 0) {
      s_hist[34] = base;
      if (!dry && g == 0) {
        a.coreset_size[b] = base;
        if (a.k_seq_used) a.k_seq_used[b] = (a.mode == DES_SEQ) ? s_hist[33] : 0;
      }
    }
  }
  __syncthreads();
  if (a.topk_idx == nullptr) return true;
  if (a.dense) {
    // The slot table of the coreset in ascending expert order, every token of the block
    // listed for every slot; stage 2 fills in who is routed where.
    if (!dry) {
      const int size = s_hist[34];
      for (int e = threadIdx.x; e < M; e += kRtThreads) {
        const int sl = s_level[e] < a.n_slots ? s_level[e] : -1;
        a.slot_of[e] = sl;
        if (sl >= 0) {
          a.slots[sl] = make_int4(e, sl * N, N, 0);
          a.tokmask[sl] = 0u;
        }
      }
      for (int sl = size + threadIdx.x; sl < a.n_slots; sl += kRtThreads) a.slots[sl] = make_int4(-1, 0, 0, 0);
      if (threadIdx.x == 0) {
        a.meta[0] = size;
        a.meta[1] = 0;
        a.meta[2] = 0;
        // provisional: the combine launch counts the experts that received a token
        a.n_unique[0] = (a.prev_n_unique != nullptr && a.prev_n_unique[0] < 0) ? -1 : size;
      }
    }
    return true;
  }

  DES_STAMP(a, 4);
  // ------------------------------ stage 2: constrained local routing + gates
  // With several selector workgroups the permutation runs in a workgroup of its own
  // and reads S_n from memory: the indices then travel with device-scope stores
  // and loads, like the logits, so the hand-off needs no fence.
  const bool idx_dev = a.use_flags && a.B * a.groups > 1;
  auto put_idx = [&](int32_t* p, int v) {
    if (idx_dev) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
  };
  const int keff = min(a.k_route, s_hist[34]);  // experts per token: Alg. 1 stage 2 with k <= K
  const bool reuse_sort = single_pass && a.mode != DES_VANILLA;  // stage 1 sorted this token

  for (int n0 = g * TPP; n0 + wave * RPW < N; n0 += G * TPP) {
    const int n = n0 + slot;
    const bool live = n < N && !dry;
    if (!reuse_sort) {
      float val[kEpl];
      uint32_t key[kEpl];
      load_sort(n, val, key);
    }
    // candidates: sorted positions whose expert sits in the coreset
    uint32_t cmask = 0;
#pragma unroll
    for (int sp = 0; sp < kEpl; ++sp) {
      const int e = rl * kEpl + static_cast<int>((sidx >> (3 * sp)) & 7u);
      cmask |= (static_cast<uint32_t>(sp) < nvalid && s_core[e] != 0) ? (1u << sp) : 0u;
    }
    Head hd;
    head_set(hd, cmask, my_sorted);
    const size_t o = (static_cast<size_t>(b) * N + (live ? n : 0)) * K;
    uint32_t mkey[NW], m0 = 0u;  // keys drawn at iterations rl, rl + LPT, ...; the first key
#pragma unroll
    for (int q = 0; q < NW; ++q) mkey[q] = 0u;
    int have = keff;  // experts this token found (fewer only under a group limit)
    for (int it = 0; it < keff; ++it) {  // S_n = TopK(I_n restricted to C, K), best first
      bool mine;
      const uint32_t m = row_draw<LPT>(hd, mine);  // every lane of the row sees the drawn key
      if (it == 0) m0 = m;
      if (m == 0u) have = min(have, it);
#pragma unroll
      for (int q = 0; q < NW; ++q)
        if (it == q * LPT + rl) mkey[q] = m;
      if (mine) {
        const int e = rl * kEpl + static_cast<int>((sidx >> (3 * hd.h)) & 7u);
        if (live) {
          put_idx(a.topk_idx + o + it, e);
          // (a block of at most 32 tokens in one workgroup: the expert's token bitmap is
          // all the permutation needs; integer LDS atomics, independent of arrival order)
          if (a.small_perm) atomicOr(&s_mask[e], 1u << n);
        }
        head_set(hd, hd.mask & (hd.mask - 1u), my_sorted);
      }
    }
    // gate numerators of this lane's slots, then the row's sum in a fixed order
    const float mx = key_to_f32(m0);
    float mye[NW], part = 0.f;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      mye[q] = !mkey[q] ? 0.f
               : a.sigmoid ? sigmoid_f(key_to_f32(mkey[q]))
                           : exp_neg(key_to_f32(mkey[q]) - mx);
      part += mye[q];
    }
    float den = row_sum_f32<LPT>(part);
    DES_STAMP(a, 17);
    int keep = have;
    if (a.skip_beta > 0.f && keff > 1) {
      // Sec. 5.1 (Baselines), adapted NAEE rule: drop experts i..k when their
      // gates sum to less than beta of the total.  Tail sums from the weakest
      // expert upwards, fp32, rank order; numerators suffice (the ratio to the
      // total does not depend on the normalisation).
      const float thr = a.skip_beta * den;
      float suf = 0.f;
      for (int it = keff - 1; it >= 1; --it) {  // keff is the same for every row
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
          const float c = __shfl(mye[q], (lane & ~(LPT - 1)) + (it % LPT));
          if (it / LPT == q) v = c;
        }
        suf += v;
        if (it < have && suf < thr) keep = it;
      }
      part = 0.f;
#pragma unroll
      for (int q = 0; q < NW; ++q) part += (q * LPT + rl < keep) ? mye[q] : 0.f;
      den = row_sum_f32<LPT>(part);  // gates re-normalised over the survivors
    }
    // g_n = softmax of the selected logits (Alg. 1 stage 2); unused slots -1 / 0
    if (live) {
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        const int it = q * LPT + rl;
        if (it < K) {
          a.topk_w[o + it] = it < keep ? mye[q] / den : 0.f;
          if (it >= keep) put_idx(a.topk_idx + o + it, -1);
        }
      }
    }
  }
  return true;
}

// ----------------------------------------------------- role P: permutation
// Because a token names an expert at most once, the pairs of expert e ordered
// by (token, slot) are ordered by token alone, so a per-expert bitmap over the
// tokens gives every pair's sorted position with popcounts: no sort, no float,
// integer LDS atomics only (their result does not depend on arrival order).
// The popcounts before each bitmap word are kept too, so a pair's position is one
// table entry and one popcount whatever the number of tokens.
// idx_dev: S_n was written by other workgroups of this launch with device-scope
// stores (read it the same way).
// MP = the kernel's padded expert count (M <= MP): the counters are kept for MP
// experts (zero past M) so that the ranking below has compile-time trip counts.
// part / parts: a launch of its own may spread the pairs over several workgroups.
// Each builds the whole bitmap (reading the indices is cheap), places its share of
// the pairs, and the first also writes the tables; nobody reads what another wrote.
// What bounds it is latency: one workgroup on one compute unit, so the index loads of
// a thread are requested eight at a time, and the work per pair does not grow with
// the block (16384 pairs of 128 experts: 16.0 us; walking the bitmap words per pair in
// one workgroup took 127 us).
template <int MP>
__device__ void permute_all(const RoutingArgs& a, char* smem, bool idx_dev, int part, int parts) {
  const int T = a.B * a.N, K = a.K, M = a.M;
  const int words = (T + 31) / 32;
  uint32_t* member = reinterpret_cast<uint32_t*>(smem);           // [M][words]
  int* s_cnt = reinterpret_cast<int*>(member + static_cast<size_t>(M) * words);  // [MP]
  int* s_off = s_cnt + MP;                                         // [M+1]
  int* s_liv = s_off + M + 1;                                      // [M+1]
  int* s_slot = s_liv + M + 1;                                     // [MP] slot of a live expert
  int* s_uoff = s_slot + MP;                                       // [MP] its first unit
  uint16_t* s_pre = reinterpret_cast<uint16_t*>(s_uoff + MP);      // [M][words] pairs before the word
  const int tid = threadIdx.x;
  const int TK = T * K;

  auto get_idx = [&](int p) {
    return idx_dev ? __hip_atomic_load(a.topk_idx + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                   : a.topk_idx[p];
  };
  // every pair of [p0, p1), `kBatch` indices of a thread in flight at a time
  constexpr int kBatch = 8;
  auto for_pairs = [&](int p0, int p1, auto&& f) {
    for (int p = p0 + tid; p < p1; p += kBatch * kRtThreads) {
      int e[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) e[i] = p + i * kRtThreads < p1 ? get_idx(p + i * kRtThreads) : -1;
#pragma unroll
      for (int i = 0; i < kBatch; ++i)
        if (p + i * kRtThreads < p1) f(p + i * kRtThreads, e[i]);
    }
  };
  constexpr int kKeep = 2;  // up to 2048 pairs stay in registers for the second pass
  const bool keep = TK <= kKeep * kRtThreads;
  int kept[kKeep];
#pragma unroll
  for (int i = 0; i < kKeep; ++i)
    kept[i] = keep && tid + i * kRtThreads < TK ? get_idx(tid + i * kRtThreads) : -1;
  for (int i = tid; i < M * words; i += kRtThreads) member[i] = 0u;
  __syncthreads();
  auto mark = [&](int p, int e) {
    if (e >= 0) {
      const int t = p / K;
      atomicOr(&member[static_cast<size_t>(e) * words + (t >> 5)], 1u << (t & 31));
    }
  };
  if (keep) {
#pragma unroll
    for (int i = 0; i < kKeep; ++i) mark(tid + i * kRtThreads, kept[i]);
  } else {
    for_pairs(0, TK, mark);
  }
  __syncthreads();
  // counts and the popcounts before each word: a thread per expert while that is a short
  // loop, else eight lanes per expert, each a run of consecutive words, scanned over the eight
  auto count_expert = [&](int e, int c) {
    s_cnt[e] = c;
    s_slot[e] = 0;
    s_uoff[e] = 0;
    if (e < M && part == 0) a.expert_counts[e] = c;
  };
  if (words <= 8) {
    for (int e = tid; e < MP; e += kRtThreads) {
      int c = 0;
      if (e < M)
        for (int w = 0; w < words; ++w) {
          const size_t i = static_cast<size_t>(e) * words + w;
          s_pre[i] = static_cast<uint16_t>(c);
          c += __popc(member[i]);
        }
      count_expert(e, c);
    }
  } else {
    constexpr int GL = 8;
    const int run = (words + GL - 1) / GL, gl = tid % GL;
    for (int e = tid / GL; e < MP; e += kRtThreads / GL) {
      const int w0 = min(gl * run, words), w1 = min(w0 + run, words);
      const uint32_t* mrow = member + static_cast<size_t>(e < M ? e : 0) * words;
      int c = 0;
      if (e < M)
        for (int w = w0; w < w1; ++w) c += __popc(mrow[w]);
      int inc = c;
#pragma unroll
      for (int d = 1; d < GL; d <<= 1) {
        const int o = __shfl_up(inc, d, GL);
        if (gl >= d) inc += o;
      }
      if (e < M) {
        int pre = inc - c;
        for (int w = w0; w < w1; ++w) {
          s_pre[static_cast<size_t>(e) * words + w] = static_cast<uint16_t>(pre);
          pre += __popc(mrow[w]);
        }
      }
      if (gl == GL - 1) count_expert(e, inc);
    }
  }
  __syncthreads();
  // Slot order.  Up to 32 tokens every FFN task is on the chip at once and the
  // order does not matter: live experts by index.  Longer blocks: most pairs
  // first (ties to the lowest expert index), because the FFN launches hand out
  // their workgroups in slot order and, when not all of them fit on the chip at
  // once, the long ones must not be the ones that start last.  Rank by counting,
  // the comparison range split over the threads that share an expert; the
  // partial ranks meet in an integer LDS add.  The same pass counts the units
  // (groups of up to 2^rows_shift pairs) of the experts
  // ahead: the expert's place in the unit list.
  const bool by_count = T > 32;
  const int rsh = a.rows_shift;
  auto units_of = [&](int c) { return min((c + (1 << rsh) - 1) >> rsh, kMaxSplits); };
  if (by_count) {
    constexpr int P = kRtThreads / MP, CH = MP / P;  // MP * P threads: each one expert, CH rivals
    const int e = tid % MP, j0 = (tid / MP) * CH;
    const int ce = s_cnt[e];
    if (ce > 0) {
      int r = 0, uo = 0;
#pragma unroll
      for (int jj = 0; jj < CH; ++jj) {  // counts past M are zero: never ahead of a live expert
        const int cj = s_cnt[j0 + jj];
        const bool ahead = cj > ce || (cj == ce && j0 + jj < e);
        r += ahead ? 1 : 0;
        uo += ahead ? units_of(cj) : 0;
      }
      if (r) {
        atomicAdd(&s_slot[e], r);
        atomicAdd(&s_uoff[e], uo);
      }
    }
  }
  if (tid < 64) {  // exclusive scans of counts and of (count > 0), 64 experts at a time
    int base_c = 0, base_l = 0;
    for (int c0 = 0; c0 < M; c0 += 64) {
      const int e = c0 + tid;
      const int c = e < M ? s_cnt[e] : 0;
      int inc = c;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(inc, d);
        if (tid >= d) inc += o;
      }
      const unsigned long long bal = __ballot(c > 0);
      const int lpre = __popcll(bal & ((1ull << tid) - 1ull));
      if (e < M) {
        s_off[e] = base_c + inc - c;
        s_liv[e] = base_l + lpre;
      }
      base_c += __shfl(inc, 63);
      base_l += __popcll(bal);
    }
    if (tid == 0) {
      s_off[M] = base_c;
      s_liv[M] = base_l;
      if (part == 0) {
        a.meta[0] = base_l;
        a.meta[1] = base_c;
        a.meta[2] = 0;  // live units: set after the barrier by the last slot's expert, if any
        a.n_unique[0] = (a.prev_n_unique != nullptr && a.prev_n_unique[0] < 0) ? -1 : base_l;
      }
    }
  }
  __syncthreads();
  const int n_live = s_liv[M];
  if (part == 0) {
    for (int e = tid; e <= M; e += kRtThreads) a.offsets[e] = s_off[e];
    for (int e = tid; e < M; e += kRtThreads) {
      const int c = s_cnt[e];
      const int sl = by_count ? s_slot[e] : s_liv[e];
      const bool live = c > 0 && sl < a.n_slots;
      // (up to 32 tokens the expert's bitmap row is one word: the tokens routed to it)
      if (live) a.slots[sl] = make_int4(e, s_off[e], c, words == 1 ? static_cast<int>(member[e]) : 0);
      a.slot_of[e] = live ? sl : -1;
      if (live && by_count) {
        const int nu = units_of(c);
        for (int k = 0; k < nu; ++k) a.units[s_uoff[e] + k] = sl | (k << 16) | (nu << 24);
        if (sl == n_live - 1) a.meta[2] = s_uoff[e] + nu;  // the last slot closes the list
      }
    }
    for (int s = n_live + tid; s < a.n_slots; s += kRtThreads) a.slots[s] = make_int4(-1, 0, 0, 0);
  }
  auto place = [&](int p, int e) {
    if (e < 0) { a.pos[p] = -1; return; }
    const int t = p / K;
    const size_t w = static_cast<size_t>(e) * words + (t >> 5);
    const int r = s_off[e] + s_pre[w] + __popc(member[w] & ((1u << (t & 31)) - 1u));
    a.pair_tok[r] = t;
    a.pos[p] = r;
  };
  if (keep) {
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
      if (tid + i * kRtThreads < TK) place(tid + i * kRtThreads, kept[i]);
  } else {
    const int share = (TK + parts - 1) / parts;
    for_pairs(part * share, min(TK, (part + 1) * share), place);
  }
}

// A bounded wait ran out (a fault of the device, or another kernel keeps this
// launch's producers off the chip): leave an EMPTY work list, so that the FFN
// launches that follow find no expert, index nothing and the combine adds no
// routed row - y is then the shared expert's output (+ x under `residual`), and
// n_unique = -1 says so.  Every workgroup that gives up writes the same values.
__device__ void publish_empty(const RoutingArgs& a, int n_flags) {
  const int tid = threadIdx.x;
  if (a.slots != nullptr) {
    for (int s = tid; s < a.n_slots; s += kRtThreads) a.slots[s] = make_int4(-1, 0, 0, 0);
    for (int i = tid; i < a.B * a.N * a.K; i += kRtThreads) a.pos[i] = -1;
    for (int e = tid; e <= a.M; e += kRtThreads) a.offsets[e] = 0;
    for (int e = tid; e < a.M; e += kRtThreads) {
      a.slot_of[e] = -1;
      a.expert_counts[e] = 0;
    }
    if (tid < 3) a.meta[tid] = 0;
  }
  // the flags of this call are abandoned: clear them, so that a replay of a
  // captured launch (same epoch) starts from flags that no producer has set
  if (a.use_flags)
    for (int i = tid; i < n_flags; i += kRtThreads) a.flags[i] = 0ull;
  if (tid == 0 && a.n_unique) a.n_unique[0] = -1;
}

// The same outputs as permute_all for a block of at most 32 tokens whose selection
// ran in this workgroup: stage 2 has left, per expert, the bitmap of the tokens routed
// to it (s_mask), so counts are popcounts, an expert's pairs in token order are its set
// bits in order, and a pair's sorted position is a popcount below its token's bit.  No
// second pass over the indices to build bitmaps (the FFN kernels take
// the bitmap from the slot record).
template <int LPT>
__device__ void permute_small(const RoutingArgs& a, char* smem) {
  using L = SelLds<LPT>;
  const uint32_t* s_mask = reinterpret_cast<const uint32_t*>(smem + L::mask);
  int* s_off = reinterpret_cast<int*>(smem + L::off);
  int* s_liv = reinterpret_cast<int*>(smem + L::liv);
  const int tid = threadIdx.x, M = a.M, K = a.K, TK = a.B * a.N * a.K;
  if (tid < 64) {  // exclusive scans of counts and of (count > 0), 64 experts at a time
    int base_c = 0, base_l = 0;
    for (int c0 = 0; c0 < M; c0 += 64) {
      const int e = c0 + tid;
      const int c = e < M ? __popc(s_mask[e]) : 0;
      int inc = c;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(inc, d);
        if (tid >= d) inc += o;
      }
      const unsigned long long bal = __ballot(c > 0);
      const int lpre = __popcll(bal & ((1ull << tid) - 1ull));
      if (e < M) {
        s_off[e] = base_c + inc - c;
        s_liv[e] = base_l + lpre;
      }
      base_c += __shfl(inc, 63);
      base_l += __popcll(bal);
    }
    if (tid == 0) {
      s_off[M] = base_c;
      s_liv[M] = base_l;
      a.meta[0] = base_l;
      a.meta[1] = base_c;
      a.meta[2] = 0;
      a.n_unique[0] = (a.prev_n_unique != nullptr && a.prev_n_unique[0] < 0) ? -1 : base_l;
    }
  }
  __syncthreads();
  const int n_live = s_liv[M];
  for (int e = tid; e <= M; e += kRtThreads) a.offsets[e] = s_off[e];
  for (int e = tid; e < M; e += kRtThreads) {
    const uint32_t m = s_mask[e];
    const int c = __popc(m), sl = s_liv[e];
    const bool live = c > 0 && sl < a.n_slots;
    a.expert_counts[e] = c;
    if (live) a.slots[sl] = make_int4(e, s_off[e], c, static_cast<int>(m));
    a.slot_of[e] = live ? sl : -1;
  }
  for (int s = n_live + tid; s < a.n_slots; s += kRtThreads) a.slots[s] = make_int4(-1, 0, 0, 0);
  for (int p = tid; p < TK; p += kRtThreads) {
    const int e = a.topk_idx[p];  // (stored by this workgroup before the barrier above)
    if (e < 0) {
      a.pos[p] = -1;
      continue;
    }
    const int t = p / K;
    const int r = s_off[e] + __popc(s_mask[e] & ((1u << t) - 1u));
    a.pair_tok[r] = t;
    a.pos[p] = r;
  }
}

// ---------------------------------------------------------------- the kernel
// LDS of the routing kernel: the selection's carve-up, but at least what the
// router tile (32 KB, see router_tile_bf16) and the permutation (bitmap of at most 8192
// words, as many 16-bit counts and at most 5 * 512 + 2 counters, under 59 KB for every
// shape the library accepts) need.
constexpr int kMinRoutingLds = 59 * 1024;
static_assert(kMinRoutingLds >= 8192 * 6 + 4 * (5 * 512 + 2), "permutation tables");
static_assert(kMinRoutingLds >= kRtWaves * 2 * kOperandBytes, "router tile");

template <int LPT, bool EXT>
__global__ __launch_bounds__(kRtThreads) void routing_kernel(RoutingArgs a) {
  constexpr int kLds = SelLds<LPT>::total > kMinRoutingLds ? SelLds<LPT>::total : kMinRoutingLds;
  __shared__ __align__(16) char smem[kLds];
  const int n_tiles = (a.do_router && !a.skip_router_tiles && !a.solo) ? a.tiles_m * a.tiles_t : 0;
  int blk = blockIdx.x;
  if (a.xo != nullptr && blk >= a.x_first) {  // x for the gate/up launch; nobody in this launch waits for it
    const int T = a.B * a.N, pieces = T * (a.D / 8), step = (gridDim.x - a.x_first) * kRtThreads;
    for (int p = (blk - a.x_first) * kRtThreads + threadIdx.x; p < pieces; p += step) {
      const int oct = p / (4 * T) * 4 + p % 4, t = p / 4 % T;  // (four neighbouring lanes along a row)
      *reinterpret_cast<uint4*>(a.xo + (static_cast<size_t>(oct) * T + t) * 8) =
          *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.x) + static_cast<size_t>(t) * a.D + oct * 8);
    }
    return;
  }
  if (blk < n_tiles || a.solo) {  // ---- role R
    if (blk == 0) DES_STAMP(a, 8);
    if (a.bf16) router_tile_bf16(a, blk % a.tiles_m, blk / a.tiles_m, smem);
    else router_tile_f32(a, blk % a.tiles_m, blk / a.tiles_m);
    if (blk == 0) DES_STAMP(a, 9);
    if (a.use_flags) {
      stores_done();  // this thread's logits have reached the level all compute units share
      __syncthreads();
      if (threadIdx.x == 0 && !a.solo) flag_publish(a.flags + blk, a.epoch, false);
    }
    if (blk == 0) DES_STAMP(a, 10);
    if (!a.solo) return;
  }
  blk -= n_tiles;
  const int n_sel = a.do_select ? a.B * a.groups : 0;
  const int all_tiles = a.tiles_m * a.tiles_t;
  const int n_flags = all_tiles + 2 * a.B * a.groups;
  int part = 0;         // of the permutation
  bool idx_dev = false;
  if (blk < n_sel) {  // ---- role S
    DES_STAMP(a, 0);
    if (!select_sequence<LPT, EXT>(a, blk / a.groups, blk % a.groups, smem, false,
                              a.use_flags && a.do_router && !a.solo)) {
      publish_empty(a, n_flags);  // a bounded wait expired
      return;
    }
    DES_STAMP(a, 5);
    if (a.topk_idx == nullptr) return;
    if (!a.dense && !(n_sel == 1 && a.do_permute)) {  // the permutation is another workgroup's
      if (a.use_flags) {
        stores_done();
        __syncthreads();
        if (threadIdx.x == 0) flag_publish(a.flags + all_tiles + n_sel + blk, a.epoch, false);
      }
      return;
    }
    // a single selector permutes right here (a dense block has no permutation, and no stage 2
    // here): same workgroup, same compute unit, so the barrier orders the topk_idx stores
    // before the loads below, no device-scope fence needed
    __syncthreads();
    DES_STAMP(a, 6);
  } else {  // ---- role P
    part = blk - n_sel;
    if (part >= a.perm_parts || !a.do_permute || a.B * a.groups == 1) return;
    if (a.use_flags && a.do_select &&
        !flags_wait(a.flags + all_tiles + a.B * a.groups, a.B * a.groups, a.epoch, false,
                    a.max_wait)) {
      publish_empty(a, n_flags);  // a bounded wait expired
      return;
    }
    idx_dev = a.use_flags && a.do_select;
  }
  // (one place for both roles: a second copy of the permutation makes the kernel 8 KB longer,
  // 46 against 38 KB, and its code is fetched anew by every launch: selection alone +0.2 us)
  if (a.dense) {
  } else if (a.small_perm) {
    permute_small<LPT>(a, smem);
  } else {
    permute_all<SelLds<LPT>::MP>(a, smem, idx_dev, part, a.perm_parts);
  }
  DES_STAMP(a, 7);
  // every flag of this call has been consumed: clear them, so that a replay
  // of a captured launch (same epoch) cannot be satisfied by stale flags
  if (a.use_flags)
    for (int i = threadIdx.x; i < n_flags; i += kRtThreads) a.flags[i] = 0ull;
}

// The router as a launch of its own (des_route, and batches whose routing does not fit one launch):
// a workgroup has ET x TT of the 16 x 16 tiles of router_tile_bf16, each summed up in the same order.
template <int ET, int TT>
__global__ __launch_bounds__(kRtThreads, 8) void router_kernel(RoutingArgs a) {
  constexpr int U = ET * TT == 1 ? 4 : 2;  // k-steps per trip; two workgroups share a compute unit
  // of a wavefront: the operands of a k-step, then its partial tiles
  constexpr int kMine = (ET + TT > ET * TT ? ET + TT : ET * TT) * 256;  // floats
  __shared__ __align__(16) float part[kRtWaves * kMine];
  const int lane = threadIdx.x & 63;
  const int wave = uniform_int(threadIdx.x >> 6);  // (it guards matrix instructions, see stream_pipeline)
  const int T = a.B * a.N, D = a.D, M = a.M, nks = D / 32;
  const int groups = (a.tiles_m + ET - 1) / ET;
  const int i0 = blockIdx.x % groups * 16 * ET, t0 = blockIdx.x / groups * 16 * TT;
  const int r = lane & 15, row = lane >> 2, kq = (lane & 3) * 8;
  char* mine_lds = reinterpret_cast<char*>(part + wave * kMine);
  const uint16_t *ap[ET], *bp[TT];  // clamped rows are computed and dropped
#pragma unroll
  for (int e = 0; e < ET; ++e)
    ap[e] = static_cast<const uint16_t*>(a.w_router) + static_cast<size_t>(min(i0 + 16 * e + row, M - 1)) * D + kq;
#pragma unroll
  for (int t = 0; t < TT; ++t)
    bp[t] = static_cast<const uint16_t*>(a.x) + static_cast<size_t>(min(t0 + 16 * t + row, T - 1)) * D + kq;
  // the element that this thread will finish
  const int tile = threadIdx.x >> 8, er = threadIdx.x & 15, tc = (threadIdx.x >> 4) & 15;
  const int ef = i0 + 16 * (tile / TT) + er, tf = t0 + 16 * (tile % TT) + tc;
  // (its place in one register: two across the loop spill)
  const int fin = tile < ET * TT && ef < M && tf < T ? tf * M + ef : -1;
  const float bias = fin >= 0 && a.bias ? a.bias[ef] : 0.f;
  f32x4 acc[ET][TT];
#pragma unroll
  for (int e = 0; e < ET; ++e)
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[e][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int ks = wave; ks < nks; ks += U * kRtWaves) {
    bf16x8 av[U][ET], bv[U][TT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(ks + u * kRtWaves, nks - 1) * 32;  // clamped steps are skipped below
#pragma unroll
      for (int e = 0; e < ET; ++e) av[u][e] = *reinterpret_cast<const bf16x8*>(ap[e] + k);
#pragma unroll
      for (int t = 0; t < TT; ++t) bv[u][t] = *reinterpret_cast<const bf16x8*>(bp[t] + k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      turn_fence();
#pragma unroll
      for (int e = 0; e < ET; ++e) operand_write(av[u][e], mine_lds + e * kOperandBytes, lane);
#pragma unroll
      for (int t = 0; t < TT; ++t) operand_write(bv[u][t], mine_lds + (ET + t) * kOperandBytes, lane);
      turn_fence();
#pragma unroll
      for (int e = 0; e < ET; ++e) av[u][e] = operand_read(mine_lds + e * kOperandBytes, lane);
#pragma unroll
      for (int t = 0; t < TT; ++t) bv[u][t] = operand_read(mine_lds + (ET + t) * kOperandBytes, lane);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (ks + u * kRtWaves < nks)
#pragma unroll
        for (int e = 0; e < ET; ++e)
#pragma unroll
          for (int t = 0; t < TT; ++t)
            acc[e][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[u][e], bv[u][t], acc[e][t], 0, 0, 0);
  }
  turn_fence();
#pragma unroll
  for (int e = 0; e < ET; ++e)
#pragma unroll
    for (int t = 0; t < TT; ++t)
      *reinterpret_cast<f32x4*>(part + wave * kMine + (e * TT + t) * 256 + r * 16 + 4 * (lane >> 4)) = acc[e][t];
  __syncthreads();
  if (fin < 0) return;
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < kRtWaves; ++w) s += part[w * kMine + tile * 256 + tc * 16 + er];  // fixed order
  a.logits[fin] = s + bias;
}

// probs[t][:] = router weights of token t (softmax of its logits, or their
// sigmoids); one wavefront per token (des_route only).
__global__ __launch_bounds__(64) void softmax_kernel(const float* __restrict__ logits,
                                                     float* __restrict__ probs, int M, int sigmoid) {
  const int lane = threadIdx.x;
  const float* row = logits + static_cast<size_t>(blockIdx.x) * M;
  float* out = probs + static_cast<size_t>(blockIdx.x) * M;
  if (sigmoid) {
    for (int i = lane; i < M; i += 64) out[i] = sigmoid_f(row[i]);
    return;
  }
  uint32_t mk = 0;
  for (int i = lane; i < M; i += 64) mk = max(mk, order_key(row[i]));
  const float mx = key_to_f32(wave_max_u32(mk));
  float s = 0.f;
  for (int i = lane; i < M; i += 64) s += expf(row[i] - mx);
  s = wave_sum_f32(s);
  const float inv = 1.0f / s;
  for (int i = lane; i < M; i += 64) out[i] = expf(row[i] - mx) * inv;
}

// ------------------------------------------------------------------ launchers
static int launch_routing_grid(const RoutingArgs& a, int grid, int kernel_id, hipStream_t st) {
  const int lanes = (a.M + kEpl - 1) / kEpl;  // lanes a token's experts need, 8 experts each
  const dim3 g(grid), b(kRtThreads);
#define DES_LAUNCH_ROUTING(EXT)                                                     \
  do {                                                                             \
    if (lanes <= 4) launch(kernel_id, routing_kernel<4, EXT>, g, b, 0, st, a);       \
    else if (lanes <= 8) launch(kernel_id, routing_kernel<8, EXT>, g, b, 0, st, a);  \
    else if (lanes <= 16) launch(kernel_id, routing_kernel<16, EXT>, g, b, 0, st, a); \
    else if (lanes <= 32) launch(kernel_id, routing_kernel<32, EXT>, g, b, 0, st, a); \
    else launch(kernel_id, routing_kernel<64, EXT>, g, b, 0, st, a);                 \
  } while (0)
  if (a.n_group > 1 || a.vote_atomic) DES_LAUNCH_ROUTING(true);
  else DES_LAUNCH_ROUTING(false);
#undef DES_LAUNCH_ROUTING
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DES_OK : hip_fail(e, "routing launch");
}

// Compute units of the current device (kept per device, 0 = not known yet; threads may ask at the
// same time).  A routing workgroup fills a whole compute unit (16 wavefronts at up to 128
// registers), so the fused launch may use at most this many workgroups if all are to be resident.
static int device_compute_units() {
  constexpr int kDevices = 64;
  static std::atomic<int> known[kDevices];
  if (g_test_compute_units >= 0) {
    const int n = g_test_compute_units;
    g_test_compute_units = -1;
    return n;
  }
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  const bool keep = dev >= 0 && dev < kDevices;
  if (keep) n = known[dev].load(std::memory_order_relaxed);
  if (n > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (keep) known[dev].store(n, std::memory_order_relaxed);
  return n;
}

static void fill_common(RoutingArgs& a, const des_shape_t& s) {
  a = RoutingArgs{};
  a.B = s.n_seqs; a.N = s.n_tokens; a.M = s.n_experts; a.K = s.top_k; a.C = s.coreset;
  a.k_seq = s.k_seq; a.mode = s.mode; a.cap = des_coreset_capacity(&s); a.D = s.hidden;
  a.n_slots = max_live_experts(s);
  a.tiles_m = (s.n_experts + 15) / 16;
  a.tiles_t = (s.n_seqs * s.n_tokens + 15) / 16;
  a.bf16 = s.dtype == DES_BF16;
  a.groups = 1;
  a.perm_parts = 1;
  a.max_wait = g_test_max_wait > 0 ? g_test_max_wait : kMaxWaitIters;
  a.k_route = s.k_route > 0 ? s.k_route : s.top_k;
  a.skip_beta = s.skip_beta;
  a.sigmoid = s.router_act == DES_ROUTER_SIGMOID;
  a.vote_renorm = s.vote_renorm;
  a.vote_atomic = s.vote_atomic;
  if (s.n_group > 1 && s.topk_group < s.n_group) {  // keeping every group is no limit
    a.n_group = s.n_group;
    a.group_lanes = s.n_experts / s.n_group / kEpl;
    a.topk_group = s.topk_group;
    a.group_top2 = s.group_score == DES_GROUP_TOP2SUM;
  }
}

LayerForm layer_form(const des_shape_t& s) {
  const int n_tiles = ((s.n_experts + 15) / 16) * ((s.n_seqs * s.n_tokens + 15) / 16);
  int fused_limit = device_compute_units();
  if (fused_limit > kMaxFusedRoutingBlocks) fused_limit = kMaxFusedRoutingBlocks;
  // A selector workgroup handles selector_tokens_per_pass() tokens at once; a
  // longer sequence is spread over several selector workgroups when they all fit.
  const int tpp = selector_tokens_per_pass(s.n_experts);
  int groups = (s.n_tokens + tpp - 1) / tpp;
  if (groups > kMaxSelGroups / s.n_seqs) groups = kMaxSelGroups / s.n_seqs > 0 ? kMaxSelGroups / s.n_seqs : 1;
  if (n_tiles + s.n_seqs * groups + 1 > fused_limit) groups = 1;
  const int roles = n_tiles + s.n_seqs * groups + (s.n_seqs * groups > 1 ? 1 : 0);
  const bool fused = roles <= fused_limit;
  const bool dense = fused && dense_shape(s) && s.n_tokens <= tpp;
  // x in operand order, against in rows, routing and gate/up of 14 layers.  Dense blocks (gate/up takes all
  // tokens): 1, 2 and 4 tokens take 1.02, 1.01 and 1.01 of the time (of one token both are the same bytes), 6
  // to 16 0.99, 17 to 24 0.97, 32 0.94 (3072 x 1536 0.87); 512 wide 0.97 to 1.06.  Elsewhere the pieces of an
  // expert's few tokens lie further apart than their rows: 20 to 32 tokens of 1024 to 2048 0.93 to 1.01 (64
  // experts of 2048 x 512, k = 8, vanilla: 1.04), up to 17 tokens 1.01, above 2048 0.98 to 1.08.
  const int T = s.n_seqs * s.n_tokens;
  const bool x_copy = fused && s.dtype == DES_BF16 && T <= 32 && s.hidden >= 1024 &&
                      (dense ? T >= 6 : T >= 20 && s.hidden <= 2048);
  return LayerForm{groups, roles, fused, dense, x_copy};
}

void layer_plan(const des_shape_t& s, int32_t* plan) {
  const LayerForm f = layer_form(s);
  plan[0] = f.fused; plan[1] = f.dense; plan[2] = f.x_copy; plan[3] = f.groups;
}

// Four tiles per workgroup read half as much per tile, where one tile each makes more than one round of
// the chip.  One and four, in us.  Up to 1024 wide: 128 experts of 1024, 224 tiles 4.0 and 4.6, 288 5.5 and
// 4.8, 1024 8.9 and 6.1; of 256, 272 tiles level; of 128, where reading counts for little, 512 tiles 3.3 and
// 3.4, 576 4.0 and 3.4.  Wider, with many token rows: 128 experts of 2048, 256 tiles 5.4 and 6.8, 288 6.7 and
// 6.9, 320 7.4 and 6.9, 512 8.2 and 7.1; of 3072, 256 tiles 7.2 and 9.2, 264 9.7 and 9.2, 288 10.0 and 9.3.  With
// few (many experts), one tile each stays ahead up to two rounds: 256 of 2048, 320 tiles 6.2 and 7.0, 512 6.8 and
// 7.2, 576 7.6 and 7.3, 1024 10.1 and 8.4.  Between, at 160 to 224 experts, fours lose up to 7 % past the lines
// below (192 of 1536, 444 tiles: 6.5 and 7.0).
static bool wide_router(const RoutingArgs& a) {
  const int tiles = a.tiles_m * a.tiles_t;
  if (a.D <= 1024) return a.D < 256 ? tiles >= 512 : tiles > 256;
  return tiles > 512 || (a.D <= 2048 ? tiles > 288 && a.tiles_t > 35 : tiles > 256 && a.tiles_t > 32);
}

static int launch_router_tiles(const RoutingArgs& a, hipStream_t st) {
  const int tiles = a.tiles_m * a.tiles_t;
  if (!a.bf16) return launch_routing_grid(a, tiles, kKRouter, st);
  const dim3 b(kRtThreads);
  if (wide_router(a))
    launch(kKRouter, router_kernel<2, 2>, dim3((a.tiles_m + 1) / 2 * ((a.tiles_t + 1) / 2)), b, 0, st, a);
  else
    launch(kKRouter, router_kernel<1, 1>, dim3(tiles), b, 0, st, a);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DES_OK : hip_fail(e, "router launch");
}

void router_plan(const des_shape_t& s, int32_t* plan) {
  RoutingArgs a;
  fill_common(a, s);
  plan[0] = plan[1] = !a.bf16 ? 0 : wide_router(a) ? 2 : 1;
  plan[2] = plan[3] = 0;
}

int launch_router(const des_shape_t& s, const void* x, const void* w_router, const float* bias,
                  float* logits, hipStream_t st) {
  RoutingArgs a;
  fill_common(a, s);
  a.x = x; a.w_router = w_router; a.bias = bias; a.logits = logits;
  a.do_router = 1;
  return launch_router_tiles(a, st);
}

int launch_softmax(const des_shape_t& s, const float* logits, float* probs, hipStream_t st) {
  const int T = s.n_seqs * s.n_tokens;
  launch(kKSoftmax, softmax_kernel, dim3(T), dim3(64), 0, st, logits, probs, s.n_experts,
         static_cast<int>(s.router_act == DES_ROUTER_SIGMOID));
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DES_OK : hip_fail(e, "softmax launch");
}

int launch_select(const des_shape_t& s, const float* logits, int32_t* coreset_idx,
                  int32_t* coreset_size, float* votes, int32_t* k_seq_used, hipStream_t st) {
  RoutingArgs a;
  fill_common(a, s);
  a.logits = const_cast<float*>(logits);
  a.coreset_idx = coreset_idx; a.coreset_size = coreset_size; a.votes = votes;
  a.k_seq_used = k_seq_used;
  a.do_select = 1;
  return launch_routing_grid(a, a.B, kKSelect, st);
}

int launch_routing(const des_shape_t& s, const LayerForm& form, const void* x, const void* w_router,
                   const float* bias, float* logits, int32_t* coreset_idx, int32_t* coreset_size,
                   int32_t* topk_idx, float* topk_w, int32_t* expert_counts, int32_t* n_unique,
                   const int32_t* prev_n_unique, char* ws, unsigned long long epoch,
                   hipStream_t st) {
  const WsLayout w = ws_layout(s);
  RoutingArgs a;
  fill_common(a, s);
  a.prev_n_unique = prev_n_unique;
  a.x = x; a.w_router = w_router; a.bias = bias; a.logits = logits;
  a.coreset_idx = coreset_idx; a.coreset_size = coreset_size;
  a.topk_idx = topk_idx; a.topk_w = topk_w;
  a.expert_counts = expert_counts; a.n_unique = n_unique;
  a.offsets = reinterpret_cast<int32_t*>(ws + w.offsets);
  a.slots = reinterpret_cast<int4*>(ws + w.slots);
  a.meta = reinterpret_cast<int32_t*>(ws + w.meta);
  a.pair_tok = reinterpret_cast<int32_t*>(ws + w.pair_tok);
  a.pos = reinterpret_cast<int32_t*>(ws + w.pos);
  a.flags = reinterpret_cast<unsigned long long*>(ws + w.flags);
  a.epoch = epoch;
  a.slot_of = reinterpret_cast<int32_t*>(ws + w.slot_of);
  a.units = reinterpret_cast<int32_t*>(ws + w.units);
  a.rows_shift = lds_rows_pass(s.n_seqs * s.n_tokens) == 64 ? 6 : 7;
  a.sel_part = reinterpret_cast<uint32_t*>(ws + w.sel_part);
  const int n_tiles = a.tiles_m * a.tiles_t;
  // One selector workgroup and at most 32 tokens: the short permutation.  (Skipping
  // drops a token's experts after they were drawn, so the bitmaps of stage 2 would name
  // pairs that no longer exist: it keeps the general permutation.)
  const bool small = a.B == 1 && form.groups == 1 && s.n_tokens <= 32 && !(s.skip_beta > 0.0f);
  if (form.fused) {  // all workgroups resident at once: one launch
    a.groups = form.groups;
    a.small_perm = small;
    a.dense = form.dense ? 1 : 0;
    a.tokmask = reinterpret_cast<uint32_t*>(ws + w.tokmask);
    a.do_router = a.do_select = a.do_permute = 1;
    a.use_flags = 1;
    int n_x = 0;
    if (form.x_copy) {
      a.xo = reinterpret_cast<uint16_t*>(ws + w.o);
      const int pieces = s.n_seqs * s.n_tokens * (s.hidden / 8);
      n_x = pieces > 16 * kRtThreads ? 16 : (pieces + kRtThreads - 1) / kRtThreads;
    }
    if (g_test_skip_router) {  // test hook: nobody computes the logits, the selectors' wait expires
      a.skip_router_tiles = 1;
      if (g_test_skip_router == 2) g_test_skip_router = g_test_max_wait = 0;  // one launch only
      a.x_first = form.roles - n_tiles;
      return launch_routing_grid(a, a.x_first + n_x, kKRouting, st);
    }
    // A single tile: handing it to another workgroup would cost more than it saves (8 tokens, 16
    // experts of width 256, fp32: routing 14.4 -> 13.4 us).
    a.solo = n_tiles == 1 && form.roles == 2;
    a.x_first = a.solo ? 1 : form.roles;
    return launch_routing_grid(a, a.x_first + n_x, kKRouting, st);
  }
  // too large to wait inside one launch: the same roles as three launches
  RoutingArgs r = a;
  r.do_router = 1;
  int rc = launch_router_tiles(r, st);
  if (rc != DES_OK) return rc;
  RoutingArgs sel = a;
  sel.do_select = 1;
  sel.do_permute = a.B == 1 ? 1 : 0;
  sel.small_perm = a.B == 1 && s.n_tokens <= 32 && !(s.skip_beta > 0.0f);
  rc = launch_routing_grid(sel, a.B, kKSelect, st);
  if (rc != DES_OK || a.B == 1) return rc;
  RoutingArgs p = a;
  p.do_permute = 1;
  // about one pair per thread and workgroup (all of them read every index for the bitmaps,
  // so more workgroups stop paying off)
  const int pairs = s.n_seqs * s.n_tokens * s.top_k;
  p.perm_parts = pairs <= 2 * kRtThreads ? 1 : (pairs + kRtThreads - 1) / kRtThreads > 16 ? 16 : (pairs + kRtThreads - 1) / kRtThreads;
  return launch_routing_grid(p, p.perm_parts, kKPermute, st);
}

}  // namespace des
