// The attention sub-layer of a block-parallel decoding step, for gfx950: every token of
// the block attends to the cached prefix / suffix positions and to the whole block
// (Sec. 5.1 fixes that window; Fig. 2 left and Sec. 5.2 count attention among the fixed,
// non-MoE costs of a step).  The paper does not define the sub-layer; this is plain
// multi-head scaled-dot-product attention without mask, positional encoding or bias.
//
// Three launches per sub-layer:
//   1. q, k, v = x Wq^T, x Wk^T, x Wv^T     one dense-projection launch over the three
//                                            weight matrices (bf16 MFMA, fp32 accumulate)
//   2. softmax(q K^T / sqrt(dh)) V           workgroups per (sequence, key/value head), bf16 MFMA
//   3. y = heads Wo^T (+ x)                  the same projection kernel, residual fused
// For at most 32 token rows the projections are weight scans like the expert FFN: weights
// from HBM straight into MFMA operands.  Longer blocks use tiles of weight rows and token
// rows that meet in LDS (des_tile_gemm.h).
#include "des_common.h"
#include "des_stream_gemm.h"
#include "des_tile_gemm.h"

namespace des {

struct LinearArgs {
  const uint16_t* in;    // [T][Din] bf16 token rows
  const uint16_t* w[3];  // up to three weight matrices [fout[i]][Din], rows along the reduction
  uint16_t* out[3];      // [T][fout[i]] bf16
  const uint16_t* res;   // [T][fout[0]] bf16 added to out[0] before rounding, or null
  int fout[3];
  int n_mats, T, Din;
  // reduction dimension split over two workgroups (ksplit = 2):
  int ksplit;
  float* partial;             // [workgroups][tiles of a workgroup][64 lanes][4] fp32 partial tiles
  unsigned long long* flags;  // [workgroup pairs] set to `epoch` by the half that finishes first
  unsigned long long epoch;   // of this call: never zero, never repeated (stale words cannot match)
};

// out[m][t][f] = sum_d in[t][d] * w[m][f][d] for blocks of more than 32 token rows, in tiles
// of 32 MT weight rows x 32 NT token rows (tile_gemm_dma, with NB buffers; NB = 0: tile_gemm).
// KW = 2: the two halves of the reduction dimension go to the two halves of the workgroup and
// meet in LDS, first half + second half.
// Consecutive workgroups go to the eight XCDs in turn: the grid is walked so that one XCD
// has all the token tiles of a weight tile (its L2 then reads those weights once).
template <int MT, int NT, int KW, int NB>
__global__ __launch_bounds__(256 * KW, NB == 0 ? 2 : 1) void linear_tile_kernel(LinearArgs a) {
  constexpr int BM = 32 * MT, BN = 32 * NT;
  __shared__ __align__(16) char lds[NB == 0 ? tile_lds_bytes<MT, NT>() : tile_dma_lds_bytes<MT, NT, KW, NB>()];
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
  const int part = KW > 1 ? threadIdx.x >> 8 : 0;
  const int wm = wave >> 1, wn = wave & 1;
  const int kd = a.Din / KW, k0 = part * kd;
  const int tok_tiles = (a.T + BN - 1) / BN;
  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  int mb = seq / tok_tiles * 8 + xcd, m = 0;
  const int g0 = seq % tok_tiles * BN;
  for (; m < a.n_mats; ++m) {  // which matrix this workgroup belongs to
    const int per = (a.fout[m] + BM - 1) / BM;
    if (mb < per) break;
    mb -= per;
  }
  if (m >= a.n_mats) return;  // (the grid is rounded up to whole rounds of the XCDs)
  const int fout = a.fout[m], Din = a.Din, f0 = mb * BM;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (NB == 0) {  // chunks through registers (tile_gemm)
    static_assert(KW == 1, "one group");
    const uint16_t* aptr[MT];
    const uint16_t* bptr[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
      aptr[i] = a.w[m] + static_cast<size_t>(min(f0 + i * 32 + (tid >> 3), fout - 1)) * Din + (tid & 7) * 8;
#pragma unroll
    for (int i = 0; i < NT; ++i)
      bptr[i] = a.in + static_cast<size_t>(min(g0 + i * 32 + (tid >> 3), a.T - 1)) * Din + (tid & 7) * 8;
    tile_gemm<MT, NT, 2, false>(aptr, bptr, kd, lds, acc);
  } else {
    uint32_t aoff[MT], boff[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
      aoff[i] = static_cast<uint32_t>(min(i * 32 + (tid >> 3), fout - 1 - f0)) * Din * 2u + tile_piece(tid) * 16u;
#pragma unroll
    for (int i = 0; i < NT; ++i)
      boff[i] = static_cast<uint32_t>(min(i * 32 + (tid >> 3), a.T - 1 - g0)) * Din * 2u + tile_piece(tid) * 16u;
    const uint16_t* abase = uniform_ptr(a.w[m] + static_cast<size_t>(f0) * Din + k0);
    const uint16_t* bbase = uniform_ptr(a.in + static_cast<size_t>(g0) * Din + k0);
    tile_gemm_dma<MT, NT, KW, NB>(abase, bbase, aoff, boff, kd, lds, acc);
  }
  if constexpr (KW > 1) {  // (everybody is done with the buffers)
    float* other = reinterpret_cast<float*>(lds);  // [wave][MT x NT][64 lanes][4]
    if (part == 1) {
#pragma unroll
      for (int t = 0; t < MT * NT; ++t)
        *reinterpret_cast<f32x4*>(other + ((wave * MT * NT + t) * 64 + lane) * 4) = acc[t / NT][t % NT];
    }
    __syncthreads();
    if (part == 1) return;
#pragma unroll
    for (int t = 0; t < MT * NT; ++t) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(other + ((wave * MT * NT + t) * 64 + lane) * 4);
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[t / NT][t % NT][q] += v[q];
    }
  }
  uint16_t* out = a.out[m];
  const uint16_t* res = m == 0 ? a.res : nullptr;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int tok = g0 + (wn * NT + j) * 16 + (lane & 15);
    if (tok >= a.T) continue;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int f = f0 + (wm * MT + i) * 16 + 4 * (lane >> 4);
      if (f >= fout) continue;
      const size_t o = static_cast<size_t>(tok) * fout + f;
      f32x4 r = acc[i][j];
      if (res != nullptr) {
        const u16x4 rv = *reinterpret_cast<const u16x4*>(res + o);
#pragma unroll
        for (int q = 0; q < 4; ++q) r[q] += bf16_bits_to_f32(rv[q]);
      }
      u16x4 ob;
#pragma unroll
      for (int q = 0; q < 4; ++q) ob[q] = f32_to_bf16_bits(r[q]);
      *reinterpret_cast<u16x4*>(out + o) = ob;
    }
  }
}

// The same projection for blocks of at most 32 token rows, where the weights are a pure
// stream and what matters is how many wavefronts pull on it at once: a workgroup owns RT
// 16-row weight tiles, its wavefronts split the reduction dimension (each has a
// contiguous run of every row; the token rows come from L2, each fragment used for the RT
// tiles), and the partial tiles are added through LDS in wavefront order, so the result
// does not depend on timing.  Weight and token rows are both row-major: they are loaded in
// whole 128-byte lines, two stages of four k-steps in flight, and turned into operand order
// through the wavefront's own LDS.  (Loaded in operand order, 64 bytes of 16 rows at a time,
// the q/k/v launch of the 2048-wide layer took 13.7 us, now 10.3; the output 11.8, now 9.2.)
template <int RT, int NT>
__global__ __launch_bounds__(512) void linear_splitk_kernel(LinearArgs a) {
  constexpr int U = 4, kTurn = (RT + NT) * kTurnBytes;
  static_assert(kTurn >= RT * NT * 1024, "a wavefront's partial tiles take the place of its turn buffer");
  __shared__ __align__(16) char s_turn[8 * kTurn];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_waves = blockDim.x >> 6;
  char* turn = s_turn + wave * kTurn;
  const int half = blockIdx.x % a.ksplit, pair_id = blockIdx.x / a.ksplit;
  int grp_i = pair_id, m = 0;
  for (; m < a.n_mats; ++m) {  // which matrix this workgroup belongs to
    const int per = (a.fout[m] / 16 + RT - 1) / RT;
    if (grp_i < per) break;
    grp_i -= per;
  }
  if (m >= a.n_mats) return;
  const int fout = a.fout[m], Din = a.Din;
  const int n_tiles = fout / 16;
  const int kwg = Din / a.ksplit;                   // reduction elements of this workgroup
  const int kper = kwg / n_waves, nks = kper / 32;  // the host makes kper a multiple of 32
  const int k0 = half * kwg + wave * kper;
  const int col = lane & 15, grp = lane >> 4;
  // a load = 8 rows x 64 elements: lane l has piece l % 8 of row l / 8
  const uint16_t* wt[RT];
  const uint16_t* wp[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {  // a tile past the matrix repeats the last one, dropped at the store
    wt[r] = a.w[m] + static_cast<size_t>(min(grp_i * RT + r, n_tiles - 1)) * 16 * Din + k0;
    wp[r] = wt[r] + static_cast<size_t>(lane >> 3) * Din + (lane & 7) * 8;
  }
  const uint16_t* xp[NT][2];
#pragma unroll
  for (int i = 0; i < NT; ++i)  // rows past the block repeat the last token, dropped at the store
#pragma unroll
    for (int q = 0; q < 2; ++q)
      xp[i][q] = a.in + static_cast<size_t>(min(i * 16 + q * 8 + (lane >> 3), a.T - 1)) * Din + k0 + (lane & 7) * 8;
  f32x4 acc[RT][NT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[r][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](const bf16x8 (&w)[RT], const bf16x8 (&x)[NT]) {
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int i = 0; i < NT; ++i) acc[r][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[r], x[i], acc[r][i], 0, 0, 0);
  };
  bf16x8 aw[2][U / 2][RT][2], bx[2][U / 2][NT][2];
  auto load = [&](int st, auto set) {
    constexpr int z = decltype(set)::value;
#pragma unroll
    for (int b = 0; b < U / 2; ++b) {
      const int k = (st * U / 2 + b) * 64;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int r = 0; r < RT; ++r)
          aw[z][b][r][q] = __builtin_nontemporal_load(
              reinterpret_cast<const bf16x8*>(wp[r] + static_cast<size_t>(q) * 8 * Din + k));
#pragma unroll
        for (int i = 0; i < NT; ++i) bx[z][b][i][q] = *reinterpret_cast<const bf16x8*>(xp[i][q] + k);
      }
    }
  };
  auto compute = [&](auto set) {
    constexpr int z = decltype(set)::value;
#pragma unroll
    for (int b = 0; b < U / 2; ++b) {
      turn_fence();
#pragma unroll
      for (int r = 0; r < RT; ++r) turn_write(aw[z][b][r][0], aw[z][b][r][1], turn + r * kTurnBytes, lane);
#pragma unroll
      for (int i = 0; i < NT; ++i) turn_write(bx[z][b][i][0], bx[z][b][i][1], turn + (RT + i) * kTurnBytes, lane);
      turn_fence();
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bf16x8 w[RT], x[NT];
#pragma unroll
        for (int r = 0; r < RT; ++r) w[r] = turn_read(turn + r * kTurnBytes, u, lane);
#pragma unroll
        for (int i = 0; i < NT; ++i) x[i] = turn_read(turn + (RT + i) * kTurnBytes, u, lane);
        multiply(w, x);
      }
    }
  };
  stream_pipeline(nks / U, load, compute);
  for (int ks = nks / U * U; ks < nks; ++ks) {  // k-steps left over by the stages, in operand order
    bf16x8 w[RT], x[NT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
      w[r] = *reinterpret_cast<const bf16x8*>(wt[r] + static_cast<size_t>(col) * Din + ks * 32 + grp * 8);
#pragma unroll
    for (int i = 0; i < NT; ++i)
      x[i] = *reinterpret_cast<const bf16x8*>(a.in + static_cast<size_t>(min(i * 16 + col, a.T - 1)) * Din + k0 +
                                              ks * 32 + grp * 8);
    multiply(w, x);
  }
  // partial tiles: [wave][RT x NT][64 lanes][4], each in its wavefront's part of the LDS
  auto partial = [&](int w, int t) { return reinterpret_cast<float*>(s_turn + w * kTurn) + (t * 64 + lane) * 4; };
  turn_fence();
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int i = 0; i < NT; ++i) *reinterpret_cast<f32x4*>(partial(wave, r * NT + i)) = acc[r][i];
  __syncthreads();
  // wavefront w finishes the tiles w, w + n_waves, ... of the workgroup's RT x NT
  uint16_t* out = a.out[m];
  const uint16_t* res = m == 0 ? a.res : nullptr;
  if (a.ksplit == 2) {
    // Two workgroups share these rows, each with half of the reduction dimension.  Both
    // write their partial tiles with device-scope stores, wait for them, and swap the
    // call's epoch into the pair's flag: the one that gets the epoch back is the second to
    // arrive, and it alone goes on - with both partials read back and added as
    // (first half) + (second half), whoever finished first.  No spinning: nobody waits.
    float* mine = a.partial + static_cast<size_t>(blockIdx.x) * (RT * NT * 256);
    for (int t = wave; t < RT * NT; t += n_waves) {
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
      for (int w = 0; w < n_waves; ++w) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(partial(w, t));
#pragma unroll
        for (int q = 0; q < 4; ++q) sum[q] += v[q];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        __hip_atomic_store(mine + (t * 64 + lane) * 4 + q, sum[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's partials have left the compute unit
    __shared__ int s_second;
    __syncthreads();
    if (tid == 0) {
      const unsigned long long old =
          __hip_atomic_exchange(a.flags + pair_id, a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_second = old == a.epoch ? 1 : 0;
      // the pair is complete: clear the flag, so that a replay of a captured launch (same
      // epoch) starts from a flag nobody has set
      if (old == a.epoch) __hip_atomic_store(a.flags + pair_id, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!s_second) return;
  }
  const float* p0 = a.partial + static_cast<size_t>(pair_id) * 2 * (RT * NT * 256);
  for (int t = wave; t < RT * NT; t += n_waves) {
    const int r = t / NT, i = t % NT;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    if (a.ksplit == 2) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float lo = __hip_atomic_load(p0 + (t * 64 + lane) * 4 + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float hi = __hip_atomic_load(p0 + RT * NT * 256 + (t * 64 + lane) * 4 + q, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
        sum[q] = lo + hi;
      }
    } else {
      for (int w = 0; w < n_waves; ++w) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(partial(w, t));
#pragma unroll
        for (int q = 0; q < 4; ++q) sum[q] += v[q];
      }
    }
    const int tok = i * 16 + col, tile = grp_i * RT + r;
    if (tok < a.T && tile < n_tiles) {
      const size_t o = static_cast<size_t>(tok) * fout + tile * 16 + 4 * grp;
      if (res != nullptr) {
        const u16x4 rv = *reinterpret_cast<const u16x4*>(res + o);
#pragma unroll
        for (int q = 0; q < 4; ++q) sum[q] += bf16_bits_to_f32(rv[q]);
      }
      u16x4 ob;
#pragma unroll
      for (int q = 0; q < 4; ++q) ob[q] = f32_to_bf16_bits(sum[q]);
      *reinterpret_cast<u16x4*>(out + o) = ob;
    }
  }
}

struct AttnArgs {
  const uint16_t *q, *k, *v;           // [T][H*dh], [T][Hkv*dh], [T][Hkv*dh] of the block's own tokens
  const uint16_t *k_cache, *v_cache;   // [B][Hkv][P][dh] cached positions (prefix, then suffix)
  uint16_t* o;                         // [T][H*dh] per-head outputs
  int B, N, H, Hkv, dh, P;
  int splits, tiles;                   // of a workgroup: parts of the window x query tiles (wavefronts)
  int turn;                            // cut window: queries and keys go through LDS into operand order
  float scale;                         // 1 / sqrt(dh)
};

// LDS that the parts of a cut window exchange, after the values: maxima [8 wavefronts][16 queries],
// running sums of the weights [tiles][64 lanes], the weights of two parts [2][tiles][steps][64 lanes][8]
// (before the weights, the same place may turn the wavefronts' keys into operand order).
__host__ __device__ constexpr size_t exchange_bytes(int tiles, int steps_of_part) {
  return 512 + tiles * 256 + 2 * static_cast<size_t>(tiles) * steps_of_part * 1024;
}

// How the work of one (sequence, key/value head) is cut.  Its query rows - the block's
// tokens under each query head that shares the keys - form tiles of 16; a wavefront takes
// one tile and one part of the window, a workgroup up to eight wavefronts that share the
// transposed values in LDS.  A window whose scores fit a wavefront's registers is not cut.
// A longer window is cut until the scores of a part fit, and further while
// the launch has fewer than 2048 wavefronts (eight per compute unit), as long as a part keeps
// 64 positions (what a wavefront requests at once anyway); then the tiles are spread over more
// workgroups until every compute unit has one (each stages the values again, from L2).
// Where workgroups full of tiles cover the compute units already, cutting only stages the values
// more often (64 sequences of 32 tokens, 32 heads on 4 of width 128): up to 512 positions stay
// whole, half the keys requested ahead (496: 102 us, cut 169 us); beyond that, if the values
// leave a compute unit one workgroup anyway, the scores are computed twice (576: 157 us, cut 287
// us).  So they are where no cut into at most eight parts fits (windows beyond 2048).
constexpr int kWholeWindow = 256;  // positions whose scores a wavefront keeps in registers
constexpr int kWideWindow = 512;   // ... if it requests half as many keys ahead
//
// Queries and keys of 128-wide heads under a cut window are loaded along their rows and turned into operand
// order (`turn`) where four wavefronts or more share a compute unit: there their loads in operand order
// queue up (see operand_write).  Eight sequences over 496 positions 19.3 -> 16.3 us, 128 tokens over 568 16.0
// -> 14.2, 30 x 17 over 457 49.4 -> 42.4.  With fewer the way through LDS is what counts (one block over 272
// positions, 256 wavefronts: 11.4 and 11.9; whole windows: 64 positions 6.0 and 6.4, 16 x 128 over 528 level),
// and so it is for other widths (104: 30 launches over 272 to 640 positions take 3 to 12 % longer; 96, 30 x 17:
// 26.6 and 27.9; 64: 16.6 and 20.0) and for few query tiles per key/value head, where the keys come from memory:
// one or two (16 heads on 16, 16 x 16 over 416: 15.2 and 16.1; 30 x 17 over 457: 39.6 and 40.5), and four to
// seven above 48 MB of keys and values (32 heads on 8: 32 x 16 over 400, 52 MB, 33.0 and 34.4; 24 x 16 over 480,
// 47 MB, 34.7 and 32.0).
struct AttnPlan { int splits, tiles, groups; size_t lds; bool turn; };
static AttnPlan attn_plan(const AttnArgs& a, size_t value_bytes) {
  const int rows = a.H / a.Hkv * a.N, tiles = (rows + 15) / 16, steps = (a.P + a.N + 31) / 32;
  const int heads = a.B * a.Hkv;
  AttnPlan p{1, 8, 1, value_bytes, false};
  auto part = [&]() { return (steps + p.splits - 1) / p.splits; };  // steps of a part
  auto spread = [&]() {
    p.tiles = 8 / p.splits;
    while (p.tiles > 1 && heads * ((tiles + p.tiles - 1) / p.tiles) < 256) p.tiles /= 2;
    if (p.tiles > tiles) p.tiles = tiles;
  };
  auto fits = [&]() {
    return part() * 32 <= kWholeWindow && value_bytes + exchange_bytes(p.tiles, part()) <= 160 * 1024;
  };
  const bool full = tiles >= 8 && heads * ((tiles + 7) / 8) >= 256;
  const bool whole = a.P + a.N <= (full ? kWideWindow : kWholeWindow) || (full && value_bytes > 80 * 1024);
  if (!whole) {
    p.splits = 2;
    spread();
    while (p.splits < 8 && (!fits() || (4 * p.splits <= steps && heads * tiles * p.splits < 2048))) {
      p.splits *= 2;
      spread();
    }
    if (!fits()) p.splits = 1;
  }
  spread();
  if (p.splits > 1) p.lds += exchange_bytes(p.tiles, part());
  p.groups = (tiles + p.tiles - 1) / p.tiles;
  const int query_tiles = p.groups * p.tiles, waves = p.splits * p.tiles;
  const size_t with_turn = value_bytes + 512 + p.tiles * 256 + (waves < 4 ? 4 : waves) * kOperandBytes;
  const size_t window_bytes = static_cast<size_t>(heads) * (a.P + a.N) * a.dh * 4;  // keys and values
  p.turn = p.splits > 1 && a.dh == 128 && heads * query_tiles * p.splits >= 1024 &&
           (query_tiles >= 8 || (query_tiles >= 4 && window_bytes <= (48u << 20))) && with_turn <= 160 * 1024;
  if (p.turn && with_turn > p.lds) p.lds = with_turn;
  return p;
}

// Both contractions are bf16 MFMA with fp32 accumulation, laid out so that no operand
// needs a transpose between them:
//   S^T = K Q^T    A = keys (16 per tile, straight from global memory), B = the 16 queries
//                  -> lane l holds query l % 16, keys 4 (l / 16) .. + 3 of the tile
//   O^T = V^T P^T  B = the weights of two score tiles as they sit in those registers (the
//                  contraction only needs A and B to agree on which key a slot means),
//                  A = values transposed in LDS, read with that same key order
//                  -> lane l holds query l % 16, coordinates 4 (l / 16) .. + 3 of the tile
// The maximum of the whole window comes first, the weights after it; all sums run over the
// window in order, whatever the cut, so a query's result does not depend on how many others
// the launch has.  Keys are read 64 at a time with the next 128 requested ahead.  Forms:
//   kWhole  up to 256 positions: one wavefront per tile, all scores stay in registers;
//   kWide   the same up to 512 positions, half as many keys requested ahead;
//   kParts  the wavefronts of a tile score their parts of the window, exchange their maxima and
//           form their weights side by side.  The weights then pass through LDS part after part;
//           each wavefront adds up its share of the coordinates over the whole window;
//   kTwice  one wavefront per tile, the scores computed twice.
// Weights are rounded to bf16 for the second contraction, their sum is kept in fp32.
// What bounds it is latency - the loads behind one another, then the staging of the
// values: eight sequences of 32 tokens over 496 positions, 32 heads on 4, take 16.3 us
// (one workgroup per query head, half of its wavefronts idle, scores computed twice and
// values transposed two bytes at a time: 49.6 us); one block over 64 positions 5.3 us.
// A running maximum with the parts added up at the end was 1.6 us faster, but then the
// rounding of the weights depends on the cut, and a part whose scores are all -inf has none.
// NKS = 32-element steps of the head width.
typedef short i16x4 __attribute__((ext_vector_type(4)));
enum AttnForm { kWhole, kWide, kParts, kTwice };
template <int NKS, int FORM, bool ROWS>
__global__ __launch_bounds__(512) void attention_core_kernel(AttnArgs a) {
  constexpr int NDT = 2 * NKS;
  // Queries and keys of 128-wide heads under a cut window may be loaded along their rows (a.turn)
  const bool along = FORM == kParts && NKS == 4 && ROWS && a.turn;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  uint16_t* vt = reinterpret_cast<uint16_t*>(smem_raw);  // [ndt * 16][ldv]: values, transposed (unless ROWS)
  const int N = a.N, dh = a.dh, P = a.P, nk = a.P + a.N;
  const int nkp = (nk + 31) & ~31, ldv = nkp + 4, steps = nkp / 32;
  const int ndt = (dh + 15) / 16;
  const int tid = threadIdx.x, lane = tid & 63, n_threads = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x / a.Hkv, g = blockIdx.x % a.Hkv;
  const int rep = a.H / a.Hkv, rows = rep * N;
  const int S = a.splits, part = wave % S;
  const size_t cbase = (static_cast<size_t>(b) * a.Hkv + g) * P * dh;
  const uint16_t* kc = a.k_cache + cbase;  // cached keys / values of this head (unused if P == 0)
  const uint16_t* vc = a.v_cache + cbase;
  const size_t brow = static_cast<size_t>(b) * N * a.Hkv * dh + static_cast<size_t>(g) * dh;
  const uint16_t* kb = a.k + brow;         // the block's own keys / values, row stride Hkv * dh
  const uint16_t* vb = a.v + brow;
  const int bstride = a.Hkv * dh;
  const int col = lane & 15, grp = lane >> 4;
  const float neg_inf = -__builtin_inff();
  auto row_of = [&](const uint16_t* cache, const uint16_t* block, int j) -> const uint16_t* {
    return j < P ? cache + static_cast<size_t>(j) * dh : block + static_cast<size_t>(j - P) * bstride;
  };
  const int lrow = along ? lane >> 2 : col, lpiece = along ? lane & 3 : grp;  // of a 16 x 32 operand, loading
  char* turn = reinterpret_cast<char*>(smem_raw) + static_cast<size_t>(ndt) * 16 * ldv * 2 +
               512 + a.tiles * 256 + wave * kOperandBytes;  // (in the place of the ring)
  auto load8 = [&](const uint16_t* row, int s) -> bf16x8 {  // elements 32 s + 8 lpiece .. + 7, zeros past dh
    const int e = 32 * s + 8 * lpiece;
    uint4 raw = make_uint4(0u, 0u, 0u, 0u);
    if (e < dh) raw = *reinterpret_cast<const uint4*>(row + e);
    return __builtin_bit_cast(bf16x8, raw);
  };
  // this lane's query row (rows past the last repeat it and are not stored)
  const int row0 = (blockIdx.y * a.tiles + wave / S) * 16, row = row0 + col;
  auto query_off = [&](int r) {
    r = min(r, rows - 1);
    return (static_cast<size_t>(b) * N + r % N) * (a.H * dh) + static_cast<size_t>(g * rep + r / N) * dh;
  };
  bf16x8 qf[NKS];
  {
    const uint16_t* q = a.q + query_off(row0 + lrow);
#pragma unroll
    for (int s = 0; s < NKS; ++s) qf[s] = load8(q, s);
  }
  // this wavefront's part of the window, in steps of 32 positions
  const int per = (steps + S - 1) / S;
  const int s0 = min(part * per, steps), s1 = wave < S * a.tiles ? min(s0 + per, steps) : s0;
  constexpr int KT = FORM == kWide ? 2 : 4, KS = KT / 2;  // key tiles requested together; steps of them
  bf16x8 kf[2][KT][NKS];
  auto load_keys = [&](int st, auto set) {  // KT key tiles (KS steps); tiles past the part are skipped
    constexpr int z = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < KT; ++i) {
      const uint16_t* krow = row_of(kc, kb, min(32 * st + 16 * i + lrow, nk - 1));
#pragma unroll
      for (int s = 0; s < NKS; ++s) kf[z][i][s] = st + i / 2 < s1 ? load8(krow, s) : bf16x8{};
    }
  };
  if (s0 < s1) load_keys(s0, S0{});
  if (s0 + KS < s1) load_keys(s0 + KS, S1{});

  // ROWS (heads of 64 or 128): the values lie in LDS as rows, brought there by direct loads while the
  // scores are computed, and the transposing LDS read turns four positions x 16 coordinates into the
  // operand.  Rows of kRow bytes, the 32-byte segment g of row r at g ^ value_swizzle(r): the 16 rows
  // of an operand read spread over all banks.  (Through registers, transposed 8 bytes at a time, the
  // staging was a phase of its own with conflicts in its LDS writes: 8 sequences over 496 positions,
  // 22.1 us; so, and with the operands of the weights formed outside the turns below, 19.6.)
  constexpr int kRow = ROWS ? NKS * 64 : 256, kPieces = kRow / 16;
  auto value_swizzle = [](int r) { return kRow == 256 ? (r & 7) : ((r >> 1) & 3); };
  if constexpr (ROWS) {
    constexpr int kRows = 1024 / kRow;  // of one direct load
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<size_t>(DES_LDS_PTR(smem_raw)));
    const int sub = lane / kPieces, p = lane % kPieces, n_waves = n_threads >> 6;
    for (int i = wave; i < nkp / kRows; i += n_waves) {
      const int j = i * kRows + sub;
      if (j < nk) {
        const uint16_t* src = row_of(vc, vb, j) + (p ^ (value_swizzle(j) << 1)) * 8;
        // (the wait state between the write of M0 and the load, see dma_stream_gemm)
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds0 + i * 1024)
                     : "m0");
      } else {  // slots beyond the window hold zeros (their weights are zero too, but 0 x garbage could be NaN)
        *reinterpret_cast<uint4*>(smem_raw + i * 1024 + lane * 16) = make_uint4(0u, 0u, 0u, 0u);
      }
    }
  } else
  // values -> LDS, transposed: a thread takes 8 coordinates of 4 consecutive positions and
  // writes 8 bytes per coordinate.  Slots beyond the window hold zeros.
  {
    const int vec = dh / 8, n_piece = nkp / 4 * vec;
    auto fetch = [&](int i, uint4 (&raw)[4]) {
      const int j = i / vec * 4, c = (i % vec) * 8;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        raw[q] = (i < n_piece && j + q < nk) ? *reinterpret_cast<const uint4*>(row_of(vc, vb, j + q) + c)
                                             : make_uint4(0u, 0u, 0u, 0u);
    };
    auto put = [&](int i, const uint4 (&raw)[4]) {
      if (i >= n_piece) return;
      uint16_t* dst = vt + (i % vec) * 8 * ldv + i / vec * 4;
      const uint32_t w[4][4] = {{raw[0].x, raw[1].x, raw[2].x, raw[3].x}, {raw[0].y, raw[1].y, raw[2].y, raw[3].y},
                                {raw[0].z, raw[1].z, raw[2].z, raw[3].z}, {raw[0].w, raw[1].w, raw[2].w, raw[3].w}};
#pragma unroll
      for (int q = 0; q < 4; ++q) {  // coordinates 2q (low halves) and 2q + 1 (high halves)
        *reinterpret_cast<uint2*>(dst + 2 * q * ldv) =
            make_uint2((w[q][0] & 0xffffu) | (w[q][1] << 16), (w[q][2] & 0xffffu) | (w[q][3] << 16));
        *reinterpret_cast<uint2*>(dst + (2 * q + 1) * ldv) =
            make_uint2((w[q][0] >> 16) | (w[q][1] & 0xffff0000u), (w[q][2] >> 16) | (w[q][3] & 0xffff0000u));
      }
    };
    for (int i = tid; i < n_piece; i += 2 * n_threads) {
      uint4 r0[4], r1[4];
      fetch(i, r0);
      fetch(i + n_threads, r1);
      put(i, r0);
      put(i + n_threads, r1);
    }
  }
  // the values are there (direct loads: the compiler does not know of them)
  auto values_ready = [&]() {
    if (ROWS) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  if (!ROWS) values_ready();

  if (FORM != kParts && wave >= a.tiles) {  // it only helped with the values
    if (ROWS) values_ready();
    return;
  }
  float mx = neg_inf, lsum = 0.f;
  f32x4 oacc[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt) oacc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (along) {
#pragma unroll
    for (int s = 0; s < NKS; ++s) qf[s] = operand_turn(qf[s], turn, lane);
  }
  // positions of this lane from step st on that count: inside the window and inside the part
  auto limit = [&](int st) { return min(nk, 32 * s1) - (32 * st + 4 * grp); };
  // scores of the key tiles of a set; the maximum takes them in
  auto scores = [&](int st, auto set, f32x4* sc) {
    constexpr int z = decltype(set)::value;
    if (along) {
#pragma unroll
      for (int i = 0; i < KT; ++i)
#pragma unroll
        for (int s = 0; s < NKS; ++s) kf[z][i][s] = operand_turn(kf[z][i][s], turn, lane);
    }
#pragma unroll
    for (int i = 0; i < KT; ++i) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NKS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[z][i][s], qf[s], acc, 0, 0, 0);
      sc[i] = acc;
    }
    const int lim = limit(st);
#pragma unroll
    for (int i = 0; i < KT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = 16 * i + r < lim ? fmaxf(mx, sc[i][r]) : mx;
  };
  auto query_max = [&]() {  // over the lanes that hold a query's scores
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
  };
  // the weights of step st from the scores of its two tiles
  auto form = [&](int st, const f32x4* sc, f32x4 (&w)[2]) {
    const int lim = limit(st);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) w[i][r] = 16 * i + r < lim ? expf((sc[i][r] - mx) * a.scale) : 0.f;
  };
  // ... into their sum, and as an operand (the pack rounds to nearest even, like f32_to_bf16_bits)
  auto add_to_sum = [&](const f32x4 (&w)[2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) lsum += w[i][r];
  };
  auto operand = [&](const f32x4 (&w)[2]) -> bf16x8 {
    return __builtin_convertvector(__builtin_shufflevector(w[0], w[1], 0, 1, 2, 3, 4, 5, 6, 7), bf16x8);
  };
  auto add_values = [&](int st, int dt, const bf16x8& pb, f32x4& o) {  // coordinates 16 dt .. + 15 of step st
    struct { u16x4 lo, hi; } vv;
    if constexpr (ROWS) {
      typedef __attribute__((address_space(3))) i16x4 LdsI16x4;
      // lanes 4 i .. 4 i + 3 of 16 address position i's 16 coordinates; a lane gets four positions of its own
      const int j = 32 * st + 4 * grp + (col >> 2);  // (16 rows on: the same swizzle)
      unsigned char* at = smem_raw + j * kRow + ((dt ^ value_swizzle(j)) << 5) + (col & 3) * 8;
      vv.lo = __builtin_bit_cast(u16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsI16x4*)DES_LDS_PTR(at)));
      vv.hi = __builtin_bit_cast(u16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsI16x4*)DES_LDS_PTR(at + 16 * kRow)));
    } else {
      const uint16_t* vrow = vt + (16 * dt + col) * ldv + 32 * st + 4 * grp;
      vv.lo = *reinterpret_cast<const u16x4*>(vrow);
      vv.hi = *reinterpret_cast<const u16x4*>(vrow + 16);
    }
    o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vv), pb, o, 0, 0, 0);
  };
  auto weigh = [&](int st, const f32x4* sc) __attribute__((always_inline)) {  // the steps of a set, all coordinates
#pragma unroll
    for (int c = 0; c < KS; ++c) {
      if (st + c < s1) {
        f32x4 w[2];
        form(st + c, sc + 2 * c, w);
        add_to_sum(w);
        const bf16x8 pb = operand(w);
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
          if (dt < ndt) add_values(st + c, dt, pb, oacc[dt]);
      }
    }
  };
  uint16_t* orow = a.o + query_off(row);
  auto store = [&](int dt, const f32x4& o, float inv) {
    const int d0 = 16 * dt + 4 * grp;
    if (row < rows && d0 < dh) {
      u16x4 ob;
#pragma unroll
      for (int r = 0; r < 4; ++r) ob[r] = f32_to_bf16_bits(o[r] * inv);
      *reinterpret_cast<u16x4*>(orow + d0) = ob;
    }
  };
  if constexpr (FORM == kTwice) {
    auto walk = [&](auto&& f) {  // the keys, 64 at a time: f(first step, scores)
      f32x4 sc[KT];
      for (int st = 0; st < s1; st += 2 * KS) {
        scores(st, S0{}, sc);
        if (st + 2 * KS < s1) load_keys(st + 2 * KS, S0{});
        f(st, sc);
        if (st + KS < s1) {
          scores(st + KS, S1{}, sc);
          if (st + 3 * KS < s1) load_keys(st + 3 * KS, S1{});
          f(st + KS, sc);
        }
      }
    };
    walk([](int, const f32x4*) {});
    if (ROWS) values_ready();
    query_max();
    load_keys(0, S0{});
    load_keys(KS, S1{});
    walk(weigh);
  } else {
    constexpr int kSets = (FORM == kWide ? kWideWindow : kWholeWindow) / (16 * KT);
    f32x4 sc[kSets][KT];
    static_for(std::make_integer_sequence<int, kSets>{}, [&](auto i) {
      constexpr int I = decltype(i)::value;
      typedef std::integral_constant<int, I & 1> Set;
      const int st = s0 + KS * I;
      if (st < s1) scores(st, Set{}, sc[I]);
      if (st + 2 * KS < s1) load_keys(st + 2 * KS, Set{});
    });
    query_max();
    if (ROWS && FORM != kParts) values_ready();
    if constexpr (FORM != kParts) {
      static_for(std::make_integer_sequence<int, kSets>{}, [&](auto i) {
        constexpr int I = decltype(i)::value;
        if (KS * I < s1) weigh(KS * I, sc[I]);
      });
    } else {
      const int q = wave / S;  // this wavefront's tile, if below a.tiles
      const bool busy = q < a.tiles;
      char* after = reinterpret_cast<char*>(smem_raw) + static_cast<size_t>(ndt) * 16 * ldv * 2;
      float* part_max = reinterpret_cast<float*>(after);        // (see exchange_bytes)
      float* part_sum = reinterpret_cast<float*>(after + 512) + (busy ? q : 0) * 64 + lane;
      uint16_t* ring = reinterpret_cast<uint16_t*>(after + 512 + a.tiles * 256) + lane * 8;
      if (grp == 0) part_max[wave * 16 + col] = mx;
      values_ready();
      for (int p = 0; p < S; ++p) mx = fmaxf(mx, part_max[(wave - part + p) * 16 + col]);
      constexpr int kSteps = kWholeWindow / 32;
      f32x4 w[kSteps][2];
      bf16x8 wp[kSteps];  // (all parts form theirs side by side, a turn below only adds them up)
      static_for(std::make_integer_sequence<int, kSteps>{}, [&](auto i) {
        constexpr int I = decltype(i)::value;
        if (s0 + I < s1) {
          form(s0 + I, &sc[I / 2][I % 2 * 2], w[I]);
          wp[I] = operand(w[I]);
        }
      });
      // Turn p: the weights of part p meet the values, those of part p + 1 are put in place and added
      // to the sum (the ring holds two parts; a turn's barrier separates its uses).
      constexpr int kShare = NDT / 2;  // coordinate tiles of a wavefront: part, part + S, ...
      for (int p = -1; p < S; ++p) {
        if (busy && part == p + 1) {
          if (p >= 0) lsum = *part_sum;
          uint16_t* dst = ring + ((part & 1) * a.tiles + q) * per * 512;
          static_for(std::make_integer_sequence<int, kSteps>{}, [&](auto i) {
            constexpr int I = decltype(i)::value;
            if (s0 + I < s1) {
              *reinterpret_cast<bf16x8*>(dst + I * 512) = wp[I];
              add_to_sum(w[I]);
            }
          });
          *part_sum = lsum;
        }
        if (busy && p >= 0) {
          const uint16_t* src = ring + ((p & 1) * a.tiles + q) * per * 512;
          const int first = p * per, last = min(first + per, steps);
          for (int st = first; st < last; ++st) {
            const bf16x8 pb = *reinterpret_cast<const bf16x8*>(src + (st - first) * 512);
#pragma unroll
            for (int i = 0; i < kShare; ++i)
              if (part + i * S < ndt) add_values(st, part + i * S, pb, oacc[i]);
          }
        }
        if (p < S - 1) __syncthreads();
      }
      if (!busy) return;
      lsum = *part_sum;  // (complete since the turn before the last)
    }
  }
  lsum += __shfl_xor(lsum, 16);
  lsum += __shfl_xor(lsum, 32);
  const float inv = 1.0f / lsum;
#pragma unroll
  for (int dt = 0; dt < (FORM == kParts ? NDT / 2 : NDT); ++dt) store(FORM == kParts ? part + dt * S : dt, oacc[dt], inv);
}

// Blocks of more than 32 token rows: is the reduction cut in two?  Where a launch of one
// workgroup per 64 weight rows and 128 (64 if that makes fewer than 100) token rows has fewer
// than 150: half of the compute units would have four wavefronts or none (2048 x 4096 weights
// on 256 token rows: 20.5 us whole, 17.0 us cut).  The cut decides the order of the sums, so it
// depends on sizes alone.
struct LongCut { int workgroups; bool cut; };
static LongCut long_cut(int T, const int* fout, int n_mats, int Din) {
  int b64 = 0;
  for (int m = 0; m < n_mats; ++m) b64 += (fout[m] / 32 + 1) / 2;
  const int rows = b64 * ((T + 127) / 128) < 100 ? 64 : 128;
  const int workgroups = b64 * ((T + rows - 1) / rows);
  return LongCut{workgroups, workgroups < 150 && Din % 512 == 0};
}

// The tile of such a block (32 mt weight rows x 32 nt token rows) and its number of workgroups.
//
// A launch is bound by what a compute unit can pull into its LDS: (mt + nt) x 32 rows of the reduction
// per tile, for as many tiles as the fullest unit has.  Small tiles spread over all units, large ones
// reload less.  Measured in two states, because a layer's weights come from memory in a model (the
// experts of the layer before have streamed through the last-level cache) and from that cache when one
// layer is called again: 13 pairs of widths x 29 batches of 33 to 4096 rows, both projections, every
// tile; the second of two figures is with the cache flushed.  Chunks that pass through registers (64 x
// 64 or 128 x 128) were the only form once; against them the launches take 17 % and 12 % less, at most
// 6 % and 16 % longer, and 1.7 % longer than in the best of the tiles (2048 x 4096 weights, 256 rows:
// 17.0 / 21.0 us, now 13.5 / 17.3; 1024 rows 32.5 / 35.2, now 26.8 / 37.2).
//
// Where 128 x 128 tiles fill the units they are the best, in one of two forms.  Straight into LDS, one
// chunk ahead: two tiles share a unit and hide each other's waits, so an even number of tiles per unit
// takes 19 % and 9 % less than in registers (2048 x 4096 weights, 4096 rows: 67.7 / 80.5 us against 84.0
// / 85.3).  With an odd number the last tile waits alone for every chunk, which costs more the further
// away the weights are (6144 x 2048, 1760 rows, three tiles: 53.8 / 69.4 against 60.9 / 63.4; 4096 x
// 4096, 1024 rows, one: 47.3 / 61.2 against 49.4 / 51.0): through registers, two chunks ahead.  So do
// launches of more than eight tiles per unit (level, and 17 % longer where 18 fill their rounds) and
// reductions beyond 8192 (16384: 466 against 324).
//
// Else the cheapest by the relative times below, per row and tile on one unit: tiles side by side on a
// unit overlap, so a second one costs a third, a third one and more about their own time; two groups of
// 64 x 64 or more take a unit's LDS for themselves, a second such tile comes after the first.
struct TileLinearPlan { int mt, nt, blocks, kw; bool regs; };
static TileLinearPlan tile_linear_plan(int T, const int* fout, int n_mats, int Din) {
  const int kw = long_cut(T, fout, n_mats, Din).cut ? 2 : 1;
  constexpr int kTiles[][2] = {{4, 4}, {4, 2}, {2, 2}, {2, 1}, {1, 1}};
  auto blocks = [&](int mt, int nt) {
    int b = 0;
    for (int m = 0; m < n_mats; ++m) b += (fout[m] + 32 * mt - 1) / (32 * mt);
    return (b + 7) / 8 * 8 * ((T + 32 * nt - 1) / (32 * nt));
  };
  // (filled: two tiles per unit, or, where a tile is long enough to pay for its start, one, if the last
  // round of units is at least two thirds full)
  if (const int b4 = blocks(4, 4), k = (b4 + 255) / 256;
      kw == 1 && (b4 >= 512 || (Din >= 2048 && b4 >= 256 && 2 * 256 * k <= 3 * b4)))
    return TileLinearPlan{4, 4, b4, 1, k % 2 != 0 || k > 8 || Din > 8192};
  TileLinearPlan best{0, 0, 0, kw, false};
  long best_cost = 0;
  for (const auto& t : kTiles) {
    const int mt = t[0], nt = t[1];
    if (mt * nt == 16 && kw == 2) continue;  // (15 % longer at best)
    const int b = blocks(mt, nt);
    const long k = (b + 255) / 256;  // tiles of the fullest compute unit
    const long unit = kw == 2         ? (mt * nt >= 4 && k > 1 ? 400 * k : 270 * k + 10)
                      : mt * nt == 16 ? (k == 1 ? 250 : k == 2 ? 330 : 205 * k)
                      : mt * nt == 8  ? (k == 1 ? 210 : k == 2 ? 280 : 155 * k)
                                      : (k == 1 ? 190 : k == 2 ? (mt > nt ? 256 : 247) : 140 * k + 20);
    const long cost = unit * (mt + nt);
    if (best.mt == 0 || cost < best_cost) {
      best = TileLinearPlan{mt, nt, b, kw, false};
      best_cost = cost;
    }
  }
  return best;
}

// of one half of a cut reduction: 4 weight tiles x up to 8 token tiles x 1 KB
constexpr size_t kLongPartialBytes = 4 * 8 * 1024;

// Scratch of one attention sub-layer (bytes from a 256-byte aligned base): q, k, v and the
// per-head outputs of the block's tokens, bf16.
AttnLayout attn_layout(const des_shape_t& s, const des_attn_shape_t& t) {
  const size_t T = static_cast<size_t>(s.n_seqs) * s.n_tokens;
  AttnLayout l;
  size_t p = 0;
  l.q = p; p = align256(p + 2 * T * t.n_heads * t.head_dim);
  l.k = p; p = align256(p + 2 * T * t.n_kv_heads * t.head_dim);
  l.v = p; p = align256(p + 2 * T * t.n_kv_heads * t.head_dim);
  l.o = p; p = align256(p + 2 * T * t.n_heads * t.head_dim);
  // short blocks, reduction split over two workgroups: fp32 partial tiles (two halves x two
  // token tiles x 1 KB per 16-row weight tile) and one flag per 16 rows, for the larger of
  // the two projection launches (they run one after the other)
  const size_t tiles_qkv = static_cast<size_t>(t.n_heads + 2 * t.n_kv_heads) * t.head_dim / 16;
  const size_t tiles_out = static_cast<size_t>(s.hidden) / 16;
  const size_t tiles = tiles_qkv > tiles_out ? tiles_qkv : tiles_out;
  size_t part_bytes = tiles * 4096, n_flags = tiles;
  if (T > 32) {
    // Longer blocks need none (the halves of a cut reduction meet in LDS), but the size is part
    // of the interface: a caller keeps one buffer for its longest block and the remainders after
    // it, which do.  So it stays at 32 KB for each half of a workgroup's cut reduction and a flag
    // per workgroup (2048-wide layer, 32 heads: 5.85 MB at 33 tokens, 1.90 MB at 32).
    const int f_qkv[3] = {t.n_heads * t.head_dim, t.n_kv_heads * t.head_dim, t.n_kv_heads * t.head_dim};
    const int f_out[1] = {s.hidden};
    const LongCut a = long_cut(static_cast<int>(T), f_qkv, 3, s.hidden);
    const LongCut b = long_cut(static_cast<int>(T), f_out, 1, t.n_heads * t.head_dim);
    const size_t wa = a.workgroups, wb = b.workgroups;
    const size_t pa = a.cut ? wa * 2 * kLongPartialBytes : 0, pb = b.cut ? wb * 2 * kLongPartialBytes : 0;
    part_bytes = pa > pb ? pa : pb;
    n_flags = wa > wb ? wa : wb;
  }
  l.partial = p; p = align256(p + part_bytes);
  l.flags = p; p = align256(p + n_flags * 8);
  l.total = p;
  return l;
}

void projection_plan(const des_shape_t& s, const des_attn_shape_t& t, bool output, int32_t* plan) {
  const int T = s.n_seqs * s.n_tokens, HD = t.n_heads * t.head_dim, KD = t.n_kv_heads * t.head_dim;
  const int f_qkv[3] = {HD, KD, KD}, f_out[1] = {s.hidden};
  plan[0] = plan[1] = plan[2] = plan[3] = 0;
  if (T <= 32) return;
  const TileLinearPlan p = output ? tile_linear_plan(T, f_out, 1, HD) : tile_linear_plan(T, f_qkv, 3, s.hidden);
  plan[0] = p.mt; plan[1] = p.nt; plan[2] = p.kw; plan[3] = p.regs;
}

size_t attn_core_lds(const des_shape_t& s, const des_attn_shape_t& t) {
  // the head's values, transposed: (dh rounded up to 16) rows of (window rounded up to 32) + 4 bf16
  const size_t nk = static_cast<size_t>(attn_cached(t)) + s.n_tokens;
  const size_t nkp = (nk + 31) / 32 * 32;
  return static_cast<size_t>((t.head_dim + 15) / 16 * 16) * (nkp + 4) * 2;
}

static void launch_linear(const LinearArgs& a, int kernel_id, hipStream_t st) {
  if (a.T <= 32) {
    // Row tiles per workgroup: two halve the token-row traffic from L2, which costs as much
    // as the weight stream here (q/k/v of the 2048-wide layer, 320 tiles, 32 rows: 8.4 us
    // against 11.2 us with one), but only while the workgroups still cover most compute units
    // (its output projection, 128 tiles: 8.1 us with one, 9.2 us with two; 256 tiles of 2048:
    // 7.1 and 9.4 us).
    // Fewer than 150 workgroups: the reduction dimension is split over two workgroups as
    // well (the output projection 9.1 -> 8.1 us; q/k/v with 160 workgroups would take 11.9 us
    // instead of 8.4).  At 1024 x 1024 the exchange of partial tiles costs more than the spread
    // gains (4.2 us whole, 5.2 us split): the split stays there because it decides the order of
    // the sums.  (Times with the weights in the last-level cache.)
    // Wavefronts per workgroup (k-slices): a whole number of 32-element steps each, at
    // least 256 reduction elements per row, at most 8.
    int tiles = 0;
    for (int m = 0; m < a.n_mats; ++m) tiles += a.fout[m] / 16;
    const bool two = tiles >= 2 * 150;
    int groups = 0;
    for (int m = 0; m < a.n_mats; ++m) groups += two ? (a.fout[m] / 16 + 1) / 2 : a.fout[m] / 16;
    LinearArgs b = a;
    b.ksplit = (groups < 150 && a.Din % 64 == 0 && a.Din >= 1024 && b.partial != nullptr) ? 2 : 1;
    const int kwg = a.Din / b.ksplit;
    int nw = 8;
    while (nw > 1 && (kwg % (32 * nw) != 0 || kwg / nw < 256)) nw >>= 1;
    const dim3 g(groups * b.ksplit), blk(nw * kWave);
    if (two) {
      if (a.T <= 16) launch(kernel_id, linear_splitk_kernel<2, 1>, g, blk, 0, st, b);
      else launch(kernel_id, linear_splitk_kernel<2, 2>, g, blk, 0, st, b);
    } else {
      if (a.T <= 16) launch(kernel_id, linear_splitk_kernel<1, 1>, g, blk, 0, st, b);
      else launch(kernel_id, linear_splitk_kernel<1, 2>, g, blk, 0, st, b);
    }
    return;
  }
  const TileLinearPlan pl = tile_linear_plan(a.T, a.fout, a.n_mats, a.Din);
  const dim3 g(pl.blocks), b(256 * pl.kw);
  // (buffers of a chunk: three, two for the largest tile so that two workgroups share a compute unit)
  auto pick = [&](auto kernel1, auto kernel2) { launch(kernel_id, pl.kw == 2 ? kernel2 : kernel1, g, b, 0, st, a); };
  if (pl.regs) launch(kernel_id, linear_tile_kernel<4, 4, 1, 0>, g, b, 0, st, a);
  else if (pl.nt == 4) launch(kernel_id, linear_tile_kernel<4, 4, 1, 2>, g, b, 0, st, a);
  else if (pl.mt == 4) pick(linear_tile_kernel<4, 2, 1, 3>, linear_tile_kernel<4, 2, 2, 3>);
  else if (pl.nt == 2) pick(linear_tile_kernel<2, 2, 1, 3>, linear_tile_kernel<2, 2, 2, 3>);
  else if (pl.mt == 2) pick(linear_tile_kernel<2, 1, 1, 3>, linear_tile_kernel<2, 1, 2, 3>);
  else pick(linear_tile_kernel<1, 1, 1, 3>, linear_tile_kernel<1, 1, 2, 3>);
}

static AttnArgs core_args(const des_shape_t& s, const des_attn_shape_t& t) {  // (sizes only)
  AttnArgs c{};
  c.B = s.n_seqs; c.N = s.n_tokens; c.H = t.n_heads; c.Hkv = t.n_kv_heads; c.dh = t.head_dim;
  c.P = attn_cached(t);
  return c;
}

void core_plan(const des_shape_t& s, const des_attn_shape_t& t, bool sizes, int32_t* plan) {
  const AttnPlan p = attn_plan(core_args(s, t), attn_core_lds(s, t));
  plan[0] = sizes ? static_cast<int32_t>(p.lds) : p.splits;
  plan[1] = sizes ? static_cast<int32_t>(attn_core_lds(s, t)) : p.tiles;
  plan[2] = sizes ? 0 : p.groups;
  plan[3] = sizes ? 0 : p.turn;
}

int launch_attention(const des_shape_t& s, const des_attn_shape_t& t, const void* x, const void* wq,
                     const void* wk, const void* wv, const void* wo, const void* k_cache,
                     const void* v_cache, void* y, char* ws, unsigned long long epoch, hipStream_t st) {
  const AttnLayout l = attn_layout(s, t);
  const int T = s.n_seqs * s.n_tokens;
  const int HD = t.n_heads * t.head_dim, KD_ = t.n_kv_heads * t.head_dim;
  LinearArgs p{};
  p.in = static_cast<const uint16_t*>(x);
  p.w[0] = static_cast<const uint16_t*>(wq);
  p.w[1] = static_cast<const uint16_t*>(wk);
  p.w[2] = static_cast<const uint16_t*>(wv);
  p.out[0] = reinterpret_cast<uint16_t*>(ws + l.q);
  p.out[1] = reinterpret_cast<uint16_t*>(ws + l.k);
  p.out[2] = reinterpret_cast<uint16_t*>(ws + l.v);
  p.fout[0] = HD; p.fout[1] = KD_; p.fout[2] = KD_;
  p.n_mats = 3; p.T = T; p.Din = s.hidden; p.res = nullptr;
  p.ksplit = 1;
  p.partial = reinterpret_cast<float*>(ws + l.partial);
  p.flags = reinterpret_cast<unsigned long long*>(ws + l.flags);
  p.epoch = epoch;
  launch_linear(p, kKAttnProj, st);

  AttnArgs c = core_args(s, t);
  c.q = p.out[0]; c.k = p.out[1]; c.v = p.out[2];
  c.k_cache = static_cast<const uint16_t*>(k_cache);
  c.v_cache = static_cast<const uint16_t*>(v_cache);
  c.o = reinterpret_cast<uint16_t*>(ws + l.o);
  c.scale = 1.0f / sqrtf(static_cast<float>(t.head_dim));
  const AttnPlan pl = attn_plan(c, attn_core_lds(s, t));
  c.splits = pl.splits;
  c.tiles = pl.tiles;
  c.turn = pl.turn;
  const int waves = pl.splits * pl.tiles, nks = (t.head_dim + 31) / 32;
  const size_t lds = pl.lds;
  // (four wavefronts stage faster than one)
  const dim3 grid(s.n_seqs * t.n_kv_heads, pl.groups), block((waves < 4 ? 4 : waves) * kWave);
  auto core = [&](auto kernel) -> int {
    if (lds > 48 * 1024) {  // (a property of the function on the current device; cheap to repeat)
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (e != hipSuccess) return hip_fail(e, "attention LDS size");
    }
    launch(kKAttnCore, kernel, grid, block, lds, st, c);
    return DES_OK;
  };
  // Values as rows (64 or 128 coordinates: whole numbers of the swizzled 32-byte segments), except
  // under short windows in workgroups full of tiles, where the staging is little and shared by eight
  // tiles (64 positions, 64 sequences of 32 tokens: 21.5 us transposed, 22.9 as rows; 132 positions:
  // 39.1 and 37.6; 16 sequences over 64 positions, four tiles: 8.4 and 8.1).
  const bool rows = c.P + c.N > 96 || pl.tiles < 8;
  auto pick = [&](auto form) -> int {
    constexpr int W = decltype(form)::value;
    if (rows && t.head_dim == 64) return core(attention_core_kernel<2, W, true>);
    if (rows && t.head_dim == 128) return core(attention_core_kernel<4, W, true>);
    return nks == 1 ? core(attention_core_kernel<1, W, false>) : nks == 2 ? core(attention_core_kernel<2, W, false>)
         : nks == 3 ? core(attention_core_kernel<3, W, false>) : core(attention_core_kernel<4, W, false>);
  };
  const int rc = pl.splits > 1 ? pick(std::integral_constant<int, kParts>{})
               : c.P + c.N <= kWholeWindow ? pick(std::integral_constant<int, kWhole>{})
               : c.P + c.N <= kWideWindow ? pick(std::integral_constant<int, kWide>{})
                                           : pick(std::integral_constant<int, kTwice>{});
  if (rc != DES_OK) return rc;

  LinearArgs o{};
  o.in = c.o;
  o.w[0] = static_cast<const uint16_t*>(wo);
  o.out[0] = static_cast<uint16_t*>(y);
  o.fout[0] = s.hidden;
  o.n_mats = 1; o.T = T; o.Din = HD;
  o.ksplit = 1;
  o.partial = p.partial;
  o.flags = p.flags;
  o.epoch = epoch;
  o.res = s.residual ? static_cast<const uint16_t*>(x) : nullptr;
  launch_linear(o, kKAttnOut, st);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DES_OK : hip_fail(e, "attention launch");
}

}  // namespace des
