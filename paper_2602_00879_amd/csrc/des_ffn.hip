// Grouped SwiGLU expert FFN and weighted combine (Alg. 1 stage 2, last line:
// y_n = sum_{i in S_n} g_{n,i} E_i(x_n)), for gfx950.
//
// The layer is bound by the one-time read of the live experts' weights
// (Eq. 2: the b * |union S_n| term), so the kernels are organised around the
// weight stream, not around the tokens:
//   * at most 32 tokens: a wavefront owns 16 or 32 intermediate units (their gate and up
//     rows), or 32 or 64 down rows, of one expert and walks the whole reduction dimension,
//     loading each weight fragment straight into the matrix-core A operand with 16-byte
//     loads - every weight byte is read by exactly one wavefront, exactly once; the expert's
//     tokens are the B operand (one or two tiles of 16), so a partly empty token tile
//     wastes matrix-core cycles, which are free here, and no bandwidth;
//   * more: an expert's tokens form units of up to 128 rows that go through LDS and are
//     shared by a workgroup's wavefronts, the weights straight into operands (streamed) or
//     through LDS as well (tiles);
//   * the grid is sized for the worst case and every wavefront looks its
//     expert up in the device-resident live list, so the host never waits for
//     the routing result.
// Nothing is accumulated with floating-point atomics: gate/up writes the
// SwiGLU activations H, down writes one fp32 row per (token, expert) pair, and
// the combine adds a token's K rows in slot order.
#include <type_traits>

#include "des_common.h"
#include "des_select.h"
#include "des_stream_gemm.h"
#include "des_tile_gemm.h"

namespace des {


struct FfnArgs {
  const void* x;
  const void *wg, *wu, *wd;     // routed experts
  const void *sg, *su, *sd;     // shared expert (or null)
  const int32_t* topk_idx;      // [T][K]
  const float* topk_w;          // [T][K]
  const int4* slots;            // [n_slots] {expert, first sorted pair, pairs, 0}
  const int32_t *meta, *pair_tok, *pos;
  void* h;                      // [(TK) x F] then [T x Fs]
  float* o;                     // [(TK + T) x D] outputs per pair (bf16)
  void* y;                      // [T][D]
  int T, D, M, F, Fs, K, n_slots, residual;
  int splits;                   // units the shared expert's rows are spread over (LDS kernels)
  const int32_t* units;         // live units of the routed experts, longest expert first:
                                // slot | split << 16 | splits of that slot << 24; meta[2] of them
  size_t h_rows;                // routed rows of H (the shared expert's rows follow them)
  const uint16_t* xo;           // x in operand order (see operand_off), or null
  DenseArgs dn;                 // dense short block: stage 2 beside gate/up, see des_common.h
};

#ifdef DES_FFN_STAMPS  // development aid (build with DES_FFN_STAMPS=1): per-task 100 MHz
                       // timestamps of the gate/up kernels, [start, task found, end, hardware id
                       // or pairs], read back with des_debug_ffn_stamps()
__device__ long long g_ffn_stamps[8192 * 4];
#define DES_FSTAMP(task, i) do { if ((threadIdx.x & 63) == 0 && (task) < 8192) g_ffn_stamps[(task) * 4 + (i)] = wall_clock64(); } while (0)
#else
#define DES_FSTAMP(task, i) do { } while (0)
#endif

// Work item of one wavefront: which expert's rows, which pairs.
struct Task {
  const uint16_t *w0, *w1;  // weight matrices of the expert (gate, up) or (down, -)
  int slot;                 // slot of the expert (-1 for the shared expert)
  int pre_tok[2];           // blocks of <= 32 tokens: this lane's token in the slot's token tiles
  int count;                // pairs of this expert
  int pair0;                // first sorted position (routed) or 0 (shared)
  bool shared;
  uint32_t dmask;           // dense short block, down projection: the slot's routed tokens
  size_t row_base;          // first H / O row of these pairs
  int fdim;                 // F of this expert (F or Fs)
};

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + expf(-z)); }

// ------------------------------------------------------------------ bf16 path
// MFMA 16x16x32 bf16: lane l supplies row (l%16), reduction elements
// 8*(l/16)..+7 of both operands; the accumulator of lane l holds token column
// (l%16) and weight rows 4*(l/16)..+3.
//
// Weight fragment address for (row tile rt, k-step ks):
//   row-major [rows][kd]:  base + (rt*16 + l%16)*kd + ks*32 + 8*(l/16)
//   packed tiles          :  base + ((rt*(kd/32) + ks)*64 + l)*8
template <bool PACKED>
__device__ __forceinline__ const uint16_t* frag_ptr(const uint16_t* base, int rt, int kd, int lane) {
  if (PACKED) return base + (static_cast<size_t>(rt) * (kd / 32) * 64 + lane) * 8;
  return base + (static_cast<size_t>(rt) * 16 + (lane & 15)) * kd + (lane >> 4) * 8;
}

__device__ __forceinline__ bf16x8 ld8(const uint16_t* p) {
  return *reinterpret_cast<const bf16x8*>(p);
}
// Weights are read once and never again: a non-temporal load keeps them from
// displacing the activations in L2 / the last-level cache.
__device__ __forceinline__ bf16x8 ld8_stream(const uint16_t* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(p));
}
// This lane's place in the loads of row tile rt: packed tiles are in operand order already.
template <bool PACKED>
__device__ __forceinline__ const uint16_t* load_ptr(const uint16_t* base, int rt, int kd, int lane) {
  if (PACKED) return frag_ptr<true>(base, rt, kd, lane);
  return base + (static_cast<size_t>(rt) * 16 + (lane >> 3)) * kd + (lane & 7) * 8;
}
// Load i of a tile's stream: k-step i (packed), or half i % 2 of 64-element block i / 2.
template <bool PACKED>
__device__ __forceinline__ size_t load_off(int i, int kd) {
  return PACKED ? static_cast<size_t>(i) * 512 : static_cast<size_t>(i & 1) * 8 * kd + (i >> 1) * 64;
}

// x of at most 32 tokens in operand order, eight elements of a token next to the same eight of the
// following ones: element offset of piece `oct` (elements 8 * oct ..) of token t.  The lanes of an
// operand load then read runs of 256 bytes; in rows they read four rows per four lanes, at a quarter of
// the rate (see operand_write), which bounds the kernel where a wavefront has few weight rows per token
// fragment (17 experts of 2048 x 512, 32 tokens, 16 units per wavefront: 20.0 -> 18.4 us; 32 of
// 2048 x 768 in 32 units, where the weights do: 34.5 -> 34.0).
__device__ __forceinline__ int operand_off(int oct, int t, int T) { return (oct * T + t) * 8; }

// gate/up for the task's pairs (at most 16*NT), intermediate rows
// (ft0 .. ft0+FT-1)*16..+15.  The FT row tiles share every token fragment.
template <int FT, int NT, int U, bool PACKED>
__device__ __forceinline__ void gateup_group(const FfnArgs& a, const Task& t, int ft0, int lane,
                                             char* turn) {
  static_assert(PACKED || U % 2 == 0, "row-major stages are whole 64-element blocks");
  const int D = a.D;
  const int nks = D / 32;
  const uint16_t* x = static_cast<const uint16_t*>(a.x);
  const uint16_t* gp[FT];
  const uint16_t* up[FT];
#pragma unroll
  for (int f = 0; f < FT; ++f) {
    gp[f] = load_ptr<PACKED>(t.w0, ft0 + f, D, lane);
    up[f] = load_ptr<PACKED>(t.w1, ft0 + f, D, lane);
  }
  const uint16_t* xp[NT];
  const int xstep = a.xo ? 32 * a.T : 32;  // elements to the next k-step
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    int pi = min(i * 16 + (lane & 15), t.count - 1);  // clamped rows are dropped at the store
    const int tok = t.shared ? pi : t.pre_tok[i];
    xp[i] = a.xo ? a.xo + operand_off(lane >> 4, tok, a.T) : x + static_cast<size_t>(tok) * D + (lane >> 4) * 8;
  }
  f32x4 accg[FT][NT], accu[FT][NT];
#pragma unroll
  for (int f = 0; f < FT; ++f)
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      accg[f][i] = f32x4{0.f, 0.f, 0.f, 0.f};
      accu[f][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  bf16x8 ag[2][U][FT], au[2][U][FT], bx[2][U][NT];
  auto load = [&](int st, auto stage) {
    constexpr int s = decltype(stage)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ks = st * U + u;
#pragma unroll
      for (int f = 0; f < FT; ++f) {
        ag[s][u][f] = ld8_stream(gp[f] + load_off<PACKED>(ks, D));
        au[s][u][f] = ld8_stream(up[f] + load_off<PACKED>(ks, D));
      }
#pragma unroll
      for (int i = 0; i < NT; ++i) bx[s][u][i] = ld8(xp[i] + ks * xstep);
    }
  };
  auto compute = [&](auto stage) {
    constexpr int s = decltype(stage)::value;
    if constexpr (!PACKED) {
      turn_fence();
#pragma unroll
      for (int u = 0; u < U; u += 2)
#pragma unroll
        for (int f = 0; f < FT; ++f) {
          turn_write(ag[s][u][f], ag[s][u + 1][f], turn + (u / 2 * 2 * FT + 2 * f) * kTurnBytes, lane);
          turn_write(au[s][u][f], au[s][u + 1][f], turn + (u / 2 * 2 * FT + 2 * f + 1) * kTurnBytes, lane);
        }
      turn_fence();
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int f = 0; f < FT; ++f) {
          ag[s][u][f] = turn_read(turn + (u / 2 * 2 * FT + 2 * f) * kTurnBytes, u & 1, lane);
          au[s][u][f] = turn_read(turn + (u / 2 * 2 * FT + 2 * f + 1) * kTurnBytes, u & 1, lane);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int i = 0; i < NT; ++i) {
          accg[f][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ag[s][u][f], bx[s][u][i], accg[f][i], 0, 0, 0);
          accu[f][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(au[s][u][f], bx[s][u][i], accu[f][i], 0, 0, 0);
        }
  };
  stream_pipeline(nks / U, load, compute);
  for (int ks = nks / U * U; ks < nks; ++ks) {  // k-steps left over by the stages
    bf16x8 x1[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) x1[i] = ld8(xp[i] + ks * xstep);
#pragma unroll
    for (int f = 0; f < FT; ++f) {
      const bf16x8 g1 = ld8_stream(frag_ptr<PACKED>(t.w0, ft0 + f, D, lane) + static_cast<size_t>(ks) * frag_step<PACKED>());
      const bf16x8 u1 = ld8_stream(frag_ptr<PACKED>(t.w1, ft0 + f, D, lane) + static_cast<size_t>(ks) * frag_step<PACKED>());
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        accg[f][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(g1, x1[i], accg[f][i], 0, 0, 0);
        accu[f][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u1, x1[i], accu[f][i], 0, 0, 0);
      }
    }
  }
  uint16_t* h = static_cast<uint16_t*>(a.h);
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int pi = i * 16 + (lane & 15);
    if (pi < t.count) {
#pragma unroll
      for (int f = 0; f < FT; ++f) {
        u16x4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = f32_to_bf16_bits(silu_f(accg[f][i][q]) * accu[f][i][q]);
        uint16_t* dst = h + (t.row_base + pi) * t.fdim + (ft0 + f) * 16 + 4 * (lane >> 4);
        *reinterpret_cast<u16x4*>(dst) = v;
      }
    }
  }
}

__device__ __forceinline__ bool make_task(const FfnArgs& a, int slot_or_shared, bool shared,
                                          bool down, Task& t, int lane) {
  const size_t TK = static_cast<size_t>(a.T) * a.K;
  t.dmask = 0u;  // (every path: the down projection tests it)
  if (!shared) {
    const int4 sl = a.slots[slot_or_shared];
    // an unused slot; also refuses a record that does not fit the problem (the
    // workspace is the caller's memory: never index weights or pairs with it blindly)
    if (sl.x < 0 || sl.x >= a.M || sl.y < 0 || sl.z < 1 ||
        static_cast<long long>(sl.y) + sl.z > static_cast<long long>(a.h_rows))
      return false;
    const int e = sl.x;
    const int off = sl.y;
    if (a.dn.on) {
      // every token of the block, in order: H row = first row of the slot + token
      t.pre_tok[0] = min(lane & 15, a.T - 1);
      t.pre_tok[1] = min(16 + (lane & 15), a.T - 1);
      if (down) {
        // the expert's pairs are the set bits of its bitmap, in order (positions past
        // the count repeat the last one; their results are dropped)
        t.dmask = a.dn.tokmask[slot_or_shared] & (a.T >= 32 ? 0xffffffffu : ((1u << a.T) - 1u));
        if (t.dmask == 0u) return false;  // nobody was routed to this expert
        const int cnt = __popc(t.dmask);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int want = min(i * 16 + (lane & 15), cnt - 1);
          uint32_t mm = t.dmask;
          for (int k = 0; k < want; ++k) mm &= mm - 1u;
          t.pre_tok[i] = __builtin_ctz(mm);
        }
      }
    } else if (!down && a.T <= 32) {
      // at most 32 tokens: the record carries the bitmap of the expert's tokens; its pairs
      // in order are the set bits in order (positions past the count repeat the last one)
      const uint32_t m = static_cast<uint32_t>(sl.w);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int want = min(i * 16 + (lane & 15), sl.z - 1);
        uint32_t mm = m;
        for (int k = 0; k < want; ++k) mm &= mm - 1u;
        t.pre_tok[i] = mm ? min(__builtin_ctz(mm), a.T - 1) : 0;
      }
    }
    t.slot = slot_or_shared;
    // (dense, down: only the routed tokens count, so a slot with at most 16 of them takes
    // the one-tile path)
    t.count = t.dmask ? __popc(t.dmask) : sl.z;
    t.pair0 = off;
    t.shared = false;
    t.row_base = static_cast<size_t>(off);
    t.fdim = a.F;
    const size_t mat = static_cast<size_t>(a.F) * a.D;
    if (down) {
      t.w0 = static_cast<const uint16_t*>(a.wd) + e * mat;
      t.w1 = nullptr;
    } else {
      t.w0 = static_cast<const uint16_t*>(a.wg) + e * mat;
      t.w1 = static_cast<const uint16_t*>(a.wu) + e * mat;
    }
  } else {
    t.slot = -1;
    t.count = a.T;
    t.pair0 = 0;
    t.shared = true;
    t.row_base = TK;  // H: row index in units of its own stride, see h_base below
    t.fdim = a.Fs;
    t.w0 = static_cast<const uint16_t*>(down ? a.sd : a.sg);
    t.w1 = static_cast<const uint16_t*>(down ? nullptr : a.su);
  }
  return true;
}

// H rows of the shared expert start after the TK routed rows of width F; they
// have width Fs.  Express that start as a row offset in Fs-wide rows by
// shifting the base pointer instead (keeps one indexing formula).
__device__ __forceinline__ FfnArgs shared_view(const FfnArgs& a, Task& t, size_t elem_size) {
  FfnArgs v = a;
  v.h = static_cast<char*>(a.h) + a.h_rows * a.F * elem_size;
  t.row_base = 0;
  return v;
}

#ifndef DES_FFN_WAVES
#define DES_FFN_WAVES 1
#endif
constexpr int kFfnWaves = DES_FFN_WAVES;  // wavefronts per workgroup; each is an independent task
// The wavefront's task, a scalar: it guards matrix instructions (see stream_pipeline).
__device__ __forceinline__ int ffn_task() {
  return blockIdx.x * kFfnWaves + (kFfnWaves == 1 ? 0 : uniform_int(threadIdx.x >> 6));
}
constexpr int kGuTiles = 2;   // gate/up row tiles per task (F % 32 == 0, so F/16 is even)

// One gate/up task (see the kernel comment): returns false if the slot is unused.
template <int MAXNT, bool PACKED, int U1 = 2, int U2 = 2, int GT = kGuTiles>
__device__ __forceinline__ bool gateup_task(const FfnArgs& a, int task, int lane, char* turn) {
  const int tiles_r = a.F / (16 * GT);
  const int routed = a.n_slots * tiles_r;
  Task t;
  int ft;
  FfnArgs v = a;
  DES_FSTAMP(task, 0);
  if (task < routed) {
    if (!make_task(a, task / tiles_r, false, false, t, lane)) return false;
    DES_FSTAMP(task, 1);
    ft = (task % tiles_r) * GT;
  } else {
    make_task(a, 0, true, false, t, lane);
    v = shared_view(a, t, 2);
    ft = (task - routed) * GT;
  }
  if (MAXNT == 1 || uniform_int(t.count) <= 16) gateup_group<GT, 1, U1, PACKED>(v, t, ft, lane, turn);
  else gateup_group<GT, MAXNT, U2, PACKED>(v, t, ft, lane, turn);
  DES_FSTAMP(task, 2);
#ifdef DES_FFN_STAMPS
  if ((threadIdx.x & 63) == 0 && task < 8192)
    g_ffn_stamps[task * 4 + 3] = (static_cast<long long>(__builtin_amdgcn_s_getreg(20 | (31 << 11))) << 32) |
                                 static_cast<unsigned>(__builtin_amdgcn_s_getreg(4 | (31 << 11)));
#endif
  return true;
}

// MAXNT bounds the token tiles a task can have (the host knows T >= any expert's
// count), so that small blocks get a kernel with few registers.  U1 / U2 are
// the k-steps per stage of the one- and two-token-tile paths.
// GT = row tiles per task: 2 normally, 1 when the launch would otherwise have
// too few wavefronts to keep enough bytes in flight (small coresets).
template <int MAXNT, bool PACKED, int U1 = 2, int U2 = 2, int GT = kGuTiles>
__global__ __launch_bounds__(kFfnWaves* kWave) void gateup_bf16_kernel(FfnArgs a) {
  const int lane = threadIdx.x & 63;
  int task = ffn_task();
  {
    if (a.dn.on) {
      // dense short block: the first wavefronts of the grid re-route the block's tokens
      // (Alg. 1 stage 2) while the others stream the coreset's weights
      const int n_s2 = (a.T * a.dn.lpt + 63) / 64;
      if (task < n_s2) {
        __shared__ uint32_t s_sorted[kFfnWaves * kEpl * 64];
        uint32_t* srt = s_sorted + (threadIdx.x >> 6) * (kEpl * 64);
        const int n_core = uniform_int(a.meta[0]);
        if (n_core <= 0) return;  // the routing launch gave up: nothing was elected
        switch (a.dn.lpt) {
          case 4: stage2_wave<4>(a.dn, a.T, a.M, a.K, n_core, task, srt); break;
          case 8: stage2_wave<8>(a.dn, a.T, a.M, a.K, n_core, task, srt); break;
          case 16: stage2_wave<16>(a.dn, a.T, a.M, a.K, n_core, task, srt); break;
          case 32: stage2_wave<32>(a.dn, a.T, a.M, a.K, n_core, task, srt); break;
          default: stage2_wave<64>(a.dn, a.T, a.M, a.K, n_core, task, srt); break;
        }
        return;
      }
      task -= n_s2;
    }
  }
  const int tasks = a.n_slots * (a.F / (16 * GT)) + a.Fs / (16 * GT);
  // row-major: the stage's tiles (2 per row tile, U k-steps) in operand order, per wavefront
  constexpr int kUmax = (U1 > U2 ? U1 : U2) > 2 ? (U1 > U2 ? U1 : U2) : 2;
  constexpr int kTurn = PACKED ? 16 : kUmax / 2 * 2 * GT * kTurnBytes;
  __shared__ __align__(16) char s_turn[kFfnWaves * kTurn];
  if (task < tasks) gateup_task<MAXNT, PACKED, U1, U2, GT>(a, task, lane, s_turn + (threadIdx.x >> 6) * kTurn);
}

// down for the task's pairs (at most 16*NT), output rows (dt0 .. dt0+RT-1)*16
template <int RT, int NT, int U, bool PACKED>
__device__ __forceinline__ void down_group(const FfnArgs& a, const Task& t, int dt0, int lane,
                                           char* turn) {
  static_assert(PACKED || U % 2 == 0, "row-major stages are whole 64-element blocks");
  // the trip counts are uniform (see stream_pipeline); the addresses of row-major tiles are
  // better derived in vector registers (33 experts of 2048 x 768: 23.2 us against 26.1 us, the
  // compiler spends scalar instructions per load otherwise), packed ones in scalars (19.7, 20.1)
  const int F = PACKED ? uniform_int(t.fdim) : t.fdim;
  const int nks = uniform_int(F / 32);
  const uint16_t* h = static_cast<const uint16_t*>(a.h);
  const uint16_t* ap[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) ap[r] = load_ptr<PACKED>(t.w0, dt0 + r, F, lane);
  const uint16_t* hp[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int pi = min(i * 16 + (lane & 15), t.count - 1);
    // (dense short block: H holds every token of the block for this slot; the routed
    // ones, in order, are this expert's pairs)
    const int hrow = t.dmask ? t.pre_tok[i] : pi;
    hp[i] = h + (t.row_base + hrow) * F + (lane >> 4) * 8;
  }
  f32x4 acc[RT][NT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[r][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 aw[2][U][RT], bh[2][U][NT];
  auto load = [&](int st, auto stage) {
    constexpr int s = decltype(stage)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ks = st * U + u;
#pragma unroll
      for (int r = 0; r < RT; ++r)
        aw[s][u][r] = ld8_stream(ap[r] + load_off<PACKED>(ks, F));
#pragma unroll
      for (int i = 0; i < NT; ++i) bh[s][u][i] = ld8(hp[i] + ks * 32);
    }
  };
  auto compute = [&](auto stage) {
    constexpr int s = decltype(stage)::value;
    if constexpr (!PACKED) {
      turn_fence();
#pragma unroll
      for (int u = 0; u < U; u += 2)
#pragma unroll
        for (int r = 0; r < RT; ++r)
          turn_write(aw[s][u][r], aw[s][u + 1][r], turn + (u / 2 * RT + r) * kTurnBytes, lane);
      turn_fence();
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int r = 0; r < RT; ++r) aw[s][u][r] = turn_read(turn + (u / 2 * RT + r) * kTurnBytes, u & 1, lane);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int i = 0; i < NT; ++i)
          acc[r][i] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[s][u][r], bh[s][u][i], acc[r][i], 0, 0, 0);
  };
  stream_pipeline(nks / U, load, compute);
  for (int ks = nks / U * U; ks < nks; ++ks) {  // k-steps left over by the stages
    bf16x8 h1[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) h1[i] = ld8(hp[i] + ks * 32);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const bf16x8 w1 = ld8_stream(frag_ptr<PACKED>(t.w0, dt0 + r, F, lane) + static_cast<size_t>(ks) * frag_step<PACKED>());
#pragma unroll
      for (int i = 0; i < NT; ++i)
        acc[r][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, h1[i], acc[r][i], 0, 0, 0);
    }
  }
  const size_t orow0 = t.shared ? static_cast<size_t>(a.T) * a.K : static_cast<size_t>(t.pair0);
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int pi = i * 16 + (lane & 15);
    if (pi < t.count) {
      size_t orow = orow0 + pi;
      if (t.dmask) {
        // dense short block: the pair's row is token * K + (which of the token's
        // choices this expert is)
        const int tok = t.pre_tok[i];
        orow = static_cast<size_t>(tok) * a.K + a.dn.choice[t.slot * 32 + tok];
      }
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        float* dst = a.o + orow * a.D + (dt0 + r) * 16 + 4 * (lane >> 4);
        *reinterpret_cast<f32x4*>(dst) = acc[r][i];
      }
    }
  }
}

// One down task: 64 output rows of one expert for all of its pairs.
template <int MAXNT, bool PACKED, int U1 = 2, int U2 = 2, int RTG = 4>
__device__ __forceinline__ bool down_task(const FfnArgs& a, int task, int lane, char* turn) {
  const int dtiles = a.D / 16;
  const int groups = (dtiles + RTG - 1) / RTG;  // 16 * RTG output rows per task
  const int routed = a.n_slots * groups;
  Task t;
  int dg;
  FfnArgs v = a;
  if (task < routed) {
    const int slot = task / groups;
    if (!make_task(a, slot, false, true, t, lane)) return false;
    dg = task % groups;
  } else {
    make_task(a, 0, true, true, t, lane);
    v = shared_view(a, t, 2);
    dg = task - routed;
  }
  const int dt_begin = dg * RTG;
  const int dt_end = min(dt_begin + RTG, dtiles);
  if (uniform_int(dt_end - dt_begin) < RTG) {  // ragged row group: one row tile at a time
    for (int dt = uniform_int(dt_begin); dt < uniform_int(dt_end); ++dt) down_group<1, MAXNT, 2, PACKED>(v, t, dt, lane, turn);
  } else if (MAXNT == 1 || uniform_int(t.count) <= 16) {
    down_group<RTG, 1, U1, PACKED>(v, t, dt_begin, lane, turn);
  } else {
    down_group<RTG, MAXNT, U2, PACKED>(v, t, dt_begin, lane, turn);
  }
  return true;
}

template <int MAXNT, bool PACKED, int U1 = 2, int U2 = 2, int RTG = 4>
__global__ __launch_bounds__(kFfnWaves* kWave) void down_bf16_kernel(FfnArgs a) {
  const int lane = threadIdx.x & 63;
  const int task = ffn_task();
  const int groups = (a.D / 16 + RTG - 1) / RTG;
  const int tasks = a.n_slots * groups + (a.Fs > 0 ? groups : 0);
  constexpr int kUmax = (U1 > U2 ? U1 : U2) > 2 ? (U1 > U2 ? U1 : U2) : 2;
  constexpr int kTurn = PACKED ? 16 : kUmax / 2 * RTG * kTurnBytes;
  __shared__ __align__(16) char s_turn[kFfnWaves * kTurn];
  if (task < tasks) down_task<MAXNT, PACKED, U1, U2, RTG>(a, task, lane, s_turn + (threadIdx.x >> 6) * kTurn);
}

// ------------------------------------------ larger blocks: activations via LDS
// (the streaming building block dma_stream_gemm lives in des_stream_gemm.h)
// Which expert, which of its weight-row groups and which pairs a workgroup works on.  The grid is
// one-dimensional and read in hand-out order: the shared expert first (every token: the longest
// workgroups), then the live units of the routed experts as the permutation lists them - longest
// expert first, an expert's units next to each other.  So when the workgroups do not all fit on
// the chip at once the long ones start first, consecutive workgroups carry similar work, and the
// grid's tail beyond the live units exits on one scalar load.
//
// The units of an expert read the same weights.  The hardware deals workgroups out to the eight
// XCDs in turn, each with an L2 of its own: an expert's workgroups are numbered so that an XCD gets
// a run of its row groups with all their units, which then stream those weights side by side, one
// from memory and the others from that L2 (2048 tokens, 1024 on each of 16 experts of 2048 x 768:
// gate/up 161 -> 122 us, the next form's 146 -> 105; with every unit's groups on one XCD instead,
// which saves fetches of token rows, 162).  The weights of an expert with one unit are read once
// on the chip and loaded non-temporally: kept in L2 and the last-level cache they displace the
// token rows (128 tokens: 40.0 -> 44.2 us).
struct LdsTask {
  int group;        // weight-row group of the expert
  int g0, rows;     // its pairs [g0, g0 + rows)
  bool alone;       // no other workgroup reads these weights
};
__device__ __forceinline__ void unit_share(int i, int per, int nsplit, int& group, int& split) {
  if (nsplit == 1) {  // (a run of row groups per XCD is no help: 80 tokens, 2048 x 512, down 13.4 -> 14.9 us)
    group = i;
    split = 0;
    return;
  }
  // blocks of eight units: with all of an expert's side by side their token rows would not stay in an L2
  const int block = i / (8 * per), m = min(8, nsplit - 8 * block);
  i -= block * 8 * per;
  const int n = m * per, j = i & 7;  // workgroup i of the block's n; those with the same j share an XCD
  const int p = j * (n >> 3) + min(j, n & 7) + (i >> 3);
  group = p / m;
  split = 8 * block + p % m;
}
// EVEN: an expert's units have the same number of rows, so that they keep the same pace (else all but
// the last have as many as a unit can: fewer tiles of 32 rows in all, which is what the tile kernels pay for).
template <bool DOWN, bool EVEN>
__device__ __forceinline__ bool lds_task(const FfnArgs& a, int per_expert, int per_shared, int max_rows, LdsTask& k,
                                         Task& t, FfnArgs& v, int lane) {
  int bx = blockIdx.x, split, nsplit;
  v = a;
  if (bx < per_shared * a.splits) {
    make_task(a, 0, true, DOWN, t, lane);
    v = shared_view(a, t, 2);
    nsplit = a.splits;
    unit_share(bx, per_shared, nsplit, k.group, split);
  } else {
    bx -= per_shared * a.splits;
    const int u = bx / per_expert;
    if (u >= uniform_int(a.meta[2])) return false;
    const int rec = uniform_int(a.units[u]);
    nsplit = rec >> 24;
    if ((rec & 0xffff) >= a.n_slots || nsplit < 1 || nsplit > kMaxSplits || ((rec >> 16) & 0xff) >= nsplit) return false;
    unit_share(bx - (u - ((rec >> 16) & 0xff)) * per_expert, per_expert, nsplit, k.group, split);
    if (!make_task(a, rec & 0xffff, false, DOWN, t, lane)) return false;
  }
  const int count = uniform_int(t.count);  // (scalars: they guard matrix instructions, see stream_pipeline)
  const int share = EVEN ? min(max_rows, (count + nsplit - 1) / nsplit) : max_rows;
  k.g0 = split * share;
  k.rows = min(share, count - k.g0);
  k.alone = nsplit == 1;
  return k.rows > 0;
}

// Calls f(token tiles, alone) with the number of 16-row token tiles that the code is built for
// (even units of an expert with several have more than half of the rows they can have).
template <int MAXNT, typename F>
__device__ __forceinline__ void by_token_tiles(int rows, bool alone, F&& f) {
  const int nt = (rows + 15) / 16;
  if (MAXNT < 8 || alone) {
    if (nt <= 1) f(std::integral_constant<int, 1>{}, std::true_type{});
    else if (nt <= 2) f(std::integral_constant<int, 2>{}, std::true_type{});
    else if (MAXNT < 8 || nt <= 4) f(std::integral_constant<int, 4>{}, std::true_type{});
    else if constexpr (MAXNT >= 8) {
      if (nt <= 6) f(std::integral_constant<int, 6>{}, std::true_type{});
      else f(std::integral_constant<int, 8>{}, std::true_type{});
    }
  } else if constexpr (MAXNT >= 8) {
    if (nt <= 6) f(std::integral_constant<int, 6>{}, std::false_type{});
    else f(std::integral_constant<int, 8>{}, std::false_type{});
  }
}

// MAXNT = token tiles of a unit at most (the LDS buffer holds 16*MAXNT rows); LW = wavefronts
// per workgroup; KD = the reduction length when the host knows it to be one of the unrolled
// cases, else 0; RT = weight tiles of a wavefront, for gate/up half of them gate and half up.
template <int MAXNT, int LW, int KD, int RT>
__global__ __launch_bounds__(LW* kWave, ((KD > 0 || MAXNT <= 4 || RT == 4) ? 2 : 1)) void gateup_lds_kernel(FfnArgs a) {
  constexpr int HT = RT / 2;
  __shared__ __align__(16) uint16_t lds[lds_elems(RT, KD)];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  Task t;
  LdsTask k;
  FfnArgs v;
  const int per_r = (a.F / 16 + LW * HT - 1) / (LW * HT);
  const int per_s = (a.Fs / 16 + LW * HT - 1) / (LW * HT);
  DES_FSTAMP(blockIdx.x, 0);
  if (!lds_task<false, true>(a, per_r, per_s, 16 * MAXNT, k, t, v, lane)) return;  // uniform per workgroup
  const int tiles = t.fdim / 16, tile = (k.group * LW + wave) * HT;
  const uint16_t* wp[RT];
#pragma unroll
  for (int i = 0; i < HT; ++i) {  // a tile past the matrix repeats the last one, dropped at the store
    wp[i] = tile_base(uniform_ptr(t.w0), min(tile + i, tiles - 1), a.D);
    wp[HT + i] = tile_base(uniform_ptr(t.w1), min(tile + i, tiles - 1), a.D);
  }
  const uint32_t wlo = tile_lane_off(lane);
  const uint16_t* x = uniform_ptr(static_cast<const uint16_t*>(a.x));
  auto row_off = [&](int r) {
    const int tok = t.shared ? k.g0 + r : a.pair_tok[t.pair0 + k.g0 + r];
    return tok * a.D;
  };
  by_token_tiles<MAXNT>(k.rows, k.alone, [&](auto ntc, auto alone) {
    constexpr int NT = decltype(ntc)::value;
    f32x4 acc[RT][NT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int i = 0; i < NT; ++i) acc[r][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int KC = NT <= 4 && RT == 2 ? 128 : 64;  // rows * KC: at most one 16 KB buffer
    dma_stream_gemm<RT, NT, (MAXNT < 8 || KC == 128 ? 64 : 128), LW, KC, KD, decltype(alone)::value>(
        wp, wlo, wave, a.D, k.rows, x, row_off, lds, acc);
    uint16_t* h = static_cast<uint16_t*>(v.h) + (t.row_base + k.g0) * t.fdim + 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int r = i * 16 + (lane & 15);
      if (r >= k.rows) continue;
#pragma unroll
      for (int f = 0; f < HT; ++f) {
        if (tile + f >= tiles) continue;
        u16x4 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = f32_to_bf16_bits(silu_f(acc[f][i][q]) * acc[HT + f][i][q]);
        *reinterpret_cast<u16x4*>(h + static_cast<size_t>(r) * t.fdim + (tile + f) * 16) = o;
      }
    }
  });
#ifdef DES_FFN_STAMPS
  DES_FSTAMP(blockIdx.x, 2);
  if (threadIdx.x == 0 && blockIdx.x < 8192) {  // pairs this workgroup worked on, where it ran
    g_ffn_stamps[blockIdx.x * 4 + 3] = k.rows;
    g_ffn_stamps[blockIdx.x * 4 + 1] =
        (static_cast<long long>(__builtin_amdgcn_s_getreg(20 | (31 << 11))) << 32) |
        static_cast<unsigned>(__builtin_amdgcn_s_getreg(4 | (31 << 11)));
  }
#endif
}

template <int MAXNT, int LW, int KD, int RT>
__global__ __launch_bounds__(LW* kWave, ((KD > 0 || MAXNT <= 4 || RT == 4) ? 2 : 1)) void down_lds_kernel(FfnArgs a) {
  __shared__ __align__(16) uint16_t lds[lds_elems(RT, KD)];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  Task t;
  LdsTask k;
  FfnArgs v;
  const int dtiles = a.D / 16, per = (dtiles + RT * LW - 1) / (RT * LW);
  if (!lds_task<true, true>(a, per, a.Fs > 0 ? per : 0, 16 * MAXNT, k, t, v, lane)) return;
  const int dt0 = (k.group * LW + wave) * RT;
  const int F = uniform_int(t.fdim);  // guards matrix instructions
  const uint16_t* wp[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) wp[r] = tile_base(uniform_ptr(t.w0), min(dt0 + r, dtiles - 1), F);
  const uint32_t wlo = tile_lane_off(lane);
  const uint16_t* h = uniform_ptr(static_cast<const uint16_t*>(v.h) + (t.row_base + k.g0) * F);
  const size_t orow0 = (t.shared ? static_cast<size_t>(a.T) * a.K : static_cast<size_t>(t.pair0)) + k.g0;
  auto row_off = [&](int r) { return r * F; };
  by_token_tiles<MAXNT>(k.rows, k.alone, [&](auto ntc, auto alone) {
    constexpr int NT = decltype(ntc)::value;
    f32x4 acc[RT][NT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int i = 0; i < NT; ++i) acc[r][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int KC = NT <= 4 && RT == 2 ? 128 : 64;
    dma_stream_gemm<RT, NT, (MAXNT < 8 || KC == 128 ? 64 : 128), LW, KC, KD, decltype(alone)::value>(
        wp, wlo, wave, F, k.rows, h, row_off, lds, acc);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int r = i * 16 + (lane & 15);
      if (r >= k.rows) continue;
      float* dst = a.o + (orow0 + r) * a.D + dt0 * 16 + 4 * (lane >> 4);
#pragma unroll
      for (int q = 0; q < RT; ++q)
        if (dt0 + q < dtiles) *reinterpret_cast<f32x4*>(dst + 16 * q) = acc[q][i];
    }
  });
}

// ------------------------------------------ many token rows: weights and tokens in LDS tiles
// The same work list (a unit = up to 128 token rows of an expert), the tiles of
// des_tile_gemm.h: a workgroup has 16 MT intermediate units (their gate and up rows), or 32 MT
// output rows, of one unit.  Every sum runs over the reduction in the same order as in the
// other kernels, so which of them ran cannot be told from the results.  P = chunks of the
// reduction in registers on their way, where at most 64 token rows leave the room.
template <bool PACKED, int MAXNT, int MT, int P>
__global__ __launch_bounds__(kTileThreads, 2) void gateup_tile_kernel(FfnArgs a) {
  constexpr int HT = MT / 2, kRows = 32 * MAXNT;
  // Packed weights, two chunks ahead, units sized for 128 rows (many experts with a few pairs each): two
  // workgroups per compute unit are faster than the three whose tiles fit (96 experts of 2016 x 288 and a
  // shared one, 80 tokens: 36.1 us against 39.9, with the last-level cache flushed 40.3 against 44.1).  Not
  // so for row-major weights (128 experts of 2048 x 768, 65 tokens: 63.2 against 57.6) and in the down
  // projection (32 experts of 1024 x 352, 2048 tokens: 16.7 against 14.8).
  constexpr int kLds = PACKED && P == 2 && MAXNT == 4 ? 56 * 1024 : tile_lds_bytes<MT, MAXNT>();
  __shared__ __align__(16) char lds[kLds];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  Task t;
  LdsTask k;
  FfnArgs v;
  if (!lds_task<false, false>(a, (a.F / 16 + MT - 1) / MT, (a.Fs / 16 + MT - 1) / MT, kRows, k, t, v, lane)) return;
  const int tiles = t.fdim / 16, f0 = k.group * MT;  // this workgroup's first 16 units
  const uint16_t* x = static_cast<const uint16_t*>(a.x);
  uint16_t* h = static_cast<uint16_t*>(v.h);
  // row tile q of the workgroup: wavefronts wm have gate tiles, then the up tiles of the same units
  const uint16_t* aptr[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int q = 2 * i + (tid >> 7), ft = min(f0 + q / MT * HT + q % HT, tiles - 1);
    aptr[i] = tile_weight_ptr<PACKED>((q % MT < HT ? t.w0 : t.w1) + static_cast<size_t>(ft) * 16 * a.D, a.D, tid);
  }
  const int g0 = k.g0, rows = k.rows;
  auto run = [&](auto ntc) {
    constexpr int NT = decltype(ntc)::value;
    const uint16_t* bptr[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int r = g0 + min(i * 32 + (tid >> 3), rows - 1);
      bptr[i] = x + static_cast<size_t>(t.shared ? r : a.pair_tok[t.pair0 + r]) * a.D + (tid & 7) * 8;
    }
    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    tile_gemm<MT, NT, (NT <= 2 ? P : 1), PACKED>(aptr, bptr, a.D, lds, acc);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int r = (wn * NT + j) * 16 + (lane & 15);
      if (r >= rows) continue;
#pragma unroll
      for (int i = 0; i < HT; ++i) {
        const int ft = f0 + wm * HT + i;
        if (ft >= tiles) continue;
        u16x4 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = f32_to_bf16_bits(silu_f(acc[i][j][q]) * acc[HT + i][j][q]);
        *reinterpret_cast<u16x4*>(h + (t.row_base + g0 + r) * t.fdim + ft * 16 + 4 * (lane >> 4)) = o;
      }
    }
  };
  if (rows <= 32) run(std::integral_constant<int, 1>{});
  else if (rows <= 64) run(std::integral_constant<int, 2>{});
  else if (rows <= 96) run(std::integral_constant<int, MAXNT < 3 ? MAXNT : 3>{});
  else run(std::integral_constant<int, MAXNT>{});
}

template <bool PACKED, int MAXNT, int MT, int P>
__global__ __launch_bounds__(kTileThreads, 2) void down_tile_kernel(FfnArgs a) {
  constexpr int kRows = 32 * MAXNT;
  __shared__ __align__(16) char lds[tile_lds_bytes<MT, MAXNT>()];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  Task t;
  LdsTask k;
  FfnArgs v;
  const int tiles = a.D / 16, per = (tiles + 2 * MT - 1) / (2 * MT);
  if (!lds_task<true, false>(a, per, a.Fs > 0 ? per : 0, kRows, k, t, v, lane)) return;
  const int F = uniform_int(t.fdim), d0 = k.group * 2 * MT;  // (see stream_pipeline)
  const uint16_t* h = static_cast<const uint16_t*>(v.h);
  const size_t orow0 = t.shared ? static_cast<size_t>(a.T) * a.K : static_cast<size_t>(t.pair0);
  const uint16_t* aptr[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
    aptr[i] = tile_weight_ptr<PACKED>(
        t.w0 + static_cast<size_t>(min(d0 + 2 * i + (tid >> 7), tiles - 1)) * 16 * F, F, tid);
  const int g0 = k.g0, rows = k.rows;
  auto run = [&](auto ntc) {
    constexpr int NT = decltype(ntc)::value;
    const uint16_t* bptr[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
      bptr[i] = h + (t.row_base + g0 + min(i * 32 + (tid >> 3), rows - 1)) * F + (tid & 7) * 8;
    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    tile_gemm<MT, NT, (NT <= 2 ? P : 1), PACKED>(aptr, bptr, F, lds, acc);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int r = (wn * NT + j) * 16 + (lane & 15);
      if (r >= rows) continue;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int dt = d0 + wm * MT + i;
        if (dt < tiles)
          *reinterpret_cast<f32x4*>(a.o + (orow0 + g0 + r) * a.D + dt * 16 + 4 * (lane >> 4)) = acc[i][j];
      }
    }
  };
  if (rows <= 32) run(std::integral_constant<int, 1>{});
  else if (rows <= 64) run(std::integral_constant<int, 2>{});
  else if (rows <= 96) run(std::integral_constant<int, MAXNT < 3 ? MAXNT : 3>{});
  else run(std::integral_constant<int, MAXNT>{});
}

// ------------------------------------------------------------------ fp32 path
// Plain fused-multiply-add kernels for the small fp32 configuration: lanes stride the reduction
// dimension with 16-byte loads, fixed-order wave reduction.  Launches and dependent loads bound small
// blocks, reading the weights again for every pair large ones.  So there are two launches, a pair's expert
// is read straight from the choices (pair t * K + j has row t * K + j of H), and a wavefront of the second
// one has one output element with all the choices of its token, whose products it adds in slot order as the
// combine does (8 tokens, 16 experts of 256 x 128: down and combine were 4.4 + 4.2 us, now 4.0; the layer
// 22.0 -> 19.6).  F32Form has the rest.
__device__ __forceinline__ float dot_f32(const float* a, const float* b, int n, int lane) {
  const float4* pa = reinterpret_cast<const float4*>(a);
  const float4* pb = reinterpret_cast<const float4*>(b);
  float s = 0.f;
  for (int v = lane; v < n / 4; v += 64) {
    const float4 p = pa[v], q = pb[v];
    s = fmaf(p.x, q.x, s);
    s = fmaf(p.y, q.y, s);
    s = fmaf(p.z, q.z, s);
    s = fmaf(p.w, q.w, s);
  }
  return wave_sum_f32(s);
}

// Expert of pair p = t * K + j, or -1: an unused choice, or a routing launch that gave up (it
// leaves no pair a position).
__device__ __forceinline__ int f32_expert(const FfnArgs& a, int p) {
  const int pos = a.pos[p], e = a.topk_idx[p];
  return pos >= 0 && e < a.M ? e : -1;
}

// grid.x = pair, then the shared expert's tokens; grid.y tiles the F rows.
// SORTED: pairs in the order of their experts, so that workgroups that run together read the same rows.
template <bool SORTED>
__global__ __launch_bounds__(256) void gateup_f32_kernel(FfnArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int TK = a.T * a.K;
  const bool sh = static_cast<int>(blockIdx.x) >= TK;
  int r = blockIdx.x;
  if (SORTED && !sh) {
    if (r >= a.meta[1]) return;  // (fewer pairs than choices)
    const int p0 = a.pair_tok[r] * a.K;
    int j = 0;
    while (j < a.K - 1 && a.pos[p0 + j] != r) ++j;
    r = p0 + j;
  }
  const int e = sh ? 0 : f32_expert(a, r);
  if (e < 0) return;
  const int F = sh ? a.Fs : a.F, tok = sh ? r - TK : r / a.K;
  const float* xg = static_cast<const float*>(a.x) + static_cast<size_t>(tok) * a.D;
  const float* wg = sh ? static_cast<const float*>(a.sg)
                       : static_cast<const float*>(a.wg) + static_cast<size_t>(e) * a.F * a.D;
  const float* wu = sh ? static_cast<const float*>(a.su)
                       : static_cast<const float*>(a.wu) + static_cast<size_t>(e) * a.F * a.D;
  float* h = static_cast<float*>(a.h) +
             (sh ? static_cast<size_t>(TK) * a.F + static_cast<size_t>(tok) * a.Fs : static_cast<size_t>(r) * a.F);
  for (int f = blockIdx.y * 4 + wave; f < F; f += gridDim.y * 4) {
    const float g = dot_f32(xg, wg + static_cast<size_t>(f) * a.D, a.D, lane);
    const float u = dot_f32(xg, wu + static_cast<size_t>(f) * a.D, a.D, lane);
    if (lane == 0) h[f] = silu_f(g) * u;
  }
}

// y[t][d]: grid.x = token, grid.y tiles the D rows.  J choices at a time: their rows of H and
// of the weights are in flight together.
template <int J>
__global__ __launch_bounds__(256) void down_combine_f32_kernel(FfnArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = blockIdx.x, K = a.K, D = a.D, n4 = a.F / 4;
  const size_t TK = static_cast<size_t>(a.T) * K;
  const float* h = static_cast<const float*>(a.h);
  for (int d = blockIdx.y * 4 + wave; d < D; d += gridDim.y * 4) {
    const size_t yo = static_cast<size_t>(t) * D + d;
    const float xv = a.residual ? static_cast<const float*>(a.x)[yo] : 0.f;
    float acc = 0.f;
    for (int j0 = 0; j0 < K; j0 += J) {
      const float4 *ph[J], *pw[J];
      float g[J], s[J];
      int e[J];
#pragma unroll
      for (int u = 0; u < J; ++u) {
        const int p = t * K + min(j0 + u, K - 1);
        e[u] = j0 + u < K ? f32_expert(a, p) : -1;
        g[u] = a.topk_w[p];
        s[u] = 0.f;
        ph[u] = reinterpret_cast<const float4*>(h + static_cast<size_t>(p) * a.F);
        pw[u] = reinterpret_cast<const float4*>(static_cast<const float*>(a.wd) +
                                                (static_cast<size_t>(max(e[u], 0)) * D + d) * a.F);
      }
      if (J == 1) {
        const float *hr = reinterpret_cast<const float*>(ph[0]), *wr = reinterpret_cast<const float*>(pw[0]);
        if (e[0] >= 0) acc = fmaf(g[0], dot_f32(hr, wr, a.F, lane), acc);
        continue;
      }
      for (int v = lane; v < n4; v += 64) {
        float4 q[J], w[J];
#pragma unroll
        for (int u = 0; u < J; ++u)
          if (e[u] >= 0) {
            q[u] = ph[u][v];
            w[u] = pw[u][v];
          }
#pragma unroll
        for (int u = 0; u < J; ++u)
          if (e[u] >= 0) {
            s[u] = fmaf(q[u].x, w[u].x, s[u]);
            s[u] = fmaf(q[u].y, w[u].y, s[u]);
            s[u] = fmaf(q[u].z, w[u].z, s[u]);
            s[u] = fmaf(q[u].w, w[u].w, s[u]);
          }
      }
#pragma unroll
      for (int u = 0; u < J; ++u)
        if (e[u] >= 0) acc = fmaf(g[u], wave_sum_f32(s[u]), acc);
    }
    if (a.Fs > 0)
      acc += dot_f32(h + TK * a.F + static_cast<size_t>(t) * a.Fs,
                     static_cast<const float*>(a.sd) + static_cast<size_t>(d) * a.Fs, a.Fs, lane);
    if (a.residual) acc += xv;
    if (lane == 0) static_cast<float*>(a.y)[yo] = acc;
  }
}

// ---------------------------------------------------------------- combine
// y[t][d] = sum_j topk_w[t][j] * O[pos[t*K+j]][d]  (slot order j = 0..K-1)
//           (+ O[TK + t][d] shared) (+ x[t][d] residual); 4 columns per thread.
__global__ __launch_bounds__(256) void combine_kernel(FfnArgs a) {
  const int t = blockIdx.x;
  const int d = (blockIdx.y * 256 + threadIdx.x) * 4;
  if (a.dn.on && blockIdx.x == 0 && blockIdx.y == 0) {
    // dense short block: cnt_i and the number of experts that received a token, from
    // the bitmaps stage 2 left (integer work, the same whatever the order)
    __shared__ int s_live;
    if (threadIdx.x == 0) s_live = 0;
    __syncthreads();
    int live = 0;
    for (int e = threadIdx.x; e < a.M; e += 256) {
      const int sl = a.dn.slot_of[e];
      const int c = (sl >= 0 && sl < a.n_slots) ? __popc(a.dn.tokmask[sl]) : 0;
      a.dn.expert_counts[e] = c;
      live += c > 0 ? 1 : 0;
    }
    if (live) atomicAdd(&s_live, live);
    __syncthreads();
    // (a negative value was put there by a routing launch that gave up, or carried over
    // from an earlier layer of a stack: it stays)
    if (threadIdx.x == 0 && a.dn.n_unique[0] >= 0) a.dn.n_unique[0] = s_live;
  }
  if (d >= a.D) return;
  const int K = a.K;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  // eight slots at a time: their position, gate and output-row loads are all in
  // flight together; the sum still runs in slot order
  for (int j0 = 0; j0 < K; j0 += 8) {
    int r[8];
    float w[8];
    float4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool in = j0 + u < K;
      r[u] = in ? a.pos[t * K + j0 + u] : -1;
      w[u] = in ? a.topk_w[t * K + j0 + u] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = r[u] >= 0 ? *reinterpret_cast<const float4*>(a.o + static_cast<size_t>(r[u]) * a.D + d)
                       : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (r[u] < 0) continue;
      acc.x = fmaf(w[u], v[u].x, acc.x);
      acc.y = fmaf(w[u], v[u].y, acc.y);
      acc.z = fmaf(w[u], v[u].z, acc.z);
      acc.w = fmaf(w[u], v[u].w, acc.w);
    }
  }
  if (a.Fs > 0) {
    const size_t r = static_cast<size_t>(a.T) * K + t;
    const float4 v = *reinterpret_cast<const float4*>(a.o + r * a.D + d);
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  const size_t xo = static_cast<size_t>(t) * a.D + d;
  if (a.residual) {
    const u16x4 xv = *reinterpret_cast<const u16x4*>(static_cast<const uint16_t*>(a.x) + xo);
    acc.x += bf16_bits_to_f32(xv[0]); acc.y += bf16_bits_to_f32(xv[1]);
    acc.z += bf16_bits_to_f32(xv[2]); acc.w += bf16_bits_to_f32(xv[3]);
  }
  u16x4 out;
  out[0] = f32_to_bf16_bits(acc.x); out[1] = f32_to_bf16_bits(acc.y);
  out[2] = f32_to_bf16_bits(acc.z); out[3] = f32_to_bf16_bits(acc.w);
  *reinterpret_cast<u16x4*>(static_cast<uint16_t*>(a.y) + xo) = out;
}

// ------------------------------------------------------------------ packing
// dst tile layout documented in des.h (des_pack_expert_weights).
__global__ __launch_bounds__(256) void pack_kernel(const uint16_t* __restrict__ src,
                                                   uint16_t* __restrict__ dst, int rows, int cols,
                                                   long long groups_total) {
  // one thread per group of 8 values
  const long long g = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x;
  if (g >= groups_total) return;
  const long long per_mat = static_cast<long long>(rows) * cols / 8;
  const long long m = g / per_mat;
  long long q = g % per_mat;
  const int l = static_cast<int>(q % 64);
  q /= 64;
  const int ct = static_cast<int>(q % (cols / 32));
  const int rt = static_cast<int>(q / (cols / 32));
  const uint16_t* s = src + m * rows * cols + static_cast<long long>(rt * 16 + (l & 15)) * cols +
                      ct * 32 + 8 * (l >> 4);
  *reinterpret_cast<uint4*>(dst + g * 8) = *reinterpret_cast<const uint4*>(s);
}

int launch_pack(const void* src, void* dst, int64_t n_mats, int rows, int cols, hipStream_t st) {
  const long long groups = n_mats * rows * static_cast<long long>(cols) / 8;
  const long long blocks = (groups + 255) / 256;
  launch(kKPack, pack_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st,
         static_cast<const uint16_t*>(src), static_cast<uint16_t*>(dst), rows, cols, groups);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DES_OK : hip_fail(e, "pack launch");
}

// ------------------------------------------------------------- read ceiling
// Bare streaming read: every wavefront pulls one contiguous 64 KB chunk with
// sixteen 16-byte loads per lane in flight and does nothing else.  What this
// reaches is the machine's practical ceiling for a weight scan, the figure
// the FFN kernels are quoted against beside the 8 TB/s data-sheet peak.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int kProbeChunk = 65536;

__global__ __launch_bounds__(kWave) void read_probe_kernel(const u32x4* __restrict__ src,
                                                           u32x4* __restrict__ sink) {
  constexpr int kVecs = kProbeChunk / 16, kU = 16;
  const u32x4* p = src + static_cast<size_t>(blockIdx.x) * kVecs + threadIdx.x;
  u32x4 acc = {0, 0, 0, 0};
  for (int i = 0; i < kVecs; i += kWave * kU) {
    u32x4 v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = __builtin_nontemporal_load(p + i + u * kWave);
#pragma unroll
    for (int u = 0; u < kU; ++u) acc ^= v[u];
  }
  // keeps the loads alive; the pattern does not occur in real data
  if (acc.x == 0x12345678u && acc.y == 0x9abcdef0u && acc.z == 0x0fedcba9u) sink[0] = acc;
}

int launch_read_probe(const void* src, size_t bytes, void* sink, hipStream_t st) {
  launch(kKProbe, read_probe_kernel, dim3(static_cast<unsigned>(bytes / kProbeChunk)), dim3(kWave), 0,
         st, static_cast<const u32x4*>(src), static_cast<u32x4*>(sink));
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DES_OK : hip_fail(e, "read probe launch");
}

// ------------------------------------------------------------------ launcher
// How an fp32 layer's two launches run (times are of the launch concerned, in us).
struct F32Form {
  bool sorted;     // gate/up takes the pairs in the order of their experts
  int at_once;     // choices of a token whose rows down has in flight together
  int down_tiles;  // workgroups of down per token
};
static F32Form f32_form(const des_shape_t& s) {
  const int TK = s.n_seqs * s.n_tokens * s.top_k;
  // The order of the experts costs dependent loads and spreads a token's row of x, and it pays where an
  // expert is large and the pairs are more than run together: 128 experts of 2048 x 768, k = 8, vanilla, 128
  // tokens 1088 in the order of the tokens and 974 in that of the experts, 512 tokens 4444 and 3579; a coreset
  // of 32 of them, 8 tokens 106 and 130, 128 level, 256 2126 and 1851; 16 of 4096 x 1024, 128 pairs 293 and 269,
  // 1024 pairs 2109 and 1923.  Experts of 1024 x 512 and less stay ahead in token order up to 4096 pairs
  // (1029 and 1174; of 512 x 256 270 and 341).  At 96 to 192 pairs without a coreset the line costs up to 7 %.
  const size_t expert = static_cast<size_t>(s.ffn) * s.hidden;
  const int pairs = expert >= (4u << 20) ? 128 : 2 * max_live_experts(s) > s.n_experts ? 256 : 1024;
  // Choices side by side hide the loads of few tokens (16 tokens: 16 experts of 4096 x 1024, k = 4, 81 and one
  // after the other 104; 32 of 1536 x 1408 58 and 69); with more the chip is full without (64 tokens, 128 of
  // 2048 x 768, k = 8: 270 and 248).
  const int at_once = s.top_k == 1 || TK > 128 ? 1 : 4;
  // A wavefront per output element: one token of width 2048, k = 8, takes 10 us so, 38 in 64 workgroups.  With
  // one choice per token what leads to the first product is worth sharing among several elements: 512 tokens,
  // 16 experts of 512 x 256, 45 and 34.
  const int most = s.top_k == 1 && s.n_seqs * s.n_tokens >= 64 ? 64 : 1024, d4 = (s.hidden + 3) / 4;
  return F32Form{expert >= (1u << 20) && TK >= pairs, at_once, d4 < most ? d4 : most};
}

void f32_plan(const des_shape_t& s, int32_t* plan) {
  const F32Form f = f32_form(s);
  const bool on = s.dtype == DES_F32;
  plan[0] = on && f.sorted; plan[1] = on ? f.at_once : 0; plan[2] = on ? f.down_tiles : 0; plan[3] = 0;
}

int launch_ffn(const des_shape_t& s, const LayerForm& form, const void* x, const void* w_gate,
               const void* w_up, const void* w_down, const void* ws_gate, const void* ws_up,
               const void* ws_down, const float* logits, int32_t* topk_idx, float* topk_w, int32_t* expert_counts,
               int32_t* n_unique, void* y, char* ws, unsigned long long epoch, hipStream_t st) {
  const WsLayout w = ws_layout(s);
  FfnArgs a;
  a.x = x;
  a.wg = w_gate; a.wu = w_up; a.wd = w_down;
  a.sg = ws_gate; a.su = ws_up; a.sd = ws_down;
  a.topk_idx = topk_idx;
  a.topk_w = topk_w;
  a.slots = reinterpret_cast<const int4*>(ws + w.slots);
  a.meta = reinterpret_cast<const int32_t*>(ws + w.meta);
  a.pair_tok = reinterpret_cast<const int32_t*>(ws + w.pair_tok);
  a.units = reinterpret_cast<const int32_t*>(ws + w.units);
  a.pos = reinterpret_cast<const int32_t*>(ws + w.pos);
  a.h = ws + w.h;
  a.o = reinterpret_cast<float*>(ws + w.o);
  a.y = y;
  a.T = s.n_seqs * s.n_tokens;
  a.D = s.hidden; a.M = s.n_experts; a.F = s.ffn; a.Fs = s.ffn_shared; a.K = s.top_k;
  a.n_slots = max_live_experts(s);
  a.residual = s.residual;
  a.splits = 1;
  a.h_rows = w.h_rows;
  a.xo = form.x_copy ? reinterpret_cast<const uint16_t*>(ws + w.o) : nullptr;
  a.dn = DenseArgs{};
  int n_s2 = 0;  // wavefronts of the gate/up launch that run stage 2 (dense short block)
  if (form.dense) {
    a.dn.on = 1;
    a.dn.lpt = 1024 / selector_tokens_per_pass(s.n_experts);
    a.dn.sigmoid = s.router_act == DES_ROUTER_SIGMOID;
    a.dn.logits = logits;
    a.dn.topk_idx = topk_idx;
    a.dn.topk_w = topk_w;
    a.dn.slot_of = reinterpret_cast<const int32_t*>(ws + w.slot_of);
    a.dn.tokmask = reinterpret_cast<uint32_t*>(ws + w.tokmask);
    a.dn.choice = reinterpret_cast<uint8_t*>(ws + w.choice);
    a.dn.pos = reinterpret_cast<int32_t*>(ws + w.pos);
    a.dn.expert_counts = expert_counts;
    a.dn.n_unique = n_unique;
    n_s2 = (a.T * a.dn.lpt + 63) / 64;
  }
  const int TK = a.T * a.K;

  if (s.dtype == DES_BF16) {
    const bool packed = s.weight_layout == DES_LAYOUT_PACKED;
    const int gu_tasks = a.n_slots * (a.F / (16 * kGuTiles)) + a.Fs / (16 * kGuTiles);
    const int gu_blocks = (gu_tasks + n_s2 + kFfnWaves - 1) / kFfnWaves;
    const int groups = (a.D / 16 + 3) / 4;
    const int dn_tasks = a.n_slots * groups + (a.Fs > 0 ? groups : 0);
    const int dn_blocks = (dn_tasks + kFfnWaves - 1) / kFfnWaves;
    // an expert serves a token at most once, so no task has more than T pairs
    const int maxnt = (a.T + 15) / 16;
    const dim3 blk(kFfnWaves * kWave);
    // Few experts (small coreset): halve the task size so that enough wavefronts keep bytes in
    // flight; a halved down task should still stream >= 48 KB (F >= 768).  2048 x 768, whole and
    // halved tasks, in us: gate/up under 8 tokens 13.5 and 9.4 at 192 tasks, 16.8 and 17.2 at
    // 384, 25.9 and 24.8 at 768; under 32 tokens 15.7 and 13.4, 20.1 and 20.1, 32.7 and 37.0.
    // Down under 8 tokens 7.8 and 6.1 at 256 tasks, 9.4 and 9.3 at 512, 12.1 and 11.9 at 1024;
    // under 32 tokens 9.8 and 9.4, 11.3 and 12.7, 20.4 and 19.7.
    const bool gu_fine = gu_tasks < 512;
    const bool dn_fine = dn_tasks <= 1024 && a.F >= 768;
    const int gu_fine_tasks = a.n_slots * (a.F / 16) + a.Fs / 16;
    const int dn_fine_groups = (a.D / 16 + 1) / 2;
    const int dn_fine_tasks = a.n_slots * dn_fine_groups + (a.Fs > 0 ? dn_fine_groups : 0);
#define DES_LAUNCH_FFN(NTV, PK)                                                             \
  do {                                                                                      \
    if (gu_fine)                                                                \
      launch(kKGateUp, gateup_bf16_kernel<NTV, PK, 4, 4, 1>, dim3(gu_fine_tasks + n_s2), blk, 0, st, a); \
    else                                                                                    \
      launch(kKGateUp, gateup_bf16_kernel<NTV, PK>, dim3(gu_blocks), blk, 0, st, a);        \
    if (dn_fine)                                                                \
      launch(kKDown, down_bf16_kernel<NTV, PK, 4, 4, 2>, dim3(dn_fine_tasks), blk, 0, st, a); \
    else                                                                                    \
      launch(kKDown, down_bf16_kernel<NTV, PK>, dim3(dn_blocks), blk, 0, st, a);            \
  } while (0)
    if (a.T > 32) {
      // Longer blocks: units of 64 token rows while no expert can have more, else 128; an
      // expert with more pairs has several of them (the unit list).
      //
      // Three forms of each kernel: streamed with four weight tiles per wavefront (below), streamed
      // with two, tiles.  Streamed (weights straight into operands, token rows through LDS): packed
      // weights whose reduction is one of the unrolled ones - or, with fewer than 32 pairs per
      // possible expert, any whole number of its chunks.  Tiles (both through LDS): everything else.
      // 128 experts of 2048 x 768 under 256 tokens, gate/up + down: packed 68.3 + 40.0 us streamed,
      // 77.6 + 43.6 in tiles; row-major (64 bytes of a row per operand load) 99.9 + 54.8 and 81.3 +
      // 45.0.  64 experts of 1536 x 1408, packed, not unrolled: 16 pairs per expert 78.0 + 50.0 and
      // 80.5 + 51.6, 32 pairs 111 + 64.9 and 98.5 + 56.5, 128 pairs 223 + 126 and 168 + 97.  Sizes
      // that are no multiple of the streamed chunk had one wavefront per 16 or 32 weight rows gather
      // everything from L2 (64 experts of 1440 x 288, packed, 200 tokens, 12 pairs per expert:
      // gate/up 60.2, in tiles 22.8).
      const int rows_pass = lds_rows_pass(a.T);
      const bool small = rows_pass == 64;
      int splits = (a.T + rows_pass - 1) / rows_pass;  // of the shared expert (all T rows)
      if (splits > kMaxSplits) splits = kMaxSplits;
      a.splits = splits;
      const int n_units = max_units(s);
      // unrolled reduction lengths (the shared expert shares the down launch)
      const int gu_kd = a.D == 2048 ? 2048 : 0;
      const int dn_kd = (a.Fs != 0 && a.Fs != a.F) ? 0 : (a.F == 768 || a.F == 512) ? a.F : 0;
      const bool few = TK < 32 * a.n_slots;
      const bool gu_stream = packed && a.D % kKC == 0 && (gu_kd > 0 || few);
      const bool dn_stream = packed && a.F % kKC == 0 && a.Fs % kKC == 0 && (dn_kd > 0 || few);
#define DES_LAUNCH_GU(MNT, LWV)                                                             \
  do {                                                                                      \
    if (gu_kd == 2048) launch(kKGateUp, gateup_lds_kernel<MNT, LWV, 2048, 2>, gg, dim3(LWV* kWave), 0, st, a); \
    else launch(kKGateUp, gateup_lds_kernel<MNT, LWV, 0, 2>, gg, dim3(LWV* kWave), 0, st, a);  \
  } while (0)
#define DES_LAUNCH_DN(MNT, LWV)                                                             \
  do {                                                                                      \
    if (dn_kd == 768) launch(kKDown, down_lds_kernel<MNT, LWV, 768, 2>, dg, dim3(LWV* kWave), 0, st, a); \
    else if (dn_kd == 512) launch(kKDown, down_lds_kernel<MNT, LWV, 512, 2>, dg, dim3(LWV* kWave), 0, st, a); \
    else launch(kKDown, down_lds_kernel<MNT, LWV, 0, 2>, dg, dim3(LWV* kWave), 0, st, a);      \
  } while (0)
#define DES_LAUNCH_TILE(id, kernel, g, MT, P)                                               \
  do {                                                                                      \
    const dim3 tb(kTileThreads);                                                            \
    if (packed && small) launch(id, kernel<true, 2, MT, P>, g, tb, 0, st, a);               \
    else if (packed) launch(id, kernel<true, 4, MT, P>, g, tb, 0, st, a);                   \
    else if (small) launch(id, kernel<false, 2, MT, P>, g, tb, 0, st, a);                   \
    else launch(id, kernel<false, 4, MT, P>, g, tb, 0, st, a);                              \
  } while (0)
      // Tiles: four row tiles per wavefront share a token fragment where there is enough to do,
      // two make twice the workgroups where there is not, and with two chunks requested ahead
      // they hide more of a chunk's way.  Counted in workgroups of the larger tile (for the most
      // experts that can be live).  Gate/up: below one per compute unit, two and two (4 experts
      // of 7168 x 2048, row-major, 64 tokens: 100 us -> 50, streamed 71; packed, 8 experts of
      // 4096 x 1408, 128 tokens: 60 -> 53, streamed 54); up to 1.75 per unit, two tiles but one
      // chunk (128 experts of 2048 x 768, coreset of 32, row-major, 72 tokens: 39.4 -> 36.7, with
      // two chunks 44.9; above that 128 experts under 64 tokens, vanilla: 62.6 -> 69.8).  Experts
      // with a few pairs each under units sized for 128 rows: two and two as well (128 experts of
      // 2048 x 768, 80 tokens, 5 pairs each: 76 -> 58.5, streamed 64.7).  Down: two and two up to
      // 1.5 workgroups per unit (512 x 896, 64 tokens: 10.8 -> 7.0, streamed 9.3; 592 workgroups:
      // 21.4 -> 23.5).
      auto units_of = [&](int width) { return (width + 63) / 64; };  // of 4 row tiles
      const int gu_wgs = n_units * units_of(a.F) + splits * units_of(a.Fs);
      const int dn_wgs = (n_units + (a.Fs > 0 ? splits : 0)) * ((a.D + 127) / 128);
      const bool gu_two = gu_wgs < 256 || (!small && TK < 8 * a.n_slots);
      const int gu_mt = gu_two || gu_wgs < 448 ? 2 : 4, dn_mt = dn_wgs < 384 ? 2 : 4;
      // Streamed with four weight tiles per wavefront instead of two, for packed weights and many
      // pairs per expert: a token fragment from LDS meets twice the weights and the launch can
      // reach the matrix cores' rate (16 experts of 2048 x 768, 1024 pairs each: gate/up 160 us in
      // two tiles, 105; 16 of 4096 x 1408, 2048 tokens, k = 2: 176 in LDS tiles, 121; 64 sequences
      // of 32 tokens on 128 experts: 204 and 168).  It has half as many wavefronts, each with
      // half of the room for requested weights: from 120 pairs per possible expert on, where the
      // reduction is not one of the unrolled ones and not short from 40 on (24 experts of 640 x 1152,
      // 43 pairs: 15.3 against 17.8), and with fewer than 224 workgroups (for the most experts that
      // can be live) never (32 experts of 1280 x 384, 64 pairs, 144 workgroups: 18.6 against 26.0).
      auto four = [&](int kd, bool unrolled, int wgs) {
        return packed && !small && kd % kKC == 0 && wgs >= 224 &&
               (TK >= 120 * a.n_slots || (kd >= 1152 && !unrolled && TK >= 40 * a.n_slots));
      };
      const int gu_four_wgs = n_units * ((a.F + 127) / 128) + splits * ((a.Fs + 127) / 128);
      const int dn_four_wgs = (n_units + (a.Fs > 0 ? splits : 0)) * ((a.D + 255) / 256);
      if (four(a.D, gu_kd > 0, gu_four_wgs)) {
        launch(kKGateUp, gateup_lds_kernel<8, 4, 0, 4>, dim3(gu_four_wgs), dim3(4 * kWave), 0, st, a);
      } else if (gu_stream) {
        // Wavefronts per workgroup: two give the finest spread of the weight bytes over the
        // compute units; four share the staged activations among more weight rows, which
        // measured better once experts have many tokens (48-layer stack: 7.7 ms against
        // 8.0 ms; down projection at T = 128: 23 us against 27 us).
        const int lw = a.T <= 128 ? 2 : 4;
        const dim3 gg(n_units * ((a.F / 16 + lw - 1) / lw) + splits * ((a.Fs / 16 + lw - 1) / lw));
        if (small) DES_LAUNCH_GU(4, 2);
        else if (lw == 2) DES_LAUNCH_GU(8, 2);
        else DES_LAUNCH_GU(8, 4);
      } else {
        const dim3 gg(n_units * ((a.F / 16 + gu_mt - 1) / gu_mt) + splits * ((a.Fs / 16 + gu_mt - 1) / gu_mt));
        if (gu_two) DES_LAUNCH_TILE(kKGateUp, gateup_tile_kernel, gg, 2, 2);
        else if (gu_mt == 2) DES_LAUNCH_TILE(kKGateUp, gateup_tile_kernel, gg, 2, 1);
        else DES_LAUNCH_TILE(kKGateUp, gateup_tile_kernel, gg, 4, 1);
      }
      if (a.Fs % kKC == 0 && four(a.F, dn_kd > 0, dn_four_wgs)) {
        launch(kKDown, down_lds_kernel<8, 4, 0, 4>, dim3(dn_four_wgs), dim3(4 * kWave), 0, st, a);
      } else if (dn_stream) {
        const int lw = a.T <= 64 ? 2 : 4;
        const int per = (a.D / 32 + lw - 1) / lw;
        const dim3 dg(n_units * per + (a.Fs > 0 ? splits * per : 0));
        if (small) DES_LAUNCH_DN(4, 2);
        else DES_LAUNCH_DN(8, 4);
      } else {
        const int per = (a.D / 16 + 2 * dn_mt - 1) / (2 * dn_mt);
        const dim3 dg(n_units * per + (a.Fs > 0 ? splits * per : 0));
        if (dn_mt == 2) DES_LAUNCH_TILE(kKDown, down_tile_kernel, dg, 2, 2);
        else DES_LAUNCH_TILE(kKDown, down_tile_kernel, dg, 4, 1);
      }
#undef DES_LAUNCH_GU
#undef DES_LAUNCH_DN
#undef DES_LAUNCH_TILE
    } else if (packed) {
      if (maxnt <= 1) DES_LAUNCH_FFN(1, true);
      else DES_LAUNCH_FFN(2, true);
    } else {
      if (maxnt <= 1) DES_LAUNCH_FFN(1, false);
      else DES_LAUNCH_FFN(2, false);
    }
#undef DES_LAUNCH_FFN
    dim3 cg(a.T, (a.D / 4 + 255) / 256);
    launch(kKCombine, combine_kernel, cg, dim3(256), 0, st, a);
  } else {
    const int rows = TK + (a.Fs > 0 ? a.T : 0);
    const int Fm = a.F > a.Fs ? a.F : a.Fs;
    const F32Form f = f32_form(s);
    const dim3 gu(rows, (Fm + 3) / 4 > 64 ? 64 : (Fm + 3) / 4), gd(a.T, f.down_tiles), block(256);
    if (f.sorted) launch(kKGateUp, gateup_f32_kernel<true>, gu, block, 0, st, a);
    else launch(kKGateUp, gateup_f32_kernel<false>, gu, block, 0, st, a);
    if (f.at_once == 1) launch(kKDown, down_combine_f32_kernel<1>, gd, block, 0, st, a);
    else launch(kKDown, down_combine_f32_kernel<4>, gd, block, 0, st, a);
  }
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DES_OK : hip_fail(e, "ffn launch");
}

}  // namespace des

#ifdef DES_FFN_STAMPS
extern "C" int des_debug_ffn_stamps(long long* host, int n) {
  return hipMemcpyFromSymbol(host, HIP_SYMBOL(des::g_ffn_stamps), sizeof(long long) * n) == hipSuccess
             ? 0 : -6;
}
#endif
