// Streaming GEMM building blocks: the pieces that the short-block kernels share, and the one
// of the expert FFN's kernels that stage token rows through LDS (packed weights, more than 32
// tokens): weights from HBM straight into MFMA operands, token rows from L2 into LDS by direct
// loads, explicit wait counts.  gfx950 only.
#pragma once

#include <type_traits>
#include <utility>

#include "des_common.h"

namespace des {

typedef std::integral_constant<int, 0> S0;
typedef std::integral_constant<int, 1> S1;

// elements between consecutive k-steps of a 16-row weight tile
template <bool PACKED>
__device__ __forceinline__ constexpr int frag_step() { return PACKED ? 512 : 32; }

// ------------------------------------------ short blocks: weights straight into operands
// The weight stream of one wavefront: `steps` stages in two register sets.  load(st, set)
// requests stage st, compute(set) multiplies it.  The trips carry no branch, so the
// compiler waits for exactly the stage it needs and the next one stays in flight (with a
// test for the end around each load it waited for everything outstanding); the scheduling
// barriers keep a stage's loads together in front of the multiplies.  More sets do not
// help: what bounds these kernels is the chip's read rate and its spread over the compute
// units (128-expert layer, 32 tokens: 34.4 us with two, three or four sets of two k-steps;
// where fewer wavefronts are in flight the branch-free form pays: 16 of 256 experts 22.3 ->
// 20.0 us, 4 tokens 20.2 -> 18.6 us, the down projections 12.1 -> 11.1 and 12.0 -> 10.6).
// Every condition around a matrix instruction must be uniform to the compiler as well as in
// fact (`steps` from kernel arguments, or through uniform_int): matrix instructions ignore
// the execution mask, and a short block under a mask that the compiler takes for divergent
// may be entered with all lanes off.
template <typename Load, typename Compute>
__device__ __forceinline__ void stream_pipeline(int steps, Load&& load, Compute&& compute) {
  if (steps > 0) load(0, S0{});
  int st = 0;
  for (; st + 3 <= steps; st += 2) {
    load(st + 1, S1{});
    __builtin_amdgcn_sched_barrier(0);
    compute(S0{});
    __builtin_amdgcn_sched_barrier(0);
    load(st + 2, S0{});
    __builtin_amdgcn_sched_barrier(0);
    compute(S1{});
    __builtin_amdgcn_sched_barrier(0);
  }
  if (st < steps) {
    if (st + 1 < steps) load(st + 1, S1{});
    compute(S0{});
    if (st + 1 < steps) compute(S1{});
  }
}

// Row-major weights.  An MFMA A operand takes 16 rows x 32 elements, 64 bytes of each
// row: a load in operand order touches 16 half lines, and the kernels then ran at 3.6 TB/s
// where packed tiles reach 5.8 (33 experts of 2048 x 768: gate/up 58.4 us, down 31.8 us; as
// below 44.4 and 23.2, packed 42.5 and 21.8).  So row-major tiles are loaded in whole
// 128-byte lines (a load = 8 rows x 64 elements, lane l has piece l % 8 of row l / 8) and
// turned into operand order through a few KB of LDS that belong to the wavefront alone: two loads (v[0], v[1]: rows 0-7 and 8-15) become the
// operands of two k-steps.  16-byte piece p of row r is kept at piece p ^ (r / 2 % 8), so
// writes and reads both spread over all banks.
constexpr int kTurnBytes = 2048;  // of LDS per 16 x 64 tile
__device__ __forceinline__ void turn_write(const bf16x8& v0, const bf16x8& v1, char* tile, int lane) {
  const int r = lane >> 3, p = lane & 7;
  *reinterpret_cast<bf16x8*>(tile + r * 128 + ((p ^ (r >> 1)) << 4)) = v0;
  *reinterpret_cast<bf16x8*>(tile + (r + 8) * 128 + ((p ^ ((r >> 1) + 4)) << 4)) = v1;
}
__device__ __forceinline__ bf16x8 turn_read(const char* tile, int u, int lane) {
  const int r = lane & 15, p = u * 4 + (lane >> 4);
  return *reinterpret_cast<const bf16x8*>(tile + r * 128 + ((p ^ (r >> 1)) << 4));
}
// the wavefront's LDS accesses stay in program order (they execute in order)
__device__ __forceinline__ void turn_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------ token rows via LDS, weights via registers
// With more than two token tiles per expert the direct scheme above runs out
// of registers for its prefetch (every token fragment is double-buffered in
// registers).  For T > 32 the expert's activation rows go through LDS instead:
//   * a workgroup of LW wavefronts works on LW weight-row groups of one expert;
//     each wavefront streams its own two weight tiles from HBM straight into
//     MFMA operands, three chunks of 128 reduction elements deep, so that two
//     chunks (16 KB per wavefront) stay in flight across every barrier;
//   * the expert's token rows of the next chunk are gathered from L2 into LDS
//     by direct global-to-LDS loads (no staging registers), double-buffered;
//   * LDS rows are 256 B with the 16-byte pieces of row r stored at piece
//     index p ^ (r & 15): a direct load writes lane l at base + 16*l, so the
//     swizzle is applied on the global side (which piece a lane fetches), and
//     the 16 token rows an MFMA operand reads fall into 16 different banks.
// The compiler does not know about the direct loads (they are asm): it neither waits for
// them nor for the weights, explicit vmcnt counts do.  The token fragments are volatile LDS
// reads, which keeps them in program order with the asm statements and the barriers; the
// compiler counts them itself, so the next fragments are on their way while one group is
// multiplied (128-expert layer, 128 tokens: gate/up 41.9 us with a wait after every group,
// 39.9 us so; experts of 512 x 896, 112 tokens: 11.3 and 10.3 us; 8 x 32 and 64 x 32 tokens of
// the former: no difference).  None of the asm statements claims
// to touch memory (a "memory" clobber makes the compiler wait for every pending load first);
// they are volatile, which keeps them in program order with each other and the barriers.
constexpr int kKC = 128;            // reduction lengths must be multiples of this
#define DES_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// One 16-byte weight fragment, asynchronously: the register is valid only after
// a wait_weights() that names it.  (The compiler's own vmcnt bookkeeping gives
// up across the rotating stages and early exits of the chunk loop and waits for
// everything at every use, which would drain the prefetch; so these loads and
// their waits are explicit.)
template <int OFF>
__device__ __forceinline__ void ld8_async(bf16x8& v, const uint16_t* ubase, uint32_t lane_off) {
  // s_nop 4: the base may have just been written by a vector instruction (a
  // scalar register restored from a spill lane); a vector-memory instruction
  // needs five wait states after that, and the compiler adds none inside asm.
  asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %1, %2 offset:%3 nt"
               : "=v"(v)
               : "v"(lane_off), "s"(ubase), "n"(OFF));
}
// A pointer the compiler may keep in scalar registers (the value is the same in all lanes).
template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return reinterpret_cast<T*>((static_cast<unsigned long long>(hi) << 32) | lo);
}
// Weight tile rt of a packed [rows][kd] matrix (uniform), and a lane's byte offset in a fragment.
__device__ __forceinline__ const uint16_t* tile_base(const uint16_t* base, int rt, int kd) {
  return base + static_cast<size_t>(rt) * 16 * kd;
}
__device__ __forceinline__ uint32_t tile_lane_off(int lane) { return lane * 16u; }
// Waits until at most N vector-memory operations are outstanding and makes the
// fragments of a stage depend on that wait.
template <int N>
__device__ __forceinline__ void wait_weights(bf16x8 (&a)[4], bf16x8 (&b)[4]) {
  asm volatile("s_waitcnt vmcnt(%8)"
               : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]),
                 "+v"(b[3])
               : "n"(N));
}
template <int N>
__device__ __forceinline__ void wait_weights(bf16x8 (&a)[2], bf16x8 (&b)[2]) {
  asm volatile("s_waitcnt vmcnt(%4)" : "+v"(a[0]), "+v"(a[1]), "+v"(b[0]), "+v"(b[1]) : "n"(N));
}

template <int... I, typename F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}

// acc0/acc1 += A0/A1 (this wavefront's two 16-row weight tiles, reduction
// length kd) x token rows.  KC = reduction elements per chunk (128 or 64), KD =
// the reduction length if known at compile time (then kd == KD), else 0; kd is a
// multiple of KC.  Row r of the pass (r < 16*NT) is `base + row_off(min(r,
// rows_valid-1))`.  `lds` is the workgroup's buffer of NB * ROWS * 2*KC bytes
// (ROWS >= 16*NT), NB = 3 if KD > 0, else 2.  All LW wavefronts of the workgroup call it together;
// a0, a1, base and `wave` are wavefront-uniform; w_lane_off is the lane's byte
// offset inside a weight fragment.
//
// LDS rows hold one chunk of a token row (2*KC bytes) with the 16-byte piece p
// of row r stored at piece index p ^ swz(r), swz(r) = r & 15 for 256-byte rows,
// (r >> 1) & 7 for 128-byte rows: the 16 token rows an MFMA operand reads fall
// into 16 different bank groups.  A direct load writes lane l at base + 16*l,
// so the swizzle is applied on the global side (which piece a lane fetches).
//
// A wavefront without a tile of its own (row tiles not a multiple of LW) runs
// on tile 0 and drops its result.
template <int NT, int ROWS, int LW, int KC, int KD, typename RowOff>
__device__ __forceinline__ void dma_stream_gemm(const uint16_t* a0, const uint16_t* a1,
                                                uint32_t w_lane_off, int wave, int kd,
                                                int rows_valid, const uint16_t* base,
                                                RowOff row_off, uint16_t* lds,
                                                f32x4 (&acc0)[NT], f32x4 (&acc1)[NT]) {
  static_assert(KC == 128 || KC == 64, "chunk of 4 or 2 k-steps");
  static_assert(KD % KC == 0, "reduction length must be whole chunks");
  const int lane = threadIdx.x & 63;
  const int nchunks = kd / KC;
  constexpr int NCH = KD / KC;
  constexpr int KS = KC / 32;        // k-steps per chunk
  constexpr int RB = KC * 2;         // bytes of a token row in LDS
  constexpr int PP = KC / 8;         // 16-byte pieces per row
  constexpr int RPI = 64 / PP;       // rows one direct load (64 lanes x 16 B) covers
  constexpr int NG = 16 * NT / RPI;  // direct loads per chunk (RPI rows each)
  constexpr int ND = (NG + LW - 1) / LW;  // ... per wavefront: every wavefront issues as many,
                                     // so that the wait counts below hold for all of them; one
                                     // without a group of its own repeats the last group
                                     // (same bytes to the same place)
  constexpr int NW = 2 * KS;         // weight loads per wavefront and chunk
  constexpr int kBufBytes = ROWS * RB;
  constexpr int kTile = 16 * RB;     // bytes of one token tile in a buffer
  constexpr int kFragBytes = frag_step<true>() * 2;  // between k-steps of a weight tile
  auto swz = [](int r) { return KC == 128 ? (r & 15) : ((r >> 1) & 7); };
  // All addresses are a uniform base, advanced per chunk in scalar registers,
  // plus a per-lane byte offset that never changes.
  uint32_t off[ND];                  // byte offset of this lane's piece of its rows, chunk 0
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int row = min(i * LW + wave, NG - 1) * RPI + lane / PP;
    off[i] = (static_cast<uint32_t>(row_off(min(row, rows_valid - 1))) +
              (((lane % PP) ^ swz(row)) << 3)) * 2u;
  }
  // (asm, not the builtin: after the builtin the compiler waits for all
  // outstanding loads as soon as an address register is reused)
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<size_t>(DES_LDS_PTR(lds)));
  auto dma = [&](int chunk, auto bufc) {
    constexpr int bs = decltype(bufc)::value;
    const uint16_t* g = base + chunk * KC;  // uniform
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const uint32_t dst = lds0 + bs * kBufBytes + min(i * LW + wave, NG - 1) * 1024;  // uniform
      const uint32_t o = off[i];
      // Wait states the compiler would insert for its own instructions but does
      // not for asm: one between the write of M0 and the load, five between a
      // vector instruction that wrote the base registers (a scalar register
      // restored from a spill lane) and the load.
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, %1"
                   ::"v"(o), "s"(g), "s"(dst)
                   : "m0");
    }
  };
  bf16x8 aw0[KD > 0 ? 3 : 2][KS], aw1[KD > 0 ? 3 : 2][KS];
  auto loadw = [&](int chunk, auto stage) {
    constexpr int s = decltype(stage)::value;
    const uint16_t* q0 = a0 + static_cast<size_t>(chunk) * KS * frag_step<true>();
    const uint16_t* q1 = a1 + static_cast<size_t>(chunk) * KS * frag_step<true>();
    ld8_async<0 * kFragBytes>(aw0[s][0], q0, w_lane_off);
    ld8_async<0 * kFragBytes>(aw1[s][0], q1, w_lane_off);
    ld8_async<1 * kFragBytes>(aw0[s][1], q0, w_lane_off);
    ld8_async<1 * kFragBytes>(aw1[s][1], q1, w_lane_off);
    if constexpr (KS == 4) {
      ld8_async<2 * kFragBytes>(aw0[s][2], q0, w_lane_off);
      ld8_async<2 * kFragBytes>(aw1[s][2], q1, w_lane_off);
      ld8_async<3 * kFragBytes>(aw0[s][3], q0, w_lane_off);
      ld8_async<3 * kFragBytes>(aw1[s][3], q1, w_lane_off);
    }
  };
  // byte offset in a buffer of this lane's fragment of token tile 0, k-step u of a chunk
  uint32_t fa[KS];
#pragma unroll
  for (int u = 0; u < KS; ++u) fa[u] = (lane & 15) * RB + (((u * 4 + (lane >> 4)) ^ swz(lane & 15)) << 4);
  typedef __attribute__((address_space(3))) const volatile bf16x8 LdsFrag;
  const auto lds_base = reinterpret_cast<__attribute__((address_space(3))) const volatile char*>(DES_LDS_PTR(lds));
  auto compute = [&](auto bufc, auto stage) {
    constexpr int bs = decltype(bufc)::value;
    constexpr int s = decltype(stage)::value;
    constexpr int G = NT > 4 ? NT / 2 : NT;  // token tiles fetched from LDS at a time
    constexpr int NGR = NT / G, STEPS = KS * NGR;
    bf16x8 b[2][G];
    auto fetch = [&](auto stepc) {
      constexpr int st = decltype(stepc)::value, u = st / NGR, g = st % NGR * G;
#pragma unroll
      for (int i = 0; i < G; ++i)
        b[st & 1][i] = *reinterpret_cast<LdsFrag*>(lds_base + fa[u] + bs * kBufBytes + (g + i) * kTile);
    };
    fetch(S0{});
    static_for(std::make_integer_sequence<int, STEPS>{}, [&](auto stepc) {
      constexpr int st = decltype(stepc)::value, u = st / NGR, g = st % NGR * G;
      if constexpr (st + 1 < STEPS) fetch(std::integral_constant<int, st + 1>{});
      __builtin_amdgcn_sched_barrier(0);  // (the next fragments are requested before these multiplies)
#pragma unroll
      for (int i = 0; i < G; ++i) {
        acc0[g + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw0[s][u], b[st & 1][i], acc0[g + i], 0, 0, 0);
        acc1[g + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw1[s][u], b[st & 1][i], acc1[g + i], 0, 0, 0);
      }
    });
    // every read of this buffer has come back before the next barrier lets it be overwritten
    asm volatile("s_waitcnt lgkmcnt(0)");
  };
  if constexpr (KD > 0) {
    // Reduction length known at compile time, three LDS buffers: straight-line
    // code, activations and weights both two chunks ahead.  Issue order of
    // vector-memory operations (A = this wavefront's ND activation loads of a
    // chunk, W = its NW weight loads):
    //   A(0) W(0) A(1) W(1) | step 0: A(2) W(2) | step 1: A(3) W(3) | ...
    // They complete in order, so "at most ND + NW outstanding" at the top of
    // step c means A(c) and W(c) have landed while chunk c+1 is still in flight.
    // A(c+2) overwrites the buffer chunk c-1 was read from; the barrier of step
    // c comes after everybody's reads of it.
    static_assert(ND + NW <= 63, "wait count must fit the counter");
    dma(0, S0{});
    loadw(0, S0{});
    if constexpr (NCH > 1) {
      dma(1, S1{});
      loadw(1, S1{});
    }
    static_for(std::make_integer_sequence<int, NCH>{}, [&](auto cc) {
      constexpr int c = decltype(cc)::value;
      typedef std::integral_constant<int, c % 3> Cur;
      typedef std::integral_constant<int, (c + 2) % 3> Nxt;
      if constexpr (c + 1 < NCH) wait_weights<ND + NW>(aw0[c % 3], aw1[c % 3]);
      else wait_weights<0>(aw0[c % 3], aw1[c % 3]);
      __builtin_amdgcn_s_barrier();
      if constexpr (c + 2 < NCH) {
        dma(c + 2, Nxt{});
        loadw(c + 2, Nxt{});
      }
      compute(Cur{}, Cur{});
    });
  } else {
    // Any reduction length: two stages.  Step c: everything this wavefront asked
    // for (its share of the activations of chunk c, its weights of chunk c) has
    // landed; the barrier then says the same of the other wavefronts' shares, and
    // that everybody is done reading the other buffer, which the loads of chunk
    // c+1 overwrite while chunk c is multiplied.
    auto step = [&](int c, auto bufc, auto nextbuf) {
      constexpr int s = decltype(bufc)::value;
      wait_weights<0>(aw0[s], aw1[s]);
      __builtin_amdgcn_s_barrier();
      if (c + 1 < nchunks) {
        dma(c + 1, nextbuf);
        loadw(c + 1, nextbuf);
      }
      compute(bufc, bufc);
    };
    dma(0, S0{});
    loadw(0, S0{});
    for (int c = 0; c < nchunks; c += 2) {
      step(c, S0{}, S1{});
      if (c + 1 >= nchunks) break;
      step(c + 1, S1{}, S0{});
    }
  }
  __builtin_amdgcn_s_barrier();  // nobody still reads a buffer the next pass refills
}

// Every pass works in buffers of 16 KB: up to 64 token rows with chunks of 128
// reduction elements, or up to 128 rows with chunks of 64.  Three buffers when
// the reduction length is a compile-time constant (48 KB: three workgroups per
// compute unit), else two.
constexpr int kLdsBufElems = 8192;
__host__ __device__ constexpr int lds_elems(int kd) { return (kd > 0 ? 3 : 2) * kLdsBufElems; }

}  // namespace des
