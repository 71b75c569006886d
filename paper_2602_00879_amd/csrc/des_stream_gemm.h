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
// turned into operand order through a few KB of LDS that belong to the wavefront alone: two loads
// (v[0], v[1]: rows 0-7 and 8-15) become the operands of two k-steps.  16-byte piece p of row r is kept at piece p ^ (r / 2 % 8), so
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

// Operands of 16 row-major rows x 32 elements (64 bytes of each row).  A compute unit serves a load of
// 64 x 16 bytes in 7.6 ns while every four neighbouring lanes read one 64-byte segment; in operand
// order, where they read four rows, it takes 27 ns.  So such a load runs along the rows - lane l has
// piece l % 4 of row l / 4 - and 1 KB of the wavefront's own LDS turns it into operand order.
// Piece p of row r is kept at p ^ (r / 4): the writes and any 16 consecutive lanes' reads spread over all
// banks.  The LDS does not serve a read in such runs, though: counted in the attention core, a turn has four
// cycles of bank conflicts (294,912 in 73,728 turns), where the core has none without turns.
constexpr int kOperandBytes = 1024;
__device__ __forceinline__ void operand_write(const bf16x8& v, char* at, int lane) {
  const int r = lane >> 2, p = lane & 3;
  *reinterpret_cast<bf16x8*>(at + r * 64 + ((p ^ (r >> 2)) << 4)) = v;
}
__device__ __forceinline__ bf16x8 operand_read(const char* at, int lane) {
  const int r = lane & 15, p = lane >> 4;
  return *reinterpret_cast<const bf16x8*>(at + r * 64 + ((p ^ (r >> 2)) << 4));
}
// ... one after the other through the same place
__device__ __forceinline__ bf16x8 operand_turn(const bf16x8& v, char* at, int lane) {
  turn_fence();
  operand_write(v, at, lane);
  turn_fence();
  return operand_read(at, lane);
}

// ------------------------------------------ token rows via LDS, weights via registers
// With more than two token tiles per expert the direct scheme above runs out
// of registers for its prefetch (every token fragment is double-buffered in
// registers).  For T > 32 the expert's activation rows go through LDS instead:
//   * a workgroup of LW wavefronts works on LW weight-row groups of one expert;
//     each wavefront streams its own weight tiles straight into MFMA operands;
//   * the expert's token rows are gathered from L2 into LDS by direct
//     global-to-LDS loads (no staging registers).
// Three forms: two weight tiles and a reduction known at compile time, or four tiles and any
// even number of chunks, have both requested two chunks ahead (three buffers of token rows),
// so that they stay in flight across every barrier; two tiles and any number of chunks, one
// chunk ahead (two buffers).
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
// NT_HINT: a non-temporal load, for weights that one workgroup alone reads.
template <int OFF, bool NT_HINT>
__device__ __forceinline__ void ld8_async(bf16x8& v, const uint16_t* ubase, uint32_t lane_off) {
  // s_nop 4: the base may have just been written by a vector instruction (a
  // scalar register restored from a spill lane); a vector-memory instruction
  // needs five wait states after that, and the compiler adds none inside asm.
  if constexpr (NT_HINT)
    asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %1, %2 offset:%3 nt"
                 : "=v"(v)
                 : "v"(lane_off), "s"(ubase), "n"(OFF));
  else
    asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %1, %2 offset:%3"
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
template <int N, int KS, int RT>
__device__ __forceinline__ void wait_weights(bf16x8 (&a)[KS][RT]) {
  static_assert(RT * KS == 4 || RT * KS == 8, "fragments of a stage");
  bf16x8* p = &a[0][0];
  if constexpr (RT * KS == 8)
    asm volatile("s_waitcnt vmcnt(%8)"
                 : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]), "+v"(p[4]), "+v"(p[5]), "+v"(p[6]), "+v"(p[7])
                 : "n"(N));
  else
    asm volatile("s_waitcnt vmcnt(%4)" : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]) : "n"(N));
}

template <int... I, typename F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}

// acc[r] += A[r] (this wavefront's RT 16-row weight tiles, reduction length kd) x token rows.
// KC = reduction elements per chunk (128 or 64), KD = the reduction length if known at compile
// time (then kd == KD), else 0; kd is a multiple of KC, of 2 KC with RT = 4.  Row r of the pass
// (r < 16*NT) is `base + row_off(min(r, rows_valid-1))`.  `lds` is the workgroup's buffer of
// NB * ROWS * 2*KC bytes (ROWS >= 16*NT), NB = 2 if RT = 2 and KD = 0, else 3.  All LW wavefronts
// of the workgroup call it together; a[], base and `wave` are wavefront-uniform; w_lane_off is
// the lane's byte offset inside a weight fragment.  NT_HINT: see ld8_async.
//
// LDS rows hold one chunk of a token row (2*KC bytes) with the 16-byte piece p
// of row r stored at piece index p ^ swz(r), swz(r) = r & 15 for 256-byte rows,
// (r >> 1) & 7 for 128-byte rows: the 16 token rows an MFMA operand reads fall
// into 16 different bank groups.  A direct load writes lane l at base + 16*l,
// so the swizzle is applied on the global side (which piece a lane fetches).
//
// A tile past the matrix repeats another (the caller drops its result).
template <int RT, int NT, int ROWS, int LW, int KC, int KD, bool NT_HINT, typename RowOff>
__device__ __forceinline__ void dma_stream_gemm(const uint16_t* const (&a)[RT], uint32_t w_lane_off, int wave,
                                                int kd, int rows_valid, const uint16_t* base, RowOff row_off,
                                                uint16_t* lds, f32x4 (&acc)[RT][NT]) {
  static_assert(KC == 128 || KC == 64, "chunk of 4 or 2 k-steps");
  static_assert(KD % KC == 0, "reduction length must be whole chunks");
  static_assert(RT == 2 || (RT == 4 && KC == 64 && KD == 0), "forms below");
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
  constexpr int NW = RT * KS;        // weight loads per wavefront and chunk
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
  auto dma = [&](int chunk, uint32_t buf) {  // buf: byte offset of the buffer, uniform
    const uint16_t* g = base + chunk * KC;  // uniform
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const uint32_t dst = lds0 + buf + min(i * LW + wave, NG - 1) * 1024;  // uniform
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
  bf16x8 aw[KD > 0 ? 3 : 2][KS][RT];
  auto loadw1 = [&](int chunk, auto stage, auto uc) {  // the fragments of k-step u of a chunk
    constexpr int s = decltype(stage)::value, u = decltype(uc)::value;
#pragma unroll
    for (int r = 0; r < RT; ++r)
      ld8_async<u * kFragBytes, NT_HINT>(aw[s][u][r], a[r] + static_cast<size_t>(chunk) * KS * frag_step<true>(),
                                         w_lane_off);
  };
  auto loadw = [&](int chunk, auto stage) {
    static_for(std::make_integer_sequence<int, KS>{}, [&](auto uc) { loadw1(chunk, stage, uc); });
  };
  // byte offset in a buffer of this lane's fragment of token tile 0, k-step u of a chunk
  uint32_t fa[KS];
#pragma unroll
  for (int u = 0; u < KS; ++u) fa[u] = (lane & 15) * RB + (((u * 4 + (lane >> 4)) ^ swz(lane & 15)) << 4);
  typedef __attribute__((address_space(3))) const volatile bf16x8 LdsFrag;
  const auto lds_base = reinterpret_cast<__attribute__((address_space(3))) const volatile char*>(DES_LDS_PTR(lds));
  // multiplies the chunk in buffer `buf` with the weights of a stage; done(u): k-step u's weights are free
  auto compute = [&](uint32_t buf, auto stage, auto&& done) {
    constexpr int s = decltype(stage)::value;
    constexpr int G = NT <= 4 ? NT : RT == 4 ? 2 : NT / 2;  // token tiles fetched from LDS at a time
    constexpr int NGR = NT / G, STEPS = KS * NGR;
    bf16x8 b[2][G];
    auto fetch = [&](auto stepc) {
      constexpr int st = decltype(stepc)::value, u = st / NGR, g = st % NGR * G;
#pragma unroll
      for (int i = 0; i < G; ++i)
        b[st & 1][i] = *reinterpret_cast<LdsFrag*>(lds_base + (fa[u] + buf) + (g + i) * kTile);
    };
    fetch(S0{});
    static_for(std::make_integer_sequence<int, STEPS>{}, [&](auto stepc) {
      constexpr int st = decltype(stepc)::value, u = st / NGR, g = st % NGR * G;
      if constexpr (st + 1 < STEPS) fetch(std::integral_constant<int, st + 1>{});
      __builtin_amdgcn_sched_barrier(0);  // (the next fragments are requested before these multiplies)
#pragma unroll
      for (int i = 0; i < G; ++i)
#pragma unroll
        for (int r = 0; r < RT; ++r)
          acc[r][g + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[s][u][r], b[st & 1][i], acc[r][g + i], 0, 0, 0);
      if constexpr (g + G == NT) done(std::integral_constant<int, u>{});
    });
    // every read of this buffer has come back before the next barrier lets it be overwritten
    asm volatile("s_waitcnt lgkmcnt(0)");
  };
  const auto nothing = [](auto) {};
  static_assert(ND + NW <= 63, "wait count must fit the counter");
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
    dma(0, 0);
    loadw(0, S0{});
    if constexpr (NCH > 1) {
      dma(1, kBufBytes);
      loadw(1, S1{});
    }
    static_for(std::make_integer_sequence<int, NCH>{}, [&](auto cc) {
      constexpr int c = decltype(cc)::value;
      typedef std::integral_constant<int, c % 3> Cur;
      typedef std::integral_constant<int, (c + 2) % 3> Nxt;
      wait_weights<(c + 1 < NCH) ? ND + NW : 0>(aw[c % 3]);
      __builtin_amdgcn_s_barrier();
      if constexpr (c + 2 < NCH) {
        dma(c + 2, Nxt::value * kBufBytes);
        loadw(c + 2, Nxt{});
      }
      compute(Cur::value * kBufBytes, Cur{}, nothing);
    });
  } else if constexpr (RT == 4) {
    // Any even number of chunks, in the order above, but the weights have two stages only (the
    // accumulators take half of the registers): a k-step's fragments are requested for two
    // chunks later as soon as they have been multiplied.
    uint32_t cur = 0;  // the current chunk's buffer
    auto step = [&](int c, auto stage, auto more, auto last) {  // more: chunk c + 2 exists
      constexpr int s = decltype(stage)::value;
      wait_weights<last ? 0 : ND + NW>(aw[s]);
      __builtin_amdgcn_s_barrier();
      if constexpr (more) dma(c + 2, cur >= kBufBytes ? cur - kBufBytes : 2 * kBufBytes);
      compute(cur, stage, [&](auto uc) {
        if constexpr (more) {
          __builtin_amdgcn_sched_barrier(0);
          loadw1(c + 2, stage, uc);
        }
      });
      cur = cur == 2 * kBufBytes ? 0 : cur + kBufBytes;
    };
    dma(0, 0);
    loadw(0, S0{});
    dma(1, kBufBytes);
    loadw(1, S1{});
    int c = 0;
    for (; c + 2 < nchunks; c += 2) {
      step(c, S0{}, std::true_type{}, std::false_type{});
      step(c + 1, S1{}, std::true_type{}, std::false_type{});
    }
    step(c, S0{}, std::false_type{}, std::false_type{});
    step(c + 1, S1{}, std::false_type{}, std::true_type{});
  } else {
    // Any reduction length: two stages.  Step c: everything this wavefront asked
    // for (its share of the activations of chunk c, its weights of chunk c) has
    // landed; the barrier then says the same of the other wavefronts' shares, and
    // that everybody is done reading the other buffer, which the loads of chunk
    // c+1 overwrite while chunk c is multiplied.
    auto step = [&](int c, auto bufc, auto nextbuf) {
      constexpr int s = decltype(bufc)::value;
      wait_weights<0>(aw[s]);
      __builtin_amdgcn_s_barrier();
      if (c + 1 < nchunks) {
        dma(c + 1, decltype(nextbuf)::value * kBufBytes);
        loadw(c + 1, nextbuf);
      }
      compute(s * kBufBytes, bufc, nothing);
    };
    dma(0, 0);
    loadw(0, S0{});
    for (int c = 0; c < nchunks; c += 2) {
      step(c, S0{}, S1{});
      if (c + 1 >= nchunks) break;
      step(c + 1, S1{}, S0{});
    }
    // Nothing is outstanding (the last step requests nothing and has waited for the rest).  The check of
    // the generated code for reads of a register whose load is under way cannot know that: this tells it.
    asm volatile("s_waitcnt vmcnt(0)");
  }
}

// Every pass works in buffers of 16 KB: up to 64 token rows with chunks of 128
// reduction elements, or up to 128 rows with chunks of 64.  Three buffers (48 KB) where
// chunks are requested two ahead, else two.
constexpr int kLdsBufElems = 8192;
__host__ __device__ constexpr int lds_elems(int rt, int kd) { return (rt > 2 || kd > 0 ? 3 : 2) * kLdsBufElems; }

}  // namespace des
