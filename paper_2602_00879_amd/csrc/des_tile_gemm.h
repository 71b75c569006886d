// Tiled GEMM building block for the cases where many token rows meet one weight matrix (the
// attention projections of longer blocks, experts with many pairs): weight rows and token
// rows are both staged through LDS and shared by the four wavefronts of a workgroup.
// gfx950 only.
//
// Where a matrix has at most a few dozen token rows the weights are a pure stream and go
// from HBM straight into MFMA operands (des_stream_gemm.h).  With more, that form leaves a
// wavefront with one long chain - read the token fragments from LDS, wait, multiply - and,
// for one dense matrix, the chip with too few wavefronts.  Here a tile's reduction runs in
// chunks of 64.  tile_gemm (experts): two LDS buffers, the next P chunks in registers on their way;
// ordinary loads, the compiler places their waits.  tile_gemm_dma (attention projections): straight
// into LDS.
#pragma once

#include "des_common.h"
#include "des_stream_gemm.h"

namespace des {

constexpr int kTileK = 64;          // reduction elements per chunk
constexpr int kTileThreads = 256;   // four wavefronts, 2 x 2 over the tile

// LDS of one workgroup: two buffers of one chunk of (32 MT weight + 32 NT token) rows x 128 bytes.
template <int MT, int NT>
constexpr int tile_lds_bytes() { return 2 * 32 * (MT + NT) * kTileK * 2; }

// acc[m][n] += weight tile m x token tile n of this wavefront, over a reduction of `kd`
// elements (a multiple of 32; uniform to the compiler too, see stream_pipeline).  A group of
// four wavefronts works on a tile of 32 MT weight
// rows x 32 NT token rows; wavefront (wm, wn) of the 2 x 2 has weight rows 16 MT wm .. and
// token rows 16 NT wn ..
// Pointers of this thread (t = thread of the workgroup): aptr[i] = tile_weight_ptr() of row tile
// 2 i + t / 128 of the weight tile (row tiles 0 .. MT - 1 are wavefronts wm = 0's, the others
// wm = 1's); bptr[i] = element 8 * (t % 8) of token row i * 32 + t / 8 (a tile or row past the
// end repeats another, the caller drops its results).  PACKED: the weights' layout, operand
// tiles of 16 rows x 32 elements.  The whole workgroup calls it together.
// Every sum runs over the reduction in ascending steps of 32 whatever the tile, so the
// results do not depend on MT or NT.
//
// Rows lie 128 bytes apart in LDS, the 16-byte piece p of row r at p ^ (r / 2 % 8): a
// wavefront's writes (8 rows) and its operand reads (16 rows, one piece) both fall into
// different banks.
template <bool PACKED>
__device__ __forceinline__ const uint16_t* tile_weight_ptr(const uint16_t* row_tile, int kd, int t) {
  return PACKED ? row_tile + (t & 63) * 8 : row_tile + static_cast<size_t>((t >> 3) & 15) * kd + (t & 7) * 8;
}
template <int MT, int NT, int P, bool PACKED>
__device__ __forceinline__ void tile_gemm(const uint16_t* const (&aptr)[MT], const uint16_t* const (&bptr)[NT],
                                          int kd, char* lds, f32x4 (&acc)[MT][NT]) {
  constexpr int kBuf = 32 * (MT + NT) * kTileK * 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int steps = (kd + kTileK - 1) / kTileK;
  const int piece = tid & 7, srow = tid >> 3;
  const int sdst = srow * 128 + ((piece ^ ((srow >> 1) & 7)) << 4);  // + 32 rows: the same swizzle
  // weights: the same place (row-major), or two operand tiles per chunk (packed): this wavefront
  // loads the first or the second, lane l has piece l / 16 of row l % 16 of it
  const int arow = PACKED ? (wave >> 1) * 16 + (lane & 15) : srow;
  const int apiece = PACKED ? (wave & 1) * 4 + (lane >> 4) : piece;
  const int adst = arow * 128 + ((apiece ^ ((arow >> 1) & 7)) << 4);
  uint4 ra[P][MT], rb[P][NT];
  auto load = [&](int st, auto set) {
    constexpr int z = decltype(set)::value;
    // pieces past the end of the reduction fetch its last elements; store() replaces them
    // with zeros
    const int k = min(st * kTileK + piece * 8, kd - 8) - piece * 8;
    const size_t ka = PACKED ? static_cast<size_t>(min(2 * st + (wave & 1), kd / 32 - 1)) * 512 : k;
#pragma unroll
    for (int i = 0; i < MT; ++i) ra[z][i] = *reinterpret_cast<const uint4*>(aptr[i] + ka);
#pragma unroll
    for (int i = 0; i < NT; ++i) rb[z][i] = *reinterpret_cast<const uint4*>(bptr[i] + k);
  };
  auto store = [&](int st, auto set) {
    constexpr int z = decltype(set)::value;
    if ((st + 1) * kTileK > kd) {
      if (st * kTileK + apiece * 8 >= kd) {
#pragma unroll
        for (int i = 0; i < MT; ++i) ra[z][i] = make_uint4(0u, 0u, 0u, 0u);
      }
      if (st * kTileK + piece * 8 >= kd) {
#pragma unroll
        for (int i = 0; i < NT; ++i) rb[z][i] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
    char* buf = lds + (st & 1) * kBuf;
#pragma unroll
    for (int i = 0; i < MT; ++i) *reinterpret_cast<uint4*>(buf + i * 4096 + adst) = ra[z][i];
#pragma unroll
    for (int i = 0; i < NT; ++i) *reinterpret_cast<uint4*>(buf + (MT + i) * 4096 + sdst) = rb[z][i];
  };
  const int r = lane & 15, g = lane >> 4, sw = (r >> 1) & 7;
  auto compute = [&](int st) {
    const char* a = lds + (st & 1) * kBuf + (wm * MT * 16 + r) * 128;
    const char* b = lds + (st & 1) * kBuf + 32 * MT * 128 + (wn * NT * 16 + r) * 128;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int off = ((u * 4 + g) ^ sw) << 4;
      bf16x8 fa[MT], fb[NT];
#pragma unroll
      for (int i = 0; i < MT; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(a + i * 2048 + off);
#pragma unroll
      for (int i = 0; i < NT; ++i) fb[i] = *reinterpret_cast<const bf16x8*>(b + i * 2048 + off);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
  };
  auto step = [&](int st, auto i, auto more) {  // chunk st is in LDS; i = st % P
    typedef std::integral_constant<int, (decltype(i)::value + 1) % P> Next;
    if (more || st + 1 < steps) store(st + 1, Next{});
    if (more || st + 1 + P < steps) load(st + 1 + P, Next{});
    compute(st);
    __syncthreads();
  };
  auto unrolled = std::make_integer_sequence<int, P>{};
  static_for(unrolled, [&](auto i) {
    if (i < steps) load(i, i);
  });
  store(0, S0{});
  if (P < steps) load(P, S0{});
  __syncthreads();
  // step st: the next chunk goes from registers to the buffer that the one before was read
  // from (everybody is past the barrier that ended it), the one after P more is requested
  int st = 0;
  for (; st + 2 * P < steps; st += P)
    static_for(unrolled, [&](auto i) { step(st + i, i, std::true_type{}); });
  for (; st < steps; st += P)
    static_for(unrolled, [&](auto i) {
      if (st + i < steps) step(st + i, i, std::false_type{});
    });
}

// The same tile for whole chunks only (kd a multiple of 64), both operands row-major: weight and
// token rows go from global memory straight into LDS (no registers, no LDS writes of the
// wavefronts' own), NB buffers of a chunk each, NB - 1 chunks requested ahead, one barrier per chunk.
// abase / bbase: the reduction's first element of the tile's first weight and token row, uniform;
// aoff / boff: byte offset of this thread's piece of row 32 i + t / 8, which is
// row * stride + tile_piece(t) * 16 (a row past the end repeats another).
// Sums run in the same order as in tile_gemm.
//
// The direct loads are asm (des_stream_gemm.h says why): the compiler does not know of them, the wait
// before each barrier is explicit, and the operand reads are volatile, which keeps them in program
// order with the barriers.
//
// A group of four wavefronts works on a tile as in tile_gemm.  KW = 2: the workgroup has two such
// groups, each with its half of the reduction (kd and the bases are the group's own, the lengths are
// equal) and buffers of its own.
__device__ __forceinline__ int tile_piece(int t) { return (t & 7) ^ ((t >> 4) & 7); }
template <int MT, int NT, int KW, int NB>
constexpr int tile_dma_lds_bytes() { return KW * NB * 32 * (MT + NT) * kTileK * 2; }
template <int MT, int NT, int KW, int NB>
__device__ __forceinline__ void tile_gemm_dma(const uint16_t* abase, const uint16_t* bbase, const uint32_t (&aoff)[MT],
                                              const uint32_t (&boff)[NT], int kd, char* lds, f32x4 (&acc)[MT][NT]) {
  constexpr int kBuf = 32 * (MT + NT) * kTileK * 2, ND = MT + NT;
  const int grp = KW > 1 ? uniform_int(threadIdx.x >> 8) : 0;
  const int lane = threadIdx.x & 63, wave = uniform_int((threadIdx.x >> 6) & 3);
  const int wm = wave >> 1, wn = wave & 1;
  const int steps = kd / kTileK;
  lds += grp * NB * kBuf;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<size_t>(DES_LDS_PTR(lds))) + wave * 1024;
  auto load = [&](const uint16_t* base, uint32_t off, uint32_t dst) {
    // (wait states after the writes of M0 and of the base, see dma_stream_gemm)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(dst) : "m0");
  };
  auto request = [&](int st, uint32_t buf) {
    const uint16_t *ga = abase + st * kTileK, *gb = bbase + st * kTileK;
#pragma unroll
    for (int i = 0; i < MT; ++i) load(ga, aoff[i], lds0 + buf + i * 4096);
#pragma unroll
    for (int i = 0; i < NT; ++i) load(gb, boff[i], lds0 + buf + (MT + i) * 4096);
  };
  const int r = lane & 15, g = lane >> 4, sw = (r >> 1) & 7;
  typedef __attribute__((address_space(3))) const volatile bf16x8 LdsFrag;
  const auto lds_base = reinterpret_cast<__attribute__((address_space(3))) const volatile char*>(DES_LDS_PTR(lds));
  const uint32_t a0 = (wm * MT * 16 + r) * 128, b0 = 32 * MT * 128 + (wn * NT * 16 + r) * 128;
  auto compute = [&](uint32_t buf) {
    bf16x8 fa[2][MT], fb[2][NT];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t off = buf + (((u * 4 + g) ^ sw) << 4);
#pragma unroll
      for (int i = 0; i < MT; ++i) fa[u][i] = *reinterpret_cast<LdsFrag*>(lds_base + (a0 + off) + i * 2048);
#pragma unroll
      for (int i = 0; i < NT; ++i) fb[u][i] = *reinterpret_cast<LdsFrag*>(lds_base + (b0 + off) + i * 2048);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[u][i], fb[u][j], acc[i][j], 0, 0, 0);
  };
  static_assert(NB == 2 || NB == 3, "chunks ahead");
  static_assert((NB - 1) * ND <= 63, "wait counts must fit the counter");
#pragma unroll
  for (int i = 0; i < NB - 1; ++i)
    if (i < steps) request(i, i * kBuf);
  uint32_t cur = 0;
  for (int st = 0; st < steps; ++st) {
    // chunk st has landed (loads complete in order; the chunks after it stay in flight) ...
    if (st + NB - 2 < steps) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NB - 2) * ND));
    else asm volatile("s_waitcnt vmcnt(0)");
    // ... everybody's share of it, and everybody has read the buffer that is filled next
    asm volatile("s_waitcnt lgkmcnt(0)");
    __builtin_amdgcn_s_barrier();
    if (st + NB - 1 < steps) request(st + NB - 1, cur >= kBuf ? cur - kBuf : (NB - 1) * kBuf);
    compute(cur);
    cur = cur == (NB - 1) * kBuf ? 0 : cur + kBuf;
  }
  // (whoever uses the LDS next waits for everybody's reads of it first)
  asm volatile("s_waitcnt lgkmcnt(0)");
  __builtin_amdgcn_s_barrier();
}

}  // namespace des
