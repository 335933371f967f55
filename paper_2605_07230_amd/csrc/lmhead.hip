// lmhead_softmax_cfg kernels for gfx950: final projection with the guidance mix in the epilogue
// (Sec. 4.2: the O(hV) projection dominates; App. "Configuration Details": guidance scale,
// temperature, top-k), then one kernel for the per-row softmax statistics.
//
// bf16 projection: both operands reach the matrix cores through a ring of LDS stages filled by LDS-direct loads.
// lmhead_bf16_ring_kernel takes rows and weights as they lie in memory (or packed weights) and comes in tiles from
// 64 x 64 to 256 x 128; lmhead_bf16_tiled_kernel takes both operands packed and carries the large tiles of steps with
// several hundred rows.  lm_plan chooses by estimated time, and gives the columns that do not fill a round a smaller tile.
#include "common.h"

namespace {

struct LmParams {
  const void* h_cond;
  const void* h_uncond;
  const void* w;
  float* logits;
  float* row_max;
  float* row_thr;
  float* row_lse;
  const uint4* hp_cond;     // packed hidden states (MFMA operand order), when the packed path runs
  const uint4* hp_uncond;
  int n_nodes, hidden, vocab;
  int col0;                 // first vocabulary column of the launch
  float cfg_scale, temperature;
  int top_k;
  int sample_rank;          // row statistics: entries of the sample at and above the cut
};

// ------------------------------------------------------------------------------------------ f32
// Workgroup = 16 vocabulary entries x 16 NB nodes (conditional and unconditional rows of the same nodes); the four waves
// take every fourth 16-wide step of the hidden dimension and are summed through LDS.  v_mfma_f32_16x16x4_f32 takes one
// value per lane and operand, k = lane / 16; a lane loads the 16 bytes at 4 (lane / 16) of its row's step and feeds
// element c of both operands to the c-th product, so every product sees the same four k on both sides.
// Bound by latency at the sizes this path serves (15 nodes x 4096 x 512: 8.4 MB): the one-thread-per-entry loop it
// replaces read 256 rows 4 bytes at a time, 58 us; 16-entry workgroups fill the chip: 4.9 us.
// VEC: hidden is a multiple of 4 and the pointers are 16-byte aligned; otherwise elements are loaded one at a time.
template <int NB, bool CFG, bool VEC>
__global__ __launch_bounds__(256) void lmhead_f32_kernel(LmParams p) {
  constexpr int NR = NB * (CFG ? 2 : 1);
  __shared__ float red[4][NR][4][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int K = p.hidden, v0 = blockIdx.x * 16, node0 = blockIdx.y * 16 * NB;
  const float* wr = (const float*)p.w + (int64_t)min(v0 + l16, p.vocab - 1) * K;   // clamped, never stored
  const float* hr[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) hr[i] = (const float*)(i < NB ? p.h_cond : p.h_uncond) + (int64_t)min(node0 + 16 * (i % NB) + l16, p.n_nodes - 1) * K;
  auto load4 = [&](const float* row, int k) {
    if (VEC) return k < K ? *(const f32x4*)(row + k) : f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 x;
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = k + c < K ? row[k + c] : 0.f;
    return x;
  };
  f32x4 acc[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int UN = NR > 4 ? 2 : 4;   // steps requested together; past the end they are zero
  for (int k0 = 16 * wave; k0 < K; k0 += 64 * UN) {
    f32x4 a[UN][NR], b[UN];
#pragma unroll
    for (int s = 0; s < UN; ++s) {
      const int k = k0 + 64 * s + 4 * g;
      b[s] = load4(wr, k);
#pragma unroll
      for (int i = 0; i < NR; ++i) a[s][i] = load4(hr[i], k);
    }
#pragma unroll
    for (int s = 0; s < UN; ++s)
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][i][c], b[s][c], acc[i], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < NR; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][i][r][lane] = acc[i][r];
  __syncthreads();
  // register r of lane (l16, g) is node 4 g + r of its block, entry l16; wave w finishes blocks w, w + 4, ...
  for (int i = wave; i < NB; i += 4)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float c = ((red[0][i][r][lane] + red[1][i][r][lane]) + red[2][i][r][lane]) + red[3][i][r][lane];
      float gmix = c;
      if (CFG) {
        const int j = NB + i;
        const float u = ((red[0][j][r][lane] + red[1][j][r][lane]) + red[2][j][r][lane]) + red[3][j][r][lane];
        gmix = u + p.cfg_scale * (c - u);
      }
      const int node = node0 + 16 * i + 4 * g + r;
      if (node < p.n_nodes && v0 + l16 < p.vocab) p.logits[(int64_t)node * p.vocab + v0 + l16] = gmix / p.temperature;
    }
}

// ----------------------------------------------------------------------------------------- bf16
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
union Frag8 {
  bf16x8 v;
  uint4 u;
  u32x4 n;
};

// ------------------------------------------------------------------------- bf16, packed operands
// Operand order: for a block of 32 rows rb and a 16-wide k step ks, 64 x 16 bytes where entry
// l = (r32, half) holds src[32*rb + r32][16*ks + 8*half .. +7]; the ks blocks of one rb follow
// each other.  One wave-wide 16-byte load per MFMA operand, 1 KiB contiguous.
__global__ __launch_bounds__(256) void pack32_kernel(const uint16_t* __restrict__ src0, uint4* __restrict__ dst0,
                                                      const uint16_t* __restrict__ src1, uint4* __restrict__ dst1, int rows, int K) {
  const uint16_t* src = blockIdx.z ? src1 : src0;
  uint4* dst = blockIdx.z ? dst1 : dst0;
  const int lane = threadIdx.x & 63, r32 = lane & 31, half = lane >> 5;
  const int ks = blockIdx.x * 4 + (threadIdx.x >> 6), rb = blockIdx.y;
  if (ks >= K / 16) return;
  const int row = 32 * rb + r32;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row < rows) v = *(const uint4*)(src + (int64_t)row * K + 16 * ks + 8 * half);
  dst[((int64_t)rb * (K / 16) + ks) * 64 + lane] = v;
}

// eight guidance-mixed elements u + s (c - u), float32, rounded once to bf16
__device__ __forceinline__ uint4 mix16(const uint4& c, const uint4& u, float s) {
  const uint32_t cw[4] = {c.x, c.y, c.z, c.w}, uw[4] = {u.x, u.y, u.z, u.w};
  uint32_t m[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float c0 = __uint_as_float(cw[i] << 16), c1 = __uint_as_float(cw[i] & 0xffff0000u);
    const float u0 = __uint_as_float(uw[i] << 16), u1 = __uint_as_float(uw[i] & 0xffff0000u);
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const b2 r = __builtin_convertvector(f2{u0 + s * (c0 - u0), u1 + s * (c1 - u1)}, b2);   // round to nearest even
    m[i] = *(const uint32_t*)&r;
  }
  return make_uint4(m[0], m[1], m[2], m[3]);
}

// The same operand order for the guidance-mixed rows u + s (c - u) (float32, rounded once to bf16): the
// projection is linear, so one product over these rows gives the mixed logits.  dst_rows: the rows as they lie, too.
__global__ __launch_bounds__(256) void pack32_mix_kernel(const uint16_t* __restrict__ src_c, const uint16_t* __restrict__ src_u,
                                                          uint4* __restrict__ dst, uint4* __restrict__ dst_rows, int rows, int K, float s) {
  const int lane = threadIdx.x & 63, r32 = lane & 31, half = lane >> 5;
  const int ks = blockIdx.x * 4 + (threadIdx.x >> 6), rb = blockIdx.y;
  if (ks >= K / 16) return;
  const int row = 32 * rb + r32;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row < rows) {
    const int64_t o = (int64_t)row * K + 16 * ks + 8 * half;
    const uint4 c = *(const uint4*)(src_c + o), u = *(const uint4*)(src_u + o);
    v = mix16(c, u, s);
    if (dst_rows) dst_rows[o / 8] = v;
  }
  dst[((int64_t)rb * (K / 16) + ks) * 64 + lane] = v;
}

// The same mixed rows, left row-major (what the ring kernel reads).
__global__ __launch_bounds__(256) void mix_rows_kernel(const uint4* __restrict__ src_c, const uint4* __restrict__ src_u,
                                                        uint4* __restrict__ dst, int n16, float s) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n16) dst[i] = mix16(src_c[i], src_u[i], s);
}

// ----------------------------------------------------------------------------------- bf16, ring of stages
// Tile = 32 AM WM rows x 32 AN WN vocabulary columns per workgroup of eight waves; a wave owns AM x AN blocks of
// 32 x 32 and every KW-th k16 step of a stage (KW groups of waves split the hidden dimension inside the workgroup and
// are summed through LDS at the end, in a fixed order).  A stage = KS k16 steps of every row and column block of the
// tile; NST stages are in flight or in use.  With guidance a wave's two row blocks are the conditional and the
// unconditional rows of the same 32 nodes, so the mix stays in registers.
//
// What bounds it: the bytes a compute unit has in flight.  Loads alone (no multiplications, no LDS reads) take 90 % of
// the kernel's time at every tile, and requesting more than ~64 KB ahead changes nothing (48 KB: 33 us, 72 KB: 29.6,
// 120 KB: 29.6 at 60 x 16384 x 4096), so a tile costs about (weight bytes x HBM latency + row bytes x L2 latency) / 64 KB.
// Hence tiles as large as the row count justifies, each weight byte loaded once per row tile, no padding traffic.
// Rows are read as they lie in memory: a wave's 1 KiB request covers whole 128-byte pieces of eight rows (eight lanes per
// row), and no packing pass precedes the kernel (row-major rows measured the same as packed ones).  LDS-direct loads put
// lane l's 16 bytes at 16 l, so bank conflicts are avoided by WHICH piece a lane fetches: slot q of row r holds piece
// q ^ ((r >> 1) & 7), and the 16 rows that a fragment read touches together land in 16 different 16-byte slots.  Packed
// weights (contiguous 1 KiB operand blocks) are 4 us faster than row-major ones at 16384 x 4096.
// Large weights are streamed (nt): a step reads them once, or once per row tile at the same time, and everything else it touches
// would be displaced from the caches by them.  Steps over weights that the caches do not hold yet: 60 rows x 16384 28.9 ->
// 25.9 us, 60 x 65536 103.8 -> 92.7 (5.8 TB/s), 60 guidance pairs, row-major 40.7 -> 38.1, and the kernels after it find
// their rows again (whole step of 60 x 16384: 66 -> 58).  lm_streams says which launches do.  They are instances of their own:
// two loops in one kernel, or one that chooses at every request, made the launches that do not stream 2-8 % slower
// (512 rows x 16384 x 4096 74.7 -> 79.5 us, 300 x 8192 x 2048 24.4 -> 25.1, 686 row-major rows x 16384 x 4096 123 -> 131).
// Measured against the kernels this replaced (64 x 64 tiles, operands loaded to registers, hidden 4096; us, without the
// packing pass of 4 us that they needed): 60 rows x 16384: 30.2 -> 27.4; 60 x 65536: 110 -> 101 (5.3 TB/s);
// 120 x 16384: 45 -> 35; 230 x 16384: 75 -> 45; 60 guidance pairs, row-major weights: 63 -> 37.
// DIRECT = false: rows or weights that do not start on a 16-byte boundary.  LDS-direct loads are counted on for aligned
// addresses only; ordinary loads take any, pass through registers and are stored to the same places, one stage ahead in two
// slots (so the stages are twice as long).  60 rows x 16384 x 4096: 26 us aligned, 38 with rows at 8 bytes past a boundary,
// 47 with packed weights 2 bytes past one (36 in the register-staged kernel); 60 pairs, row-major: 36, 62, 78 (93); 230 rows:
// 44, 58, 78 (109).
template <int AM, int AN, int WM, int WN, int KW, int KS, int NST, bool CFG, bool PW, bool DIRECT, bool STREAM>
__global__ __launch_bounds__(512) void lmhead_bf16_ring_kernel(LmParams p, int n_mtiles) {
  static_assert(WM * WN * KW == 8 && KS % KW == 0 && KS % 4 == 0 && (!CFG || AM == 2), "eight waves; guidance pairs are a wave's two row blocks");
  constexpr int BM = 32 * AM * WM, BN = 32 * AN * WN, NA = BM / 32, NBLK = NA + BN / 32, STAGE = NBLK * KS * 1024;
  constexpr int LPW = NBLK * KS / 8, SPW = KS / KW;
  // DEALT: a wave's requests of a stage are LPA chunks of rows, then chunks of weights.  Streamed weights need that, 256 x 128 tiles
  // take it: with consecutive chunks some waves request nothing but weights, and all wait for them (343 pairs x 33088 x 2048
  // packed 122.0 us, dealt 116.5, 500 pairs 157.8 and 152.6, 450 pairs x 49152 x 2048 row-major 225.3 and 217.5).  The smaller tiles
  // do not: 64 x 64 over 8192 x 4096 gets up to 10 % slower.
  constexpr bool DEALT = STREAM || WM == 4;
  constexpr int LPA = NA * KS / 8;
  static_assert(NA * KS % 8 == 0 && NBLK * KS % 8 == 0 && (DIRECT || !STREAM), "every wave requests the same number of 1 KiB chunks");
  extern __shared__ __align__(1024) char ring_lds[];   // [NST stages][NBLK blocks][KS KiB]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, half = lane >> 5;
  const int K = p.hidden, n_stages = K / (16 * KS);    // hidden is a multiple of 128
  // XCD-aware order: contiguous ranges of tiles per XCD (any grid size), row tiles of one column tile adjacent in its L2
  const int nwg = gridDim.x, xcd = blockIdx.x & 7;
  const int logical = xcd * (nwg >> 3) + min(xcd, nwg & 7) + (blockIdx.x >> 3);
  const int nt = logical / n_mtiles, mt = logical % n_mtiles;

  // loader: request i of a wave is chunk id of a stage: block id / KS, KiB id % KS of it (one k16 step of packed operands, or
  // eight rows x 128 bytes of row-major ones, four of which make a 32-row x 64-column piece).  Where they are dealt, which requests are
  // weights is known at compile time.
  auto chunk = [&](int i) { return !DEALT ? wave * LPW + i : (i < LPA ? wave * LPA + i : NA * KS + wave * (LPW - LPA) + (i - LPA)); };
  auto weights = [&](int i) { return DEALT ? i >= LPA : chunk(i) / KS >= NA; };
  unsigned voff[LPW];
  const char* src[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int id = chunk(i), blk = id / KS, q = id % KS;
    const char* base;
    int row0, rows;
    if (!weights(i)) {
      base = (const char*)((CFG && (blk & 1)) ? p.h_uncond : p.h_cond);
      row0 = CFG ? mt * (BM / 2) + 32 * (blk >> 1) : mt * BM + 32 * blk;
      rows = p.n_nodes;
    } else {
      base = (const char*)p.w;
      row0 = p.col0 + nt * BN + 32 * (blk - NA);
      rows = p.vocab;
    }
    if (PW && weights(i)) {
      src[i] = base + ((int64_t)min(row0 / 32, rows / 32 - 1) * (K / 16) + q) * 1024;   // columns past the end: clamped, never stored
      voff[i] = 16u * lane;
    } else {
      const int lr = 8 * (q & 3) + (lane >> 3), first = min(row0, rows - 1);
      src[i] = base + (int64_t)first * 2 * K + (q >> 2) * 128;
      voff[i] = (unsigned)(min(row0 + lr, rows - 1) - first) * (unsigned)(2 * K) + 16u * (unsigned)((lane & 7) ^ ((lr >> 1) & 7));
    }
  }
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)ring_lds);
  u32x4 held[DIRECT ? 1 : LPW];   // (ordinary loads) the stage on its way
  auto store_held = [&](int slot) {   // complete before the next barrier, which waits for the wave's LDS operations
#pragma unroll
    for (int i = 0; i < (DIRECT ? 0 : LPW); ++i) *(u32x4*)(ring_lds + chunk(i) * 1024 + slot * STAGE + 16 * lane) = held[i];
  };
  auto request = [&](int t, int slot) {   // t past the end: clamped, that data is never multiplied
    const int tc = min(t, n_stages - 1);
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const char* g = src[i] + (int64_t)tc * ((PW && weights(i)) ? KS * 1024 : KS * 32);
      if constexpr (!DIRECT) { __builtin_memcpy(&held[i], g + voff[i], 16); continue; }
      const unsigned l = lds0 + slot * STAGE + chunk(i) * 1024;
      if (STREAM && i >= LPA) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(l), "v"(voff[i]), "s"(g) : "memory");
      else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(voff[i]), "s"(g) : "memory");
    }
  };
  const int kw = wave / (WM * WN), wm = (wave / WN) % WM, wn = wave % WN;
  // byte offset of k16 step s of a block for this lane (its 16 bytes of row r32)
  auto packed_at = [&](int s) { return (unsigned)(s * 1024 + lane * 16); };
  auto rows_at = [&](int s) { return (unsigned)((s >> 2) * 4096 + r32 * 128 + (((2 * (s & 3) + half) ^ ((r32 >> 1) & 7)) * 16)); };

  f32x16 acc[AM][AN];
#pragma unroll
  for (int i = 0; i < AM; ++i)
#pragma unroll
    for (int j = 0; j < AN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // every sum over the hidden dimension is four chains, over the KW groups of waves and within a wave: one chain of 4096
  // terms is off by 3.7e-7 of the row (2-norm, against float64), two 2.5e-7, four 1.7e-7
  constexpr int CH = 4 / KW;
  f32x16 done[AM][AN];   // (CH > 1) the finished chains
#pragma unroll
  for (int t = 0; t < NST - 1; ++t) { request(t, t); store_held(t); }
  int slot = 0, t = 0;
  for (int c = 1; c <= CH; ++c) {
    for (const int t_end = n_stages * c / CH; t < t_end; ++t) {
      // own chunks of stage t landed (the NST - 2 later stages may be in flight), own LDS reads of stage t - 1 done; bare
      // barrier: everybody's chunks are there and stage t - 1's slot is free
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LPW * (NST - 2)) : "memory");
      const int free_slot = slot == 0 ? NST - 1 : slot - 1;
      request(t + NST - 1, free_slot);
      if (!DIRECT) __builtin_amdgcn_sched_barrier(0);   // left alone, each load sinks to the store of its value
      const char* st = ring_lds + slot * STAGE;
      Frag8 a[SPW][AM], b[SPW][AN];
#pragma unroll
      for (int ss = 0; ss < SPW; ++ss) {
        const int s = kw * SPW + ss;
#pragma unroll
        for (int i = 0; i < AM; ++i) a[ss][i].n = *(const u32x4*)(st + (AM * wm + i) * KS * 1024 + rows_at(s));
#pragma unroll
        for (int j = 0; j < AN; ++j) b[ss][j].n = *(const u32x4*)(st + (NA + AN * wn + j) * KS * 1024 + (PW ? packed_at(s) : rows_at(s)));
      }
#pragma unroll
      for (int ss = 0; ss < SPW; ++ss)
#pragma unroll
        for (int i = 0; i < AM; ++i)
#pragma unroll
          for (int j = 0; j < AN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ss][i].v, b[ss][j].v, acc[i][j], 0, 0, 0);
      store_held(free_slot);
      slot = slot + 1 == NST ? 0 : slot + 1;
    }
    if (CH > 1)
#pragma unroll
      for (int i = 0; i < AM; ++i)
#pragma unroll
        for (int j = 0; j < AN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float x = c > 1 ? done[i][j][r] + acc[i][j][r] : acc[i][j][r];
            done[i][j][r] = x;
            acc[i][j][r] = c < CH ? 0.f : x;
          }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the clamped extra requests must not outlive the workgroup's LDS

  // epilogue: accumulator (i, j), register r of lane (r32, half) is row 8 (r / 4) + 4 half + r % 4, column r32
  constexpr int NI = CFG ? 1 : AM;   // node blocks of a wave
  auto emit = [&](int i, int j, int r, float x0, float x1) {
    const int node = (CFG ? mt * (BM / 2) + 32 * wm : mt * BM + 32 * (AM * wm + i)) + 8 * (r >> 2) + 4 * half + (r & 3);
    const int col = p.col0 + nt * BN + 32 * (AN * wn + j) + r32;
    const float gmix = CFG ? x1 + p.cfg_scale * (x0 - x1) : x0;
    if (node < p.n_nodes && col < p.vocab) p.logits[(int64_t)node * p.vocab + col] = gmix / p.temperature;
  };
  if constexpr (KW == 1) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < AN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) emit(i, j, r, acc[i][j][r], CFG ? acc[AM - 1][j][r] : 0.f);
  } else {
    // the KW partial tiles meet in LDS; wave group kw finishes every KW-th of the wave tile's values
    __syncthreads();
    constexpr int NV = AM * AN * 16, PER = NI * AN * 16 / KW;
    float* red = (float*)ring_lds;   // [8 waves][NV values][64 lanes]
#pragma unroll
    for (int i = 0; i < AM; ++i)
#pragma unroll
      for (int j = 0; j < AN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) red[(wave * NV + (i * AN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
    __syncthreads();
#pragma unroll
    for (int e0 = 0; e0 < PER; ++e0) {
      const int e = kw * PER + e0;
      float x0 = 0.f, x1 = 0.f;
#pragma unroll
      for (int g = 0; g < KW; ++g) {
        const float* part = red + (wave % (WM * WN) + g * WM * WN) * NV * 64 + lane;
        x0 += part[e * 64];
        if (CFG) x1 += part[(AN * 16 + e) * 64];
      }
      emit(e / (AN * 16), (e >> 4) % AN, e & 15, x0, x1);
    }
  }
}

// ------------------------------------------------------------------- bf16, packed, many rows
// LDS-tiled projection for the large tiles of steps with several hundred rows (batched prompts), where the kernel is
// bound by the matrix cores instead of by streaming W.  Workgroup tile = 256 rows x 256 vocabulary
// columns: with guidance 128 nodes (4 conditional + 4 unconditional 32-row blocks), without 256
// nodes.  The eight waves form a 2 x 4 grid; a wave owns 4 row blocks (two node blocks, conditional
// and unconditional, so the mix stays in registers) x 2 column blocks = 8 accumulators, two waves
// share a SIMD and one wave's waits are covered by the other's MFMAs (four waves with 16
// accumulators each were 10 % slower).
//
// Both operands are packed in MFMA operand order and never pass through registers on their way in:
// gfx950's 16-byte LDS-direct loads write each wave-wide 1 KiB block straight into a ring of four
// half-stages (2 k16 steps = 32 KiB each), so there are no staging registers, no LDS store
// instructions and no register pressure in the loop (a register-staged version of this kernel ran
// at the 256-register limit; a single spilled address in its loop was reloaded behind a wait for
// all outstanding loads and cost 8 %).  Per half-stage h:
//   - step 0 is multiplied; between the multiplications (each occupies the matrix core for 32
//     cycles, so the other instructions are free) step 1's fragments are read and the loads of
//     half-stage h + 3 are issued into the buffer that h - 1 was read from;
//   - the wave waits for its own loads of h + 1 and for its LDS reads, then the workgroup barrier
//     (bare: a fenced barrier would wait for every outstanding load);
//   - step 1 is multiplied while the first fragments of h + 1 are read.
// The barrier sits before the last step's multiplications, which cover it.
// HALF (no guidance only): 128-row tiles for steps whose 256-row tiles would leave compute units idle - a wave owns
// 2 x 2 accumulators; the tile has four H blocks per k16 step, eight per half-stage: wave w requests block w % 4 of
// step w / 4, so every wave issues three loads per half-stage (one H, two W) and the wait counts stay uniform.
template <bool CFG, bool HALF, bool STREAM>
__global__ __launch_bounds__(512) void lmhead_bf16_tiled_kernel(LmParams p, int n_mtiles) {
  static_assert(!(CFG && HALF) && (HALF || !STREAM), "half tiles exist for the plain projection only, and only they stream");
  constexpr int NI = HALF ? 2 : 4;   // row blocks per wave
  extern __shared__ u32x4 lds[];     // [4 half-stages][2 k16 steps][16 blocks: 8 H then 8 W][64 lanes]
  constexpr int NBUF = 4, HS = 2, HBYTES = HS * 16 * 1024;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: everything derived from it stays scalar
  const int r32 = lane & 31, half = lane >> 5;
  const int KS = p.hidden / 16, n_half = KS / HS;
  const unsigned lane_off = 16u * lane;                        // byte offset of this lane's 16-byte piece in a block

  // the row tiles of a column share an XCD's L2, as in the ring kernel and for any grid: streamed weights that every XCD fetched
  // for its own row tile came from HBM each time (400 rows x 33024 x 4096, 516 tiles: 249 us, so 180; with plain weights 223 and 182)
  const int nwg = gridDim.x, xcd = blockIdx.x & 7;
  const int logical = xcd * (nwg >> 3) + min(xcd, nwg & 7) + (blockIdx.x >> 3);
  const int nt = logical / n_mtiles, mt = logical % n_mtiles;

  // loader: per k16 step a wave copies block wave (H) and block wave + 8 (W); both base pointers are scalars
  const char* src[2];
#pragma unroll
  for (int b4 = 0; b4 < 2; ++b4) {
    const char* base;
    int64_t rb;   // 32-row block index in the source matrix
    if (b4 == 0) {
      if (CFG) { base = (const char*)(wave < 4 ? p.hp_cond : p.hp_uncond); rb = (int64_t)mt * 4 + (wave & 3); }
      else if (HALF) { base = (const char*)p.hp_cond; rb = (int64_t)mt * 4 + (wave & 3); }
      else { base = (const char*)p.hp_cond; rb = (int64_t)mt * 8 + wave; }
    } else {
      base = (const char*)p.w;
      rb = min(p.col0 / 32 + nt * 8 + wave, p.vocab / 32 - 1);   // a last column tile past the vocabulary re-reads its last block, never stored
    }
    src[b4] = base + rb * KS * 1024;
  }
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)lds);
  const int last = n_half - 1;
  // request i of a half-stage: k16 step i / 2, H (i even) or W (i odd).  Half tiles may stream W like the ring
  // kernel (see lm_streams), whole ones do not (400 rows x 65536 x 2048 122 -> 129).  h may run past the end:
  // clamped, that data is never multiplied.  M0 carries the LDS address of the wave's 1 KiB block;
  // each lane's 16 bytes land at 16 * lane behind it.
  auto request = [&](int h, int buf, int i) {
    if (HALF && i == 2) return;                                   // (i is a constant after unrolling)
    const int ks = (HALF && i == 0) ? (wave >> 2) : (i >> 1);     // half tiles: the wave's one H block belongs to step wave / 4
    const char* g = src[i & 1] + ((int64_t)min(h, last) * HS + ks) * 1024;
    const int slot = (i & 1) ? 8 + wave : (HALF ? (wave & 3) : wave);
    const unsigned l = lds0 + buf * HBYTES + (ks * 16 + slot) * 1024;
    if (STREAM && (i & 1)) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(l), "v"(lane_off), "s"(g) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(lane_off), "s"(g) : "memory");
  };
  // A wave's own loads of the next half-stage have landed when at most the 2 x 4 later ones are
  // outstanding; its LDS reads are complete at lgkmcnt(0).
  auto land_and_sync = [&]() {
    if (HALF) asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // 2 x 3 later loads
    else asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };

  // LDS read addresses: one base register per 64 KiB and role, the rest is an immediate.  The bases
  // are made opaque so that the compiler neither re-derives them nor keeps further sums alive.
  char* const lds_b = (char*)lds;
  auto opaque = [](unsigned x) { asm volatile("" : "+v"(x)); return x; };
  const int wm = wave >> 2, wn = wave & 3;
  // row blocks of wave row wm: with guidance 2 wm, 2 wm + 1 (conditional) and the same two of the
  // unconditional half (+4); without, 4 wm .. 4 wm + 3
  const unsigned a_base = 1024u * ((CFG || HALF) ? 2 * wm : 4 * wm) + lane_off, b_base = 1024u * (8 + 2 * wn) + lane_off;
  const unsigned a_off[2] = {opaque(a_base), opaque(a_base + 65536u)};
  const unsigned b_off[2] = {opaque(b_base), opaque(b_base + 65536u)};

  f32x16 acc[NI][2];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  Frag8 fa[2][NI], fb[2][2];   // operand fragments, double-buffered by k16 step
  auto read_one = [&](int slot, int buf, int ks, int idx) {   // idx 0 .. NI-1: H fragment, NI, NI+1: W fragment
    const int byte0 = buf * HBYTES + ks * 16 * 1024;          // compile-time after unrolling
    if (idx < NI) {
      const int rel = CFG ? (idx & 1) + 4 * (idx >> 1) : idx;
      fa[slot][idx].n = *(const u32x4*)(lds_b + a_off[byte0 >> 16] + ((byte0 & 65535) + rel * 1024));
    } else {
      fb[slot][idx - NI].n = *(const u32x4*)(lds_b + b_off[byte0 >> 16] + ((byte0 & 65535) + (idx - NI) * 1024));
    }
  };
  // 2 NI multiplications; after the k-th one, side(k) issues its piece of the other work
  auto multiply_with = [&](int slot, auto&& side) {
#pragma unroll
    for (int k = 0; k < 2 * NI; ++k) {
      __builtin_amdgcn_sched_barrier(0);
      acc[k >> 1][k & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[slot][k >> 1].v, fb[slot][k & 1].v, acc[k >> 1][k & 1], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      side(k);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr int NFR = NI + 2;                          // fragments per k16 step
  constexpr int FRAG_ORDER[6] = {0, NI, NI + 1, 1, 2, 3};   // the order in which the multiplications first need them

#pragma unroll
  for (int h = 0; h < NBUF - 1; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) request(h, h, i);
  land_and_sync();
#pragma unroll
  for (int k = 0; k < NFR; ++k) read_one(0, 0, 0, FRAG_ORDER[k]);
  constexpr int CH = HALF ? 4 : 1;   // chains of the sum over the hidden dimension (256-row tiles have no registers for more than one)
  f32x16 done[NI][2];                // (CH > 1) the finished chains
  int h0 = 0;
  for (int c = 1; c <= CH; ++c) {
    for (const int h_end = n_half / NBUF * c / CH * NBUF; h0 < h_end; h0 += NBUF) {   // hidden is a multiple of 128: four half-stages always divide it
#pragma unroll
      for (int b = 0; b < NBUF; ++b) {
        const int hn = h0 + b + NBUF - 1, bn = (b + NBUF - 1) % NBUF;
        multiply_with(0, [&](int k) {
          if (HALF) { read_one(1, b, 1, FRAG_ORDER[k]); request(hn, bn, k); }   // four multiplications: a read and a request behind each
          else if (k < 6) read_one(1, b, 1, FRAG_ORDER[k]);
          else { request(hn, bn, 2 * (k - 6)); request(hn, bn, 2 * (k - 6) + 1); }
        });
        land_and_sync();
        multiply_with(1, [&](int k) { if (k < NFR) read_one(0, (b + 1) % NBUF, 0, FRAG_ORDER[k]); });
      }
    }
    if (CH > 1)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float x = c > 1 ? done[i][j][r] + acc[i][j][r] : acc[i][j][r];
            done[i][j][r] = x;
            acc[i][j][r] = c < CH ? 0.f : x;
          }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the clamped extra requests must not outlive the workgroup's LDS

  // epilogue: accumulator (i, j), register r of lane (r32, half) is row 8 (r / 4) + 4 half + r % 4, column r32
  const int v0 = p.col0 + nt * 256 + 64 * wn;
#pragma unroll
  for (int i = 0; i < (CFG ? 2 : NI); ++i) {
    const int node0 = (CFG || HALF) ? mt * 128 + 32 * (2 * wm + i) : mt * 256 + 32 * (4 * wm + i);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n_here = v0 + 32 * j < p.vocab ? p.n_nodes : 0;   // nothing to store past the vocabulary
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float c = acc[i][j][r];
        const float gmix = CFG ? acc[i + 2][j][r] + p.cfg_scale * (c - acc[i + 2][j][r]) : c;
        const int node = node0 + 8 * (r >> 2) + 4 * half + (r & 3);
        if (node < n_here) p.logits[(int64_t)node * p.vocab + v0 + 32 * j + r32] = gmix / p.temperature;
        if (r == 15) __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

// ------------------------------------------------------------------------------------ row stats
// One workgroup of 1024 threads per row; the row lives in registers (VPT values per thread).
// row_max, exact k-th largest (radix select on order-preserving integer keys), and log-sum-exp
// over the kept entries.
__device__ __forceinline__ uint32_t f32_key(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_f32(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Exact k-th largest by three rounds of radix selection over the order-preserving keys held in
// registers: a 4096-bin LDS histogram (integer atomics) of key bits 31..20, then 1024 bins of bits
// 19..10 among the keys of the chosen bin, then 1024 bins of bits 9..0.  After each round a scan
// from the top bin finds the bin that holds the k-th largest and how many keys lie above it.
// (A row whose entries all share one bin, e.g. all equal, serialises on one LDS address: slow, exact.)
template <int NB, int NT>   // bins (the workgroup's NT threads take NB / NT each, highest first)
__device__ __forceinline__ void find_bin_from_top(const int* hist, int k, int tid, int lane, int wave, int* s_wsum, int* s_bin,
                                                  int* s_above) {
  constexpr int BPT = NB / NT;
  int hb[BPT], loc = 0;
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    const int b = NB - 1 - (BPT * tid + i);
    hb[i] = hist[b];
    loc += hb[i];
  }
  const int incl = wave_scan_incl_i(loc);
  if (lane == 63) s_wsum[wave] = incl;
  __syncthreads();
  // lane l holds the sum of waves 0 .. l % 16
  int upto = s_wsum[lane & 15];
  upto += dpp_i32<0x111, 0xf>(0, upto);
  upto += dpp_i32<0x112, 0xf>(0, upto);
  upto += dpp_i32<0x114, 0xf>(0, upto);
  upto += dpp_i32<0x118, 0xf>(0, upto);
  int before = incl - loc + (wave > 0 ? __builtin_amdgcn_readlane(upto, __builtin_amdgcn_readfirstlane(wave - 1) & 15) : 0);
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    if (before < k && before + hb[i] >= k) { *s_bin = NB - 1 - (BPT * tid + i); *s_above = before; }
    before += hb[i];
  }
  __syncthreads();
}

// Row statistics.  One workgroup of NT = 1024 or 512 threads per row; the row lives in registers (VPT values per thread,
// loaded 16 bytes at a time when the row allows it).
//
// Fast path (top-k active): the order-preserving radix rounds above put sign, exponent and three mantissa bits
// into the first digit, so a row of logits lands in a few dozen of its 4096 bins and the 65536 LDS atomics of
// a long row serialise on them.  Instead the first round bins LINEARLY, bin(x) = clamp(int(x s + c), 0, 4095),
// over the range of a sample of the row (each thread's first load: 4096 entries, in 512 threads 2048), while the rest of the row is
// still arriving.  Any non-decreasing bin function keeps the selection exact: with `above` entries in the bins
// over bin B and above < k <= above + hist[B], the k-th largest is the (k - above)-th largest of bin B.  A
// second sweep over the registers re-evaluates the same fused multiply-add and files every entry of bin B or
// higher (some k + a few dozen of them) into a list of its wave in LDS, by ballots; the candidates of bin B are then
// ranked exactly by their integer keys, and only the listed entries see an exponential - two rounds of a wave's lanes
// for k = 2000, where one list per thread took as many as the fullest of 64 lists (6 to 8), and rows whose kept entries crowd
// into some threads fell back.  What bounds a row once it is in registers is the instructions of its 16 waves and the
// barriers between the stages; values that a wave has no hit among, most of them for small k, cost it a comparison and a branch
// (700 x 65536 with k = 50 47.4 us with a list per thread, 50.9 with a ballot and a count for every value, 45 so).  60 rows x 16384 6.6 ->
// 6.0 us, 462 x 16384 15.3 -> 14.1, 300 x 33088 with k = 8000, where lists per thread overflowed, 0.27 of the time, 1024 x 65536
// 76.6 -> 74.0.  (Two workgroups per compute unit, at 64 registers: 462 x 16384 16.3 us, spilled from 24576 entries on.)
// CUT, rows of more than 32768 entries: counting every entry in LDS is most of the work there.  The entries of the sample alone are counted,
// while the rest of the row arrives, and give a value that somewhat more than k entries of the row are expected to reach; the one sweep lists
// those, and the bins are filled from the lists.  Any cut that at least k entries reach keeps the selection exact; where fewer do, a
// list is full, or the sample's cut lies in its lowest bin, every entry is counted after all.
// 1024 rows x 65536 71.1 -> 65.7 us (see launch_row_stats_long for where it pays).
// Where there is a cut, and in the kernels of 512 threads, each wave begins elsewhere in the row (the sample is a run of 256 entries per wave), so that
// the sample stands for rows whose entries are ordered as well: 1024 x 65536 of which one range of a quarter is finite 479 -> 60 us, 300 x 8192 falling
// along the row, k = 5000, 25 -> 8 with samples from the row's beginning and so.
// Rows the fast path does not fit (degenerate or non-finite sample range, k-th largest in the lowest bin, more
// than RS_CAND candidates, a wave with more than RS_CAP - 64 listed entries) take the radix rounds: slow, exact.
constexpr int RS_LIST = 12288;  // listed entries, dealt evenly to the waves of a workgroup
constexpr int RS_CAND = 1024;   // candidates ranked by counting
constexpr int RS_PRE_OFFSET = 80 * 1024;   // 80 KiB prefetch buffer behind the structure below (1 KiB aligned)

struct RowStatsSmem {
  int hist1[4096], hist2[1024], hist3[1024];
  float list[RS_LIST];          // wave after wave
  float cand[RS_CAND];
  float f_rng[32], f_max[16], f_sum[16];
  int s_wsum[16], n_listed[16];
  int s_bin, s_above, n_cand, flag;
  float s_thr;
};

// Workgroups are persistent: workgroup b takes rows b, b + gridDim.x, ...; the loads of its next row are issued
// as soon as the registers of the current one are no longer needed, so that they overlap the row's tail (list
// processing, candidate ranking, reductions).
// VPT = values per thread: 4, 8, 16, 24, 32, 40, 48 or 64 (rows that are not 16-byte aligned: 4, 16 or 64; NT = 512: 8, 16, 32 or 48),
// the smallest that holds the row.  A chunk that the row does not fill files only its real entries: 33088 entries in a 65536-entry
// frame used to send 32448 padding entries through LDS atomics on one bin, one after the other (78 us for 343 rows, now
// 22; 46 -> 10 us for 200 x 24000).
// NT = 512: two rows on a compute unit, each with half of its waves and registers; while one row is loaded, the other is searched.
template <int VPT, bool VEC, int NT, bool CUT>   // VEC: rows start on 16-byte boundaries and V is a multiple of 4
__global__ __launch_bounds__(NT, 4) void row_stats_kernel(LmParams p) {
  constexpr int NW = NT / 64, RS_CAP = RS_LIST / NW;   // waves, listed entries of one
  extern __shared__ __align__(1024) char rs_smem_raw[];
  RowStatsSmem& sm = *(RowStatsSmem*)rs_smem_raw;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int V = p.vocab;
  const bool topk = p.top_k > 0 && p.top_k < V;
  constexpr int NCH = VPT / 4;
  constexpr bool SPREAD = CUT || NT == 512;   // wave w begins w / NW of the way through the whole chunks
  static_assert(!SPREAD || VEC, "the first load of every wave lies in the row");
  const int rot = SPREAD ? __builtin_amdgcn_readfirstlane(wave) * (V / (4 * NT)) / NW : 0;
  // chunks that the row fills for sure (it did not fit the next smaller frame)
  constexpr int SURE = NT == 512 ? NCH - 4 : VEC ? (VPT == 64 ? 12 : (VPT == 16 ? 2 : (VPT >= 24 ? NCH - 2 : (VPT == 8 ? 1 : 0)))) : (VPT == 64 ? 4 : (VPT == 16 ? 1 : 0));
  // Long rows: the last NPRE 16 KiB chunks of the NEXT row are fetched into LDS (LDS-direct loads, no registers
  // needed) while the current row's registers are still in use - HBM would otherwise idle between the end of a
  // row's loads and the moment its registers are free.  A thread reads back exactly the 16 bytes its own lane
  // fetched, so no barrier is involved.
  constexpr int NPRE = (VEC && NT == 1024 && VPT == 64) ? 5 : 0;
  constexpr int NREG = NCH - NPRE;   // chunks loaded into registers
  float* const pre = (float*)(rs_smem_raw + RS_PRE_OFFSET);
  const unsigned pre_lds = __builtin_amdgcn_readfirstlane((unsigned)(size_t)pre) + 1024u * (unsigned)__builtin_amdgcn_readfirstlane(wave);
  // Slot jj of this thread, element c, holds vocabulary entry 4 (tid + NT mch(jj)) + c: chunk jj of the row, or, where samples are spread, the
  // jj-th from the one that the thread's wave begins with, around the row's end.  Slots 0 .. NREG-1 are loaded into registers (and swept in the order they
  // arrive; slot 0, always inside the row if that fills a chunk, is the sample), slots NREG .. NCH-1 come from LDS and are swept last.  Entries
  // past V are masked to -inf before use.  Every load is unconditional (addresses clamped into the row): all of them are in flight at once.
  auto mch = [&](int jj) { return !SPREAD ? jj : (jj + rot < NCH ? jj + rot : jj + rot - NCH); };   // chunk that slot jj holds
  const bool whole = V == VPT * NT;   // workgroup-uniform: a full row needs no masking
  float x[VPT];
  // (The thread index is passed through an empty asm so that the per-chunk offsets and masks below are recomputed
  // where they are used instead of being kept in registers across the whole row loop.)
  auto load_row = [&](int row) {
    const char* g = (const char*)(p.logits + (int64_t)row * V);   // uniform base + 32-bit byte offsets
    int t = tid;
    asm volatile("" : "+v"(t));
    if (VEC) {
#pragma unroll
      for (int jj = 0; jj < NREG; ++jj) {
        const float4 q = *(const float4*)(g + 4u * (unsigned)min(4 * (t + NT * mch(jj)), V - 4));
        x[4 * jj] = q.x; x[4 * jj + 1] = q.y; x[4 * jj + 2] = q.z; x[4 * jj + 3] = q.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < VPT; ++i) x[i] = *(const float*)(g + 4u * (unsigned)min(4 * (t + NT * (i >> 2)) + (i & 3), V - 1));
    }
  };
  auto prefetch_row = [&](int row) {   // chunks NREG .. NCH-1 -> LDS, lane l's 16 bytes at 16 l behind M0
    const char* g = (const char*)(p.logits + (int64_t)row * V);
    int t = tid;
    asm volatile("" : "+v"(t));
#pragma unroll
    for (int m = 0; m < NPRE; ++m) {
      const unsigned voff = 4u * (unsigned)min(4 * (t + NT * mch(NREG + m)), V - 4);
      const unsigned l = pre_lds + 16384u * m;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(voff), "s"(g) : "memory");
    }
  };
  auto mask_chunks = [&](int jj0, int jj1) {
    if (!whole) {
      int t = tid;
      asm volatile("" : "+v"(t));
#pragma unroll
      for (int jj = SPREAD || jj0 > SURE ? jj0 : SURE; jj < jj1; ++jj)
        if (!SPREAD || 4 * NT * (mch(jj) + 1) > V)   // (a branch of the wave)
#pragma unroll
          for (int c = 0; c < 4; ++c) x[4 * jj + c] = 4 * (t + NT * mch(jj)) + c < V ? x[4 * jj + c] : -INFINITY;
    }
  };
  int row = blockIdx.x;
  if (row < p.n_nodes) {
    prefetch_row(row);   // (the first row has nothing to hide behind: same loads, issued first)
    load_row(row);
  }
  for (; row < p.n_nodes; row += gridDim.x) {
    const int next = row + gridDim.x;
    mask_chunks(0, NREG);
#pragma unroll
    for (int i = 0; i < 4096 / NT; ++i) sm.hist1[tid + NT * i] = 0;
    if (tid == 0) { sm.n_cand = 0; sm.flag = 0; }

    // ---- range of the sample (first chunk of every thread)
    float smax = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    float smin = INFINITY;
#pragma unroll
    for (int c = 0; c < 4; ++c) smin = fminf(smin, x[c] == -INFINITY ? INFINITY : x[c]);   // padding (and -inf logits) aside
    smax = wave_max(smax);
    smin = -wave_max(-smin);
    if (lane == 0) { sm.f_rng[wave] = smax; sm.f_rng[16 + wave] = smin; }
    __syncthreads();
    smax = sm.f_rng[0]; smin = sm.f_rng[16];
#pragma unroll
    for (int w = 1; w < NW; ++w) { smax = fmaxf(smax, sm.f_rng[w]); smin = fminf(smin, sm.f_rng[16 + w]); }
    const float bs = 4096.f / (smax - smin), bc = -smin * bs;
    // usable: finite positive scale and offset (rules out equal, infinite or NaN sample bounds)
    const bool fast = topk && bs > 0.f && bs < INFINITY && fabsf(bc) < INFINITY;

    float mx = -INFINITY;
    auto sweep = [&](int jj0, int jj1) {   // row maximum and first-round histogram of x-chunks jj0 .. jj1-1
      auto chunk = [&](int jj, auto in_row) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          mx = fmaxf(mx, x[4 * jj + c]);
          const float t = __builtin_amdgcn_fmed3f(fmaf(x[4 * jj + c], bs, bc), 0.f, 4095.f);
          if (in_row(c)) atomicAdd(&sm.hist1[(int)t], 1);
        }
        __builtin_amdgcn_sched_barrier(0);   // keep the unrolled sweep from piling up temporaries
      };
      auto always = [](int) { return true; };
      if (fast && whole) {
#pragma unroll
        for (int jj = jj0; jj < jj1; ++jj) chunk(jj, always);
      } else if (fast) {
        int t = tid;
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int jj = jj0; jj < jj1; ++jj) {
          if ((!SPREAD && jj < SURE) || 4 * NT * (mch(jj) + 1) <= V) chunk(jj, always);   // uniform in a wave
          else chunk(jj, [&](int c) { return 4 * (t + NT * mch(jj)) + c < V; });
        }
      } else {
#pragma unroll
        for (int i = 4 * jj0; i < 4 * jj1; ++i) mx = fmaxf(mx, x[i]);
      }
    };
    // ---- the cut: the value that p.sample_rank entries of the sample reach
    float cut = 0.f;
    bool cutting = false;   // workgroup-uniform
    int n_list = 0, most = 0;   // entries listed by this wave
    float* const list = sm.list + wave * RS_CAP;
    // values i0 .. i1 - 1 of this thread that pass go to its wave's list
    auto file = [&](int i0, int i1, auto&& passes) {
#pragma unroll
      for (int i = i0; i < i1; ++i) {
        const bool hit = passes(x[i]);
        const unsigned long long m = __ballot(hit);
        if (m) {
          const int at = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, (unsigned)n_list));
          if (hit) list[at] = x[i];
          n_list += __popcll(m);
          most = max(most, n_list);
          n_list = min(n_list, RS_CAP - 64);         // room for the next 64
        }
        if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (CUT && fast) {
#pragma unroll
      for (int c = 0; c < 4; ++c) atomicAdd(&sm.hist1[(int)__builtin_amdgcn_fmed3f(fmaf(x[c], bs, bc), 0.f, 4095.f)], 1);
      __syncthreads();
      find_bin_from_top<4096, NT>(sm.hist1, p.sample_rank, tid, lane, wave, sm.s_wsum, &sm.s_bin, &sm.s_above);
      const int Bs = sm.s_bin;
      cutting = Bs > 0;
      cut = ((float)Bs - bc) / bs;
#pragma unroll
      for (int i = 0; i < 4096 / NT; ++i) sm.hist1[tid + NT * i] = 0;
    }
    auto first_sweep = [&](int jj0, int jj1) {
      if (CUT && cutting) file(4 * jj0, 4 * jj1, [&](float v) { return v >= cut; });
      else {
        if (CUT && jj0 == 0) __syncthreads();   // the sweep counts into the bins that other waves have just cleared
        sweep(jj0, jj1);
      }
    };
    first_sweep(0, NREG);
    if (NPRE > 0) {
      // every load of this row that went to registers has been waited for; the LDS-direct ones were issued before
      // them and complete in order - waited for explicitly all the same
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      int t = tid;
      asm volatile("" : "+v"(t));
#pragma unroll
      for (int m = 0; m < NPRE; ++m) {
        const float4 q = *(const float4*)(pre + 4096 * m + 4 * t);
        x[4 * (NREG + m)] = q.x; x[4 * (NREG + m) + 1] = q.y; x[4 * (NREG + m) + 2] = q.z; x[4 * (NREG + m) + 3] = q.w;
      }
      mask_chunks(NREG, NCH);
      first_sweep(NREG, NCH);
      // the values are in registers (the sweep consumed them): the buffer can take the next row's chunks
      if (next < p.n_nodes) prefetch_row(next);
    }
    if (CUT && cutting)
      for (int j = lane; j < n_list; j += 64) mx = fmaxf(mx, list[j]);
    auto row_max = [&]() {
      mx = wave_max(mx);
      if (lane == 0) {
        sm.f_max[wave] = mx;
        sm.n_listed[wave] = most > RS_CAP - 64 ? -(1 << 20) : n_list;
      }
      __syncthreads();                       // maxima, lists and every atomic of the sweep
      mx = sm.f_max[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) mx = fmaxf(mx, sm.f_max[w]);
    };
    row_max();
    if (CUT && cutting) {
      int total = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) total += sm.n_listed[w];
      if (total >= p.top_k) {
        for (int j = lane; j < n_list; j += 64) atomicAdd(&sm.hist1[(int)__builtin_amdgcn_fmed3f(fmaf(list[j], bs, bc), 0.f, 4095.f)], 1);
        __syncthreads();
      } else {   // the sample was misleading, or a list is full: every entry is looked at, as in narrower rows
        __syncthreads();   // everyone has read the counts and maxima that are written again
        cutting = false;
        n_list = most = 0;
        mx = -INFINITY;
        sweep(0, NCH);
        row_max();
      }
    }

    float thr = -INFINITY, se = 0.f;
    bool done = false;
    int B = 0, n_c = 0, k = p.top_k;
    if (fast) {
      find_bin_from_top<4096, NT>(sm.hist1, k, tid, lane, wave, sm.s_wsum, &sm.s_bin, &sm.s_above);
      B = sm.s_bin;
      n_c = sm.hist1[B];
      k -= sm.s_above;                     // rank of the k-th largest inside bin B, 1 = largest
      if (B > 0 && n_c <= RS_CAND) {       // workgroup-uniform
        if (!cutting) {
          const float Bf = (float)B;
          file(0, VPT, [&](float v) { return fmaf(v, bs, bc) >= Bf; });   // bin(x) >= B (B >= 1: the clamp at 0 plays no part; the one at 4095 cannot matter)
          if (most > RS_CAP - 64 && lane == 0) sm.flag = 1;
          __syncthreads();
        }
        done = sm.flag == 0;
      }
    }
    // Without top-k every entry is kept: the sum is taken from the registers (padding is -inf and adds nothing).  Read again four
    // bytes at a time, as by the rounds below, it took 60 rows x 16384 from 4.1 to 5.5 us, x 33088 from 5.2 to 8.8, x 65536
    // from 7.2 to 14.7.
    if (!topk)
#pragma unroll
      for (int i = 0; i < VPT; i += 4) se += (__expf(x[i] - mx) + __expf(x[i + 1] - mx)) + (__expf(x[i + 2] - mx) + __expf(x[i + 3] - mx));
    // The registers are free (the rounds below re-read the row): the next row arrives during this row's tail.
    if (next < p.n_nodes) load_row(next);
    if (done) {
      // listed entries: above bin B -> kept; in bin B -> candidate; below (where there was a cut) -> not kept
      const float Bf = (float)B, B1f = (float)(B + 1);
      for (int j = lane; j < n_list; j += 64) {
        const float xv = list[j], t = fmaf(xv, bs, bc);
        if (B < 4095 && t >= B1f) se += __expf(xv - mx);
        else if (t >= Bf) sm.cand[atomicAdd(&sm.n_cand, 1)] = xv;
      }
      __syncthreads();
      // exact k-th largest of the n_c candidates by counting (ties: lower list index first); wave w ranks
      // candidates w, w + NW, ..., its lanes share the comparisons
      for (int i = wave; i < n_c; i += NW) {
        const uint32_t ki = f32_key(sm.cand[i]);
        int rank = 0;
        for (int j = lane; j < n_c; j += 64) {
          const uint32_t kj = f32_key(sm.cand[j]);
          rank += (kj > ki || (kj == ki && j < i)) ? 1 : 0;
        }
        rank = wave_sum_i(rank);
        if (lane == 0 && rank == k - 1) sm.s_thr = key_f32(ki);
      }
      __syncthreads();
      thr = sm.s_thr;
      const uint32_t tk = f32_key(thr);
      for (int i = tid; i < n_c; i += NT) {
        const float xi = sm.cand[i];
        if (f32_key(xi) >= tk) se += __expf(xi - mx);
      }
    } else if (topk) {
      // Radix rounds on the order-preserving keys.  Slow and exact: the row is read again from memory (mostly the
      // caches) in every round, a few registers at a time.
      const float* g = p.logits + (int64_t)row * V;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4096 / NT; ++i) sm.hist1[tid + NT * i] = 0;
#pragma unroll
      for (int i = 0; i < 1024 / NT; ++i) sm.hist2[tid + NT * i] = sm.hist3[tid + NT * i] = 0;
      __syncthreads();
      k = p.top_k;
      for (int v = tid; v < V; v += NT) atomicAdd(&sm.hist1[f32_key(g[v]) >> 20], 1);
      __syncthreads();
      find_bin_from_top<4096, NT>(sm.hist1, k, tid, lane, wave, sm.s_wsum, &sm.s_bin, &sm.s_above);
      const uint32_t b1 = (uint32_t)sm.s_bin;
      k -= sm.s_above;
      __syncthreads();   // s_bin / s_above are rewritten by the next round
      for (int v = tid; v < V; v += NT) {
        const uint32_t key = f32_key(g[v]);
        if ((key >> 20) == b1) atomicAdd(&sm.hist2[(key >> 10) & 1023u], 1);
      }
      __syncthreads();
      find_bin_from_top<1024, NT>(sm.hist2, k, tid, lane, wave, sm.s_wsum, &sm.s_bin, &sm.s_above);
      const uint32_t b12 = (b1 << 10) | (uint32_t)sm.s_bin;
      k -= sm.s_above;
      __syncthreads();
      for (int v = tid; v < V; v += NT) {
        const uint32_t key = f32_key(g[v]);
        if ((key >> 10) == b12) atomicAdd(&sm.hist3[key & 1023u], 1);
      }
      __syncthreads();
      find_bin_from_top<1024, NT>(sm.hist3, k, tid, lane, wave, sm.s_wsum, &sm.s_bin, &sm.s_above);
      const uint32_t thr_key = (b12 << 10) | (uint32_t)sm.s_bin;
      thr = key_f32(thr_key);
      for (int v = tid; v < V; v += NT) {
        const float xv = g[v];
        if (f32_key(xv) >= thr_key) se += __expf(xv - mx);
      }
    }
    se = wave_sum(se);
    if (lane == 0) sm.f_sum[wave] = se;
    __syncthreads();
    if (tid == 0) {
      float tot = 0.f;
      for (int w = 0; w < NW; ++w) tot += sm.f_sum[w];
      p.row_max[row] = mx;
      p.row_thr[row] = thr;
      p.row_lse[row] = mx + logf(tot);
    }
  }
}

LmParams make_params(const lmhead_args* a) {
  LmParams p;
  p.h_cond = a->h_cond;
  p.h_uncond = a->h_uncond;
  p.w = a->w;
  p.logits = a->logits;
  p.row_max = a->row_max;
  p.row_thr = a->row_thr;
  p.row_lse = a->row_lse;
  p.hp_cond = nullptr;
  p.hp_uncond = nullptr;
  p.n_nodes = a->n_nodes;
  p.hidden = a->hidden;
  p.vocab = a->vocab;
  p.col0 = 0;
  p.cfg_scale = a->cfg_scale;
  p.temperature = a->temperature;
  p.top_k = a->top_k;
  p.sample_rank = 0;
  return p;
}

}  // namespace

hipError_t launch_lmhead_f32(cascade_ctx* ctx, const lmhead_args* a) {
  hipStream_t stream = ctx->stream;
  KernelTimer t(ctx, CASCADE_K_LMHEAD);
  LmParams p = make_params(a);
  const bool vec = a->hidden % 4 == 0 && (((uintptr_t)a->h_cond | (uintptr_t)a->h_uncond | (uintptr_t)a->w) & 15) == 0;
  const bool few = a->n_nodes <= 16;   // one node block per workgroup, or four sharing the weights they load
  dim3 grid((a->vocab + 15) / 16, few ? 1 : (a->n_nodes + 63) / 64);
#define CASCADE_LAUNCH_F32(NB, CFG, VEC) CASCADE_TIMED_LAUNCH(t, (lmhead_f32_kernel<NB, CFG, VEC>), grid, dim3(256), 0, stream, p)
  if (a->h_uncond) {
    if (few) { if (vec) CASCADE_LAUNCH_F32(1, true, true); else CASCADE_LAUNCH_F32(1, true, false); }
    else { if (vec) CASCADE_LAUNCH_F32(4, true, true); else CASCADE_LAUNCH_F32(4, true, false); }
  } else {
    if (few) { if (vec) CASCADE_LAUNCH_F32(1, false, true); else CASCADE_LAUNCH_F32(1, false, false); }
    else { if (vec) CASCADE_LAUNCH_F32(4, false, true); else CASCADE_LAUNCH_F32(4, false, false); }
  }
#undef CASCADE_LAUNCH_F32
  return hipGetLastError();
}

template <int AM, int AN, int WM, int WN, int KW, int KS, int NST, bool CFG, bool PW, bool DIRECT, bool STREAM>
hipError_t launch_ring_k(cascade_ctx* ctx, const LmParams& p, int n_cols) {
  constexpr int BM = 32 * AM * WM, BN = 32 * AN * WN, NODES = CFG ? BM / 2 : BM;
  constexpr int RING = NST * (BM + BN) / 32 * KS * 1024, RED = KW > 1 ? 8 * AM * AN * 4096 : 0;
  constexpr int smem = RING > RED ? RING : RED;
  static_assert(smem <= 160 * 1024, "LDS of a compute unit");
  auto kern = lmhead_bf16_ring_kernel<AM, AN, WM, WN, KW, KS, NST, CFG, PW, DIRECT, STREAM>;
  static bool attr_done = false;   // one flag per template instance
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const int n_mtiles = (p.n_nodes + NODES - 1) / NODES;
  KernelTimer t(ctx, CASCADE_K_LMHEAD);
  CASCADE_TIMED_LAUNCH(t, kern, dim3((n_cols + BN - 1) / BN * n_mtiles), dim3(512), smem, ctx->stream, p, n_mtiles);
  return hipGetLastError();
}
template <int AM, int AN, int WM, int WN, int KW, int KS, int NST, bool CFG, bool PW>
hipError_t launch_ring_t(cascade_ctx* ctx, const LmParams& p, int n_cols, bool stream) {
  return stream ? launch_ring_k<AM, AN, WM, WN, KW, KS, NST, CFG, PW, true, true>(ctx, p, n_cols)
                : launch_ring_k<AM, AN, WM, WN, KW, KS, NST, CFG, PW, true, false>(ctx, p, n_cols);
}
constexpr int LM_UNALIGNED = -1;   // ordinary loads: 64 x 64 or 128 x 128
template <bool CFG, bool PW>
hipError_t launch_ring(cascade_ctx* ctx, const LmParams& p, int tile, int n_cols, bool stream) {
  switch (tile) {
    case 0: return launch_ring_t<2, 1, 1, 2, 4, 4, 6, CFG, PW>(ctx, p, n_cols, stream);
    case 1: return launch_ring_t<2, 2, 2, 1, 4, 4, 4, CFG, PW>(ctx, p, n_cols, stream);
    case 2: return launch_ring_t<2, 2, 1, 4, 2, 4, 3, CFG, PW>(ctx, p, n_cols, stream);
    case 3: return launch_ring_t<2, 2, 2, 2, 2, 4, 4, CFG, PW>(ctx, p, n_cols, stream);
    case LM_UNALIGNED: return p.n_nodes * (CFG ? 2 : 1) <= 64 ? launch_ring_k<2, 1, 1, 2, 4, 8, 2, CFG, PW, false, false>(ctx, p, n_cols)
                                                              : launch_ring_k<2, 2, 2, 2, 2, 8, 2, CFG, PW, false, false>(ctx, p, n_cols);
    default: return launch_ring_t<2, 2, 4, 2, 1, 4, 3, CFG, PW>(ctx, p, n_cols, stream);
  }
}

// Tiles of the projection: ring kernel 0-4, tiled kernel 5 (128 x 256, plain rows only) and 6 (256 x 256).  us = one tile
// on every compute unit, hidden 4096, the weight stream aside; a last round that fills few units costs `few` of that plus
// the filled share of the rest (the clock rises when units idle), a tile of padding rows only `pad` (zeros draw less
// power).  Fitted to 100 sizes (16-1024 rows, 16384-65536 columns, plain, pairs and row-major weights), all seven tiles each, before
// weights were streamed; see lm_estimate_us for how well they choose since.
struct LmTile {
  int rows, cols;
  float us, few, pad;
};
constexpr LmTile LM_TILES[7] = {{64, 64, 17.6f, 1.f, 0.83f}, {128, 64, 26.8f, 1.f, 0.64f}, {64, 256, 46.5f, 0.91f, 1.f}, {128, 128, 41.f, 0.83f, 0.8f},
                                {256, 128, 72.f, 0.77f, 0.9f}, {128, 256, 68.5f, 0.87f, 0.77f}, {256, 256, 115.4f, 0.66f, 0.58f}};
constexpr int LM_RING_TILES = 5;

// Weights from this size on are streamed (see the ring kernel): a third of the last-level cache.  A step of 60 nodes whose
// weights no cache holds, default policy and streamed: 8192 x 4096 (67 MB) 56.8 and 52.1 us, 16384 x 3072 (101 MB) 59 and 53, 16384 x
// 4096 63 and 56, 40000 x 4096 111 and 100.  Three smaller matrices used in turn stay in the cache together: 4096 x 2048 38.0 and
// 41.1, 8192 x 4096 49.5 and 52.2, but 16384 x 3072 57 and 53.
// The rule counts on the layers of a model that pass between two projections.  The projection alone, default policy and
// streamed, behind a copy of 1 GiB: 60 x 16384 x 4096 38.4 and 27.1 us, 120 x 33088 x 2048 (128 x 128) 64.2 and 51.8, 256 x 65536 x 4096
// (256 x 128) 163 and 147; over copies of the weights in turn, of which the cache keeps some: 25.7 and 24.4, 51.3 and 50.2, 152
// and 155.  A caller that repeats it on one matrix of at most 256 MB with nothing between finds that in the cache only without
// streaming: 60 x 16384 x 4096 23 and 24 us, 120 x 16384 x 4096 26 and 33, 60 pairs x 33088 x 2048 row-major 23 and 35.
constexpr int64_t LM_STREAM_BYTES = (int64_t)85 << 20;

// Whether a launch of tiles over `rows` rows streams its weights.  In the ring kernel, three row tiles and more that share a column
// of weights are bound by the matrix cores: 343 pairs x 33088 x 2048 the same over cold weights (122 us), 116 against 122 where the
// cache holds them.  128 x 256 tiles stream for any number of them: behind a copy of 1 GiB 300 rows x 16384 x 4096 69.7 -> 61.5 us, 480 x 16384 x 4096
// 71.2 -> 66.0, 480 x 65536 x 2048 152 -> 142; over copies in turn 400 x 33088 x 4096 146.4 -> 143.1, 256 x 65536 x 4096 157.3 -> 153.7,
// 200 x 65536 x 2048 80.9 -> 85.1.  Smaller weights, not streamed and streamed: 300 x 20480 x 2048 over copies in turn 38.0 and 38.7,
// repeated 34.9 and 38.5.
bool lm_streams(int tile, int rows, int vocab, int hidden) {
  if (tile < 0 || tile > 5 || (int64_t)vocab * hidden * 2 < LM_STREAM_BYTES) return false;
  return tile == 5 || (rows + LM_TILES[tile].rows - 1) / LM_TILES[tile].rows <= 2;
}

// 256 x 128 tiles that stream their weights to one tile of mixed rows (up to 256), fitted again since they do: whole rounds take less, of that a part
// whatever the hidden dimension (start and stores), and a round that is not full takes nearly as long.  Projection in 128 x 256 tiles, where each weight
// is requested twice, which were taken, and so, us: 256 x 65536 x 4096 154.1 and 151.5, 184 rows 154.5 and 144.3, 130 rows 149.7 and 139.5, 200 x
// 40000 x 4096 111.5 and 104.8, 200 x 65536 x 2048 88.1 and 87.9; with two tiles of rows the other way round, 400 x 36032 x 4096 154.5 and 161.4.
// (Plain rows, for which 256 x 128 is up to 10 % faster as well, still take the old costs.)
constexpr LmTile LM_STREAMED_256X128 = {256, 128, 63.f, 0.937f, 0.9f};
constexpr float LM_STREAMED_START_US = 8.f;

// Time of the tiles of a launch over n_cols columns: rounds over the compute units.
float lm_rounds_us(int i, int rows, int n_cols, int vocab, int hidden, bool mixed, int n_cu) {
  const bool streamed = i == 4 && mixed && rows <= 256 && lm_streams(i, rows, vocab, hidden);
  const LmTile& tile = streamed ? LM_STREAMED_256X128 : LM_TILES[i];
  const float start = streamed ? LM_STREAMED_START_US : 0.f;
  const int n_mtiles = (rows + tile.rows - 1) / tile.rows;
  const long tiles = (long)n_mtiles * ((n_cols + tile.cols - 1) / tile.cols);
  const float last = (float)(tiles % n_cu) / n_cu, used = (float)rows / ((float)n_mtiles * tile.rows);
  const float rounds = (float)(tiles / n_cu) + (last > 0.f ? tile.few + (1.f - tile.few) * last : 0.f);
  return rounds * (start + (tile.us - start) * (hidden / 4096.f)) * (tile.pad + (1.f - tile.pad) * used);
}
// Estimated time of the whole projection: that, and the weight stream at 6.2 TB/s, which overlap only partly.  Over 250
// sizes (16-800 rows, 16384-65536 columns, hidden 2048 and 4096, weights from HBM, streamed where lm_streams says so) a single tile, where one is
// chosen, is 1.0 % behind the fastest one in the mean, at worst 23 % (90 rows x 49152 x 2048: 54.3 us in 128 x 64, 44.0 in 128 x 256;
// 16 pairs of row-major rows x 49152 x 2048 48.5 in 64 x 256, 39.3 in 64 x 64).
float lm_estimate_us(float a, int vocab, int hidden) {
  const float b = (float)vocab * hidden * 2.f / 6.2e6f;
  return sqrtf(a * a + b * b);
}

// How a projection is cut: columns [0, split) in tiles of one shape, [split, vocab) in tiles of another (split = vocab: one
// launch).  A last round that fills few compute units costs as much as a full one, so the columns that fill whole rounds
// take the large tile and the rest a smaller one in a second launch: 686 rows (guidance pairs) x 33088 x 2048 are 777
// tiles of 256 x 128, four rounds of 256 units (133 us); 768 of them and 55 of 64 x 64: 122 us.  Where columns are cut (71 of
// those 250 sizes) that is 10 % faster than the fastest single tile in the mean, 27 % at best and 4 % slower at worst (300 pairs x
// 33024 x 2048: 103.9 us, 100.3 in 256 x 256).
struct LmPlan {
  int main, rest, split;
  float us;
};
constexpr float LM_SECOND_LAUNCH_US = 4.f;

LmPlan lm_plan(const lmhead_args* a, bool packed_w, bool premix, bool cfg, int n_cu) {
  const int rows = a->n_nodes * (cfg ? 2 : 1), V = a->vocab;
  auto usable = [&](int i) {
    if (i >= LM_RING_TILES && !packed_w) return false;
    if (i == 5) return !cfg;
    // 256 x 256 tiles sum the hidden dimension in one chain; faster for fewer rows as well (256 x 65536: 138 us against 169),
    // but there every other tile is twice as close to the exact sums
    return i != 6 || (V % 256 == 0 && rows >= (cfg ? 512 : 257));
  };
  LmPlan best = {0, 0, V, INFINITY};
  for (int i = 0; i < 7; ++i) {
    if (!usable(i)) continue;
    const float pack = i >= LM_RING_TILES && !premix ? 4.f : 0.f;   // the tiled kernel needs its rows packed (the mix packs them on the way)
    const LmTile& t = LM_TILES[i];
    const float whole = lm_estimate_us(lm_rounds_us(i, rows, V, V, a->hidden, premix, n_cu), V, a->hidden) + pack;
    if (whole < best.us) best = {i, i, V, whole};
    const int n_mtiles = (rows + t.rows - 1) / t.rows, n_ntiles = (V + t.cols - 1) / t.cols;
    const int full = (int)((long)n_mtiles * n_ntiles / n_cu) * n_cu / n_mtiles;   // column tiles in whole rounds
    if (full == 0 || full * t.cols >= V) continue;
    for (int j = 0; j < 7; ++j) {
      if (!usable(j) || (i < LM_RING_TILES && j >= LM_RING_TILES)) continue;
      const float c = lm_rounds_us(i, rows, full * t.cols, V, a->hidden, premix, n_cu) + lm_rounds_us(j, rows, V - full * t.cols, V, a->hidden, premix, n_cu);
      const float us = lm_estimate_us(c, V, a->hidden) + pack + LM_SECOND_LAUNCH_US;
      if (us < best.us) best = {i, j, full * t.cols, us};
    }
  }
  return best;
}

// guidance mixed into the hidden rows in front of the projection: from there on a plain projection of n_nodes rows
bool lm_premix(const lmhead_args* a) {
  return a->h_uncond != nullptr && a->cfg_mix == CASCADE_CFG_MIX_HIDDEN && a->w_layout == CASCADE_W_PACKED32;
}

LmPlan lm_choose(const lmhead_args* a, int n_cu) {
  const bool premix = lm_premix(a), cfg = a->h_uncond != nullptr && !premix;
  LmPlan plan = lm_plan(a, a->w_layout == CASCADE_W_PACKED32, premix, cfg, n_cu);
  // (mixed and packed rows lie in the workspace; both passes that write them read the caller's rows with ordinary loads)
  const bool rows_direct = !premix && (plan.main < LM_RING_TILES || plan.rest < LM_RING_TILES);
  if (((uintptr_t)a->w | (rows_direct ? (uintptr_t)a->h_cond | (uintptr_t)(cfg ? a->h_uncond : nullptr) : 0)) & 15)
    plan.main = plan.rest = LM_UNALIGNED, plan.split = a->vocab;
  return plan;
}

// one launch over columns [p.col0, p.col0 + n_cols)
hipError_t launch_lm_tile(cascade_ctx* ctx, const LmParams& p, int tile, bool cfg, bool packed_w, int n_cols) {
  const bool stream = lm_streams(tile, p.n_nodes * (cfg ? 2 : 1), p.vocab, p.hidden);
  if (tile < LM_RING_TILES) {
    if (packed_w) return cfg ? launch_ring<true, true>(ctx, p, tile, n_cols, stream) : launch_ring<false, true>(ctx, p, tile, n_cols, stream);
    return cfg ? launch_ring<true, false>(ctx, p, tile, n_cols, stream) : launch_ring<false, false>(ctx, p, tile, n_cols, stream);
  }
  const bool half = tile == 5;
  const int nodes_per_tile = (cfg || half) ? 128 : 256, n_mtiles = (p.n_nodes + nodes_per_tile - 1) / nodes_per_tile;
  const size_t smem = (size_t)4 * 32 * 1024;   // ring of four 32 KiB half-stages
  static bool attr_done[4] = {false, false, false, false};
  auto kern = cfg ? lmhead_bf16_tiled_kernel<true, false, false>
                  : (half ? (stream ? lmhead_bf16_tiled_kernel<false, true, true> : lmhead_bf16_tiled_kernel<false, true, false>)
                          : lmhead_bf16_tiled_kernel<false, false, false>);
  const int which = cfg ? 0 : (half ? 1 + stream : 3);
  if (!attr_done[which]) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_done[which] = true;
  }
  KernelTimer t(ctx, CASCADE_K_LMHEAD);
  CASCADE_TIMED_LAUNCH(t, kern, dim3((n_cols + 255) / 256 * n_mtiles), dim3(512), smem, ctx->stream, p, n_mtiles);
  return hipGetLastError();
}

void plan_lmhead_streams(const lmhead_args* a, int n_cu, int32_t* streams, int32_t* rest_streams) {
  const LmPlan plan = lm_choose(a, n_cu);
  const int rows = a->n_nodes * (a->h_uncond != nullptr && !lm_premix(a) ? 2 : 1);
  *streams = lm_streams(plan.main, rows, a->vocab, a->hidden);
  *rest_streams = lm_streams(plan.rest, rows, a->vocab, a->hidden);
}

void plan_lmhead_bf16(const lmhead_args* a, int n_cu, int32_t* tile, int32_t* rest_tile, int32_t* rest_column) {
  const LmPlan plan = lm_choose(a, n_cu);
  *tile = plan.main;
  *rest_tile = plan.rest;
  *rest_column = plan.split;
}

hipError_t launch_lmhead_bf16(cascade_ctx* ctx, const lmhead_args* a) {
  LmParams p = make_params(a);
  const bool packed_w = a->w_layout == CASCADE_W_PACKED32;
  const bool premix = lm_premix(a), cfg = a->h_uncond != nullptr && !premix;
  const LmPlan plan = lm_choose(a, ctx->n_cu);
  uint4* hc = (uint4*)ctx->hpack_ws;
  if (plan.main < LM_RING_TILES) {
    if (premix) {
      const int64_t n16 = (int64_t)a->n_nodes * a->hidden / 8;
      if ((size_t)n16 * 16 > ctx->hpack_ws_bytes) return hipErrorInvalidValue;
      KernelTimer t(ctx, CASCADE_K_PACK);
      CASCADE_TIMED_LAUNCH(t, mix_rows_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, ctx->stream, (const uint4*)a->h_cond,
                           (const uint4*)a->h_uncond, hc, (int)n16, a->cfg_scale);
      p.h_cond = hc;
    }
  } else {
    // this step's hidden states in operand order (zero rows up to a whole tile)
    const int rblocks = (a->n_nodes + 255) / 256 * 8;
    const size_t per = (size_t)rblocks * 32 * a->hidden * 2;
    if (per * (cfg ? 2 : 1) > ctx->hpack_ws_bytes) return hipErrorInvalidValue;
    uint4* hu = (uint4*)(ctx->hpack_ws + per);
    dim3 pgrid((a->hidden / 16 + 3) / 4, rblocks, cfg ? 2 : 1);
    KernelTimer t(ctx, CASCADE_K_PACK);
    if (premix) {
      CASCADE_TIMED_LAUNCH(t, pack32_mix_kernel, pgrid, dim3(256), 0, ctx->stream, (const uint16_t*)a->h_cond,
                           (const uint16_t*)a->h_uncond, hc, plan.rest < LM_RING_TILES ? hu : nullptr, a->n_nodes, a->hidden, a->cfg_scale);
      if (plan.rest < LM_RING_TILES) p.h_cond = hu;
    } else {
      CASCADE_TIMED_LAUNCH(t, pack32_kernel, pgrid, dim3(256), 0, ctx->stream, (const uint16_t*)a->h_cond, hc,
                           (const uint16_t*)a->h_uncond, hu, a->n_nodes, a->hidden);
    }
    p.hp_cond = hc;
    p.hp_uncond = hu;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_lm_tile(ctx, p, plan.main, cfg, packed_w, plan.split);
  if (e != hipSuccess || plan.split == a->vocab) return e;
  p.col0 = plan.split;
  return launch_lm_tile(ctx, p, plan.rest, cfg, packed_w, a->vocab - plan.split);
}

hipError_t launch_pack_w(cascade_ctx* ctx, const void* w, int vocab, int hidden, void* w_packed) {
  dim3 grid((hidden / 16 + 3) / 4, vocab / 32);
  hipLaunchKernelGGL(pack32_kernel, grid, dim3(256), 0, ctx->stream, (const uint16_t*)w, (uint4*)w_packed,
                     (const uint16_t*)nullptr, (uint4*)nullptr, vocab, hidden);
  return hipGetLastError();
}

template <int VPT, bool VEC, int NT, bool CUT = false>
hipError_t launch_row_stats_t(cascade_ctx* ctx, const LmParams& p) {
  constexpr int PER_CU = 1024 / NT;
  static_assert(sizeof(RowStatsSmem) <= RS_PRE_OFFSET, "the prefetch buffer starts behind the structure");
  static_assert(PER_CU * sizeof(RowStatsSmem) <= 160 * 1024, "LDS of a compute unit");
  const size_t smem = (VEC && NT == 1024 && VPT == 64) ? RS_PRE_OFFSET + 80 * 1024 : sizeof(RowStatsSmem);
  auto kern = row_stats_kernel<VPT, VEC, NT, CUT>;
  static bool attr_done = false;   // one flag per template instance
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  KernelTimer t(ctx, CASCADE_K_ROW_STATS);
  // as many workgroups as the compute units hold (128 registers for each of 1024 threads), each walking its share of the rows
  const int most = PER_CU * ctx->n_cu, grid = p.n_nodes < most ? p.n_nodes : most;
  CASCADE_TIMED_LAUNCH(t, kern, dim3(grid), dim3(NT), smem, ctx->stream, p);
  return hipGetLastError();
}
// Rows of more than 32768 entries, with a cut where it pays.  Every entry counted and a cut, us: 60 rows x 49152 10.6 and 10.3, x 65536 13.5 and
// 12.8; 400 x 33088 22.0 and 21.0, x 57344 33.0 and 30.0; 1024 x 65536 71.1 and 65.7; but 60 x 33088 9.3 and 9.8, where the search in
// the sample takes longer than the counting, and with long lists 60 x 65536 with k = 8000 14.7 and 14.9, 400 such rows 38.8 and 41.0.
template <int VPT>
hipError_t launch_row_stats_long(cascade_ctx* ctx, LmParams& p) {
  // The sample is sixteen runs of 256 entries.  If they stand for the row, the cut lets four standard deviations of a random sample's count more
  // than k entries through; where neighbours are alike it may let through fewer, or too many for the lists (704 per wave).  A tenth of the row is asked for at most.
  const float mean = (float)p.top_k * 4096 / p.vocab, rank = mean + 4.f * sqrtf(mean) + 8.f;
  const bool cut = (VPT > 40 || p.n_nodes >= 128) && p.top_k > 0 && rank <= 0.1f * 4096;
  p.sample_rank = cut ? (int)rank : 0;
  return cut ? launch_row_stats_t<VPT, true, 1024, true>(ctx, p) : launch_row_stats_t<VPT, true, 1024, false>(ctx, p);
}

hipError_t launch_row_stats(cascade_ctx* ctx, const lmhead_args* a) {
  LmParams p = make_params(a);
  const int V = a->vocab;
  // 16-byte loads need every row to start on a 16-byte boundary
  const bool vec = V % 4 == 0 && ((uintptr_t)a->logits & 15u) == 0;
  if (!vec) return V <= 4096 ? launch_row_stats_t<4, false, 1024>(ctx, p) : (V <= 16384 ? launch_row_stats_t<16, false, 1024>(ctx, p) : launch_row_stats_t<64, false, 1024>(ctx, p));
  // More rows than compute units: two on each at a time, 512 threads for a row.  1024 threads for one at a time and so, us: 280 rows x 4096
  // 8.3 and 6.4, x 8192 9.3 and 6.8, x 16384 12.4 and 9.7; 400 x 16384 13.3 and 10.3, x 24576 16.6 and 12.9; 1024 x 8192 18.2 and
  // 13.1, x 16384 25.4 and 19.2, x 24576 33.1 and 23.8.  Fewer rows have the whole compute unit (60 x 16384 6.2 us, 6.8 in 512
  // threads), and wider ones are bound by its instructions (400 x 33088 22.1 and 21.6, and registers are spilled).
  if (a->n_nodes > ctx->n_cu && V <= 24576) {
    if (V <= 4096) return launch_row_stats_t<8, true, 512>(ctx, p);
    if (V <= 8192) return launch_row_stats_t<16, true, 512>(ctx, p);
    return V <= 16384 ? launch_row_stats_t<32, true, 512>(ctx, p) : launch_row_stats_t<48, true, 512>(ctx, p);
  }
  switch ((V + 8191) / 8192) {
    case 1: return V <= 4096 ? launch_row_stats_t<4, true, 1024>(ctx, p) : launch_row_stats_t<8, true, 1024>(ctx, p);
    case 2: return launch_row_stats_t<16, true, 1024>(ctx, p);
    case 3: return launch_row_stats_t<24, true, 1024>(ctx, p);
    case 4: return launch_row_stats_t<32, true, 1024>(ctx, p);
    case 5: return launch_row_stats_long<40>(ctx, p);
    case 6: return launch_row_stats_long<48>(ctx, p);
    default: return launch_row_stats_long<64>(ctx, p);
  }
}
