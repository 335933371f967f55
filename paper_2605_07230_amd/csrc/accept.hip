// cascade_accept kernel for gfx950 (Sec. 4.1 cosine similarity of target hidden states; Eq. 1
// interchangeable set; Eq. 2 convergence set; Eq. 3 aggregated mass).
//
// One workgroup per node a (several where its rows are wide and do not go through the matrix cores).  Everything a needs is the cosine of its own feature row against its
// parent, its siblings and its children: one row against at most 1 + 63 + 64 others.  The others
// are taken in blocks of 15; with a as the 16th row, one 16 x 16 Gram tile per block gives every
// a . x (row of a) and every |x|^2 (diagonal) at once.  For bf16 hidden states the tile runs on
// v_mfma_f32_16x16x32_bf16 with the four waves splitting the hidden dimension (operands loaded
// straight from global memory as 16-byte k-contiguous pieces); f32 rows (and logit-space
// similarity) are swept once for eight others at a time on the vector ALU (narrow ones for four, by each wave).  The probabilities of the siblings' and children's
// tokens under the parent's distribution are gathered while the rows are still in flight; the sets
// I_a and C_a, the distinct-token masses and all outputs then need only ballots and LDS.
#include <type_traits>

#include "common.h"

namespace {

constexpr int MAXW = CASCADE_MAX_WIDTH;   // children per node
constexpr int GN = MAXW + 1;              // rows of the Gram matrix: parent + children
constexpr int GP = GN + 1;                // LDS pitch

// probability of vocabulary entry t under a row's filtered softmax
__device__ __forceinline__ float prob_of(const float* logits_row, float thr, float lse, int t) {
  const float gv = logits_row[t];
  return gv >= thr ? __expf(gv - lse) : 0.f;
}

__device__ __forceinline__ float cos_from(float ab, float aa, float bb) {
  return (aa > 0.f && bb > 0.f) ? ab / (sqrtf(aa) * sqrtf(bb)) : 0.f;
}

union Frag8 {
  bf16x8 v;
  uint4 u;
};

// Gram tile of 16 rows with themselves over k in [k0, k1), (k1 - k0) a multiple of 32; row is this lane's row, g its 8-wide k group.  Eight
// steps' loads are issued together.  Lanes of rows that a tile does not have (live = false) load nothing: a tile holds 7 to 8 rows in the mean; their
// entries of the result are not looked at.  In steps of four, every lane loading: 60 nodes x 2048 6.0 -> 4.8 us, x 5120 9.8 -> 6.3, four such
// trees x 5120 11.2 -> 8.0 (steps of four, so: 5.2, 7.5, 8.8; of sixteen: 5.3, 7.6, 9.6).
__device__ __forceinline__ f32x4 gram_tile(const uint16_t* row, bool live, int k0, int k1, int g) {
  f32x4 acc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto steps = [&](auto count, int k) {
    constexpr int N = decltype(count)::value;
    Frag8 f[N];
#pragma unroll
    for (int s = 0; s < N; ++s) f[s].u = make_uint4(0, 0, 0, 0);
    if (live)
#pragma unroll
      for (int s = 0; s < N; ++s) f[s].u = *(const uint4*)(row + k + 32 * s + 8 * g);
#pragma unroll
    for (int s = 0; s < N; ++s) acc[s & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[s].v, f[s].v, acc[s & 3], 0, 0, 0);
  };
  int k = k0;
  for (; k + 256 <= k1; k += 256) steps(std::integral_constant<int, 8>{}, k);
  for (; k < k1; k += 32) steps(std::integral_constant<int, 1>{}, k);
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// The same Gram tile of one row set with itself over NS k-steps, all of the lane's NS 16-byte pieces
// requested before the first multiplication (one round trip instead of NS / 4), side() issued
// behind them (loads return in order, so what side() requests arrives after the rows), four
// independent accumulator chains.  (Every lane loads: with the lanes of missing rows masked off 60 nodes x 4096 5.4 -> 5.7 us.)
template <int NS, typename F>
__device__ __forceinline__ f32x4 gram_tile_deep(const uint16_t* row, int k0, int g, F&& side) {
  Frag8 f[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) f[s].u = *(const uint4*)(row + k0 + 32 * s + 8 * g);
  side();
  f32x4 acc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < NS; ++s) acc[s & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[s].v, f[s].v, acc[s & 3], 0, 0, 0);
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// Rows that do not go through the matrix cores (f32; bf16 of a width that is no multiple of 128): the whole workgroup
// sweeps the row of a once per group of DG other rows and keeps a.x, x.x of each in registers, NT x 16 bytes of every
// row per step.  Bound by the bytes a compute unit has in flight (each node reads all of its relatives' rows): the former
// one-row-per-wave loop had one 4-byte load per lane and row in flight - 235 us for 120 nodes x 16384 logits, 19-22 so (and
// less in parts, see launch_accept).
// Narrow rows would spend their time on the 17 sums over eight waves and two barriers per group: up to NARROW elements (an
// eighth where they are loaded one at a time) a wave takes a group of WG rows by itself.  Two trees of 64 nodes, cold caches,
// with one row per wave, swept by the workgroup, swept by a wave: f32 x 64 6.1, 8.6, 5.6 us; x 512 15.0, 8.5, 5.6; x 1024 25.4, 8.2,
// 6.3; bf16 x 72 6.4, 8.9, 6.4; x 1016 7.1, 8.5, 6.6.  Wider rows: f32 x 2048 37.0, 6.6; bf16 x 1976 the wave is slower in small trees
// (40 nodes: 6.6 and 7.4).
constexpr int DG = 8, WG = 4, NARROW = 1024;
template <typename T> struct Piece;   // 16 bytes of a row, or one element of rows that are not 16-byte aligned
template <> struct Piece<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void get(const float* p, float (&x)[N]) { const float4 v = *(const float4*)p; x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w; }
};
template <> struct Piece<uint16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void get(const uint16_t* p, float (&x)[N]) {
    const uint4 v = *(const uint4*)p;
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) { x[2 * i] = __uint_as_float(w[i] << 16); x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u); }
  }
};
// sums over this thread's share of elements h0 .. h - 1 of the row (NT threads): s[2 j] = a.x_j, s[2 j + 1] = x_j.x_j, s[2 G] = a.a
template <int G, int NT, typename T>
__device__ __forceinline__ void dot_group(const T* a, const T* const (&x)[G], int h0, int h, bool aligned, int tid, float (&s)[2 * G + 1]) {
  constexpr int N = Piece<T>::N;
#pragma unroll
  for (int j = 0; j < 2 * G + 1; ++j) s[j] = 0.f;
  if (aligned) {
#pragma unroll 2
    for (int k = h0 + tid * N; k < h; k += NT * N) {   // h0 and h are multiples of N
      float av[N], xv[G][N];
      Piece<T>::get(a + k, av);
#pragma unroll
      for (int j = 0; j < G; ++j) Piece<T>::get(x[j] + k, xv[j]);
#pragma unroll
      for (int c = 0; c < N; ++c) {
        s[2 * G] = fmaf(av[c], av[c], s[2 * G]);
#pragma unroll
        for (int j = 0; j < G; ++j) { s[2 * j] = fmaf(av[c], xv[j][c], s[2 * j]); s[2 * j + 1] = fmaf(xv[j][c], xv[j][c], s[2 * j + 1]); }
      }
    }
  } else {
    for (int k = h0 + tid; k < h; k += NT) {
      const float av = load_f32(a + k);
      s[2 * G] = fmaf(av, av, s[2 * G]);
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const float xv = load_f32(x[j] + k);
        s[2 * j] = fmaf(av, xv, s[2 * j]);
        s[2 * j + 1] = fmaf(xv, xv, s[2 * j + 1]);
      }
    }
  }
}

constexpr int MAXO = 2 * MAXW;   // others of a node: parent + (siblings - 1) + children <= 1 + 63 + 64
static_assert(MAXO + 1 == ACCEPT_SUMS, "the workspace is sized for these");

constexpr unsigned CU_LDS = 160 << 10;   // of a compute unit, in bytes

// Where the workgroups of one node meet (wide rows): a counter that is zero between calls, and the partial sums.
struct AcceptShare {
  int* arrived;                 // [nodes]
  unsigned long long* sums;     // [nodes][parts][MAXO + 1]: a.x and x.x of every other row, a.a
};

// How a node's row is taken against the others: by the workgroup on the vector ALU, by single waves, or in Gram tiles (bf16 rows of a multiple of
// 128; of 4096: the whole part of a wave in flight at once).  Kernels of their own: the less code stands in one, the sooner a cold launch is through it.
enum AcceptRows { ROWS_SWEPT, ROWS_NARROW, ROWS_TILES, ROWS_TILES_4096 };

template <typename T, int NT, AcceptRows HOW>   // NT threads; the Gram tiles of bf16 rows are laid out for 256
__global__ __launch_bounds__(NT) void accept_node_kernel(accept_args a, AcceptShare share, int* dev_status) {
  constexpr int NWV = NT / 64;
  __shared__ float gq[NWV][256];        // the waves' partial Gram tiles over their parts of K; generic path: their partial sums
  __shared__ float s_cos[MAXO];         // cos(a, other)
  __shared__ int s_other[MAXO];         // node index of every other row: parent, siblings (without a), children
  __shared__ int s_stok[MAXW], s_ctok[MAXW];   // tokens of the siblings (by rank, a included) and of the children
  __shared__ int s_sib[MAXW], s_chl[MAXW];     // node indices of the siblings (by rank, a included) and of the children
  __shared__ float s_sq[MAXW], s_cq[MAXW];     // their probabilities under the parent's distribution
  __shared__ int s_ks, s_kc, s_rank;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.z, node = blockIdx.y, n_grid = gridDim.y;
  const int lo = a.node_off[b], Tn = a.node_off[b + 1] - lo;
  if (node == 0 && Tn > n_grid) {
    // the launch was sized for smaller trees: the nodes beyond it are flagged and written as zeros
    if (tid == 0) atomicOr(dev_status, CASCADE_FLAG_TREE_SIZE);
    for (int j = n_grid + tid; j < Tn && lo + j < a.n_nodes_total; j += NT) {
      a.q_tok[lo + j] = 0.f; a.m_int[lo + j] = 0.f; a.cos_parent[lo + j] = 0.f; a.n_int[lo + j] = 0;
      a.m_conv[lo + j] = 0.f; a.n_conv[lo + j] = 0;
    }
  }
  if (node >= Tn) return;
  const int64_t gi = lo + node;
  // wave 0 scans the tree for siblings and children, SCAN chunks of 64 nodes per round trip; the first
  // SCAN chunks (parents and tokens) are requested here, before anything waits for this node's own parent
  // pointer
  constexpr int SCAN = 4;
  int pj0[SCAN], tk0[SCAN];
  auto request_chunks = [&](int base) {
#pragma unroll
    for (int c = 0; c < SCAN; ++c) {
      const int j = base + 64 * c + lane;
      pj0[c] = j < Tn ? a.parent[lo + j] : -2;
      tk0[c] = j < Tn ? a.token[lo + j] : -1;
    }
  };
  if (wave == 0) request_chunks(0);
  const int par = a.parent[gi];
  auto write_zero = [&]() {
    if (tid == 0) {
      a.q_tok[gi] = 0.f; a.m_int[gi] = 0.f; a.cos_parent[gi] = 0.f; a.n_int[gi] = 0;
      a.m_conv[gi] = 0.f; a.n_conv[gi] = 0;
    }
  };
  if (node == 0 || par < 0 || par >= node) {   // roots, and nodes whose parent pointer is unusable
    if (tid == 0 && (node > 0 || par != -1)) atomicOr(dev_status, CASCADE_FLAG_PARENT);
    write_zero();
    return;
  }
  const int h = a.hidden;
  const T* H = (const T*)a.h_cond;
  const float* Lp = a.logits + (int64_t)(lo + par) * a.vocab;
  const float thr = a.row_thr[lo + par], lse = a.row_lse[lo + par];

  if (wave == 0) {   // siblings (children of par, in index order, a included) and children of a
    int ks = 0, kc = 0, rank = -1;
    for (int base = 0; base < Tn; base += 64 * SCAN) {
      if (base > 0) request_chunks(base);
#pragma unroll
      for (int c = 0; c < SCAN; ++c) {
        if (base + 64 * c >= Tn) break;
        const int j = base + 64 * c + lane;
        const int pj = pj0[c], tk = tk0[c];
        const bool sib = pj == par && j > par;
        const unsigned long long sm = __ballot(sib);
        if (sib) {
          const int r = ks + __popcll(sm & ((1ull << lane) - 1ull));
          if (r < MAXW) {
            s_sib[r] = j;
            s_stok[r] = tk;
            // other index: parent is 0; siblings keep their rank order with a left out
            if (j != node) s_other[1 + r - (j > node ? 1 : 0)] = j;
          }
          if (j == node) rank = r;
        }
        ks += __popcll(sm);
        const bool ch = pj == node && j > node;
        const unsigned long long cm = __ballot(ch);
        if (ch) {
          const int r = kc + __popcll(cm & ((1ull << lane) - 1ull));
          if (r < MAXW) { s_chl[r] = j; s_ctok[r] = tk; }
        }
        kc += __popcll(cm);
      }
    }
    rank = wave_max_i(rank);
    if (ks > MAXW || kc > MAXW) {
      if (lane == 0) atomicOr(dev_status, CASCADE_FLAG_WIDTH);
      ks = min(ks, MAXW);
      kc = min(kc, MAXW);
    }
    if (lane == 0) { s_ks = ks; s_kc = kc; s_rank = rank; s_other[0] = par; }
  }
  __syncthreads();
  const int ks = s_ks, kc = s_kc, rank = s_rank;
  if (rank < 0 || rank >= MAXW) {   // beyond the width limit (flagged above): not verified
    write_zero();
    return;
  }
  const int n_sib = ks - 1;              // siblings without a
  const int n_other = 1 + n_sib + kc;
  if (tid < kc) s_other[1 + n_sib + tid] = s_chl[tid];   // the children come after the siblings
  __syncthreads();

  // tokens of the siblings (threads 0 .. ks-1) and of the children (threads 64 .. 64+kc-1), left in LDS by
  // the scan; their probabilities under the parent's distribution are gathered while the feature rows are in flight
  const bool own_sib = tid < ks, own_ch = tid >= 64 && tid < 64 + kc;
  int my_tok = -1;
  if (own_sib) my_tok = s_stok[tid];
  else if (own_ch) my_tok = s_ctok[tid - 64];
  float my_q = 0.f, my_logit = -INFINITY;
  const bool q_wanted = (own_sib || own_ch) && my_tok >= 0 && my_tok < a.vocab;
  auto request_q = [&]() {   // the load only; its value is turned into a probability later
    if (q_wanted) my_logit = Lp[my_tok];
  };
  auto finish_q = [&]() { my_q = (q_wanted && my_logit >= thr) ? __expf(my_logit - lse) : 0.f; };
  auto gather_q = [&]() { request_q(); finish_q(); };

  const T* row_a = H + (int64_t)gi * h;
  if constexpr (HOW >= ROWS_TILES) {
    const int l16 = lane & 15, g = lane >> 4;
    const int kq = h / NWV;   // a multiple of 32
    for (int blk = 0; blk * 15 < n_other; ++blk) {
      // tile rows: 0 = a, 1..15 = others 15 blk .. 15 blk + 14 (clamped: extra rows repeat the last one)
      const int o = 15 * blk + l16 - 1;
      const uint16_t* ra = l16 == 0 ? (const uint16_t*)row_a
                                    : (const uint16_t*)(H + (int64_t)(lo + s_other[min(o, n_other - 1)]) * h);
      f32x4 acc;
      if constexpr (HOW == ROWS_TILES_4096) {   // the wave's whole part in flight at once
        acc = gram_tile_deep<128 / NWV>(ra, wave * kq, g, [&]() { if (blk == 0) request_q(); });
      } else {
        if (blk == 0) request_q();
        acc = gram_tile(ra, l16 == 0 || o < n_other, wave * kq, (wave + 1) * kq, g);
      }
      if (blk == 0) finish_q();
      if (blk > 0) __syncthreads();   // the previous block's partial tiles have been consumed
#pragma unroll
      for (int r = 0; r < 4; ++r) gq[wave][(4 * g + r) * 16 + l16] = acc[r];
      __syncthreads();
      if (tid >= 1 && tid < 16 && 15 * blk + tid - 1 < n_other) {
        // row 0 of the tile: a . x_j ; diagonal: |x_j|^2 ; entry (0, 0): |a|^2
        const int j = tid;
        float ax = gq[0][j], xx = gq[0][17 * j], aa = gq[0][0];
#pragma unroll
        for (int w = 1; w < NWV; ++w) { ax += gq[w][j]; xx += gq[w][17 * j]; aa += gq[w][0]; }
        s_cos[15 * blk + j - 1] = cos_from(ax, aa, xx);
      }
    }
  }
  if constexpr (HOW < ROWS_TILES) {
    gather_q();
    const bool aligned = (h * sizeof(T)) % 16 == 0 && ((uintptr_t)H & 15) == 0;
    if constexpr (HOW == ROWS_NARROW) {
      for (int o0 = WG * wave; o0 < n_other; o0 += NT / 64 * WG) {
        const T* x[WG];
#pragma unroll
        for (int j = 0; j < WG; ++j)   // past the end: the last one again
          x[j] = H + (int64_t)(lo + __builtin_amdgcn_readfirstlane(s_other[min(o0 + j, n_other - 1)])) * h;
        float s[2 * WG + 1];
        dot_group<WG, 64>(row_a, x, 0, h, aligned, lane, s);
        const float aa = wave_sum(s[2 * WG]);
#pragma unroll
        for (int j = 0; j < WG; ++j) {
          const float ax = wave_sum(s[2 * j]), xx = wave_sum(s[2 * j + 1]);
          if (lane == j && o0 + j < n_other) s_cos[o0 + j] = cos_from(ax, aa, xx);
        }
      }
    } else {
      float* part = &gq[0][0];   // [NWV waves][2 DG + 1]
      static_assert(NWV * (2 * DG + 1) <= NWV * 256, "partial sums fit");
      // Wide rows: gridDim.x workgroups, dealt to different XCDs, take the same part of every node's elements, leave their sums in memory that all XCDs see
      // (agent-scope accesses go past their L2s) and count themselves in; the one that arrives last adds the parts up in their
      // order and goes on, the others are done.  No workgroup ever waits for another.  A node whose relatives fit one sweep of rows
      // below 16384 elements saves less than the meeting takes: one of its workgroups does it alone (15 and 40 nodes x 8192 floats,
      // no family of more than eight: 6.9 and 7.4 us, 7.7 and 7.8 with a meeting).
      const int launched = gridDim.x;
      const bool alone = n_other <= DG && h < 16384;
      if (alone && (int)blockIdx.x != (node * launched >> 3) % launched) return;   // (the one: spread over the XCDs)
      const int parts = alone ? 1 : launched, width = ((h + parts - 1) / parts + 63) & ~63;
      const int h0 = alone ? 0 : min((int)blockIdx.x * width, h), h1 = min(h0 + width, h);
      unsigned long long* const shared = share.sums + (gi * parts + blockIdx.x) * (MAXO + 1);
      auto pair = [](float x, float y) { return (unsigned long long)__float_as_uint(x) | ((unsigned long long)__float_as_uint(y) << 32); };
      auto group = [&](int o0, auto size) {   // others o0 .. o0 + G - 1
        constexpr int G = decltype(size)::value;
        const T* x[G];
#pragma unroll
        for (int j = 0; j < G; ++j)   // past the end: the last one again
          x[j] = H + (int64_t)(lo + __builtin_amdgcn_readfirstlane(s_other[min(o0 + j, n_other - 1)])) * h;
        float s[2 * G + 1];
        dot_group<G, NT>(row_a, x, h0, h1, aligned, tid, s);
        if (o0 > 0) __syncthreads();   // the previous group's sums have been consumed
#pragma unroll
        for (int j = 0; j < 2 * G + 1; ++j) s[j] = wave_sum(s[j]);
        if (lane == 0)
#pragma unroll
          for (int j = 0; j < 2 * G + 1; ++j) part[wave * (2 * G + 1) + j] = s[j];
        __syncthreads();
        if (tid < G && o0 + tid < n_other) {
          float ax = 0.f, xx = 0.f, aa = 0.f;
          for (int w = 0; w < NWV; ++w) {
            const float* q = part + w * (2 * G + 1);
            ax += q[2 * tid];
            xx += q[2 * tid + 1];
            aa += q[2 * G];
          }
          if (parts == 1) s_cos[o0 + tid] = cos_from(ax, aa, xx);
          else {
            __hip_atomic_store(shared + o0 + tid, pair(ax, xx), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (o0 + tid == 0) __hip_atomic_store(shared + MAXO, pair(aa, 0.f), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      };
      // A last group of up to four others reads four rows, not eight: one tree of 60 nodes x 16384 floats 10.2 -> 9.2 us, of 100 x 30016 14.2 -> 12.4,
      // four of 60 x 8192 14.3 -> 13.0.
      for (int o0 = 0; o0 < n_other; o0 += DG) {
        if (n_other - o0 <= DG / 2) group(o0, std::integral_constant<int, DG / 2>{});   // (the last one)
        else group(o0, std::integral_constant<int, DG>{});
      }
      if (parts > 1) {
        __shared__ int s_before;
        if (wave == 0) {   // the wave that stored the sums
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          if (lane == 0) s_before = __hip_atomic_fetch_add(share.arrived + gi, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (s_before != parts - 1) return;
        if (tid == 0) __hip_atomic_store(share.arrived + gi, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next call
        if (tid < n_other) {
          float ax = 0.f, xx = 0.f, aa = 0.f;
          for (int q = 0; q < parts; ++q) {
            const unsigned long long* from = share.sums + (gi * parts + q) * (MAXO + 1);
            const unsigned long long v = __hip_atomic_load(from + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            aa += __uint_as_float((unsigned)__hip_atomic_load(from + MAXO, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            ax += __uint_as_float((unsigned)v);
            xx += __uint_as_float((unsigned)(v >> 32));
          }
          s_cos[tid] = cos_from(ax, aa, xx);
        }
      }
    }
  }
  if (own_sib) { s_stok[tid] = my_tok; s_sq[tid] = my_q; }
  else if (own_ch) { s_ctok[tid - 64] = my_tok; s_cq[tid - 64] = my_q; }
  __syncthreads();

  if (wave == 0) {
    const int ta = s_stok[rank];
    const bool tok_ok = ta >= 0 && ta < a.vocab;
    // I_a among the siblings, by rank (lane = rank)
    bool member = false;
    int tj = -1;
    if (lane < ks && lane != rank) {
      tj = s_stok[lane];
      member = s_cos[1 + lane - (lane > rank ? 1 : 0)] >= a.tau_pos;
    }
    const unsigned long long imask = __ballot(member);
    float mi = 0.f;
    if (member && tj != ta && tj >= 0 && tj < a.vocab) {
      bool dup = false;
      for (unsigned long long m = imask & ((1ull << lane) - 1ull); m; m &= m - 1) dup |= (s_stok[__ffsll((long long)m) - 1] == tj);
      if (!dup) mi = s_sq[lane];
    }
    mi = wave_sum(mi);
    // C_a among the children (lane = child rank)
    bool conv = false;
    int tc = -1;
    if (lane < kc) {
      tc = s_ctok[lane];
      conv = s_cos[1 + n_sib + lane] >= a.tau_seq;
    }
    const unsigned long long cmask = __ballot(conv);
    float mc = 0.f;
    if (conv && tc != ta && tc >= 0 && tc < a.vocab) {
      bool dup = false;
      for (unsigned long long m = imask; m; m &= m - 1) dup |= (s_stok[__ffsll((long long)m) - 1] == tc);
      for (unsigned long long m = cmask & ((1ull << lane) - 1ull); m; m &= m - 1) dup |= (s_ctok[__ffsll((long long)m) - 1] == tc);
      if (!dup) mc = s_cq[lane];
    }
    mc = wave_sum(mc);
    if (lane == 0) {
      if (!tok_ok) atomicOr(dev_status, CASCADE_FLAG_TOKEN);
      a.q_tok[gi] = tok_ok ? s_sq[rank] : 0.f;
      a.m_int[gi] = mi;
      a.n_int[gi] = __popcll(imask);
      a.m_conv[gi] = mc;
      a.n_conv[gi] = __popcll(cmask);
      a.cos_parent[gi] = s_cos[0];
    }
  }
}

}  // namespace

hipError_t launch_accept(cascade_ctx* ctx, const accept_args* a) {
  KernelTimer t(ctx, CASCADE_K_ACCEPT);
  dim3 grid(1, ctx->lim.max_nodes_per_tree, a->n_prompts);
  const bool bf16 = a->h_dtype == CASCADE_BF16, mfma = bf16 && a->hidden % 128 == 0;
  const bool aligned = (a->hidden * (bf16 ? 2 : 4)) % 16 == 0 && ((uintptr_t)a->h_cond & 15) == 0;
  const bool narrow = !mfma && a->hidden <= (aligned ? NARROW : NARROW / 8);
  // Wide rows that the vector ALU sweeps: a node with many relatives reads 20 of them and more, through one compute unit.  Parts of
  // at least 8 KiB of rows of 8192 elements and more (16 KiB from 16384 floats on), two workgroups per compute unit (what its
  // registers hold), and 2, 4 or 8 of them, so that an XCD holds one part of every row.  f32, one tree: 60 nodes x 4096 8.5 us
  // whole, 8.8 in two parts; 60 x 8192 11.3 whole, 10.9 in two, 10.0 in four; 60 x 16384 16.5 whole, 11.0 in four, 11.9 in
  // eight; 120 x 16384 16.3 whole, 11.6-12.0 in four; 80 x 33088 26.6, 14.3 in four, 15.1 in six; 96 x 65536 44.4 whole, 20.7 in four, 24.8 in five.
  AcceptShare share = {(int*)ctx->accept_ws, (unsigned long long*)ctx->accept_sums};
  int parts = 1;
  if (!mfma && !narrow) {
    const int by_bytes = (int64_t)a->hidden * (bf16 ? 2 : 4) / 8192, by_room = ACCEPT_PER_CU * ctx->n_cu / a->n_nodes_total;
    const int by_width = a->hidden < 8192 ? 1 : (a->hidden < 32768 ? 4 : 8);
    while (2 * parts <= by_width && 2 * parts <= by_bytes && 2 * parts <= by_room) parts *= 2;
    if (parts > 1 && recorded(ctx->stream)) parts = 1;
  }
  grid.x = parts;
  // Rows of 4096, up to two nodes per compute unit: LDS is set aside so that two workgroups fit on one and no third, although the registers would
  // hold three; the nodes then spread over the whole chip, where three on one unit end last.  Only where all workgroups of the launch
  // could be resident at three per unit, those of nodes that a tree does not have included: more of them wait for places that are fewer so.
  // Rows cold, registers' limit and so, us, means over eight sets of ragged trees of at most 512 nodes: 8 prompts x 40-80 nodes 12.4 and 11.6, 12 x 20-56 11.5
  // and 10.7, 16 x 20-40 10.9 and 10.7, 4 x 60-140 12.0 and 11.9 (rows warm 10.7 and 10.6, 10.0 and 9.8, 9.5 and 9.8, 10.7 and 11.2); in contexts for trees
  // twice as large 12 prompts 11.4 and 11.5, 16 prompts 11.2 and 12.6.  Beyond two nodes per unit three at a time hide more of the latency (1024 nodes 17.5, two
  // at a time 17.8).  Other widths, whose kernel the registers let stand six times on a unit, are mostly slower so (2048: 16 x 20-40 8.5 and 9.5, 1536: 496
  // nodes 8.5 and 11.4, 1152: 511 nodes 8.5 and 9.5).
  const bool spread = mfma && a->hidden == 4096 && a->n_nodes_total <= 2 * ctx->n_cu && grid.y * grid.z <= 3u * ctx->n_cu;
  const unsigned apart = spread ? CU_LDS / 3 : 0;   // beside the kernel's own, more than a third
  // (Gram tiles on eight waves: 462 nodes 10.2 -> 12.1 us, 1024 nodes 18 -> 23.6, fewer nodes the same)
#define CASCADE_LAUNCH_ACCEPT(T, NT, HOW) CASCADE_TIMED_LAUNCH(t, (accept_node_kernel<T, NT, HOW>), grid, dim3(NT), apart, ctx->stream, *a, share, ctx->dev_status)
  if (mfma) { if (a->hidden == 4096) CASCADE_LAUNCH_ACCEPT(uint16_t, 256, ROWS_TILES_4096); else CASCADE_LAUNCH_ACCEPT(uint16_t, 256, ROWS_TILES); }
  else if (bf16) { if (narrow) CASCADE_LAUNCH_ACCEPT(uint16_t, 256, ROWS_NARROW); else CASCADE_LAUNCH_ACCEPT(uint16_t, 256, ROWS_SWEPT); }
  else { if (narrow) CASCADE_LAUNCH_ACCEPT(float, 512, ROWS_NARROW); else CASCADE_LAUNCH_ACCEPT(float, 512, ROWS_SWEPT); }
#undef CASCADE_LAUNCH_ACCEPT
  return hipGetLastError();
}
