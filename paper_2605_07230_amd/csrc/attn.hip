// tree_verify_attn kernels for gfx950.
//
// Every node of a row attends the row's prefix KV positions plus its ancestors in the drafted
// tree plus itself (Preliminaries: parallel target pass; tree decoding with a tree mask).
//
// bf16 path: one workgroup = (row, kv head, query super-block, kv split).  K and V tiles (64 keys) are
// both staged row-major ([key][d]) in LDS; the K operand of the score MFMA is read as 16-byte words, the
// V operand of the second MFMA through the transposing LDS read (ds_read_b64_tr_b16), so no tile is ever
// transposed in memory.  Scores are produced TRANSPOSED, S^T = K Q^T, with v_mfma_f32_16x16x32_bf16: a
// lane then owns one query column, so the online-softmax statistics are per-lane scalars and the
// probabilities are already laid out as the B operand of O^T = V^T P^T.  The ancestor mask of the 64
// tree keys of a tile is one 64-bit word per query, built in LDS by climbing parent pointers.  One body
// (ring_body: tiles in an LDS ring filled by LDS-direct loads) serves 64 to 256 query rows per workgroup,
// the smaller ones with the keys split across workgroups where that fills the chip (partials to the
// workspace, a small merge kernel); the smallest steps split the query rows over workgroups instead and
// the keys over waves.  attn_choose chooses by estimated time.
//
// f32 path: one kernel on the f32 matrix instructions, 16 query rows per workgroup, used by the small fp32 configuration.
#include <type_traits>

#include "common.h"

namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

struct AttnParams {
  const int32_t* node_off;
  const int32_t* parent;
  const int32_t* prefix_len;
  const void* q;
  const void* k_tree;
  const void* v_tree;
  const void* k_cache;
  const void* v_cache;
  int64_t sr, sh, sp;
  void* out;
  float* lse;
  float* ws_o;     // [n_split][N*Hq][D]
  float* ws_ml;    // [n_split][N*Hq][2]
  int* dev_status;
  int n_heads, n_kv_heads, group;
  int n_split, n_sb;
  int n_rows_total;  // N * Hq
  int max_tree;      // the host's bound on any row's node count (the grid was sized for it)
  int round_rows;    // rows of the batch that one workgroup per compute unit covers; 0: less than one
  float scale_log2e;
};

// 2^x for x <= 0 or -inf (v_exp_f32; no range handling needed here)
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ------------------------------------------------------------------------------------------ f32
// Workgroup = (16 query rows of one row of the batch, kv head); its NW waves take every NW-th tile of 16 keys and meet in
// LDS.  Both products run on v_mfma_f32_16x16x4_f32 (one value per lane and operand, k = lane / 16 = g):
//   S^T = K Q^T   lane (l16, g) loads 16 bytes at d = 16 ks + 4 g of key / query l16 and feeds element c of both to the
//                 c-th product; the result holds keys 4 g + r of query l16;
//   O^T = V^T P^T product r takes P^T straight from register r of that result, and element c of the 16 bytes of key 4 g + r's
//                 value at d = 64 h + 4 l16: its row l16 stands for that d + c (element loads: d = 16 db + l16).
// Nothing passes through LDS before the merge.  Bound by the trips to memory, one after the other (the row's place; queries, parents and
// the first tile), by the 50 GB/s at which one compute unit receives keys and values that no cache near it holds (8 heads x 271 keys are 139 KB for
// each of 8 units: 2.8 us), and by the tile that some wave has to do alone at the end.  15 nodes x 8 heads x 64, 256 keys: 10.6 us with
// parents staged in LDS behind a barrier, values loaded four bytes at a time and sixteen parts read by every thread of the merge, now 9.7 (a step 28.3 and 26.9);
// 60 nodes, 1000 keys 23.9 and 20.3-20.9, 200 nodes, 320 keys 14.9 and 13.2-14.5.  Two or three tiles of a wave side by side in 8 or 12 waves are
// slower (10.1-10.4, 20.6-22.0).
// DB = 16-wide blocks of head_dim; VEC, VEC_V: queries and keys, and values, can be read 16 bytes at a time (otherwise element by element, values of
// neighbouring lanes side by side: two trees of 60 nodes x 4 heads x 70, 400 keys 29.7 us with four neighbouring elements per lane, 25.5 so; values alone off
// the 16-byte grid, four trees of 60 nodes x 8 heads x 64, 1000 keys 54.5 with element loads for everything, 21.6 so).
template <int DB, int NW, bool VEC, bool VEC_V>
__global__ __launch_bounds__(64 * NW) void attn_f32_kernel(AttnParams p, int n_rows, int D) {
  extern __shared__ __align__(16) float f32_smem[];   // [NW][16 queries][16 DB + 4] partial outputs, [NW][16][2] (m, l)
  __shared__ int s_parent[CASCADE_MAX_TREE];
  constexpr int OP = 16 * DB + 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4, kvh = blockIdx.y, G = p.group;
  // which row of the batch this query block belongs to: the grid counts the blocks of all rows
  int s = -1, lo = 0, T = 0, P = 0, sb = blockIdx.x;
  for (int base = 0; base < n_rows && s < 0; base += 64) {
    const int r = base + lane;
    const int lo_l = r < n_rows ? p.node_off[r] : 0, t_l = r < n_rows ? p.node_off[r + 1] - lo_l : 0;
    const int p_l = r < n_rows ? p.prefix_len[r] : 0;
    const int nb = (t_l * G + 15) / 16, incl = wave_scan_incl_i(nb);
    const unsigned long long hit = __ballot(sb < incl);
    if (hit) {
      const int l = __ffsll((long long)hit) - 1;
      s = base + l;
      lo = __builtin_amdgcn_readlane(lo_l, l);
      T = __builtin_amdgcn_readlane(t_l, l);
      P = __builtin_amdgcn_readlane(p_l, l);
      sb -= __builtin_amdgcn_readlane(incl - nb, l);
    } else {
      sb -= __builtin_amdgcn_readlane(incl, 63);
    }
  }
  if (s < 0) return;   // the grid is an upper bound of the number of blocks
  const int M = T * G;
  const int qr = min(16 * sb + l16, M - 1);   // rows past the end repeat the last one, never stored
  const int qh = G == 1 ? 0 : qr / T, qi = qr - qh * T;
  const int64_t q_row = (int64_t)(lo + qi) * p.n_heads + kvh * G + qh;
  const int n_pt = (P + 15) / 16, nt = n_pt + (T + 15) / 16;
  auto load4 = [&](const float* row, int d) {
    if (VEC) return d < D ? *(const f32x4*)(row + d) : f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 x;
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = d + c < D ? row[d + c] : 0.f;
    return x;
  };
  const float* kc = (const float*)p.k_cache + s * p.sr + kvh * p.sh;
  const float* vc = (const float*)p.v_cache + s * p.sr + kvh * p.sh;
  const float* ktr = (const float*)p.k_tree + ((int64_t)lo * p.n_kv_heads + kvh) * D;
  const float* vtr = (const float*)p.v_tree + ((int64_t)lo * p.n_kv_heads + kvh) * D;
  const int64_t tree_pitch = (int64_t)p.n_kv_heads * D;
  // tile registers; keys past the end of the tile's source: clamped, masked below
  static_assert(VEC || !VEC_V, "load4 serves both");
  f32x4 q[DB], ot[DB], k[DB], v[4][DB / 4];
  auto request_k = [&](int t) {
    const bool tree = t >= n_pt;
    const int key = min(16 * (tree ? t - n_pt : t) + l16, (tree ? T : P) - 1);
    const float* row = (tree ? ktr : kc) + (int64_t)key * (tree ? tree_pitch : p.sp);
#pragma unroll
    for (int db = 0; db < DB; ++db) k[db] = load4(row, 16 * db + 4 * g);
  };
  auto request_v = [&](int t) {
    const bool tree = t >= n_pt;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = min(16 * (tree ? t - n_pt : t) + 4 * g + r, (tree ? T : P) - 1);
      const float* row = (tree ? vtr : vc) + (int64_t)key * (tree ? tree_pitch : p.sp);
#pragma unroll
      for (int h = 0; h < DB / 4; ++h)
        if (VEC_V) v[r][h] = load4(row, 64 * h + 4 * l16);
        else
#pragma unroll
          for (int c = 0; c < 4; ++c) v[r][h][c] = row[min(64 * h + 16 * c + l16, D - 1)];
    }
  };
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    q[db] = load4((const float*)p.q + q_row * D, 16 * db + 4 * g);
    ot[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // Trees of up to 128 nodes: every wave holds the parents in its lanes (like the query-split kernel), requested together with the
  // queries and the first tiles.  Larger ones are staged, behind a barrier.
  const bool in_lanes = T <= 128;
  int pa[2] = {-1, -1};
  if (in_lanes) {
#pragma unroll
    for (int j = 0; j < 2; ++j) pa[j] = p.parent[lo + min(64 * j + lane, T - 1)];
  }
  const int t0 = __builtin_amdgcn_readfirstlane(wave);
  if (t0 < nt) { request_k(t0); request_v(t0); }
  if (in_lanes) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (64 * j + lane < T && pa[j] >= 64 * j + lane) { atomicOr(p.dev_status, CASCADE_FLAG_PARENT); pa[j] = -1; }   // keeps the climb finite; any negative parent ends it
  } else {
    for (int i = tid; i < T; i += 64 * NW) {
      int pi = p.parent[lo + i];
      if (pi >= i) { atomicOr(p.dev_status, CASCADE_FLAG_PARENT); pi = -1; }
      if (i < CASCADE_MAX_TREE) s_parent[i] = pi;
    }
    __syncthreads();
  }
  // node a's parent: smaller than a, or negative.  Nothing but the array in LDS bounds a tree here; nodes past it read memory.
  auto parent_of = [&](int a) {
    if (a < CASCADE_MAX_TREE) return s_parent[a];
    const int pi = p.parent[lo + a];
    return pi >= a ? -1 : pi;
  };
  // keys of tile t that query l16 sees
  auto seen = [&](int t) {
    if (t < n_pt) {
      const int left = P - 16 * t;
      return left >= 16 ? 0xffffu : (1u << left) - 1u;
    }
    const int kb = 16 * (t - n_pt);
    unsigned bits = 0;
    int a = qi, steps = 0;
    // the node and its MAX_DEPTH nearest ancestors; a longer path is flagged
    if (in_lanes) {
      while (__any(a >= kb)) {   // kb >= 0
        if (a >= kb && ++steps > CASCADE_MAX_DEPTH + 1) { atomicOr(p.dev_status, CASCADE_FLAG_DEPTH); a = -1; }
        if (a >= kb && a - kb < 16) bits |= 1u << (a - kb);
        int up = __builtin_amdgcn_ds_bpermute(4 * (a & 63), pa[0]);
        if (T > 64) {
          const int hi = __builtin_amdgcn_ds_bpermute(4 * (a & 63), pa[1]);
          up = a >= 64 ? hi : up;
        }
        a = a >= kb ? up : a;
      }
    } else {
      while (a >= kb) {
        if (++steps > CASCADE_MAX_DEPTH + 1) { atomicOr(p.dev_status, CASCADE_FLAG_DEPTH); break; }
        if (a - kb < 16) bits |= 1u << (a - kb);
        a = parent_of(a);
      }
    }
    return bits;
  };
  float m = -INFINITY, l = 0.f;
  auto step = [&](int t, auto more) {   // more: another tile of the wave follows
    constexpr bool MORE = decltype(more)::value;
    const unsigned bits = seen(t);
    f32x4 st = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int c = 0; c < 4; ++c) st = __builtin_amdgcn_mfma_f32_16x16x4f32(k[db][c], q[db][c], st, 0, 0, 0);
    if constexpr (MORE) request_k(t + NW);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      st[r] = ((bits >> (4 * g + r)) & 1u) ? st[r] * p.scale_log2e : -INFINITY;
      mx = fmaxf(mx, st[r]);
    }
    const float m_new = fmaxf(m, rows4_max(mx)), m_use = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = fast_exp2(m - m_use);
    float ls = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      st[r] = fast_exp2(st[r] - m_use);
      ls += st[r];
    }
    l = l * alpha + ls;
    m = m_new;
    // A masked key has probability 0, but 0 x inf and 0 x NaN are NaN: a tile that some query does not see whole is looked
    // through for such values, and if it holds any its keys are added one at a time, to the queries that see them.
    bool whole_keys = true;
    if (__any(bits != 0xffffu)) {
      float z = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int db = 0; db < DB; ++db) z = fmaf(v[r][db / 4][db % 4], 0.f, z);
      whole_keys = !__any(z != 0.f);
    }
#pragma unroll
    for (int db = 0; db < DB; ++db) ot[db] *= alpha;
    if (whole_keys) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) ot[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[r][db / 4][db % 4], st[r], ot[db], 0, 0, 0);
    } else {
      for (int kg = 0; kg < 4; ++kg)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool sees = (bits >> (4 * kg + r)) & 1u;
#pragma unroll
          for (int db = 0; db < DB; ++db) {
            const f32x4 o = __builtin_amdgcn_mfma_f32_16x16x4f32(g == kg ? v[r][db / 4][db % 4] : 0.f, st[r], ot[db], 0, 0, 0);
#pragma unroll
            for (int c = 0; c < 4; ++c) ot[db][c] = sees ? o[c] : ot[db][c];
          }
        }
    }
    if constexpr (MORE) request_v(t + NW);
  };
  int t = t0;
  for (; t + NW < nt; t += NW) step(t, std::true_type{});
  if (t < nt) step(t, std::false_type{});
  // merge: lane (l16, g) holds d = 64 (db / 4) + 16 g + 4 c + db % 4 of query l16 (a value's 16 bytes feed four products; element
  // loads: d = 16 db + 4 g + c)
  l = rows4_sum(l);
  float* mo = f32_smem + (wave * 16 + l16) * OP;
  float* ml = f32_smem + NW * 16 * OP;
#pragma unroll
  for (int h = 0; h < DB / 4; ++h)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (VEC_V) *(f32x4*)(mo + 64 * h + 16 * g + 4 * c) = f32x4{ot[4 * h][c], ot[4 * h + 1][c], ot[4 * h + 2][c], ot[4 * h + 3][c]};
      else *(f32x4*)(mo + 64 * h + 16 * c + 4 * g) = ot[4 * h + c];
    }
  if (g == 0) {
    ml[(wave * 16 + l16) * 2] = m;
    ml[(wave * 16 + l16) * 2 + 1] = l;
  }
  __syncthreads();
  // a wave finishes whole rows: lane w holds the factor of wave w's part
  const int rows = min(16, M - 16 * sb);
  for (int r = __builtin_amdgcn_readfirstlane(wave); r < rows; r += NW) {
    const int row = 16 * sb + r, w = lane & 15;
    const float mw = w < NW ? ml[(w * 16 + r) * 2] : -INFINITY, lw = w < NW ? ml[(w * 16 + r) * 2 + 1] : 0.f;
    const float mm = wave_max(mw), f = fast_exp2(mw - mm);   // a wave without visible keys: 0
    const float ll = wave_sum(lane < NW ? f * lw : 0.f);
    const int64_t rowg = (int64_t)(lo + row % T) * p.n_heads + kvh * G + row / T;
    for (int d = lane; d < D; d += 64) {
      float o = 0.f;
#pragma unroll
      for (int i = 0; i < NW; ++i) o = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), i)), f32_smem[(i * 16 + r) * OP + d], o);
      ((float*)p.out)[rowg * D + d] = o / ll;
    }
    if (lane == 0 && p.lse) p.lse[rowg] = mm * LN2 + logf(ll);
  }
}

// ----------------------------------------------------------------------------------------- bf16
constexpr int KT = 64;  // keys per tile

// Workgroups are dispatched in index order, and with ragged prefixes the rows differ several-fold in
// work: a heavy row that happens to sit at the end of the batch would start when the rest of the grid
// is almost done and finish alone.  Dispatch position z therefore takes the z-th heaviest row
// (keys = prefix + tree nodes; ties by index), computed redundantly by every wave from the two small
// arrays it reads anyway.  Batches of more than 64 rows keep their order.
// Workgroups beyond one per compute unit land beside an earlier one: every second round of p.round_rows rows is taken in
// reverse, so that the heaviest row of a round shares its unit with the lightest of the next.
// The row's first node, node count and prefix length come back with it: the lanes already hold them, so the
// workgroup does not go to memory a second time for three values that the next loads depend on.
struct RowInfo {
  int s, lo, T, P;
};
__device__ __forceinline__ RowInfo row_by_work_rank(const AttnParams& p, int z, int n_rows, int lane) {
  RowInfo ri;
  if (n_rows > 64 || n_rows <= 1) {
    ri.s = z;
    ri.lo = p.node_off[z];
    ri.T = p.node_off[z + 1] - ri.lo;
    ri.P = p.prefix_len[z];
    return ri;
  }
  int lo_l = 0, t_l = 0, p_l = 0, work = -1;
  if (lane < n_rows) {
    lo_l = p.node_off[lane];
    t_l = p.node_off[lane + 1] - lo_l;
    p_l = p.prefix_len[lane];
    work = p_l + t_l;
  }
  int rank = 0;
  for (int r = 0; r < n_rows; ++r) {
    const int wr = __builtin_amdgcn_readlane(work, r);
    rank += (wr > work || (wr == work && r < lane)) ? 1 : 0;
  }
  if (p.round_rows > 0 && ((z / p.round_rows) & 1)) {
    const int first = z / p.round_rows * p.round_rows;
    z = first + min(first + p.round_rows, n_rows) - 1 - z;
  }
  const unsigned long long hit = __ballot(lane < n_rows && rank == z);
  ri.s = hit ? __ffsll((long long)hit) - 1 : z;   // (ranks are a permutation: some lane always hits)
  ri.lo = __builtin_amdgcn_readlane(lo_l, ri.s);
  ri.T = __builtin_amdgcn_readlane(t_l, ri.s);
  ri.P = __builtin_amdgcn_readlane(p_l, ri.s);
  return ri;
}

// Workgroups are dealt round-robin to the 8 XCDs (one L2 each) in launch order: hardware id h runs on
// XCD h % 8.  A unit = the nx workgroups of one (row, kv head).  This renumbering keeps a unit's
// workgroups on one XCD (they meet in one L2) while consecutive units still go to different XCDs, so
// rows with long and short prefixes stay spread over the chip.  Needs a unit count divisible by 8;
// otherwise the launch order is kept.
__device__ __forceinline__ unsigned xcd_local_order(unsigned h, unsigned nx, unsigned n_units) {
  if (n_units & 7u) return h;
  const unsigned x = h & 7u, k = h >> 3;          // XCD, slot inside the XCD
  return ((k / nx) * 8u + x) * nx + k % nx;       // unit (k / nx) * 8 + x, workgroup k % nx of it
}


// A row whose tree has more nodes than the host's bound is not computed (the grid and the LDS arrays
// were sized for the bound): the precondition flag is raised and the row's outputs are still defined -
// zeros and lse = -inf, or empty split partials that the merge kernel turns into the same.  Called by
// every workgroup of such a row; the one with query block 0 of each (kv head, split) does the writing.
template <int D, bool SPLIT>
__device__ __forceinline__ void skip_oversize_row(const AttnParams& p, int lo, int T, int kvh, int sb, int split, int tid, int nthreads) {
  if (sb != 0) return;
  if (tid == 0) atomicOr(p.dev_status, CASCADE_FLAG_TREE_SIZE);
  const int G = p.group;
  const int Tc = min(T, p.n_rows_total / p.n_heads - lo);   // never past the packed arrays
  for (int r = tid; r < Tc * G; r += nthreads) {
    const int64_t rowg = (int64_t)(lo + r / G) * p.n_heads + kvh * G + r % G;
    if (SPLIT) {
      float* wm = p.ws_ml + ((int64_t)split * p.n_rows_total + rowg) * 2;
      wm[0] = -INFINITY;
      wm[1] = 0.f;
    } else {
      uint4* o = (uint4*)((uint16_t*)p.out + rowg * D);
#pragma unroll
      for (int c = 0; c < D / 8; ++c) o[c] = make_uint4(0, 0, 0, 0);
      if (p.lse) p.lse[rowg] = -INFINITY;
    }
  }
}

// two floats -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const bf16x2_t v = __builtin_convertvector(f32x2_t{a, b}, bf16x2_t);
  return *(const uint32_t*)&v;
}

union Frag8 {
  bf16x8 v;
  uint4 u;
  uint2 h[2];
};

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// A wave's own LDS-direct loads have landed when at most the N youngest are outstanding; its LDS writes and
// reads are complete at lgkmcnt(0); then the workgroup barrier, bare (a fenced barrier would wait for every
// outstanding load, i.e. for the whole prefetch ring).
template <int N>
__device__ __forceinline__ void wait_and_sync() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// ---------------------------------------------------------------------- bf16, ring of tiles
// Workgroup = (row, kv head, 16 NQ NW query rows, kv split): NW waves x NQ 16-row query blocks share every
// 64-key K / V tile.  Tiles never pass through registers on their way in: 16-byte LDS-direct loads
// (global_load_lds_dwordx4, M0 = LDS address of the wave's 1 KiB chunk) write them into two rings of NS
// tiles each, NS - 1 tiles ahead of their use; a wave waits only for its own chunks of the tile that is
// needed next (vmcnt), then one bare s_barrier per tile makes everybody's chunks visible and the oldest
// tile's buffer free.  An LDS-direct load puts lane l's 16 bytes at 16 l behind M0, so a tile cannot be
// padded; bank conflicts are avoided by choosing WHICH 16-byte piece of a key row each lane fetches: LDS
// slot q of row r holds piece q ^ swz(r) (K: the 16 keys a score MFMA reads together land in 16 different
// slots; V: the 8 keys x 32 bytes of half a transposing read likewise).
// The loop is software-pipelined inside a wave: the score MFMAs of tile t+1 are issued between the
// exponentials of tile t (matrix cores and vector ALU run side by side), then the PV MFMAs of tile t.
// The running maximum that the exponentials refer to is only moved when a row's maximum has grown by
// more than 2^8 (the result does not depend on the reference, p <= 256 is exact enough in bf16 and far
// from overflow in the float accumulators), so the accumulator rescale is a rarely taken branch.  That holds
// for the 256-row kernel.  The smaller ones move it with every new maximum, whose probability is then exactly 1 and whose
// neighbours round finest; with FINE the exponentials of a tile refer to the tile's own maximum, and its sums and products
// are scaled to the running one in float32 when they are added.  2-norm against float64: 2.08e-3 with FINE at every shape
// measured (1 to 16 rows, 90-4200 keys), 2.14e-3 to 2.25e-3 without, 2.34e-3 in the 256-row kernel.
template <int D>
struct RingGeom {
  static constexpr int RB = 2 * D;        // bytes per key row
  static constexpr int PPR = RB / 16;     // 16-byte pieces per row
  static constexpr int RPC = 1024 / RB;   // rows per 1 KiB chunk (one wave-wide LDS-direct load)
  static constexpr int CPT = KT / RPC;    // chunks per tile
  static constexpr int TILE = KT * RB;    // bytes per K (or V) tile
  // slot swizzles (see above); both depend on the key index modulo 16 only
  __device__ static constexpr int kswz(int key) { return D == 128 ? (key & 15) : ((key >> 1) & 7); }
  __device__ static constexpr int vswz(int key) { return D == 128 ? 2 * (key & 7) : 2 * ((key >> 1) & 3); }
};

constexpr float RESCALE_STEP = 8.f;   // log2 units (256-row kernel)

// Maxima of MFMA results (or -inf).  The IEEE-754-2019 maximum maps to v_maximum3_f32 without the input-quieting
// copies that fmaxf costs in IEEE mode.  It must stay a compiler-visible operation: a vector ALU instruction that
// reads a register too soon after the matrix core was told to write it gets the register's OLD contents, the
// hardware does not interlock that case, and the compiler pads only the instructions it can see - the same
// maximum written as inline assembly read stale registers whenever the scheduler put it right behind its MFMA.
__device__ __forceinline__ float vmax3(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}
__device__ __forceinline__ float vmax2(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float rows4_max_raw(float v) {
  cascade_u32x2 a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = vmax2(__uint_as_float(a.x), __uint_as_float(a.y));
  cascade_u32x2 b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return vmax2(__uint_as_float(b.x), __uint_as_float(b.y));
}

//
// DIRECT = false: keys and values that do not start on a 16-byte boundary, or positions more than 64 MiB apart.  LDS-direct
// loads are counted on for aligned addresses only and take 32-bit offsets inside a tile; ordinary loads with 64-bit addresses
// take any.  They pass through registers and are stored to the same places at the end of the step that requested them.
template <int D, int NS, int NQ, int NW, bool WHOLE, bool FINE, bool DIRECT, bool STREAM>
__device__ __forceinline__ void ring_body(const AttnParams& p) {
  using GM = RingGeom<D>;
  constexpr int NT = 64 * NW, RW = 16 * NQ * NW;
  constexpr int KS = D / 32, DB = D / 16;
  static_assert(!(WHOLE && FINE) && (DIRECT || !STREAM), "the 256-row kernel lets the reference lag; LDS-direct loads stream");
  constexpr int LW = GM::CPT % NW == 0 ? NW : 4;   // waves that load: all, or the first four when the chunks do not divide
  constexpr int CPW = GM::CPT / LW;     // chunks of K (and of V) a loading wave fetches per tile
  constexpr int LPI = 2 * CPW;          // LDS-direct loads a wave issues per iteration
  static_assert(DIRECT || LW == NW, "every wave stores what it has requested");
  static_assert(GM::CPT % LW == 0 && NW >= LW && (NS == 2 || NS == 3), "ring geometry: the loop below is unrolled NS times");
  extern __shared__ __align__(1024) char ring_smem[];
  char* const smem_raw = ring_smem;
  // [K ring: NS tiles][V ring: NS tiles][parent: CASCADE_MAX_TREE ints][ancestor words: 2 x RW]
  int* s_parent = (int*)(smem_raw + 2 * NS * GM::TILE);
  unsigned long long* s_anc = (unsigned long long*)(s_parent + CASCADE_MAX_TREE);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const unsigned nx = gridDim.x, ny = gridDim.y;
  const unsigned lid = xcd_local_order(blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z), nx, ny * gridDim.z);
  const int bx = (int)(lid % nx), kvh = (int)((lid / nx) % ny);
  const RowInfo ri = row_by_work_rank(p, (int)(lid / (nx * ny)), (int)gridDim.z, lane);
  const int s = ri.s, lo = ri.lo, T = ri.T, P = ri.P;
  const int n_split = WHOLE ? 1 : p.n_split;
  const int split = bx % n_split, sb = bx / n_split;
  const int G = p.group;
  const int M = T * G;
  const int row0 = sb * RW;
  if (T > p.max_tree) {
    if (n_split > 1) skip_oversize_row<D, true>(p, lo, T, kvh, sb, split, tid, NT);
    else skip_oversize_row<D, false>(p, lo, T, kvh, sb, split, tid, NT);
    return;
  }
  if (row0 >= M || T > CASCADE_MAX_TREE) return;
  const int n_pt = (P + KT - 1) / KT, n_tt = (T + KT - 1) / KT, nt = n_pt + n_tt;   // nt >= 1: a tree has at least its root
  const int per = WHOLE ? nt : (nt + n_split - 1) / n_split;
  const int t_begin = split * per, t_end = min(nt, t_begin + per);
  if (!WHOLE && t_begin >= t_end) {   // a row with fewer tiles than splits: an empty partial
    for (int r = row0 + tid; r < min(row0 + RW, M); r += NT) {
      float* wm = p.ws_ml + ((int64_t)split * p.n_rows_total + (int64_t)(lo + r % T) * p.n_heads + kvh * G + r / T) * 2;
      wm[0] = -INFINITY;
      wm[1] = 0.f;
    }
    return;
  }

  const char* kc = (const char*)((const uint16_t*)p.k_cache + s * p.sr + kvh * p.sh);
  const char* vc = (const char*)((const uint16_t*)p.v_cache + s * p.sr + kvh * p.sh);
  const char* ktr = (const char*)((const uint16_t*)p.k_tree + ((int64_t)lo * p.n_kv_heads + kvh) * D);
  const char* vtr = (const char*)((const uint16_t*)p.v_tree + ((int64_t)lo * p.n_kv_heads + kvh) * D);
  const unsigned tree_pitch_b = (unsigned)(p.n_kv_heads * D * 2), cache_pitch_b = (unsigned)(p.sp * 2);
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)smem_raw);

  // ---- loader: chunk c = CPW wave + i of a tile; lane -> row c RPC + lane / PPR, LDS slot lane % PPR.
  // Ring stages are numbered by the workgroup's own tile count (tile t lives in stage (t - t_begin) % NS), so
  // that inside the loop, which is unrolled NS times, every LDS address is a per-lane register + a constant.
  int ld_row[CPW];
  unsigned ld_kpiece[CPW], ld_vpiece[CPW], ld_kfull[CPW], ld_vfull[CPW];
#pragma unroll
  for (int i = 0; i < CPW; ++i) {
    const int r = (CPW * wave + i) * GM::RPC + lane / GM::PPR, q = lane % GM::PPR;
    ld_row[i] = r;
    ld_kpiece[i] = 16u * (unsigned)(q ^ GM::kswz(r));
    ld_vpiece[i] = 16u * (unsigned)(q ^ GM::vswz(r));
    ld_kfull[i] = (unsigned)r * cache_pitch_b + ld_kpiece[i];   // offsets inside a whole prefix tile
    ld_vfull[i] = (unsigned)r * cache_pitch_b + ld_vpiece[i];
  }
  // One matrix (K or V) of tile tk into ring stage `stage`.  tk is clamped to the workgroup's last tile (the
  // extra requests keep the per-iteration load count fixed; their data lands in a free stage and is never
  // used); rows past the end of the tile's source are read from its last row (always in bounds; their scores
  // are masked, so the finite clamped values contribute exactly nothing).
  u32x4 held[2][DIRECT ? 1 : CPW];   // (ordinary loads) K and V on their way
  auto store_held = [&](int stage, bool is_v) {
#pragma unroll
    for (int i = 0; i < (DIRECT ? 0 : CPW); ++i)
      *(u32x4*)(smem_raw + (is_v ? NS * GM::TILE : 0) + stage * GM::TILE + (CPW * wave + i) * 1024 + 16 * lane) = held[is_v][i];
  };
  // STREAM: a prefix that one workgroup per (row, kv head) reads, once, is streamed: 16 rows of 100-600 keys 39.6 -> 35.9 us and 3 us
  // off the step behind it, 8 rows 1 us off the step.  With keys in parts (2 rows of 1289 keys) and 256-row workgroups (8 rows of
  // 4200) it changes nothing; prefixes that several query blocks read meet in an L2 and stay with the default policy.  The rule
  // counts on the other layers of a model between two steps: attention alone behind a copy of 1 GiB, 8 rows of 1289 keys, 60 nodes
  // 61 -> 40 us, 16 of 312 keys 40 -> 34; repeated on the same prefixes, which the last-level cache then keeps, 32.6 -> 36 and 26.1 -> 26.5.
  // Instances of their own: chosen at every request it made the others up to 4 % slower (4 rows of 1289 keys, 119 nodes, head_dim 64:
  // 25.3 -> 26.2).
  auto request = [&](int tk, int stage, bool is_v) {
    if (LW < NW && wave >= LW) return;
    const int tc = min(tk, t_end - 1);
    if constexpr (!DIRECT) {
      const bool tree_tile = tc >= n_pt;
      const int kb = tree_tile ? (tc - n_pt) * KT : tc * KT;
      const int lim = (tree_tile ? T : P) - 1 - kb;                 // last valid row of the tile, >= 0
      const int64_t pitch_b = tree_tile ? (int64_t)tree_pitch_b : 2 * p.sp;
      const char* src = (is_v ? (tree_tile ? vtr : vc) : (tree_tile ? ktr : kc)) + (int64_t)kb * pitch_b;
#pragma unroll
      for (int i = 0; i < CPW; ++i) __builtin_memcpy(&held[is_v][i], src + min(ld_row[i], lim) * pitch_b + (is_v ? ld_vpiece[i] : ld_kpiece[i]), 16);
      return;
    }
    const unsigned ldst = lds0 + (is_v ? NS * GM::TILE : 0) + stage * GM::TILE + CPW * wave * 1024;
    if (tc < n_pt && (tc + 1) * KT <= P) {
      // a whole tile of the prefix: nothing to clamp, the per-lane offsets are constants
      const char* src = (is_v ? vc : kc) + (int64_t)tc * KT * cache_pitch_b;
#pragma unroll
      for (int i = 0; i < CPW; ++i) {
        const unsigned l = ldst + i * 1024;
        if (STREAM) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(l), "v"(is_v ? ld_vfull[i] : ld_kfull[i]), "s"(src) : "memory");
        else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(is_v ? ld_vfull[i] : ld_kfull[i]), "s"(src) : "memory");
      }
    } else {
      const bool tree_tile = tc >= n_pt;
      const int kb = tree_tile ? (tc - n_pt) * KT : tc * KT;
      const int lim = (tree_tile ? T : P) - 1 - kb;                 // last valid row of the tile, >= 0
      const unsigned pitch_b = tree_tile ? tree_pitch_b : cache_pitch_b;
      const char* src = (is_v ? (tree_tile ? vtr : vc) : (tree_tile ? ktr : kc)) + (int64_t)kb * pitch_b;
#pragma unroll
      for (int i = 0; i < CPW; ++i) {
        const unsigned voff = (unsigned)min(ld_row[i], lim) * pitch_b + (is_v ? ld_vpiece[i] : ld_kpiece[i]);
        const unsigned l = ldst + i * 1024;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(voff), "s"(src) : "memory");
      }
    }
  };

  // ancestor-or-self words of tree tile tt (tile index in the workgroup's numbering) for the workgroup's query rows
  auto build_mask = [&](int tt) {
    if (tid < RW) {
      const int kbase = (tt - n_pt) * KT;
      const int r = row0 + tid;
      unsigned long long wbits = 0ull;
      if (r < M) {
        int a = r % T, guard = 0;
        while (a >= 0 && guard++ <= CASCADE_MAX_TREE) {
          const int rel = a - kbase;
          if (rel < 0) break;   // ancestors only get smaller
          if (rel < 64) wbits |= 1ull << rel;
          a = s_parent[a];
        }
      }
      s_anc[(tt & 1) * RW + tid] = wbits;
    }
  };

  // ---- prologue: K(t_begin) first, then the steady-state order K(t + NS), V(t + NS - 1) of iterations -NS+1 .. -1
  request(t_begin, 0, false);
  store_held(0, false);
#pragma unroll
  for (int i = 1 - NS; i < 0; ++i) {
    request(t_begin + i + NS, (i + NS) % NS, false);
    store_held((i + NS) % NS, false);
    request(t_begin + i + NS - 1, (i + NS - 1) % NS, true);
    store_held((i + NS - 1) % NS, true);
  }
  if (t_end > n_pt) {
    for (int i = tid; i < T; i += NT) {
      int pi = p.parent[lo + i];
      if (pi >= i || pi < -1 || (i == 0 && pi != -1) || (i > 0 && pi < 0)) {
        atomicOr(p.dev_status, CASCADE_FLAG_PARENT);
        pi = (i == 0) ? -1 : 0;   // keep the climb finite
      }
      s_parent[i] = pi;
    }
  }
  // query fragments (B operand of S^T): lane = (query l16, d group g)
  Frag8 qf[NQ][KS];
  int64_t out_row[NQ];   // index into [N*Hq] or -1
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    const int r = row0 + 16 * (wave + NW * n) + l16;
    const bool ok = r < M;
    const int i = ok ? r % T : 0, hg = ok ? r / T : 0;
    const int64_t rowg = (int64_t)(lo + i) * p.n_heads + kvh * G + hg;
    out_row[n] = ok ? rowg : -1;
    const uint16_t* qp = (const uint16_t*)p.q + rowg * D + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ok) qf[n][ks].u = *(const uint4*)(qp + 32 * ks);
      else qf[n][ks].u = make_uint4(0, 0, 0, 0);
    }
  }
  f32x4 ot[NQ][DB];
  f32x4 lsum[NQ];        // row sums of the (bf16) probabilities, produced by the matrix cores: every entry holds the sum
  float m_ref[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    m_ref[n] = -INFINITY;
    lsum[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int db = 0; db < DB; ++db) ot[n][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  Frag8 ones;            // a V^T fragment of bf16 ones: ones x P^T = the probabilities' row sums
  ones.u = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);

  // ---- LDS read addresses.  K fragment (kt, ks): key 16 kt + l16, pieces of d 32 ks + 8 g: slot (4 ks + g) ^ swz;
  // V operand (db, j): keys 32 j + 4 g + (l16 >> 2) (+ 16), 4 consecutive d at 16 db + 4 (l16 & 3): slot
  // (2 db + ((l16 & 3) >> 1)) ^ swz.  ks and db enter by XOR into a per-lane constant (one register each), the
  // stage, kt and j are compile-time byte offsets.
  const unsigned k_lane = (unsigned)(l16 * GM::RB) + 16u * (unsigned)(g ^ GM::kswz(l16));
  const int vkey = 4 * g + (l16 >> 2);
  const unsigned v_lane = (unsigned)(vkey * GM::RB) + ((16u * (unsigned)((l16 & 3) >> 1)) ^ (16u * (unsigned)GM::vswz(vkey))) + 8u * (unsigned)(l16 & 1);
  static_assert(GM::kswz(0) == GM::kswz(16) && GM::vswz(3) == GM::vswz(19) && GM::vswz(3) == GM::vswz(35), "swizzles have period 16");
  const char* k_addr[KS];
  const char* v_addr[DB];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) k_addr[ks] = smem_raw + (k_lane ^ (unsigned)(64 * ks));
#pragma unroll
  for (int db = 0; db < DB; ++db) v_addr[db] = smem_raw + NS * GM::TILE + (v_lane ^ (unsigned)(32 * db));

  f32x4 st[NQ][4];   // scores: st[n][kt] holds keys 16 kt + 4 g + c for query l16
  // K fragments of one 16-key sub-tile kt of the tile in K stage `stage` (A operand of S^T = K Q^T)
  auto load_kfrags = [&](Frag8 (&kf)[KS], int stage, int kt) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[ks].u = *(const uint4*)(k_addr[ks] + stage * GM::TILE + 16 * kt * GM::RB);
  };
  auto score_kt = [&](const Frag8 (&kf)[KS], int kt) {
#pragma unroll
    for (int n = 0; n < NQ; ++n) st[n][kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int n = 0; n < NQ; ++n) st[n][kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks].v, qf[n][ks].v, st[n][kt], 0, 0, 0);
  };
  // V operand of step i = (db, j) = (i / 2, i % 2) of the tile in V stage `stage`: keys 32 j + 4 g + {0..3} and
  // 32 j + 16 + 4 g + {0..3} at d = 16 db + l16, fetched by two transposing loads from the row-major tile
  union VFrag { Frag8 f; s16x4 h[2]; };
  auto load_vfrag = [&](VFrag& vf, int stage, int i) {
    const char* vp = v_addr[i >> 1] + stage * GM::TILE + 32 * (i & 1) * GM::RB;
    vf.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(vp));
    vf.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(vp + 16 * GM::RB));
  };
  // largest of a lane's 16 scores of query block n (raw, before the scale)
  auto lane_max = [&](int n) {
    float a = vmax3(st[n][0][0], st[n][0][1], st[n][0][2]);
    a = vmax3(a, st[n][0][3], st[n][1][0]);
    a = vmax3(a, st[n][1][1], st[n][1][2]);
    a = vmax3(a, st[n][1][3], st[n][2][0]);
    a = vmax3(a, st[n][2][1], st[n][2][2]);
    a = vmax3(a, st[n][2][3], st[n][3][0]);
    a = vmax3(a, st[n][3][1], st[n][3][2]);
    return vmax2(a, st[n][3][3]);
  };

  __syncthreads();                    // parent array complete (the compiler's own waits cover its loads)
  if (t_begin >= n_pt) build_mask(t_begin);
  wait_and_sync<LPI * (NS - 1)>();    // K(t_begin) everywhere (and the first mask)
  float lmax[NQ];                     // lane_max of the scores in st (FINE: the row's), for tiles that need no mask
  {
    Frag8 kf[2][KS];
    load_kfrags(kf[0], 0, 0);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      if (kt < 3) load_kfrags(kf[(kt + 1) & 1], 0, kt + 1);
      score_kt(kf[kt & 1], kt);
    }
#pragma unroll
    for (int n = 0; n < NQ; ++n) lmax[n] = FINE ? rows4_max_raw(lane_max(n)) : lane_max(n);
  }

  // One tile.  ST = ring stage of tile t (compile time: the loop below is unrolled NS times).
  auto tile_step = [&](int t, auto st_const) {
    constexpr int ST = decltype(st_const)::value;
    constexpr int ST_K = (ST + 1) % NS;             // stage of K(t+1)
    constexpr int ST_VNEW = (ST + NS - 1) % NS;     // stage V(t + NS - 1) goes to (V(t-1) has been consumed)
    const bool tree_tile = t >= n_pt;
    const int kbase = tree_tile ? (t - n_pt) * KT : t * KT;
    const int rem = (tree_tile ? T : P) - kbase;
    wait_and_sync<LPI * (NS - 2)>();   // K(t+1), V(t) landed everywhere; K(t), V(t-1) free
    request(t + NS, ST, false);
    request(t + NS - 1, ST_VNEW, true);
    if (!DIRECT) __builtin_amdgcn_sched_barrier(0);   // left alone, each load sinks to the store of its value
    Frag8 kf[2][KS];
    load_kfrags(kf[0], ST_K, 0);       // in flight during the reference check
    if (t + 1 < t_end && t + 1 >= n_pt) build_mask(t + 1);   // read after the next barrier

    // ---- masks (tree tiles and the ragged last prefix tile) and the reference of the exponentials
    if (tree_tile || rem < KT) {
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        unsigned long long valid = tree_tile ? s_anc[(t & 1) * RW + 16 * (wave + NW * n) + l16]
                                             : (rem >= 64 ? ~0ull : ((1ull << rem) - 1ull));
        if (out_row[n] < 0) valid = 0ull;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
          const uint32_t nib = (uint32_t)(valid >> (16 * kt + 4 * g));   // this lane's 4 keys of sub-tile kt
#pragma unroll
          for (int c = 0; c < 4; ++c) st[n][kt][c] = ((nib >> c) & 1u) ? st[n][kt][c] : -INFINITY;
        }
        lmax[n] = FINE ? rows4_max_raw(lane_max(n)) : lane_max(n);
      }
    }
    // a lane sees 16 of its row's 64 scores; if none of a wave's lanes exceeds its row's reference by more than
    // the step, no row does, and the reference stays (scale > 0: the maximum commutes with it)
    constexpr float STEP = WHOLE ? RESCALE_STEP : 0.f;
    float m_tile[NQ];
    bool moved = false;
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      m_tile[n] = lmax[n] * p.scale_log2e;   // FINE: the row's in this tile, otherwise this lane's
      moved |= m_tile[n] > m_ref[n] + STEP;   // -inf + 8 = -inf: a first finite score always moves it
    }
    if (__ballot(moved) != 0ull) {
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        const float mx = FINE ? m_tile[n] : rows4_max_raw(lmax[n]) * p.scale_log2e;
        const float m_new = (mx > m_ref[n] + STEP) ? mx : m_ref[n];
        const float use_new = (m_new == -INFINITY) ? 0.f : m_new;
        const float alpha = fast_exp2(m_ref[n] - use_new);   // -inf - finite = -inf -> 0 ; equal -> 1
        lsum[n] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) ot[n][db] *= alpha;
        m_ref[n] = m_new;
      }
    }
    float m_neg[NQ], beta[NQ], ltile[NQ];   // (FINE) 2^(the tile's maximum - the running one); this lane's part of the tile's row sums
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      const float m = FINE ? m_tile[n] : m_ref[n];
      m_neg[n] = (m == -INFINITY) ? 0.f : -m;
      if (FINE) beta[n] = (m == -INFINITY) ? 0.f : fast_exp2(m - m_ref[n]);   // no visible key: nothing to add
      ltile[n] = 0.f;
    }

    // ---- probabilities of tile t and scores of tile t+1.  Sub-tile kt's scores are consumed by the exponentials
    // (and packed as the B operand of the second MFMA) before the MFMAs of tile t+1 overwrite the same registers,
    // so the matrix cores work on sub-tile kt while the vector ALU is busy with sub-tile kt + 1.
    Frag8 pf[NQ][2];
    auto probs_kt = [&](int kt) {
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        float e[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) e[c] = fast_exp2(fmaf(st[n][kt][c], p.scale_log2e, m_neg[n]));   // -inf stays -inf -> 0
        const float sum = (e[0] + e[1]) + (e[2] + e[3]);   // this lane's keys, before they are rounded
        if (FINE) ltile[n] += sum;
        else if (!WHOLE) lsum[n][0] += sum;
        const uint32_t lo2 = pack_bf16x2(e[0], e[1]), hi2 = pack_bf16x2(e[2], e[3]);
        if (kt & 1) { pf[n][kt >> 1].u.z = lo2; pf[n][kt >> 1].u.w = hi2; }
        else { pf[n][kt >> 1].u.x = lo2; pf[n][kt >> 1].u.y = hi2; }
      }
    };
    constexpr int NVS = 2 * DB, VW = 4;   // V steps per tile, steps whose fragments are requested ahead
    VFrag vf[VW];
    probs_kt(0);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      if (kt < 3) load_kfrags(kf[(kt + 1) & 1], ST_K, kt + 1);
      else {
#pragma unroll
        for (int i = 0; i < VW; ++i) load_vfrag(vf[i], ST, i);
        // left to itself the scheduler sinks every V read to just in front of its MFMA (fewer live registers) and
        // the second half of the step then waits out one LDS round trip per pair of MFMAs
        __builtin_amdgcn_sched_barrier(0);
      }
      score_kt(kf[kt & 1], kt);
      if (kt < 3) probs_kt(kt + 1);
    }

    // ---- O^T += V^T P^T, row sums += ones P^T; the vector ALU meanwhile looks at the next tile's scores
#pragma unroll
    for (int n = 0; n < NQ; ++n)
#pragma unroll
      for (int j = 0; j < (WHOLE ? 2 : 0); ++j) lsum[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones.v, pf[n][j].v, lsum[n], 0, 0, 0);
    if (FINE)
#pragma unroll
      for (int n = 0; n < NQ; ++n) lsum[n][0] = fmaf(beta[n], ltile[n], lsum[n][0]);
#pragma unroll
    for (int n = 0; n < NQ; ++n) lmax[n] = lane_max(n);
    f32x4 pv[2][NQ];   // (FINE) the tile's product for this d block and the one before, which is added meanwhile
    auto add_pv = [&](int db) {
#pragma unroll
      for (int n = 0; n < NQ; ++n)
#pragma unroll
        for (int c = 0; c < 4; ++c) ot[n][db][c] = fmaf(beta[n], pv[db & 1][n][c], ot[n][db][c]);
    };
#pragma unroll
    for (int i = 0; i < NVS; ++i) {
      if (FINE && i == 2)   // under the products' cover: nothing else stands between the barrier and the exponentials
#pragma unroll
        for (int n = 0; n < NQ; ++n) lmax[n] = rows4_max_raw(lmax[n]);
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        f32x4& o = FINE ? pv[(i >> 1) & 1][n] : ot[n][i >> 1];
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[i % VW].f.v, pf[n][i & 1].v, FINE && (i & 1) == 0 ? zero : o, 0, 0, 0);
      }
      if (FINE && (i & 1) && i > 1) add_pv((i >> 1) - 1);
      if (i + VW < NVS) load_vfrag(vf[i % VW], ST, i + VW);
      __builtin_amdgcn_sched_barrier(0);   // keeps the read of step i + VW here, VW steps ahead of its use
    }
    if (FINE) add_pv(DB - 1);
    store_held(ST, false);       // K(t) and V(t - 1) are free (see above); complete before the next barrier, which waits for LDS
    store_held(ST_VNEW, true);
  };

  for (int t = t_begin; t < t_end; t += NS) {
    tile_step(t, std::integral_constant<int, 0>{});
    if (t + 1 >= t_end) break;
    tile_step(t + 1, std::integral_constant<int, 1>{});
    if constexpr (NS > 2) {
      if (t + 2 >= t_end) break;
      tile_step(t + 2, std::integral_constant<int, 2>{});
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the clamped extra requests must not outlive the workgroup's LDS

  // epilogue: lane (query l16, g) owns d = 16*db + 4*g + c
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    const float l = WHOLE ? lsum[n][0] : rows4_sum(lsum[n][0]);
    if (out_row[n] < 0) continue;
    if (n_split > 1) {
      float* wo = p.ws_o + ((int64_t)split * p.n_rows_total + out_row[n]) * D;
#pragma unroll
      for (int db = 0; db < DB; ++db) *(f32x4*)(wo + 16 * db + 4 * g) = ot[n][db];
      if (g == 0) {
        float* wm = p.ws_ml + ((int64_t)split * p.n_rows_total + out_row[n]) * 2;
        wm[0] = m_ref[n];
        wm[1] = l;
      }
      continue;
    }
    const float inv = 1.f / l;   // l >= 1: the node's own key is never masked
    uint16_t* o = (uint16_t*)p.out + out_row[n] * D;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      uint2 w;
      w.x = pack_bf16x2(ot[n][db][0] * inv, ot[n][db][1] * inv);
      w.y = pack_bf16x2(ot[n][db][2] * inv, ot[n][db][3] * inv);
      *(uint2*)(o + 16 * db + 4 * g) = w;
    }
    if (g == 0 && p.lse) p.lse[out_row[n]] = m_ref[n] * LN2 + logf(l);
  }
}

template <int D, int NS>
__global__ __launch_bounds__(512, 1) void attn_bf16_ring_kernel(AttnParams p) { ring_body<D, NS, 2, 8, true, false, true, false>(p); }

// 64 (4 waves), 80 (5), 96 (6) or, with two query blocks per wave, 128 rows per workgroup: two workgroups share a compute
// unit (two-deep rings, 64 KiB) and cover each other's waits.  One workgroup as large as the row's tree reads every key once:
// trees of 65 to 80 nodes used to take two 64-row workgroups.  Deeper rings (96, 128 KiB: one workgroup per unit) measured
// the same or slower at every shape.  Against the kernels this replaced, in a step (us): 16 rows of 113-680 keys, 40-80
// nodes: 46 -> 37; 10 rows of 107-1619 keys, 8 kv heads of 4: 54 -> 34; 8 rows of 140-680 keys: 25 -> 22; 2 rows of 4200 keys
// and 256 nodes, keys in four parts: 65 -> 59 with the merge; 2 rows of 1289 keys, four parts: 23 -> 21.
template <int D, int NS, int NQ, int NW, int OCC, bool FINE, bool DIRECT, bool STREAM>
__global__ __launch_bounds__(64 * NW, OCC) void attn_bf16_rows_kernel(AttnParams p) { ring_body<D, NS, NQ, NW, false, FINE, DIRECT, STREAM>(p); }

// ---------------------------------------------------------------------- bf16, few query rows
// When a step has so few (row, kv head) pairs and keys that the chain of tiles of one workgroup is what takes the time,
// the query rows are split instead of the keys: workgroup = (row, kv head, 16 query rows), eight
// waves, wave w owning the 64-key tiles w, w + 8, ... of the whole key range.  A wave keeps its
// tile to itself: K is loaded from global memory directly in MFMA operand order (16-byte pieces of
// one key row per lane), V goes through a wave-private LDS region only to be read back transposed.
// No workgroup barrier inside the tile loop; the eight (m, l, O) partials are merged through LDS at
// the end.  Keys and values are read by every query block of a (row, kv head) - from L2.
// What bounds it is the chain of one wave: lookups, queries, its tile, the merge.  Parents in the lanes of the wave that owns a
// tree tile, no division where heads are not grouped and no barrier before the merge: 2 rows x 312 keys, 60 nodes 11.4 -> 10.4 us.
template <int D>
__global__ __launch_bounds__(512) void attn_bf16_qsplit_kernel(AttnParams p) {
  constexpr int NWV = 8, NT = 512;
  constexpr int KS = D / 32, DB = D / 16, DC = D / 8;
  constexpr int VP = D + 16;           // V row pitch (elements), as in the other kernels
  constexpr int OP = D + 4;            // merge buffer row pitch (floats)
  constexpr int NVC = KT * DC / 64;    // 16-byte pieces of V per lane per tile
  extern __shared__ __align__(16) char smem_raw[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  uint16_t* vt = (uint16_t*)smem_raw + (size_t)wave * KT * VP;                         // this wave's V tile

  // the query blocks of a (row, kv head) share an L2
  const unsigned nx = gridDim.x, ny = gridDim.y;
  const unsigned lid = xcd_local_order(blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z), nx, ny * gridDim.z);
  const int sb = (int)(lid % nx), kvh = (int)((lid / nx) % ny), s = (int)(lid / (nx * ny));
  const int lo = p.node_off[s];
  const int T = p.node_off[s + 1] - lo;
  const int P = p.prefix_len[s];
  const int G = p.group;
  const int M = T * G;
  const int row0 = sb * 16;
  if (T > p.max_tree) { skip_oversize_row<D, false>(p, lo, T, kvh, sb, 0, tid, NT); return; }
  if (row0 >= M || T > 128) return;
  const int n_pt = (P + KT - 1) / KT, n_tt = (T + KT - 1) / KT, nt = n_pt + n_tt;

  const uint16_t* kc = (const uint16_t*)p.k_cache + s * p.sr + kvh * p.sh;
  const uint16_t* vc = (const uint16_t*)p.v_cache + s * p.sr + kvh * p.sh;
  const uint16_t* ktr = (const uint16_t*)p.k_tree + ((int64_t)lo * p.n_kv_heads + kvh) * D;
  const uint16_t* vtr = (const uint16_t*)p.v_tree + ((int64_t)lo * p.n_kv_heads + kvh) * D;
  const int64_t tree_pitch = (int64_t)p.n_kv_heads * D;

  // tile registers: K fragments kf[kt][ks] = key 16 kt + l16, d 32 ks + 8 g .. + 7 ; V pieces c = lane + 64 it
  u32x4 kf[4][KS], vr[NVC];
  auto request_tile = [&](int t) {
    const bool tree_tile = t >= n_pt;
    const int kbase = tree_tile ? (t - n_pt) * KT : t * KT;
    const int klimit = tree_tile ? T : P;
    const uint16_t* ksrc = tree_tile ? ktr : kc;
    const uint16_t* vsrc = tree_tile ? vtr : vc;
    const int64_t pitch = tree_tile ? tree_pitch : p.sp;
    // Keys past the end of the tile's source are read from its last row (clamped: always in bounds)
    // and are NOT zeroed here: their scores are masked to -inf below, so their probabilities are
    // exactly 0 and the clamped (finite) K and V rows contribute nothing.  A select on the loaded
    // value would make the compiler wait for every load right here, before the next one is issued.
    const int last = max(klimit - 1, 0);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      const int key = kbase + 16 * kt + l16;
      const uint16_t* kp = ksrc + (int64_t)min(key, last) * pitch + 8 * g;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[kt][ks] = *(const u32x4*)(kp + 32 * ks);
    }
#pragma unroll
    for (int it = 0; it < NVC; ++it) {
      const int c = lane + 64 * it, key = kbase + c / DC, dc = c % DC;
      vr[it] = *(const u32x4*)(vsrc + (int64_t)min(key, last) * pitch + 8 * dc);
    }
  };
  // The tree tile that this wave owns, if any (there are at most two, in consecutive waves): the wave takes the parents of the
  // whole tree into its lanes and climbs there, so nothing is staged and no barrier stands in front of the tile loop.
  const int t_tree = n_pt + ((wave - n_pt) & (NWV - 1));
  const bool owns_tree = t_tree < nt;
  int pa[2] = {-1, -1};
  if (owns_tree) {
#pragma unroll
    for (int j = 0; j < 2; ++j) pa[j] = p.parent[lo + min(64 * j + lane, T - 1)];
  }

  // the workgroup's 16 query rows (B operand of S^T): lane = (query l16, d group g); rows past the end repeat the last one,
  // masked and never stored
  Frag8 qf[KS];
  const bool q_ok = row0 + l16 < M;
  const int qr = min(row0 + l16, M - 1);
  const int qh = G == 1 ? 0 : qr / T, qi = qr - qh * T;
  const int64_t rowg = (int64_t)(lo + qi) * p.n_heads + kvh * G + qh;
  {
    const uint16_t* qp = (const uint16_t*)p.q + rowg * D + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks].u = *(const uint4*)(qp + 32 * ks);
  }
  // The first tile is requested AFTER the parent and query loads: loads return in order, so the wait
  // for the parents below leaves the tile's loads in flight instead of draining them.
  unsigned long long seen = 0ull;   // keys of the tree tile that query l16 sees: itself and its ancestors
  if (wave < nt) {
    request_tile(wave);
    if (owns_tree) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int i = 64 * j + lane;
        const bool bad = i < T && (i == 0 ? pa[j] != -1 : (pa[j] >= i || pa[j] < 0));
        if (bad) { atomicOr(p.dev_status, CASCADE_FLAG_PARENT); pa[j] = i == 0 ? -1 : 0; }   // keeps the climb finite
      }
      const int kbase = (t_tree - n_pt) * KT;
      int a = q_ok ? qi : -1;
      while (__any(a >= kbase)) {   // kbase >= 0; ancestors only get smaller
        if (a >= kbase && a - kbase < 64) seen |= 1ull << (a - kbase);
        const int at = 4 * (a & 63);
        int up = __builtin_amdgcn_ds_bpermute(at, pa[0]);
        if (T > 64) {
          const int hi = __builtin_amdgcn_ds_bpermute(at, pa[1]);
          up = a >= 64 ? hi : up;
        }
        a = a > 0 ? up : -1;
      }
    }
  }

  f32x4 ot[DB];
  float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
  for (int db = 0; db < DB; ++db) ot[db] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int t = wave; t < nt; t += NWV) {
    const bool tree_tile = t >= n_pt;
    const int kbase = tree_tile ? (t - n_pt) * KT : t * KT;
    const int klimit = tree_tile ? T : P;
    // S^T = K Q^T from the register fragments (K was requested before V and arrives first)
    f32x4 st[4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      st[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        Frag8 a8;
        a8.u = make_uint4(kf[kt][ks][0], kf[kt][ks][1], kf[kt][ks][2], kf[kt][ks][3]);
        st[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a8.v, qf[ks].v, st[kt], 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // V: registers -> this wave's LDS tile (row-major); the previous tile's reads are complete (same wave, in order)
#pragma unroll
    for (int it = 0; it < NVC; ++it) {
      const int c = lane + 64 * it;
      *(u32x4*)(&vt[(c / DC) * VP + 8 * (c % DC)]) = vr[it];
    }
    __builtin_amdgcn_wave_barrier();   // keep the tile's stores ahead of its transposing reads in program order
    if (t + NWV < nt) request_tile(t + NWV);   // next tile of this wave streams in during the softmax

    unsigned long long valid;
    if (tree_tile) {
      valid = seen;   // (the wave's only tree tile)
    } else {
      const int rem = klimit - kbase;
      valid = rem >= 64 ? ~0ull : ((1ull << rem) - 1ull);
    }
    if (!q_ok) valid = 0ull;
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      const uint32_t nib = (uint32_t)(valid >> (16 * kt + 4 * g));   // this lane's 4 keys of sub-tile kt
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float z = ((nib >> c) & 1u) ? st[kt][c] * p.scale_log2e : -INFINITY;
        st[kt][c] = z;
        mx = fmaxf(mx, z);
      }
    }
    mx = rows4_max(mx);
    const float m_new = fmaxf(m_run, mx);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = fast_exp2(m_run - m_use);
    float ls = 0.f;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float e = fast_exp2(st[kt][c] - m_use);
        st[kt][c] = e;
        ls += e;
      }
    l_run = l_run * alpha + ls;
    m_run = m_new;
#pragma unroll
    for (int db = 0; db < DB; ++db) ot[db] *= alpha;
    Frag8 pf[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      pf[j].u.x = pack_bf16x2(st[2 * j][0], st[2 * j][1]);
      pf[j].u.y = pack_bf16x2(st[2 * j][2], st[2 * j][3]);
      pf[j].u.z = pack_bf16x2(st[2 * j + 1][0], st[2 * j + 1][1]);
      pf[j].u.w = pack_bf16x2(st[2 * j + 1][2], st[2 * j + 1][3]);
    }
    // O^T += V^T P^T with transposing reads of the wave's V tile (LDS operations of one wave complete in order)
#pragma unroll
    for (int db = 0; db < DB; ++db) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint16_t* vp = &vt[(32 * j + 4 * g + (l16 >> 2)) * VP + 16 * db + 4 * (l16 & 3)];
        union { Frag8 f; s16x4 h[2]; } vf;
        vf.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(vp));
        vf.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(vp + 16 * VP));
        ot[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf.f.v, pf[j].v, ot[db], 0, 0, 0);
      }
    }
    __builtin_amdgcn_wave_barrier();   // and the reads ahead of the next tile's stores
  }

  // merge the eight waves' partials through LDS (the V tiles are reused)
  l_run = rows4_sum(l_run);
  __syncthreads();
  float* mo = (float*)smem_raw;                 // [NWV][16 rows][OP]
  float* mml = mo + NWV * 16 * OP;              // [NWV][16 rows][2]
  {
    float* orow = mo + (wave * 16 + l16) * OP;
#pragma unroll
    for (int db = 0; db < DB; ++db) *(f32x4*)(orow + 16 * db + 4 * g) = ot[db];
    if (g == 0) {
      mml[(wave * 16 + l16) * 2] = m_run;
      mml[(wave * 16 + l16) * 2 + 1] = l_run;
    }
  }
  __syncthreads();
  {
    constexpr int TPR = NT / 16;                 // threads per output row
    constexpr int DQ = D / TPR;                  // d range of one thread (4 for D = 128, 2 for D = 64)
    const int row = tid / TPR, dq = tid % TPR;
    const int rr = row0 + row;
    if (rr < M) {
      float mw[NWV], m = -INFINITY;
#pragma unroll
      for (int w = 0; w < NWV; ++w) { mw[w] = mml[(w * 16 + row) * 2]; m = fmaxf(m, mw[w]); }
      float l = 0.f, o[DQ];
#pragma unroll
      for (int d = 0; d < DQ; ++d) o[d] = 0.f;
#pragma unroll
      for (int w = 0; w < NWV; ++w) {
        if (mw[w] == -INFINITY) continue;
        const float sc = fast_exp2(mw[w] - m);
        l += sc * mml[(w * 16 + row) * 2 + 1];
        const float* orow = mo + (w * 16 + row) * OP + DQ * dq;
#pragma unroll
        for (int d = 0; d < DQ; ++d) o[d] += sc * orow[d];
      }
      const int i = rr % T, hg = rr / T;
      const int64_t rg = (int64_t)(lo + i) * p.n_heads + kvh * G + hg;
      const float inv = 1.f / l;
      uint16_t* op = (uint16_t*)p.out + rg * D + DQ * dq;
#pragma unroll
      for (int d = 0; d < DQ; d += 2) *(uint32_t*)(op + d) = pack_bf16x2(o[d] * inv, o[d + 1] * inv);
      if (dq == 0 && p.lse) p.lse[rg] = m * LN2 + logf(l);
    }
  }
}

// log-sum-exp merge of the split partials: D/4 lanes per output row (a float4 each), 256 threads
template <int D>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnParams p) {
  constexpr int LPR = D / 4;             // lanes per row
  constexpr int RPB = 256 / LPR;         // rows per block
  const int64_t row = (int64_t)blockIdx.x * RPB + threadIdx.x / LPR;
  const int d4 = threadIdx.x % LPR;
  if (row >= p.n_rows_total) return;
  float m = -INFINITY;
  for (int c = 0; c < p.n_split; ++c) m = fmaxf(m, p.ws_ml[((int64_t)c * p.n_rows_total + row) * 2]);
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  float l = 0.f;
  for (int c = 0; c < p.n_split; ++c) {
    const float* ml = p.ws_ml + ((int64_t)c * p.n_rows_total + row) * 2;
    const float mc = ml[0];
    if (mc == -INFINITY) continue;
    const float w = exp2f(mc - m);
    l += w * ml[1];
    o += w * *(const f32x4*)(p.ws_o + ((int64_t)c * p.n_rows_total + row) * D + 4 * d4);
  }
  const float inv = l > 0.f ? 1.f / l : 0.f;   // a skipped row (every partial empty) comes out as zeros, lse = -inf
  uint2 packed;
  packed.x = pack_bf16x2(o[0] * inv, o[1] * inv);
  packed.y = pack_bf16x2(o[2] * inv, o[3] * inv);
  *(uint2*)((uint16_t*)p.out + row * D + 4 * d4) = packed;
  if (d4 == 0 && p.lse) p.lse[row] = m * LN2 + logf(l);
}

AttnParams make_params(cascade_ctx* ctx, const tree_attn_args* a) {
  AttnParams p;
  p.node_off = a->node_off;
  p.parent = a->parent;
  p.prefix_len = a->prefix_len;
  p.q = a->q;
  p.k_tree = a->k_tree;
  p.v_tree = a->v_tree;
  p.k_cache = a->k_cache;
  p.v_cache = a->v_cache;
  p.sr = a->cache_stride_row;
  p.sh = a->cache_stride_head;
  p.sp = a->cache_stride_pos;
  p.out = a->out;
  p.lse = a->lse;
  p.ws_o = nullptr;
  p.ws_ml = nullptr;
  p.dev_status = ctx->dev_status;
  p.n_heads = a->n_heads;
  p.n_kv_heads = a->n_kv_heads;
  p.group = a->n_heads / a->n_kv_heads;
  p.n_split = 1;
  p.n_sb = 1;
  p.round_rows = 0;
  p.n_rows_total = a->n_nodes_total * a->n_heads;
  p.max_tree = a->max_nodes_per_tree;
  const float scale = a->scale != 0.f ? a->scale : 1.f / sqrtf((float)a->head_dim);
  p.scale_log2e = scale * LOG2E;
  return p;
}

// whole rows of keys per workgroup (n_split == 1): the ring kernel
template <int D>
hipError_t launch_ring_t(cascade_ctx* ctx, const AttnParams& p, dim3 grid) {
  constexpr int NS = 3;
  const size_t smem = 2 * NS * RingGeom<D>::TILE + CASCADE_MAX_TREE * sizeof(int) + 2 * 256 * sizeof(unsigned long long);
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)attn_bf16_ring_kernel<D, NS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  KernelTimer t(ctx, CASCADE_K_ATTN);
  CASCADE_TIMED_LAUNCH(t, (attn_bf16_ring_kernel<D, NS>), grid, dim3(512), smem, ctx->stream, p);
  return hipGetLastError();
}

}  // namespace

template <int DB, int NW, bool VEC, bool VEC_V>
hipError_t launch_f32_k(cascade_ctx* ctx, const AttnParams& p, dim3 grid, int n_rows, int D) {
  constexpr int smem = (NW * 16 * (16 * DB + 4) + NW * 32) * 4;
  auto kern = attn_f32_kernel<DB, NW, VEC, VEC_V>;
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  KernelTimer t(ctx, CASCADE_K_ATTN);
  CASCADE_TIMED_LAUNCH(t, kern, grid, dim3(64 * NW), smem, ctx->stream, p, n_rows, D);
  return hipGetLastError();
}
template <int DB, int NW>
hipError_t launch_f32_t(cascade_ctx* ctx, const AttnParams& p, dim3 grid, int n_rows, int D, bool vec, bool vec_v) {
  if (vec) return vec_v ? launch_f32_k<DB, NW, true, true>(ctx, p, grid, n_rows, D) : launch_f32_k<DB, NW, true, false>(ctx, p, grid, n_rows, D);
  return launch_f32_k<DB, NW, false, false>(ctx, p, grid, n_rows, D);
}

hipError_t launch_tree_attn_f32(cascade_ctx* ctx, const tree_attn_args* a) {
  AttnParams p = make_params(ctx, a);
  const int D = a->head_dim;
  // blocks of 16 query rows: at most one partly filled one per row of the batch
  dim3 grid((unsigned)((int64_t)a->n_nodes_total * p.group / 16 + a->n_rows), a->n_kv_heads);
  const bool vec = D % 4 == 0 && ((a->cache_stride_row | a->cache_stride_head | a->cache_stride_pos) & 3) == 0 &&
                   (((uintptr_t)a->q | (uintptr_t)a->k_tree | (uintptr_t)a->k_cache) & 15) == 0;
  const bool vec_v = (((uintptr_t)a->v_tree | (uintptr_t)a->v_cache) & 15) == 0;
  if (D <= 64) return launch_f32_t<4, 16>(ctx, p, grid, a->n_rows, D, vec, vec_v);
  if (D <= 128) return launch_f32_t<8, 8>(ctx, p, grid, a->n_rows, D, vec, vec_v);
  return launch_f32_t<16, 4>(ctx, p, grid, a->n_rows, D, vec, vec_v);
}

// 16 NQ NW query rows per workgroup, keys split p.n_split ways (partials, then the merge kernel)
template <int D, int NQ, int NW, int OCC, bool FINE, bool DIRECT, bool STREAM>
hipError_t launch_rows_k(cascade_ctx* ctx, const AttnParams& p, dim3 grid) {
  constexpr int NS = 2, RW = 16 * NQ * NW;
  constexpr int smem = 2 * NS * RingGeom<D>::TILE + CASCADE_MAX_TREE * (int)sizeof(int) + 2 * RW * (int)sizeof(unsigned long long);
  auto kern = attn_bf16_rows_kernel<D, NS, NQ, NW, OCC, FINE, DIRECT, STREAM>;
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  {
    KernelTimer t(ctx, CASCADE_K_ATTN);
    CASCADE_TIMED_LAUNCH(t, kern, grid, dim3(64 * NW), smem, ctx->stream, p);
  }
  if (p.n_split > 1) {
    KernelTimer t(ctx, CASCADE_K_ATTN_MERGE);
    CASCADE_TIMED_LAUNCH(t, (attn_merge_kernel<D>), dim3((p.n_rows_total + (1024 / D) - 1) / (1024 / D)), dim3(256), 0, ctx->stream, p);
  }
  return hipGetLastError();
}
// a prefix that one workgroup reads, once, is streamed (see ring_body)
template <int D, int NQ, int NW, int OCC, bool FINE>
hipError_t launch_rows_t(cascade_ctx* ctx, const AttnParams& p, dim3 grid) {
  return p.n_sb == 1 && p.n_split == 1 ? launch_rows_k<D, NQ, NW, OCC, FINE, true, true>(ctx, p, grid)
                                       : launch_rows_k<D, NQ, NW, OCC, FINE, true, false>(ctx, p, grid);
}

template <int D>
hipError_t launch_qsplit_t(cascade_ctx* ctx, const AttnParams& p, dim3 grid) {
  constexpr int VP = D + 16;
  const size_t smem = (size_t)8 * KT * VP * sizeof(uint16_t);
  static_assert(8 * 16 * (D + 4) * 4 + 8 * 16 * 2 * 4 <= 8 * KT * (D + 16) * 2, "merge buffers fit in the V tiles");
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)attn_bf16_qsplit_kernel<D>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  KernelTimer t(ctx, CASCADE_K_ATTN);
  CASCADE_TIMED_LAUNCH(t, (attn_bf16_qsplit_kernel<D>), grid, dim3(512), smem, ctx->stream, p);
  return hipGetLastError();
}

// How a step's attention can be cut.  Shapes 0-4: query rows per workgroup, and what one 64-key tile costs a workgroup (us
// at head_dim 128, inside a step, i.e. with cold caches): on a mostly idle chip (c0: its chain of waits), with one workgroup
// on every compute unit (c1), with two (c2; c2_hbm when every tile comes from HBM because no other query block shares it:
// the bytes in flight bind).  Shape 5 is the query-split kernel.
struct AttnShape {
  int rows;
  float c0, c1, c2, c2_hbm;
  int per_cu;
};
constexpr int ATTN_N_SHAPES = 6, ATTN_RING = 4, ATTN_QSPLIT = 5;
constexpr AttnShape ATTN_SHAPES[ATTN_N_SHAPES] = {{64, 1.0f, 1.0f, 1.5f, 3.0f, 2}, {80, 1.0f, 1.15f, 1.9f, 3.0f, 2}, {96, 1.0f, 1.2f, 2.1f, 3.0f, 2},
                                                  {128, 1.2f, 1.45f, 2.5f, 2.5f, 2}, {256, 1.7f, 2.3f, 2.3f, 2.3f, 1}, {16, 0.75f, 0.75f, 0.75f, 0.75f, 1}};

// head_dim 64: the tile's cost against that at 128, shape by shape (half the bytes and products, the same exponentials and
// waits).  Fitted, with the fixed part, to every cut of 20 steps (1-16 rows, 90-4200 keys, 16-256 nodes, 1 or 4 heads per kv
// head, cold caches): the cut chosen is 2 % behind the fastest in the mean, 5 % with one factor of 0.65.  2 rows x 1289 keys,
// 60 nodes: query split 16.9 us, 64 rows in four splits 18.9; 4 x 2000 keys, 256 nodes, 8 kv heads of 4: 64 rows 47.0, 128 rows
// 51.6; 2 x 2400 keys, 128 nodes: 64 rows in four splits 28.3, 128 rows in eight 33.4.
constexpr float ATTN_NARROW[ATTN_N_SHAPES] = {0.75f, 0.75f, 0.75f, 0.83f, 0.62f, 0.73f};

// Estimated time of a step's attention, us.  Against measured steps (32 heads, head_dim 128): 2 rows x 312 keys, 60 nodes:
// query split 10.5 (10.3), 64 rows 13.4 (13.4); 2 x 1289 keys: query split 22.5 (23.1), 64 rows whole 29 (29.5) and in four
// splits 19 (20.7); 2 x 4200 keys, 256 nodes: 64 rows 77 (79), 128 rows in four splits 62 (59); 8 such rows: 256 rows
// 168 (167), 128 rows 182 (172); 16 rows of 113-680 keys, 40-80 nodes: 128 rows 37 (37), 80 rows 43 (44); 10 rows of
// 107-1619 keys, 8 kv heads of 4: 64 rows 40 (34), 128 rows in two splits 43 (38).  With cold caches, query split and 64 rows: 8 rows
// of 29 keys, 54 nodes (four rounds) 25.5 and 12.7, at head_dim 64 18.6 and 10.3; 16 x 110 keys, 29 nodes, 8 kv heads of 4 (three)
// 24.7 and 13.7; 64 rows in four, eight and sixteen parts: 2 x 1269 keys, 29 nodes, 8 heads 18.6, 18.4, 21.0.  Over 72 steps
// (1-16 rows, 24-4200 keys, 15-256 nodes) the cut chosen was 2.5 % behind the fastest in the mean when the costs were fitted; over
// 340 others (the same ranges, 32 or 8 kv heads, both head widths, inputs from HBM) it is 4.3 % behind.  At worst: 96 rows in
// several blocks (8 rows x 700 keys, 119 nodes, 8 kv heads of 4: 48.5 us, 64 rows 32.3; x 2400 keys 111 and 68) and 128 rows for
// 16 rows of 60 nodes at head_dim 64 (700 keys: 31.9 us, 64 rows 24.2).
float attn_estimate_us(int shape, const tree_attn_args* a, int group, int n_split, int n_cu) {
  const AttnShape& sh = ATTN_SHAPES[shape];
  const int M = a->max_nodes_per_tree * group, n_sb = (M + sh.rows - 1) / sh.rows;
  const int tiles = (a->max_prefix_len + KT - 1) / KT + (a->max_nodes_per_tree + KT - 1) / KT;
  const bool narrow = a->head_dim == 64;
  const float d = narrow ? ATTN_NARROW[shape] : 1.f;
  // query blocks that hold rows: ragged trees leave some of the launched ones empty
  float blocks = (float)a->n_rows * n_sb;
  if (n_sb > 1) blocks = fminf(blocks, (float)a->n_nodes_total * group / sh.rows + 0.5f * a->n_rows);
  const float x = blocks * a->n_kv_heads * n_split / n_cu;   // workgroups per compute unit
  if (shape == ATTN_QSPLIT) {   // one workgroup fills a compute unit's LDS: whole rounds, each with its own start and merge
    const float chain = tiles * sh.c1 * d;
    return 6.f + chain + (fmaxf(ceilf(x), 1.f) - 1.f) * ((narrow ? 2.7f : 4.f) + chain);
  }
  const float c2 = sh.c2_hbm + (sh.c2 - sh.c2_hbm) * fminf(blocks / a->n_rows - 1.f, 1.f);
  const float per_tile = x <= 1.f ? sh.c0 + (sh.c1 - sh.c0) * x
                       : (sh.per_cu == 1 ? sh.c1 * ceilf(x) : (x <= 2.f ? sh.c1 + (c2 - sh.c1) * (x - 1.f) : c2 * 0.5f * x));
  float us = (narrow ? 9.3f : 7.4f) + (float)((tiles + n_split - 1) / n_split) * per_tile * d;
  if (n_split > 1)   // a second launch, which reads the parts one after the other, and partials written and read (mostly through the caches)
    us += 3.8f + 0.3f * n_split + (float)n_split * a->n_nodes_total * a->n_heads * (a->head_dim + 2) * 4.f / 7e6f;
  return us;
}

// shapes that exist with ordinary loads as well (the query-split kernel has no others)
bool attn_shape_loads_any(int shape) { return shape == 0 || shape == 3 || shape == ATTN_QSPLIT; }

// Whether a tile's exponentials refer to its own maximum (see ring_body).  On a full chip that costs time: it adds 1.2 us to a
// step of 16 rows of 113-680 keys (153 us), 3.2 to one of 10 rows of 107-1619 keys with 8 kv heads of 4 (210), 4.4 to one of
// 2 rows of 4200 keys and 256 nodes in four parts (290).  Fewer workgroups mostly wait (0.5 us of 161 at 2 rows of 1289 keys,
// 0.9 of 94 at 4 rows of 240-560), and one running maximum rounds more coarsely there than the 2 to 16 groups of waves, each
// with a maximum of its own, that such steps' keys were cut into before (2.16e-3 against 2.12e-3 and 2.17e-3 against 2.14e-3
// from float64; 2.08e-3 so).  It is taken there, unless 256-row workgroups that fill the chip would have no more parts.
bool attn_fine(const tree_attn_args* a, int group, int n_split, int n_cu) {
  const long M = (long)a->max_nodes_per_tree * group, heads = (long)a->n_rows * a->n_kv_heads;
  if (M <= 128) return a->head_dim == 64 || heads * ((M + 63) / 64) < 2 * n_cu;
  return n_split < n_cu / (heads * ((M + 255) / 256));
}

template <int D, bool FINE>
hipError_t launch_rows(cascade_ctx* ctx, const AttnParams& p, int shape, dim3 grid) {
  switch (shape) {
    case 0: return launch_rows_t<D, 1, 4, 2, FINE>(ctx, p, grid);
    case 1: return launch_rows_t<D, 1, 5, 3, FINE>(ctx, p, grid);
    case 2: return launch_rows_t<D, 1, 6, 3, FINE>(ctx, p, grid);
    default: return launch_rows_t<D, 2, 4, 2, FINE>(ctx, p, grid);
  }
}

template <int D>
hipError_t launch_bf16_t(cascade_ctx* ctx, const AttnParams& p, int shape, bool fine, bool direct, dim3 grid) {
  if (shape == ATTN_RING) return launch_ring_t<D>(ctx, p, grid);
  if (shape == ATTN_QSPLIT) return launch_qsplit_t<D>(ctx, p, grid);
  if (!direct) return shape == 0 ? launch_rows_k<D, 1, 4, 2, true, false, false>(ctx, p, grid) : launch_rows_k<D, 1, 8, 2, true, false, false>(ctx, p, grid);
  return fine ? launch_rows<D, true>(ctx, p, shape, grid) : launch_rows<D, false>(ctx, p, shape, grid);
}

struct AttnCut {
  int shape, n_split;
  bool fine, direct;
};

AttnCut attn_choose(const tree_attn_args* a, int n_cu, size_t ws_bytes) {
  const int group = a->n_heads / a->n_kv_heads, M = a->max_nodes_per_tree * group;   // query rows per (row, kv head)
  const int n_tiles = (a->max_prefix_len + KT - 1) / KT + (a->max_nodes_per_tree + KT - 1) / KT;
  const size_t per_split = (size_t)a->n_nodes_total * a->n_heads * (a->head_dim + 2) * sizeof(float);
  AttnCut cut = {0, 1, false, true};
  // keys and values are fetched by LDS-direct loads where their addresses allow it (strides are multiples of 16 bytes)
  cut.direct = (((uintptr_t)a->k_tree | (uintptr_t)a->v_tree | (uintptr_t)a->k_cache | (uintptr_t)a->v_cache) & 15) == 0 &&
               a->cache_stride_pos <= (int64_t)1 << 25;
  float best = INFINITY;
  for (int i = 0; i < ATTN_N_SHAPES; ++i) {
    if (!cut.direct && !attn_shape_loads_any(i)) continue;
    if (i == ATTN_QSPLIT && (M > 128 || a->max_nodes_per_tree > 128)) continue;   // its LDS holds trees of 128 nodes
    for (int n = 1; n <= 16 && n <= n_tiles; n = n < 4 ? n + 1 : n * 2) {
      if (n > 1 && (i >= ATTN_RING || per_split * n > ws_bytes)) break;   // these take whole rows of keys
      const float us = attn_estimate_us(i, a, group, n, n_cu);
      if (us < best) { best = us; cut.shape = i; cut.n_split = n; }
    }
  }
  cut.fine = attn_fine(a, group, cut.n_split, n_cu);
  return cut;
}

void plan_tree_attn_bf16(const tree_attn_args* a, int n_cu, size_t ws_bytes, int32_t* query_rows, int32_t* key_parts) {
  const AttnCut cut = attn_choose(a, n_cu, ws_bytes);
  *query_rows = ATTN_SHAPES[cut.shape].rows;
  *key_parts = cut.n_split;
}

hipError_t launch_tree_attn_bf16(cascade_ctx* ctx, const tree_attn_args* a) {
  AttnParams p = make_params(ctx, a);
  const AttnCut cut = attn_choose(a, ctx->n_cu, ctx->attn_ws_bytes);
  p.n_split = cut.n_split;
  p.n_sb = (a->max_nodes_per_tree * p.group + ATTN_SHAPES[cut.shape].rows - 1) / ATTN_SHAPES[cut.shape].rows;
  if (p.n_split > 1) {
    p.ws_o = (float*)ctx->attn_ws;
    p.ws_ml = (float*)(ctx->attn_ws + (size_t)p.n_split * p.n_rows_total * a->head_dim * sizeof(float));
  }
  dim3 grid(p.n_split * p.n_sb, a->n_kv_heads, a->n_rows);
  // rows of the batch that one round of workgroups over the compute units covers (see row_by_work_rank)
  p.round_rows = ctx->n_cu / (int)(grid.x * grid.y);
  return a->head_dim == 128 ? launch_bf16_t<128>(ctx, p, cut.shape, cut.fine, cut.direct, grid)
                            : launch_bf16_t<64>(ctx, p, cut.shape, cut.fine, cut.direct, grid);
}
