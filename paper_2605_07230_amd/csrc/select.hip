// select_path kernel for gfx950: as many workgroups per prompt as its row has passes of 4096 entries, where the chip has room.
//
// SEQUENTIAL (Alg. 2 as printed): wave 0 holds the per-node scalars of the whole tree in registers
// (one node per lane per 64-node chunk).  The children of the current node are found with one
// ballot per chunk, and the serial budget / acceptance arithmetic of the tried children runs on
// values fetched with readlane, so a level costs no memory access at all.
// LONGEST: the same rule along every root-to-leaf path on its own is a top-down recurrence
// (state of a node = f(state of its parent)); it is evaluated level by level in LDS, then the
// best leaf is picked with an integer atomic max.
// Both end with Alg. 1's correction step: inverse CDF over the terminal node's filtered softmax
// with the rejected tokens removed, as per-256-entry chunk sums, a scan over the chunk sums and
// a scan inside the crossing chunk.
#include "common.h"

namespace {

constexpr int MAXCHUNKS = CASCADE_MAX_VOCAB / 256;

__device__ __forceinline__ float readlane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

struct Try {
  bool pass;
  float tvd;
};
// Alg. 2 body for one tried node: budget-gated aggregation (a mass of 0 changes nothing, so the set
// sizes need not be consulted), then Alg. 1's test r * p < q
__device__ __forceinline__ Try try_node(float q, float mi, float mc, float up, float tvd, float eps) {
  if (tvd + mi <= eps) { q += mi; tvd += mi; }
  if (tvd + mc <= eps) { q += mc; tvd += mc; }
  Try r;
  r.pass = up < q;
  r.tvd = tvd;
  return r;
}

// Where the workgroups of one prompt meet: the sums of their vocabulary chunks and a counter that is zero between calls.
struct SelectShare {
  int* arrived;     // [prompts]
  float* sums;      // [prompts][MAXCHUNKS]
};

// TCH = 64-node chunks of the tree held in registers by the walking wave (Tn <= 64 * TCH); CPW = 256-entry vocabulary chunks
// that each of the eight waves sums per pass
template <int TCH, int CPW>
__global__ __launch_bounds__(512) void select_kernel(select_args a, SelectShare share, int* dev_status) {
  constexpr int SEL_THREADS = 512, SEL_WAVES = 8, PASS = SEL_WAVES * CPW;
  __shared__ int s_tok[CASCADE_MAX_DEPTH];   // tokens of the accepted path
  __shared__ int s_path[CASCADE_MAX_DEPTH];
  __shared__ int s_tried[CASCADE_MAX_WIDTH];
  __shared__ int s_len, s_cur, s_ntried, s_best;
  __shared__ float s_tvd;
  __shared__ float s_chunk[MAXCHUNKS];
  __shared__ float s_total;
  __shared__ int s_last;
  // LONGEST only
  __shared__ int s_par[CASCADE_MAX_TREE];
  __shared__ float s_ntvd[CASCADE_MAX_TREE];
  __shared__ unsigned char s_alive[CASCADE_MAX_TREE], s_ready[CASCADE_MAX_TREE], s_depth[CASCADE_MAX_TREE], s_haschild[CASCADE_MAX_TREE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.y, parts = gridDim.x;
  const int lo = a.node_off[b], Tn = min(a.node_off[b + 1] - lo, 64 * TCH);
  // a tree larger than the launch was sized for is walked over its first 64 * TCH nodes only, and flagged
  if (tid == 0 && a.node_off[b + 1] - lo > 64 * TCH) atomicOr(dev_status, CASCADE_FLAG_TREE_SIZE);
  const int maxd = min(a.max_depth, CASCADE_MAX_DEPTH);
  const float eps = a.eps_tvd;

  if (a.mode == CASCADE_WALK_SEQUENTIAL) {
    if (wave == 0) {
      const int nch = (Tn + 63) >> 6;
      int par[TCH], tok[TCH];
      float qv[TCH], mi[TCH], mc[TCH], up[TCH];
      // the loads of several chunks are in flight together (all of them in trees of at most 256 nodes): clamped, because a
      // branch per chunk made every chunk wait for its own
      constexpr int GC = TCH > 4 ? 2 : TCH;
#pragma unroll
      for (int c0 = 0; c0 < TCH; c0 += GC) {
#pragma unroll
        for (int c = c0; c < c0 + GC; ++c) { par[c] = -2; tok[c] = -1; qv[c] = mi[c] = mc[c] = up[c] = 0.f; }
        if (c0 * 64 < Tn) {
          float pr[GC];
#pragma unroll
          for (int c = c0; c < c0 + GC; ++c) {
            const int at = lo + min(c * 64 + lane, Tn - 1);
            par[c] = a.parent[at];
            tok[c] = a.token[at];
            qv[c] = a.q_tok[at];
            mi[c] = a.m_int[at];
            mc[c] = a.m_conv[at];
            up[c] = a.u[at];
            pr[c - c0] = 1.f;
          }
          if (a.draft_prob)
#pragma unroll
            for (int c = c0; c < c0 + GC; ++c) pr[c - c0] = a.draft_prob[lo + min(c * 64 + lane, Tn - 1)];
#pragma unroll
          for (int c = c0; c < c0 + GC; ++c) {
            up[c] *= pr[c - c0];
            if (c * 64 + lane >= Tn) par[c] = -2;   // no node: nobody's child
          }
        }
      }
      int cur = 0, len = 0, ntried = 0;
      float tvd = 0.f;
      while (true) {
        int accepted = -1;
        ntried = 0;
#pragma unroll
        for (int c = 0; c < TCH; ++c) {
          if (c < nch && accepted < 0) {
            const int j = c * 64 + lane;
            unsigned long long kids = __ballot(par[c] == cur && j > cur);
            while (kids) {
              const int l = __ffsll((long long)kids) - 1;
              kids &= kids - 1;
              const Try r = try_node(readlane_f(qv[c], l), readlane_f(mi[c], l), readlane_f(mc[c], l),
                                     readlane_f(up[c], l), tvd, eps);
              tvd = r.tvd;
              if (r.pass) { accepted = c * 64 + l; break; }
              const int tt = __builtin_amdgcn_readlane(tok[c], l);
              if (ntried < CASCADE_MAX_WIDTH) { if (lane == 0) s_tried[ntried] = tt; ++ntried; }
              else if (lane == 0) atomicOr(dev_status, CASCADE_FLAG_WIDTH);
            }
          }
        }
        if (accepted < 0) break;
        if (len >= maxd) { if (lane == 0) atomicOr(dev_status, CASCADE_FLAG_DEPTH); break; }
        int at = tok[0];   // (of the accepted node's chunk)
#pragma unroll
        for (int c = 1; c < TCH; ++c) at = (accepted >> 6) == c ? tok[c] : at;
        at = __builtin_amdgcn_readlane(at, accepted & 63);
        if (lane == 0) { s_path[len] = accepted; s_tok[len] = at; }
        ++len;
        cur = accepted;
      }
      if (lane == 0) { s_len = len; s_cur = cur; s_ntried = ntried; s_tvd = tvd; }
    }
  } else {
    // top-down recurrence over the tree, one level per round; every value a round needs is requested before the first one
    // (a load inside a round costs it a trip to memory: 119 nodes and nine rounds x 33088 entries 10.1 -> 9.4 us)
    constexpr int SLOTS = 64 * TCH / SEL_THREADS > 0 ? 64 * TCH / SEL_THREADS : 1;   // nodes of a thread
    int par[SLOTS];
    float qv[SLOTS], mi[SLOTS], mc[SLOTS], up[SLOTS];
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) {
      const int i = tid + k * SEL_THREADS, at = lo + max(min(i, Tn - 1), 0);
      par[k] = -1;
      qv[k] = mi[k] = mc[k] = up[k] = 0.f;
      if (k * SEL_THREADS < Tn) {
        par[k] = a.parent[at];
        qv[k] = a.q_tok[at];
        mi[k] = a.m_int[at];
        mc[k] = a.m_conv[at];
        up[k] = a.u[at];
        if (a.draft_prob) up[k] *= a.draft_prob[at];
      }
      if (i >= Tn) continue;
      if (i == 0) par[k] = -1;
      else if (par[k] < 0 || par[k] >= i) { atomicOr(dev_status, CASCADE_FLAG_PARENT); par[k] = -1; }   // orphan: never reached
      s_par[i] = par[k];
      s_alive[i] = i == 0;
      s_ready[i] = i == 0;
      s_depth[i] = 0;
      s_ntvd[i] = 0.f;
      s_haschild[i] = 0;
    }
    if (tid == 0) s_best = -1;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SLOTS; ++k)
      if (tid + k * SEL_THREADS < Tn && par[k] >= 0) s_haschild[par[k]] = 1;
    for (int round = 0; round < maxd; ++round) {
      bool can[SLOTS];
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) {
        const int i = tid + k * SEL_THREADS;
        can[k] = i < Tn && !s_ready[i] && par[k] >= 0 && s_ready[par[k]];
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) {
        const int i = tid + k * SEL_THREADS;
        if (can[k]) {
          const int pi = par[k];
          float t = s_ntvd[pi];
          bool alive = false;
          if (s_alive[pi]) {
            const Try r = try_node(qv[k], mi[k], mc[k], up[k], t, eps);
            t = r.tvd;
            alive = r.pass;
          }
          s_ntvd[i] = t;
          s_alive[i] = alive;
          s_depth[i] = s_depth[pi] + 1;
          s_ready[i] = 1;
        }
      }
      __syncthreads();
    }
    // every leaf: deepest accepted node on its chain; best = longest, ties to the smallest leaf index
    for (int i = tid; i < Tn; i += SEL_THREADS) {
      if (!s_ready[i] && s_par[i] >= 0) atomicOr(dev_status, CASCADE_FLAG_DEPTH);
      if (!s_haschild[i]) {
        int x = i;
        while (x >= 0 && !s_alive[x]) x = s_par[x];   // parents have smaller indices: ends at the root, or at -1 under an orphan
        if (x >= 0) atomicMax(&s_best, (int)s_depth[x] * CASCADE_MAX_TREE + (CASCADE_MAX_TREE - 1 - i));
      }
    }
    __syncthreads();
    if (tid == 0) {
      const int best = max(s_best, CASCADE_MAX_TREE - 1);   // no usable leaf (bad parent array): root only
      const int leaf = CASCADE_MAX_TREE - 1 - (best % CASCADE_MAX_TREE);
      int x = leaf, first_dead = -1;
      while (x > 0 && !s_alive[x]) { first_dead = x; x = s_par[x]; }
      if (x < 0) { x = 0; first_dead = -1; }
      const int len = s_depth[x];
      s_len = len;
      s_cur = x;
      s_tvd = first_dead >= 0 ? s_ntvd[first_dead] : s_ntvd[x];
      s_ntried = first_dead >= 0 ? 1 : 0;
      if (first_dead >= 0) s_tried[0] = a.token[lo + first_dead];
      for (int d = len - 1, y = x; d >= 0; --d) { s_path[d] = y; s_tok[d] = a.token[lo + y]; y = s_par[y]; }
    }
  }
  __syncthreads();

  // ---- correction / bonus token: inverse CDF over the terminal node's distribution
  const int len = s_len, cur = s_cur, ntried = s_ntried;
  const int V = a.vocab;
  const float* Lr = a.logits + (int64_t)(lo + cur) * V;
  const float thr = a.row_thr[lo + cur], lse = a.row_lse[lo + cur];
  const int nchunks = (V + 255) >> 8;
  const bool vec = (V & 3) == 0;
  const float ub = a.u_bonus[b];

  // Chunk sums.  A pass of a workgroup covers PASS chunks, CPW per wave; all loads of a pass are in flight together: clamped
  // into the row (entries past its end are masked), because a guard around every load made every chunk wait for the one
  // before.  What bounds this part is the chain of instructions of a wave (a dependent one issues every 8 cycles) and, in long
  // rows, the exponentials of the one compute unit: the scans of a pass advance side by side without branches, the rejected
  // tokens are visited once per pass by the wave that owns them, and the passes of a prompt are dealt to `parts` workgroups.
  // Each of those walks the tree by itself (nothing is exchanged before the sums), leaves its sums in memory and counts itself
  // in; the one that arrives last goes on, the others are done, so no workgroup ever waits for another.
  const int ban = lane < ntried ? s_tried[lane] : -1;   // lane e holds the e-th rejected token
  const int n_pass = (nchunks + PASS - 1) / PASS;
  auto sum_chunks = [&](int first, int step, bool use_ban, auto&& put) {
#pragma unroll 1
    for (int ps = first; ps < n_pass; ps += step) {
      const int c0 = ps * PASS + wave;   // this wave's chunks: c0, c0 + SEL_WAVES, ...
      f32x4 r[CPW];
#pragma unroll
      for (int ci = 0; ci < CPW; ++ci) {
        const int e0 = (c0 + SEL_WAVES * ci) * 256 + 4 * lane;
        if (vec) r[ci] = *(const f32x4*)(Lr + min(e0, V - 4));
        else
#pragma unroll
          for (int i = 0; i < 4; ++i) r[ci][i] = Lr[min(e0 + i, V - 1)];
      }
#pragma unroll
      for (int ci = 0; ci < CPW; ++ci)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float x = __expf(r[ci][i] - lse);
          r[ci][i] = r[ci][i] >= thr ? x : 0.f;
        }
      if ((ps + 1) * PASS * 256 > V)   // the pass reaches past the row
#pragma unroll
        for (int ci = 0; ci < CPW; ++ci)
#pragma unroll
          for (int i = 0; i < 4; ++i) r[ci][i] = (c0 + SEL_WAVES * ci) * 256 + 4 * lane + i < V ? r[ci][i] : 0.f;
      for (int e = 0; use_ban && e < ntried; ++e) {
        const int t = __builtin_amdgcn_readlane(ban, e);
        if (t >= 0 && t / (256 * PASS) == ps && ((t >> 8) & (SEL_WAVES - 1)) == wave)
#pragma unroll
          for (int ci = 0; ci < CPW; ++ci)
#pragma unroll
            for (int i = 0; i < 4; ++i) r[ci][i] = (c0 + SEL_WAVES * ci) * 256 + 4 * lane + i == t ? 0.f : r[ci][i];
      }
      float cs[CPW];
#pragma unroll
      for (int ci = 0; ci < CPW; ++ci) cs[ci] = ((r[ci][0] + r[ci][1]) + r[ci][2]) + r[ci][3];
      auto scan_step = [&](auto shift) {
#pragma unroll
        for (int ci = 0; ci < CPW; ++ci) cs[ci] += shift(cs[ci]);
      };
      scan_step([](float v) { return dpp_f32<0x111, 0xf>(0.f, v); });   // wave_sum's steps: lane 63 ends up with the total
      scan_step([](float v) { return dpp_f32<0x112, 0xf>(0.f, v); });
      scan_step([](float v) { return dpp_f32<0x114, 0xf>(0.f, v); });
      scan_step([](float v) { return dpp_f32<0x118, 0xf>(0.f, v); });
      scan_step([](float v) { return dpp_f32<0x142, 0xa>(0.f, v); });
      scan_step([](float v) { return dpp_f32<0x143, 0xc>(0.f, v); });
      if (lane == 63)
#pragma unroll
        for (int ci = 0; ci < CPW; ++ci) put(c0 + SEL_WAVES * ci, cs[ci]);   // chunks past the row: 0
    }
  };
  auto to_lds = [&](int c, float x) { if (c < MAXCHUNKS) s_chunk[c] = x; };

  float cs[4];   // wave 0: lane l owns chunks 4 l .. 4 l + 3
  bool last = parts == 1;   // wave 0: this workgroup goes on
  if (parts > 1) {
    // Sums and counter pass through memory that all XCDs see (agent-scope accesses go past their L2s), so no cache has to be
    // written back; the wait puts every wave's sums there before the workgroup counts itself in.
    float* shared = share.sums + (size_t)b * MAXCHUNKS;
    sum_chunks(blockIdx.x, parts, true, [&](int c, float x) {
      if (c < nchunks) __hip_atomic_store(shared + c, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (wave == 0) {
      int n = 0;
      if (lane == 0) n = __hip_atomic_fetch_add(share.arrived + b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last = __builtin_amdgcn_readfirstlane(n) == parts - 1;
      if (lane == 0) {
        s_last = last;
        if (last) __hip_atomic_store(share.arrived + b, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next call
      }
      if (last)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          cs[i] = 4 * lane + i < nchunks ? __hip_atomic_load(shared + 4 * lane + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.f;
    }
  } else {
    sum_chunks(0, 1, true, to_lds);
    __syncthreads();
    if (wave == 0)
#pragma unroll
      for (int i = 0; i < 4; ++i) cs[i] = 4 * lane + i < nchunks ? s_chunk[4 * lane + i] : 0.f;
  }
  // wave 0 of the workgroup that goes on
  float total = 0.f, base = 0.f;
  int cstar = -1;
  bool lastkept = false;
  auto find_chunk = [&]() {   // the chunk in which the running sum crosses the target
    const float loc = ((0.f + cs[0]) + cs[1]) + cs[2] + cs[3];
    const float incl = wave_scan_incl_f(loc);
    total = readlane_f(incl, 63);
    const float target = ub * total;
    float run = incl - loc;
    int cand = 0x7fffffff;
    float cbase = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (cand == 0x7fffffff && cs[i] > 0.f && run + cs[i] > target) { cand = 4 * lane + i; cbase = run; }
      run += cs[i];
    }
    cstar = wave_min_i(cand);
    lastkept = cstar == 0x7fffffff;
    if (lastkept) {
      // rounding kept the running sum at or below the target: take the last chunk that holds mass
      int lastc = -1;
#pragma unroll
      for (int i = 0; i < 4; ++i) if (cs[i] > 0.f) lastc = 4 * lane + i;
      cstar = wave_max_i(lastc);
      base = 0.f;
    } else {
      base = readlane_f(cbase, __ffsll((long long)__ballot(cand == cstar)) - 1);
    }
  };
  if (wave == 0 && last) {
    find_chunk();
    if (lane == 0) s_total = total;
  }
  __syncthreads();
  if (parts > 1 && !s_last) return;
  bool use_ban = true;
  if (!(s_total > 0.f)) {   // every kept entry was removed: the unfiltered row, which this workgroup sums by itself
    use_ban = false;
    sum_chunks(0, 1, false, to_lds);
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) cs[i] = 4 * lane + i < nchunks ? s_chunk[4 * lane + i] : 0.f;
      find_chunk();
    }
  }

  if (wave == 0) {
    int x = -1;
    if (total > 0.f && cstar >= 0) {
      const float target = ub * total;
      const int e0 = cstar * 256 + lane * 4;
      float m[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float g = Lr[min(e0 + i, V - 1)], p = __expf(g - lse);
        m[i] = (g >= thr && e0 + i < V) ? p : 0.f;
      }
      for (int e = 0; use_ban && e < ntried; ++e) {
        const int t = __builtin_amdgcn_readlane(ban, e);
#pragma unroll
        for (int i = 0; i < 4; ++i) m[i] = e0 + i == t ? 0.f : m[i];
      }
      const float p0 = m[0], p1 = p0 + m[1], p2 = p1 + m[2], p3 = p2 + m[3];
      const float incl = wave_scan_incl_f(p3);
      const float run = base + (incl - p3);
      int cand = 0x7fffffff;
      if (!lastkept) {
        if (m[0] > 0.f && run + p0 > target) cand = e0;
        else if (m[1] > 0.f && run + p1 > target) cand = e0 + 1;
        else if (m[2] > 0.f && run + p2 > target) cand = e0 + 2;
        else if (m[3] > 0.f && run + p3 > target) cand = e0 + 3;
      }
      x = wave_min_i(cand);
      if (x == 0x7fffffff) {
        int last = -1;
#pragma unroll
        for (int i = 0; i < 4; ++i) if (m[i] > 0.f) last = e0 + i;
        x = wave_max_i(last);
      }
    }
    if (lane == 0) {
      a.emitted[(int64_t)b * (a.max_depth + 1) + len] = x;
      a.accept_len[b] = len;
      a.terminal[b] = cur;
      a.tvd_used[b] = s_tvd;
    }
  } else if (wave == 1) {
    for (int d = lane; d <= a.max_depth; d += 64) {
      if (d < a.max_depth) a.path_nodes[(int64_t)b * a.max_depth + d] = d < len ? s_path[d] : -1;
      if (d != len) a.emitted[(int64_t)b * (a.max_depth + 1) + d] = d < len ? s_tok[d] : -1;
    }
  }
}

}  // namespace

hipError_t launch_select(cascade_ctx* ctx, const select_args* a) {
  KernelTimer t(ctx, CASCADE_K_SELECT);
  SelectShare share = {(int*)ctx->select_ws, (float*)(ctx->select_ws + SELECT_MAX_SHARED * sizeof(int))};
  const bool small_tree = ctx->lim.max_nodes_per_tree <= 256;
  // Passes of 4096 entries, dealt to up to two workgroups per compute unit: a row's exponentials take a lone compute unit 1 us per
  // 16384 entries, the meeting of the workgroups 1.5 us.  In a step, with one workgroup per prompt and as built now: 60 nodes x
  // 16384 entries 9.0 -> 6.4 us, 60 x 65536 13.3 -> 6.7, four trees of 256 x 65536 15.0 -> 8.3.  Trees of 12 nodes, walk alone:
  // 48 prompts x 65536 12.4 -> 8.3, 100 x 33088 9.4 -> 8.4, 100 x 65536 13.4 -> 10.4 (with one workgroup per compute unit, two
  // parts: 10.3 and 14.5).  More than 128 prompts fill the chip by themselves.
  const int pass = 4096, n_pass = (a->vocab + pass - 1) / pass;
  int parts = a->n_prompts <= SELECT_MAX_SHARED ? 2 * ctx->n_cu / a->n_prompts : 1;
  parts = parts < 1 ? 1 : (parts < n_pass ? parts : n_pass);
  if (parts > 1 && recorded(ctx->stream)) parts = 1;
  // A lone workgroup takes up to eight chunks per wave and pass, and as many in every pass as it can: 33088 entries are 130 chunks, 17
  // per wave, three passes of six (200 prompts: 9.9 us, with eight 11.4).
  const int per_wave = ((a->vocab + 255) / 256 + 7) / 8, alone = (per_wave + 7) / 8, cpw = parts > 1 || n_pass == 1 ? 2 : ((per_wave + alone - 1) / alone <= 6 ? 6 : 8);
  dim3 grid(parts, a->n_prompts);
#define CASCADE_LAUNCH_SELECT(TCH, CPW) CASCADE_TIMED_LAUNCH(t, (select_kernel<TCH, CPW>), grid, dim3(512), 0, ctx->stream, *a, share, ctx->dev_status)
  if (cpw == 2) { if (small_tree) CASCADE_LAUNCH_SELECT(4, 2); else CASCADE_LAUNCH_SELECT(16, 2); }
  else if (cpw == 6) { if (small_tree) CASCADE_LAUNCH_SELECT(4, 6); else CASCADE_LAUNCH_SELECT(16, 6); }
  else { if (small_tree) CASCADE_LAUNCH_SELECT(4, 8); else CASCADE_LAUNCH_SELECT(16, 8); }
#undef CASCADE_LAUNCH_SELECT
  return hipGetLastError();
}
