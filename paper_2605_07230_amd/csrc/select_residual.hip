// select_path with full drafter distributions: the SEQUENTIAL walk of Alg. 2 in which every
// rejection replaces the verifying distribution f by Alg. 1's residual norm([f - p]_+) against the
// rejected node's drafter row, and the last token is drawn from what is left.
//
// One workgroup of 16 waves per prompt.  The verifying distribution lives in registers for the
// whole walk: wave w owns the vocabulary segment [w * SEG, (w + 1) * SEG), SEG = 256 * VQ, as VQ
// four-wide vectors per lane (entry = w * SEG + 256 * i + 4 * lane + c).  A rejection costs one
// coalesced read of the drafter row, a workgroup sum and a rescale; an acceptance one read of the
// new node's logits row.  All decisions are taken by every thread on the same broadcast scalars,
// so control flow stays uniform.  The inverse CDF at the end runs over the same registers.
// Bound by the chain of dependent trips to memory: the scalars of all nodes (and, but for the widest frame, the drafter's
// probability of each node's token) are fetched once, by a thread per node, and the drafter row of a rejected child's sibling is on
// its way while the child's residual is summed.  In a step, with a trip per tried child for each of these before: 60 nodes x 16384,
// four prompts 22.4 -> 15.6 us, 60 x 4096 10.7 -> 9.2, 60 x 20480 50.6 -> 14.6 (also: frames of its own up to 32768 and
// 49152 entries), 50 x 33088, two prompts 53.5 -> 26.2.  The row of a node's first child is not requested before its test:
// chains of eight accepted first children 9.7 -> 8.9 us (1000 entries), 13.0 -> 12.5 (8192), 13.7 -> 12.8 (16384), with a row for each of
// them 10.5, 15.9 and 15.0.
#include "common.h"

namespace {

constexpr int NW = 16;

struct Try {
  bool pass;
  float tvd;
};
__device__ __forceinline__ Try try_node(float q, float mi, float mc, float up, float tvd, float eps) {
  if (tvd + mi <= eps) { q += mi; tvd += mi; }
  if (tvd + mc <= eps) { q += mc; tvd += mc; }
  Try r;
  r.pass = up < q;
  r.tvd = tvd;
  return r;
}

__device__ __forceinline__ float readlane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// EXACT: vocab == 16 * SEG, every lane's entries exist (no clamping, plain immediate offsets)
template <int VQ, bool EXACT>
__global__ __launch_bounds__(1024) void select_residual_kernel(select_args a, int* dev_status) {
  constexpr int SEG = 256 * VQ;
  __shared__ int s_child[CASCADE_MAX_WIDTH];
  __shared__ int s_par[CASCADE_MAX_TREE], s_tok[CASCADE_MAX_TREE];                       // the tree's nodes
  __shared__ float s_mi[CASCADE_MAX_TREE], s_mc[CASCADE_MAX_TREE], s_up[CASCADE_MAX_TREE];   // s_up: u, times the drafter's probability (GATHER)
  __shared__ int s_path[CASCADE_MAX_DEPTH];
  __shared__ int s_m, s_x;
  __shared__ float s_q;
  __shared__ float s_wsum[NW];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x;
  const int lo = a.node_off[b], Tn = min(a.node_off[b + 1] - lo, CASCADE_MAX_TREE);
  if (tid == 0 && a.node_off[b + 1] - lo > CASCADE_MAX_TREE) atomicOr(dev_status, CASCADE_FLAG_TREE_SIZE);
  const int V = a.vocab;   // a multiple of 4, at most 16 * SEG (checked by the host)
  const int maxd = min(a.max_depth, CASCADE_MAX_DEPTH);
  const float eps = a.eps_tvd;
  const int e_base = wave * SEG + lane * 4;

  f32x4 f[VQ];
  auto load_target = [&](int node) {
    const float* Lr = a.logits + (int64_t)(lo + node) * V;
    const float thr = a.row_thr[lo + node], lse = a.row_lse[lo + node];
#pragma unroll
    for (int i = 0; i < VQ; ++i) {
      const int e = e_base + 256 * i;
      const f32x4 g = *(const f32x4*)((const char*)Lr + 4u * (unsigned)(EXACT ? e : min(e, V - 4)));   // clamped: always in bounds, masked below
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float x = __expf(g[c] - lse);
        f[i][c] = ((EXACT || e < V) && g[c] >= thr) ? x : 0.f;
      }
      if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // at most four row loads in flight: registers
    }
  };

  // AHEAD: the drafter row of a child is requested before it is known whether the child is rejected (frames of 8 vectors and more
  // have no registers for it and read the row when they need it, twice).  GATHER: probabilities of all tokens at once; 250
  // nodes x 65536 are as many lines and pages (16 prompts 43.0 -> 46.8 us, with one at a time 41.6).
  constexpr bool AHEAD = VQ <= 4, GATHER = VQ < 16;
  f32x4 pr[AHEAD ? VQ : 1];
  auto load_draft = [&](int node) {
    const float* prow = a.draft_dist + (int64_t)(lo + node) * V;
#pragma unroll
    for (int i = 0; i < (AHEAD ? VQ : 0); ++i) {
      const int e = e_base + 256 * i;
      pr[i] = *(const f32x4*)((const char*)prow + 4u * (unsigned)(EXACT ? e : min(e, V - 4)));   // (a select on it would wait for it here)
    }
  };

  // Everything a tried child needs is fetched for all nodes at once: thread i is node i (a tree has at most 1024).
  static_assert(CASCADE_MAX_TREE <= 64 * NW, "a thread per node");
  if (tid < Tn) {
    const int tok = a.token[lo + tid];
    const float u = a.u[lo + tid];
    s_par[tid] = a.parent[lo + tid];
    s_mi[tid] = a.m_int[lo + tid];
    s_mc[tid] = a.m_conv[lo + tid];
    s_tok[tid] = tok;
    s_up[tid] = GATHER && tok >= 0 && tok < V ? u * a.draft_dist[(int64_t)(lo + tid) * V + tok] : u;
  }
  int cur = 0, len = 0;
  float tvd = 0.f;
  load_target(0);
  __syncthreads();
  while (true) {
    if (wave == 0) {   // ordered list of cur's children
      int k = 0;
      for (int base = (cur + 1) & ~63; base < Tn; base += 64) {
        const int j = base + lane;
        const bool is = j < Tn && j > cur && s_par[j] == cur;
        const unsigned long long m = __ballot(is);
        if (is) {
          const int idx = k + __popcll(m & ((1ull << lane) - 1ull));
          if (idx < CASCADE_MAX_WIDTH) s_child[idx] = j;
        }
        k += __popcll(m);
      }
      if (k > CASCADE_MAX_WIDTH) {
        if (lane == 0) atomicOr(dev_status, CASCADE_FLAG_WIDTH);
        k = CASCADE_MAX_WIDTH;
      }
      if (lane == 0) s_m = k;
    }
    __syncthreads();
    const int m = s_m;
    int accepted = -1;
    for (int j = 0; j < m; ++j) {
      const int ch = s_child[j];
      const int ta = s_tok[ch];
      const bool tok_ok = ta >= 0 && ta < V;
      const float* prow = a.draft_dist + (int64_t)(lo + ch) * V;
      if (tok_ok) {
        const int w_owner = ta / SEG, r = ta - w_owner * SEG;
        if (wave == w_owner && lane == ((r & 255) >> 2)) {
          float val = 0.f;
#pragma unroll
          for (int i = 0; i < VQ; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c)
              if ((r >> 8) == i && (r & 3) == c) val = f[i][c];
          s_q = val;
        }
      } else if (tid == 0) {
        atomicOr(dev_status, CASCADE_FLAG_TOKEN);
        s_q = 0.f;
      }
      const float px = !GATHER && tok_ok ? prow[ta] : 1.f;
      __syncthreads();
      const Try t = try_node(s_q, s_mi[ch], s_mc[ch], s_up[ch] * px, tvd, eps);
      tvd = t.tvd;
      if (t.pass) { accepted = ch; break; }
      // rejected: f <- norm([f - p]_+), kept as it is when nothing would be left
      if (AHEAD && j == 0) load_draft(ch);
      float loc = 0.f;
      f32x4 left[AHEAD ? VQ : 1];
      auto take_away = [&](int i, const f32x4& p4) {
        f32x4 d;
#pragma unroll
        for (int c = 0; c < 4; ++c) d[c] = fmaxf(f[i][c] - p4[c], 0.f);
        return d;
      };
      auto row_of = [&](int i) {
        const int e = e_base + 256 * i;
        f32x4 p4 = *(const f32x4*)((const char*)prow + 4u * (unsigned)(EXACT ? e : min(e, V - 4)));
        if (!EXACT && e >= V) p4 = f32x4{0.f, 0.f, 0.f, 0.f};   // f is 0 there as well
        return p4;
      };
#pragma unroll
      for (int i = 0; i < VQ; ++i) {
        f32x4 d = take_away(i, AHEAD ? pr[AHEAD ? i : 0] : row_of(i));
        if (AHEAD && !EXACT && e_base + 256 * i >= V) d = f32x4{0.f, 0.f, 0.f, 0.f};   // past the row: f is 0 and stays 0
        loc += ((d[0] + d[1]) + d[2]) + d[3];
        if (AHEAD) left[AHEAD ? i : 0] = d;
        if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
      }
      if (AHEAD && j + 1 < m) load_draft(s_child[j + 1]);
      const float ws = wave_sum(loc);
      if (lane == 0) s_wsum[wave] = ws;
      __syncthreads();
      float Z = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) Z += s_wsum[w];
      if (Z > 0.f) {
        const float inv = 1.f / Z;
#pragma unroll
        for (int i = 0; i < VQ; ++i) {   // (the second read of the row hits the cache: no second register copy of f)
          const f32x4 d = AHEAD ? left[AHEAD ? i : 0] : take_away(i, row_of(i));
          f[i] = d * inv;
          if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (accepted < 0) break;
    if (len >= maxd) {
      if (tid == 0) atomicOr(dev_status, CASCADE_FLAG_DEPTH);
      break;
    }
    if (tid == 0) s_path[len] = accepted;
    ++len;
    cur = accepted;
    load_target(cur);
  }
  __syncthreads();   // the last reads of s_wsum / s_q are done

  // ---- last token: inverse CDF over f, vocabulary order = (wave, i, lane, c)
  float cs[VQ], wt = 0.f;
#pragma unroll
  for (int i = 0; i < VQ; ++i) {
    cs[i] = wave_sum(((f[i][0] + f[i][1]) + f[i][2]) + f[i][3]);
    wt += cs[i];
  }
  if (lane == 0) s_wsum[wave] = wt;
  if (tid == 0) s_x = -1;
  __syncthreads();
  float total = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) total += s_wsum[w];
  const float target = a.u_bonus[b] * total;
  // the wave whose segment crosses the target; if rounding lets no segment cross, the last one with mass
  int wstar = -1, wlast = -1;
  float base = 0.f, run = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float x = s_wsum[w];
    if (x > 0.f) wlast = w;
    if (wstar < 0 && x > 0.f && run + x > target) { wstar = w; base = run; }
    run += x;
  }
  const bool forced_last = wstar < 0;
  if (forced_last) wstar = wlast;
  if (total > 0.f && wave == wstar) {
    int x = 0x7fffffff, last = -1;
    float r0 = base;
    bool done = false;
#pragma unroll
    for (int i = 0; i < VQ; ++i) {
      const int e0 = e_base + 256 * i;
#pragma unroll
      for (int c = 0; c < 4; ++c) if (f[i][c] > 0.f) last = e0 + c;
      if (!done && !forced_last && cs[i] > 0.f && r0 + cs[i] > target) {
        const float p0 = f[i][0], p1 = p0 + f[i][1], p2 = p1 + f[i][2], p3 = p2 + f[i][3];
        const float incl = wave_scan_incl_f(p3);
        const float rl = r0 + (incl - p3);
        int cand = 0x7fffffff;
        if (f[i][0] > 0.f && rl + p0 > target) cand = e0;
        else if (f[i][1] > 0.f && rl + p1 > target) cand = e0 + 1;
        else if (f[i][2] > 0.f && rl + p2 > target) cand = e0 + 2;
        else if (f[i][3] > 0.f && rl + p3 > target) cand = e0 + 3;
        x = wave_min_i(cand);
        done = x != 0x7fffffff;   // rounding inside the chunk may leave no crossing: fall through to later chunks
      }
      if (!done) r0 += cs[i];
    }
    if (x == 0x7fffffff) x = wave_max_i(last);
    if (lane == 0) s_x = x;
  }
  __syncthreads();

  for (int d = tid; d < a.max_depth; d += 1024)
    a.path_nodes[(int64_t)b * a.max_depth + d] = d < len ? s_path[d] : -1;
  for (int d = tid; d <= a.max_depth; d += 1024) {
    int v = -1;
    if (d < len) v = s_tok[s_path[d]];
    else if (d == len) v = s_x;
    a.emitted[(int64_t)b * (a.max_depth + 1) + d] = v;
  }
  if (tid == 0) {
    a.accept_len[b] = len;
    a.terminal[b] = cur;
    a.tvd_used[b] = tvd;
  }
}

}  // namespace

hipError_t launch_select_residual(cascade_ctx* ctx, const select_args* a) {
  KernelTimer t(ctx, CASCADE_K_SELECT);
  dim3 grid(a->n_prompts);
  const int V = a->vocab;
#define CASCADE_LAUNCH_RESIDUAL(VQ, EX) \
  CASCADE_TIMED_LAUNCH(t, (select_residual_kernel<VQ, EX>), grid, dim3(1024), 0, ctx->stream, *a, ctx->dev_status)
  if (V <= 16 * 256) { if (V == 16 * 256) CASCADE_LAUNCH_RESIDUAL(1, true); else CASCADE_LAUNCH_RESIDUAL(1, false); }
  else if (V <= 16 * 1024) { if (V == 16 * 1024) CASCADE_LAUNCH_RESIDUAL(4, true); else CASCADE_LAUNCH_RESIDUAL(4, false); }
  else if (V <= 16 * 2048) CASCADE_LAUNCH_RESIDUAL(8, false);
  else if (V <= 16 * 3072) CASCADE_LAUNCH_RESIDUAL(12, false);
  else { if (V == 16 * 4096) CASCADE_LAUNCH_RESIDUAL(16, true); else CASCADE_LAUNCH_RESIDUAL(16, false); }
#undef CASCADE_LAUNCH_RESIDUAL
  return hipGetLastError();
}
