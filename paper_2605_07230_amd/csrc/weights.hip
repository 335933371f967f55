// convergence_weights: the Eq. 4 weight mask of the drafter-training loss.  For every pair of
// consecutive positions (k, k+1) of a target-generated sequence: cos(F_k, F_{k+1}) >= tau_seq (the
// convergence set of Eq. 2 between neighbours) gives weight c, otherwise 1.
//
// Bandwidth-bound: every feature row should cross HBM once.  A run of consecutive pairs belongs to the waves that share
// its rows: the four waves of a workgroup take a quarter of every row each (narrow rows: fewer waves per run), in 1 KiB
// pieces, with seven rows requested ahead.  Only the first row of a run is read twice.  8 sequences x 2356 x 4096 bf16:
// 30.3 us (154 MB, 5.1 TB/s); with whole rows per wave the chip filled only with runs of 9 pairs, 11 % of the rows were
// read twice, and it took 36.0.
#include "common.h"

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr int MAX_RUN = 128;   // pairs of a run (their partial sums wait in LDS)

template <typename T> struct Acc;
template <> struct Acc<float> {
  static __device__ __forceinline__ void dot(const u32x4& a, const u32x4& b, float& ab, float& bb) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = __uint_as_float(a[i]), y = __uint_as_float(b[i]);
      ab = fmaf(x, y, ab);
      bb = fmaf(y, y, bb);
    }
  }
};
template <> struct Acc<uint16_t> {   // bf16 pairs packed in 32-bit words
  static __device__ __forceinline__ void dot(const u32x4& a, const u32x4& b, float& ab, float& bb) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x0 = __uint_as_float(a[i] << 16), x1 = __uint_as_float(a[i] & 0xffff0000u);
      const float y0 = __uint_as_float(b[i] << 16), y1 = __uint_as_float(b[i] & 0xffff0000u);
      ab = fmaf(x0, y0, ab);
      ab = fmaf(x1, y1, ab);
      bb = fmaf(y0, y0, bb);
      bb = fmaf(y1, y1, bb);
    }
  }
};

// CS waves share a run of consecutive rows, each with every CS-th KiB of a row (NV of them), and the next R - 1 rows
// requested; a workgroup of four waves holds 4 / CS runs.  Each wave leaves its part of every row's norm and of every
// pair's product in LDS, and they are added once at the end of the run, so the loop has no barrier.
template <typename T, int NV, int CS, int R>
__global__ __launch_bounds__(256) void conv_weight_kernel(conv_weight_args a, int runs_per_seq, int run_len) {
  constexpr int RUNS = 4 / CS;
  __shared__ float s_dot[RUNS][CS][MAX_RUN], s_norm[RUNS][CS][MAX_RUN + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int part = wave % CS, mine = wave / CS;
  const long long run_id = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * RUNS + mine;
  const bool exists = run_id < (long long)a.n_seqs * runs_per_seq;
  const int seq = exists ? (int)(run_id / runs_per_seq) : 0, run = exists ? (int)(run_id % runs_per_seq) : 0;
  const int K = a.seq_len;
  const int nvec = a.hidden * (int)sizeof(T) / 16;   // 16-byte vectors per row
  const u32x4* base = (const u32x4*)a.features + (long long)seq * K * nvec;
  const int k0 = run * run_len, n = exists ? min(run_len, K - 1 - k0) : 0;   // pairs (k, k+1) for k in [k0, k0 + n)

  if (n > 0) {
    u32x4 r[R][NV];
    auto load_row = [&](int i, u32x4 (&dst)[NV]) {   // row i of the run; past its end the last one again (a cache hit)
      const u32x4* row = base + (long long)(k0 + min(i, n)) * nvec;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int idx = (v * CS + part) * 64 + lane;
        const u32x4 x = row[min(idx, nvec - 1)];   // clamped, zeroed below
        dst[v] = idx < nvec ? x : u32x4{0u, 0u, 0u, 0u};
      }
    };
#pragma unroll
    for (int i = 0; i < R; ++i) load_row(i, r[i]);
    float pp = 0.f, dummy = 0.f;
#pragma unroll
    for (int v = 0; v < NV; ++v) Acc<T>::dot(r[0][v], r[0][v], dummy, pp);
    pp = wave_sum(pp);
    if (lane == 0) s_norm[mine][part][0] = pp;
    for (int i0 = 0; i0 < n; i0 += R) {
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const int i = i0 + u;
        if (i >= n) break;
        float ab = 0.f, bb = 0.f;
#pragma unroll
        for (int v = 0; v < NV; ++v) Acc<T>::dot(r[u][v], r[(u + 1) % R][v], ab, bb);
        load_row(i + R, r[u]);
        ab = wave_sum(ab);
        bb = wave_sum(bb);
        if (lane == 0) { s_dot[mine][part][i] = ab; s_norm[mine][part][i + 1] = bb; }
      }
    }
  }
  __syncthreads();
  float* wout = a.weights + (long long)seq * K;
  float* cout = a.cos_next ? a.cos_next + (long long)seq * K : nullptr;
  for (int i = part * 64 + lane; i < n; i += 64 * CS) {
    float ab = 0.f, aa = 0.f, bb = 0.f;
#pragma unroll
    for (int c = 0; c < CS; ++c) { ab += s_dot[mine][c][i]; aa += s_norm[mine][c][i]; bb += s_norm[mine][c][i + 1]; }
    const float cs = (aa > 0.f && bb > 0.f) ? ab / (sqrtf(aa) * sqrtf(bb)) : 0.f;
    wout[k0 + i] = cs >= a.tau_seq ? a.c : 1.f;
    if (cout) cout[k0 + i] = cs;
  }
  if (exists && run == runs_per_seq - 1 && part == 0 && lane == 0) {   // the last position has no successor
    wout[K - 1] = 1.f;
    if (cout) cout[K - 1] = 0.f;
  }
}

template <typename T, int NV, int CS, int R>
hipError_t launch_cs(cascade_ctx* ctx, const conv_weight_args* a) {
  // one run per group of CS waves with eight waves on every compute unit: long runs re-read fewer boundary rows
  const long long pairs = (long long)a->n_seqs * (a->seq_len - 1), groups = (long long)ctx->n_cu * 8 / CS;
  long long run_len = (pairs + groups - 1) / groups;
  run_len = run_len < 4 ? 4 : (run_len > MAX_RUN ? MAX_RUN : run_len);
  const int runs_per_seq = a->seq_len > 1 ? (int)((a->seq_len - 1 + run_len - 1) / run_len) : 1;
  const long long blocks = ((long long)a->n_seqs * runs_per_seq + 4 / CS - 1) / (4 / CS);
  const long long gy = (blocks + (1 << 22) - 1) >> 22;   // a grid dimension holds fewer than 2^32 threads
  KernelTimer t(ctx, CASCADE_K_WEIGHTS);
  CASCADE_TIMED_LAUNCH(t, (conv_weight_kernel<T, NV, CS, R>), dim3((unsigned)((blocks + gy - 1) / gy), (unsigned)gy), dim3(256), 0, ctx->stream, *a,
                       runs_per_seq, (int)run_len);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_t(cascade_ctx* ctx, const conv_weight_args* a) {
  const int kib = (a->hidden * (int)sizeof(T) + 1023) / 1024;   // at most 16
  if (kib <= 1) return launch_cs<T, 1, 1, 8>(ctx, a);
  if (kib <= 2) return launch_cs<T, 1, 2, 8>(ctx, a);
  if (kib <= 4) return launch_cs<T, 1, 4, 8>(ctx, a);
  if (kib <= 8) return launch_cs<T, 2, 4, 8>(ctx, a);
  return launch_cs<T, 4, 4, 4>(ctx, a);
}

}  // namespace

hipError_t launch_conv_weights(cascade_ctx* ctx, const conv_weight_args* a) {
  return a->dtype == CASCADE_BF16 ? launch_t<uint16_t>(ctx, a) : launch_t<float>(ctx, a);
}
