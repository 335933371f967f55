// kv_commit: append the root and the accepted path of every row's tree to that row's prefix cache,
// for all layers (Preliminaries: accepted tokens are appended to the prefix).  A pure gather /
// scatter of 16-byte pieces.
//
// One workgroup per (row, layer, keys or values, 2 KiB of a node row) copies all of the row's slots, or a group of them: the row's lookups are
// three trips to memory (prompt, lengths and tree; accepted length and path; the data), made once for all slots with the path
// in the lanes of a wave.  Bound by the copy: 47 MB (8 pairs of rows, 30 layers, 32 heads x 128) 15.4 -> 11.8 us, against 9.4 at
// the rate of a large copy.  One workgroup per (row, slot, layer) made two thirds of the launched ones find out by three
// dependent trips that their slot was empty, and dirty lines that stay in the L2s are written back after the last
// workgroup has ended: streaming (non-temporal) stores alone are worth 2 us.  Streaming loads cost 6; two, four or eight pieces of a
// thread in flight up to 1 (few slots have that many).  Only paths near 64 nodes in every row are slower than they were with a
// workgroup per slot: 1 GB (30 layers, 16 rows, 65 slots each) 196 -> 216 us, 21 slots 53.5 -> 49.5.
#include "common.h"

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct CommitParams {
  kv_commit_args a;
  int* dev_status;
  int row_vec;       // 16-byte pieces per node row (n_kv_heads * head_dim * elem / 16)
  int head_vec;      // 16-byte pieces per head
  int part_vec;      // 16-byte pieces of a node row that one workgroup copies
  int parts;         // such parts of a node row
  int slots;         // slots that one workgroup copies
  long long sl, sr, sh, sp;   // cache strides in 16-byte pieces
  long long tree_layer_vec;   // 16-byte pieces per layer of k_tree / v_tree
};

constexpr int COMMIT_THREADS = 256;

__global__ __launch_bounds__(COMMIT_THREADS) void kv_commit_kernel(CommitParams p) {
  __shared__ int s_node[CASCADE_MAX_DEPTH + 1];   // tree node of every slot, -1: nothing to copy
  const kv_commit_args& a = p.a;
  const int s = blockIdx.x, layer = blockIdx.y, part = (blockIdx.z >> 1) % p.parts, slot0 = (blockIdx.z >> 1) / p.parts * p.slots;
  const bool values = blockIdx.z & 1;
  const int tid = threadIdx.x;
  const bool reporter = layer == 0 && blockIdx.z == 0 && tid == 0;

  const int b = a.row_prompt[s], P = a.prefix_len[s];
  const int base = a.node_off[s], n_tree = a.node_off[s + 1] - base;
  if (b < 0 || b >= a.n_prompts) {
    if (reporter) { atomicOr(p.dev_status, CASCADE_FLAG_PATH); a.prefix_len_out[s] = P; }
    return;
  }
  const int n_acc = a.accept_len[b];
  int node = 0;      // slot tid: the root, then the path
  if (tid > 0 && tid <= a.max_depth) node = a.path_nodes[(long long)b * a.max_depth + tid - 1];
  if (n_acc < 0 || n_acc > a.max_depth) {
    if (reporter) { atomicOr(p.dev_status, CASCADE_FLAG_DEPTH); a.prefix_len_out[s] = P; }
    return;
  }
  if (P < 0 || P + 1 + n_acc > a.prefix_cap) {
    if (reporter) { atomicOr(p.dev_status, CASCADE_FLAG_CAPACITY); a.prefix_len_out[s] = P; }
    return;
  }
  if (reporter) a.prefix_len_out[s] = P + 1 + n_acc;
  const int n_slots = min(1 + n_acc - slot0, p.slots);   // of this workgroup
  if (n_slots <= 0) return;
  if (tid <= n_acc) {   // at most CASCADE_MAX_DEPTH + 1 slots
    if (node < 0 || node >= n_tree || base < 0 || base + node >= a.n_nodes_total) {
      if (layer == 0 && blockIdx.z == 0) atomicOr(p.dev_status, CASCADE_FLAG_PATH);
      node = -1;
    }
    s_node[tid] = node;
  }
  __syncthreads();
  const u32x4* src = (const u32x4*)(values ? a.v_tree : a.k_tree) + (long long)layer * p.tree_layer_vec + (long long)base * p.row_vec;
  u32x4* dst = (u32x4*)(values ? a.v_cache : a.k_cache) + (long long)layer * p.sl + (long long)s * p.sr + (long long)P * p.sp;
  const int v0 = part * p.part_vec, n_vec = min(p.part_vec, p.row_vec - v0), total = n_slots * n_vec;   // n_vec >= 1
  for (int i = tid; i < total; i += COMMIT_THREADS) {
    const unsigned j = (unsigned)i / (unsigned)n_vec, slot = slot0 + j, v = v0 + i - j * n_vec, head = v / (unsigned)p.head_vec;
    const int nd = s_node[slot];
    if (nd >= 0)
      __builtin_nontemporal_store(src[(long long)nd * p.row_vec + v], dst + (long long)slot * p.sp + (long long)head * p.sh + (v - head * p.head_vec));
  }
}

}  // namespace

hipError_t launch_kv_commit(cascade_ctx* ctx, const kv_commit_args* a) {
  const int e = a->dtype == CASCADE_BF16 ? 2 : 4;
  CommitParams p;
  p.a = *a;
  p.dev_status = ctx->dev_status;
  p.head_vec = a->head_dim * e / 16;
  p.row_vec = a->n_kv_heads * p.head_vec;
  p.sl = a->cache_stride_layer * e / 16;
  p.sr = a->cache_stride_row * e / 16;
  p.sh = a->cache_stride_head * e / 16;
  p.sp = a->cache_stride_pos * e / 16;
  p.tree_layer_vec = (long long)a->n_nodes_total * p.row_vec;
  // 2 KiB of every node row per workgroup: 47 MB (30 layers x 16 rows x 8 KiB) 11.8 us with parts of 2 or 4 KiB, 12.7 with whole rows
  p.part_vec = p.row_vec < 128 ? p.row_vec : 128;
  p.parts = (p.row_vec + p.part_vec - 1) / p.part_vec;
  // Few workgroups share the slots, eight each at least: one that copies 65 slots alone is a chain of 33 pieces per thread.  Paths of 64
  // nodes: 2 rows x 1 layer 11.4 -> 4.2 us, 16 x 1 11.8 -> 5.8, 2 x 4 11.5 -> 4.4.  Where the rows and layers make four workgroups per
  // compute unit by themselves, more would mostly find out that their slots are empty (16 rows x 30 layers, paths of 0 to 2 nodes
  // of at most 64: 5.4-7.6 us, in groups of eight slots 22-23).
  const int all = 1 + a->max_depth;
  const int64_t base = (int64_t)a->n_rows * a->n_layers * 2 * p.parts, room = 4 * ctx->n_cu / base;
  const int groups = (int)(room < 1 ? 1 : (room < (all + 7) / 8 ? room : (all + 7) / 8));
  p.slots = (all + groups - 1) / groups;
  dim3 grid((unsigned)a->n_rows, (unsigned)a->n_layers, 2u * p.parts * groups);
  KernelTimer t(ctx, CASCADE_K_COMMIT);
  CASCADE_TIMED_LAUNCH(t, kv_commit_kernel, grid, dim3(COMMIT_THREADS), 0, ctx->stream, p);
  return hipGetLastError();
}
