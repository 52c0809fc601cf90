// Host side of the one-launch decoding steps (decode_stack.hip).
#pragma once

#include "percache_internal.hpp"

namespace pc {
namespace stackdec {

constexpr int kWaves = 8;            // wavefronts of a workgroup
constexpr int kRing = 64 * 1024;     // LDS of a workgroup's weights in flight, or of two K/V tiles
constexpr int kMaxRows = 4;          // token rows
constexpr int kMaxQueryRows = 16;    // query rows per kv head
constexpr int kMaxLayers = 32;       // per launch (their pointers are launch arguments)

struct LayerPtrs {
  const __bf16 *gain1, *wqkv, *wo, *gain2, *w_gate, *w_up, *w_down, *qkv_bias, *q_norm, *k_norm;
};

struct Args {
  LayerPtrs w[kMaxLayers];
  // handed over: the blocks of a layer (n_*: their elements), those of the next one s_word words of 4 bytes further on
  __bf16 *h;              // the layer's input [M, H]
  float *h_b;             // and in blocks for the norm in front
  __bf16 *mid;            // the same between attention and ffn
  float *mid_b;
  float *qsum, *part;
  __bf16 *attn, *act;
  __bf16 *h_out;          // takes the rows of layer out_layer
  const __bf16 *gain_after;   // gain1 of the layer behind this launch's last
  __bf16 *k_dense, *v_dense;
  const int32_t *table, *append;
  const float2 *rope;
  unsigned *ticket;
  __bf16 *k16, *v16;
  const uint8_t *k8, *v8;
  const float *k_scale, *v_scale;
  size_t layer_stride, layer_stride8, scale_stride;
  size_t s_word, n_h, n_block, n_qsum, n_part, n_attn, n_act, l_kv;
  float eps, inv_h, scale_log2e;
  int M, T, H, Hq, Hkv, ffn, C, n_slots16, tbl_stride, n_splits, n_layers, out_layer;
  int n_q, n_t, n_x, n_o, n_g, per_layer;   // items of a layer
  int n_items;                              // of this launch
  int x_bytes, x_share_log2;                // LDS of a wavefront's token rows; lanes that share 8 columns in the merge
};

// Workspace of a step through n_layers layers over queries of at most max_tiles cached 64-key tiles (0: the shape does not take this path).
size_t workspace_bytes(const percache_config &c, int n_cu, int32_t batch, int32_t t_fresh, int32_t ffn, int n_layers, int max_tiles);
// Whether a step through n_layers layers over queries of at most max_tiles cached 64-key tiles takes it.
bool takes(const percache_config &c, int n_cu, int32_t batch, int32_t t_fresh, int32_t ffn, int n_layers, int max_tiles);
// The step.  rows: the chunk lists and, behind them, (slot, tokens) per query if append.  table: where they go (with_rows) or stand.
pc_status launch(percache_ctx *ctx, const percache_block_weights *layers, int n_layers, int ffn, float eps, const __bf16 *h_in, int batch, int t_fresh,
                 const std::vector<int32_t> *rows, int32_t *table, int tbl_stride, bool append, int max_tiles, int formats, __bf16 *h_out, void *ws,
                 const __bf16 **k_dense, const __bf16 **v_dense, size_t *dense_stride, hipStream_t stream);

}  // namespace stackdec
}  // namespace pc
