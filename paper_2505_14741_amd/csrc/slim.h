// Interface of slim.hip.
#pragma once
#include "common.h"

namespace ps {

struct SlimLayer { const float *W_qkv, *W_o, *W_1, *W_2, *b_qkv, *b_o, *b_1, *b_2; };
struct SlimArgs {
    const float *x, *ctx, *W_pe, *b_pe, *W_out, *b_out, *mod, *modf, *rope, *qkv;
    float *X, *qkv_out, *eps_out;
    long ctx_bs, mod_bs;
    PatchGeom pg;
    int tokens, text_tokens, head_dim, layer;
    float eps, scale;
};

// What slim.hip takes: fp32, hidden 32 or 64 in heads of 16 or 32, mlp_ratio 4, whole 16-value blocks of up to 64 values
// per patch, up to 1024 tokens.  us per forward of 2 layers, a launch per operation / this: hidden 64, 4 heads: 32 tokens 94 /
// 42, 416 tokens 112 / 55, 976 tokens 141 / 77 (16 samples 326 / 230).  A head of 64 keeps one wave per workgroup busy for
// long (416 tokens 156 / 183), and a hidden size of 128 has too much to do per token for one workgroup (416 tokens, 8 heads
// 135 / 143; both of when hidden 64 took 125 / 71).
constexpr int SLIM_TOKENS = 1024;
constexpr bool slim_network(int dtype, int hidden, int head_dim, int mlp_ratio, int patch_values, int tokens) {
    return dtype == PS_F32 && (hidden == 32 || hidden == 64) && head_dim <= 32 && mlp_ratio == 4 && patch_values % 16 == 0 &&
           patch_values <= 64 && tokens <= SLIM_TOKENS;
}

// A forward is launch_slim_begin and one launch_slim_layer per layer; the conditioning (mod, modf, rope) is there already.
// g.qkv_out: where the launch leaves the q, k, v [batch * tokens, 3 * hidden] of the layer that follows; g.qkv: where a
// layer's own were left, other memory (a workgroup's next ones must not overwrite keys others still read).
hipError_t launch_slim_begin(const SlimArgs& g, int hidden, const SlimLayer& first, int batch, hipStream_t st);
// layer number g.layer; next: the one after it, NULL after the last
hipError_t launch_slim_layer(const SlimArgs& g, int hidden, const SlimLayer& layer, const SlimLayer* next, int batch, hipStream_t st);

}  // namespace ps
