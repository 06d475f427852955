// Batched frozen-weight engine (batch.hip): forward, gradient sums and
// per-sample gradients of many samples layer by layer.  Plain data shared
// with the host API.
#pragma once

#include "chaos_internal.h"

namespace chaos {

// i / d for 32-bit i with i * d < 2^32 (every index here): one multiply-high
struct FastDiv {
    uint32_t m, d;
};

// One convolution or fully connected layer with the pooling layer after it.
// Activations live in memory as fp32 [sample][position][map]; a fully
// connected layer sees its input as one position with C = inputs channels
// (flat), in that order.
struct Stage {
    int C, H, W;            // input maps and map size (flat: H = W = 1)
    int O, K, Ho, Wo;       // output maps, kernel side (flat: 1), conv output size
    int p, Hp, Wp;          // pooling window side (1: none) and pooled size
    int flat;
    int P, Pp, T;           // conv positions, pooled positions, kernel positions
    int nin, nout;          // floats per sample in and out
    int prevP, prevC;       // flat: maps and positions of the flattened input
    int w_off, w_stride, b_off;  // weights W[o][...] and biases in the device layout
    int cw_off, cb_off;          // and in the canonical one
    // operand packs (bf16, three planes), in bf16 elements from the pack's start
    int C8, st;             // 8-channel chunks per position; bytes per staged position
    int O8, ost;            // the same of the output deltas
    int CT, KS;             // forward: column tiles, K steps of 32
    int KSO, RTB;           // backward data: K steps, row tiles
    int64_t fpack, bpack;
    // workspace per sample: floats before this stage's outputs, argmax bytes
    int64_t y_off, a_off;
};

struct BatchPlan {
    bool ok = false;
    int n_stages = 0;
    Stage s[kMaxLayers];
    int64_t pack_elems = 0;     // both packs of every stage
    int64_t act_floats = 0;     // y of every stage, per sample
    int64_t arg_bytes = 0;      // argmax of every pooled stage, per sample (multiple of 16)
    int last_c = 0, last_p = 0; // the output layer's maps and positions
};

// The engine's entry points are weak: the host API also builds alone, without
// the kernels (its argument checks under a sanitizer), and then has no engine.
#define CHAOS_WEAK __attribute__((weak))

// Whether and how the engine serves a net (geometry only).
CHAOS_WEAK void batch_plan(const Net &net, const ParamLayout &layout, BatchPlan &plan);

// Memory one call works in.
struct BatchWork {
    uint16_t *pack;        // plan.pack_elems
    float *act;            // samples * act_floats (y), then as many (errors) for gradients
    uint8_t *arg;          // samples * arg_bytes
    int64_t samples;       // samples per pass over the layers, a multiple of 4
    float *part;           // weight-gradient partial rows
    int64_t part_floats;   // floats there
};
// The workspace of `samples` samples (a multiple of 4) carved from buf.
inline BatchWork batch_work(const BatchPlan &plan, uint16_t *pack, void *buf, int64_t samples, bool grads) {
    BatchWork w{};
    w.pack = pack;
    w.act = static_cast<float *>(buf);
    w.arg = reinterpret_cast<uint8_t *>(w.act + samples * plan.act_floats * (grads ? 2 : 1));
    w.samples = samples;
    return w;
}

struct BatchCall {
    const float *params, *x;
    const int32_t *labels;
    int64_t n;
    float *out, *loss, *grad_sum, *grad_each;
    int32_t *n_wrong;
    int64_t n_params;
};

// Bytes of activation workspace per sample (forward only / with gradients).
CHAOS_WEAK int64_t batch_sample_bytes(const BatchPlan &plan, bool grads);
// Floats of partial rows that a gradient sum over n samples is best run with,
// and the fewest it can be run with.
CHAOS_WEAK int64_t batch_part_floats(const BatchPlan &plan, int64_t n);
CHAOS_WEAK int64_t batch_part_min(const BatchPlan &plan);
CHAOS_WEAK hipError_t launch_batch(const BatchPlan &plan, const BatchWork &w, const BatchCall &c, hipStream_t s);

// ---- training worker with its per-sample state in LDS (worker_lds.hip) ----
// One convolution or fully connected layer with the pooling layer after it;
// activations are [map][position], LDS offsets in floats.
struct LdsStage {
    int fc, C, H, W, O, K, Ho, Wo, p, Hp, Wp;
    int w_off, b_off;
    int y_off, arg_off, tab_off;  // outputs, argmax bytes, offsets of (map, kernel) in the input
};
struct LdsPlan {
    int n, in_size, n_out;
    int z_off, red_off, e_off[2];  // conv outputs / framed deltas; partial tiles; errors
    int64_t bytes;
    LdsStage s[kMaxLayers];
};
CHAOS_WEAK bool worker_lds_plan(const Net &net, LdsPlan &plan);
CHAOS_WEAK int worker_lds_blocks_per_cu(const LdsPlan &plan);
CHAOS_WEAK hipError_t launch_worker_lds(int mode, const LdsPlan &plan, const WorkArgs &a, int grid, hipStream_t s);

} // namespace chaos
