// The row-block form of the online update (update_rows.hip): arguments of its two launches.
#pragma once
#include "internal.hpp"

namespace ab {

// One matrix product of the rows launch: a layer forward, or backward (its weights used transposed).
struct RowsJob {
    const unsigned char *W;
    uint32_t ld;                             // bytes of a row of W
    uint16_t n_blk, n_slices;                // blocks of inputs (128 bytes of W's rows; backward 64 (fp32: 32) rows), 64-column slices
    uint16_t ks_shift, passes;               // narrow layers: 1 << ks_shift wavefronts share a slice's inputs; wide ones: passes
    uint16_t recip, back;                    // ceil(32 / n_slices) (n_slices <= 4); backward
};

struct RowsArgs {
    RowsJob job[2 * AB_MAX_HIDDEN - 1];      // filled by the launcher
    const void *x;                           // [Bp, l[0].in] transformed rows, zero in the padding
    struct L {
        const void *W; const float *b;       // [out, in], 16-byte aligned rows (layer 0: the padded copy); [out]
        void *h, *d;                         // [Bp, out] activations and deltas (d only from layer k0 on)
        int32_t in, out;                     // multiples of 64
    } l[AB_MAX_HIDDEN];
    const void *w_out; const float *b_out, *target;
    float *dout, *lossrow;                   // [Bp, n_out], [Bp]
    int64_t B;
    int32_t D, k0, n_out, loss_kind, n_jobs;
    int32_t o_even, o_odd, o_bias, o_wout, o_bout, o_tgt, o_mask, o_dout, o_scratch;     // LDS layout, filled by the launcher
};
// ... of blocks of 32 rows.  The kernel of 16 does without these fields and bytes: with them (and its opening through touch_arguments)
// a step of 200 rows of 54-64-64-1 in fp32 took 20.88 us instead of 20.76.
struct Rows32Args : RowsArgs {
    int32_t o_sums;                          // the output unit's partial sums
    uint32_t folds;                          // two bits a job: 1 << fold shares of the inputs one after the other in a wavefront, summed apart
};
static_assert(sizeof(RowsArgs) == 792, "what the kernel of 16 rows is passed");
static_assert(2 * (2 * AB_MAX_HIDDEN - 1) <= 32, "two bits a job");

struct GradsArgs {
    struct L {
        const void *d, *h_in;                // deltas [Bp, H], the layer's inputs [Bp, in_w]
        float *gw, *gb;                      // [splits, H, in_w], [splits, H]
        int32_t H, in_w, start;              // start: first tile of the layer
    } l[AB_MAX_HIDDEN];
    int32_t n, splits;
    int64_t B, Bp;
    const void *h_last; const float *dout, *lossrow;
    float *gw_out, *gb_out, *loss_out;       // (gb_out: [n_out]; loss_out may be NULL)
    int32_t H_last, n_out;
    int32_t out_splits;                      // of gw_out: [out_splits, n_out, H_last]
    unsigned n_out_blocks, n_tile_blocks;    // work-groups of the output unit's gradient, of the tiles (n_out + 1 between them)
};

// The gradients launch that takes the Adam step as well: each work-group has the whole batch of its part.
struct AdamTensor { float *w, *m, *v; void *wc; };                  // master, moments, compute-type copy (NULL for biases)
struct StepArgs {
    struct L {
        const void *d, *h_in;                // deltas [Bp, H], the layer's inputs [Bp, in_w]
        AdamTensor W, b;
        int32_t H, in_w, cols, start;        // cols: of W itself (layer 0's inputs are padded); start: first tile of the layer
    } l[AB_MAX_HIDDEN];
    int32_t n, n_tiles;
    int64_t B, Bp;
    const void *h_last; const float *dout, *lossrow;
    AdamTensor Wo, bo;
    float *loss_out;                         // may be NULL
    int32_t H_last, n_out;
    unsigned n_out_blocks;
    const float *scal;                       // {1 - beta1^t, 1 - beta2^t}
    float lr, beta1, beta2, eps;
};
hipError_t launch_update_step(int dtype, const StepArgs &a, hipStream_t st);

bool update_rows_supported(const RowsArgs &shape, int dtype);      // looks at D, n_out and the widths only
int update_rows32_fold(const RowsArgs &shape, int dtype);          // of blocks of 32 rows (for tests)
hipError_t launch_update_rows(int dtype, RowsArgs a, hipStream_t st);
hipError_t launch_update_grads(int dtype, int tile, const GradsArgs &a, hipStream_t st);     // tile: 64 or 128

}  // namespace ab
