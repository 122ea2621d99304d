// Launch wrappers of the gfx950 kernels (host side).  All pointers are device pointers.
#ifndef SS_KERNELS_H
#define SS_KERNELS_H

#include <hip/hip_runtime.h>

#include <cstdint>

#include "ss_plan.h"

namespace ss {

typedef uint16_t bf16_t;  // bf16 bit pattern (source tensors, embedding rows, norm gains)
typedef uint16_t f16_t;   // IEEE half bit pattern: both operands of every projection (packed weights, packed activations)
typedef uint16_t kv_t;    // key/value cache slot: IEEE half bit pattern

// Packed weight matrix: N output rows (multiple of 16), K inputs padded to Kp (multiple of 64).
struct PackedMat {
    f16_t* p = nullptr;
    void* pn = nullptr;   // the same values in the 12-bit form, or null (see k_narrow_weight)
    int N = 0, K = 0, Kp = 0;
};

// Per-micro-batch device state read and written by the kernels, so that one decode step can be
// replayed without any host-side scalar changing.
struct MbState {
    int32_t* d_n;        // [1] token-rows of the next forward
    int32_t* d_step;     // [1] tokens generated so far by every live row (rows advance in lockstep)
    int32_t* tr_tok;     // [n_max] token id fed by token-row j
    int32_t* tr_row;     // [n_max] micro-batch row of token-row j
    int32_t* tr_pos;     // [n_max] position of token-row j inside its row
    int32_t* live_row;   // [B]     rows still in the live batch, in slot order
    int32_t* d_nlive;    // [1]
    int32_t* d_active;   // [1] rows that still owe tokens after the last bookkeeping step
    int32_t* row_plen;   // [B] prompt length
    int32_t* row_j0;     // [B] first token-row of the row in a prompt forward
    int32_t* row_limit;  // [B] min(target, cap): tokens the row emits; lowered by the device when the row emits its end id
    const int32_t* row_stay;   // [B] or null: forwards that the row takes part in (micro-batches that share theirs)
    int64_t* row_so;     // [B] first key/value slot of the row's slab
    int32_t* row_cap;    // [B] slots in the row's slab (prompt + cap)
    int32_t* am;         // [n_sel_max] argmax of the selected rows' logits
    int32_t* out_tok;    // [B][max_new]
    int32_t max_new;
};

constexpr size_t kZeroBlkBytes = 4096;   // a 12-bit group (3 KiB) or an operand block (1 KiB)

struct GemmArgs {
    const f16_t* W;      // packed [N, Kp]
    const void* Wn;      // the same matrix in the 12-bit form; read instead of W when `narrow`
    const f16_t* X;      // packed [rows, Kp] activations
    float* out;          // EPI_PARTIAL: [ksplit][m_stride][N] fp32
    f16_t* out_packed;   // EPI_SWIGLU: packed [rows, kp_out], column f = silu(gate_f) * up_f
    int N, Kp, m_rows;   // m_rows: rows to compute (stores are guarded by it)
    int m_stride;        // row stride (in rows) between k-slices of `out`
    int kp_out;          // padded K of out_packed
    int ksplit;          // outer k-slices (gemm_plan)
    int nb, kd;          // skinny kernel shape (gemm_plan)
    int block;           // >= 0: block kernel with this tile (gemm_plan)
    int sweep_p;         // > 0: sweep kernel with this many waves per workgroup (gemm_plan)
    int sweep_gn;        //      its workgroups per k-slice
    int narrow;          // sweep and skinny kernels: read Wn (the plan allows it and the matrix has one)
    int sweep_kh;        //      2: two waves per unit, each half of every chunk's k-blocks (gemm_plan)
    const f16_t* zero_blk;   // kZeroBlkBytes of zeros: read in place of weights beyond a range (sweep kernel)
};

void launch_pack_weight(const void* src, int src_f32, f16_t* dst, int n_src, int k, int kp, int blk_stride,
                        int blk_off, int head_strips, hipStream_t s);
// Writes the 12-bit form of a packed [N, Kp] matrix (Kp a multiple of 128; narrow_strip); sets *unfit if a value has no such
// form.  dst == nullptr: only that.
void launch_narrow_weight(const f16_t* src, void* dst, int N, int Kp, int32_t* unfit, hipStream_t s);
void launch_cast_rows(const void* src, int src_f32, bf16_t* dst, size_t count, hipStream_t s);
void launch_embed(const MbState& st, const bf16_t* embed, float* x, int d, int n_max, hipStream_t s);
void launch_rmsnorm(const MbState& st, float* x, const float* part, int ksplit, size_t part_stride,
                    const bf16_t* w, float eps, const int32_t* sel, const int32_t* d_nsel, f16_t* h_packed, int d,
                    int n_max, hipStream_t s);
// Where an EPI_QKV launch puts its results: q rotated, fp32 [rows, d]; k rotated and v into the rows' slabs.
struct QkvOut {
    MbState st;
    float* qrot;
    kv_t *kc, *vc;
    const float *rcos, *rsin;
    int hd;
};

// EPI_QKV and EPI_RESIDUAL (out += sums) need a plan for the block kernel without k-slices; EPI_QKV needs `qkv`.
void launch_gemm(const GemmArgs& a, int epilogue, hipStream_t s, const QkvOut* qkv = nullptr);
// Up to kFewRows rows, 12-bit weights (few_plan).  EPI_PARTIAL and EPI_SWIGLU: of the normalised rows of x [n_rows, Kp]; EPI_PARTIAL: whole
// sums to out [n_rows, N]; EPI_RESIDUAL: of the packed rows X, added to out [n_rows, N].
struct FewArgs {
    const void* Wn;
    const float* x;
    const bf16_t* gain;
    const f16_t* X;
    float* out;
    f16_t* out_packed;
    FewPlan plan;
    int N, Kp, kp_out, units;   // units: strips, or pairs of them with EPI_SWIGLU
    float eps;
};
void launch_gemm_few(const FewArgs& a, int n_rows, int epilogue, hipStream_t s);
void launch_rope_append(const MbState& st, const float* qkv_part, int ksplit, size_t part_stride, float* qrot,
                        kv_t* kcache, kv_t* vcache, const float* rope_cos, const float* rope_sin, int d, int H,
                        int hd, int n_max, hipStream_t s);
// Causal attention of a prompt forward: B rows, row i holding st.row_plen[i] token-rows that start at token-row
// st.row_j0[i]; max_len = the longest row (sizes the grid).
void launch_attention_prompt(const MbState& st, const float* qrot, const kv_t* kcache, const kv_t* vcache,
                             f16_t* out_packed, int d, int H, int hd, int B, int max_len, hipStream_t s);
// n_max: rows of this launch; plan_rows, mb_rows, max_ctx: rows to choose its shape for (n_max, or those of one micro-batch
// of several), rows of the micro-batch, finished ones included, and an upper bound of its contexts in this forward (they
// choose the launch shape).  scratch: kWorkspaceRows rows of d floats (attention_split keeps to them).
void launch_attention_decode(const MbState& st, const float* qkv_part, int ksplit, size_t part_stride,
                             kv_t* kcache, kv_t* vcache, const float* rope_cos, const float* rope_sin,
                             f16_t* out_packed, int d, int H, int hd, int n_max, int plan_rows, int mb_rows,
                             int max_ctx, float* scratch, hipStream_t s);
// Decode steps of n_max rows (at most), one workgroup each, from the embedding to the logits of row j at logits + j * V and,
// with am, their argmax (row_step_plan says when).  steps > 0: greedy rows with known ends; each takes that many steps on its own
// tokens, or with `compact` those that it owes, and writes them out itself (the tables of live rows stay as they are).
struct RowStepArgs {
    struct Layer {
        const f16_t* w[4];   // q|k|v, o, gate|up, down
        const bf16_t *attn_norm, *mlp_norm;
    } layer[kRowMaxLayers];
    const bf16_t *embed, *final_norm;
    const f16_t* lm_head;
    kv_t* kv;                 // layer l: keys at kv + 2 * l * kv_layer_stride, values kv_layer_stride behind
    size_t kv_layer_stride;
    const float *rope_cos, *rope_sin;
    float* logits;
    int32_t* am;
    int n_layers, d, H, F, Fp, V;
    int steps, compact;
    float eps;
};
void launch_row_step(const MbState& st, const RowStepArgs& a, int hd, int n_max, hipStream_t s);
void launch_argmax(const float* logits, int vocab, const int32_t* d_nsel, int32_t* am, int n_max, hipStream_t s);
// Temperature sampling in place of the argmax: st.am[j] for the first *d_nsel selected rows.  The draw of slot j
// (row r = st.live_row[j], token number t = *st.d_step) is draws[r * st.max_new + t], or with draws == nullptr
// the counter-based generator's draw for (ids[r], t) under `seed`.
void launch_sample(const float* logits, int vocab, const int32_t* d_nsel, const MbState& st, const float* draws,
                   const int32_t* ids, uint64_t seed, float inv_temp, int n_max, hipStream_t s);
// eos_id: -1 when rows end only at their limit.
void launch_step_update(const MbState& st, int compact, int eos_id, hipStream_t s);
// Reads the first bytes/65536 chunks of 64 KiB at p and discards them (bandwidth probe).
void launch_read_stream(const f16_t* p, size_t bytes, uint32_t* sink, hipStream_t s);
void launch_fill_i32(int32_t* p, int32_t v, size_t n, hipStream_t s);

}  // namespace ss

#endif
