// Launchers of the small kernels of the verify step (see step_kernels.hip).
#pragma once
#include "../../include/cerberus.h"
#include "common.h"

namespace cerb {

struct Dims {
  int n_layers, d, nH, dh, F, Fpad, V, Hc, R, sb, dtype, Bmax, cap, topk, T;
  int R64;  // rows allocated per activation plane
  float eps, threshold;
};

enum { ASSEMBLE_BY_FLAG = 0, ASSEMBLE_FORCE_AR = 1, ASSEMBLE_FULL_TREE = 2, ASSEMBLE_PROMPT = 3 };

// Prompt pass: sequence `seq` runs `n` rows carrying tokens[0..n), every other sequence sits out.  The prompt counts in
// pieces of `piece` tokens (the last one may be shorter): a piece is committed whole, the first one that the cache has no
// room for ends the prompt (the rest of its pass and the passes after it commit nothing), and the output taps see the rows
// of the prompt's last piece, from slot 0 on.  A pass holds whole pieces; the `first` one starts the prompt, and `last` holds
// its last piece, whose rows alone go on to the LM head.
struct PromptArgs {
  const int* tokens;
  int n, seq, piece, first, last;
};

struct ResFinishArgs {
  const float* part[CERBERUS_MAX_HEADS];   // GEMM partials of head i: [S][16][width]
  const float* bias[CERBERUS_MAX_HEADS];   // fp32 [width]
  size_t pstride[CERBERUS_MAX_HEADS];
  int S[CERBERUS_MAX_HEADS];
  int width[CERBERUS_MAX_HEADS];
};

enum { TOPK_MAX_PARTS = 16 };               // vocabulary slices of 4096 entries: up to 65536
struct TopkArgs {
  const float* logits[CERBERUS_MAX_HEADS];  // head i: [16][V]
  const int* seq_T;                         // [B] rows of each sequence this step (0: sat out)
  float* part_v;                            // [Hc][B][TOPK_MAX_PARTS][CERBERUS_MAX_TOPK] best entries of every slice, in order
  int* part_i;
};

hipError_t launch_assemble(const Dims& D, const TreeDev& tr, const RowMap& rm, const cerberus_state& st,
                           const cerberus_taps& tp, int batch, int mode, const PromptArgs& pa, const AttnPlanCfg& ap, hipStream_t s);
// after the layers of a prompt pass: commits the rows; in the last pass the row map becomes that of the tail rows
hipError_t launch_prompt_commit(const RowMap& rm, const cerberus_state& st, int* last_row, int batch, int seq, int last_pass,
                                hipStream_t s);
// after the LM head of the last pass: the pending token
hipError_t launch_prompt_root(const cerberus_state& st, const int* g, const int* last_row, int seq, hipStream_t s);
// also fills rope_cs[row][j] = (cos, sin)(pos(row) * inv_freq[j]), j < dh/2, the angle formed in double
hipError_t launch_embed(const Dims& D, const RowMap& rm, const void* embed, float* x, const double* inv_freq, float2* rope_cs,
                        int rows_max, hipStream_t s);
// S_dev: if set, the number of partial planes is read from there (at most S)
hipError_t launch_add_rmsnorm(const Dims& D, const RowMap& rm, float* x, const float* part, int S, const int* S_dev, size_t pstride,
                              const float* gain, void* out, float* out_f32, float* tap, const int* src0, int rows_max, hipStream_t s);
// How a GEMM input lies in memory: row-major planes, or MFMA A-fragment order (bf16; see FusedQkvArgs and TileGemmArgs)
enum { A_ROWS = 0, A_FRAG64 = 1, A_FRAG = 2 };
// residual add + x * gain + per-block sums of x^2 (the RMSNorm scalar is applied by the consumer of the next GEMM)
int add_gain_blocks(int d, int order);   // sums per row
hipError_t launch_add_gain(const Dims& D, const RowMap& rm, float* x, const float* part, int S, const int* S_dev, size_t pstride,
                           const float* gain, void* out, float* ssq, int rows_max, hipStream_t s, int order = A_ROWS);
hipError_t launch_rope_kv(const Dims& D, const RowMap& rm, const float* part, int S, size_t pstride,
                          const float2* rope_cs, void* q, void* kv_layer, void* ktree, void* vtree, const float* ssq,
                          int rows_max, hipStream_t s);
// Whole-K GEMMs with fused epilogues (gemm_fused.hip), launches of up to 64 rows in bf16 mode.
// At: the GEMM input in MFMA A-fragment order, piece [((ks * 2 + plane) * 4 + mt) * 64 + lane] = the 8 values
// of row mt*16 + lane%16 at columns ks*32 + (lane/16)*8.., plane 0 = hi, 1 = lo (written by launch_add_gain
// in order A_FRAG64).  slabs: [grid][ns] 16-column slabs of every workgroup, -1 = none; positions (2p, 2p+1) form a pair.
struct FusedQkvArgs {
  const void* W;            // [3d][K] in the stream order of this kernel's grid and slab table (launch_pack_stream)
  const void* At;
  const int* slabs;         // pairs: slabs i and i + dh/32 of a q or k head; or one or two v slabs
  int ksteps;               // padded K / 32
  const float* ssq;         // block sums of x^2 of the pending attention norm
  int nb;
  const float2* rope_cs;    // [rows][dh/2] (cos, sin) of every row's rotation angles (written by launch_embed)
  RowMap rm;
  bf16_t* q;                // [rows][d] hi, lo plane lo_off later
  bf16_t* kv_layer;         // [2][Bmax][nH][cap][dh]
  bf16_t* ktree;
  bf16_t* vtree;
  size_t lo_off;
  Dims D;
};
struct FusedGateUpArgs {
  const void* W;            // [2F][K] (gate rows first) in the stream order of this kernel's grid and slab table
  const void* At;
  const int* slabs;         // pairs: (gate slab s, up slab F/16 + s): the same 16 FFN columns
  int ksteps;
  const float* ssq;
  int nb, d;
  float eps;
  RowMap rm;
  bf16_t* act;              // [rows][Fpad] hi, lo plane lo_off later (launch_tile_gate_up, lo_off 0: fragment order, Fpad / 32 k-steps)
  size_t lo_off;
  int Fpad;
};
hipError_t launch_qkv_rope(const FusedQkvArgs& a, int ns, int grid, hipStream_t s);
hipError_t launch_gate_up_swiglu(const FusedGateUpArgs& a, int ns, int grid, hipStream_t s);
size_t fused_stream_pieces(int ns, int grid, int ksteps);   // 16-byte pieces of a stream-order weight copy
hipError_t launch_pack_stream(const void* packed, void* dst, const int* table, int ns, int grid, int ksteps, hipStream_t s);
// Whole-K GEMMs with fused epilogues for more rows (gemm_tile.h, bf16 mode).
struct TileGemmArgs {
  const void* W;            // pre-tiled weights: fragment (slab, k-step) is 1 KB at (slab * ksteps + ks) * 1024
  const void* A;            // fragment (row tile, k-step, plane) is 1 KB at ((mt * ksteps + ks) * 2 + plane) * 1024 (A_FRAG)
  int ksteps, pairs;        // padded K / 32 (a multiple of 8); slab pairs of the launch
  const int* n_rows;        // device row count; null: rows_cap rows
  int rows_cap;             // upper bound of it
  // launch_tile_planes
  int max_splits;           // most k ranges
  int* splits_out;          // how many the launch made is left here: planes for the consumer to sum
  size_t lda, lo_off;       // if lda: A is row-major [rows][lda] instead, the lo plane lo_off elements later
};
hipError_t init_tile_qkv();       // each once per device, before the first launch
hipError_t init_tile_gate_up();
hipError_t init_tile_planes();
int tile_plane_splits(int pairs, int ksteps, int grid, int most, bool rows);   // most k ranges whatever the row count; rows: A is row-major
// out[k range][row][pairs * 32]
hipError_t launch_tile_planes(const TileGemmArgs& a, float* out, size_t pstride, int grid, hipStream_t s);
hipError_t launch_tile_qkv(const TileGemmArgs& a, const FusedQkvArgs& f, int grid, hipStream_t s);           // W, A, k-steps and rows: of a
hipError_t launch_tile_gate_up(const TileGemmArgs& a, const FusedGateUpArgs& g, int grid, hipStream_t s);
hipError_t launch_swiglu(const Dims& D, const RowMap& rm, const float* part, int S, size_t pstride, void* act,
                         const float* ssq, int rows_max, hipStream_t s);
hipError_t launch_row_argmax(const Dims& D, const RowMap& rm, const float* part, int S, size_t pstride, int* g,
                             const cerberus_taps& tp, int rows_max, hipStream_t s);
hipError_t launch_accept(const Dims& D, const TreeDev& tr, const RowMap& rm, const int* g, const int* tok,
                         const cerberus_state& st, int* path, int* last_row, int batch, hipStream_t s);
hipError_t launch_compact(const Dims& D, const RowMap& rm, const cerberus_state& st, const int* path, int batch,
                          hipStream_t s);
// entropy of `rows` vectors: vector r is forced[r] if forced != nullptr, else base[row_index ? row_index[r] : r];
// rows with seq_T[r] <= 0 (when seq_T != nullptr) are left untouched.
// Seeding of the decoding heads' stage-0 state by the gate launch; hsF == nullptr: none.
struct HeadsPrep {
  float* hsF;     // [Hc][16][2d] fp32 state
  void* hsA;      // same as the GEMM input type (bf16: lo plane lo_off elements later)
  size_t lo_off;
  int Hc, sb;     // number of heads; index of the special block
};
hipError_t launch_gate(int d, float threshold, const float* base, const int* row_index, const float* forced,
                       const int* seq_T, int rows, float* entropy, int* flag, const HeadsPrep& hp, int dtype, hipStream_t s);
hipError_t launch_resblock_finish(const Dims& D, const ResFinishArgs& a, const float* curF, float* nxtF, void* nxtA,
                                  int link_next, int batch, hipStream_t s);
hipError_t launch_topk(const Dims& D, const TopkArgs& a, const cerberus_state& st, const cerberus_taps& tp, int batch,
                       hipStream_t s);
hipError_t launch_log_tokens(const Dims& D, const cerberus_state& st, int batch, int* out, int cap, int* count,
                             hipStream_t s);
hipError_t launch_to_f32(const void* in, float* out, int n, int dtype, hipStream_t s);

}  // namespace cerb
