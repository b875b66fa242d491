// launch.h -- host-side launchers of the libmxattn kernels (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mxattn {

// Shared-scale rule of the MXFP4 quantizer.
// kRuleQmax is the ceil rule of a general boundary q (Boundary in
// device_common.h), a run-time argument of the quantizers.
enum Rule { kRuleOcp = 0, kRuleUos = 1, kRuleQmax = 2 };

// Query rows per workgroup of the fused attention kernel, and its KV tile
// B_c: the running maximum is updated once per kKvTile keys.
constexpr int kQueryTile = 128;
constexpr int kKvTile = 128;

hipError_t launch_quantize_headdim(const void* x, uint8_t* codes, uint8_t* scales, int64_t rows,
                                   int rule, hipStream_t stream, double qmax = 0.0);

// Q/K of the rotated mode: rows multiplied by R_H = H/sqrt(128) first.
hipError_t launch_quantize_headdim_rotated(const void* x, uint8_t* codes, uint8_t* scales, int64_t rows,
                                           int rule, hipStream_t stream);

hipError_t launch_quantize_tokens(const void* x, uint8_t* codes, uint8_t* scales, int64_t BH,
                                  int64_t N, int rule, hipStream_t stream, double qmax = 0.0);

// The quantized operands of a forward call, in the attention kernel's layouts
// (AttnArgs), in one launch: K^, V^ and their scales; Q^ too where q is not
// null (the rotated mode).
struct PrepareArgs {
    const uint4 *q, *k, *v;  // bf16 [BH, Nq or N, 128]
    uint8_t *qc, *qs;        // [BH, Nq, 64], [BH, Nq, 4]
    uint8_t* kc;             // [BH, N, 64]
    uint8_t* vc;             // [BH, ntiles, 128, vrow]
    uint8_t* sc;             // [BH, ntiles, 1024]
    int64_t BH;
    int N, Nq, ntiles;  // tiles of 128 tokens of a head
    int vrow;           // v_tile_row_bytes(N)
    int64_t first;      // set by the launcher: first workgroup of a launch
};
// Bytes of a channel in a tile of V^ codes stored tile by tile: those of the tile's
// four blocks, or of the blocks that there are in a head shorter than a tile (one
// block: 2 KiB per head instead of 8).
inline int v_tile_row_bytes(int64_t N) { return N > 96 ? 64 : (int)((N + 31) / 32) * 16; }
hipError_t launch_prepare_operands(const PrepareArgs& a, int rule, bool rotated, hipStream_t stream);

// Per-head squared-error sweep over boundaries (qmax.hip).  The histogram
// pass writes partial sums to a workspace of qmax_sse_workspace_bytes(...)
// bytes; the reduction turns them into sse[BH, nq] (fp64).
constexpr int kMaxBoundaries = 64;
int64_t qmax_sse_workspace_bytes(int axis, int64_t BH, int64_t N);
hipError_t launch_qmax_sse(const void* x, int axis, const double* qs, int nq, double* sse,
                           void* workspace, int64_t BH, int64_t N, hipStream_t stream);

struct AttnArgs {
    const uint8_t* qc;  // [BH, Nq, 64]
    const uint8_t* qs;  // [BH, Nq, 4]
    const uint16_t* qraw;  // bf16 Q [BH, Nq, 128] if the kernel quantizes Q itself, else null
    const uint8_t* kc;  // [BH, N, 64]
    const uint8_t* vc;  // V^ codes: channel d of tile t at head * vhead + t * vtile + d * vrow, 64 B (16 B per block)
    const uint8_t* sc;  // [BH, ntiles, 1024]: K^ and V^ scales in MFMA operand order
    uint16_t* out;      // [BH, Nq, 128] bf16
    int N;              // keys / values per head
    int Nq;             // queries per head (Q^ codes/scales and out are [BH, Nq, ...])
    int vrow, vtile, vhead;  // bytes; [BH, 128, nb * 16] or [BH, ntiles, 128, v_tile_row_bytes]
    int qtiles;
    int total_tiles;    // workgroups that do work
    int per_xcd;
    int nchunks;        // resident kernel: workgroups per (batch, head)
    int nsplit;         // runs the keys of a head are divided into (1: not divided), and their workspace:
    int score_parts;    // parts of a run in the pass over the scores
    float* run_max;     // [BH, qtiles, nsplit * score_parts, 128]: largest score of a part
    float2* part_ml;    // [BH, qtiles, nsplit, 128]: m and l after a run
    float4* part_o;     // [BH, qtiles, nsplit, 4 waves, 16, 64 lanes]: O~ of a run
};

// Runs the keys of a head are divided into, from the shape alone (so every
// entry point divides alike): see attention.hip.
int key_splits(int64_t BH, int64_t Nq, int64_t Nkv);
// Workspace of a divided call: at most kMaxSplitWorkgroups workgroups' worth.
constexpr int kMaxSplitWorkgroups = 512;
constexpr int kScoreParts = 4;  // at most
constexpr size_t kSplitBytesPerWorkgroup = 128 * (128 * 4 + 8 + 4 * kScoreParts);
inline size_t split_bytes(int64_t BH, int64_t Nq, int nsplit) {
    return nsplit <= 1 ? 0 : (size_t)(BH * ((Nq + kQueryTile - 1) / kQueryTile) * nsplit) * kSplitBytesPerWorkgroup;
}

// Largest key (and value) length of the fused attention kernel: one head's
// K^ codes (64 B per key) and V^ codes (128 channels x 16 B per 32 keys) are
// addressed through buffer resources with 32-bit byte offsets, which stay
// below 2^31 up to this length.
constexpr int64_t kMaxKeys = (int64_t)1 << 24;

// Keys up to which the whole of K^ and V^ of a head stays in LDS for the
// workgroup's lifetime (launch_attention then runs the resident kernel).
constexpr int kResidentKeys = 512;

// Scales of K^ and V^ in the attention kernel's operand order (AttnArgs::sc);
// out holds tile_scales_bytes(BH, N) bytes.
inline int64_t tile_scales_bytes(int64_t BH, int64_t N) { return BH * ((N + 127) / 128) * 1024; }
hipError_t launch_tile_scales(const uint8_t* ks, const uint8_t* vs, uint8_t* out, int64_t BH, int64_t N,
                              hipStream_t stream);

// Row-sum diagnostics (rowsum.hip).  Attention rows [row0, row0 + rows) of
// every head: either p [BH, rows, ld] fp32 stored, or their quantization
// statistics written to stats [BH, Nq, 8] (fp64).
enum RowsOut { kRowsStoreP = 0, kRowsDiagUos = 1, kRowsDiagOcp = 2 };
struct SoftmaxRowsArgs {
    const uint16_t* q;  // [BH, Nq, 128] bf16
    const uint16_t* k;  // [BH, Nkv, 128] bf16
    float* p;           // [BH, rows, ld] (kRowsStoreP)
    int Nq, Nkv, row0, rows, ld;
    float gamma;        // pre-scale (diagnostics)
    double g;           // fp64(1 / gamma)
    double* stats;      // [BH, Nq, 8] (diagnostics)
    int qtiles, runs;   // set by the launcher: row tiles, runs of key tiles
    float c;            // set by the launcher: log2(e) / sqrt(128)
};
hipError_t launch_attn_rows(const SoftmaxRowsArgs& a, int64_t BH, int out, hipStream_t stream);

// Diagnostics of rows of p [n_rows, ld] (first N entries), written to
// stats[((r / rows_per_head) * out_rows_per_head + out_row0 + r % rows_per_head) * 8 + i].
struct RowsumDiagArgs {
    const float* p;
    int64_t N, ld;
    float gamma;  // pre-scale
    double g;     // fp64(1 / gamma)
    double* stats;
    int64_t rows_per_head, out_rows_per_head, out_row0;
};
hipError_t launch_rowsum_diag(const RowsumDiagArgs& a, int64_t n_rows, int rule, hipStream_t stream);

// mode: 0 OCP + direct, 1 UOS + direct, 2 UOS + PNQ
hipError_t launch_attention(const AttnArgs& a, int mode, hipStream_t stream);

}  // namespace mxattn
