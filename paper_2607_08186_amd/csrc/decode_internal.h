// decode_internal.h -- host-side geometry and launcher of the parallel-stream decode
// kernels inside libhd.so (sfa_decode_bf16.hip).
#pragma once

#include "hd_internal.h"

namespace hd {

struct DecGeom {
    int B, Lcap, n, Hq, Hkv, D, G;
    int mode;          // 0 intra, 1 full cross-stream, 2 local cross-stream
    int window;        // local layers: positions p - window < p' <= p; else a huge value
    float scale_log2;  // scale * log2(e)
    int gchunk;        // query heads per problem (their query slots fit 32 MFMA columns)
    int ngc;           // head chunks per key/value head, G / gchunk
    int nchunk;        // 256-row chunks of the cache per problem (for the longest context)
    int nsplit;        // workgroups per problem (for the longest context), at most nchunk
    int problems;      // B * Hkv * ngc (* n for intra-stream layers)
    int nslot;         // query slots per problem: gchunk (intra-stream) or n * gchunk
};

// Rows per workgroup of a problem with `rows` cached rows to read.  Up to kDecSingle rows one
// workgroup takes them all, with no combine pass (300 rows of 32 problems at D=128: 13.0
// against 14.5 us; 778 rows 16.8 against 14.1).  Beyond, the rows are spread so that all
// problems together make about as many workgroups as the chip holds at once
// (kDecTarget at D=128: two per CU), in whole tiles of four waves and at least kDecChunk
// rows each (the workspace has room for that many partials).  16 sequences x 4096 tokens,
// n=4, 32/8 heads of 128, full cross-stream: 177 us with 512 workgroups, 192 with 1024, 199
// with 2048 (more partials, and more prologues that load nothing), 243 with one per 256 rows.
constexpr int kDecChunk = 256;
constexpr int kDecSingle = 384;
constexpr int kDecTarget = 512;
__host__ __device__ inline int dec_target(int D) { return kDecTarget * (128 / D); }
__host__ __device__ inline int dec_split_rows(int problems, int D, int rows)
{
    if (rows <= kDecSingle) return kDecSingle;
    const int target = dec_target(D);
    const int64_t per = ((int64_t)rows * problems + target - 1) / target;
    return per <= kDecChunk ? kDecChunk : (int)((per + 127) / 128 * 128);
}
// upper bound of the splits over all sequences of at most `rows` rows
inline int dec_max_splits(int problems, int D, int rows)
{
    if (rows <= kDecSingle) return 1;
    const int by_rows = (rows + kDecChunk - 1) / kDecChunk;
    const int by_target = (dec_target(D) + problems - 1) / problems;
    return by_rows < by_target ? by_rows : by_target;
}
// Four waves per workgroup in place of two where that still leaves one workgroup's place per CU:
// few rows in all, whose latency counts (8 problems x 3112 rows 16.1 against 19.3 us);
// with more, two workgroups of two waves overlap each other's prologue and merge (32 x 4096
// rows 20.0 against 22.5, 32 x 8004 rows 35 against 48).
inline bool dec_wide(int problems, int D, int nsplit)
{
    return (int64_t)problems * nsplit <= dec_target(D) / 2;
}

DecGeom make_dec_geom(int B, int Lcap, int n, int Hq, int Hkv, int D, int mode, int window,
                      float scale, int max_ctx);
size_t decode_workspace_bytes(const DecGeom &g);
hipError_t launch_decode_bf16(const void *q, const void *kc, const void *vc, const int32_t *ctx,
                              void *o, float *lse, const DecGeom &g, void *ws, hipStream_t s);

// Library-owned scratch for the decode partials of callers that cannot allocate: a
// device array of kDecodeScratchBytes per GPU, held until the process ends and shared
// by every such call on that GPU.  decode_scratch returns its address on the current
// device (looked up once per device).
constexpr size_t kDecodeScratchBytes = (size_t)128 << 20;
hipError_t decode_scratch(void **ptr);

}  // namespace hd
