// decode_internal.h -- host-side geometry and launcher of the parallel-stream decode
// kernels inside libhd.so (sfa_decode_bf16.hip).
#pragma once

#include "hd_internal.h"

namespace hd {

struct DecGeom {
    int B, Lcap, n, Hq, Hkv, D, G;
    int mode;          // 0 intra, 1 full cross-stream, 2 local cross-stream
    int window;        // local layers: positions p - window < p' <= p; else a huge value
    int max_ctx;       // bound on the contexts
    float scale_log2;  // scale * log2(e)
    int gchunk;        // query heads per problem (their query slots fit 32 MFMA columns)
    int ngc;           // head chunks per key/value head, G / gchunk
    int nchunk;        // 256-row chunks of the cache per problem (for the longest context)
    int nsplit;        // workgroups per problem (for the longest context), at most nchunk
    int problems;      // B * Hkv * ngc (* n for intra-stream layers)
    int nslot;         // query slots per problem: gchunk (intra-stream) or n * gchunk
    int waves;         // per workgroup of the partial kernel: 2, 4 or 8
    int heads;         // neighbouring key/value heads that one XCD takes together
    int single;        // cached rows up to which one workgroup takes a whole problem
};

// Split of a problem's cached rows over workgroups.  Up to `single` rows one workgroup takes
// them all, with no combine pass.  Beyond, they go in equal parts to as many workgroups as
// leave all problems together no more of them than the chip holds at once (kDecTarget at D=128:
// two per CU), in whole tiles and at least kDecChunk rows each (the workspace has room for
// that many partials).  16 sequences x 4096 tokens, n=4, 32/8 heads of 128, full cross-stream:
// 177 us with 512 workgroups, 192 with 1024, 199 with 2048 (more partials, and more prologues
// that load nothing), 243 with one per 256 rows.  Rounded up instead, the workgroups beyond 512
// run after the others (144 problems of up to 5619 rows: 88.5 us with 4 splits, 69 with 3).
// Between target / 2 and 2 * target problems long ones go in parts of kDecWhole rows at most, so
// that contexts of different lengths even out (320 problems of up to 4096 rows, D=128: 120 us
// whole, 106 in parts; 832 of up to 4796, D=64: 187 and 138; 768 of 2501 rows, D=128, 180 and
// 173), but not where whole ones about fill the chip (512 of 4096 rows: 175 and 185); with more
// the chip goes through several rounds of whole ones.  At D=32, where two heads' rows share a
// line, the parts are of kDecChunk rows (1280 problems of 3001 rows: 188 us whole, 157 in
// parts of 1024, 106 in parts of 256).
constexpr int kDecChunk = 256;
constexpr int kDecTarget = 512;
__host__ __device__ inline int dec_target(int D) { return kDecTarget * (128 / D); }
constexpr int kDecWhole = 1024;
__host__ __device__ inline int dec_splits(int problems, int D, int single, int rows)
{
    const int target = dec_target(D);
    if (rows <= single || (D > 32 && problems >= 2 * target)) return 1;
    if (D > 32 && problems <= target && problems >= target / 16 * 15) return 1;
    const int splits = target / problems;
    const int whole = D > 32 ? kDecWhole : kDecChunk;
    if (splits <= 1) return (rows + whole - 1) / whole;
    const int by_rows = (rows + kDecChunk - 1) / kDecChunk;
    return by_rows < splits ? by_rows : splits;
}
__host__ __device__ inline int dec_split_rows(int problems, int D, int single, int rows)
{
    const int splits = dec_splits(problems, D, single, rows);
    const int per = (rows + splits - 1) / splits;
    return splits == 1 ? rows : (per > kDecChunk ? (per + 63) / 64 * 64 : kDecChunk);
}

// Neighbouring key/value heads that one XCD takes together.  At D=32 two heads' rows share a line,
// and on large grids their lying side by side counts as well, so up to eight (D=32, 16 sequences x
// 4096 rows x 4 streams: 50 us, 87 a head at a time; D=64, 1280 problems of 3000 rows: 164 and 182);
// below, single heads spread a step better (D=64, 128 problems of 16384 rows: 98 and 106).
inline int dec_heads(int problems, int D, int Hkv)
{
    int h = D == 32 || problems > 256 ? 8 : 1;
    while (Hkv % h) h /= 2;
    return h;
}

// Waves per workgroup and `single`, from the most rows that the cache can hold (and not from
// the bound on this call's contexts, so that a sequence's result does not depend on it):
//   8 waves, one tile in flight each, where at most one problem per CU has at most 1024
//     rows: the whole problem in one launch (D=128, launch to launch: 256 problems x 501 rows
//     22.1 us in 2 splits, 15.5 in one; x 1001 rows 32 and 26.5; 128 x 801 rows 18.6 and
//     15.9).  With 64 problems or fewer the split's larger grid wins earlier (64 x 516 rows
//     15.8 and 14.7, 32 x 764 rows 15.1 and 15.6);
//   4 waves, two tiles in flight each, where that leaves at most one workgroup per CU: few
//     rows in all, whose latency counts (8 problems x 3112 rows: 16.1 us against 19.3);
//   2 waves else: two workgroups per CU overlap each other's prologue and merge (32 problems
//     x 4096 rows 20.0 us against 22.5, 32 x 8004 rows 35 against 48).
inline void dec_shape(int problems, int D, int cap_rows, int &waves, int &single)
{
    const int most = problems <= 64 ? 640 : 1024;
    const bool few = problems <= 256 && cap_rows <= most;
    single = few ? most : 384;
    const int64_t wgs = (int64_t)problems * dec_splits(problems, D, single, cap_rows);
    waves = few ? 8 : wgs <= dec_target(D) / 2 ? 4 : 2;
}

// Cached rows of a problem that some query row of it sees: [klo, kvlen), the first one
// rounded down to a tile of kDecTile; they are split over workgroups, `per` rows each.  A
// context outside [0, max_ctx], for which neither grid nor workspace is made, counts as the
// nearest one inside.
constexpr int kDecTile = 32;  // cached rows per wave and step
struct DecRows {
    int ctx, klo, kvlen, per;
};
__host__ __device__ inline DecRows dec_rows(const DecGeom &g, int ctx)
{
    DecRows r;
    r.ctx = ctx < 0 ? 0 : ctx > g.max_ctx ? g.max_ctx : ctx;
    r.kvlen = g.mode == 0 ? r.ctx + 1 : (r.ctx + 1) * g.n;
    const int lo = r.ctx * g.n - g.window + 1;  // first position in the window of stream 0
    r.klo = (g.mode == 2 && lo > 0 ? lo : 0) / kDecTile * kDecTile;
    r.per = dec_split_rows(g.problems, g.D, g.single, r.kvlen - r.klo);
    return r;
}

// A problem and its query slots: cross-stream layers: slot = s * gchunk + head-in-chunk (all
// streams of the token); intra-stream layers: one problem per stream, slot = head-in-chunk.
struct DecProblem {
    int b, hk, gc, s;
};

__host__ __device__ inline int dec_index(const DecGeom &g, const DecProblem &r)
{
    return ((r.b * g.Hkv + r.hk) * g.ngc + r.gc) * (g.mode == 0 ? g.n : 1) + r.s;
}

// Workgroup id -> problem and split.  Ids go round-robin over the 8 XCDs; `heads` neighbouring
// key/value heads, whose rows share lines or lie side by side, follow each other on one XCD, and
// such units are dealt out over the XCDs split by split, so that splits past the end of a short
// context leave no XCD out.  False: no work.
__host__ __device__ inline bool dec_place(const DecGeom &g, int id, DecProblem &r, int &split)
{
    const int j = id >> 3, unit = (j / g.heads << 3) + (id & 7), units = g.problems / g.heads;
    split = unit / units;
    if (split >= g.nsplit) return false;
    int p = unit % units;
    r.s = 0;
    if (g.mode == 0) {
        r.s = p % g.n;
        p /= g.n;
    }
    r.gc = p % g.ngc;
    p /= g.ngc;
    const int sets = g.Hkv / g.heads;
    r.hk = p % sets * g.heads + j % g.heads;
    r.b = p / sets;
    return true;
}

// workgroup ids that dec_place maps
inline int64_t dec_grid(const DecGeom &g)
{
    return ((int64_t)g.problems / g.heads * g.nsplit + 7) / 8 * 8 * g.heads;
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
