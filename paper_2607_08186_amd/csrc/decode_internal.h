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
    int problems;      // B * Hkv * ngc (* n for intra-stream layers)
    int nslot;         // query slots per problem: gchunk (intra-stream) or n * gchunk
    int waves;         // per workgroup of the partial kernel: 8 or 4
    int heads;         // neighbouring key/value heads that one XCD takes together
    int single, fill, whole, part;  // see dec_splits
    int nsplit;        // workgroups per problem (for the longest context), at most nchunk
};

// Split of a problem's cached rows over workgroups.  It follows from the number of problems,
// the head dim and the sequence's own rows, and neither from the cache's capacity nor from the
// bound on the contexts: these change no bit of a result, and no short context pays for a large
// cache (D=128, launch to launch, 32 to 256 problems of 100 to 1000 rows in a cache of 4096:
// 10.7 to 22 us, as in a tight one; shaped by the capacity they took 14.7 to 28.6).
//   Workgroups: eight waves, one workgroup per CU, up to 256 problems at D=128; half of that each
//     beyond (256 CUs; 264 problems of 700 rows 23.6 -> 22.7 us) and, where a tile is half the
//     bytes or less, from 65 problems on (D=64: 96 of 2000 rows 18.9 -> 15.5).
//   Up to `single` rows one workgroup takes a problem, and where that holds for all of them the
//     combine is not launched (64 problems x 499 rows 11.4 us, 14.8 in parts; 256 x 1000 rows 22 and
//     32; but 32 x 777 rows are faster in parts, 13.8 and 15.6).
//   Beyond, at least `fill` parts, with which all problems together fill the chip once, of at
//     least kDecChunk rows each (the workspace has room for that many partials).  More of them
//     mean more prologues and partials (16 x 4096 tokens, n=4, 32/8 heads of 128, full
//     cross-stream: 169 us in 2 parts, 174 in 4).
//   Above 256 problems parts of at most `part` rows even out contexts of different lengths and
//     the last round of workgroups (264 problems of 6000 rows at D=128: 149 us, 182 whole; 560 of
//     4500 at D=64: 106 and 142), and at D=64 above 128, where `fill` is 4 to 7 parts that do not
//     fill the 1024 places (208 problems of 12000 rows 127 -> 116 us, of up to 12000 108 -> 98;
//     136 of 9000 64 -> 60).  So do they where `fill` is one part for 129 to 170 problems, a
//     third of the CUs or more idle, in long contexts (`whole`; 160 of up to 6000 rows, D=128: 70
//     us, 80 whole; but 184 of 6000 rows 109 and 93).  Not at D=128 where whole ones fill seven
//     eighths or more of the 512 places (448 of 4500 rows: 175 us in parts, 166 whole; 512 of
//     4096: 172 and 165; 384 of 4500: 149 and 154).
constexpr int kDecSlots = 8;  // waves that a CU holds at D=128, each with a K and a V tile in LDS
constexpr int kDecChunk = 256;
__host__ __device__ inline int dec_splits(const DecGeom &g, int rows)
{
    if (rows <= g.single) return 1;
    const int by_rows = (rows + kDecChunk - 1) / kDecChunk;
    const int parts = rows <= g.whole ? 1 : (rows + g.part - 1) / g.part;
    const int want = parts > g.fill ? parts : g.fill;
    return want < by_rows ? want : by_rows;
}
__host__ __device__ inline int dec_split_rows(const DecGeom &g, int rows)
{
    const int splits = dec_splits(g, rows);
    const int per = (rows + splits - 1) / splits;
    return splits == 1 ? rows : (per > kDecChunk ? (per + 63) / 64 * 64 : kDecChunk);
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
    r.per = dec_split_rows(g, r.kvlen - r.klo);
    return r;
}

// Shape of the launch (see dec_splits), for problems of at most `rows` visible rows.
//   heads: at D=32 two heads' rows share a line, and on large grids their lying side by side
//     counts as well, so one XCD takes up to eight neighbouring heads together (D=32, 16 sequences
//     x 4096 rows x 4 streams: 50 us, 87 a head at a time; D=64, 1280 problems of 3000 rows: 164 and
//     182); below, single heads spread a step better (D=64, 128 problems of 16384 rows: 98 and 106).
inline void dec_launch(DecGeom &g, int rows)
{
    const int P = g.problems;
    g.waves = P <= (g.D == 128 ? 256 : 64) ? 8 : 4;
    g.single = P <= 64 ? 640 : P <= 256 ? 1024 : 384;
    g.fill = kCus * (kDecSlots / g.waves) * (128 / g.D) / P;
    g.part = g.D == 128 ? 2048 : 1024;
    g.whole = P > 256 || (g.D == 64 && P > 128) ? g.part : 1 << 30;
    if (g.D == 128 && P > 128 && P <= 170) g.whole = 4096;
    if (g.D == 128 && P >= 448 && P <= 512) g.whole = 1 << 30;
    g.heads = g.D == 32 || P > 256 ? 8 : 1;
    while (g.Hkv % g.heads) g.heads /= 2;
    g.nsplit = dec_splits(g, rows);  // grows with the rows
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
