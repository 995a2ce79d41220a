// embed_bwd.hip -- gradient of the multi-stream token expansion with respect to the
// n tables, and cyclic replication of the tables.
//
// The expansion of eq. (expansion) is a gather, out[b][t*n + s] = tables[s][ids[b][t]],
// so its gradient is a scatter-add: table s at token id x receives the sum of the
// upstream rows t*n + s of every token t with id x.  Done deterministically, without
// atomics on the data:
//   1. a stable sort of the (id, token position) pairs by id; ids outside [0, V) get
//      the key V and sort to the end.  Up to kSmallSortMax tokens the sorted position
//      of a token is counted directly (the number of tokens whose (key, position) is
//      smaller; one launch spread over M / 16 workgroups).  Up to kMidSortMax tokens an
//      LSD radix sort with 9-bit digits in two launches a pass; larger batches take 8-bit
//      digits (per-block digit histograms, one device-wide exclusive scan, then a
//      scatter in which every block ranks its chunk stably with eight 1-bit splits in
//      LDS);
//   2. the run starts of the sorted ids give the distinct ids in ascending order and
//      each run's index (token positions ascend within a run, as the sort is stable);
//   3. a gather-reduce over the sorted rows: the upstream rows of a run are summed in
//      fp32 in ascending token order (HBM-bound: every upstream row is read once, every
//      gradient row written once).
// The gradient comes out sparse, as (distinct ids, rows), so nothing scales with V;
// hd_embed_grad_scatter_add adds such rows into a dense fp32 table gradient.
//
// Cyclic replication, eq. (cyclic_init): when the expansion factor grows from n to m
// (a multiple of n), table s of the new set is table s mod n of the old one.
#include <algorithm>
#include <type_traits>

#include "embed_internal.h"
#include "hd_device.h"

namespace hd {

namespace {

constexpr int kThreads = 256;
constexpr int kItems = 8;
constexpr int kChunk = kThreads * kItems;  // keys per block in the scan and sort kernels
constexpr int kWaves = kThreads / 64;

// Exclusive scan of one int per thread across the workgroup; *total gets the sum.  `sh` is
// LDS scratch of kWaves + 1 ints.
__device__ inline int block_exclusive_scan(int x, int *total, int *sh)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int v = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(v, o);
        if (lane >= o) v += y;
    }
    if (lane == 63) sh[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        int acc = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int t = sh[w];
            sh[w] = acc;
            acc += t;
        }
        sh[kWaves] = acc;
    }
    __syncthreads();
    const int r = sh[wave] + v - x;
    *total = sh[kWaves];
    __syncthreads();  // sh may be reused right away
    return r;
}

// ---------------------------------------------------------------- device-wide scan
// Exclusive scan of x[0..n) (n <= kChunk * kChunk) in three launches: per-block sums,
// a one-block scan of the sums (the grand total goes to *total), per-block apply.

__global__ __launch_bounds__(kThreads) void scan_reduce_kernel(const int *__restrict__ x, int n,
                                                               int *__restrict__ sums)
{
    __shared__ int sh[kWaves + 1];
    const int64_t base = (int64_t)blockIdx.x * kChunk + threadIdx.x * kItems;
    int acc = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j)
        if (base + j < n) acc += x[base + j];
    int total;
    block_exclusive_scan(acc, &total, sh);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kThreads) void scan_top_kernel(int *__restrict__ sums, int nb,
                                                            int *__restrict__ total)
{
    __shared__ int sh[kWaves + 1];
    const int base = threadIdx.x * kItems;
    int v[kItems], acc = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        v[j] = base + j < nb ? sums[base + j] : 0;
        acc += v[j];
    }
    int tot;
    int run = block_exclusive_scan(acc, &tot, sh);
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        if (base + j < nb) sums[base + j] = run;
        run += v[j];
    }
    if (threadIdx.x == 0 && total != nullptr) *total = tot;
}

__global__ __launch_bounds__(kThreads) void scan_apply_kernel(int *__restrict__ x, int n,
                                                              const int *__restrict__ sums)
{
    __shared__ int sh[kWaves + 1];
    const int64_t base = (int64_t)blockIdx.x * kChunk + threadIdx.x * kItems;
    int v[kItems], acc = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        v[j] = base + j < n ? x[base + j] : 0;
        acc += v[j];
    }
    int tot;
    int run = block_exclusive_scan(acc, &tot, sh) + sums[blockIdx.x];
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        if (base + j < n) x[base + j] = run;
        run += v[j];
    }
}

hipError_t scan_exclusive(int *x, int n, int *sums, int *total, hipStream_t s)
{
    const int nb = (n + kChunk - 1) / kChunk;
    scan_reduce_kernel<<<nb, kThreads, 0, s>>>(x, n, sums);
    scan_top_kernel<<<1, kThreads, 0, s>>>(sums, nb, total);
    scan_apply_kernel<<<nb, kThreads, 0, s>>>(x, n, sums);
    return hipGetLastError();
}

// ---------------------------------------------------------------- radix sort

// sort key of token i: its id, or V for an id outside [0, V)
__device__ inline uint32_t id_key(const int32_t *ids, int64_t i, int64_t V)
{
    const int32_t id = ids[i];
    return id >= 0 && (int64_t)id < V ? (uint32_t)id : (uint32_t)V;
}

// digit histogram of each block's chunk, stored digit-major: hist[d * nblk + block]
__global__ __launch_bounds__(kThreads) void radix_hist_kernel(const uint32_t *__restrict__ keys,
                                                              const int32_t *__restrict__ ids,
                                                              int M, int64_t V, int shift,
                                                              int *__restrict__ hist)
{
    __shared__ int h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kChunk + threadIdx.x * kItems;
#pragma unroll
    for (int j = 0; j < kItems; ++j)
        if (base + j < M) {
            const uint32_t key = ids != nullptr ? id_key(ids, base + j, V) : keys[base + j];
            atomicAdd(&h[(key >> shift) & 255], 1);
        }
    __syncthreads();
    hist[threadIdx.x * gridDim.x + blockIdx.x] = h[threadIdx.x];
}

// Stable scatter of one 8-bit digit pass.  offs = exclusive scan of the histograms
// (digit-major), so offs[d * nblk + block] is where this block's first key of digit d
// goes.  Keys and values come from (ids, token index) on the first pass.
__global__ __launch_bounds__(kThreads) void radix_scatter_kernel(
    const uint32_t *__restrict__ keys, const int32_t *__restrict__ vals,
    const int32_t *__restrict__ ids, int M, int64_t V, int shift, const int *__restrict__ offs,
    uint32_t *__restrict__ keys_out, int32_t *__restrict__ vals_out)
{
    __shared__ uint32_t sk[kChunk];
    __shared__ int32_t sv[kChunk];
    __shared__ int h[256];
    __shared__ int sh[kWaves + 1];
    const int64_t base = (int64_t)blockIdx.x * kChunk;
    const int valid = (int)min((int64_t)kChunk, (int64_t)M - base);
    uint32_t k[kItems];
    int32_t v[kItems];
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int c = threadIdx.x * kItems + j;
        if (c < valid) {
            k[j] = ids != nullptr ? id_key(ids, base + c, V) : keys[base + c];
            v[j] = ids != nullptr ? (int32_t)(base + c) : vals[base + c];
        } else {
            k[j] = 0xffffffffu;  // padding: digit 255, after every real key of the chunk
            v[j] = 0;
        }
    }
    // local stable sort of the chunk by the digit: one stable 1-bit split per bit
    for (int bit = 0; bit < 8; ++bit) {
        int zeros = 0;
#pragma unroll
        for (int j = 0; j < kItems; ++j) zeros += ((k[j] >> (shift + bit)) & 1) ? 0 : 1;
        int ztot;
        const int zb = block_exclusive_scan(zeros, &ztot, sh);  // zeros in earlier threads
        int zc = 0;
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            const int c = threadIdx.x * kItems + j;
            const bool one = (k[j] >> (shift + bit)) & 1;
            const int zbefore = zb + zc;  // zeros before element c
            const int dst = one ? ztot + (c - zbefore) : zbefore;
            zc += one ? 0 : 1;
            sk[dst] = k[j];
            sv[dst] = v[j];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            k[j] = sk[threadIdx.x * kItems + j];
            v[j] = sv[threadIdx.x * kItems + j];
        }
        __syncthreads();
    }
    // start of each digit's run inside the sorted chunk (real keys only)
    h[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kItems; ++j)
        if ((int)threadIdx.x * kItems + j < valid) atomicAdd(&h[(k[j] >> shift) & 255], 1);
    __syncthreads();
    int tot;
    const int start = block_exclusive_scan(h[threadIdx.x], &tot, sh);
    h[threadIdx.x] = start;
    __syncthreads();
    // the chunk's real keys are its first `valid` sorted entries
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int c = threadIdx.x * kItems + j;
        if (c < valid) {
            const int d = (k[j] >> shift) & 255;
            const int64_t dst = (int64_t)offs[d * gridDim.x + blockIdx.x] + (c - h[d]);
            keys_out[dst] = k[j];
            vals_out[dst] = v[j];
        }
    }
}

// ---------------------------------------------------------------- small batches

constexpr int kRankTokens = 16;  // tokens a rank workgroup places
constexpr int kRankChunks = 16;  // key chunks per token, one thread each

// Stable sort by counting: token i goes to position #{j : key_j < key_i, or key_j ==
// key_i and j < i}, which is the position the stable radix sort gives it.  A
// workgroup of 256 threads places 16 tokens: thread (c, i) counts over every 16th key
// from c (all M keys staged in LDS) for token i, and the 16 counts of a token are
// added in LDS, so the M x M comparisons spread over M / 16 workgroups (every CU at
// the 36-layer step's 4096 tokens).  PACKED (V < 2^19, so that every key, V included,
// fits 19 bits; vocabularies under 524288): LDS holds key << 13 | j, all distinct, and
// the order above is a single unsigned comparison of those words.  The comparisons grow
// as M^2: 15 us at 8192 tokens (23 unpacked) against 21-30 in radix passes, 27 (46) at
// 10000 against 23-32, so it stops at 8192.
constexpr int kRankIndexBits = 13;  // token indices below kSmallSortMax = 2^13
static_assert((1 << kRankIndexBits) == kSmallSortMax, "packed keys carry the token index");

template <bool PACKED>
__global__ __launch_bounds__(kRankTokens * kRankChunks) void rank_sort_kernel(
    const int32_t *__restrict__ ids, int M, int64_t V, uint32_t *__restrict__ keys_out,
    int32_t *__restrict__ vals_out)
{
    __shared__ uint32_t sk[kSmallSortMax];
    __shared__ int cnt[kRankChunks][kRankTokens];
    // all of a thread's ids in flight at once (32 at kSmallSortMax tokens): buffer loads
    // past the M ids return 0 instead of being branched around, so that no load waits
    // for the one before it
    constexpr int kFill = kSmallSortMax / (kRankTokens * kRankChunks);
    const rsrc_t rid = make_rsrc(ids, (uint32_t)M * 4);
    int32_t fid[kFill];
#pragma unroll
    for (int f = 0; f < kFill; ++f)
        fid[f] = (int32_t)ld4(rid, (uint32_t)(f * kRankTokens * kRankChunks + threadIdx.x) * 4);
#pragma unroll
    for (int f = 0; f < kFill; ++f) {
        const int j = f * kRankTokens * kRankChunks + threadIdx.x;
        if (j < M) {
            const uint32_t key = fid[f] >= 0 && (int64_t)fid[f] < V ? (uint32_t)fid[f] : (uint32_t)V;
            sk[j] = PACKED ? key << kRankIndexBits | (uint32_t)j : key;
        }
    }
    __syncthreads();
    const int t = threadIdx.x % kRankTokens, c = threadIdx.x / kRankTokens;
    const int i = blockIdx.x * kRankTokens + t;
    const uint32_t ki = i < M ? sk[i] : 0xffffffffu;
    // chunk c: keys c, c + 16, ... (the 16 threads of a chunk read the same word, the
    // four chunks of a wave four consecutive words)
    int n = 0;
#pragma unroll 8
    for (int j = c; j < M; j += kRankChunks) {
        const uint32_t kj = sk[j];
        if constexpr (PACKED)
            n += kj < ki ? 1 : 0;
        else
            n += (kj < ki || (kj == ki && j < i)) ? 1 : 0;
    }
    cnt[c][t] = n;
    __syncthreads();
    if (c == 0 && i < M) {
        int r = 0;
#pragma unroll
        for (int cc = 0; cc < kRankChunks; ++cc) r += cnt[cc][t];
        keys_out[r] = PACKED ? ki >> kRankIndexBits : ki;
        vals_out[r] = i;
    }
}

// ---------------------------------------------------------------- middle-sized batches

// Up to kMidSortMax tokens: an LSD radix sort with 9-bit digits in two launches a pass
// (digit counts, scatter).  A workgroup ranks 1024 keys: per wave and 64 keys the lanes with
// the same digit find each other by nine ballots, and a running count per (wave, digit) in
// LDS ranks them stably.  Every workgroup adds up the digit counts of all 1024-key blocks
// itself (they are few: 128 at kMidSortMax), which saves the scan launches.  32768 text-like
// ids below 151936: 35 us with the run indices, 103 us in the 26 launches of the
// general sort.  (Counting the next pass's digits inside the scatter with global atomics
// saves a launch but queues on the few addresses that frequent ids share: 48 us.)
constexpr int kMidBits = 9;
constexpr int kMidDigits = 1 << kMidBits;
constexpr int kMidItems = 4;
constexpr int kMidChunk = kThreads * kMidItems;

__global__ __launch_bounds__(kThreads) void mid_hist_kernel(const uint32_t *__restrict__ keys,
                                                            const int32_t *__restrict__ ids, int M,
                                                            int64_t V, int shift, int *__restrict__ hist)
{
    __shared__ int h[kMidDigits];
    for (int d = threadIdx.x; d < kMidDigits; d += kThreads) h[d] = 0;
    __syncthreads();
    const int base = blockIdx.x * kMidChunk;
#pragma unroll
    for (int j = 0; j < kMidItems; ++j) {
        const int i = base + j * kThreads + (int)threadIdx.x;
        if (i < M) {
            const uint32_t key = ids != nullptr ? id_key(ids, i, V) : keys[i];
            atomicAdd(&h[(key >> shift) & (kMidDigits - 1)], 1);
        }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < kMidDigits; d += kThreads) hist[(int64_t)blockIdx.x * kMidDigits + d] = h[d];
}

// Orders the LDS accesses of one wave's lanes before it against those after it (no instruction:
// a wave's LDS accesses run in order, the compiler's order is what it holds).
__device__ inline void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

__global__ __launch_bounds__(kThreads) void mid_scatter_kernel(
    const uint32_t *__restrict__ keys, const int32_t *__restrict__ vals, const int32_t *__restrict__ ids,
    int M, int64_t V, int shift, const int *__restrict__ hist, uint32_t *__restrict__ keys_out,
    int32_t *__restrict__ vals_out)
{
    constexpr int kPerThread = kMidDigits / kThreads;
    static_assert(kPerThread == 2, "digits 2t and 2t + 1 per thread");
    __shared__ int wh[kWaves][kMidDigits];
    __shared__ int sh[kWaves + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < kWaves * kMidDigits; i += kThreads) (&wh[0][0])[i] = 0;
    // digit counts of all blocks and of the blocks before this one
    const int nblk = gridDim.x;
    int tot[2] = {0, 0}, pre[2] = {0, 0};
#pragma unroll 8
    for (int b = 0; b < nblk; ++b) {
        const u32x2 c = *reinterpret_cast<const u32x2 *>(hist + (int64_t)b * kMidDigits + 2 * threadIdx.x);
        tot[0] += (int)c[0];
        tot[1] += (int)c[1];
        pre[0] += b < (int)blockIdx.x ? (int)c[0] : 0;
        pre[1] += b < (int)blockIdx.x ? (int)c[1] : 0;
    }
    // this wave's 256 keys, 64 at a time in order
    const int base = blockIdx.x * kMidChunk + wave * (kMidChunk / kWaves);
    uint32_t k[kMidItems];
    int32_t v[kMidItems];
    int rank[kMidItems];
#pragma unroll
    for (int j = 0; j < kMidItems; ++j) {
        const int i = base + j * 64 + lane;
        k[j] = 0;
        v[j] = 0;
        if (i < M) {
            k[j] = ids != nullptr ? id_key(ids, i, V) : keys[i];
            v[j] = ids != nullptr ? i : vals[i];
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kMidItems; ++j) {
        const bool ok = base + j * 64 + lane < M;
        const int d = (int)(k[j] >> shift) & (kMidDigits - 1);
        uint64_t peers = __ballot(ok);
#pragma unroll
        for (int bit = 0; bit < kMidBits; ++bit) {
            const uint64_t m = __ballot((d >> bit) & 1);
            peers &= (d >> bit) & 1 ? m : ~m;
        }
        const int below = __popcll(peers & (((uint64_t)1 << lane) - 1));
        rank[j] = 0;
        if (ok) rank[j] = wh[wave][d] + below;
        wave_fence();  // every lane has read before the first peer adds
        if (ok && below == 0) wh[wave][d] += __popcll(peers);
        wave_fence();
    }
    __syncthreads();
    // wh becomes the position of the wave's first key of each digit
    int total;
    int at = block_exclusive_scan(tot[0] + tot[1], &total, sh);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int d = 2 * threadIdx.x + e;
        int run = at + pre[e];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int c = wh[w][d];
            wh[w][d] = run;
            run += c;
        }
        at += tot[e];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kMidItems; ++j)
        if (base + j * 64 + lane < M) {
            const int dst = wh[wave][(k[j] >> shift) & (kMidDigits - 1)] + rank[j];
            keys_out[dst] = k[j];
            vals_out[dst] = v[j];
        }
}

// Runs of a sorted key array of M <= kMidSortMax entries in one launch: a workgroup takes
// 1024 keys and counts the run starts before them itself.  Every run's first row gets the
// run's index; the run of key V (if any) is the last one and is not counted as a distinct
// id.  Keys past the end read as zeros (buffer range).
__global__ __launch_bounds__(kThreads) void mid_segments_kernel(const uint32_t *__restrict__ keys, int M,
                                                                int64_t V, int *__restrict__ segidx,
                                                                int32_t *__restrict__ uniq,
                                                                int32_t *__restrict__ num_uniq)
{
    static_assert(kMidItems % 4 == 0, "whole 16-byte loads");
    __shared__ int sh[kWaves + 1];
    const rsrc_t rk = make_rsrc(keys, (uint32_t)M * 4);
    // bit e: key i + e (e < 4) starts a run; k receives the four keys
    auto heads = [&](int i, u32x4 &k) __attribute__((always_inline)) {
        k = ld16(rk, (uint32_t)i * 4);
        const uint32_t before = i > 0 ? ld4(rk, (uint32_t)(i - 1) * 4) : 0u;
        uint32_t h = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + e < M && (i + e == 0 || k[e] != (e == 0 ? before : k[e - 1]))) h |= 1u << e;
        return h;
    };
    const int b0 = blockIdx.x * kMidChunk;
    int earlier = 0;
#pragma unroll 4
    for (int i = threadIdx.x * 4; i < b0; i += kThreads * 4) {
        u32x4 k;
        earlier += __builtin_popcount(heads(i, k));
    }
    int before_block;
    block_exclusive_scan(earlier, &before_block, sh);
    const int i0 = b0 + threadIdx.x * kMidItems;
    uint32_t head = 0;
    u32x4 k[kMidItems / 4];
#pragma unroll
    for (int q = 0; q < kMidItems / 4; ++q) head |= heads(i0 + 4 * q, k[q]) << (4 * q);
    int here;
    int u = before_block + block_exclusive_scan(__builtin_popcount(head), &here, sh);
#pragma unroll
    for (int e = 0; e < kMidItems; ++e) {
        const uint32_t ke = k[e / 4][e % 4];
        if ((head >> e) & 1u) {
            segidx[i0 + e] = u;
            if (ke < (uint64_t)V) uniq[u] = (int32_t)ke;
            ++u;
        }
        if (i0 + e == M - 1) *num_uniq = before_block + here - (ke == (uint64_t)V ? 1 : 0);
    }
}

// ---------------------------------------------------------------- segments

__global__ __launch_bounds__(kThreads) void seg_flags_kernel(const uint32_t *__restrict__ keys,
                                                             int M, int *__restrict__ flags)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < M) flags[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1 : 0;
}

// segidx = exclusive scan of the head flags: a head's value is its segment's index
__global__ __launch_bounds__(kThreads) void seg_write_kernel(const uint32_t *__restrict__ keys,
                                                             const int *__restrict__ segidx,
                                                             int M, int64_t V, int32_t *__restrict__ uniq)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= M || !(i == 0 || keys[i] != keys[i - 1])) return;
    if (keys[i] < (uint64_t)V) uniq[segidx[i]] = (int32_t)keys[i];
}

// counts the distinct in-range ids (the run of key V, if any, is the last segment and is
// left out)
__global__ void seg_finish_kernel(const uint32_t *__restrict__ keys, int M, int64_t V,
                                  const int *__restrict__ nseg, int32_t *__restrict__ num_uniq)
{
    *num_uniq = *nseg - (keys[M - 1] == (uint64_t)V ? 1 : 0);
}

// ---------------------------------------------------------------- gather-reduce

// drows[s][u][:] = sum over the run of distinct id u of dout[pos*n + s][:] (fp32, in
// ascending token order).  HBM-bound: every upstream row is read once, every gradient row
// written once.  Token ids repeat very unevenly (in running text a few make up a tenth of all
// tokens, most occur once), so the work is split by sorted rows, not by ids: a wave
// takes the runs that start among R consecutive sorted rows, for one stream and 64 * VEC
// columns, loads the R rows at once, adds them in order and stores a sum at every run's
// end.  Only a run that reaches past the R rows goes on, R rows at a time; waves that see
// no run start have nothing to do.  So all loads of a wave are in flight together,
// whatever the run lengths, and a run of k rows takes k / R steps in place of k.  Measured
// (text-like ids, Dm=4096 bf16 at 4096 tokens, 290 MB; Dm=2048 at 8 x 4096, 959 MB; n=4):
// 123 -> 59 us and 684 -> 201 us against one workgroup per (id, stream) walking its run row
// by row; on ids that hardly repeat 83 -> 83 and 346 -> 292 us.  R = 4 rows: with 8 or 16
// the latter took 89 us, with fewer waves in flight while each waits for its loads.
//
// Buffer loads with an exact range per row (zero for rows outside the wave's part) keep the
// loads free of branches; the upstream rows are read once, so they carry the streaming
// hint (14% faster than cached ones on rows that are not in the caches).
template <typename E, int VEC>
struct RowChunk {
    static constexpr int kBytes = VEC * sizeof(E);
    static constexpr int kWords = kBytes < 4 ? 1 : kBytes / 4;
    uint32_t w[kWords];
    __device__ inline void load(rsrc_t r, uint32_t off)
    {
        if constexpr (kBytes >= 16) {
#pragma unroll
            for (int i = 0; i < kBytes / 16; ++i) {
                const u32x4 x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off + i * 16, 0, 2));
                w[4 * i] = x[0];
                w[4 * i + 1] = x[1];
                w[4 * i + 2] = x[2];
                w[4 * i + 3] = x[3];
            }
        } else if constexpr (kBytes == 8) {
            const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 2);
            w[0] = x[0];
            w[1] = x[1];
        } else if constexpr (kBytes == 4) {
            w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 2);
        } else {
            w[0] = __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 2);
        }
    }
    __device__ inline void add(float (&acc)[VEC]) const
    {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if constexpr (sizeof(E) == 4)
                acc[e] += __uint_as_float(w[e]);
            else
                acc[e] += (e & 1) ? bf16_hi(w[e / 2]) : bf16_lo(w[e / 2]);
        }
    }
};

// A long run: kSplit waves (the one whose rows hold its start and the next ones, which have
// no run start of their own) take a kSplit-th of the columns each, with kSplit times the
// rows in flight.  A run is long when it covers those waves' rows whole.
constexpr int kSplit = 4;

// acc of columns d0 .. d0 + VR of stream s over the run of `key` that starts at sorted row
// `at`, RR rows at a time; the next rows' keys are loaded while these are added.
template <typename E, int VR, int RR>
__device__ inline void sum_run(const E *dout, const uint32_t *keys, const int32_t *pos, int M, uint32_t key,
                               int at, int n, int Dm, int s, int c0, int lane, float (&acc)[VR])
{
    static_assert(RR <= 64, "a lane per row");
    uint32_t k = keys[min(at + lane, M - 1)];
    int p = pos[min(at + lane, M - 1)];
    for (;;) {
        const uint64_t out = ~__ballot(at + lane < M && k == key && lane < RR);
        const int cnt = out ? __builtin_ctzll(out) : 64;
        RowChunk<E, VR> x[RR];
#pragma unroll
        for (int r = 0; r < RR; ++r) {
            const int64_t row = (int64_t)__builtin_amdgcn_readlane(p, r) * n + s;
            x[r].load(make_rsrc(dout + row * Dm + c0,
                                r < cnt ? (uint32_t)min(Dm - c0, 64 * VR) * (uint32_t)sizeof(E) : 0u),
                      (uint32_t)lane * RowChunk<E, VR>::kBytes);
        }
        at += RR;
        k = keys[min(at + lane, M - 1)];
        p = pos[min(at + lane, M - 1)];
#pragma unroll
        for (int r = 0; r < RR; ++r) x[r].add(acc);
        if (cnt < RR) return;
    }
}

template <typename E, int VEC, int R>
__global__ __launch_bounds__(kThreads) void embed_grad_reduce_kernel(
    const E *__restrict__ dout, const uint32_t *__restrict__ keys, const int32_t *__restrict__ pos,
    const int *__restrict__ segidx, int M, int64_t V, int n, int Dm, int nchunk, int64_t units,
    float *__restrict__ drows)
{
    static_assert((kSplit - 1) * R < 64 && R < 64, "a lane per row looked back over, and one past R");
    constexpr bool kRuns = VEC == 8;  // long runs are split
    constexpr int VR = VEC / kSplit > 0 ? VEC / kSplit : 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int64_t unit = (int64_t)blockIdx.x * kWaves + wave; unit < units; unit += (int64_t)gridDim.x * kWaves) {
        const int c0 = (int)(unit % nchunk) * 64 * VEC;  // this wave's columns
        const int64_t us = unit / nchunk;
        const int s = (int)(us % n);
        int base = (int)(us / n) * R;
        const int d0 = c0 + lane * VEC;
        float acc[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
        int u = 0;
        auto store = [&]() __attribute__((always_inline)) {
            if (d0 >= Dm) return;
            float *o = drows + ((int64_t)s * M + u) * Dm + d0;
            if constexpr (VEC == 8) {
                *reinterpret_cast<f32x4 *>(o) = f32x4{acc[0], acc[1], acc[2], acc[3]};
                *reinterpret_cast<f32x4 *>(o + 4) = f32x4{acc[4], acc[5], acc[6], acc[7]};
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) o[e] = acc[e];
            }
        };
        // this wave's share `part` of the long run that starts at sorted row `at`
        auto long_run = [&](int at, uint32_t key, int part) __attribute__((always_inline)) {
            if constexpr (kRuns) {
                constexpr int RR = 64 / RowChunk<E, VR>::kWords;
                const int c = c0 + part * 64 * VR, d = c + lane * VR;
                if (c >= Dm) return;
                float a[VR];
#pragma unroll
                for (int e = 0; e < VR; ++e) a[e] = 0.f;
                sum_run<E, VR, RR>(dout, keys, pos, M, key, at, n, Dm, s, c, lane, a);
                if (d >= Dm) return;
                float *o = drows + ((int64_t)s * M + segidx[at]) * Dm + d;
#pragma unroll
                for (int e = 0; e < VR; ++e) o[e] = a[e];
            }
        };
        // the run that starts in rows [base, base + R) and goes on past them is long
        auto is_long = [&](int b, uint32_t key) __attribute__((always_inline)) {
            return kRuns && b + kSplit * R <= M && keys[b + kSplit * R - 1] == key;
        };
        bool first = true;
        for (;;) {
            // lane l: sorted row base + l; bit l of `head`: it starts a run; of `end`: no row of
            // an id in [0, V) (the run of key V is the last one)
            const int row = min(base + lane, M - 1);
            const uint32_t key = keys[row], before = keys[max(row - 1, 0)];
            const int at = pos[row], si = segidx[row];
            const uint64_t head = __ballot(row == 0 || key != before);
            const uint64_t end = __ballot(base + lane >= M || (uint64_t)key >= (uint64_t)V);
            const int nend = end ? __builtin_ctzll(end) : 64;
            int lo = 0, hi = min(R, nend);
            if (first) {
                lo = head ? __builtin_ctzll(head) : 64;
                if (lo >= hi) {  // no run starts here; perhaps a share of a long one
                    if (kRuns && lo >= R && nend > 0) {
                        const uint32_t k0 = __builtin_amdgcn_readfirstlane(key);
                        // lane l: row base - (kSplit - 1) R + l
                        const int back = base - (kSplit - 1) * R + lane;
                        const uint32_t kb = keys[max(back, 0)], kp = keys[max(back - 1, 0)];
                        const uint64_t h = __ballot(lane < (kSplit - 1) * R && back >= 0 && kb == k0 &&
                                                    (back == 0 || kp != k0));
                        if (h) {
                            const int start = base - (kSplit - 1) * R + __builtin_ctzll(h);
                            const int owner = start / R * R;
                            if (is_long(owner, k0)) long_run(start, k0, (base - owner) / R);
                        }
                    }
                    break;
                }
                u = __builtin_amdgcn_readlane(si, lo);
                // the last run that starts here: handled apart if it is long
                if (kRuns && hi == R && !((head >> R) & 1) && nend > R) {
                    const int last = 63 - __builtin_clzll(head & (((uint64_t)1 << R) - 1));
                    const uint32_t kl = __builtin_amdgcn_readlane(key, last);
                    if (is_long(base, kl)) {
                        long_run(base + last, kl, 0);
                        hi = last;
                        if (lo >= hi) break;
                    }
                }
            } else {
                hi = min(hi, head ? __builtin_ctzll(head) : 64);
            }
            RowChunk<E, VEC> x[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t p = (int64_t)__builtin_amdgcn_readlane(at, r) * n + s;
                const bool in = r >= lo && r < hi;
                x[r].load(make_rsrc(dout + p * Dm + c0,
                                    in ? (uint32_t)min(Dm - c0, 64 * VEC) * (uint32_t)sizeof(E) : 0u),
                          (uint32_t)lane * RowChunk<E, VEC>::kBytes);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r > lo && r < hi && ((head >> r) & 1)) {  // the next run starts
                    store();
                    ++u;
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
                }
                x[r].add(acc);
            }
            if (hi < R || nend <= R || ((head >> R) & 1)) {
                store();
                break;
            }
            base += R;
            first = false;
        }
    }
}

// dtables[s][uniq[u]][:] += drows[s][u][:] for u < *num_uniq (distinct ids: one writer
// per destination row, no atomics)
__global__ __launch_bounds__(kThreads) void embed_grad_scatter_add_kernel(
    const int32_t *__restrict__ uniq, const float *__restrict__ drows,
    const int32_t *__restrict__ num_uniq, int rows_cap, int n, int64_t V, int Dm,
    float *__restrict__ dtables)
{
    const int64_t items = (int64_t)*num_uniq * n;
    for (int64_t w = blockIdx.x; w < items; w += gridDim.x) {
        const int u = (int)(w / n), s = (int)(w % n);
        const int32_t x = uniq[u];
        if (x < 0 || (int64_t)x >= V) continue;
        const float *src = drows + ((int64_t)s * rows_cap + u) * Dm;
        float *dst = dtables + ((int64_t)s * V + x) * Dm;
        for (int d = threadIdx.x; d < Dm; d += kThreads) dst[d] += src[d];
    }
}

// ---------------------------------------------------------------- cyclic replication

// dst table s (s0 <= s < m) = src table s mod n; `words` W-sized words per table
template <typename W>
__global__ __launch_bounds__(kThreads) void cyclic_replicate_kernel(const W *__restrict__ src,
                                                                    W *__restrict__ dst, int n,
                                                                    int s0, int64_t words)
{
    const int s = s0 + blockIdx.y;
    const W *a = src + (int64_t)(s % n) * words;
    W *b = dst + (int64_t)s * words;
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < words;
         e += (int64_t)gridDim.x * kThreads)
        b[e] = a[e];
}

}  // namespace

EmbedBwdWorkspace embed_bwd_workspace(int M)
{
    EmbedBwdWorkspace w;
    const size_t m4 = align256((size_t)M * 4);
    const int nblk = (M + kChunk - 1) / kChunk;
    w.keys_a = 0;
    w.vals_a = w.keys_a + m4;
    w.keys_b = w.vals_a + m4;
    w.vals_b = w.keys_b + m4;
    w.hist = w.vals_b + m4;
    w.sums = w.hist + align256((size_t)256 * nblk * 4);
    w.scalars = w.sums + align256((size_t)kChunk * 4);
    w.segidx = w.scalars + 256;
    w.total = w.segidx + m4 + align256(((size_t)M + 1) * 4);
    return w;
}

hipError_t launch_embed_bwd(const int32_t *ids, const void *dout, int B, int L, int n, int64_t V,
                            int Dm, int esize, int32_t *uniq, float *drows, int32_t *num_uniq,
                            void *ws, hipStream_t s)
{
    const int M = B * L;
    const EmbedBwdWorkspace w = embed_bwd_workspace(M);
    char *base = static_cast<char *>(ws);
    uint32_t *ka = reinterpret_cast<uint32_t *>(base + w.keys_a);
    int32_t *va = reinterpret_cast<int32_t *>(base + w.vals_a);
    uint32_t *kb = reinterpret_cast<uint32_t *>(base + w.keys_b);
    int32_t *vb = reinterpret_cast<int32_t *>(base + w.vals_b);
    int *hist = reinterpret_cast<int *>(base + w.hist);
    int *sums = reinterpret_cast<int *>(base + w.sums);
    int *nseg = reinterpret_cast<int *>(base + w.scalars);
    int *segidx = reinterpret_cast<int *>(base + w.segidx);

    const int nblk = (M + kChunk - 1) / kChunk, nmid = (M + kMidChunk - 1) / kMidChunk;
    int bits = 0;
    while (bits < 32 && ((uint64_t)V >> bits) != 0) ++bits;  // the largest key is V

    timing_before("embed_bwd_sort", s);
    hipError_t e = hipSuccess;
    const uint32_t *kin = nullptr;
    const int32_t *vin = nullptr;
    if (M <= kSmallSortMax) {
        const unsigned nb = (M + kRankTokens - 1) / kRankTokens;
        if (V < ((int64_t)1 << (32 - kRankIndexBits)))
            rank_sort_kernel<true><<<nb, kRankTokens * kRankChunks, 0, s>>>(ids, M, V, ka, va);
        else
            rank_sort_kernel<false><<<nb, kRankTokens * kRankChunks, 0, s>>>(ids, M, V, ka, va);
        kin = ka;
        vin = va;
        e = hipGetLastError();
    } else {
        const bool mid = M <= kMidSortMax;
        const int width = mid ? kMidBits : 8;
        const int passes = (bits + width - 1) / width;
        // the digit counts of a middle-sized pass (512 per 1024 tokens) lie in the part that
        // later holds the segment indices
        for (int p = 0; p < passes && e == hipSuccess; ++p) {
            uint32_t *kout = (p & 1) ? kb : ka;
            int32_t *vout = (p & 1) ? vb : va;
            const int32_t *from_ids = p == 0 ? ids : nullptr;
            if (mid) {
                mid_hist_kernel<<<nmid, kThreads, 0, s>>>(kin, from_ids, M, V, width * p, segidx);
                mid_scatter_kernel<<<nmid, kThreads, 0, s>>>(kin, vin, from_ids, M, V, width * p, segidx,
                                                             kout, vout);
            } else {
                radix_hist_kernel<<<nblk, kThreads, 0, s>>>(kin, from_ids, M, V, width * p, hist);
                e = scan_exclusive(hist, 256 * nblk, sums, nullptr, s);
                radix_scatter_kernel<<<nblk, kThreads, 0, s>>>(kin, vin, from_ids, M, V, width * p, hist,
                                                               kout, vout);
            }
            kin = kout;
            vin = vout;
            if (e == hipSuccess) e = hipGetLastError();
        }
    }
    timing_after(s);
    if (e != hipSuccess) return e;

    timing_before("embed_bwd_segments", s);
    if (M <= kMidSortMax) {
        mid_segments_kernel<<<nmid, kThreads, 0, s>>>(kin, M, V, segidx, uniq, num_uniq);
    } else {
        const int nb1 = (M + kThreads - 1) / kThreads;
        seg_flags_kernel<<<nb1, kThreads, 0, s>>>(kin, M, segidx);
        e = scan_exclusive(segidx, M, sums, nseg, s);
        seg_write_kernel<<<nb1, kThreads, 0, s>>>(kin, segidx, M, V, uniq);
        seg_finish_kernel<<<1, 1, 0, s>>>(kin, M, V, nseg, num_uniq);
    }
    if (e == hipSuccess) e = hipGetLastError();
    timing_after(s);
    if (e != hipSuccess) return e;

    timing_before("embed_bwd_reduce", s);
    // VEC columns per lane (whole aligned words of a row), R rows in flight per wave in 64
    // registers; units beyond the grid are strided over it
    auto reduce = [&](auto elem, auto vec) {
        using E = decltype(elem);
        constexpr int VEC = decltype(vec)::value;
        constexpr int R = VEC == 8 ? 4 : 16;
        const int nchunk = (Dm + 64 * VEC - 1) / (64 * VEC);
        const int64_t units = (int64_t)((M + R - 1) / R) * n * nchunk;
        const int64_t wgs = (units + kWaves - 1) / kWaves;
        embed_grad_reduce_kernel<E, VEC, R><<<(unsigned)std::min<int64_t>(wgs, 1 << 22), kThreads, 0, s>>>(
            static_cast<const E *>(dout), kin, vin, segidx, M, V, n, Dm, nchunk, units, drows);
    };
    auto pick = [&](auto elem) {
        if (Dm % 8 == 0)
            reduce(elem, std::integral_constant<int, 8>{});
        else if (Dm % 2 == 0)
            reduce(elem, std::integral_constant<int, 2>{});
        else
            reduce(elem, std::integral_constant<int, 1>{});
    };
    if (esize == 2)
        pick(bf16{});
    else
        pick(float{});
    e = hipGetLastError();
    timing_after(s);
    return e;
}

hipError_t launch_embed_grad_scatter_add(const int32_t *uniq, const float *drows,
                                         const int32_t *num_uniq, int rows_cap, int n, int64_t V,
                                         int Dm, float *dtables, hipStream_t s)
{
    const int64_t max_items = (int64_t)rows_cap * n;
    const int grid = (int)(max_items < 8192 ? max_items : 8192);
    timing_before("embed_grad_scatter_add", s);
    embed_grad_scatter_add_kernel<<<grid, kThreads, 0, s>>>(uniq, drows, num_uniq, rows_cap, n, V,
                                                            Dm, dtables);
    hipError_t e = hipGetLastError();
    timing_after(s);
    return e;
}

hipError_t launch_cyclic_replicate(const void *src, void *dst, int n, int m, int64_t V, int Dm,
                                   int esize, hipStream_t s)
{
    const int s0 = src == dst ? n : 0;  // in place: the first n tables are already there
    if (s0 >= m) return hipSuccess;
    const int64_t bytes = V * (int64_t)Dm * esize;
    const dim3 block(kThreads);
    timing_before("cyclic_replicate", s);
    if (bytes % 16 == 0) {
        const int64_t words = bytes / 16;
        const dim3 grid((unsigned)std::min<int64_t>((words + kThreads - 1) / kThreads, 4096),
                        (unsigned)(m - s0));
        cyclic_replicate_kernel<u32x4><<<grid, block, 0, s>>>(
            static_cast<const u32x4 *>(src), static_cast<u32x4 *>(dst), n, s0, words);
    } else {
        const int64_t words = bytes / 2;
        const dim3 grid((unsigned)std::min<int64_t>((words + kThreads - 1) / kThreads, 4096),
                        (unsigned)(m - s0));
        cyclic_replicate_kernel<uint16_t><<<grid, block, 0, s>>>(
            static_cast<const uint16_t *>(src), static_cast<uint16_t *>(dst), n, s0, words);
    }
    hipError_t e = hipGetLastError();
    timing_after(s);
    return e;
}

}  // namespace hd
