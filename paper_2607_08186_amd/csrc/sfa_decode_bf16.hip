// sfa_decode_bf16.hip -- parallel-stream decode for Stream-Factorized Attention.
//
// At a decode step the n streams of each sequence's new token are run together: query
// row s of sequence b sits at expanded position ctx[b]*n + s and attends, under the
// layer's mask, to the sequence's cached rows (the new token's own n keys and values
// are already appended at rows ctx[b]*n .. ctx[b]*n + n - 1).  An intra-stream layer
// reads only its stream's rows (1/n of the cache), a full cross-stream layer the whole
// prefix, a local one the last `window` positions.
//
// HBM-bound: every cached key/value row is read once for all the query rows that use it
// (the heads of its group, and for cross-stream layers all n streams: up to 32 query
// slots per problem).  Split over the cache (dec_splits):
//   partial: a workgroup takes one split of the cached rows of one problem (b, kv-head[,
//            head chunk][, stream]); its waves take 32-row tiles in turn, K and V each through a
//            place of its own in LDS that the next tile's rows are loaded into as soon as this one's
//            are used (direct-to-LDS streaming loads of whole lines, no barrier in the loop),
//            S^T = K Q^T and O^T += V^T P^T on the matrix cores with a running maximum per
//            query slot, the waves merged through LDS into one (max, sum, unnormalised O)
//            per query slot in the workspace;
//   combine: per query row, the splits' partials reduced to o and lse.
// Where all problems have one split only (short contexts, or enough problems to fill the chip) the
// partial kernel writes o and lse itself and the combine is not launched.
// Measured at 16 x 4096 tokens, n=4, 32/8 heads of 128: 6.3 TB/s of cache rows with the combine
// (full cross-stream and intra-stream); streaming loads give 5% over cached ones.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "decode_internal.h"
#include "sfa_lds.h"

namespace hd {

namespace {

constexpr int kTile = kDecTile;               // cached rows per wave and step
constexpr int kSlots = 32;                    // query slots per problem (MFMA columns)

// What a tile's rows see: rows below < j <= limit are visible to this lane's query (they exist
// and, for cross-stream layers, lie at or before it and within the window).
struct Mask {
    int kvlen, pos0, n, window, limit, below;
    bool cross;
    __device__ inline Mask(const DecGeom &g, const DecRows &r, int slot)
        : kvlen(r.kvlen), pos0(r.ctx * g.n), n(g.n), window(g.window), cross(g.mode != 0)
    {
        const int qp = pos0 + slot / g.gchunk;  // my query's key coordinate (cross-stream layers)
        limit = cross ? min(qp, kvlen - 1) : kvlen - 1;
        below = cross ? max(-1, qp - window) : -1;
    }
    // the tile at row kb holds a pair that is not visible (uniform over the wave)
    __device__ inline bool some(int kb) const
    {
        const int last = kb + kTile - 1;
        return last >= kvlen || (cross && (last > pos0 || pos0 + n - 1 - kb >= window));
    }
};

template <int N>
__device__ inline void wait_loads_le()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// NW waves; ONCE: each line of the cache serves one problem only (streaming loads).
template <int D, int NW, bool ONCE>
__global__ __launch_bounds__(NW * 64, 1) void sfa_decode_partial_kernel(
    const bf16 *__restrict__ q, const bf16 *__restrict__ kc, const bf16 *__restrict__ vc,
    const int32_t *__restrict__ ctx_tokens, float *__restrict__ part, bf16 *__restrict__ o,
    float *__restrict__ lse, DecGeom g)
{
    constexpr int KS = D / 16, DB = D / 32;
    using T = Tile<D, kTile>;
    constexpr int LOADS = T::INSTR;  // direct-to-LDS instructions per K or V tile
    // LDS: K and V tile of each wave, reused at the end as the scratch of the merge
    // ([wave][slot][D + 1] of O: the odd row length keeps both its writes, a slot per lane, and
    // its reads, a dim per lane, off one another's banks; then [wave][slot] max and sum)
    constexpr int MERGE = NW * kSlots * (D + 1) * 4 + 2 * NW * kSlots * 4;
    constexpr int TILES = NW * 2 * T::BYTES;
    constexpr int ALL = TILES + T::BYTES;  // tiles | the query slots
    __shared__ __attribute__((aligned(1024))) char smem[MERGE > ALL ? MERGE : ALL];

    DecProblem pr;
    int split;
    if (!dec_place(g, blockIdx.x, pr, split)) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;

    const DecRows dr = dec_rows(g, ctx_tokens[pr.b]);
    // this workgroup's rows: cross-stream rows are expanded positions, intra-stream problem
    // row j is cache row j*n + s
    const int r0 = dr.klo + split * dr.per;
    if (r0 >= dr.kvlen) return;  // the combine reads the splits that have rows
    const int r1 = min(dr.kvlen, r0 + dr.per);
    const int nt = (r1 - r0 + kTile - 1) / kTile;
    const Mask mk(g, dr, l32);

    // the sequence's cached rows; rows past the context are out of range and load zeros
    const size_t cslice = (size_t)g.n * g.Lcap * g.Hkv * D;
    const uint32_t range = (uint32_t)((size_t)(dr.ctx + 1) * g.n * g.Hkv * D * 2);
    const rsrc_t rk = make_rsrc(kc + pr.b * cslice, range);
    const rsrc_t rv = make_rsrc(vc + pr.b * cslice, range);
    const uint32_t kstride = (uint32_t)(g.mode == 0 ? g.n : 1) * g.Hkv * D * 2;
    const uint32_t kbase = (uint32_t)((g.mode == 0 ? pr.s : 0) * g.Hkv + pr.hk) * D * 2;

    char *const ktile = smem + wave * 2 * T::BYTES, *const vtile = ktile + T::BYTES;
    char *const qtile = smem + TILES;
    const auto plan = T::template dma_plan<1>(kbase, kstride, 0, lane);
    // K or V rows of tile t of the split to st; tiles past the last one load zeros, so that the
    // loads in flight can be counted.
    auto issue = [&](rsrc_t rs, int t, char *st) __attribute__((always_inline)) {
        const uint32_t off = t < nt ? (uint32_t)(r0 + t * kTile) * kstride : kOob;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            if constexpr (ONCE)
                dma_lds16_nt(rs, st + i * 1024, plan.voff[i] + off);
            else
                dma_lds16(rs, st + i * 1024, plan.voff[i] + off);
        }
    };

    // The 32 query slots (column l32 of the MFMA results is slot l32), shared by the waves, and
    // behind them the first tiles.
    const int nslot = g.nslot;
    {
        const rsrc_t rq = make_rsrc(q, (uint32_t)((size_t)g.B * g.n * g.Hq * D * 2));
#pragma unroll
        for (int i = wave; i < LOADS; i += NW) {
            const int x = i * 64 + lane, slot = x / T::CH, c = (x % T::CH) ^ T::swz(slot);
            const int st = g.mode == 0 ? pr.s : slot / g.gchunk;
            const int h = pr.hk * g.G + pr.gc * g.gchunk + (g.mode == 0 ? slot : slot % g.gchunk);
            dma_lds16(rq, qtile + i * 1024,
                      slot < nslot ? (uint32_t)((((size_t)pr.b * g.n + st) * g.Hq + h) * D * 2) + c * 16 : kOob);
        }
    }
    issue(rk, wave, ktile);
    issue(rv, wave, vtile);
    uint32_t kro[KS], vto[DB][2];
    T::row_offsets(l32, hi, kro);
    T::tr_offsets(lane, vto);
    wait_loads_le<2 * LOADS>();
    lds_barrier();
    bf16x8 qr[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qr[kk] = T::row_at(qtile, kro[kk], 0);

    float m = -INFINITY, lsum = 0.f;
    f32x16 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db] = f32x16{};
    const float c2 = g.scale_log2;
    // K of the wave's next tile is loaded once the scores of this one are formed, its V once this
    // one's product is: what is waited for has landed when only the tile issued after it is in
    // flight.
    for (int t = wave; t < nt; t += NW) {
        const int kb = r0 + t * kTile;
        wait_loads_le<LOADS>();
        bf16x8 a[KS];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) a[kk] = T::row_at(ktile, kro[kk], 0);
        __builtin_amdgcn_sched_barrier(0);
        // S^T = K Q^T
        f32x16 sc = {};
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) sc = mfma32(a[kk], qr[kk], sc);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue(rk, t + NW, ktile);
        mfma_settle();
        float x[16], mx = -INFINITY;
        if (mk.some(kb)) {
            const int lim = mk.limit - kb - 4 * hi, lo = mk.below - kb - 4 * hi;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = 8 * (r >> 2) + (r & 3);
                x[r] = ((j > lim) | (j <= lo)) ? -INFINITY : sc[r] * c2;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = sc[r] * c2;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, x[r]);
        const float mn = fmaxf(m, max_xor32(mx));
        if (__any(mn > m)) {
            const float alpha = mn == m ? 1.f : fast_exp2(m - mn);
            m = mn;
            lsum *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) oacc[db] *= alpha;
        }
        const float me = m == -INFINITY ? 0.f : m;  // no visible row yet: weights exp2(-inf) = 0
        bf16x8 pb[2];
        const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                w[e] = pack_bf16(fast_exp2(x[h * 8 + 2 * e] - me), fast_exp2(x[h * 8 + 2 * e + 1] - me));
                // the sum adds the bf16 weights that the P V product uses
                lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w[e]), ones, lsum, false);
            }
            pb[h] = __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]});
        }
        // O^T (dims x slots) += V^T P^T
        wait_loads_le<LOADS>();
        bf16x8 b[DB][2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int db = 0; db < DB; ++db) b[db][kk] = T::tr_at(vtile, vto[db], kk);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int db = 0; db < DB; ++db) oacc[db] = mfma32(b[db][kk], pb[kk], oacc[db]);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue(rv, t + NW, vtile);
        mfma_settle();
    }
    wait_loads_le<0>();  // nothing may write the tiles any more
    mfma_settle();
    lsum = sum_xor32(lsum);

    // merge the waves
    __syncthreads();
    float *so = reinterpret_cast<float *>(smem);
    float *sm = so + NW * kSlots * (D + 1);
    float *sl = sm + NW * kSlots;
    if (l32 < nslot) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                so[(wave * kSlots + l32) * (D + 1) + db * 32 + 8 * (r >> 2) + 4 * hi + (r & 3)] = oacc[db][r];
        if (hi == 0) {
            sm[wave * kSlots + l32] = m;
            sl[wave * kSlots + l32] = lsum;
        }
    }
    __syncthreads();
    // partials [problem][split][slot][D + 2]: O, then max and sum, for the problem's
    // nslot slots only; with one split per problem the results themselves
    float *dst = part + ((size_t)dec_index(g, pr) * g.nsplit + split) * nslot * (D + 2);
    for (int e = tid; e < nslot * D; e += NW * 64) {
        const int sl_i = e / D, d = e % D;
        float mt = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) mt = fmaxf(mt, sm[w * kSlots + sl_i]);
        float x = 0.f, l = 0.f;
        if (mt != -INFINITY) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float a = fast_exp2(sm[w * kSlots + sl_i] - mt);
                x += a * so[(w * kSlots + sl_i) * (D + 1) + d];
                l += a * sl[w * kSlots + sl_i];
            }
        }
        if (g.nsplit == 1) {
            const int st = g.mode == 0 ? pr.s : sl_i / g.gchunk;
            const int h = pr.hk * g.G + pr.gc * g.gchunk + (g.mode == 0 ? sl_i : sl_i % g.gchunk);
            o[(((size_t)pr.b * g.n + st) * g.Hq + h) * D + d] = (bf16)(x / l);
            if (d == 0) lse[((size_t)pr.b * g.Hq + h) * g.n + st] = (mt + log2f(l)) * 0.6931471805599453f;
        } else {
            dst[sl_i * (D + 2) + d] = x;
            if (d == 0) {
                dst[sl_i * (D + 2) + D] = mt;
                dst[sl_i * (D + 2) + D + 1] = l;
            }
        }
    }
}

// one workgroup of D threads per query row (b, s, hq): reduce the splits' partials
template <int D>
__global__ __launch_bounds__(D) void sfa_decode_combine_kernel(const float *__restrict__ part,
                                                               const int32_t *__restrict__ ctx_tokens,
                                                               bf16 *__restrict__ o,
                                                               float *__restrict__ lse, DecGeom g)
{
    const int hq = blockIdx.x % g.Hq;
    const int s = (blockIdx.x / g.Hq) % g.n;
    const int b = blockIdx.x / (g.Hq * g.n);
    const int gl = (hq % g.G) % g.gchunk;
    const int prob = dec_index(g, DecProblem{b, hq / g.G, (hq % g.G) / g.gchunk, g.mode == 0 ? s : 0});
    const int slot = g.mode == 0 ? gl : s * g.gchunk + gl;
    // the splits the partial kernel wrote: those with rows
    const DecRows dr = dec_rows(g, ctx_tokens[b]);
    const int nc = (dr.kvlen - dr.klo + dr.per - 1) / dr.per;
    const float *src = part + (size_t)prob * g.nsplit * g.nslot * (D + 2) + slot * (D + 2);
    const size_t cstep = (size_t)g.nslot * (D + 2);
    // Every split has a visible row for some query of the problem, but
    // possibly none for this one (max -inf, sum 0); the query's own key is in one of
    // them, so the largest maximum m is finite.  Two passes, m first and then each
    // split's share scaled by exp2(mc - m): no load waits for the previous split's
    // arithmetic, as it would with a running maximum.
    float m = -INFINITY;
#pragma unroll 8
    for (int c = 0; c < nc; ++c) m = fmaxf(m, src[c * cstep + D]);
    float acc = 0.f, l = 0.f;
#pragma unroll 8
    for (int c = 0; c < nc; ++c) {
        const float mc = src[c * cstep + D], lc = src[c * cstep + D + 1];
        const float oc = src[c * cstep + threadIdx.x];
        const float w = fast_exp2(mc - m);  // exp2(-inf) = 0
        // a split without a visible row is skipped (select, no branch)
        acc = mc == -INFINITY ? acc : __builtin_fmaf(oc, w, acc);
        l = mc == -INFINITY ? l : __builtin_fmaf(lc, w, l);
    }
    const size_t row = ((size_t)b * g.n + s) * g.Hq + hq;
    o[row * D + threadIdx.x] = (bf16)(acc / l);
    if (threadIdx.x == 0) lse[((size_t)b * g.Hq + hq) * g.n + s] = (m + log2f(l)) * 0.6931471805599453f;
}

}  // namespace

DecGeom make_dec_geom(int B, int Lcap, int n, int Hq, int Hkv, int D, int mode, int window,
                      float scale, int max_ctx)
{
    DecGeom g;
    g.B = B; g.Lcap = Lcap; g.n = n; g.Hq = Hq; g.Hkv = Hkv; g.D = D; g.G = Hq / Hkv;
    g.mode = mode;
    g.max_ctx = max_ctx;
    g.window = mode == 2 ? window : kNoWindow;
    g.scale_log2 = scale * 1.4426950408889634f;
    // query heads per problem: the largest divisor of G whose slots fit the 32 columns
    const int per_head = mode == 0 ? 1 : n;
    g.gchunk = 1;
    for (int c = g.G; c >= 1; --c)
        if (g.G % c == 0 && c * per_head <= kSlots) {
            g.gchunk = c;
            break;
        }
    g.ngc = g.G / g.gchunk;
    const int64_t rows = mode == 0 ? (int64_t)max_ctx + 1 : ((int64_t)max_ctx + 1) * n;
    g.nchunk = (int)((rows + kDecChunk - 1) / kDecChunk);
    g.problems = B * Hkv * g.ngc * (mode == 0 ? n : 1);
    g.nslot = g.gchunk * per_head;
    // a local layer's rows span at most the window, the other streams of the token and the
    // rounding down to a tile
    const int64_t span = mode == 2 ? (int64_t)window + n + kTile : INT32_MAX;
    dec_launch(g, (int)std::min(rows, span));
    return g;
}

size_t decode_workspace_bytes(const DecGeom &g)
{
    return (size_t)g.problems * g.nchunk * g.nslot * (g.D + 2) * sizeof(float);
}

// The scratch array of the allocation-free decode entry point.  In host code its name
// stands for a host-side shadow, not for device memory: kernels get the address that
// hipGetSymbolAddress reports for the current device.
static __device__ __align__(256) char scratch[kDecodeScratchBytes];

hipError_t decode_scratch(void **ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (addr[dev] == nullptr) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

hipError_t launch_decode_bf16(const void *q, const void *kc, const void *vc, const int32_t *ctx,
                              void *o, float *lse, const DecGeom &g, void *ws, hipStream_t s)
{
    const bf16 *qq = static_cast<const bf16 *>(q), *kk = static_cast<const bf16 *>(kc),
               *vv = static_cast<const bf16 *>(vc);
    float *part = static_cast<float *>(ws);
    bf16 *oo = static_cast<bf16 *>(o);
    const unsigned grid = (unsigned)dec_grid(g);
    const int rows = g.B * g.n * g.Hq;
    auto run = [&](auto dk, const char *pname, const char *cname) {
        constexpr int DD = decltype(dk)::value;
        timing_before(pname, s);
        auto go = [&](auto once) {
            constexpr bool ONCE = decltype(once)::value;
            if (g.waves == 8)
                sfa_decode_partial_kernel<DD, 8, ONCE><<<grid, 8 * 64, 0, s>>>(qq, kk, vv, ctx, part, oo, lse, g);
            else
                sfa_decode_partial_kernel<DD, 4, ONCE><<<grid, 4 * 64, 0, s>>>(qq, kk, vv, ctx, part, oo, lse, g);
        };
        // Streaming loads, unless another head chunk reads the rows too or, at D=32, the other half
        // of the line is another head's row (16 x 2597 rows of 3 streams, 64/8 heads of 32: 50.6 us
        // streaming, 47.3 cached; at D=64 177 streaming and 195 cached).
        if (DD > 32 && g.ngc == 1)
            go(std::bool_constant<(DD > 32)>{});
        else
            go(std::false_type{});
        hipError_t e = hipGetLastError();
        timing_after(s);
        if (e != hipSuccess || g.nsplit == 1) return e;
        timing_before(cname, s);
        sfa_decode_combine_kernel<DD><<<rows, DD, 0, s>>>(part, ctx, oo, lse, g);
        e = hipGetLastError();
        timing_after(s);
        return e;
    };
    if (g.D == 32)
        return run(std::integral_constant<int, 32>{}, "sfa_decode_bf16_d32", "sfa_decode_combine_d32");
    if (g.D == 64)
        return run(std::integral_constant<int, 64>{}, "sfa_decode_bf16_d64", "sfa_decode_combine_d64");
    return run(std::integral_constant<int, 128>{}, "sfa_decode_bf16_d128", "sfa_decode_combine_d128");
}

}  // namespace hd
