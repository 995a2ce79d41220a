// sfa_f32.hip -- fp32 Stream-Factorized Attention forward/backward (with its backward
// preprocess, which forms Delta and the base-2 lse of every query row; the bf16 path
// forms its row statistics in a kernel of its own before the dK/dV pass).
//
// All products run on the matrix cores in fp32 (16x16x4 MFMA: fp32 operands, fp32
// multiply-add), softmax in fp32; same problem decomposition as the bf16 path (see
// SfaGeom).  These layers are small (gradient checks, accuracy-first runs), so what
// bounds them is the length of the longest workgroup's serial sweep and how many CUs
// have work.  Hence:
//   tiles of 16 rows: a workgroup owns 16 or 32 query rows (forward, dQ) or keys (dK/dV)
//     of one problem, and its waves (four; eight on 16-row tiles at D < 128) take the steps
//     of the sweep over the other operand in turn, each with its own accumulators, added
//     in LDS in a fixed order at the end (the forward's after scaling to the waves' common
//     row maximum);
//   no LDS and no barrier inside a sweep: operands go from memory (L1/L2) to registers in
//     the layout the MFMA takes, the next step's loads issued as soon as the registers of
//     the current one are free;
//   dK/dV and dQ in one launch, the longer dK/dV workgroups first, so that both fill the
//     chip together.
// Measured (events, forward + preprocess + backward): B=1 L=256 n=2 Hq=8 Hkv=2 D=64, full
// cross-stream, 77 us (12 TFLOP/s; 3,630 us with one lane per row on the vector units);
// 50-63 TFLOP/s once the chip is full (B=2 L=512 n=4 Hq=12 Hkv=4), of 152 that a large
// fp32 matrix product reaches.
//
// 16x16x4 MFMA layout: lane l supplies row (A) or column (B) l % 16 at k-slot l / 16; result
// register r of lane l is row 4 (l / 16) + r, column l % 16.  Two operand forms follow:
//   row form    (k-slots run along the head dim): lane (i, g) = (l % 16, l / 16) holds
//     dims 16c + 4g .. + 3 of row i for every c, 16 bytes a load; MFMA (c, e) takes
//     element e of load c on both sides;
//   column form (k-slots run along the rows): MFMA r takes row 4g + r, the rows that result
//     register r of a score tile holds, so P and dS feed the next product from
//     registers.  Lane i loads W = min(4, D/16) consecutive dims per block group, which
//     serve W MFMAs: output row i of block b is dim (b / W) 16 W + i W + b % W.
#include "hd_device.h"

namespace hd {

namespace {

constexpr int kT = 16;      // rows or keys per MFMA tile
// Waves per workgroup, splitting the sweep: two per SIMD where their registers allow (the
// backward of B=1 L=256 n=2 Hq=8 Hkv=2: 56 against 64 us at D=64, 37 against 44 at D=32;
// at D=128, and with two subtiles at D=64, eight waves would spill).
template <int D, int NS>
constexpr int kWavesOf = D < 128 && NS == 1 ? 8 : 4;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kLog2e = 1.4426950408889634f;

__device__ inline f32x4 mfma16f(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// max / sum over the four lanes l % 16 + 16 g (g = 0 .. 3) that hold one column
__device__ inline float max_groups(float v)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return max_xor32(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ inline float sum_groups(float v)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return sum_xor32(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

__device__ inline bool not_finite(float x) { return (__float_as_uint(x) & 0x7f800000u) == 0x7f800000u; }

// Rows of one problem inside a batch slice: row i at byte base + i * stride; rows outside
// [0, len) read zeros.
struct Rows {
    rsrc_t rs;
    uint32_t base, stride;
    int len;
    __device__ inline uint32_t off(int row) const
    {
        return row >= 0 && row < len ? base + (uint32_t)row * stride : kOob;
    }
};

template <int D>
struct Ops {
    static constexpr int C = D / 16;             // row form: 16-byte loads per row and lane
    static constexpr int NB = D / 16;            // column form: 16-dim output blocks
    static constexpr int W = NB < 4 ? NB : 4;    // dims per lane and load
    static_assert(W == 4 || W == 2, "16- or 8-byte column loads");

    // element 4c + e: dim 16c + 4g + e of row row0 + i
    __device__ static inline void row_form(const Rows &m, int row0, int lane, f32x4 (&a)[C])
    {
        const uint32_t off = m.off(row0 + (lane & 15)) + (lane >> 4) * 16;
#pragma unroll
        for (int c = 0; c < C; ++c) a[c] = __builtin_bit_cast(f32x4, ld16(m.rs, off + c * 64));
    }
    // a[r][b]: row row0 + 4g + r, dim of output row i in block b
    __device__ static inline void col_form(const Rows &m, int row0, int lane, float (&a)[4][NB])
    {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t off = m.off(row0 + 4 * (lane >> 4) + r) + (lane & 15) * (W * 4);
#pragma unroll
            for (int j = 0; j < NB / W; ++j) {
                if constexpr (W == 4) {
                    const f32x4 x = __builtin_bit_cast(f32x4, ld16(m.rs, off + j * (16 * W * 4)));
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[r][j * W + e] = x[e];
                } else {
                    const auto x = __builtin_amdgcn_raw_buffer_load_b64(m.rs, off, 0, 0);
                    a[r][0] = __uint_as_float(x[0]);
                    a[r][1] = __uint_as_float(x[1]);
                }
            }
        }
    }
    // acc += A B over the head dim: rows of `a` against columns (rows) of `b`
    __device__ static inline f32x4 dot(const f32x4 (&a)[C], const f32x4 (&b)[C], f32x4 acc)
    {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = mfma16f(a[c][e], b[c][e], acc);
        return acc;
    }
    // acc^T += A^T w: the 16 rows of column form `a` weighted by w (register r: row 4g + r)
    __device__ static inline void add(const float (&a)[4][NB], const f32x4 &w, f32x4 (&acc)[NB])
    {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] = mfma16f(a[r][b], w[r], acc[b]);
    }
    // Same on a tile with masked pairs, whose weights are zero.  A masked pair must add
    // nothing even where its row holds an infinity or a NaN (0 * inf is NaN), so such
    // elements leave the MFMA and are added one by one for the visible pairs.  That path is
    // rare: it works on accumulators parked in `park` (this wave's, NB * 256 floats of LDS) in
    // plain loops, so that it costs the common one no registers.  vis(j): row row0 + j is
    // visible to this lane's column.
    template <typename Vis>
    __device__ static inline void add_masked(const Rows &m, int row0, int lane, float *park,
                                             const float (&a)[4][NB], const f32x4 &w, f32x4 (&acc)[NB], Vis vis)
    {
        bool bad = false;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int b = 0; b < NB; ++b) bad = bad || not_finite(a[r][b]);
        if (__any(bad)) {
            mfma_settle();
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) park[(b * 4 + q) * 64 + lane] = acc[b][q];
#pragma unroll 1
            for (int j = 0; j < kT; ++j) {
                const int r = j & 3;
                const float wj = r == 0 ? w[0] : r == 1 ? w[1] : r == 2 ? w[2] : w[3];
                const float wr = __shfl(wj, (lane & 15) + 16 * (j >> 2));
                const uint32_t off = m.off(row0 + j);
                const bool v = vis(j);
#pragma unroll 1
                for (int x = 0; x < NB * 4; ++x) {
                    const int b = x >> 2, q = x & 3;
                    const uint32_t d = (b / W) * 16 * W + (4 * (lane >> 4) + q) * W + b % W;
                    const float y = __uint_as_float(ld4(m.rs, off + d * 4));
                    if (v && not_finite(y)) park[x * 64 + lane] = __builtin_fmaf(wr, y, park[x * 64 + lane]);
                }
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[b][q] = park[(b * 4 + q) * 64 + lane];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[b] = mfma16f(not_finite(a[r][b]) ? 0.f : a[r][b], w[r], acc[b]);
            mfma_settle();
        } else {
            add(a, w, acc);
            mfma_settle();
        }
    }
};

// Writes elements r = wave of the 16-dim blocks of one column's accumulators, summed over
// the waves: store(dim, four or two consecutive dims).
template <int D, int NS>
struct Merge {
    static constexpr int kWaves = kWavesOf<D, NS>;
    // [wave][subtile][block][register][lane]
    float v[kWaves][NS][Ops<D>::NB][4][64];
    __device__ inline void put(int wave, int sub, int lane, const f32x4 (&acc)[Ops<D>::NB])
    {
#pragma unroll
        for (int b = 0; b < Ops<D>::NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[wave][sub][b][r][lane] = acc[b][r];
    }
    // sum over the waves of block b, register r, each wave scaled by sc[wave]
    __device__ inline float sum(int sub, int b, int r, int lane, const float (&sc)[kWaves]) const
    {
        float s = v[0][sub][b][r][lane] * sc[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) s = __builtin_fmaf(v[w][sub][b][r][lane], sc[w], s);
        return s;
    }
    // register r of this lane's column, dims in order, scaled by f
    // (waves 0 .. 3, one register each)
    template <typename Store>
    __device__ inline void get(int sub, int r, int lane, const float (&sc)[kWaves], float f, Store store) const
    {
        constexpr int W = Ops<D>::W;
        if (r >= 4) return;
#pragma unroll
        for (int j = 0; j < Ops<D>::NB / W; ++j) {
            float x[W];
#pragma unroll
            for (int e = 0; e < W; ++e) x[e] = sum(sub, j * W + e, r, lane, sc) * f;
            store(j * 16 * W + (4 * (lane >> 4) + r) * W, x);
        }
    }
};

__device__ inline void store_dims(rsrc_t rs, uint32_t off, const float (&x)[4])
{
    st16(rs, off, u32x4{__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])});
}
__device__ inline void store_dims(rsrc_t rs, uint32_t off, const float (&x)[2])
{
    st8(rs, off, u32x2{__float_as_uint(x[0]), __float_as_uint(x[1])});
}

// Work item -> (problem, tile) as decode_tile does, for item counts beyond 32 bits.
__device__ inline void decode_item(int64_t id, int nprob, int ntiles, int &prob, int &tile)
{
    if ((nprob & 7) == 0) {
        const int per = nprob >> 3;
        const int64_t r = id >> 3;
        tile = ntiles - 1 - (int)(r / per);
        prob = (int)(id & 7) * per + (int)(r % per);
    } else {
        tile = ntiles - 1 - (int)(id / nprob);
        prob = (int)(id % nprob);
    }
}

// One (batch, query head[, stream]) or (batch, key head[, stream]) problem.
struct Where {
    int s, h, b;
};
__device__ inline Where where(const SfaGeom &g, int prob, int heads)
{
    return Where{prob % g.streams, prob / g.streams % heads, prob / (g.streams * heads)};
}
template <int D>
__device__ inline Rows rows_of(const float *p, const SfaGeom &g, int b, int heads, int h, int s)
{
    const size_t slice = (size_t)g.N * heads * D;
    return Rows{make_rsrc(p + b * slice, (uint32_t)(slice * 4)), (uint32_t)(s * heads + h) * D * 4,
                (uint32_t)g.rowmul * heads * D * 4, g.len};
}

// Forward: NQ * 16 query rows; the waves take 32-key steps.  S^T = K Q^T puts a query's
// scores in the four lanes of one column; O^T += V^T P^T.
template <int D, int NQ>
__global__ __launch_bounds__((kWavesOf<D, NQ> * 64), 1) void sfa_fwd_f32_kernel(const float *__restrict__ q,
                                                                  const float *__restrict__ k,
                                                                  const float *__restrict__ v,
                                                                  float *__restrict__ o,
                                                                  float *__restrict__ lse, SfaGeom g,
                                                                  int64_t items)
{
    using P = Ops<D>;
    constexpr int kWaves = kWavesOf<D, NQ>;
    constexpr int KS = 2, KT = KS * kT;  // keys per step
    __shared__ Merge<D, NQ> mg;
    __shared__ float sm[kWaves][NQ][16], sl[kWaves][NQ][16];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, gr = lane >> 4;
    const int ntiles = (g.len + NQ * kT - 1) / (NQ * kT);
    for (int64_t id = blockIdx.x; id < items; id += gridDim.x) {
        int prob, tile;
        decode_item(id, g.B * g.Hq * g.streams, ntiles, prob, tile);
        const Where at = where(g, prob, g.Hq);
        const Rows rq = rows_of<D>(q, g, at.b, g.Hq, at.h, at.s);
        const Rows rk = rows_of<D>(k, g, at.b, g.Hkv, at.h / g.G, at.s);
        const Rows rv = rows_of<D>(v, g, at.b, g.Hkv, at.h / g.G, at.s);
        const Rows ro = rows_of<D>(o, g, at.b, g.Hq, at.h, at.s);
        const int q0 = tile * NQ * kT, qlast = q0 + NQ * kT - 1;

        f32x4 qr[NQ][P::C], oacc[NQ][P::NB];
        float m[NQ], l[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            P::row_form(rq, q0 + i * kT, lane, qr[i]);
#pragma unroll
            for (int b = 0; b < P::NB; ++b) oacc[i][b] = f32x4{};
            m[i] = -INFINITY;
            l[i] = 0.f;
        }
        // 32-key steps from the first key the window reaches to the diagonal
        const int jf = max(0, q0 - g.window + 1) / KT;
        const int je = (min(g.len, qlast + 1) + KT - 1) / KT;
        f32x4 kr[KS][P::C];
        float vc[KS][4][P::NB];
        auto load_k = [&](int j) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < KS; ++t) P::row_form(rk, j * KT + t * kT, lane, kr[t]);
        };
        auto load_v = [&](int j) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < KS; ++t) P::col_form(rv, j * KT + t * kT, lane, vc[t]);
        };
        int j = jf + wave;
        if (j < je) {
            load_k(j);
            load_v(j);
        }
        for (; j < je; j += kWaves) {
            const int kb = j * KT;
            f32x4 sc[KS][NQ];
#pragma unroll
            for (int t = 0; t < KS; ++t)
#pragma unroll
                for (int i = 0; i < NQ; ++i) sc[t][i] = P::dot(kr[t], qr[i], f32x4{});
            mfma_settle();
            if (j + kWaves < je) load_k(j + kWaves);
            const bool masked = kb + KT - 1 > q0 || qlast - kb >= g.window;
            auto visible = [&](int key, int i) __attribute__((always_inline)) {
                const int d = q0 + i * kT + col - key;
                return d >= 0 && d < g.window;
            };
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                float mx = -INFINITY;
#pragma unroll
                for (int t = 0; t < KS; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float x = sc[t][i][r] * g.scale_log2;
                        if (masked && !visible(kb + t * kT + 4 * gr + r, i)) x = -INFINITY;
                        sc[t][i][r] = x;
                        mx = fmaxf(mx, x);
                    }
                const float mn = fmaxf(m[i], max_groups(mx));
                if (__any(mn > m[i])) {
                    const float alpha = mn == m[i] ? 1.f : exp2f(m[i] - mn);
                    m[i] = mn;
                    l[i] *= alpha;
#pragma unroll
                    for (int b = 0; b < P::NB; ++b) oacc[i][b] *= alpha;
                }
                // a row without a visible key so far: weights exp2(-inf) = 0, not NaN
                const float me = mn == -INFINITY ? 0.f : mn;
#pragma unroll
                for (int t = 0; t < KS; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        sc[t][i][r] = exp2f(sc[t][i][r] - me);
                        l[i] += sc[t][i][r];
                    }
            }
#pragma unroll
            for (int t = 0; t < KS; ++t)
#pragma unroll
                for (int i = 0; i < NQ; ++i)
                    if (masked)
                        P::add_masked(rv, kb + t * kT, lane, &mg.v[wave][0][0][0][0], vc[t], sc[t][i], oacc[i],
                                      [&](int x) { return visible(kb + t * kT + x, i); });
                    else
                        P::add(vc[t], sc[t][i], oacc[i]);
            if (j + kWaves < je) load_v(j + kWaves);
        }
        mfma_settle();
        // merge the waves: the row's largest maximum, then each wave's share scaled to it
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            mg.put(wave, i, lane, oacc[i]);
            const float lt = sum_groups(l[i]);
            if (gr == 0) {
                sm[wave][i][col] = m[i];
                sl[wave][i][col] = lt;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int row = q0 + i * kT + col;
            float mt = sm[0][i][col], lt = 0.f, scl[kWaves];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) mt = fmaxf(mt, sm[w][i][col]);
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                // a wave without a step of this row has m = -inf, l = 0 and O = 0
                scl[w] = sm[w][i][col] == -INFINITY && mt == -INFINITY ? 1.f : exp2f(sm[w][i][col] - mt);
                lt = __builtin_fmaf(sl[w][i][col], scl[w], lt);
            }
            const uint32_t off = ro.off(row);
            mg.get(i, wave, lane, scl, 1.f / lt,
                   [&](int d, const float(&x)[P::W]) { store_dims(ro.rs, off + d * 4, x); });
            if (wave == 0 && gr == 0 && row < g.len)
                lse[((size_t)at.b * g.Hq + at.h) * g.N + (size_t)row * g.rowmul + at.s] =
                    (mt + log2f(lt)) * kLn2;
        }
        __syncthreads();
    }
}

// Per (b, hq, p) query row: delta = sum_d dO * O and lse2 = lse * log2(e).  One group
// of lanes per row, 16 bytes per lane, reduced with xor shuffles.
template <int D>
__global__ __launch_bounds__(256) void bwd_preprocess_kernel(const float *__restrict__ o,
                                                             const float *__restrict__ dO,
                                                             const float *__restrict__ lse,
                                                             float *__restrict__ delta,
                                                             float *__restrict__ lse2, SfaGeom g)
{
    constexpr int LPR = D / 4;      // lanes per row, 4 floats each
    constexpr int RPB = 256 / LPR;  // rows per workgroup
    const size_t rows = (size_t)g.B * g.N * g.Hq;
    const size_t r = (size_t)blockIdx.x * RPB + threadIdx.x / LPR;
    const int part = threadIdx.x % LPR;
    float acc = 0.f;
    if (r < rows) {
        const u32x4 a = *reinterpret_cast<const u32x4 *>(o + r * D + part * 4);
        const u32x4 c = *reinterpret_cast<const u32x4 *>(dO + r * D + part * 4);
#pragma unroll
        for (int w = 0; w < 4; ++w) acc = __builtin_fmaf(__uint_as_float(a[w]), __uint_as_float(c[w]), acc);
    }
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (r < rows && part == 0) {
        const int hq = (int)(r % g.Hq);
        const size_t bp = r / g.Hq;  // b * N + p
        const size_t b = bp / g.N, p = bp % g.N;
        const size_t li = (b * g.Hq + hq) * g.N + p;
        delta[li] = acc;
        lse2[li] = lse[li] * kLog2e;
    }
}

// dK/dV of NS * 16 keys: the waves take (query tile, query head of the group) pairs.
// S = Q K^T and dP = dO V^T put a key's pairs in the lanes of one column;
// dV^T += dO^T P, dK^T += Q^T dS.
template <int D, int NS>
__device__ inline void dkdv_f32(const float *q, const float *k, const float *v, const float *dO,
                                const float *delta, const float *lse2, float *dk, float *dv,
                                const SfaGeom &g, int64_t id, Merge<D, NS> &mg)
{
    using P = Ops<D>;
    constexpr int kWaves = kWavesOf<D, NS>;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, gr = lane >> 4;
    const int ntiles = (g.len + NS * kT - 1) / (NS * kT);
    int prob, tile;
    decode_item(id, g.B * g.Hkv * g.streams, ntiles, prob, tile);
    tile = ntiles - 1 - tile;  // early keys, which most queries see, first
    const Where at = where(g, prob, g.Hkv);
    const Rows rk = rows_of<D>(k, g, at.b, g.Hkv, at.h, at.s);
    const Rows rv = rows_of<D>(v, g, at.b, g.Hkv, at.h, at.s);
    const int k0 = tile * NS * kT, klast = k0 + NS * kT - 1;

    f32x4 kb[NS][P::C], vb[NS][P::C], ak[NS][P::NB], av[NS][P::NB];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        P::row_form(rk, k0 + i * kT, lane, kb[i]);
        P::row_form(rv, k0 + i * kT, lane, vb[i]);
#pragma unroll
        for (int b = 0; b < P::NB; ++b) ak[i][b] = av[i][b] = f32x4{};
    }
    // query tiles that see one of the keys, every head of the group in turn
    const int tf = k0 / kT;
    const int64_t qend = min((int64_t)g.len, (int64_t)klast + g.window);
    const int nit = ((int)((qend + kT - 1) / kT) - tf) * g.G;
    f32x4 qr[P::C], dr[P::C];
    float qc[4][P::NB], dc[4][P::NB], l2[4], dl[4];
    Rows rq = rows_of<D>(q, g, at.b, g.Hq, at.h * g.G, at.s), rd = rq;
    rd.rs = rows_of<D>(dO, g, at.b, g.Hq, at.h * g.G, at.s).rs;
    const uint32_t qbase = rq.base;
    auto place = [&](int it) __attribute__((always_inline)) {  // head and first row of item `it`
        rq.base = rd.base = qbase + (uint32_t)(it % g.G) * D * 4;
        return (tf + it / g.G) * kT;
    };
    auto load_rows = [&](int it) __attribute__((always_inline)) {
        const int row0 = place(it);
        P::row_form(rq, row0, lane, qr);
        P::row_form(rd, row0, lane, dr);
        const size_t lb = ((size_t)at.b * g.Hq + at.h * g.G + it % g.G) * g.N + at.s;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const size_t x = lb + (size_t)min(row0 + 4 * gr + r, g.len - 1) * g.rowmul;
            l2[r] = lse2[x];
            dl[r] = delta[x];
        }
    };
    auto load_cols = [&](int it) __attribute__((always_inline)) {
        const int row0 = place(it);
        P::col_form(rq, row0, lane, qc);
        P::col_form(rd, row0, lane, dc);
    };
    int it = wave;
    if (it < nit) {
        load_rows(it);
        load_cols(it);
    }
    for (; it < nit; it += kWaves) {
        const int row0 = (tf + it / g.G) * kT;
        const bool masked = klast > row0 || row0 + kT - 1 - k0 >= g.window || row0 + kT > g.len;
        f32x4 p[NS], ds[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            p[i] = P::dot(qr, kb[i], f32x4{});
            ds[i] = P::dot(dr, vb[i], f32x4{});
        }
        mfma_settle();
        auto visible = [&](int row, int i) __attribute__((always_inline)) {
            const int d = row - (k0 + i * kT + col);
            return d >= 0 && d < g.window && row < g.len;
        };
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float x = exp2f(__builtin_fmaf(p[i][r], g.scale_log2, -l2[r]));
                float y = x * (ds[i][r] - dl[r]);
                if (masked && !visible(row0 + 4 * gr + r, i)) x = y = 0.f;
                p[i][r] = x;
                ds[i][r] = y;
            }
        if (it + kWaves < nit) load_rows(it + kWaves);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            if (masked) {
                place(it);
                float *park = &mg.v[wave][0][0][0][0];
                auto vis = [&](int x) { return visible(row0 + x, i); };
                P::add_masked(rd, row0, lane, park, dc, p[i], av[i], vis);
                P::add_masked(rq, row0, lane, park, qc, ds[i], ak[i], vis);
            } else {
                P::add(dc, p[i], av[i]);
                P::add(qc, ds[i], ak[i]);
            }
        }
        if (it + kWaves < nit) load_cols(it + kWaves);
    }
    mfma_settle();
    float one[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) one[w] = 1.f;
    const Rows wk = rows_of<D>(dk, g, at.b, g.Hkv, at.h, at.s);
    const Rows wv = rows_of<D>(dv, g, at.b, g.Hkv, at.h, at.s);
#pragma unroll
    for (int x = 0; x < 2; ++x) {
#pragma unroll
        for (int i = 0; i < NS; ++i) mg.put(wave, i, lane, x == 0 ? ak[i] : av[i]);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const uint32_t off = wk.off(k0 + i * kT + col);
            mg.get(i, wave, lane, one, x == 0 ? g.scale : 1.f, [&](int d, const float(&y)[P::W]) {
                store_dims(x == 0 ? wk.rs : wv.rs, off + d * 4, y);
            });
        }
        __syncthreads();
    }
}

// dQ of NS * 16 query rows: the waves take 16-key tiles.  S^T = K Q^T, dP^T = V dO^T,
// dQ^T += K^T dS^T.
template <int D, int NS>
__device__ inline void dq_f32(const float *q, const float *k, const float *v, const float *dO,
                              const float *delta, const float *lse2, float *dq, const SfaGeom &g,
                              int64_t id, Merge<D, NS> &mg)
{
    using P = Ops<D>;
    constexpr int kWaves = kWavesOf<D, NS>;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, gr = lane >> 4;
    const int ntiles = (g.len + NS * kT - 1) / (NS * kT);
    int prob, tile;
    decode_item(id, g.B * g.Hq * g.streams, ntiles, prob, tile);
    const Where at = where(g, prob, g.Hq);
    const Rows rq = rows_of<D>(q, g, at.b, g.Hq, at.h, at.s);
    const Rows rd = rows_of<D>(dO, g, at.b, g.Hq, at.h, at.s);
    const Rows rk = rows_of<D>(k, g, at.b, g.Hkv, at.h / g.G, at.s);
    const Rows rv = rows_of<D>(v, g, at.b, g.Hkv, at.h / g.G, at.s);
    const int q0 = tile * NS * kT, qlast = q0 + NS * kT - 1;

    f32x4 qb[NS][P::C], db[NS][P::C], acc[NS][P::NB];
    float l2[NS], dl[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        P::row_form(rq, q0 + i * kT, lane, qb[i]);
        P::row_form(rd, q0 + i * kT, lane, db[i]);
        const size_t x = ((size_t)at.b * g.Hq + at.h) * g.N +
                         (size_t)min(q0 + i * kT + col, g.len - 1) * g.rowmul + at.s;
        l2[i] = lse2[x];
        dl[i] = delta[x];
#pragma unroll
        for (int b = 0; b < P::NB; ++b) acc[i][b] = f32x4{};
    }
    const int jf = max(0, q0 - g.window + 1) / kT;
    const int je = (min(g.len, qlast + 1) + kT - 1) / kT;
    f32x4 kr[P::C], vr[P::C];
    float kc[4][P::NB];
    auto load_rows = [&](int j) __attribute__((always_inline)) {
        P::row_form(rk, j * kT, lane, kr);
        P::row_form(rv, j * kT, lane, vr);
    };
    int j = jf + wave;
    if (j < je) {
        load_rows(j);
        P::col_form(rk, j * kT, lane, kc);
    }
    for (; j < je; j += kWaves) {
        const int kb = j * kT;
        const bool masked = kb + kT - 1 > q0 || qlast - kb >= g.window;
        f32x4 p[NS], ds[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            p[i] = P::dot(kr, qb[i], f32x4{});
            ds[i] = P::dot(vr, db[i], f32x4{});
        }
        mfma_settle();
        if (j + kWaves < je) load_rows(j + kWaves);
        auto visible = [&](int key, int i) __attribute__((always_inline)) {
            const int d = q0 + i * kT + col - key;
            return d >= 0 && d < g.window;
        };
#pragma unroll
        for (int i = 0; i < NS; ++i) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float x = exp2f(__builtin_fmaf(p[i][r], g.scale_log2, -l2[i]));
                const float y = x * (ds[i][r] - dl[i]);
                ds[i][r] = masked && !visible(kb + 4 * gr + r, i) ? 0.f : y;
            }
            if (masked)
                P::add_masked(rk, kb, lane, &mg.v[wave][0][0][0][0], kc, ds[i], acc[i], [&](int x) { return visible(kb + x, i); });
            else
                P::add(kc, ds[i], acc[i]);
        }
        if (j + kWaves < je) P::col_form(rk, (j + kWaves) * kT, lane, kc);
    }
    mfma_settle();
    float one[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) one[w] = 1.f;
    const Rows wq = rows_of<D>(dq, g, at.b, g.Hq, at.h, at.s);
#pragma unroll
    for (int i = 0; i < NS; ++i) mg.put(wave, i, lane, acc[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const uint32_t off = wq.off(q0 + i * kT + col);
        mg.get(i, wave, lane, one, g.scale,
               [&](int d, const float(&y)[P::W]) { store_dims(wq.rs, off + d * 4, y); });
    }
    __syncthreads();
}

// dK/dV work items [0, nkv), then dQ items
template <int D, int NS>
__global__ __launch_bounds__((kWavesOf<D, NS> * 64), 1) void sfa_bwd_f32_kernel(
    const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
    const float *__restrict__ dO, const float *__restrict__ delta, const float *__restrict__ lse2,
    float *__restrict__ dq, float *__restrict__ dk, float *__restrict__ dv, SfaGeom g, int64_t nkv,
    int64_t items)
{
    __shared__ Merge<D, NS> mg;
    for (int64_t id = blockIdx.x; id < items; id += gridDim.x) {
        if (id < nkv)
            dkdv_f32<D, NS>(q, k, v, dO, delta, lse2, dk, dv, g, id, mg);
        else
            dq_f32<D, NS>(q, k, v, dO, delta, lse2, dq, g, id - nkv, mg);
    }
}

// 32 rows or keys per workgroup halve the operand bytes per product; 16 double the
// workgroups and halve the longest one.  The larger tile is taken once it still gives every
// CU two workgroups: at B=1 L=256 n=2 Hq=8 Hkv=2 D=64 (64 key tiles of 16) the backward
// takes 56 us narrow and 106 us wide, at B=2 L=512 n=4 Hq=12 Hkv=4 D=32 (512 of 32)
// 112 narrow and 88 wide.
constexpr int64_t kWideItems = 512;

// Items beyond the grid are strided over it (a grid's work-items must fit 32 bits).
unsigned grid_of(int64_t items) { return (unsigned)(items < (1 << 22) ? items : (1 << 22)); }

template <int D>
hipError_t fwd_f32_d(const float *q, const float *k, const float *v, float *o, float *lse,
                     const SfaGeom &g, hipStream_t s)
{
    const int64_t nprob = (int64_t)g.B * g.Hq * g.streams;
    const int64_t wide = (g.len + 31) / 32 * nprob, narrow = (g.len + 15) / 16 * nprob;
    timing_before("sfa_fwd_f32", s);
    if (wide >= kWideItems)
        sfa_fwd_f32_kernel<D, 2><<<grid_of(wide), kWavesOf<D, 2> * 64, 0, s>>>(q, k, v, o, lse, g, wide);
    else
        sfa_fwd_f32_kernel<D, 1><<<grid_of(narrow), kWavesOf<D, 1> * 64, 0, s>>>(q, k, v, o, lse, g, narrow);
    hipError_t e = hipGetLastError();
    timing_after(s);
    return e;
}

template <int D>
hipError_t bwd_f32_d(const float *q, const float *k, const float *v, const float *dO,
                     float *dq, float *dk, float *dv, const SfaGeom &g, float *delta,
                     float *lse2, hipStream_t s)
{
    const int64_t pq = (int64_t)g.B * g.Hq * g.streams, pk = (int64_t)g.B * g.Hkv * g.streams;
    const int64_t wide = (g.len + 31) / 32, narrow = (g.len + 15) / 16;
    timing_before("sfa_bwd_f32", s);
    // at D = 128 two key subtiles do not fit the registers
    constexpr int kWide = D < 128 ? 2 : 1;
    if (kWide == 2 && wide * pk >= kWideItems)
        sfa_bwd_f32_kernel<D, kWide><<<grid_of(wide * (pk + pq)), kWavesOf<D, kWide> * 64, 0, s>>>(
            q, k, v, dO, delta, lse2, dq, dk, dv, g, wide * pk, wide * (pk + pq));
    else
        sfa_bwd_f32_kernel<D, 1><<<grid_of(narrow * (pk + pq)), kWavesOf<D, 1> * 64, 0, s>>>(
            q, k, v, dO, delta, lse2, dq, dk, dv, g, narrow * pk, narrow * (pk + pq));
    hipError_t e = hipGetLastError();
    timing_after(s);
    return e;
}

}  // namespace

hipError_t launch_bwd_preprocess_f32(const float *o, const float *dO, const float *lse,
                                     float *delta, float *lse2, const SfaGeom &g, hipStream_t s)
{
    const size_t rows = (size_t)g.B * g.N * g.Hq;
    const int lpr = g.D * 4 / 16;
    const int rpb = 256 / lpr;
    const dim3 grid((unsigned)((rows + rpb - 1) / rpb));
    timing_before("sfa_bwd_preprocess_f32", s);
    if (g.D == 32)
        bwd_preprocess_kernel<32><<<grid, 256, 0, s>>>(o, dO, lse, delta, lse2, g);
    else if (g.D == 64)
        bwd_preprocess_kernel<64><<<grid, 256, 0, s>>>(o, dO, lse, delta, lse2, g);
    else
        bwd_preprocess_kernel<128><<<grid, 256, 0, s>>>(o, dO, lse, delta, lse2, g);
    hipError_t e = hipGetLastError();
    timing_after(s);
    return e;
}

hipError_t launch_fwd_f32(const float *q, const float *k, const float *v, float *o, float *lse,
                          const SfaGeom &g, hipStream_t s)
{
    if (g.D == 32) return fwd_f32_d<32>(q, k, v, o, lse, g, s);
    if (g.D == 64) return fwd_f32_d<64>(q, k, v, o, lse, g, s);
    return fwd_f32_d<128>(q, k, v, o, lse, g, s);
}

hipError_t launch_bwd_f32(const float *q, const float *k, const float *v, const float *o,
                          const float *lse, const float *dO, float *dq, float *dk, float *dv,
                          const SfaGeom &g, void *ws, hipStream_t s)
{
    const BwdWorkspace w = bwd_workspace(g, 4);
    float *delta = reinterpret_cast<float *>(static_cast<char *>(ws) + w.delta);
    float *lse2 = reinterpret_cast<float *>(static_cast<char *>(ws) + w.lse2);
    hipError_t e = launch_bwd_preprocess_f32(o, dO, lse, delta, lse2, g, s);
    if (e != hipSuccess) return e;
    if (g.D == 32) return bwd_f32_d<32>(q, k, v, dO, dq, dk, dv, g, delta, lse2, s);
    if (g.D == 64) return bwd_f32_d<64>(q, k, v, dO, dq, dk, dv, g, delta, lse2, s);
    return bwd_f32_d<128>(q, k, v, dO, dq, dk, dv, g, delta, lse2, s);
}

}  // namespace hd
