// sfa_fwd_bf16.hip -- Stream-Factorized Attention forward, bf16 in/out, fp32 softmax.
//
// Computes, per causal problem (see SfaGeom), O = softmax(scale Q K^T + mask) V and the
// natural-log row log-sum-exp: the forward of the intra-stream layer (eq. (mask_intra))
// and of the full cross-stream layer (causal mask of Fig. "masks"(a)).
//
// Tiling (gfx950, wave64):
//   workgroup = 8 waves = 256 query rows of one problem (two waves per SIMD); wave w
//   owns rows 32w..32w+31 and each lane keeps one query row (column l%32 of the MFMA
//   results).  (Small grids take 128-row blocks, see Shape.)  The transposed score tile S^T = K Q^T puts a row's scores in one lane,
//   so the row max / row sum need one cross-half exchange, and P^T feeds the second
//   MFMA (O^T += V^T P^T) straight from registers.
//   Key/value tiles of 64 rows are loaded HBM -> LDS by direct-to-LDS buffer loads
//   into a double buffer (one barrier per tile); K is read row-wise, V through
//   transposed LDS reads, both from the same swizzled row-major layout.
//   Only tiles at or below a wave's diagonal are computed; the causal mask is applied
//   on diagonal tiles alone.  The running max is refreshed only when it grows by more
//   than 2^8 (log2 units), so the O rescale is rare; results are exact either way
//   because the normaliser uses the same reference.
#include <type_traits>

#include "sfa_lds.h"

namespace hd {

namespace {

constexpr int kWaves = 8;
constexpr int kBM = kWaves * 32;           // query rows per workgroup
constexpr int kLoaders = 4;                // group B (waves 4-7) issues the tile loads
constexpr float kRescaleThreshold = 8.0f;  // log2 units

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// FINAL: final-stream layer (query row i at key coordinate i*n + n - 1, strided wave
// rows); otherwise query row i is key coordinate i and waves take consecutive rows.
// Block shapes.  kPlain: 256 rows, one workgroup per CU at D >= 64.  kShared (D = 64): the same
// held to 128 registers, so that two workgroups share a CU.  kSplit: a block holds 128 rows,
// both groups of waves own the same ones (wave w and w + 4 rows 32w ..) and take every second
// key tile each, group B the odd ones, through rings of their own; at the end group A adds
// group B's part, scaled to the common reference.  Half the phases per block, twice the blocks.
enum Shape { kPlain, kShared, kSplit };

template <int D, bool FINAL, Shape SHAPE>
__global__ __launch_bounds__((kWaves * 64), (SHAPE == kShared ? 4 : 2)) void sfa_fwd_bf16_kernel(
    const bf16 *__restrict__ q, const bf16 *__restrict__ k, const bf16 *__restrict__ v,
    bf16 *__restrict__ o, float *__restrict__ lse, SfaGeom g)
{
    constexpr bool SPLIT = SHAPE == kSplit;
    constexpr int KS = D / 16;  // MFMA k-steps over the head dim
    constexpr int DB = D / 32;  // 32-wide head-dim blocks of O
    using T = Tile<D>;
    // two-slot K and V rings (tile t in slot t % 2); every slot is an immediate offset
    // from one per-lane address
    // (split: one pair of rings per group, which at the end hold group B's part: per wave and
    // lane 16 DB accumulators, the reference and the row sum)
    constexpr int NR = SPLIT ? 2 : 1;
    constexpr int BM = SPLIT ? kBM / 2 : kBM;
    __shared__ __attribute__((aligned(1024))) char kv[NR][4][T::BYTES];
    static_assert(!SPLIT || sizeof(kv) >= 4 * (16 * DB + 2) * 64 * sizeof(float), "group B's part must fit in the rings");

    const int ntiles = (g.qlen + BM - 1) / BM;
    const int nprob = g.B * g.Hq * g.streams;
    int prob, tile;
    decode_tile(blockIdx.x, nprob, ntiles, prob, tile);
    const int s = prob % g.streams;
    const int hq = (prob / g.streams) % g.Hq;
    const int b = prob / (g.streams * g.Hq);
    const int hk = hq / g.G;

    // per-batch slices; all in-slice byte offsets fit in 31 bits
    const size_t qslice = (size_t)g.qN * g.Hq * D, kslice = (size_t)g.N * g.Hkv * D;
    const rsrc_t rq = make_rsrc(q + b * qslice, (uint32_t)(qslice * 2));
    const rsrc_t rk = make_rsrc(k + b * kslice, (uint32_t)(kslice * 2));
    const rsrc_t rv = make_rsrc(v + b * kslice, (uint32_t)(kslice * 2));
    const rsrc_t ro = make_rsrc(o + b * qslice, (uint32_t)(qslice * 2));
    const uint32_t qstride = (uint32_t)g.qrowmul * g.Hq * D * 2;
    const uint32_t qbase = (uint32_t)(s * g.Hq + hq) * D * 2;
    const uint32_t kstride = (uint32_t)g.rowmul * g.Hkv * D * 2;
    const uint32_t kbase0 = (uint32_t)(s * g.Hkv + hk) * D * 2;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: scalar branches
    const int group = wave >> 2;  // 0: A, 1: B (one wave of each per SIMD)
    const int l32 = lane & 31, hi = lane >> 5;
    char (&ks)[2][T::BYTES] = *reinterpret_cast<char (*)[2][T::BYTES]>(kv[SPLIT ? group : 0]);
    char (&vs)[2][T::BYTES] = *reinterpret_cast<char (*)[2][T::BYTES]>(kv[SPLIT ? group : 0] + 2);
    const int q0 = tile * BM;
    constexpr int RW = BM / 32;                // waves that share the block's rows
    const int rw = SPLIT ? wave & 3 : wave;    // my place among them
    constexpr int TS = SPLIT ? 2 : 1;          // key tiles between my tiles
    const int t0 = SPLIT ? group : 0;          // my first key tile of the block
    // This wave's 32 query rows: 32 consecutive rows, or, in final-stream layers (whose
    // queries advance n key positions per row), rows rw, rw + RW, ... of the block,
    // so that all waves reach (about) the same last key tile.
    auto P = [&](int i) __attribute__((always_inline)) { return FINAL ? qpos(g, i) : i; };
    const int row = FINAL ? q0 + rw + RW * l32 : q0 + rw * 32 + l32;
    const int wrow_min = FINAL ? q0 + rw : q0 + rw * 32;
    const int wrow_max = FINAL ? wrow_min + RW * 31 : wrow_min + 31;

    // keys of the block: up to the key coordinate of its last query row
    const int kend = min(g.len, P(min(q0 + BM, g.qlen) - 1) + 1);
    const int nkt = (kend + kRows - 1) / kRows;
    // Tiles are numbered from jf, the first one holding a key that a row of this
    // workgroup sees (0 unless the layer is local); t below counts my tiles from there:
    // tile t is key tile jf + t0 + t TS.
    const int jf = max(0, P(q0) - g.window + 1) / kRows;
    const int ntl = (nkt - jf + TS - 1) / TS;
    // last tile with keys this wave sees (split: group B may have none, -1)
    const int jlast = (min(nkt - 1, P(wrow_max) / kRows) - jf - t0 + TS) / TS - 1;
    auto key0 = [&](int t) __attribute__((always_inline)) { return (jf + t0 + t * TS) * kRows; };

    // this lane's query row as the B operand of S^T = K Q^T
    bf16x8 qr[KS];
    {
        const uint32_t off = row < g.qlen ? qbase + (uint32_t)row * qstride : kOob;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
            qr[kk] = __builtin_bit_cast(bf16x8, ld16(rq, off + (kk * 16 + hi * 8) * 2));
    }

    // per-lane address parts (K and V share the row layout)
    const bool loader = SPLIT || wave >= kWaves - kLoaders;  // the waves of group B, or of each
    const int lw = loader ? wave & (kLoaders - 1) : 0;
    const auto dma = T::template dma_plan<kLoaders>(kbase0, kstride, lw, lane);
    uint32_t kro[KS], vto[DB][2];
    T::row_offsets(l32, hi, kro);
    T::tr_offsets(lane, vto);
    // loader waves queue their shares of K of tile t+2 and V of tile t+1 in their
    // vector phase of tile t (or, once past their last tile, before the barrier that
    // ends it) and wait for them at the end of their next phase
    auto issue = [&](int t) __attribute__((always_inline)) {
        if (loader) {
            if (t + 2 < ntl)
                T::load(ks[t & 1], rk, dma, (uint32_t)key0(t + 2) * kstride, lw);
            if (t + 1 < ntl)
                T::load(vs[(t + 1) & 1], rv, dma, (uint32_t)key0(t + 1) * kstride, lw);
        }
    };

    f32x16 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db] = f32x16{};
    f32x16 sc[2];               // scores of the tile whose softmax comes next
    bf16x8 pb[4];               // bf16 weights of the tile whose P V product comes next
    float m2 = -INFINITY;       // reference max in log2 units
    float lsum0 = 0.f, lsum1 = 0.f;  // this lane half's share of the row sum (two chains)
    const float c2 = g.scale_log2;
    const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);

    // the tile holds keys past this wave's first row (diagonal) or, in a local layer,
    // keys at least a window before its last row
    auto needs_mask = [&](int t) __attribute__((always_inline)) {
        const int kb = key0(t);
        return kb + kRows - 1 > P(wrow_min) || kb <= P(wrow_max) - g.window;
    };

    // Matrix phase of tile t: the scores of tile t+1 (DO_S) and O^T += V^T P^T of
    // tile t (DO_PV).  On the tile that holds this wave's diagonal the score
    // accumulators start at -inf for keys past the lane's row, so masked scores come
    // out as -inf (exp2 -> 0) and the softmax needs no mask; other tiles start from the
    // MFMA's literal zero.  KSL/VSL: ring slots of K of tile t+1 and V of tile t.
    auto mfma_phase = [&](int t, auto do_s_, auto do_pv_, auto ksl, auto vsl) __attribute__((always_inline)) {
        constexpr bool DO_S = decltype(do_s_)::value, DO_PV = decltype(do_pv_)::value;
        const char *kt = ks[decltype(ksl)::value];
        const char *vt = vs[decltype(vsl)::value];
        if constexpr (DO_S) {
            const bf16x8 a0 = T::row_at(kt, kro[0], 0), a1 = T::row_at(kt, kro[0], 2);
            if (needs_mask(t + 1)) {
                // key = kb + c with c = mb*32 + 8*(r/4) + r%4 + 4*hi; masked if key > row
                // or row - key >= window, compared against a per-lane limit so the
                // per-element constants stay immediates
                const int lim = P(row) - 4 * hi - key0(t + 1);
                const int lo = lim - g.window;
                f32x16 bias[2];
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int c = mb * 32 + 8 * (r >> 2) + (r & 3);
                        bias[mb][r] = c > lim || c <= lo ? -INFINITY : 0.f;
                    }
                sc[0] = mfma32(a0, qr[0], bias[0]);
                sc[1] = mfma32(a1, qr[0], bias[1]);
            } else {
                sc[0] = mfma32(a0, qr[0], f32x16{});
                sc[1] = mfma32(a1, qr[0], f32x16{});
            }
        }
        // the S and P V chains interleaved
        constexpr int NS = DO_S ? 2 * KS - 2 : 0, NP = DO_PV ? 4 * DB : 0;
#pragma unroll
        for (int i = 0; i < (NS > NP ? NS : NP); ++i) {
            if (i < NP) {
                const int db = i / 4, kk = i % 4;
                oacc[db] = mfma32(T::tr_at(vt, vto[db], kk), pb[kk], oacc[db]);
            }
            if (i < NS) {
                const int kk2 = 1 + i / 2, mb = i % 2;
                sc[mb] = mfma32(T::row_at(kt, kro[kk2], mb * 2), qr[kk2], sc[mb]);
            }
        }
        // operand reads about six ahead of their MFMAs
        sched_pattern<6, NS + NP, 1, 2, 0>();
        if constexpr (DO_S) pin(sc[0], sc[1]);
    };
    // Vector phase of tile t: row max, rare rescale, P = exp2(S c2 - m2) as bf16 and
    // the row sum of those bf16 weights.
    auto vector_phase = [&]() __attribute__((always_inline)) {
        float mx = -INFINITY;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[mb][r]);
        mx = max_xor32(mx);
        const float mcand = fmaxf(m2, mx * c2);
        if (__any(mcand > m2 + kRescaleThreshold)) {
            const float alpha = mcand == -INFINITY ? 1.f : fast_exp2(m2 - mcand);
            m2 = mcand;
            lsum0 *= alpha;
            lsum1 *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) oacc[db] *= alpha;
        }
        // a row that has seen only masked keys so far (local layers) keeps m2 = -inf;
        // its weights are then exp2(-inf) = 0, not NaN
        const float m2e = m2 == -INFINITY ? 0.f : m2;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t w[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p0 = fast_exp2(__builtin_fmaf(sc[mb][h * 8 + 2 * e], c2, -m2e));
                    const float p1 = fast_exp2(__builtin_fmaf(sc[mb][h * 8 + 2 * e + 1], c2, -m2e));
                    w[e] = pack_bf16(p0, p1);
                    // the row sum adds the bf16 weights that the P V product uses
                    if (mb == 0)
                        lsum0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w[e]), ones, lsum0, false);
                    else
                        lsum1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w[e]), ones, lsum1, false);
                }
                pb[mb * 2 + h] = __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]});
            }
        pin(pb[0], pb[1], pb[2], pb[3]);
    };

    // Prologue: K of tiles 0, 1 and V of tile 0 resident (and the query row).
    if (loader) {
        T::load(ks[0], rk, dma, (uint32_t)key0(0) * kstride, lw);
        if (ntl > 1) T::load(ks[1], rk, dma, (uint32_t)key0(1) * kstride, lw);
        T::load(vs[0], rv, dma, (uint32_t)key0(0) * kstride, lw);
    }
    wait_vmcnt_le(0);
    lds_barrier();

    // Ping-pong.  Each wave runs: matrix phase of tile -1 (scores of tile 0), then for
    // t = 0 .. jlast the vector phase of tile t and the matrix phase of tile t, one
    // phase per workgroup barrier.  Group B starts one phase after group A, so on every
    // SIMD one wave feeds the matrix unit while the other uses the vector unit.  Waves
    // that finish early pass the remaining barriers idle; every wave passes
    // 2*ntl + 2 of them.  Loads (the four waves of group B, each a quarter of a tile,
    // also those whose rows end before the block's last key tile): K of t+2 goes to
    // the slot of K of t, V of t+1 to the slot of V of t-1, both last read in the
    // matrix phases of tile t-1 (phases 2t, 2t+1); they are queued in phase 2t+2 and
    // published by the barrier of phase 2t+3, before group A's matrix phase of tile
    // t+1 (phase 2t+4).  A group B wave passes barrier 2t+2 right after queueing the
    // loads of tile t and barrier 2t+3 right after waiting for them.
    using F = std::false_type;
    using Tr = std::true_type;
    using Z = std::integral_constant<int, 0>;
    using O = std::integral_constant<int, 1>;
    int nb = 0;  // barriers passed
    auto bar = [&]() __attribute__((always_inline)) { lds_barrier(); ++nb; };
    if (group == 1) bar();
    if (!SPLIT || jlast >= 0) {
        mfma_phase(-1, Tr{}, F{}, Z{}, Z{});
        bar();
        int t = 0;
        for (; t + 1 < jlast; t += 2) {
            vector_phase();
            issue(t);
            bar();
            mfma_phase(t, Tr{}, Tr{}, O{}, Z{});
            if (loader) wait_vmcnt_le(0);
            bar();
            vector_phase();
            issue(t + 1);
            bar();
            mfma_phase(t + 1, Tr{}, Tr{}, Z{}, O{});
            if (loader) wait_vmcnt_le(0);
            bar();
        }
        if (t < jlast) {  // t even
            vector_phase();
            issue(t);
            bar();
            mfma_phase(t, Tr{}, Tr{}, O{}, Z{});
            if (loader) wait_vmcnt_le(0);
            bar();
            ++t;
        }
        // t == jlast: last softmax and P V product
        vector_phase();
        issue(t);
        bar();
        if (t & 1)
            mfma_phase(t, F{}, Tr{}, Z{}, O{});
        else
            mfma_phase(t, F{}, Tr{}, Z{}, Z{});
        if (loader) wait_vmcnt_le(0);
        bar();
    } else {
        bar();
    }
    while (nb < 2 * ntl + 2) {  // idle: past this wave's last tile
        if (loader) {
            const int ph = nb - group - 1;  // 2t: the vector phase of tile t, 2t + 1: its matrix phase
            if ((ph & 1) == 0)
                issue(ph >> 1);
            else
                wait_vmcnt_le(0);
        }
        bar();
    }

    mfma_settle();
    float l = sum_xor32(lsum0 + lsum1);
    if constexpr (SPLIT) {
        // every wave has passed the last barrier: the rings are free
        float *part = reinterpret_cast<float *>(kv) + rw * (16 * DB + 2) * 64 + lane;
        if (group == 1) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) part[(db * 16 + r) * 64] = oacc[db][r];
            part[16 * DB * 64] = m2;
            part[(16 * DB + 1) * 64] = l;
        }
        lds_barrier();
        if (group == 1) return;
        // a group without a visible key has reference -inf, sum 0 and zero accumulators
        const float mb = part[16 * DB * 64], mt = fmaxf(m2, mb);
        const float wa = m2 == mt ? 1.f : fast_exp2(m2 - mt), wb = mb == mt ? 1.f : fast_exp2(mb - mt);
        l = l * wa + part[(16 * DB + 1) * 64] * wb;
        m2 = mt;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] = oacc[db][r] * wa + part[(db * 16 + r) * 64] * wb;
    }
    if (row < g.qlen) {
        const float inv = 1.f / l;
        const uint32_t obase = qbase + (uint32_t)row * qstride;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const int d0 = db * 32 + 8 * rq + 4 * hi;
                const u32x2 w = {pack_bf16(oacc[db][4 * rq] * inv, oacc[db][4 * rq + 1] * inv),
                                 pack_bf16(oacc[db][4 * rq + 2] * inv, oacc[db][4 * rq + 3] * inv)};
                st8(ro, obase + d0 * 2, w);
            }
        if (hi == 0) {
            const size_t li = ((size_t)b * g.Hq + hq) * g.qN + (size_t)row * g.qrowmul + s;
            lse[li] = (m2 + log2f(l)) * 0.6931471805599453f;
        }
    }
}

// The block shape for a grid of `wgs` 256-row blocks: split where fwd_split says so; at D=64
// above kPlainMax, two workgroups per CU: each one's softmax and barriers overlap the other's
// MFMAs (768 blocks: 115 -> 101 us, 9216 blocks: 1116 -> 985; 592 of L=500 37.3 -> 33.7, 544 of a
// window of 100 39.2 -> 33.4, 576 final-stream ones 140 -> 125), while a grid that would be
// resident at once then puts long causal blocks on one CU (288 blocks: 80 -> 87).
constexpr int kPlainMax = 512;
Shape fwd_shape(const SfaGeom &g, int64_t wgs)
{
    return fwd_split(g) ? kSplit : g.D == 64 && wgs > kPlainMax ? kShared : kPlain;
}

}  // namespace

hipError_t launch_fwd_bf16(const void *q, const void *k, const void *v, void *o, float *lse,
                           const SfaGeom &g, hipStream_t s)
{
    const int nprob = g.B * g.Hq * g.streams;
    const int wgs = (g.qlen + kBM - 1) / kBM * nprob;
    const Shape shape = fwd_shape(g, wgs);
    const dim3 grid(shape == kSplit ? (g.qlen + kBM / 2 - 1) / (kBM / 2) * nprob : wgs), block(kWaves * 64);
    const bf16 *qq = static_cast<const bf16 *>(q), *kk = static_cast<const bf16 *>(k),
               *vv = static_cast<const bf16 *>(v);
    bf16 *oo = static_cast<bf16 *>(o);
    auto launch = [&](auto dk, const char *name) {
        constexpr int DD = decltype(dk)::value;
        timing_before(name, s);
        auto go = [&](auto fin) {
            constexpr bool FIN = decltype(fin)::value;
            if (shape == kSplit)
                sfa_fwd_bf16_kernel<DD, FIN, kSplit><<<grid, block, 0, s>>>(qq, kk, vv, oo, lse, g);
            else if (DD == 64 && shape == kShared)
                sfa_fwd_bf16_kernel<DD, FIN, DD == 64 ? kShared : kPlain><<<grid, block, 0, s>>>(qq, kk, vv, oo, lse, g);
            else
                sfa_fwd_bf16_kernel<DD, FIN, kPlain><<<grid, block, 0, s>>>(qq, kk, vv, oo, lse, g);
        };
        if (g.strided_waves)
            go(std::true_type{});
        else
            go(std::false_type{});
    };
    const bool f = g.strided_waves;
    switch (g.D) {
    case 32: launch(std::integral_constant<int, 32>{}, f ? "sfa_fwd_final_bf16_d32" : "sfa_fwd_bf16_d32"); break;
    case 64: launch(std::integral_constant<int, 64>{}, f ? "sfa_fwd_final_bf16_d64" : "sfa_fwd_bf16_d64"); break;
    default: launch(std::integral_constant<int, 128>{}, f ? "sfa_fwd_final_bf16_d128" : "sfa_fwd_bf16_d128"); break;
    }
    hipError_t e = hipGetLastError();
    timing_after(s);
    return e;
}

}  // namespace hd
