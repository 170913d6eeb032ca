// rt_backward.hip -- deterministic backward of the radiance-bucket lookup for
// gfx950.
//
//   1. k_bwd_fragment   one lane per fragment: recompute the mapping, write
//                       dL/dview (chain through the bilinear weights, the
//                       clamp, Eq. 3, Eq. 1b and the normalisation) and
//                       dL/duv, and emit one record per (fragment, bucket):
//                       key = bucket << cell_bits | (y0 n + x0).
//   2. radix sort       stable LSD sort of (key, record) by digits of up to
//                       10 bits (9 for large inputs): per-tile digit
//                       histograms, one exclusive scan over (digit, tile)
//                       (small sorts: added up by the scatter's workgroups),
//                       stable in-tile ranking with wave ballots.  Equal keys
//                       keep record order, so the sorted sequence depends only
//                       on the inputs.
//   3. k_bucket_ranges  [start, end) of every bucket in the sorted records.
//      k_payload        (buckets of few records on average, in its
//                       place) the same, and the fractions and weighted
//                       upstream gradient of the records of buckets with at
//                       most 64 records, written in sorted order.
//   4. k_segacc         four or eight buckets per wavefront (pass 1): the records of a
//                       bucket with at most 64 are held in a register window
//                       (read from the payload, or gathered from the
//                       fragments) and reduced per cell by a segmented scan
//                       across lanes with a fixed shape; the four cell sums are
//                       added to the texels of the cell in four ordered phases
//                       in LDS, and the n x n x C tile is written once.
//                       Untouched buckets get zeros.  Buckets with 65..PIECE
//                       records go to k_segacc_big (rounds of 64), more to
//                       pass 2.
//   5. k_segacc_big /   pass 2: hot buckets are cut at fixed chunk boundaries of
//      k_combine_hot    the sorted records; each chunk's part is reduced as in
//                       pass 1 into a partial tile, and the partials are summed
//                       in chunk order.
// No float atomics are used, and every summation order is a function of the
// sorted records alone, so the gradient is bitwise reproducible.
#include <algorithm>

#include "rt_device.hpp"
#include "rt_kernels.hpp"

namespace rt {

constexpr int SORT_THREADS = 256;
constexpr int SORT_IPT = 16;  // keys per thread (4 or 8 in a small sort)
constexpr int SCAN_TILE = 4096;
constexpr int64_t SCAN_FUSED_BLOCKS = 4096;

// ---------------------------------------------------------------------------
// 1. per-fragment backward
// ---------------------------------------------------------------------------

// dL/dA from dL/dB through Eq. (3).  On the branch |A_x| >= |A_y|,
// B = (rho sgn A_x, rho A_y / |A_x|); the other branch mirrors it; at A = 0
// the map's limit along the axes (identity) is used.
__device__ __forceinline__ void square_vjp(float ax, float ay, float gbx, float gby, float& gax,
                                           float& gay) {
    float rho = sqrtf(ax * ax + ay * ay);
    if (!(rho > 0.f)) {
        gax = gbx;
        gay = gby;
        return;
    }
    // the branches differ in the axes' names only: evaluated once, by the larger
    // and the smaller axis (a wavefront has lanes on both)
    const bool xl = fabsf(ax) >= fabsf(ay);
    const float p = xl ? ax : ay, q = xl ? ay : ax;
    const float gbp = xl ? gbx : gby, gbq = xl ? gby : gbx;
    const float s = p >= 0.f ? 1.f : -1.f;
    const float jpp = fabsf(p) / rho, jpq = s * q / rho;
    const float jqp = -s * q * q * q / (rho * p * p);
    const float jqq = (q * q + rho * rho) / (rho * fabsf(p));
    const float gp = jpp * gbp + jqp * gbq, gq = jpq * gbp + jqq * gbq;
    gax = xl ? gp : gq;
    gay = xl ? gq : gp;
}

// sum_c g_c times the slopes of the blended texels along x and y: the
// differences of neighbouring taps are summed over the channels first, then
// weighted (8 operations a channel).
template <int C>
__device__ __forceinline__ void tap_slopes(const F4& t00, const F4& t01, const F4& t10,
                                           const F4& t11, const Foot& p, const float go[4],
                                           float& gx, float& gy) {
    float top = 0.f, bottom = 0.f, left = 0.f, right = 0.f;
#pragma unroll
    for (int c = 0; c < C; c++) {
        top += go[c] * (t01.v[c] - t00.v[c]);
        bottom += go[c] * (t11.v[c] - t10.v[c]);
        left += go[c] * (t10.v[c] - t00.v[c]);
        right += go[c] * (t11.v[c] - t01.v[c]);
    }
    gx = (1.f - p.fy) * top + p.fy * bottom;
    gy = (1.f - p.fx) * left + p.fx * right;
}

// Per-bucket part of the per-fragment backward: dL/ds (x, y).
template <int FMT, int C>
__device__ __forceinline__ void bucket_grads(const TexView& t, int64_t b, const Foot& p,
                                             const float go[4], float& dsx, float& dsy) {
    const int n = t.n;
    using Row = RowBits<FMT, C>;
    const unsigned char* src[1] = {(const unsigned char*)t.data +
                                   (b * (int64_t)(n * n) + p.y0 * n + p.x0) * Row::TEXEL};
    Row row[1][2];
    load_rows<FMT, C, 1>(src, n, row);
    F4 t00, t01, t10, t11;
    row[0][0].decode(t00, t01);
    row[0][1].decode(t10, t11);
    const float f = bucket_factor<FMT>(t.scales, b);
    float gx, gy;
    tap_slopes<C>(t00, t01, t10, t11, p, go, gx, gy);
    dsx = f * gx;
    dsy = f * gy;
}

// Bilinear-bucket mode: the slopes dL/ds of the four buckets (weighted by
// their bucket weights wb, as bucket_grads forms them) and dL/du, dL/dv.  The
// uv derivatives are formed from the differences of corresponding taps of
// neighbouring buckets, each tap times its bucket's factor, so their rounding
// follows the size of those differences rather than of the texel values:
//   dL/du = W sum_c g_c sum_taps w_tap [(1 - b)(T(i1,j0) - T(i0,j0)) + b (T(i1,j1) - T(i0,j1))]
//   dL/dv = H sum_c g_c sum_taps w_tap [(1 - a)(T(i0,j1) - T(i0,j0)) + a (T(i1,j1) - T(i1,j0))]
// with the buckets ordered (i0,j0), (i1,j0), (i0,j1), (i1,j1).
template <int FMT, int C>
__device__ __forceinline__ void pair_grads(const TexView& t, const int64_t bk[4], const float wb[4],
                                           float a, float bb, const Foot& p, const float go[4],
                                           bool want_uv, float& gsx, float& gsy, float& gu,
                                           float& gv) {
    const int n = t.n;
    using Row = RowBits<FMT, C>;
    const unsigned char* src[4];
#pragma unroll
    for (int k = 0; k < 4; k++)
        src[k] = (const unsigned char*)t.data +
                 (bk[k] * (int64_t)(n * n) + p.y0 * n + p.x0) * Row::TEXEL;
    Row row[4][2];
    load_rows<FMT, C, 4>(src, n, row);
    float T[4][4][4];  // [bucket][tap 00, 01, 10, 11][channel], times the bucket factor
    gsx = 0.f;
    gsy = 0.f;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        F4 t00, t01, t10, t11;
        row[k][0].decode(t00, t01);
        row[k][1].decode(t10, t11);
        const float f = bucket_factor<FMT>(t.scales, bk[k]);
        float gx, gy;
        tap_slopes<C>(t00, t01, t10, t11, p, go, gx, gy);
#pragma unroll
        for (int c = 0; c < C; c++) {
            T[k][0][c] = f * t00.v[c];
            T[k][1][c] = f * t01.v[c];
            T[k][2][c] = f * t10.v[c];
            T[k][3][c] = f * t11.v[c];
        }
        gsx += wb[k] * (f * gx);
        gsy += wb[k] * (f * gy);
    }
    gu = 0.f;
    gv = 0.f;
    if (!want_uv) return;
    const float w[4] = {(1.f - p.fx) * (1.f - p.fy), p.fx * (1.f - p.fy), (1.f - p.fx) * p.fy,
                        p.fx * p.fy};
    float su = 0.f, sv = 0.f;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        float top = 0.f, bottom = 0.f, left = 0.f, right = 0.f;
#pragma unroll
        for (int c = 0; c < C; c++) {
            top += go[c] * (T[1][q][c] - T[0][q][c]);
            bottom += go[c] * (T[3][q][c] - T[2][q][c]);
            left += go[c] * (T[2][q][c] - T[0][q][c]);
            right += go[c] * (T[3][q][c] - T[1][q][c]);
        }
        su += w[q] * ((1.f - bb) * top + bb * bottom);
        sv += w[q] * ((1.f - a) * left + a * right);
    }
    gu = (float)t.W * su;
    gv = (float)t.H * sv;
}

// The per-fragment outputs (view and uv gradients, and in nearest mode the
// sort keys and fractions) are stored non-temporally: they are written once
// and read back, if at all, by later passes over millions of records.
__device__ __forceinline__ void nt_store2(float* p, float a, float b) {
    __builtin_nontemporal_store(a, p);
    __builtin_nontemporal_store(b, p + 1);
}

// The words that the later passes expect at zero (the disorder word, the
// counters, the bucket ranges), cleared by the launch that makes the records:
// one launch fewer, and the stores hide behind the fragments' loads.  The host
// asks for it when a thread clears at most CLEAR_QUADS 16-byte groups (a
// 4096-fragment batch over a million buckets would clear 8 MB from 16
// workgroups); otherwise quads is 0 and a fill launch does it.
constexpr int64_t CLEAR_QUADS = 8;

struct ClearWords {
    uint4* at;
    int64_t quads;
};

__device__ __forceinline__ void clear_words(const ClearWords& z) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < z.quads; i += stride)
        z.at[i] = make_uint4(0u, 0u, 0u, 0u);
}

// With one bucket a fragment: bound by its streams (92 to 104 bytes a
// fragment, 5 TB/s).  With four: by the latency of the gathers at the wavefronts
// that fit, so the registers are held to 128 (FP8 RGBA took 148, three
// wavefronts a SIMD): 8.4M fragments, FP8 RGBA, 418 us with three wavefronts, 387
// with four and fewer instructions (982 vector instructions a wavefront, issued in
// 71% of the cycles).  Keeping fewer decoded taps (99 registers, more
// instructions) gains no fifth.
template <int FMT, int C, int MODE>
__global__ __launch_bounds__(256, 4) void k_bwd_fragment(
    TexView t, const float* __restrict__ uv, const float* __restrict__ tbn,
    const float* __restrict__ view, const float* __restrict__ grad_out,
    float* __restrict__ grad_view, float* __restrict__ grad_uv, uint32_t* __restrict__ keys,
    float* __restrict__ wrec, FragMap m, int cell_bits, uint32_t sentinel, ClearWords clear) {
    __shared__ FragStage stage;
    clear_words(clear);
    const int64_t f = frag_of(m, blockIdx.x, gridDim.x, threadIdx.x);
    const int n = t.n;
    float go[4] = {0.f, 0.f, 0.f, 0.f};
    bool zero = true;
    if (f >= 0) {
#pragma unroll
        for (int c = 0; c < C; c++) {
            go[c] = grad_out[f * C + c];
            zero = zero && go[c] == 0.f;
        }
    }
    Frag g;
    if (sentinel == 0u) {
        // every fragment contributes: its frame comes from the wavefront's
        // staged block (every lane takes part in staging it)
        g = load_frag_block(uv, tbn, view, m, f, stage);
        if (f < 0) return;
    } else if (f < 0) {
        return;
    } else if (zero) {
        // sparse plan: no contribution, no records; its gradients are 0
        if (grad_view) {
            grad_view[f * 3 + 0] = 0.f;
            grad_view[f * 3 + 1] = 0.f;
            grad_view[f * 3 + 2] = 0.f;
        }
        if (grad_uv) nt_store2(grad_uv + 2 * f, 0.f, 0.f);
        if (keys) {
            if constexpr (MODE == MODE_NEAREST) keys[f] = sentinel;
            else ((uint4*)keys)[f] = make_uint4(sentinel, sentinel, sentinel, sentinel);
        }
        return;
    } else {
        g = load_frag(uv, tbn, view, f);
    }
    Dir d = map_direction(g.m, g.w, n);
    Foot p = footprint(d.sx, d.sy, n);
    const uint32_t cell = (uint32_t)(p.y0 * n + p.x0);

    float gsx = 0.f, gsy = 0.f;
    if constexpr (MODE == MODE_NEAREST) {
        int i = bucket_of(g.u, t.W), j = bucket_of(g.v, t.H);
        int64_t b = (int64_t)j * t.W + i;
        if (grad_view) bucket_grads<FMT, C>(t, b, p, go, gsx, gsy);
        // no store before the taps have arrived: one counter tracks a
        // wavefront's loads and stores in order, so a wait for loads issued
        // after stores waits for those too
        __builtin_amdgcn_sched_barrier(0);
        if (grad_uv) nt_store2(grad_uv + 2 * f, 0.f, 0.f);
        if (keys) {
            __builtin_nontemporal_store(((uint32_t)b << cell_bits) | cell, keys + f);
            nt_store2(wrec + 2 * f, p.fx, p.fy);
        }
    } else {
        int i0, i1, j0, j1;
        float a, bb;
        bucket_pair(g.u, t.W, i0, i1, a);
        bucket_pair(g.v, t.H, j0, j1, bb);
        const int64_t bk[4] = {(int64_t)j0 * t.W + i0, (int64_t)j0 * t.W + i1,
                               (int64_t)j1 * t.W + i0, (int64_t)j1 * t.W + i1};
        const float wb[4] = {(1.f - a) * (1.f - bb), a * (1.f - bb), (1.f - a) * bb, a * bb};
        if (grad_view || grad_uv) {
            float gu, gv;
            pair_grads<FMT, C>(t, bk, wb, a, bb, p, go, grad_uv != nullptr, gsx, gsy, gu, gv);
            __builtin_amdgcn_sched_barrier(0);  // as above
            if (grad_uv) nt_store2(grad_uv + 2 * f, gu, gv);
        }
        if (keys) {
#pragma unroll
            for (int k = 0; k < 4; k++) keys[4 * f + k] = ((uint32_t)bk[k] << cell_bits) | cell;
            ((float4*)wrec)[f] = make_float4(p.fx, p.fy, a, bb);
        }
    }

    if (grad_view) {
        // dL/dB = (n/2) dL/ds on unclamped axes
        float gbx = d.clx ? 0.f : gsx * (0.5f * (float)n);
        float gby = d.cly ? 0.f : gsy * (0.5f * (float)n);
        float gax, gay;
        square_vjp(d.ax, d.ay, gbx, gby, gax, gay);
        // A = (u_x, u_y) k, k = (L (L + u_z))^(-1/2):
        // dk/du = -k^3/2 * [(u / L)(2L + u_z) + L e_z]
        float gux = 0.f, guy = 0.f, guz = 0.f;
        if (d.k > 0.f && d.L > 0.f) {
            float sdot = d.ux * gax + d.uy * gay;
            float coef = -0.5f * d.k * d.k * d.k * sdot;
            float t2 = (2.f * d.L + d.uz) / d.L;
            gux = d.k * gax + coef * d.ux * t2;
            guy = d.k * gay + coef * d.uy * t2;
            guz = coef * (d.uz * t2 + d.L);
        }
        // dL/dV = M^T dL/du
        __builtin_nontemporal_store(g.m[0] * gux + g.m[3] * guy + g.m[6] * guz, grad_view + f * 3 + 0);
        __builtin_nontemporal_store(g.m[1] * gux + g.m[4] * guy + g.m[7] * guz, grad_view + f * 3 + 1);
        __builtin_nontemporal_store(g.m[2] * gux + g.m[5] * guy + g.m[8] * guz, grad_view + f * 3 + 2);
    }
}

// Level-of-detail backward, per fragment (the lookup blends levels l0 and
// l0 + 1 with weights 1 - t and t; the level of detail is not
// differentiated).  The mapping is formed once; each of the fragment's two
// units u = 2f + s (level l0 + s) gets the upstream gradient times its weight,
// its records in the chain's bucket numbering (start[l] + the level's bucket)
// and the level's view and uv gradients, computed as in k_bwd_fragment and
// summed over the units in level order.  A unit without weight or past the
// last level makes no records (sentinel keys).  Units on a level whose
// gradient is not wanted still make theirs (only the stores are skipped), so
// the sorted positions, and with them the summation order of every written
// level, do not depend on which levels are asked for.
struct LevelStarts {
    int64_t v[MAX_LEVELS + 1];
};

template <int FMT, int C, int MODE>
__global__ __launch_bounds__(256) void k_lod_bwd_fragment(
    LevelSet ls, const float* __restrict__ uv, const float* __restrict__ tbn,
    const float* __restrict__ view, const float* __restrict__ duv,
    const float* __restrict__ grad_out, LevelStarts start,
    float* __restrict__ grad_view, float* __restrict__ grad_uv, uint32_t* __restrict__ keys,
    float* __restrict__ wrec, float* __restrict__ gl, FragMap m, int cell_bits,
    uint32_t sentinel, ClearWords clear) {
    clear_words(clear);
    const int64_t f = frag_of(m, blockIdx.x, gridDim.x, threadIdx.x);
    if (f < 0) return;
    const int n = ls.n;
    float g[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < C; c++) g[c] = grad_out[f * C + c];
    int l0;
    float tt;
    lod_split(((const float4*)duv)[f], ls.W, ls.H, ls.levels, l0, tt);
    const Frag fr = load_frag(uv, tbn, view, f);
    const Dir d = map_direction(fr.m, fr.w, n);
    const Foot p = footprint(d.sx, d.sy, n);
    const uint32_t cell = (uint32_t)(p.y0 * n + p.x0);
    float vx = 0.f, vy = 0.f, vz = 0.f, su = 0.f, sv = 0.f;
    for (int sl = 0; sl < 2; sl++) {
        const int l = l0 + sl;
        const int64_t u = 2 * f + sl;
        const float w = sl == 0 ? 1.f - tt : tt;
        float go[4] = {0.f, 0.f, 0.f, 0.f};
        bool zero = true;
#pragma unroll
        for (int c = 0; c < C; c++) {
            go[c] = w * g[c];
            zero = zero && go[c] == 0.f;
        }
        const bool live = l < ls.levels && !zero;
        const bool rec = live && keys != nullptr;
        if (!rec && keys) {
            if constexpr (MODE == MODE_NEAREST) keys[u] = sentinel;
            else ((uint4*)keys)[u] = make_uint4(sentinel, sentinel, sentinel, sentinel);
        }
        if (!live) continue;
        TexView t{};
        t.data = ls.data[0];
        t.scales = ls.scales[0];
#pragma unroll
        for (int k = 1; k < MAX_LEVELS; k++) {
            if (l == k) {
                t.data = ls.data[k];
                t.scales = ls.scales[k];
            }
        }
        t.W = max(ls.W >> l, 1);
        t.H = max(ls.H >> l, 1);
        t.n = n;
        t.C = C;
        if (rec) {
#pragma unroll
            for (int c = 0; c < C; c++) gl[u * C + c] = go[c];
        }
        const int64_t b0 = start.v[0];
        int64_t off = b0;
#pragma unroll
        for (int k = 1; k < MAX_LEVELS; k++)
            if (l == k) off = start.v[k];
        float gsx = 0.f, gsy = 0.f;
        if constexpr (MODE == MODE_NEAREST) {
            const int i = bucket_of(fr.u, t.W), j = bucket_of(fr.v, t.H);
            const int64_t b = (int64_t)j * t.W + i;
            if (grad_view) bucket_grads<FMT, C>(t, b, p, go, gsx, gsy);
            if (rec) {
                keys[u] = ((uint32_t)(off + b) << cell_bits) | cell;
                ((float2*)wrec)[u] = make_float2(p.fx, p.fy);
            }
        } else {
            int i0, i1, j0, j1;
            float a, bb;
            bucket_pair(fr.u, t.W, i0, i1, a);
            bucket_pair(fr.v, t.H, j0, j1, bb);
            const int64_t bk[4] = {(int64_t)j0 * t.W + i0, (int64_t)j0 * t.W + i1,
                                   (int64_t)j1 * t.W + i0, (int64_t)j1 * t.W + i1};
            const float wb[4] = {(1.f - a) * (1.f - bb), a * (1.f - bb), (1.f - a) * bb, a * bb};
            if (grad_view || grad_uv) {
                float gu, gv;
                pair_grads<FMT, C>(t, bk, wb, a, bb, p, go, grad_uv != nullptr, gsx, gsy, gu, gv);
                su += gu;
                sv += gv;
            }
            if (rec) {
#pragma unroll
                for (int k = 0; k < 4; k++)
                    keys[4 * u + k] = ((uint32_t)(off + bk[k]) << cell_bits) | cell;
                ((float4*)wrec)[u] = make_float4(p.fx, p.fy, a, bb);
            }
        }
        if (grad_view) {
            // as in k_bwd_fragment: dL/dB = (n/2) dL/ds on unclamped axes
            float gbx = d.clx ? 0.f : gsx * (0.5f * (float)n);
            float gby = d.cly ? 0.f : gsy * (0.5f * (float)n);
            float gax, gay;
            square_vjp(d.ax, d.ay, gbx, gby, gax, gay);
            float gux = 0.f, guy = 0.f, guz = 0.f;
            if (d.k > 0.f && d.L > 0.f) {
                float sdot = d.ux * gax + d.uy * gay;
                float coef = -0.5f * d.k * d.k * d.k * sdot;
                float t2 = (2.f * d.L + d.uz) / d.L;
                gux = d.k * gax + coef * d.ux * t2;
                guy = d.k * gay + coef * d.uy * t2;
                guz = coef * (d.uz * t2 + d.L);
            }
            vx += fr.m[0] * gux + fr.m[3] * guy + fr.m[6] * guz;
            vy += fr.m[1] * gux + fr.m[4] * guy + fr.m[7] * guz;
            vz += fr.m[2] * gux + fr.m[5] * guy + fr.m[8] * guz;
        }
    }
    if (grad_view) {
        grad_view[f * 3 + 0] = vx;
        grad_view[f * 3 + 1] = vy;
        grad_view[f * 3 + 2] = vz;
    }
    if (grad_uv) ((float2*)grad_uv)[f] = make_float2(su, sv);
}

// ---------------------------------------------------------------------------
// 2. stable LSD radix sort of (key, record index), digits of up to 10 bits
// ---------------------------------------------------------------------------

// Records made in key order already (fragments visited in the order of a
// visit plan): k_keys_in_order leaves 0 in the disorder word, every launch of
// the sort then returns at once, and the later passes read the keys where the
// per-fragment pass wrote them, each record's position being its number.  A
// stable sort of keys in order is the identity, so the results are the same
// bits either way.
__device__ __forceinline__ bool sort_skipped(const uint32_t* __restrict__ disorder) {
    return disorder != nullptr && __builtin_amdgcn_readfirstlane(*disorder) == 0u;
}

// One 16-byte group of keys starting at i0 with the keys around it (the key
// buffer is padded to 256 bytes, so the load of a partial last group stays
// inside it): k[0] the key before, k[1..4] the group, k[5] the key after.
__device__ __forceinline__ void load_key_group(const uint32_t* __restrict__ keys, int64_t i0,
                                               int64_t R, uint32_t k[6]) {
    const uint4 q = *(const uint4*)(keys + i0);
    k[0] = keys[i0 > 0 ? i0 - 1 : 0];
    k[1] = q.x;
    k[2] = q.y;
    k[3] = q.z;
    k[4] = q.w;
    k[5] = keys[i0 + 4 < R ? i0 + 4 : R - 1];
}

__device__ __forceinline__ bool group_descends(const uint32_t k[6], int64_t i0, int64_t R) {
    bool down = false;
#pragma unroll
    for (int u = 0; u < 4; u++) {
        const int64_t i = i0 + u;
        if (i > 0 && i < R && k[u + 1] < k[u]) down = true;
    }
    return down;
}

// The [start, end) of the buckets that start or end in a group of sorted keys.
__device__ __forceinline__ void group_ranges(const uint32_t k[6], int64_t i0, int64_t R,
                                             int cell_bits, int64_t nb, int2* __restrict__ range) {
#pragma unroll
    for (int u = 0; u < 4; u++) {
        const int64_t i = i0 + u;
        if (i >= R) break;
        const uint32_t bu = k[u + 1] >> cell_bits;
        if (bu >= nb) continue;  // records of a sparse plan without a bucket (sorted last)
        if (i == 0 || (k[u] >> cell_bits) != bu) range[bu].x = (int)i;
        if (i == R - 1 || (k[u + 2] >> cell_bits) != bu) range[bu].y = (int)(i + 1);
    }
}

// Whether any key is smaller than the one before it: a workgroup of 1024 keys
// that finds a descent stores 1 into *disorder (cleared before).  Every such
// workgroup stores the same value with a plain store, so nothing serialises: an
// atomic of every wave on this one word took 0.18 ms on 66M unsorted keys, and
// a flag per workgroup ORed by a second launch cost that launch on every call.
//
// With `range` the check also writes the [start, end) of every bucket as
// k_bucket_ranges forms them, from each workgroup whose 1024 keys (and the
// key before them) are in order: when all are, the sort and k_bucket_ranges
// return at once and these are the ranges; when some are not, k_bucket_ranges
// (or k_payload) writes both ends of every bucket the sorted keys hold (the
// same buckets these keys hold) after the sort, and buckets without keys keep
// the zeros filled in before.  Unsorted keys make nearly every record a
// boundary, so workgroups with a descent write nothing.
__global__ __launch_bounds__(256) void k_keys_in_order(const uint32_t* __restrict__ keys, int64_t R,
                                                       uint32_t* __restrict__ disorder,
                                                       int cell_bits, int64_t nb,
                                                       int2* __restrict__ range) {
    const int64_t i0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    uint32_t k[6] = {0u, 0u, 0u, 0u, 0u, 0u};
    bool down = false;
    if (i0 < R) {
        load_key_group(keys, i0, R, k);
        down = group_descends(k, i0, R);
    }
    const bool any = __syncthreads_or((int)down) != 0;
    if (any && threadIdx.x == 0) *disorder = 1u;
    if (range && !any && i0 < R) group_ranges(k, i0, R, cell_bits, nb, range);
}

// A tile's digit counts in LDS.  Neighbouring keys often have one digit (pixels
// of one cell, records without a bucket), and LDS additions to one word run one
// after the other, so the lanes count into COPIES = 4 tables, a quarter of the
// banks apart.  A pass over 16.6M records of two views 28.8 us, 25.3 with 16-byte
// loads, 20.1 with two tables, 17.0 with four, 16.3 with eight (twice the LDS);
// 4.1M records of a mip chain, half of them without a bucket, 17.8 us, 9.6 with
// four.
template <int D>
struct DigitCounts {
    static constexpr int B = 1 << D, COPIES = 4, STRIDE = B + 64 / COPIES;
    uint32_t at[COPIES * STRIDE];

    __device__ __forceinline__ void clear() {
        for (int d = threadIdx.x; d < COPIES * STRIDE; d += SORT_THREADS) at[d] = 0;
    }
    __device__ __forceinline__ void add(uint32_t digit) {  // its lowest D bits
        atomicAdd(&at[threadIdx.x % COPIES * STRIDE + (digit & (B - 1))], 1u);
    }
    // to the table of all tiles: hist[d * tiles + tile], or with SMALL (a small
    // sort, whose scatter adds the counts up itself) hist[tile * B + d]
    template <bool SMALL>
    __device__ __forceinline__ void store(uint32_t* __restrict__ hist, int64_t tile,
                                          int64_t tiles) const {
        for (int d = threadIdx.x; d < B; d += SORT_THREADS) {
            uint32_t sum = 0;
#pragma unroll
            for (int c = 0; c < COPIES; c++) sum += at[c * STRIDE + d];
            hist[SMALL ? tile * B + d : (int64_t)d * tiles + tile] = sum;
        }
    }
};

// The order check on one radix tile of 256 IPT keys per workgroup, which also
// counts the first pass's digits of its tile (the key's lowest D bits) as
// k_radix_hist does, so that pass needs no launch of it.
template <int D, bool SMALL, int IPT>
__global__ __launch_bounds__(256) void k_keys_in_order_hist(const uint32_t* __restrict__ keys,
                                                            int64_t R,
                                                            uint32_t* __restrict__ disorder,
                                                            int cell_bits, int64_t nb,
                                                            int2* __restrict__ range,
                                                            uint32_t* __restrict__ hist,
                                                            int64_t tiles) {
    constexpr int GROUPS = IPT / 4;
    __shared__ DigitCounts<D> cnt;
    const int t = threadIdx.x;
    cnt.clear();
    const int64_t tile = xcd_block_id(blockIdx.x, gridDim.x);
    const int64_t base = tile * (256 * IPT) + t * 4;
    uint32_t k[GROUPS][6];
    bool down = false;
#pragma unroll
    for (int g = 0; g < GROUPS; g++) {
        const int64_t i0 = base + g * 1024;
        if (i0 < R) {
            load_key_group(keys, i0, R, k[g]);
            down = down || group_descends(k[g], i0, R);
        }
    }
    const bool any = __syncthreads_or((int)down) != 0;  // cnt is zero past this
    if (any && t == 0) *disorder = 1u;
#pragma unroll
    for (int g = 0; g < GROUPS; g++) {
        const int64_t i0 = base + g * 1024;
        if (i0 >= R) break;
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (i0 + u < R) cnt.add(k[g][u + 1]);
        if (range && !any) group_ranges(k[g], i0, R, cell_bits, nb, range);
    }
    __syncthreads();
    cnt.template store<SMALL>(hist, tile, tiles);
}

// Digit counts of one tile of 256 IPT keys: hist[d * tiles + tile].  Tiles
// are renumbered so that each XCD takes a contiguous range: the counts of
// neighbouring tiles share cache lines of the digit-major table, and so the
// strided 4-byte stores of one XCD's tiles combine in its L2.  SMALL (a small
// sort, whose scatter adds the counts up itself): tile-major, hist[tile * B + d].
template <int D, bool SMALL, int IPT>
__global__ __launch_bounds__(SORT_THREADS) void k_radix_hist(const uint32_t* __restrict__ keys,
                                                             int64_t R, int shift,
                                                             uint32_t* __restrict__ hist,
                                                             int64_t tiles,
                                                             const uint32_t* __restrict__ skip) {
    __shared__ DigitCounts<D> cnt;
    if (sort_skipped(skip)) return;
    const int t = threadIdx.x;
    cnt.clear();
    __syncthreads();
    const int64_t tile = xcd_block_id(blockIdx.x, gridDim.x);
    const int64_t base = tile * (SORT_THREADS * IPT);
    uint4 k[IPT / 4];
#pragma unroll
    for (int r = 0; r < IPT / 4; r++) {
        const int64_t i = base + (r * SORT_THREADS + t) * 4;
        k[r] = *(const uint4*)(keys + (i < R ? i : 0));  // the buffer is padded to 256 bytes
    }
#pragma unroll
    for (int r = 0; r < IPT / 4; r++) {
        const int64_t i = base + (r * SORT_THREADS + t) * 4;
        const uint32_t q[4] = {k[r].x, k[r].y, k[r].z, k[r].w};
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (i + u < R) cnt.add(q[u] >> shift);
    }
    __syncthreads();
    cnt.template store<SMALL>(hist, tile, tiles);
}

// x from the lane `o` below in the wavefront, for a power of two o < 64;
// lanes under `o` receive 0 or some lane's x, which their callers mask.
// Offsets 1 and 2 take one or two DPP wavefront shifts (wave_shr:1) on the
// vector ALU instead of a trip through the LDS crossbar (ds_bpermute); the
// value is the same either way, so the segmented scans below add in the same
// order.  A lane without a source lane reads 0 (bound_ctrl), which lets the
// compiler fold the last shift into the addition that uses it
// (v_add_f32_dpp).
__device__ __forceinline__ int dpp_shr1(int x) {
    return __builtin_amdgcn_mov_dpp(x, 0x138, 0xF, 0xF, true);
}
__device__ __forceinline__ int lanes_up(int x, int o) {
    if (o == 1) return dpp_shr1(x);
    if (o == 2) return dpp_shr1(dpp_shr1(x));
    return __shfl_up(x, o, 64);
}
__device__ __forceinline__ uint32_t lanes_up(uint32_t x, int o) {
    return (uint32_t)lanes_up((int)x, o);
}
__device__ __forceinline__ float lanes_up(float x, int o) {
    return __int_as_float(lanes_up(__float_as_int(x), o));
}
// x from the lane one above (lane 63 receives 0, which its callers mask): one
// DPP wavefront shift (wave_shl:1)
__device__ __forceinline__ int lane_above(int x) {
    return __builtin_amdgcn_mov_dpp(x, 0x130, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t lane_above(uint32_t x) { return (uint32_t)lane_above((int)x); }

// exclusive prefix of v over the 256 threads of the block; *total receives the sum
__device__ __forceinline__ uint32_t block_exclusive(uint32_t v, uint32_t* wsum, uint32_t* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        uint32_t s = wsum[k];
        if (k < w) before += s;
        all += s;
    }
    __syncthreads();
    if (total) *total = all;
    return before + x - v;
}

// device-wide exclusive scan: per-block sums, a one-block scan of the sums,
// then per-block scans offset by the scanned sums; up to SCAN_FUSED_BLOCKS
// blocks (every sort of up to 2^27 records) the per-block scans add up the sums
// before them themselves, one launch fewer.  Each thread owns 16
// consecutive counts, read (and written) as four 16-byte vectors when all 16
// lie inside the array and the pointers are 16-byte aligned.
__device__ __forceinline__ void load16(const uint32_t* __restrict__ in, int64_t base, int64_t L,
                                       bool vec, uint32_t v[16]) {
    if (vec && base + 16 <= L) {
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint4 q = ((const uint4*)(in + base))[k];
            v[4 * k] = q.x;
            v[4 * k + 1] = q.y;
            v[4 * k + 2] = q.z;
            v[4 * k + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++) v[k] = (base + k < L) ? in[base + k] : 0u;
    }
}

__global__ __launch_bounds__(256) void k_scan_reduce(const uint32_t* __restrict__ in, int64_t L,
                                                     uint32_t* __restrict__ part,
                                                     const uint32_t* __restrict__ skip) {
    __shared__ uint32_t wsum[4];
    if (sort_skipped(skip)) return;
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + threadIdx.x * 16;
    const bool vec = ((uintptr_t)in & 15) == 0;
    uint32_t v[16], s = 0;
    load16(in, base, L, vec, v);
#pragma unroll
    for (int k = 0; k < 16; k++) s += v[k];
    uint32_t total;
    block_exclusive(s, wsum, &total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void k_scan_top(uint32_t* __restrict__ part, int64_t P,
                                                  const uint32_t* __restrict__ skip) {
    __shared__ uint32_t wsum[4];
    if (sort_skipped(skip)) return;
    uint32_t carry = 0;
    for (int64_t base = 0; base < P; base += 256 * 16) {
        const int64_t b = base + threadIdx.x * 16;
        uint32_t v[16], s = 0;
#pragma unroll
        for (int k = 0; k < 16; k++) {
            v[k] = (b + k < P) ? part[b + k] : 0u;
            s += v[k];
        }
        uint32_t total;
        uint32_t run = carry + block_exclusive(s, wsum, &total);
#pragma unroll
        for (int k = 0; k < 16; k++) {
            if (b + k < P) part[b + k] = run;
            run += v[k];
        }
        carry += total;
    }
}

// SCANNED: part holds the scanned block sums (k_scan_top ran); otherwise it
// holds the plain sums and the block adds up those of the blocks before it
// (at most SCAN_FUSED_BLOCKS of them, so at most 16 loads per thread).
template <bool SCANNED>
__global__ __launch_bounds__(256) void k_scan_down(const uint32_t* __restrict__ in, int64_t L,
                                                   const uint32_t* __restrict__ part,
                                                   uint32_t* __restrict__ out,
                                                   const uint32_t* __restrict__ skip) {
    __shared__ uint32_t wsum[4];
    if (sort_skipped(skip)) return;
    uint32_t offset;
    if constexpr (SCANNED) {
        offset = part[blockIdx.x];
    } else {
        uint32_t ps = 0;
        for (uint32_t j = threadIdx.x; j < blockIdx.x; j += 256) ps += part[j];
        block_exclusive(ps, wsum, &offset);
    }
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + threadIdx.x * 16;
    const bool vec = (((uintptr_t)in | (uintptr_t)out) & 15) == 0;
    uint32_t v[16], s = 0;
    load16(in, base, L, vec, v);
#pragma unroll
    for (int k = 0; k < 16; k++) s += v[k];
    uint32_t run = offset + block_exclusive(s, wsum, nullptr);
    uint32_t o[16];
#pragma unroll
    for (int k = 0; k < 16; k++) {
        o[k] = run;
        run += v[k];
    }
    if (vec && base + 16 <= L) {
#pragma unroll
        for (int k = 0; k < 4; k++)
            ((uint4*)(out + base))[k] = make_uint4(o[4 * k], o[4 * k + 1], o[4 * k + 2], o[4 * k + 3]);
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++)
            if (base + k < L) out[base + k] = o[k];
    }
}

// Lanes of the wavefront holding the same D-bit digit (at bit `shift` of k) as
// this one: one ballot per bit, and one three-input operation per half to keep
// the lanes that agree in it (truth table of a & ~(b ^ c)).
template <int D>
__device__ __forceinline__ uint2 digit_peers(uint32_t k, int shift) {
    uint2 peers = make_uint2(~0u, ~0u);
#pragma unroll
    for (int bit = 0; bit < D; bit++) {
        const int on = (int)(k << (31 - shift - bit)) >> 31;  // the bit in all bits
        const uint64_t m = __ballot(on != 0);
        peers.x = __builtin_amdgcn_bitop3_b32(peers.x, (uint32_t)m, (uint32_t)on, 0x90);
        peers.y = __builtin_amdgcn_bitop3_b32(peers.y, (uint32_t)(m >> 32), (uint32_t)on, 0x90);
    }
    return peers;
}

// Stable scatter of one radix pass.  Wave w ranks the contiguous quarter
// [w TILE/4, (w+1) TILE/4) of the tile in IPT rounds of 64 records: a
// record's rank is the number of lanes below it holding the same digit plus
// the wave's running count of that digit (kept in LDS by the digit's lowest
// lane).  The tile's order within a digit is therefore wave, round, lane: index
// order.  The tile is ordered in LDS, keys first and then, through the same
// buffer, record numbers, so that each digit's run is contiguous in memory.
// Tiles are renumbered per XCD as in the histogram: a digit's runs from
// neighbouring tiles are adjacent in the output, so their partial-line stores
// meet in one L2.  The places past R in the last tile hold the largest key, so
// they rank last and need no test until the stores.
//
// Bound by vector issue, not by its 16 bytes a record: 139 vector instructions
// a round and 45 KB of LDS (3 workgroups a CU) with the ballots combined by
// selects, bounds tests on every load and separate buffers for keys and
// record numbers.
//
// SMALL: hoff holds the tiles' digit counts (tile-major) instead of their
// scanned offsets, and the workgroup adds them up itself: every thread reads
// its digits' column of the table, one row of B counts per tile.  That takes
// the place of the two launches of the scan.
template <int D, bool SMALL, int IPT>
__global__ __launch_bounds__(SORT_THREADS) void k_radix_scatter(
    const uint32_t* __restrict__ keys_in, const uint32_t* __restrict__ vals_in,
    uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out, int64_t R, int shift,
    const uint32_t* __restrict__ hoff, int64_t tiles, const uint32_t* __restrict__ skip) {
    constexpr int B = 1 << D;
    constexpr int DPT = B / SORT_THREADS;  // digits per thread in the digit phase
    constexpr int TILE = SORT_THREADS * IPT;
    constexpr int QUARTER = TILE / 4;
    __shared__ uint32_t buf[TILE];
    // running counts of each wave, then where its records of a digit start in
    // the tile (both at most TILE)
    __shared__ uint16_t wcnt[4][B];
    __shared__ uint32_t gdiff[B];  // a digit's place in the output less its place in the tile
    __shared__ uint32_t wsum[4];
    if (sort_skipped(skip)) return;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t tile = xcd_block_id(blockIdx.x, gridDim.x);
    const int64_t base = tile * TILE;
    for (int d = t; d < 2 * B; d += SORT_THREADS) ((uint32_t*)wcnt)[d] = 0;
    uint32_t k[IPT], v[IPT], loc[IPT];
    const int64_t wbase = base + w * QUARTER + lane;
#pragma unroll
    for (int r = 0; r < IPT; r++) {
        const int64_t i = wbase + r * 64;
        const uint32_t q = keys_in[i < R ? i : R - 1];
        k[r] = i < R ? q : ~0u;
    }
    if (vals_in) {
#pragma unroll
        for (int r = 0; r < IPT; r++) {
            const int64_t i = wbase + r * 64;
            v[r] = vals_in[i < R ? i : R - 1];
        }
    } else {
#pragma unroll
        for (int r = 0; r < IPT; r++) v[r] = (uint32_t)(wbase + r * 64);
    }
    uint32_t off[DPT];  // where the tile's records of thread t's digits t DPT .. go
    if constexpr (SMALL) {
        // their counts in the tiles before this one, and in all
        uint32_t before[DPT], all[DPT], mine = 0;
#pragma unroll
        for (int j = 0; j < DPT; j++) before[j] = all[j] = 0;
#pragma unroll 8
        for (int q = 0; q < (int)tiles; q++) {
#pragma unroll
            for (int j = 0; j < DPT; j++) {
                const uint32_t c = hoff[q * B + t * DPT + j];
                all[j] += c;
                before[j] += q < (int)tile ? c : 0u;
            }
        }
#pragma unroll
        for (int j = 0; j < DPT; j++) mine += all[j];
        uint32_t start = block_exclusive(mine, wsum, nullptr);
#pragma unroll
        for (int j = 0; j < DPT; j++) {
            off[j] = start + before[j];
            start += all[j];
        }
    } else {
#pragma unroll
        for (int j = 0; j < DPT; j++) off[j] = hoff[(int64_t)(t * DPT + j) * tiles + tile];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IPT; r++) {
        const uint32_t dg = (k[r] >> shift) & (B - 1);
        const uint2 peers = digit_peers<D>(k[r], shift);
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi(peers.y, __builtin_amdgcn_mbcnt_lo(peers.x, 0u));
        const uint32_t count = (uint32_t)(__popc(peers.x) + __popc(peers.y));
        const uint32_t before = wcnt[w][dg];
        loc[r] = before + rank;
        wave_lds_sync();
        if (rank == 0) wcnt[w][dg] = (uint16_t)(before + count);
        wave_lds_sync();
    }
    __syncthreads();
    // digits: the tile's exclusive scan over digits, and prefixes over the waves
    uint32_t c[DPT][4], mine = 0;
#pragma unroll
    for (int j = 0; j < DPT; j++) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            c[j][q] = wcnt[q][t * DPT + j];
            mine += c[j][q];
        }
    }
    uint32_t run = block_exclusive(mine, wsum, nullptr);
#pragma unroll
    for (int j = 0; j < DPT; j++) {
        gdiff[t * DPT + j] = off[j] - run;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            wcnt[q][t * DPT + j] = (uint16_t)run;
            run += c[j][q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IPT; r++) {
        loc[r] += wcnt[w][(k[r] >> shift) & (B - 1)];
        buf[loc[r]] = k[r];
    }
    __syncthreads();
    const int nvalid = (int)((R - base) < TILE ? (R - base) : TILE);
#pragma unroll
    for (int r = 0; r < IPT; r++) {
        const int p = r * SORT_THREADS + t;
        const uint32_t kk = buf[p];
        k[r] = gdiff[(kk >> shift) & (B - 1)] + (uint32_t)p;  // from here on the destination
        if (p < nvalid) keys_out[k[r]] = kk;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IPT; r++) buf[loc[r]] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IPT; r++) {
        const int p = r * SORT_THREADS + t;
        if (p < nvalid) vals_out[k[r]] = buf[p];
    }
}

// ---------------------------------------------------------------------------
// 3. bucket ranges in the sorted records
// ---------------------------------------------------------------------------

// Grid-stride fill (the bucket ranges of 2^31 buckets are 2^32 words).
__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* __restrict__ p, int64_t n, uint32_t v) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) p[i] = v;
}

// Four sorted keys per thread, as in the order check.
__global__ __launch_bounds__(256) void k_bucket_ranges(const uint32_t* __restrict__ skeys,
                                                       int64_t R, int cell_bits, int64_t nb,
                                                       int2* __restrict__ range,
                                                       const uint32_t* __restrict__ disorder) {
    // records made in key order: the order check wrote the ranges
    if (sort_skipped(disorder)) return;
    const int64_t i0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i0 >= R) return;
    uint32_t k[6];
    load_key_group(skeys, i0, R, k);
    group_ranges(k, i0, R, cell_bits, nb, range);
}

// One sorted record: the ends of its bucket's range where it is the bucket's
// first or last, and its payload unless its bucket holds more than 64 records
// (their passes gather).  A record tells that from the keys 64 positions
// before and after it; the middle of a bucket of 65 to 127 records cannot, and
// writes a payload that nothing reads.
template <int C, int MODE>
__device__ __forceinline__ void payload_record(const uint32_t* __restrict__ skeys,
                                               const uint32_t* __restrict__ svals,
                                               const float* __restrict__ wrec,
                                               const float* __restrict__ grad_out,
                                               int2* __restrict__ range, int64_t i, int64_t R,
                                               int cell_bits, int64_t nb,
                                               float* __restrict__ payf,
                                               float* __restrict__ payg) {
    const uint32_t b = skeys[i] >> cell_bits;
    if (b >= nb) return;
    const uint32_t rec = svals[i];
    const uint32_t lo = skeys[i >= 1 ? i - 1 : 0] >> cell_bits;
    const uint32_t hi = skeys[i + 1 < R ? i + 1 : R - 1] >> cell_bits;
    const uint32_t lo64 = skeys[i >= 64 ? i - 64 : 0] >> cell_bits;
    const uint32_t hi64 = skeys[i + 64 < R ? i + 64 : R - 1] >> cell_bits;
    if (i == 0 || lo != b) range[b].x = (int)i;
    if (i == R - 1 || hi != b) range[b].y = (int)(i + 1);
    if ((i >= 64 && lo64 == b) || (i + 64 < R && hi64 == b)) return;
    float fx, fy, wb = 1.f;
    int64_t frag;
    if constexpr (MODE == MODE_NEAREST) {
        frag = rec;
        const float2 w2 = ((const float2*)wrec)[frag];
        fx = w2.x;
        fy = w2.y;
    } else {
        frag = rec >> 2;
        const int k = rec & 3;
        const float4 w4 = ((const float4*)wrec)[frag];
        fx = w4.x;
        fy = w4.y;
        const float aa = w4.z, bb = w4.w;
        wb = (k == 0) ? (1.f - aa) * (1.f - bb)
                      : (k == 1) ? aa * (1.f - bb) : (k == 2) ? (1.f - aa) * bb : aa * bb;
    }
    ((float2*)payf)[i] = make_float2(fx, fy);
    if constexpr (C == 4) {
        const float4 g = ((const float4*)grad_out)[frag];
        ((float4*)payg)[i] = make_float4(g.x * wb, g.y * wb, g.z * wb, g.w * wb);
    } else if constexpr (C == 2) {
        const float2 g = ((const float2*)grad_out)[frag];
        ((float2*)payg)[i] = make_float2(g.x * wb, g.y * wb);
    } else {
#pragma unroll
        for (int c = 0; c < C; c++) payg[i * C + c] = grad_out[frag * C + c] * wb;
    }
}

// The bucket ranges of the sorted records and the payload of the records of
// buckets with at most 64 (the ones the first accumulation pass serves from
// its register window), in sorted order: the fractions (fx, fy) and the
// upstream gradient times the bucket weight (1 in nearest mode).  That pass
// then reads its records contiguously instead of gathering them from the
// fragments; the passes for bigger buckets, whose records share cache lines,
// keep gathering.  Records past the last bucket (sparse plans) are skipped.
// Workgroups are renumbered per XCD (neighbouring records gather from
// neighbouring fragments); a workgroup takes PAYLOAD_PER_THREAD x 256
// consecutive records, a thread every 256th of them with its loads issued
// together, which also keeps the launch small when the records came in key
// order and there is nothing to do.
template <int C, int MODE>
__global__ __launch_bounds__(256) void k_payload(const uint32_t* __restrict__ skeys,
                                                 const uint32_t* __restrict__ svals,
                                                 const float* __restrict__ wrec,
                                                 const float* __restrict__ grad_out,
                                                 int2* __restrict__ range, int64_t R,
                                                 int cell_bits, int64_t nb,
                                                 float* __restrict__ payf,
                                                 float* __restrict__ payg,
                                                 const uint32_t* __restrict__ disorder) {
    // records in key order are read where they were made: no payload, and the
    // order check wrote their ranges
    if (sort_skipped(disorder)) return;
    const int64_t base =
        (int64_t)xcd_block_id(blockIdx.x, gridDim.x) * (256 * PAYLOAD_PER_THREAD) + threadIdx.x;
#pragma unroll
    for (int k = 0; k < PAYLOAD_PER_THREAD; k++) {
        const int64_t i = base + 256 * k;
        if (i < R)
            payload_record<C, MODE>(skeys, svals, wrec, grad_out, range, i, R, cell_bits, nb, payf,
                                    payg);
    }
}

// ---------------------------------------------------------------------------
// 4./5. segmented reduction of a bucket's records into its gradient tile
// ---------------------------------------------------------------------------

// Upstream gradient of sorted record i from the payload (bucket weight
// already applied).
template <int C>
__device__ __forceinline__ void load_payg(const float* __restrict__ payg, int64_t i, float g[C]) {
    if constexpr (C == 4) {
        const float4 q = ((const float4*)payg)[i];
        g[0] = q.x;
        g[1] = q.y;
        g[2] = q.z;
        g[3] = q.w;
    } else if constexpr (C == 2) {
        const float2 q = ((const float2*)payg)[i];
        g[0] = q.x;
        g[1] = q.y;
    } else {
#pragma unroll
        for (int c = 0; c < C; c++) g[c] = payg[i * C + c];
    }
}

// Row of a cell (cell / n) without a division: exact for cell < n * n, n <= 64
// with row_inv = ceil(2^20 / n), because then cell * (row_inv * n - 2^20) < 2^20.
__device__ __forceinline__ uint32_t row_inverse(int n) {
    return ((1u << 20) + (uint32_t)n - 1u) / (uint32_t)n;
}

// Adds C channel sums to texel `t` of the tile in one LDS access each way.
template <int C>
__device__ __forceinline__ void texel_add(float* tile, int t, const float v[C]) {
    if constexpr (C == 4) {
        f4v* p = (f4v*)tile + t;
        const f4v a = {v[0], v[1], v[2], v[3]};
        *p += a;
    } else if constexpr (C == 2) {
        float2* p = (float2*)tile + t;
        float2 q = *p;
        q.x += v[0];
        q.y += v[1];
        *p = q;
    } else {
#pragma unroll
        for (int c = 0; c < C; c++) tile[t * C + c] += v[c];
    }
}

// The lanes with `on` set, no two of them with the same cell, add their four
// sums to their cell's four texels in four phases, so no two lanes touch one
// texel at once.
template <int C>
__device__ __forceinline__ void accumulate_tails(int cell, const float v[4 * C], bool on, int n,
                                                 uint32_t row_inv, float* tile) {
    if (__ballot(on) == 0ull) return;
    int t00 = 0, dx = 0, dy = 0;
    if (on) {
        const int y0 = (int)(((uint32_t)cell * row_inv) >> 20);
        const int x0 = cell - y0 * n;
        t00 = cell;
        dx = x0 + 1 < n ? 1 : 0;
        dy = y0 + 1 < n ? n : 0;
    }
    wave_lds_sync();
    if (on) texel_add<C>(tile, t00, v);
    wave_lds_sync();
    if (on) texel_add<C>(tile, t00 + dx, v + C);
    wave_lds_sync();
    if (on) texel_add<C>(tile, t00 + dy, v + 2 * C);
    wave_lds_sync();
    if (on) texel_add<C>(tile, t00 + dx + dy, v + 3 * C);
    wave_lds_sync();
}

// One round of up to 64 sorted records of one bucket, one record per lane
// (lanes without a record carry a cell no record has), added to the tile.
// Records of one cell are a run of neighbouring lanes.  Runs are cut into
// blocks of BLOCK = 4, each block is summed by two segmented steps of DPP
// shifts, and the blocks' last lanes add to the tile, the blocks of a run one
// after the other.  Against a scan over whole runs that takes no step through
// the LDS crossbar and no carry between rounds: a bucket of 65..2048 records
// meets runs of a few records (its cells are spread by the normals and the
// views), where the scan's steps at distances 4 and up and the carry were a
// third of the vector instructions and two thirds of the LDS ones.  The LDS
// round trips of a block cost about as much as a step, so when a run reaches
// more than LONG_RUN records (two blocks) the round scans whole runs instead
// (64 views in plan order 650 us with 8 and 660 with 16, 8 views with bilinear
// buckets 525 and 530; both keep the sums of a run in a tree).
constexpr int BLOCK = 4, LONG_RUN = 8;

template <int C>
__device__ __forceinline__ void accumulate_round(int cell, float v[4 * C], bool valid, int n,
                                                 uint32_t row_inv, float* tile) {
    const int lane = threadIdx.x & 63;
    constexpr int F = 4 * C;
    const int below = lanes_up(cell, 1);  // by every lane: a shift reads active lanes only
    const uint64_t heads = __ballot(lane == 0 || below != cell);
    const uint64_t upto = heads & (~0ull >> (63 - lane));  // lane 0 is a head: never 0
    const int rank = lane - (63 - __builtin_clzll(upto));
    uint64_t firsts;  // lanes that start a summed piece
    int piece;        // its number in its run
    if (__ballot(rank >= LONG_RUN) != 0ull) {
        // a run is contiguous, so once no lane has a partner at distance o
        // every run is at most o long and the scan is complete
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const bool same = rank >= o;
            if (__ballot(same) == 0ull) break;
#pragma unroll
            for (int q = 0; q < F; q++) {
                const float ov = lanes_up(v[q], o);
                if (same) v[q] += ov;
            }
        }
        firsts = heads;
        piece = 0;
    } else {
        const int at = rank & (BLOCK - 1);
        const uint64_t rest = __ballot(at != 0);
        if (rest != 0ull) {
#pragma unroll
            for (int q = 0; q < F; q++) {
                const float ov = lanes_up(v[q], 1);
                if (at >= 1) v[q] += ov;
            }
            if (__ballot(at >= 2) != 0ull) {
#pragma unroll
                for (int q = 0; q < F; q++) {
                    const float ov = lanes_up(v[q], 2);
                    if (at >= 2) v[q] += ov;
                }
            }
        }
        firsts = ~rest;
        piece = rank / BLOCK;
    }
    const uint64_t lasts = (firsts >> 1) | (1ull << 63);
    const bool last = valid && ((lasts >> lane) & 1ull) != 0ull;
    for (int p = 0;; p++) {
        const bool on = last && piece == p;
        if (__ballot(on) == 0ull) break;
        accumulate_tails<C>(cell, v, on, n, row_inv, tile);
    }
}

// A sorted record's key and its number (in the order of the fragments): where
// the rest of it is gathered from.
struct RecIndex {
    uint32_t key, rec;
};

__device__ __forceinline__ void load_index(const uint32_t* __restrict__ skeys,
                                           const uint32_t* __restrict__ svals, int64_t i,
                                           RecIndex& r) {
    r.key = skeys[i];
    r.rec = svals ? svals[i] : (uint32_t)i;
}

// A record as loaded, nothing computed from it yet (that would wait for it): its
// bilinear fractions, in bilinear-bucket mode those of its bucket too, and its
// upstream gradient.
template <int C, int MODE>
struct RawRec {
    RecIndex at;
    float w[MODE == MODE_NEAREST ? 2 : 4];
    float g[C];
};

template <int C, int MODE>
__device__ __forceinline__ void load_raw(const float* __restrict__ wrec,
                                         const float* __restrict__ grad_out, const RecIndex& at,
                                         RawRec<C, MODE>& r) {
    r.at = at;
    int64_t frag;
    if constexpr (MODE == MODE_NEAREST) {
        frag = at.rec;
        const float2 w2 = ((const float2*)wrec)[frag];
        r.w[0] = w2.x;
        r.w[1] = w2.y;
    } else {
        frag = at.rec >> 2;
        const float4 w4 = ((const float4*)wrec)[frag];
        r.w[0] = w4.x;
        r.w[1] = w4.y;
        r.w[2] = w4.z;
        r.w[3] = w4.w;
    }
#pragma unroll
    for (int c = 0; c < C; c++) r.g[c] = grad_out[frag * C + c];
}

// The four tap contributions of a loaded record: v = (w00, w01, w10, w11) x its
// upstream gradient times its bucket's weight (1 in nearest mode).
template <int C, int MODE>
__device__ __forceinline__ void expand_raw(const RawRec<C, MODE>& r, float v[4 * C]) {
    const float fx = r.w[0], fy = r.w[1];
    const float w00 = (1.f - fx) * (1.f - fy), w01 = fx * (1.f - fy);
    const float w10 = (1.f - fx) * fy, w11 = fx * fy;
    float wb = 1.f;
    if constexpr (MODE == MODE_BILINEAR) {
        const int k = r.at.rec & 3;
        const float aa = r.w[2], bb = r.w[3];
        wb = (k == 0) ? (1.f - aa) * (1.f - bb)
                      : (k == 1) ? aa * (1.f - bb) : (k == 2) ? (1.f - aa) * bb : aa * bb;
    }
#pragma unroll
    for (int c = 0; c < C; c++) {
        const float gc = r.g[c] * wb;
        v[0 * C + c] = w00 * gc;
        v[1 * C + c] = w01 * gc;
        v[2 * C + c] = w10 * gc;
        v[3 * C + c] = w11 * gc;
    }
}

// A window of up to 64 consecutive sorted records held in registers, one per
// lane (cell, bilinear fractions and weighted upstream gradient), so that the
// small buckets of a group are served without further global loads.
template <int C>
struct RecWindow {
    int64_t start, end;  // records [start, end) are held; lane l holds start + l
    int cell;
    uint32_t key;
    float fx, fy;
    float g[C];
};

// payf == nullptr: the records are gathered from the fragments (svals, wrec,
// grad_out); otherwise they are read from the sorted payload (payf, payg).
template <int C, int MODE>
__device__ __forceinline__ void load_window(const uint32_t* __restrict__ skeys,
                                            const uint32_t* __restrict__ svals,
                                            const float* __restrict__ wrec,
                                            const float* __restrict__ grad_out,
                                            const float* __restrict__ payf,
                                            const float* __restrict__ payg, int64_t start,
                                            int64_t R, uint32_t cell_mask, RecWindow<C>& w) {
    const int lane = threadIdx.x & 63;
    w.start = start;
    w.end = (start + 64 < R) ? start + 64 : R;
    w.cell = -2 - lane;
    w.key = 0u;
    w.fx = w.fy = 0.f;
#pragma unroll
    for (int c = 0; c < C; c++) w.g[c] = 0.f;
    const int64_t i = start + lane;
    if (i < w.end) {
        w.key = skeys[i];
        w.cell = (int)(w.key & cell_mask);
        if (payf) {
            const float2 f2 = ((const float2*)payf)[i];
            w.fx = f2.x;
            w.fy = f2.y;
            load_payg<C>(payg, i, w.g);
        } else {
            const uint32_t rec = svals ? svals[i] : (uint32_t)i;
            float wb = 1.f;
            int64_t frag;
            if constexpr (MODE == MODE_NEAREST) {
                frag = rec;
                const float2 w2 = ((const float2*)wrec)[frag];
                w.fx = w2.x;
                w.fy = w2.y;
            } else {
                frag = rec >> 2;
                const int k = rec & 3;
                const float4 w4 = ((const float4*)wrec)[frag];
                w.fx = w4.x;
                w.fy = w4.y;
                const float aa = w4.z, bb = w4.w;
                wb = (k == 0) ? (1.f - aa) * (1.f - bb)
                              : (k == 1) ? aa * (1.f - bb) : (k == 2) ? (1.f - aa) * bb : aa * bb;
            }
#pragma unroll
            for (int c = 0; c < C; c++) w.g[c] = grad_out[frag * C + c] * wb;
        }
    }
}

// Segmented sums over the whole window, segments being runs of one sort key
// (bucket and cell): each run's last lane ends with its run's sum, formed by
// the same lanes and additions as a per-bucket scan would form it.
template <int C>
__device__ __forceinline__ void scan_window(const RecWindow<C>& w, float v[4 * C], bool& tail) {
    const int lane = threadIdx.x & 63;
    const int64_t i = w.start + lane;
    const bool valid = i < w.end;
    const float w00 = (1.f - w.fx) * (1.f - w.fy), w01 = w.fx * (1.f - w.fy);
    const float w10 = (1.f - w.fx) * w.fy, w11 = w.fx * w.fy;
#pragma unroll
    for (int c = 0; c < C; c++) {
        const float gc = valid ? w.g[c] : 0.f;
        v[0 * C + c] = w00 * gc;
        v[1 * C + c] = w01 * gc;
        v[2 * C + c] = w10 * gc;
        v[3 * C + c] = w11 * gc;
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t ok = lanes_up(w.key, o);
        const bool same = valid && lane >= o && ok == w.key;
        if (__ballot(same) == 0ull) break;
#pragma unroll
        for (int q = 0; q < 4 * C; q++) {
            const float ov = lanes_up(v[q], o);
            if (same) v[q] += ov;
        }
    }
    const uint32_t nk = lane_above(w.key);
    tail = valid && (lane == 63 || i + 1 >= w.end || nk != w.key);
}

__device__ __forceinline__ void tile_zero(float* tile, int te) {
    const int lane = threadIdx.x & 63;
    if ((te & 3) == 0) {
        const f4v z = {0.f, 0.f, 0.f, 0.f};
        for (int q = lane; q < te / 4; q += 64) ((f4v*)tile)[q] = z;
    } else {
        for (int q = lane; q < te; q += 64) tile[q] = 0.f;
    }
    wave_lds_sync();
}

// The dense gradient is written once and not read back by this library, so
// its stores are non-temporal (streamed past the caches).
__device__ __forceinline__ void tile_store(const float* tile, float* __restrict__ dst, int te) {
    const int lane = threadIdx.x & 63;
    wave_lds_sync();
    if ((te & 255) == 0) {
        for (int q = lane; q < te / 4; q += 64)
            __builtin_nontemporal_store(((const f4v*)tile)[q], (f4v*)dst + q);
    } else {
        for (int q = lane; q < te; q += 64) __builtin_nontemporal_store(tile[q], dst + q);
    }
    wave_lds_sync();
}

// Destination of the tile of bucket b (wave-uniform), or nullptr when the
// bucket's level is not written.  The level index is wave-uniform, so the
// table is read from the kernel arguments with scalar loads, one level at a
// time (a single level for the plain backward: no loop at all).
__device__ __forceinline__ float* tile_dst(const TileOut& o, int64_t b, int te) {
    const int64_t bu = (int64_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
    int l = 0;
#pragma unroll 1
    for (int k = 1; k < o.levels; k++)
        if (bu >= o.start[k]) l = k;
    l = __builtin_amdgcn_readfirstlane(l);
    float* g = o.grad[l];
    return g ? g + (bu - o.start[l]) * (int64_t)te : nullptr;
}

__device__ __forceinline__ void zero_store(float* __restrict__ dst, int te) {
    const int lane = threadIdx.x & 63;
    if ((te & 255) == 0) {
        const f4v z = {0.f, 0.f, 0.f, 0.f};
        for (int q = lane; q < te / 4; q += 64) __builtin_nontemporal_store(z, (f4v*)dst + q);
    } else {
        for (int q = lane; q < te; q += 64) __builtin_nontemporal_store(0.f, dst + q);
    }
}

// pass 1: each wavefront owns G consecutive buckets (their ranges come in one
// coalesced load) and writes their tiles one after the other, so the stores
// of untouched buckets are issued back to back; four wavefronts per
// workgroup.  G = 4, or SEG_GROUP (8) where most buckets are only listed (see
// launch_accumulate).  k_segacc writes the untouched buckets and those with at
// most 64 records (served from one register window) and lists those with
// 65..PIECE records for k_segacc_big (rounds of 64).  Splitting keeps the
// register footprint of the common case small.  The list is split over
// BIG_LISTS counters, one atomic per group, so that workloads where most
// buckets are big do not serialise on one address: runs of 2^big_run_log
// groups (at most BIG_RUN, see launch_accumulate) take the lists in turn,
// which keeps neighbouring buckets on one XCD in k_segacc_big.  The order
// inside a list does not matter, each bucket is reduced alone.
template <int C, int MODE, int G>
__global__ __launch_bounds__(256) void k_segacc(const uint32_t* __restrict__ skeys,
                                                const uint32_t* __restrict__ svals,
                                                const float* __restrict__ wrec,
                                                const float* __restrict__ grad_out,
                                                const float* __restrict__ payf,
                                                const float* __restrict__ payg,
                                                const int2* __restrict__ range,
                                                const TileOut out, int64_t nbuckets,
                                                int64_t R, int n, uint32_t cell_mask,
                                                uint32_t* __restrict__ big_count,
                                                uint32_t* __restrict__ big_list,
                                                int64_t big_cap, int big_run_log,
                                                const uint32_t* __restrict__ keys_made,
                                                const uint32_t* __restrict__ disorder) {
    if (sort_skipped(disorder)) {
        skeys = keys_made;
        svals = nullptr;
        payf = nullptr;
    }
    extern __shared__ float lds[];
    const int te = n * n * C;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    float* tile = lds + w * te;
    const uint32_t row_inv = row_inverse(n);
    const int64_t ngroups = (nbuckets + G - 1) / G;
    for (int64_t grp = (int64_t)xcd_block_id(blockIdx.x, gridDim.x) * 4 + w; grp < ngroups;
         grp += (int64_t)gridDim.x * 4) {
        const int64_t b0 = grp * G;
        int2 rl = make_int2(0, 0);
        if (lane < G && b0 + lane < nbuckets) rl = range[b0 + lane];
        const int nb = (int)((nbuckets - b0) < G ? (nbuckets - b0) : G);
        // list the group's buckets with 65..PIECE records (more go to pass 2)
        const int cl = rl.y - rl.x;
        const bool big = cl > 64 && cl <= PIECE;
        const uint64_t bm = __ballot(big);
        // a bucket for pass 2: raise the flag that lets its kernels run
        if (__ballot(cl > PIECE) != 0ull && lane == 0) atomicOr(big_count + HOT_FLAG, 1u);
        if (bm != 0ull) {
            const int64_t list = (grp >> big_run_log) & (BIG_LISTS - 1);
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(big_count + list * BIG_STRIDE, (uint32_t)__popcll(bm));
            base = __shfl(base, 0, 64);
            if (big) {
                const uint32_t below = (uint32_t)__popcll(bm & ((1ull << lane) - 1ull));
                big_list[list * big_cap + base + below] = (uint32_t)(b0 + lane);
            }
        }
        RecWindow<C> win;
        win.start = win.end = -1;
        float v[4 * C];
        bool tail = false;
        for (int k = 0; k < nb; k++) {
            // wave-uniform bucket range (scalar registers, scalar loop control)
            const int rx = __builtin_amdgcn_readfirstlane(__shfl(rl.x, k, 64));
            const int ry = __builtin_amdgcn_readfirstlane(__shfl(rl.y, k, 64));
            float* dst = tile_dst(out, b0 + k, te);
            const int cnt = ry - rx;
            if (cnt <= 0) {
                if (dst) zero_store(dst, te);
                continue;
            }
            if (cnt > 64 || !dst) continue;  // listed above, or hot; or not written
            if (!(rx >= win.start && ry <= win.end)) {
                load_window<C, MODE>(skeys, svals, wrec, grad_out, payf, payg, rx, R, cell_mask,
                                     win);
                scan_window<C>(win, v, tail);
            }
            tile_zero(tile, te);
            const int64_t i = win.start + lane;
            accumulate_tails<C>(win.cell, v, tail && i >= rx && i < ry, n, row_inv, tile);
            tile_store(tile, dst, te);
        }
    }
}

// Buckets with 65..PIECE records, listed by k_segacc (the first big_blocks
// workgroups): workgroup x serves list x mod BIG_LISTS, one wavefront per
// listed bucket, in rounds of 64 records.
//
// The workgroups after them are pass 2a, one wavefront per fixed chunk of PIECE
// sorted records: a hot bucket overlapping the chunk (only the chunk's first
// or last bucket can be hot) gets a partial tile, slot 0 for the first bucket
// and slot 1 for the last.  They return at once when k_segacc saw no such
// bucket.
//
// Bound by vector issue (87% of the cycles on the 64 views' 67M records, about
// 280 vector instructions a round; 58% on 8 views with bilinear buckets).  64 views: 973 us
// when rounds scanned whole runs and carried the last one, 718 without the
// carry, 650 since no round waits for a list entry, a range or an index (in image
// order, where the records are gathered, 1255 us throughout).  8 views
// with bilinear buckets (33.5M records, gathered): 600, 530, 520; 2867 buckets of
// 70 records: 39 us, 10.5 (more lists).  Six wavefronts a SIMD instead of five
// (80 registers, one spilled) give 638 us on the 64 views, but a launch that has
// scratch costs a small backward 7 us.
template <int C, int MODE>
__global__ __launch_bounds__(256) void k_segacc_big(const uint32_t* __restrict__ skeys,
                                                    const uint32_t* __restrict__ svals,
                                                    const float* __restrict__ wrec,
                                                    const float* __restrict__ grad_out,
                                                    const int2* __restrict__ range,
                                                    const TileOut out, int n, int cell_bits,
                                                    const uint32_t* __restrict__ big_count,
                                                    const uint32_t* __restrict__ big_list,
                                                    int64_t big_cap, uint32_t big_blocks,
                                                    float* __restrict__ part, int64_t R,
                                                    int64_t nb,
                                                    const uint32_t* __restrict__ keys_made,
                                                    const uint32_t* __restrict__ disorder) {
    const bool hot = blockIdx.x >= big_blocks;
    if (hot && __builtin_amdgcn_readfirstlane(big_count[HOT_FLAG]) == 0u) return;
    if (sort_skipped(disorder)) {
        skeys = keys_made;
        svals = nullptr;
    }
    extern __shared__ float lds[];
    const int te = n * n * C;
    const uint32_t cell_mask = cell_bits >= 32 ? 0xFFFFFFFFu : ((1u << cell_bits) - 1u);
    const uint32_t row_inv = row_inverse(n);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float* tile = lds + w * te;
    // the wavefront's work items: entries [item, items) of its list in steps of
    // `stride`, or the (at most two) slots of its chunk
    const int lane = threadIdx.x & 63;
    uint32_t item, items, stride;
    const uint32_t* entries = nullptr;
    int c0 = 0, c1 = 0;
    uint32_t b_first = 0, b_last = 0;  // of the chunk
    if (!hot) {
        const uint32_t list = blockIdx.x % BIG_LISTS;
        stride = big_blocks / BIG_LISTS * 4;
        item = blockIdx.x / BIG_LISTS * 4 + w;
        items = __builtin_amdgcn_readfirstlane(big_count[list * BIG_STRIDE]);
        entries = big_list + list * big_cap;
    } else {
        const int64_t first = ((int64_t)(blockIdx.x - big_blocks) * 4 + w) * PIECE;
        if (first >= R) return;
        c0 = (int)first;
        c1 = (int)((first + PIECE < R) ? first + PIECE : R);
        b_first = __builtin_amdgcn_readfirstlane(skeys[c0]) >> cell_bits;
        b_last = __builtin_amdgcn_readfirstlane(skeys[c1 - 1]) >> cell_bits;
        // records past the last bucket (sparse plans) belong to no slot
        stride = 1;
        item = 0;
        items = b_first >= nb ? 0u : b_last == b_first || b_last >= nb ? 1u : 2u;
    }
    // the next item: `left` records of one bucket from record `at` on, their
    // tile to dst.  The buckets and ranges of 64 items are held, one per lane, so
    // that an item waits for neither.
    struct Item {
        int at, left;
        float* dst;
    };
    int held = 64;  // the next item's lane; 64: read the next 64
    uint32_t hb = 0;
    int2 hr = make_int2(0, 0);
    auto next_item = [&](Item& k) {
        for (; item < items; item += stride) {
            if (held == 64) {
                const uint32_t q = item + lane * stride;
                if (q < items) {
                    hb = !hot ? entries[q] : q == 0 ? b_first : b_last;
                    hr = range[hb];
                }
                held = 0;
            }
            const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)hb, held);
            int a = __builtin_amdgcn_readlane(hr.x, held);
            int e = __builtin_amdgcn_readlane(hr.y, held);
            held++;
            if (hot) {
                if (e - a <= PIECE) continue;
                a = a > c0 ? a : c0;
                e = e < c1 ? e : c1;
                k.dst = part + (c0 / PIECE * 2 + (int64_t)item) * te;
            } else {
                k.dst = tile_dst(out, b, te);
                if (!k.dst) continue;  // a level that is not written
            }
            k.at = a;
            k.left = e - a;
            item += stride;
            return true;
        }
        return false;
    };
    // the round after `k`: the item's next records, or the next item
    auto next_round = [&](const Item& k, Item& next) {
        if (k.left <= 64) return next_item(next);
        next.at = k.at + 64;
        next.left = k.left - 64;
        next.dst = k.dst;
        return true;
    };
    // Rounds of 64 records.  While a round is summed, and before its tile is
    // stored, the next round's records are gathered and the indices of the one
    // after that are loaded, so no round waits for an index.  (On gfx950 one
    // counter tracks a wavefront's loads and stores: loads after the stores
    // would wait for them.)
    Item cur_item, nxt_item{}, far_item{};
    if (!next_item(cur_item)) return;
    RecIndex cur_at{}, nxt_at{}, far_at{};
    if (lane < cur_item.left) load_index(skeys, svals, cur_item.at + lane, cur_at);
    bool more = next_round(cur_item, nxt_item);
    if (more && lane < nxt_item.left) load_index(skeys, svals, nxt_item.at + lane, nxt_at);
    RawRec<C, MODE> cur{}, nxt{};
    if (lane < cur_item.left) load_raw<C, MODE>(wrec, grad_out, cur_at, cur);
    tile_zero(tile, te);
    for (;;) {
        if (more && lane < nxt_item.left) load_raw<C, MODE>(wrec, grad_out, nxt_at, nxt);
        const bool after = more && next_round(nxt_item, far_item);
        if (after && lane < far_item.left) load_index(skeys, svals, far_item.at + lane, far_at);
        const bool valid = lane < cur_item.left;
        float v[4 * C];
        expand_raw<C, MODE>(cur, v);
        const int cell = valid ? (int)(cur.at.key & cell_mask) : -2 - lane;
        accumulate_round<C>(cell, v, valid, n, row_inv, tile);
        if (cur_item.left <= 64) {
            tile_store(tile, cur_item.dst, te);
            if (!more) return;
            tile_zero(tile, te);
        }
        cur = nxt;
        cur_item = nxt_item;
        nxt_at = far_at;
        nxt_item = far_item;
        more = after;
    }
}

// pass 2b: the chunk in which a hot bucket starts sums its partial tiles in
// chunk order and writes the bucket's tile.
__global__ __launch_bounds__(64) void k_combine_hot(const uint32_t* __restrict__ skeys,
                                                    const int2* __restrict__ range,
                                                    const float* __restrict__ part,
                                                    const TileOut out, int64_t R,
                                                    int te, int cell_bits, int64_t nb,
                                                    const uint32_t* __restrict__ keys_made,
                                                    const uint32_t* __restrict__ disorder,
                                                    const uint32_t* __restrict__ hot) {
    if (__builtin_amdgcn_readfirstlane(hot[0]) == 0u) return;  // no bucket for pass 2
    if (sort_skipped(disorder)) skeys = keys_made;
    const int lane = threadIdx.x;
    const int64_t k = blockIdx.x;
    const int64_t c0 = k * PIECE;
    const int64_t c1 = (c0 + PIECE < R) ? c0 + PIECE : R;
    const uint32_t bf = skeys[c0] >> cell_bits;
    const uint32_t bl = skeys[c1 - 1] >> cell_bits;
    for (int slot = 0; slot < 2; slot++) {
        const uint32_t b = slot == 0 ? bf : bl;
        if (slot == 1 && bl == bf) break;
        if (b >= nb) break;  // the records past the last bucket (sparse plans)
        const int2 r = range[b];
        if ((int64_t)r.y - r.x <= PIECE) continue;
        if ((int64_t)r.x / PIECE != k) continue;  // combined by the chunk it starts in
        const int64_t k0 = (int64_t)r.x / PIECE, k1 = ((int64_t)r.y - 1) / PIECE;
        float* dst = tile_dst(out, b, te);
        if (!dst) continue;
        for (int q0 = 0; q0 < te; q0 += 64 * 8) {
            float acc[8];
#pragma unroll
            for (int u = 0; u < 8; u++) acc[u] = 0.f;
            for (int64_t kc = k0; kc <= k1; kc++) {
                const int s = ((skeys[kc * PIECE] >> cell_bits) == b) ? 0 : 1;
                const float* src = part + (kc * 2 + s) * (int64_t)te;
#pragma unroll
                for (int u = 0; u < 8; u++) {
                    const int q = q0 + u * 64 + lane;
                    if (q < te) acc[u] += src[q];
                }
            }
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const int q = q0 + u * 64 + lane;
                if (q < te) dst[q] = acc[u];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// planning and launch sequence
// ---------------------------------------------------------------------------

static int ceil_log2(uint64_t x) {
    int b = 0;
    while ((1ull << b) < x) b++;
    return b;
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Radix tiles of R records with ipt keys per thread.
static int64_t radix_tiles(int64_t R, int ipt) {
    return (R + SORT_THREADS * ipt - 1) / (SORT_THREADS * ipt);
}

// Digits of at most 10 bits up to this many records, 9 beyond, where the
// histograms, their scan and the scatter's LDS, which grow as 2^D, cost more than
// a pass saves.
constexpr int64_t WIDE_DIGIT_RECORDS = int64_t(1) << 22;

// log2 of the counts of a tile: the bits spread evenly over as few passes as
// digits of `most` bits allow, in a kernel of at least 8.
static int tile_bits(int key_bits, int most) {
    const int passes = (key_bits + most - 1) / most;
    return std::max(8, (key_bits + passes - 1) / passes);
}

// The digit counts of the sort, their scanned offsets and the scan's sums, from
// offset o of the workspace on; returns where they end.  A small sort needs the
// counts only.  A workspace of some size serves fewer records as well, so a sort
// reserves as many counts as any of fewer records has: fewer keys per thread make
// more of them (up to SMALL_SORT_COUNTS / 2), and so do wider digits.
static size_t place_tables(BwdPlan* p, size_t o) {
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += align256(bytes);
        return at;
    };
    const int64_t least = std::min<int64_t>(SMALL_SORT_COUNTS / 2,
                                            (int64_t)p->bins * radix_tiles(p->records, 4));
    int64_t counts = std::max(p->scan_len, least);
    if (p->records > WIDE_DIGIT_RECORDS)
        counts = std::max(counts, radix_tiles(WIDE_DIGIT_RECORDS, SORT_IPT)
                                      << tile_bits(std::max(1, p->key_bits), 10));
    p->off_hist = take((size_t)counts * 4);
    p->off_hoff = take(p->small_sort ? 0 : (size_t)counts * 4);
    p->off_scanp = take(p->small_sort ? 0 : (size_t)((counts + SCAN_TILE - 1) / SCAN_TILE + 1) * 4);
    return o;
}

bool plan_backward(int W, int H, int n, int C, int64_t N, int mode, BwdPlan* p, bool sparse) {
    // the accumulation holds four bucket tiles per workgroup in LDS (64 KiB)
    if ((int64_t)n * n * C > 4096) return false;
    const int64_t nb = (int64_t)W * H;
    // a sparse plan keeps the all-ones key free for records without a bucket
    const int bucket_bits = ceil_log2((uint64_t)nb + (sparse ? 1 : 0));
    const int cell_bits = ceil_log2((uint64_t)n * n);
    if (bucket_bits + cell_bits > 32) return false;
    const int64_t R = mode == MODE_NEAREST ? N : 4 * N;
    if (R >= (1ll << 31)) return false;
    p->records = R;
    p->key_bits = bucket_bits + cell_bits;
    p->cell_bits = cell_bits;
    p->buckets = nb;
    p->sentinel = !sparse ? 0u
                  : (p->key_bits >= 32 ? 0xFFFFFFFFu : (uint32_t)((1ull << p->key_bits) - 1));
    const int kb = std::max(1, p->key_bits);
    const int maxd = R <= WIDE_DIGIT_RECORDS ? 10 : 9;
    p->passes = (kb + maxd - 1) / maxd;
    int at = 0;
    for (int q = 0; q < 4; q++) {
        const int bits = q < p->passes ? kb / p->passes + (q < kb % p->passes ? 1 : 0) : 0;
        p->digit_bits[q] = bits;
        p->digit_shift[q] = at;
        at += bits;
    }
    // A small sort is bound by its launches, so it makes fewer (its scatters add
    // the tiles' digit counts up themselves, see launch_sort_records), at the
    // price of a read of the whole table of counts by every workgroup.  A whole
    // backward of 200,000 records took 104 us with the scans and 77 without (49
    // tiles, 2^8 digits), 600,000 the same either way (147 tiles, 2^8 digits),
    // 1,000,000 343 and 398 us (245 tiles, 2^10 digits).
    p->bins = 1 << tile_bits(kb, maxd);
    p->sort_ipt = SORT_IPT;
    p->small_sort = radix_tiles(R, SORT_IPT) * p->bins <= SMALL_SORT_COUNTS;
    // Its few tiles leave most of the chip idle, and the rounds of a tile run one
    // after the other: fewer keys per thread while the table stays below half
    // that size (65,536 records and 2^9 digits: 46.8 us with 16, 44.7 with 8, 40.1
    // with 4 keys; 50,001 and 2^10, past it: 45.7 with 8, 50.0 with 4).
    while (p->small_sort && p->sort_ipt > 4 &&
           radix_tiles(R, p->sort_ipt / 2) * p->bins <= SMALL_SORT_COUNTS / 2)
        p->sort_ipt /= 2;
    p->tiles = radix_tiles(R, p->sort_ipt);
    p->scan_len = (int64_t)p->bins * p->tiles;
    p->scan_blocks = (p->scan_len + SCAN_TILE - 1) / SCAN_TILE;
    p->chunks = (R + PIECE - 1) / PIECE;
    p->tile_elems = (int64_t)n * n * C;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o += align256(bytes);
        return at;
    };
    p->off_keys0 = take((size_t)R * 4);
    p->off_keys1 = take((size_t)R * 4);
    p->off_vals0 = take((size_t)R * 4);
    p->off_vals1 = take((size_t)R * 4);
    // the disorder word, and right after it (both are cleared in one go) the
    // big-bucket counters and the bucket ranges
    p->off_disorder = take(256);
    p->off_range = take((size_t)BIG_LISTS * BIG_STRIDE * 4 + (size_t)nb * 8);
    p->clear_bytes = o - p->off_disorder;
    p->off_wrec = take((size_t)N * (mode == MODE_NEAREST ? 8 : 16));
    // The sort's tables share the memory of what is written after the sort (12
    // bytes a record and more: the tables add nothing from 2049 records on).  From
    // 16,384 records on, where those bytes hold the padding too, they start on 64
    // KB: every workgroup of a small sort reads the whole table of counts.  A
    // backward of 1,048,576 records and 24 a bucket took 109.2 us with the tables on
    // 256 bytes or 4 KB, depending on the matrix, and 105.1 on 64 KB, 800,000 records
    // 98.5 and 95.5.
    const size_t page = R >= 16384 ? 65536 : 256;
    const size_t tables_end = place_tables(p, (o + page - 1) / page * page);
    p->off_payf = take((size_t)R * 8);
    p->off_payg = take((size_t)R * 4 * C);
    // big-bucket lists: list l receives the runs r of BIG_RUN groups with
    // r mod BIG_LISTS = l, at most ceil(ngroups / (BIG_RUN BIG_LISTS)) runs of
    // BIG_RUN * SEG_GROUP buckets, and no list exceeds the R/65 buckets that
    // can hold more than 64 records
    const int64_t ngroups = (nb + SEG_GROUP - 1) / SEG_GROUP;
    const int64_t runs_per_list = (ngroups + BIG_RUN * BIG_LISTS - 1) / (BIG_RUN * BIG_LISTS);
    const int64_t per_list = runs_per_list * BIG_RUN * SEG_GROUP;
    p->big_cap = std::max<int64_t>(1, std::min<int64_t>(per_list, R / 65));
    p->off_biglist = take((size_t)BIG_LISTS * p->big_cap * 4);
    p->off_part = take((size_t)p->chunks * 2 * p->tile_elems * 4);
    p->total = std::max(o, tables_end);
    return true;
}

bool plan_visit(int W, int H, int n, int64_t N, BwdPlan* p) {
    if (!plan_backward(W, H, n, 1, N, MODE_NEAREST, p)) return false;
    p->total = place_tables(p, p->off_range);
    return true;
}

template <int FMT, int MODE>
static void launch_bwd_fragment_c(const TexView& t, const float* uv, const float* tbn,
                                  const float* view, const float* go, float* gview, float* guv,
                                  uint32_t* keys, float* wrec, const FragMap& m, int cell_bits,
                                  uint32_t sentinel, const ClearWords& clear, hipStream_t s) {
    const uint32_t blocks = fragmap_blocks(m);
    switch (t.C) {
    case 1: hipLaunchKernelGGL((k_bwd_fragment<FMT, 1, MODE>), dim3(blocks), dim3(256), 0, s, t, uv, tbn, view, go, gview, guv, keys, wrec, m, cell_bits, sentinel, clear); break;
    case 2: hipLaunchKernelGGL((k_bwd_fragment<FMT, 2, MODE>), dim3(blocks), dim3(256), 0, s, t, uv, tbn, view, go, gview, guv, keys, wrec, m, cell_bits, sentinel, clear); break;
    case 3: hipLaunchKernelGGL((k_bwd_fragment<FMT, 3, MODE>), dim3(blocks), dim3(256), 0, s, t, uv, tbn, view, go, gview, guv, keys, wrec, m, cell_bits, sentinel, clear); break;
    default: hipLaunchKernelGGL((k_bwd_fragment<FMT, 4, MODE>), dim3(blocks), dim3(256), 0, s, t, uv, tbn, view, go, gview, guv, keys, wrec, m, cell_bits, sentinel, clear); break;
    }
}

template <int MODE, int G>
static void launch_segacc_c(int C, dim3 grid, size_t shm, hipStream_t s, const uint32_t* sk,
                            const uint32_t* sv, const float* wrec, const float* go,
                            const float* pf, const float* pg,
                            const int2* range, const TileOut& gt, int64_t nb, int64_t R, int n,
                            uint32_t mask, uint32_t* bc, uint32_t* bl, int64_t cap,
                            int run_log, const uint32_t* km, const uint32_t* dis) {
    switch (C) {
    case 1: hipLaunchKernelGGL((k_segacc<1, MODE, G>), grid, dim3(256), shm, s, sk, sv, wrec, go, pf, pg, range, gt, nb, R, n, mask, bc, bl, cap, run_log, km, dis); break;
    case 2: hipLaunchKernelGGL((k_segacc<2, MODE, G>), grid, dim3(256), shm, s, sk, sv, wrec, go, pf, pg, range, gt, nb, R, n, mask, bc, bl, cap, run_log, km, dis); break;
    case 3: hipLaunchKernelGGL((k_segacc<3, MODE, G>), grid, dim3(256), shm, s, sk, sv, wrec, go, pf, pg, range, gt, nb, R, n, mask, bc, bl, cap, run_log, km, dis); break;
    default: hipLaunchKernelGGL((k_segacc<4, MODE, G>), grid, dim3(256), shm, s, sk, sv, wrec, go, pf, pg, range, gt, nb, R, n, mask, bc, bl, cap, run_log, km, dis); break;
    }
}

template <int MODE>
static void launch_segacc_big_c(int C, dim3 grid, size_t shm, hipStream_t s, const uint32_t* sk,
                                const uint32_t* sv, const float* wrec, const float* go,
                                const int2* range, const TileOut& gt, int n, int cb,
                                const uint32_t* bc, const uint32_t* bl, int64_t cap,
                                uint32_t big_blocks, float* part, int64_t R, int64_t nb,
                                const uint32_t* km, const uint32_t* dis) {
    switch (C) {
    case 1: hipLaunchKernelGGL((k_segacc_big<1, MODE>), grid, dim3(256), shm, s, sk, sv, wrec, go, range, gt, n, cb, bc, bl, cap, big_blocks, part, R, nb, km, dis); break;
    case 2: hipLaunchKernelGGL((k_segacc_big<2, MODE>), grid, dim3(256), shm, s, sk, sv, wrec, go, range, gt, n, cb, bc, bl, cap, big_blocks, part, R, nb, km, dis); break;
    case 3: hipLaunchKernelGGL((k_segacc_big<3, MODE>), grid, dim3(256), shm, s, sk, sv, wrec, go, range, gt, n, cb, bc, bl, cap, big_blocks, part, R, nb, km, dis); break;
    default: hipLaunchKernelGGL((k_segacc_big<4, MODE>), grid, dim3(256), shm, s, sk, sv, wrec, go, range, gt, n, cb, bc, bl, cap, big_blocks, part, R, nb, km, dis); break;
    }
}

template <int MODE>
static void launch_payload_c(int C, dim3 grid, hipStream_t s, const uint32_t* sk,
                             const uint32_t* sv, const float* wrec, const float* go,
                             int2* range, int64_t R, int cb, int64_t nb, float* pf,
                             float* pg, const uint32_t* dis) {
    switch (C) {
    case 1: hipLaunchKernelGGL((k_payload<1, MODE>), grid, dim3(256), 0, s, sk, sv, wrec, go, range, R, cb, nb, pf, pg, dis); break;
    case 2: hipLaunchKernelGGL((k_payload<2, MODE>), grid, dim3(256), 0, s, sk, sv, wrec, go, range, R, cb, nb, pf, pg, dis); break;
    case 3: hipLaunchKernelGGL((k_payload<3, MODE>), grid, dim3(256), 0, s, sk, sv, wrec, go, range, R, cb, nb, pf, pg, dis); break;
    default: hipLaunchKernelGGL((k_payload<4, MODE>), grid, dim3(256), 0, s, sk, sv, wrec, go, range, R, cb, nb, pf, pg, dis); break;
    }
}

static void launch_fill(uint32_t* p, int64_t n, uint32_t v, hipStream_t s) {
    if (n <= 0) return;
    prof_begin(K_FILL, s);
    const uint32_t blocks = (uint32_t)std::min<int64_t>((n + 255) / 256, int64_t(1) << 20);
    hipLaunchKernelGGL(k_fill_u32, dim3(blocks), dim3(256), 0, s, p, n, v);
    prof_end(K_FILL, s);
}

static void launch_scan(const uint32_t* in, uint32_t* out, uint32_t* part, int64_t L,
                        int64_t blocks, hipStream_t s, const uint32_t* skip = nullptr) {
    prof_begin(K_SCAN, s);
    hipLaunchKernelGGL(k_scan_reduce, dim3((uint32_t)blocks), dim3(256), 0, s, in, L, part, skip);
    if (blocks <= SCAN_FUSED_BLOCKS) {
        hipLaunchKernelGGL(k_scan_down<false>, dim3((uint32_t)blocks), dim3(256), 0, s, in, L,
                           part, out, skip);
    } else {
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(256), 0, s, part, blocks, skip);
        hipLaunchKernelGGL(k_scan_down<true>, dim3((uint32_t)blocks), dim3(256), 0, s, in, L,
                           part, out, skip);
    }
    prof_end(K_SCAN, s);
}

hipError_t launch_exclusive_scan(const uint32_t* in, uint32_t* out, uint32_t* part, int64_t L,
                                 hipStream_t s) {
    if (L <= 0) return hipSuccess;
    launch_scan(in, out, part, L, (L + SCAN_TILE - 1) / SCAN_TILE, s);
    return hipGetLastError();
}

// What the per-fragment launch of `blocks` workgroups clears: everything, or
// nothing when that is too much for its threads (see CLEAR_QUADS).
static ClearWords clear_in_launch(const BwdPlan& plan, void* ws, uint32_t blocks) {
    const int64_t quads = (int64_t)(plan.clear_bytes / 16);
    if (quads > CLEAR_QUADS * 256 * (int64_t)blocks) return ClearWords{nullptr, 0};
    return ClearWords{(uint4*)((char*)ws + plan.off_disorder), quads};
}

hipError_t launch_backward(const TexView& t, int fmt, int mode, const float* uv,
                           const float* tbn, const float* view, const float* grad_out,
                           float* grad_tex, float* grad_view, float* grad_uv,
                           const FragMap& frags, const BwdPlan& plan, void* ws, hipStream_t s) {
    const FragMap m = with_frame_staging(frags, t, fmt);
    const int64_t N = m.N;
    char* wsb = (char*)ws;
    uint32_t* keys0 = (uint32_t*)(wsb + plan.off_keys0);
    float* wrec = (float*)(wsb + plan.off_wrec);
    const bool want_tex = grad_tex != nullptr;
    ClearWords clear{nullptr, 0};
    if (want_tex && N > 0) clear = clear_in_launch(plan, ws, fragmap_blocks(m));

    // 1. per fragment
    if (N > 0 && (want_tex || grad_view || grad_uv)) {
        prof_begin(K_BWD_FRAGMENT, s);
        uint32_t* kp = want_tex ? keys0 : nullptr;
        if (mode == MODE_NEAREST) {
            if (fmt == FMT_F32) launch_bwd_fragment_c<FMT_F32, MODE_NEAREST>(t, uv, tbn, view, grad_out, grad_view, grad_uv, kp, wrec, m, plan.cell_bits, plan.sentinel, clear, s);
            else if (fmt == FMT_BF16) launch_bwd_fragment_c<FMT_BF16, MODE_NEAREST>(t, uv, tbn, view, grad_out, grad_view, grad_uv, kp, wrec, m, plan.cell_bits, plan.sentinel, clear, s);
            else launch_bwd_fragment_c<FMT_FP8, MODE_NEAREST>(t, uv, tbn, view, grad_out, grad_view, grad_uv, kp, wrec, m, plan.cell_bits, plan.sentinel, clear, s);
        } else {
            if (fmt == FMT_F32) launch_bwd_fragment_c<FMT_F32, MODE_BILINEAR>(t, uv, tbn, view, grad_out, grad_view, grad_uv, kp, wrec, m, plan.cell_bits, plan.sentinel, clear, s);
            else if (fmt == FMT_BF16) launch_bwd_fragment_c<FMT_BF16, MODE_BILINEAR>(t, uv, tbn, view, grad_out, grad_view, grad_uv, kp, wrec, m, plan.cell_bits, plan.sentinel, clear, s);
            else launch_bwd_fragment_c<FMT_FP8, MODE_BILINEAR>(t, uv, tbn, view, grad_out, grad_view, grad_uv, kp, wrec, m, plan.cell_bits, plan.sentinel, clear, s);
        }
        prof_end(K_BWD_FRAGMENT, s);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (!want_tex) return hipSuccess;

    TileOut out{};
    out.levels = 1;
    out.start[0] = 0;
    out.start[1] = (int64_t)t.W * t.H;
    out.grad[0] = grad_tex;
    return launch_accumulate(t.n, t.C, mode, grad_out, out, plan, ws, clear.quads > 0, s);
}

template <bool SMALL, int IPT>
static void launch_radix_hist(int D, const BwdPlan& plan, hipStream_t s, const uint32_t* kin,
                              int shift, uint32_t* hist, const uint32_t* disorder) {
    const dim3 grid((uint32_t)plan.tiles), block(SORT_THREADS);
    prof_begin(K_RADIX_HIST, s);
    if (D == 8) hipLaunchKernelGGL((k_radix_hist<8, SMALL, IPT>), grid, block, 0, s, kin, plan.records, shift, hist, plan.tiles, disorder);
    else if (D == 9) hipLaunchKernelGGL((k_radix_hist<9, SMALL, IPT>), grid, block, 0, s, kin, plan.records, shift, hist, plan.tiles, disorder);
    else hipLaunchKernelGGL((k_radix_hist<10, SMALL, IPT>), grid, block, 0, s, kin, plan.records, shift, hist, plan.tiles, disorder);
    prof_end(K_RADIX_HIST, s);
}

template <bool SMALL, int IPT>
static void launch_radix_scatter(int D, const BwdPlan& plan, hipStream_t s, const uint32_t* kin,
                                 const uint32_t* vin, uint32_t* kout, uint32_t* vout, int shift,
                                 const uint32_t* hoff, const uint32_t* disorder) {
    const dim3 grid((uint32_t)plan.tiles), block(SORT_THREADS);
    prof_begin(K_RADIX_SCATTER, s);
    if (D == 8) hipLaunchKernelGGL((k_radix_scatter<8, SMALL, IPT>), grid, block, 0, s, kin, vin, kout, vout, plan.records, shift, hoff, plan.tiles, disorder);
    else if (D == 9) hipLaunchKernelGGL((k_radix_scatter<9, SMALL, IPT>), grid, block, 0, s, kin, vin, kout, vout, plan.records, shift, hoff, plan.tiles, disorder);
    else hipLaunchKernelGGL((k_radix_scatter<10, SMALL, IPT>), grid, block, 0, s, kin, vin, kout, vout, plan.records, shift, hoff, plan.tiles, disorder);
    prof_end(K_RADIX_SCATTER, s);
}

// The digits of a pass counted, the first one's by the order check (`check`).
template <bool SMALL, int IPT>
static void launch_counts(int pass, bool check, int D, const BwdPlan& plan, hipStream_t s,
                          const uint32_t* kin, uint32_t* hist, uint32_t* disorder, int2* range) {
    if (pass == 0 && check) {
        const dim3 grid((uint32_t)plan.tiles), block(SORT_THREADS);
        prof_begin(K_ORDER_CHECK, s);
        if (D == 8) hipLaunchKernelGGL((k_keys_in_order_hist<8, SMALL, IPT>), grid, block, 0, s, kin, plan.records, disorder, plan.cell_bits, plan.buckets, range, hist, plan.tiles);
        else if (D == 9) hipLaunchKernelGGL((k_keys_in_order_hist<9, SMALL, IPT>), grid, block, 0, s, kin, plan.records, disorder, plan.cell_bits, plan.buckets, range, hist, plan.tiles);
        else hipLaunchKernelGGL((k_keys_in_order_hist<10, SMALL, IPT>), grid, block, 0, s, kin, plan.records, disorder, plan.cell_bits, plan.buckets, range, hist, plan.tiles);
        prof_end(K_ORDER_CHECK, s);
    } else {
        launch_radix_hist<SMALL, IPT>(D, plan, s, kin, plan.digit_shift[pass], hist, disorder);
    }
}

// One pass of a small sort.
template <int IPT>
static void launch_small_pass(int pass, int D, const BwdPlan& plan, hipStream_t s,
                              const uint32_t* kin, const uint32_t* vin, uint32_t* kout,
                              uint32_t* vout, uint32_t* hist, uint32_t* disorder, int2* range) {
    launch_counts<true, IPT>(pass, true, D, plan, s, kin, hist, disorder, range);
    launch_radix_scatter<true, IPT>(D, plan, s, kin, vin, kout, vout, plan.digit_shift[pass], hist,
                                    disorder);
}

// Whether the R keys in keys0 are in order, and their stable sort (record
// numbers implied by position) if they are not: the order check leaves 0 or 1
// in the workspace's disorder word (cleared before, returned), and with 0
// every launch of the sort returns at once.  With `range` (zero-filled before)
// the check also writes the bucket ranges the keys give if they are in order.
// The sorted keys and their record numbers end in *skeys, *svals.
//
// The order check counts the first pass's digits too where that costs ordered
// keys no more than the launch it saves: up to COUNTING_CHECK records (check and
// counts, us, ordered keys: 2.6M 25.5 and 23, 8.4M 36 and 34, 16.8M 43 and 49, 67M 96
// and 124; unordered: 4.2M 31 and 28, 33.5M 142 and 137), and for a visit plan
// (no ranges), whose keys are seldom ordered (16.6M: 85 and 73).  A small sort
// (see plan_backward) makes fewer launches still: its scatters add the counts
// up themselves (2 launches a pass, 1 for the first, instead of 4).
constexpr int64_t COUNTING_CHECK = int64_t(1) << 23;
static const uint32_t* launch_sort_records(const BwdPlan& plan, void* ws, int2* range,
                                           hipStream_t s, const uint32_t** skeys_out,
                                           const uint32_t** svals_out) {
    char* wsb = (char*)ws;
    uint32_t* keys0 = (uint32_t*)(wsb + plan.off_keys0);
    uint32_t* keys1 = (uint32_t*)(wsb + plan.off_keys1);
    uint32_t* vals0 = (uint32_t*)(wsb + plan.off_vals0);
    uint32_t* vals1 = (uint32_t*)(wsb + plan.off_vals1);
    uint32_t* hist = (uint32_t*)(wsb + plan.off_hist);
    uint32_t* hoff = (uint32_t*)(wsb + plan.off_hoff);
    uint32_t* scanp = (uint32_t*)(wsb + plan.off_scanp);
    uint32_t* disorder = (uint32_t*)(wsb + plan.off_disorder);
    const int64_t R = plan.records;
    const bool small = plan.small_sort;
    const uint32_t* kin = keys0;
    const uint32_t* vin = nullptr;
    const bool counting = small || !range || R <= COUNTING_CHECK;
    if (!counting) {
        prof_begin(K_ORDER_CHECK, s);
        hipLaunchKernelGGL(k_keys_in_order, dim3((uint32_t)((R + 1023) / 1024)), dim3(256), 0, s,
                           keys0, R, disorder, plan.cell_bits, plan.buckets, range);
        prof_end(K_ORDER_CHECK, s);
    }
    for (int pass = 0; pass < plan.passes; pass++) {
        uint32_t* kout = (pass & 1) ? keys0 : keys1;
        uint32_t* vout = (pass & 1) ? vals0 : vals1;
        const int shift = plan.digit_shift[pass];
        const int D = std::max(8, plan.digit_bits[pass]);
        if (small && plan.sort_ipt == 4) {
            launch_small_pass<4>(pass, D, plan, s, kin, vin, kout, vout, hist, disorder, range);
        } else if (small && plan.sort_ipt == 8) {
            launch_small_pass<8>(pass, D, plan, s, kin, vin, kout, vout, hist, disorder, range);
        } else if (small) {
            launch_small_pass<16>(pass, D, plan, s, kin, vin, kout, vout, hist, disorder, range);
        } else {
            const int64_t len = ((int64_t)1 << D) * plan.tiles;
            launch_counts<false, SORT_IPT>(pass, counting, D, plan, s, kin, hist, disorder, range);
            launch_scan(hist, hoff, scanp, len, (len + SCAN_TILE - 1) / SCAN_TILE, s, disorder);
            launch_radix_scatter<false, SORT_IPT>(D, plan, s, kin, vin, kout, vout, shift, hoff,
                                                  disorder);
        }
        kin = kout;
        vin = vout;
    }
    *skeys_out = kin;
    *svals_out = vin;
    return disorder;
}

hipError_t launch_accumulate(int n, int C, int mode, const float* grad_out, const TileOut& out,
                             const BwdPlan& plan, void* ws, bool cleared, hipStream_t s) {
    char* wsb = (char*)ws;
    uint32_t* keys0 = (uint32_t*)(wsb + plan.off_keys0);
    float* wrec = (float*)(wsb + plan.off_wrec);
    float* payf = (float*)(wsb + plan.off_payf);
    float* payg = (float*)(wsb + plan.off_payg);
    uint32_t* big_count = (uint32_t*)(wsb + plan.off_range);  // BIG_LISTS counters
    int2* range = (int2*)(big_count + BIG_LISTS * BIG_STRIDE);
    uint32_t* big_list = (uint32_t*)(wsb + plan.off_biglist);
    float* part = (float*)(wsb + plan.off_part);
    const int64_t R = plan.records;

    // 2. sort, skipped on the device when the records were made in key order
    // (the order check then also writes the bucket ranges)
    const int64_t nb = plan.buckets;
    if (!cleared)  // the disorder word, the counters and the ranges
        launch_fill((uint32_t*)(wsb + plan.off_disorder), (int64_t)(plan.clear_bytes / 4), 0u, s);
    const uint32_t* skeys = keys0;
    const uint32_t* svals = nullptr;
    const uint32_t* dis = nullptr;
    if (R > 0) dis = launch_sort_records(plan, ws, range, s, &skeys, &svals);

    // 3. ranges of the sorted records, with the records' payload in sorted
    // order when buckets hold few records on average: a window of 64 records then
    // serves several buckets, of which each would gather again.  Few is 8 up to
    // 2^23 fragments, which the last-level cache holds, and 24 beyond, where the
    // payload's own kernel has more gathers in flight.  Both return at once when the
    // sort did.  Payload, windows and big pass against ranges, windows and big pass,
    // us: 2M records, 2 a bucket 756 and 788; 4.1M, 12: 317 and 299; 1.3M, 20: 70 and
    // 63; 8.3M, 32: 436 and 381; 4.2M, 64 (RGB): 133 and 95; 16.6M, 16: 1180 and
    // 1239; 33M, 32: 1649 and 1594; 66M, 16: 4610 and 5211, 64: 2846 and 2325.
    // Four buckets (four records a fragment; whole backwards of RGBA): 10.5M records
    // of random rays, 8 a bucket 952 and 741, 16: 740 and 536; of four views in image
    // order, 11: 803 and 735; 33M of random rays, 12: 2687 and 2236, of views, 11:
    // 2685 and 2625, 14: 2368 and 2046; 33M of one view of a height field, 32: 1609
    // and 1596.  Rays without any order lose where the gathers are short: 33M rays of
    // one channel, 32 a bucket, 2776 and 3001 (four views of as many, 14: 2107 and
    // 1826, so the line does not follow them).
    const int64_t frags = mode == MODE_NEAREST ? R : R / 4;
    const bool pay = R > 0 && R <= (frags <= (int64_t(1) << 23) ? 8 : 24) * nb;
    if (R > 0 && !pay) {
        prof_begin(K_BUCKET_RANGES, s);
        hipLaunchKernelGGL(k_bucket_ranges, dim3((uint32_t)((R + 1023) / 1024)), dim3(256), 0, s,
                           skeys, R, plan.cell_bits, nb, range, dis);
        prof_end(K_BUCKET_RANGES, s);
    }
    if (pay) {
        const int64_t per_block = 256 * PAYLOAD_PER_THREAD;
        const dim3 gp((uint32_t)((R + per_block - 1) / per_block));
        prof_begin(K_PAYLOAD, s);
        if (mode == MODE_NEAREST) launch_payload_c<MODE_NEAREST>(C, gp, s, skeys, svals, wrec, grad_out, range, R, plan.cell_bits, nb, payf, payg, dis);
        else launch_payload_c<MODE_BILINEAR>(C, gp, s, skeys, svals, wrec, grad_out, range, R, plan.cell_bits, nb, payf, payg, dis);
        prof_end(K_PAYLOAD, s);
    }
    const int te = (int)plan.tile_elems;
    const uint32_t cell_mask = plan.cell_bits >= 32 ? 0xFFFFFFFFu : ((1u << plan.cell_bits) - 1u);
    // Buckets per wavefront: 4, so that more wavefronts share the windows' loads
    // (us with 8 and with 4: 20 records a bucket 57 and 50, 48: 100 and 86, 64: 50
    // and 43, 128 with bilinear buckets 165 and 153, 2867 buckets of 70: 22 and
    // 15), unless nearly all buckets go to the big pass and are only listed here
    // (256: 48 and 61).  The big-bucket lists' capacity (planned for SEG_GROUP)
    // also holds the lists of groups of 4: a run covers as many buckets.
    const int G = R <= 128 * nb ? 4 : SEG_GROUP;
    const int64_t groups = (nb + G - 1) / G;
    // Consecutive groups that append to one big-bucket list: BIG_RUN (of
    // SEG_GROUP buckets) where that gives every list several runs, fewer for fewer
    // groups, so that all lists (and with them all of the big pass's workgroups)
    // get work.  With BIG_RUN throughout, the 2867 buckets of a 61 x 47 matrix went to 6 of the 64
    // lists and the pass took 38 us.  Powers of two up to BIG_RUN keep the lists
    // within the capacity planned for BIG_RUN.
    int run_log = 0;
    while ((G << (run_log + 1)) <= BIG_RUN * SEG_GROUP &&
           (groups >> (run_log + 1)) >= 4 * BIG_LISTS) run_log++;
    // the workgroups stride over the groups, so at most 2^20 of them keep the
    // launch within one dispatch (2^28 buckets and more at small n)
    const dim3 g1((uint32_t)std::min<int64_t>((groups + 3) / 4, int64_t(1) << 20));
    const float* pf = pay ? payf : nullptr;
    prof_begin(K_SEGACC, s);
    if (mode == MODE_NEAREST) {
        if (G == 4) launch_segacc_c<MODE_NEAREST, 4>(C, g1, (size_t)4 * te * 4, s, skeys, svals, wrec, grad_out, pf, payg, range, out, nb, R, n, cell_mask, big_count, big_list, plan.big_cap, run_log, keys0, dis);
        else launch_segacc_c<MODE_NEAREST, SEG_GROUP>(C, g1, (size_t)4 * te * 4, s, skeys, svals, wrec, grad_out, pf, payg, range, out, nb, R, n, cell_mask, big_count, big_list, plan.big_cap, run_log, keys0, dis);
    } else {
        if (G == 4) launch_segacc_c<MODE_BILINEAR, 4>(C, g1, (size_t)4 * te * 4, s, skeys, svals, wrec, grad_out, pf, payg, range, out, nb, R, n, cell_mask, big_count, big_list, plan.big_cap, run_log, keys0, dis);
        else launch_segacc_c<MODE_BILINEAR, SEG_GROUP>(C, g1, (size_t)4 * te * 4, s, skeys, svals, wrec, grad_out, pf, payg, range, out, nb, R, n, cell_mask, big_count, big_list, plan.big_cap, run_log, keys0, dis);
    }
    prof_end(K_SEGACC, s);
    if (R > 64) {
        // BIG_LISTS x parts workgroups, four wavefronts each; parts grows with
        // the number of buckets that can be big.  Buckets with more than PIECE
        // records: one wavefront per chunk in the same launch, then combined.
        const int64_t parts = std::min<int64_t>(std::max<int64_t>(
            1, (R / 65 + 4 * BIG_LISTS - 1) / (4 * BIG_LISTS)), 64);
        const uint32_t big_blocks = (uint32_t)(BIG_LISTS * parts);
        const uint32_t hot_blocks = R > PIECE ? (uint32_t)((plan.chunks + 3) / 4) : 0u;
        const dim3 g2(big_blocks + hot_blocks);
        prof_begin(K_SEGACC_BIG, s);
        if (mode == MODE_NEAREST)
            launch_segacc_big_c<MODE_NEAREST>(C, g2, (size_t)4 * te * 4, s, skeys, svals, wrec, grad_out, range, out, n, plan.cell_bits, big_count, big_list, plan.big_cap, big_blocks, part, R, nb, keys0, dis);
        else
            launch_segacc_big_c<MODE_BILINEAR>(C, g2, (size_t)4 * te * 4, s, skeys, svals, wrec, grad_out, range, out, n, plan.cell_bits, big_count, big_list, plan.big_cap, big_blocks, part, R, nb, keys0, dis);
        prof_end(K_SEGACC_BIG, s);
    }

    // 5. the chunks of buckets with more than PIECE records
    if (R > PIECE) {
        const dim3 g2((uint32_t)plan.chunks);
        prof_begin(K_COMBINE_HOT, s);
        hipLaunchKernelGGL(k_combine_hot, g2, dim3(64), 0, s, skeys, range, part, out, R, te,
                           plan.cell_bits, nb, keys0, dis, big_count + HOT_FLAG);
        prof_end(K_COMBINE_HOT, s);
    }
    return hipGetLastError();
}


// ---------------------------------------------------------------------------
// visit plan
// ---------------------------------------------------------------------------

// The record key of each fragment as k_bwd_fragment makes it in the nearest
// mode (bucket << cell_bits | cell of its footprint); in the bilinear-bucket
// mode the key of its first bucket (i0, j0) with its cell.
template <int MODE>
__global__ __launch_bounds__(256) void k_plan_keys(int W, int H, int n,
                                                   const float* __restrict__ uv,
                                                   const float* __restrict__ tbn,
                                                   const float* __restrict__ view,
                                                   uint32_t* __restrict__ keys, FragMap m,
                                                   int cell_bits,
                                                   uint32_t* __restrict__ disorder) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *disorder = 0u;  // for the order check
    const int64_t f = frag_of(m, blockIdx.x, gridDim.x, threadIdx.x);
    if (f < 0) return;
    const Frag g = load_frag(uv, tbn, view, f);
    const Dir d = map_direction(g.m, g.w, n);
    const Foot p = footprint(d.sx, d.sy, n);
    int64_t b;
    if constexpr (MODE == MODE_NEAREST) {
        const int i = bucket_of(g.u, W), j = bucket_of(g.v, H);
        b = (int64_t)j * W + i;
    } else {
        int i0, i1, j0, j1;
        float a, bb;
        bucket_pair(g.u, W, i0, i1, a);
        bucket_pair(g.v, H, j0, j1, bb);
        b = (int64_t)j0 * W + i0;
    }
    keys[f] = ((uint32_t)b << cell_bits) | (uint32_t)(p.y0 * n + p.x0);
}

// Planned fragment k is the caller's fragment svals[k] (k itself when the
// keys came in order): its index and its 56-byte record are copied.  A frame is
// moved by three lanes, 12 bytes each: a wavefront's 64 frames are then read
// with one access a line instead of three, and stored by consecutive lanes,
// past the caches, which keep the lines that later records gather from.  16.6M
// records (two 4K views): 630 us with a lane per record, 498 with its stores
// through LDS, 478 so (2.0 GB moved, 4.2 TB/s; the address unit is busy 85% of
// the time).
__global__ __launch_bounds__(256) void k_plan_gather(const uint32_t* __restrict__ svals,
                                                     int64_t N, const float* __restrict__ uv,
                                                     const float* __restrict__ tbn,
                                                     const float* __restrict__ view,
                                                     int32_t* __restrict__ order,
                                                     float* __restrict__ uv_out,
                                                     float* __restrict__ tbn_out,
                                                     float* __restrict__ view_out,
                                                     const uint32_t* __restrict__ disorder) {
    if (sort_skipped(disorder)) svals = nullptr;
    const int lane = threadIdx.x & 63;
    const int64_t k0 = (int64_t)xcd_block_id(blockIdx.x, gridDim.x) * 256 + (threadIdx.x & ~63u);
    const int64_t k = k0 + lane;
    uint32_t f = 0;  // past the end: fragment 0, not stored
    if (k < N) f = svals ? svals[k] : (uint32_t)k;
    float m[3][3], v[3];
#pragma unroll
    for (int p = 0; p < 3; p++) {  // third q % 3 of frame q / 3
        const int q = lane + 64 * p;
        const float* src = tbn + (int64_t)(uint32_t)__shfl((int)f, q / 3, 64) * 9 + q % 3 * 3;
#pragma unroll
        for (int c = 0; c < 3; c++) m[p][c] = src[c];
    }
#pragma unroll
    for (int c = 0; c < 3; c++) v[c] = view[(int64_t)f * 3 + c];
    const float2 t = ((const float2*)uv)[f];
#pragma unroll
    for (int p = 0; p < 3; p++) {
        const int q = lane + 64 * p;
        if (k0 + q / 3 < N) {
#pragma unroll
            for (int c = 0; c < 3; c++)
                __builtin_nontemporal_store(m[p][c], tbn_out + (k0 * 3 + q) * 3 + c);
        }
    }
    if (k >= N) return;
#pragma unroll
    for (int c = 0; c < 3; c++) __builtin_nontemporal_store(v[c], view_out + k * 3 + c);
    nt_store2(uv_out + 2 * k, t.x, t.y);
    __builtin_nontemporal_store((int32_t)f, order + k);
}

// Rows of a per-fragment array moved by a plan's order: gather (dst[k] =
// src[order[k]], into plan order) or scatter (dst[order[k]] = src[k], back to
// the caller's order).  Rows of `row` 4-byte words; 16-byte accesses when the
// row is a whole number of them and both arrays are 16-byte aligned.
template <bool VEC>
__global__ __launch_bounds__(256) void k_permute_rows(const int32_t* __restrict__ order,
                                                      int64_t N, int row,
                                                      const uint32_t* __restrict__ src,
                                                      uint32_t* __restrict__ dst, int scatter) {
    const int64_t k = (int64_t)xcd_block_id(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
    if (k >= N) return;
    const int64_t o = order[k];
    if (o < 0 || o >= N) return;  // not an index of the array: no row moves
    const int64_t from = scatter ? k : o, to = scatter ? o : k;
    if constexpr (VEC) {
        const int q = row / 4;
        const uint4* s4 = (const uint4*)src + from * q;
        uint4* d4 = (uint4*)dst + to * q;
        for (int i = 0; i < q; i++) d4[i] = s4[i];
    } else {
        for (int i = 0; i < row; i++) dst[to * row + i] = src[from * row + i];
    }
}

hipError_t launch_permute_rows(const int32_t* order, int64_t N, int row_words, const void* src,
                               void* dst, bool scatter, hipStream_t s) {
    if (N <= 0) return hipSuccess;
    const bool vec = row_words % 4 == 0 && ((uintptr_t)src % 16) == 0 && ((uintptr_t)dst % 16) == 0;
    const dim3 grid((uint32_t)((N + 255) / 256));
    prof_begin(K_PERMUTE, s);
    if (vec)
        hipLaunchKernelGGL(k_permute_rows<true>, grid, dim3(256), 0, s, order, N, row_words,
                           (const uint32_t*)src, (uint32_t*)dst, (int)scatter);
    else
        hipLaunchKernelGGL(k_permute_rows<false>, grid, dim3(256), 0, s, order, N, row_words,
                           (const uint32_t*)src, (uint32_t*)dst, (int)scatter);
    prof_end(K_PERMUTE, s);
    return hipGetLastError();
}

hipError_t launch_plan(const TexView& t, int mode, const float* uv, const float* tbn,
                       const float* view, const FragMap& m, const BwdPlan& plan, void* ws,
                       int32_t* order, float* uv_out, float* tbn_out, float* view_out,
                       hipStream_t s) {
    const int64_t N = m.N;
    if (N <= 0) return hipSuccess;
    uint32_t* keys0 = (uint32_t*)((char*)ws + plan.off_keys0);
    uint32_t* disorder = (uint32_t*)((char*)ws + plan.off_disorder);
    prof_begin(K_PLAN_KEYS, s);
    if (mode == MODE_NEAREST)
        hipLaunchKernelGGL(k_plan_keys<MODE_NEAREST>, dim3(fragmap_blocks(m)), dim3(256), 0, s,
                           t.W, t.H, t.n, uv, tbn, view, keys0, m, plan.cell_bits, disorder);
    else
        hipLaunchKernelGGL(k_plan_keys<MODE_BILINEAR>, dim3(fragmap_blocks(m)), dim3(256), 0, s,
                           t.W, t.H, t.n, uv, tbn, view, keys0, m, plan.cell_bits, disorder);
    prof_end(K_PLAN_KEYS, s);
    const uint32_t *skeys = nullptr, *svals = nullptr;
    const uint32_t* dis = launch_sort_records(plan, ws, nullptr, s, &skeys, &svals);
    prof_begin(K_PLAN_GATHER, s);
    hipLaunchKernelGGL(k_plan_gather, dim3((uint32_t)((N + 255) / 256)), dim3(256), 0, s, svals,
                       N, uv, tbn, view, order, uv_out, tbn_out, view_out, dis);
    prof_end(K_PLAN_GATHER, s);
    return hipGetLastError();
}

template <int FMT, int MODE>
static void launch_lod_frag_c(int C, dim3 grid, hipStream_t s, const LevelSet& ls,
                              const float* uv, const float* tbn, const float* view,
                              const float* duv, const float* go, const LevelStarts& st, float* gview, float* guv, uint32_t* keys,
                              float* wrec, float* gl, const FragMap& m, int cb, uint32_t sent,
                              const ClearWords& clear) {
    switch (C) {
    case 1: hipLaunchKernelGGL((k_lod_bwd_fragment<FMT, 1, MODE>), grid, dim3(256), 0, s, ls, uv, tbn, view, duv, go, st, gview, guv, keys, wrec, gl, m, cb, sent, clear); break;
    case 2: hipLaunchKernelGGL((k_lod_bwd_fragment<FMT, 2, MODE>), grid, dim3(256), 0, s, ls, uv, tbn, view, duv, go, st, gview, guv, keys, wrec, gl, m, cb, sent, clear); break;
    case 3: hipLaunchKernelGGL((k_lod_bwd_fragment<FMT, 3, MODE>), grid, dim3(256), 0, s, ls, uv, tbn, view, duv, go, st, gview, guv, keys, wrec, gl, m, cb, sent, clear); break;
    default: hipLaunchKernelGGL((k_lod_bwd_fragment<FMT, 4, MODE>), grid, dim3(256), 0, s, ls, uv, tbn, view, duv, go, st, gview, guv, keys, wrec, gl, m, cb, sent, clear); break;
    }
}

hipError_t launch_lod_bwd_fragment(const LevelSet& ls, int fmt, int mode, const float* uv,
                                   const float* tbn, const float* view, const float* duv,
                                   const float* grad_out, const int64_t* start, float* grad_view, float* grad_uv,
                                   uint32_t* keys, float* wrec, float* gl, const FragMap& m,
                                   const BwdPlan& plan, void* ws, bool* cleared, hipStream_t s) {
    LevelStarts st{};
    for (int l = 0; l <= ls.levels && l <= MAX_LEVELS; l++) st.v[l] = start[l];
    const dim3 grid(fragmap_blocks(m));
    const int C = ls.C;
    ClearWords clear{nullptr, 0};
    if (keys) clear = clear_in_launch(plan, ws, grid.x);
    *cleared = clear.quads > 0;
    prof_begin(K_LOD_BWD_FRAGMENT, s);
    if (mode == MODE_NEAREST) {
        if (fmt == FMT_F32) launch_lod_frag_c<FMT_F32, MODE_NEAREST>(C, grid, s, ls, uv, tbn, view, duv, grad_out, st, grad_view, grad_uv, keys, wrec, gl, m, plan.cell_bits, plan.sentinel, clear);
        else if (fmt == FMT_BF16) launch_lod_frag_c<FMT_BF16, MODE_NEAREST>(C, grid, s, ls, uv, tbn, view, duv, grad_out, st, grad_view, grad_uv, keys, wrec, gl, m, plan.cell_bits, plan.sentinel, clear);
        else launch_lod_frag_c<FMT_FP8, MODE_NEAREST>(C, grid, s, ls, uv, tbn, view, duv, grad_out, st, grad_view, grad_uv, keys, wrec, gl, m, plan.cell_bits, plan.sentinel, clear);
    } else {
        if (fmt == FMT_F32) launch_lod_frag_c<FMT_F32, MODE_BILINEAR>(C, grid, s, ls, uv, tbn, view, duv, grad_out, st, grad_view, grad_uv, keys, wrec, gl, m, plan.cell_bits, plan.sentinel, clear);
        else if (fmt == FMT_BF16) launch_lod_frag_c<FMT_BF16, MODE_BILINEAR>(C, grid, s, ls, uv, tbn, view, duv, grad_out, st, grad_view, grad_uv, keys, wrec, gl, m, plan.cell_bits, plan.sentinel, clear);
        else launch_lod_frag_c<FMT_FP8, MODE_BILINEAR>(C, grid, s, ls, uv, tbn, view, duv, grad_out, st, grad_view, grad_uv, keys, wrec, gl, m, plan.cell_bits, plan.sentinel, clear);
    }
    prof_end(K_LOD_BWD_FRAGMENT, s);
    return hipGetLastError();
}

}  // namespace rt
