// rt_device.hpp -- device-side building blocks shared by the gfx950 kernels of
// the radiance-bucket lookup: the incidence -> bucket mapping in binary32,
// texel loads and decodes for the storage formats, the sample directions of
// the bake, and launch helpers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rt {

constexpr int FMT_F32 = 0;
constexpr int FMT_BF16 = 1;
constexpr int FMT_FP8 = 2;
constexpr int FMT_BIT1 = 3;  // one bit per sample, one channel

// 32-bit words per bucket of the 1-bit storage: sample k = y n + x is bit
// k % 32 of word k / 32 of its bucket; the bits past n n are zero.
__host__ __device__ __forceinline__ int bit_words(int n) { return (n * n + 31) >> 5; }

constexpr int MODE_NEAREST = 0;
constexpr int MODE_BILINEAR = 1;

// Native vector types (for non-temporal loads and stores).
typedef float f4v __attribute__((ext_vector_type(4)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));

// Texture as seen by a kernel: bucket-major [H][W][n][n][C].  A bucket
// dictionary keeps `entries` buckets in data (its codebook) and an index map
// [H][W] (1, 2 or 4 bytes per bucket) naming each bucket's entry, with an
// optional gain per bucket.
struct TexView {
    const void* data;     // FMT_BIT1: uint32 words, bit_words(n) per bucket
    const float* scales;  // [H][W], FP8 only
    int W, H, n, C;
    const void* index;    // dictionary: entry of each bucket, or nullptr
    const float* gains;   // dictionary: gain of each bucket, or nullptr (1)
    int index_bytes;      // 1, 2 or 4
    int entries;          // dictionary: codebook entries K
};

// Entry of bucket b of a dictionary; numbers past the codebook read its last
// entry (the index map is caller data that the host cannot check).
__device__ __forceinline__ int64_t dict_entry(const TexView& t, int64_t b) {
    uint32_t e;
    if (t.index_bytes == 1) e = ((const uint8_t*)t.index)[b];
    else if (t.index_bytes == 2) e = ((const uint16_t*)t.index)[b];
    else e = ((const uint32_t*)t.index)[b];
    return (int64_t)min(e, (uint32_t)(t.entries - 1));
}

// A mip chain: level l has max(1, W >> l) x max(1, H >> l) buckets of the
// same n, C and format; only the storage pointers differ per level.
constexpr int MAX_LEVELS = 17;
struct LevelSet {
    const void* data[MAX_LEVELS];
    const float* scales[MAX_LEVELS];
    int levels;
    int W, H, n, C;  // level 0
};

// ---------------------------------------------------------------------------
// Launch geometry: gfx950 places consecutive workgroups of a launch on its 8
// XCDs round-robin.  Renumbering the workgroups so that each XCD receives a
// contiguous range of the logical index space keeps neighbouring fragments
// (which land in the same buckets) on the same L2.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t xcd_block_id(uint32_t bid, uint32_t nblocks) {
    constexpr uint32_t XCDS = 8;
    uint32_t xcd = bid % XCDS;
    uint32_t q = nblocks / XCDS, r = nblocks % XCDS;
    uint32_t before = xcd * q + (xcd < r ? xcd : r);
    return before + bid / XCDS;
}

// ---------------------------------------------------------------------------
// Decodes.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// E4M3 byte -> binary32 value divided by 2^8.  The byte's exponent and
// mantissa fields are placed in the corresponding fields of a binary16 (whose
// exponent bias is 8 larger), which represents e4m3 * 2^-8 exactly for every
// finite code, subnormals included; the 2^8 is folded into the bucket scale.
__device__ __forceinline__ float e4m3_div256(uint32_t byte) {
    uint32_t h = ((byte & 0x80u) << 8) | ((byte & 0x7Fu) << 7);
    return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
}

// The codes in bytes 1 and 3 of a word, as e4m3_div256 decodes them (three
// integer operations for both).
__device__ __forceinline__ void e4m3_div256_odd(uint32_t w, float& one, float& three) {
    const uint32_t h = (w & 0x80008000u) | ((w >> 1) & 0x3F803F80u);
    one = (float)__builtin_bit_cast(_Float16, (unsigned short)h);
    three = (float)__builtin_bit_cast(_Float16, (unsigned short)(h >> 16));
}

struct F4 {
    float v[4];
};

// Load the C channels of texel `t` (index in texels, bucket-major) as
// binary32.  For FP8 the values are e4m3/256; the caller multiplies by
// 256 * scale once per bucket.
template <int FMT, int C>
__device__ __forceinline__ F4 load_texel(const void* __restrict__ data, int64_t t) {
    F4 r;
#pragma unroll
    for (int c = 0; c < 4; c++) r.v[c] = 0.f;
    if constexpr (FMT == FMT_F32) {
        const float* p = (const float*)data;
        if constexpr (C == 4) {
            float4 q = ((const float4*)p)[t];
            r.v[0] = q.x; r.v[1] = q.y; r.v[2] = q.z; r.v[3] = q.w;
        } else if constexpr (C == 2) {
            float2 q = ((const float2*)p)[t];
            r.v[0] = q.x; r.v[1] = q.y;
        } else {
#pragma unroll
            for (int c = 0; c < C; c++) r.v[c] = p[t * C + c];
        }
    } else if constexpr (FMT == FMT_BF16) {
        const uint16_t* p = (const uint16_t*)data;
        if constexpr (C == 4) {
            uint2 q = ((const uint2*)p)[t];
            r.v[0] = bf16_lo(q.x); r.v[1] = bf16_hi(q.x);
            r.v[2] = bf16_lo(q.y); r.v[3] = bf16_hi(q.y);
        } else if constexpr (C == 2) {
            uint32_t q = ((const uint32_t*)p)[t];
            r.v[0] = bf16_lo(q); r.v[1] = bf16_hi(q);
        } else {
#pragma unroll
            for (int c = 0; c < C; c++) r.v[c] = bf16_lo((uint32_t)p[t * C + c]);
        }
    } else {
        const uint8_t* p = (const uint8_t*)data;
        if constexpr (C == 4) {
            uint32_t q = ((const uint32_t*)p)[t];
#pragma unroll
            for (int c = 0; c < 4; c++) r.v[c] = e4m3_div256((q >> (8 * c)) & 0xFFu);
        } else if constexpr (C == 2) {
            uint32_t q = ((const uint16_t*)p)[t];
            r.v[0] = e4m3_div256(q & 0xFFu); r.v[1] = e4m3_div256(q >> 8);
        } else {
#pragma unroll
            for (int c = 0; c < C; c++) r.v[c] = e4m3_div256((uint32_t)p[t * C + c]);
        }
    }
    return r;
}

// Bytes of one stored sample value (channel) in format FMT (not RT_FMT_BIT1).
template <int FMT>
__host__ __device__ constexpr int storage_bytes() {
    return FMT == FMT_F32 ? 4 : FMT == FMT_BF16 ? 2 : 1;
}

// The two texels of a footprint's row as stored: texels t and t + 1 of a
// bucket.
template <int FMT, int C>
struct RowBits {
    static constexpr int SIZE = storage_bytes<FMT>(), TEXEL = C * SIZE;
    // alignment of a texel (C = 3: of one value); gfx950 reads global memory at
    // any byte address
    static constexpr int ALIGN = C == 3 ? SIZE : TEXEL;
    static constexpr int WORDS = (2 * TEXEL + 3) / 4;
    uint32_t w[WORDS];

    // the first BYTES bytes of w from src, the rest of their last word 0
    template <int BYTES>
    __device__ __forceinline__ void take(const unsigned char* src) {
        struct __attribute__((packed, aligned(ALIGN))) Raw {
            unsigned char byte[BYTES];
        };
        const Raw raw = *(const Raw*)src;
        if constexpr (BYTES % 4 == 0) {
            __builtin_memcpy(w, &raw, BYTES);
        } else {
#pragma unroll
            for (int k = 0; k < (BYTES + 3) / 4; k++) {
                w[k] = 0u;
                __builtin_memcpy(&w[k], raw.byte + 4 * k, BYTES - 4 * k < 4 ? BYTES - 4 * k : 4);
            }
        }
    }
    // exactly the two texels' bytes
    __device__ __forceinline__ void load_two(const unsigned char* src) { take<2 * TEXEL>(src); }
    // the same for texels of three 2-byte values, by a 4-byte aligned access of 12
    // bytes (from the value before src where src lies between words) and one of
    // the last value
    __device__ __forceinline__ void load_two_aligned(const unsigned char* src) {
        static_assert(TEXEL == 6, "12 bytes, 2-byte aligned");
        struct __attribute__((packed, aligned(4))) Words {
            uint32_t x, y, z;
        };
        const uint32_t odd = (uint32_t)(uintptr_t)src & 2u;
        const Words p = *(const Words*)(src - odd);
        const uint32_t last = *(const uint16_t*)(src + 10);
        w[0] = __builtin_amdgcn_alignbit(p.y, p.x, 8 * odd);
        w[1] = __builtin_amdgcn_alignbit(p.z, p.y, 8 * odd);
        w[2] = __builtin_amdgcn_alignbit(last, p.z, 8 * odd);
    }
    // the texels at a and b
    __device__ __forceinline__ void load_each(const unsigned char* a, const unsigned char* b) {
        static_assert(TEXEL % 4 == 0, "whole words");
        RowBits first, second;
        first.template take<TEXEL>(a);
        second.template take<TEXEL>(b);
#pragma unroll
        for (int k = 0; k < TEXEL / 4; k++) {
            w[k] = first.w[k];
            w[TEXEL / 4 + k] = second.w[k];
        }
    }
    // a bucket of one sample: it stands for both
    __device__ __forceinline__ void load_one(const unsigned char* src) {
        RowBits a;
        a.template take<TEXEL>(src);
#pragma unroll
        for (int k = 0; k < WORDS; k++) {
            // bytes 4k .. 4k + 3 of the texel followed by itself
            uint32_t word = 0u;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int at = (4 * k + j) % TEXEL;
                word |= ((a.w[at / 4] >> (8 * (at % 4))) & 0xFFu) << (8 * j);
            }
            w[k] = word;
        }
    }
    // the values as load_texel gives them
    __device__ __forceinline__ void decode(F4& a, F4& b) const {
        float code[4 * WORDS];  // FP8
        if constexpr (FMT == FMT_FP8) {
#pragma unroll
            for (int k = 0; k < WORDS; k++) {
                e4m3_div256_odd(w[k] << 8, code[4 * k], code[4 * k + 2]);
                e4m3_div256_odd(w[k], code[4 * k + 1], code[4 * k + 3]);
            }
        }
#pragma unroll
        for (int e = 0; e < 8; e++) {
            float v = 0.f;
            if (e % 4 < C) {
                const int k = e / 4 * C + e % 4;
                if constexpr (FMT == FMT_F32) v = __uint_as_float(w[k]);
                else if constexpr (FMT == FMT_BF16) v = (k & 1) ? bf16_hi(w[k / 2]) : bf16_lo(w[k / 2]);
                else v = code[k];
            }
            (e < 4 ? a : b).v[e % 4] = v;
        }
    }
};

// The rows of NB footprints, one in each of NB buckets of n x n samples, the
// first texel of each at src[k].  All loads are issued before any of them is
// waited for.  Two texels of a row by one access halve the instructions of a
// gather, which is bound by the lines that each of them touches (64 when every
// lane reads another bucket).  Four buckets, 8.4M fragments of an FP8 RGBA
// texture: lookup 511 -> 285 us, fragment pass of the backward 509 -> 418 (387
// with the rest of it shortened); 2.1M fragments of a BF16 RGBA one: lookup 205 ->
// 155.  One bucket: the same to 5% less.
//
// The order of the loads is fixed, bucket by bucket (the barriers): one such load
// brings as many lines as a quarter of the L1 holds, and the accesses to a bucket's
// lines have to follow each other while they are there.  Left to the scheduler,
// 2.5M random rays on a 64 x 32 matrix of 8 x 8, four buckets: FP8 RGBA 97 us and
// 68 so, BF16 RGBA 91 and 71, FP32 88 and 59, FP32 RGBA 135 and 98 (a texel a load,
// waited for by bucket: 133, 119, 66, 104).
//
// Four buckets of FP32 RGBA hold 12 to 23 more registers than texels waited for
// by bucket.  Before and after, us: lookup (eight wavefronts a SIMD, then six; 4M
// fragments) 66.8 and 68.0 in image order, 655 and 655 of random rays; with the
// level of detail (six, five) 157 and 148, 1157 and 1166; a light of 16 samples (six,
// four; 2M) 282 and 270, 5603 and 4728.  A dictionary's codebook is in the caches, so
// there the order costs more than it saves in image order (FP32 RGB 66 and 71, RGBA
// 75 and 79) and less on random rays (280 and 261, 259 and 257).  One bucket of FP32
// or BF16: 4% slower to 2% faster on a 256 x 256 matrix of 16 x 16, 10 to 34% faster
// on the 64 x 32 one of 8 x 8.
//
// ALIGNED (texels of three 2-byte values): by word-aligned accesses, for lookups
// that come back to a bucket, as a light of several samples does: accesses of 12
// bytes off the word boundaries lose what the L1 holds of it.  BF16 RGB, a light
// of 16 samples, one bucket, 2M fragments on a 512 x 512 matrix of 16 x 16, a texel
// an access, two by one, two aligned: random rays 920, 1360 and 911 us, image
// order 257, 109 and 107; on a 64 x 32 matrix of 8 x 8 546, 362 and 316.  With four
// buckets in image order the aligned form is the slower one (687, 270 and 305).
template <int FMT, int C, int NB, bool ALIGNED = false>
__device__ __forceinline__ void load_rows(const unsigned char* const src[NB], int n,
                                          RowBits<FMT, C> row[NB][2]) {
    using Row = RowBits<FMT, C>;
    const int below = n >= 2 ? n * Row::TEXEL : 0;
    if constexpr (Row::TEXEL == 16) {  // an access a texel in any case
        const int second = n >= 2 ? 16 : 0;
#pragma unroll
        for (int k = 0; k < NB; k++) {
            row[k][0].load_each(src[k], src[k] + second);
            row[k][1].load_each(src[k] + below, src[k] + below + second);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else if (n >= 2) {  // the second column is x0 + 1 (see footprint)
#pragma unroll
        for (int k = 0; k < NB; k++) {
            if constexpr (ALIGNED) {
                row[k][0].load_two_aligned(src[k]);
                row[k][1].load_two_aligned(src[k] + below);
            } else {
                row[k][0].load_two(src[k]);
                row[k][1].load_two(src[k] + below);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int k = 0; k < NB; k++) {
            row[k][0].load_one(src[k]);
            // (either for the wide or for the narrow texels, the other way
            // leaves the row in memory)
            if constexpr (Row::TEXEL > 4) row[k][1] = row[k][0];
            else row[k][1].load_one(src[k]);
        }
    }
}

// Orders a wavefront's LDS accesses before and after it (the wavefront owns
// the memory, so no workgroup barrier is needed).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Factor applied to a bucket's decoded samples: 1, or 256 * scale for FP8.
template <int FMT>
__device__ __forceinline__ float bucket_factor(const float* __restrict__ scales, int64_t b) {
    if constexpr (FMT == FMT_FP8) return 256.0f * scales[b];
    else return 1.0f;
}

// ---------------------------------------------------------------------------
// Fragment inputs.
// ---------------------------------------------------------------------------

// Which fragment a thread handles.  Flat: workgroup b, thread t -> 256 b + t.
// Tiled (the caller's images of height x width pixels): workgroup b is one
// TILE_X x TILE_Y pixel tile, tiles row-major within an image and images in
// order, so the fragments of one workgroup are neighbouring pixels and
// neighbouring workgroups are neighbouring tiles.  Either way the workgroup
// index is first renumbered with xcd_block_id.
constexpr int TILE_X = 32, TILE_Y = 8;
static_assert(TILE_X * TILE_Y == 256, "one tile per 256-thread workgroup");

struct FragMap {
    int64_t N;
    int32_t width, height;     // 0: flat
    int32_t tiles_x, tiles_y;  // tiles per row and per column of an image
    int32_t stage;             // flat launches: stage the frames in LDS
};

inline FragMap make_fragmap(int64_t N, int32_t views, int32_t height, int32_t width) {
    FragMap m{N, 0, 0, 0, 0, 0};
    if (views > 0 && height > 0 && width > 0) {
        m.width = width;
        m.height = height;
        m.tiles_x = (width + TILE_X - 1) / TILE_X;
        m.tiles_y = (height + TILE_Y - 1) / TILE_Y;
    }
    return m;
}

// Flat launches of the lookup and of its per-fragment backward stage their
// fragments' frames and view vectors through LDS (load_frag_block) when the
// texture is larger than the caches.  Then the taps come from HBM and the
// launch is bound by its memory instructions, which the 16-byte staging
// loads reduce; on a texture the caches hold the launch is bound by issue,
// and the staging's LDS traffic costs more than it saves.
constexpr int64_t STAGE_FRAMES_MIN_TEXTURE_BYTES = int64_t(1) << 30;

inline FragMap with_frame_staging(FragMap m, const TexView& t, int fmt) {
    int64_t bytes = 0;
    if (!t.index) {
        const int64_t buckets = (int64_t)t.W * t.H;
        if (fmt == FMT_BIT1) bytes = buckets * bit_words(t.n) * 4;
        else bytes = buckets * t.n * t.n * t.C * (fmt == FMT_F32 ? 4 : fmt == FMT_BF16 ? 2 : 1);
    }
    m.stage = m.width == 0 && bytes >= STAGE_FRAMES_MIN_TEXTURE_BYTES ? 1 : 0;
    return m;
}

// workgroups of a launch over all fragments
inline uint32_t fragmap_blocks(const FragMap& m) {
    if (m.width == 0) return (uint32_t)((m.N + 255) / 256);
    const int64_t views = m.N / ((int64_t)m.width * m.height);
    return (uint32_t)(views * m.tiles_x * m.tiles_y);
}

// fragment of thread `tid` in workgroup `bid`, or -1 past the end / outside
// the image
__device__ __forceinline__ int64_t frag_of(const FragMap& m, uint32_t bid, uint32_t nblocks,
                                           int tid) {
    const uint32_t b = xcd_block_id(bid, nblocks);
    if (m.width == 0) {
        const int64_t f = (int64_t)b * 256 + tid;
        return f < m.N ? f : -1;
    }
    const uint32_t per_view = (uint32_t)(m.tiles_x * m.tiles_y);
    const uint32_t v = b / per_view, r = b - v * per_view;
    const uint32_t ty = r / (uint32_t)m.tiles_x, tx = r - ty * (uint32_t)m.tiles_x;
    const int x = (int)tx * TILE_X + (tid % TILE_X), y = (int)ty * TILE_Y + (tid / TILE_X);
    if (x >= m.width || y >= m.height) return -1;
    return ((int64_t)v * m.height + y) * m.width + x;
}

struct Frag {
    float u, v;
    float m[9];
    float w[3];
};

__device__ __forceinline__ Frag load_frag(const float* __restrict__ uv, const float* __restrict__ tbn,
                                          const float* __restrict__ view, int64_t f) {
    Frag r;
    float2 t = ((const float2*)uv)[f];
    r.u = t.x;
    r.v = t.y;
#pragma unroll
    for (int k = 0; k < 9; k++) r.m[k] = tbn[f * 9 + k];
#pragma unroll
    for (int k = 0; k < 3; k++) r.w[k] = view[f * 3 + k];
    return r;
}

// The frames and view vectors of a flat launch's wavefront (64 consecutive
// fragments) staged in LDS.  A fragment's 36 + 12 bytes do not fall on a
// lane's 16-byte vector, but the wavefront's 2304 + 768 bytes do: they are
// read with 16-byte loads when both arrays are 16-byte aligned there, else
// with 4-byte loads, and every lane then takes its own record from LDS (a
// stride of 9 or 3 words: no bank conflicts).  Each wavefront stages its own
// records, so no workgroup barrier couples the wavefronts.  Tiled launches
// read per lane.
struct FragStage {
    float tbn[256 * 9];
    float view[256 * 3];
};

// Returns the record of fragment f (f >= 0); every lane of a wavefront must
// reach it together.
__device__ __forceinline__ Frag load_frag_block(const float* __restrict__ uv,
                                                const float* __restrict__ tbn,
                                                const float* __restrict__ view, const FragMap& m,
                                                int64_t f, FragStage& s) {
    if (m.width != 0 || !m.stage) return f >= 0 ? load_frag(uv, tbn, view, f) : Frag{};
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t f0 = (int64_t)xcd_block_id(blockIdx.x, gridDim.x) * 256 + w * 64;
    const int nf = (int)(m.N - f0 < 64 ? (m.N - f0 > 0 ? m.N - f0 : 0) : 64);
    const float* bt = tbn + f0 * 9;
    const float* bv = view + f0 * 3;
    float* st = s.tbn + w * 64 * 9;
    float* sv = s.view + w * 64 * 3;
    if (nf == 64 && ((((uintptr_t)bt) | ((uintptr_t)bv)) & 15) == 0) {
        for (int q = lane; q < 144; q += 64) ((f4v*)st)[q] = ((const f4v*)bt)[q];
        if (lane < 48) ((f4v*)sv)[lane] = ((const f4v*)bv)[lane];
    } else {
        for (int q = lane; q < nf * 9; q += 64) st[q] = bt[q];
        for (int q = lane; q < nf * 3; q += 64) sv[q] = bv[q];
    }
    wave_lds_sync();
    Frag r{};
    if (f >= 0) {
        const float2 t = ((const float2*)uv)[f];
        r.u = t.x;
        r.v = t.y;
#pragma unroll
        for (int k = 0; k < 9; k++) r.m[k] = st[lane * 9 + k];
#pragma unroll
        for (int k = 0; k < 3; k++) r.w[k] = sv[lane * 3 + k];
    }
    return r;
}

// ---------------------------------------------------------------------------
// Incidence -> in-bucket sample coordinate, binary32.
//
//   u = M V (rows T, B, N), L = |u|
//   Eq. (1b) with I = u / L:  A = sqrt(2) (I_x, I_y) / |(I_x, I_y, I_z + 1)|.
//   For unit I, |(I_x, I_y, I_z + 1)|^2 = 2 (1 + I_z), so A = (u_x, u_y) k with
//   k = 1 / sqrt(L (L + u_z)); this form avoids normalising u first.
//   Eq. (3): B = (|A|_2 / max(|A_x|, |A_y|)) A, B = 0 at A = 0.
//   Clamp (Note after Eq. 3) and texel centres: s = clamp((B + 1) n/2 - 1/2, 0, n-1).
// ---------------------------------------------------------------------------
struct Dir {
    float sx, sy;        // clamped sample coordinates
    bool clx, cly;       // axis at or beyond its clamp bound
    float ax, ay;        // A
    float ux, uy, uz, L; // tangent-space incidence before normalisation
    float k;             // 1 / sqrt(L (L + u_z))
};

// The mapping is evaluated with one rounding per operation (no fused
// multiply-adds), so that every kernel that maps a fragment -- the lookups,
// the backward, the visit plan -- computes the same sample coordinate and the
// same footprint for it, whatever the surrounding code lets the compiler fuse.
__device__ __forceinline__ Dir map_direction(const float m[9], const float w[3], int n) {
#pragma clang fp contract(off)
    Dir d;
    d.ux = m[0] * w[0] + m[1] * w[1] + m[2] * w[2];
    d.uy = m[3] * w[0] + m[4] * w[1] + m[5] * w[2];
    d.uz = m[6] * w[0] + m[7] * w[1] + m[8] * w[2];
    d.L = sqrtf(d.ux * d.ux + d.uy * d.uy + d.uz * d.uz);
    float q = d.L * (d.L + d.uz);
    d.k = q > 0.f ? 1.0f / sqrtf(q) : 0.f;  // q = 0: I = -N (or u = 0): A = 0
    d.ax = d.ux * d.k;
    d.ay = d.uy * d.k;
    float rho = sqrtf(d.ax * d.ax + d.ay * d.ay);
    float mx = fmaxf(fabsf(d.ax), fabsf(d.ay));
    float r = mx > 0.f ? rho / mx : 0.f;
    float bx = d.ax * r, by = d.ay * r;
    float half_n = 0.5f * (float)n;
    float top = (float)(n - 1);
    float sx = (bx + 1.0f) * half_n - 0.5f;
    float sy = (by + 1.0f) * half_n - 0.5f;
    d.clx = !(sx > 0.f && sx < top);
    d.cly = !(sy > 0.f && sy < top);
    d.sx = fminf(fmaxf(sx, 0.f), top);  // NaN -> 0
    d.sy = fminf(fmaxf(sy, 0.f), top);
    return d;
}

// Bilinear footprint inside a bucket.  The first sample is kept at or below
// n-2 so that the second is always x0+1 (at s = n-1 the weight of the first is
// then exactly 0); for n = 1 both are sample 0.
struct Foot {
    int x0, y0, x1, y1;
    float fx, fy;
};

__device__ __forceinline__ Foot footprint(float sx, float sy, int n) {
#pragma clang fp contract(off)
    Foot p;
    int hi = n >= 2 ? n - 2 : 0;
    p.x0 = min((int)sx, hi);
    p.y0 = min((int)sy, hi);
    p.x1 = min(p.x0 + 1, n - 1);
    p.y1 = min(p.y0 + 1, n - 1);
    p.fx = sx - (float)p.x0;
    p.fy = sy - (float)p.y0;
    if (n == 1) { p.fx = 0.f; p.fy = 0.f; }
    return p;
}

// k mod W in [0, W).  A wavefront with every k there already (a texture that
// does not repeat) skips the division, about 20 instructions.
__device__ __forceinline__ int wrap(int k, int W) {
    if ((uint32_t)k >= (uint32_t)W) {
        k %= W;
        k = k < 0 ? k + W : k;
    }
    return k;
}

// Bucket column (or row) of a texture coordinate: floor(frac(u) W) with the UV
// plane repeating.  It is evaluated as floor(u W) mod W, which is the same
// integer, because u W is exact for a power-of-two W whereas frac(u) = u + 1
// of a small negative u is not representable in binary32.  Non-finite and
// huge coordinates (where binary32 has no fraction left) select bucket 0.
__device__ __forceinline__ int bucket_of(float u, int W) {
    const float fq = floorf(u * (float)W);
    if (!(fabsf(fq) < 1073741824.0f)) return 0;
    return wrap((int)fq, W);
}

// Bilinear-bucket footprint in UV: p = frac(u) W - 1/2, columns floor(p) and
// floor(p)+1 (wrapping), weight a = p - floor(p).  Evaluated from t = u W
// (exact for a power-of-two W) split into floor(t) and r = t - floor(t)
// (exact, except for -1/2 < t < 0 where it rounds by at most 2^-25); then
// a = r - 1/2 (exact) or r + 1/2 (rounded by at most 2^-25).  The weight is
// thus within 2^-24 however large u W is, whereas forming u W - 1/2 first
// would round it to the ulp of u W.  Non-finite and huge coordinates behave
// as u = 0.
__device__ __forceinline__ void bucket_pair(float u, int W, int& i0, int& i1, float& a) {
    const float t = u * (float)W;
    const float ft = floorf(t);
    if (!(fabsf(ft) < 1073741824.0f)) {
        i0 = W - 1;
        i1 = 0;
        a = 0.5f;
        return;
    }
    const float r = t - ft;
    int k = (int)ft;
    if (r >= 0.5f) {
        a = r - 0.5f;
    } else {
        a = r + 0.5f;
        k -= 1;
    }
    i0 = wrap(k, W);
    i1 = i0 + 1 == W ? 0 : i0 + 1;
}

// Level of detail of a fragment from its UV screen derivatives d = (du/dx,
// dv/dx, du/dy, dv/dy): rho = the larger pixel footprint in buckets of level 0
// (W x H), lambda = log2 rho clamped to [0, levels - 1] (0 when rho is 0 or
// not finite); the lookup blends levels l0 = floor(lambda) and l0 + 1 with
// weights 1 - t and t (t = 0 on the last level).
__device__ __forceinline__ void lod_split(const float4 d, int W, int H, int levels, int& l0,
                                          float& t) {
    const float ax = d.x * (float)W, ay = d.y * (float)H;
    const float bx = d.z * (float)W, by = d.w * (float)H;
    const float rho = fmaxf(sqrtf(ax * ax + ay * ay), sqrtf(bx * bx + by * by));
    float lambda = 0.f;
    if (rho > 0.f && rho <= 3.0e38f) lambda = fminf(fmaxf(log2f(rho), 0.f), (float)(levels - 1));
    l0 = (int)floorf(lambda);
    t = lambda - (float)l0;
    if (l0 >= levels - 1) {
        l0 = levels - 1;
        t = 0.f;
    }
}

// ---------------------------------------------------------------------------
// Sample centres of a bucket as directions (the write side: Eqs. 4a, 4b, 2c).
// At sample (x, y) of an n x n bucket: B = ((2x+1)/n - 1, (2y+1)/n - 1);
// A = max(|B_x|, |B_y|) / |B| B (A = 0 at B = 0); the reflection vector
// R = (-A_x w, -A_y w, 1 - |A|^2), w = sqrt(2 - |A|^2), and the incidence
// I = (A_x w, A_y w, 1 - |A|^2) that the lookup maps onto the sample (R
// mirrored about the normal).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void sample_directions(int x, int y, int n, float R[3], float I[3]) {
    const float bx = (float)(2 * x + 1) / (float)n - 1.f;
    const float by = (float)(2 * y + 1) / (float)n - 1.f;
    const float rho = sqrtf(bx * bx + by * by);
    const float m = fmaxf(fabsf(bx), fabsf(by));
    float ax = 0.f, ay = 0.f;
    if (rho > 0.f) {
        const float f = m / rho;
        ax = f * bx;
        ay = f * by;
    }
    const float r2 = ax * ax + ay * ay;
    const float w = sqrtf(fmaxf(0.f, 2.f - r2));
    R[0] = -ax * w;
    R[1] = -ay * w;
    R[2] = 1.f - r2;
    I[0] = ax * w;
    I[1] = ay * w;
    I[2] = 1.f - r2;
}

}  // namespace rt
