// One dense fp32 product per workgroup grid on 16x16x4 MFMA, operands straight from global memory
// into the registers the instruction reads: the device code of the fp32 train step's layered
// products, shared by the kernels that run one product per launch and by the launch that runs a
// product beside the weight-gradient tiles.
#pragma once
#include <hip/hip_runtime.h>

namespace rp {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) char* gbytes;   // global memory, byte-addressed

constexpr unsigned int kMmThreads = 256;

enum { MM_BIAS_RELU = 0, MM_BIAS = 1, MM_MASK = 2, MM_PARTIAL = 3 };

// C = A B (+ epilogue).  A is [M x K] with K contiguous.  NT: B is [N x K], K contiguous;
// otherwise B is [K x N], N contiguous.  The M rows come in `parts` equal parts (1, or 2: the
// rows of s and the rows of s'); a tile never straddles two parts, and the tiles of part 1 take
// B_hi and bias_hi (the frozen target network's layer) instead of B and bias.
struct MmArgs {
    const float* A;
    unsigned int lda;
    const float* B;
    const float* B_hi;
    unsigned int ldb;
    const float* bias;
    const float* bias_hi;
    const float* mask;       // MM_MASK: [M x N], the output is kept where mask > 0
    unsigned int ldmask;
    float* C;
    unsigned int ldc;
    unsigned int rows_per_part, parts, tiles_per_part;
    unsigned int N, K;       // K: what one workgroup contracts over
    // MM_PARTIAL: the contraction is split over gridDim.z workgroups per tile as well, K columns
    // each; workgroup z stores its partial product (no bias) c_stride elements after the one before.
    size_t c_stride;
};

// One wavefront's 16 x 16 tile of C over the K range [k_lo, k_lo + 16 * ngroups).
// Lane l = 16 q + c of a 16x16x4 MFMA supplies A[row c][k slot q] and B[k slot q][column c] and
// receives C[rows 4 q .. 4 q + 3][column c].  A group is 16 consecutive k: MFMA j of a group
// takes k = 16 g + 4 q + j in slot q, so that a lane's share of A (and of B when it is K
// contiguous) for a whole group is one 16-byte load.  P groups are in flight at a time: the
// loads of group g + P are requested as soon as group g has been multiplied.  Loads never
// branch: a group past the end re-reads the last one and is multiplied by zero.
template <bool NT, int P>
__device__ __forceinline__ f32x4 mm_tile(const float* __restrict__ A, unsigned int lda, unsigned int arow,
                                         const float* __restrict__ B, unsigned int ldb, unsigned int bcol,
                                         unsigned int k_lo, unsigned int ngroups, unsigned int lane) {
    const unsigned int q = lane >> 4;
    const gbytes ap = (gbytes)reinterpret_cast<const char*>(A) + ((size_t)arow * lda + k_lo + 4u * q) * 4u;
    const gbytes bp = NT ? (gbytes)reinterpret_cast<const char*>(B) + ((size_t)bcol * ldb + k_lo + 4u * q) * 4u
                         : (gbytes)reinterpret_cast<const char*>(B) + ((size_t)(k_lo + 4u * q) * ldb + bcol) * 4u;
    f32x4 a[P], b[P];
    auto load = [&](int s, unsigned int g) {
        const unsigned int gc = g < ngroups ? g : ngroups - 1u;
        a[s] = *(const __attribute__((address_space(1))) f32x4*)(ap + (size_t)gc * 64u);
        if (NT) {
            b[s] = *(const __attribute__((address_space(1))) f32x4*)(bp + (size_t)gc * 64u);
        } else {
            const gbytes rb = bp + (size_t)gc * 16u * ldb * 4u;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                b[s][j] = *(const __attribute__((address_space(1))) float*)(rb + (size_t)j * ldb * 4u);
        }
    };
#pragma unroll
    for (int s = 0; s < P; ++s) load(s, (unsigned int)s);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (unsigned int g0 = 0; g0 < ngroups; g0 += P) {
#pragma unroll
        for (int s = 0; s < P; ++s) {
            const bool live = g0 + s < ngroups;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(live ? a[s][j] : 0.f, b[s][j], acc, 0, 0, 0);
            load(s, g0 + s + P);
        }
    }
    return acc;
}

// Few tiles and a long contraction: 16 x 16 per workgroup with K split over its four wavefronts,
// summed through LDS in a fixed order.
// (bx, by, bz: the workgroup's place in the product's grid; part: 3 KB of LDS)
template <bool NT, int EPI, int P>
__device__ __forceinline__ void mm_f32_block(const MmArgs& p, unsigned int bx, unsigned int by, unsigned int bz,
                                             float (*part)[64][4]) {
    const unsigned int lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const unsigned int c = lane & 15u, q = lane >> 4;
    const unsigned int part_id = by / p.tiles_per_part;
    const unsigned int m_begin = part_id * p.rows_per_part, m_end = m_begin + p.rows_per_part;
    const unsigned int m0 = m_begin + (by - part_id * p.tiles_per_part) * 16u, n0 = bx * 16u;
    const float* Bm = part_id ? p.B_hi : p.B;
    const float* bias = part_id ? p.bias_hi : p.bias;
    // rows past the part's end re-read its last row; they are not stored
    const unsigned int arow = min(m0 + c, m_end - 1u);
    const unsigned int ng = p.K >> 6;
    const unsigned int k_lo = (EPI == MM_PARTIAL ? bz * p.K : 0u) + wave * ng * 16u;
    f32x4 acc = mm_tile<NT, P>(p.A, p.lda, arow, Bm, p.ldb, n0 + c, k_lo, ng, lane);
    if (wave) {
#pragma unroll
        for (int v = 0; v < 4; ++v) part[wave - 1u][lane][v] = acc[v];
    }
    __syncthreads();
    if (wave) return;
#pragma unroll
    for (unsigned int w = 0; w < 3; ++w)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] += part[w][lane][v];
    const unsigned int n = n0 + c;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const unsigned int m = m0 + 4u * q + v;
        if (m >= m_end) continue;
        float x = acc[v];
        if (EPI == MM_BIAS_RELU) {
            x += bias[n];
            x = x > 0.f ? x : 0.f;
        } else if (EPI == MM_BIAS) {
            x += bias[n];
        } else if (EPI == MM_MASK) {
            if (!(p.mask[(size_t)m * p.ldmask + n] > 0.f)) x = 0.f;
        }
        p.C[(EPI == MM_PARTIAL ? bz * p.c_stride : 0) + (size_t)m * p.ldc + n] = x;
    }
}

// Workgroups are dealt to the eight XCDs, each with an L2 of its own, round-robin: a launch's
// workgroup `block` of `count` takes number block_to_tile of its tiles, so that an XCD gets a
// contiguous range of them (the last count mod 8 are left where they are).
__device__ __forceinline__ unsigned int block_to_tile(unsigned int block, unsigned int count) {
    const unsigned int per = count >> 3;
    return block < 8u * per ? (block & 7u) * per + (block >> 3) : block;
}

// Many tiles: 32 x 32 of C per workgroup of W wavefronts, which split K: wavefront w takes the groups
// of 16 consecutive k with numbers w, w + W, .. and forms the whole tile from them, and the
// partial tiles are added through LDS in a fixed order, E = 16 / W adjacent columns per thread.
// What bounds such a product is the compute unit's vector-memory path, which takes a load
// instruction about every sixteen cycles (a 16-byte one takes as long as it needs for 1 KB), so
// what counts is MFMAs per load: here 16 MFMAs on six loads (two of A; four of B, two columns wide)
// or four (NT: 16 bytes along K for both), where a 16 x 16 quarter per wavefront takes 4 on five.
// P groups are in flight at a time; groups past the end re-read the last one and count as zero, so P is no
// more than a wavefront has (a contraction of up to 64: one each; with two, half of the loads were
// repeats, and the steps below took 23.8, 27.2 and 43.6 us).
// Quarters -> this, us per launch: 1024 x 512 x 512 14.3 -> 11.0 (of which 3.4 are the MFMAs at peak),
// NT 512 x 512 x 512 10.9 -> 8.5; us per step where the contractions are 32 and 64: 27-256-64-30 at batch
// 128 22.7 -> 22.0, 27-1024-64-30 at batch 128 26.1 -> 25.4, at batch 600 46.9 -> 39.6.
constexpr unsigned int kMmTile = 32, kMmTileLd = kMmTile + 4;
template <bool NT, int EPI, int W, int P>
__device__ __forceinline__ void mm_f32_tile32(const MmArgs& p, unsigned int bx, unsigned int by,
                                              float (*part)[kMmTile][kMmTileLd]) {
    static_assert(EPI != MM_PARTIAL && (W == 4 || W == 8), "whole products, four or eight wavefronts");
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const unsigned int tid = threadIdx.x, lane = tid & 63u;
    const unsigned int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned int c = lane & 15u, q = lane >> 4;
    const unsigned int part_id = by / p.tiles_per_part;
    const unsigned int m_begin = part_id * p.rows_per_part, m_end = m_begin + p.rows_per_part;
    const unsigned int m0 = m_begin + (by - part_id * p.tiles_per_part) * kMmTile, n0 = bx * kMmTile;
    const float* Bm = part_id ? p.B_hi : p.B;
    const float* bias = part_id ? p.bias_hi : p.bias;
    const unsigned int groups = p.K >> 4;
    // (rows past the part's end re-read its last row; they are not stored)
    gbytes ap[2], bp[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const unsigned int m = min(m0 + 16u * i + c, m_end - 1u);
        ap[i] = (gbytes)reinterpret_cast<const char*>(p.A) + ((size_t)m * p.lda + 4u * q) * 4u;
        bp[i] = NT ? (gbytes)reinterpret_cast<const char*>(Bm) + ((size_t)(n0 + 16u * i + c) * p.ldb + 4u * q) * 4u
                   : (gbytes)reinterpret_cast<const char*>(Bm) + ((size_t)(4u * q) * p.ldb + n0 + 2u * c) * 4u;
    }
    f32x4 a[P][2], b[P][2];   // b: NT: [column block][k]; otherwise the pairs of columns of k = 2 i, 2 i + 1
    auto load = [&](int s, unsigned int t) {
        const unsigned int g = min(wave + (unsigned int)W * t, groups - 1u);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[s][i] = *(const __attribute__((address_space(1))) f32x4*)(ap[i] + (size_t)g * 64u);
            if constexpr (NT) {
                b[s][i] = *(const __attribute__((address_space(1))) f32x4*)(bp[i] + (size_t)g * 64u);
            } else {
                const gbytes rb = bp[0] + ((size_t)g * 16u + 2u * i) * p.ldb * 4u;
                const f32x2 b0 = *(const __attribute__((address_space(1))) f32x2*)rb;
                const f32x2 b1 = *(const __attribute__((address_space(1))) f32x2*)(rb + (size_t)p.ldb * 4u);
                b[s][i] = f32x4{b0[0], b0[1], b1[0], b1[1]};
            }
        }
    };
#pragma unroll
    for (int s = 0; s < P; ++s) load(s, (unsigned int)s);
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k = 0; k < 2; ++k) acc[i][k] = f32x4{0.f, 0.f, 0.f, 0.f};
    const unsigned int rounds = (groups + W - 1u) / W;
    for (unsigned int t0 = 0; t0 < rounds; t0 += P) {
#pragma unroll
        for (int s = 0; s < P; ++s) {
            const bool live = wave + W * (t0 + s) < groups;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            live ? a[s][i][j] : 0.f, live ? (NT ? b[s][k][j] : b[s][j >> 1][2 * (j & 1) + k]) : 0.f,
                            acc[i][k], 0, 0, 0);
            if (t0 + P < rounds) load(s, t0 + P + s);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float* row = part[wave][16u * i + 4u * q + v];
            if constexpr (NT) {
                row[c] = acc[i][0][v];
                row[16u + c] = acc[i][1][v];
            } else {
                *reinterpret_cast<f32x2*>(row + 2u * c) = f32x2{acc[i][0][v], acc[i][1][v]};
            }
        }
    __syncthreads();
    constexpr unsigned int E = 16u / W;
    typedef float f32xE __attribute__((ext_vector_type(E)));
    const unsigned int r = tid / (kMmTile / E), col = (tid % (kMmTile / E)) * E;
    const unsigned int m = m0 + r, n = n0 + col;
    f32xE x = *reinterpret_cast<const f32xE*>(&part[0][r][col]);
#pragma unroll
    for (int w = 1; w < W; ++w) x += *reinterpret_cast<const f32xE*>(&part[w][r][col]);
    if (m >= m_end) return;
    if constexpr (EPI == MM_MASK) {
        const f32xE k = *reinterpret_cast<const f32xE*>(p.mask + (size_t)m * p.ldmask + n);
#pragma unroll
        for (unsigned int e = 0; e < E; ++e)
            if (!(k[e] > 0.f)) x[e] = 0.f;
    } else {
        x += *reinterpret_cast<const f32xE*>(bias + n);
        if constexpr (EPI == MM_BIAS_RELU) {
#pragma unroll
            for (unsigned int e = 0; e < E; ++e) x[e] = x[e] > 0.f ? x[e] : 0.f;
        }
    }
    *reinterpret_cast<f32xE*>(p.C + (size_t)m * p.ldc + n) = x;
}

// K is split over a workgroup's wavefronts when a product has few tiles and a long contraction.
inline bool want_ksplit(unsigned int M, unsigned int N, unsigned int K) {
    const unsigned int tiles32 = ((M + 31u) / 32u) * (N / 32u);
    return K >= 256u && K % 64u == 0 && tiles32 < 256u;
}

// Whether dZ1 = (dZ2 W2^T) masked, [B x H] over K = G, runs in the launch of the weight-gradient
// tiles rather than in one of its own: that launch holds one variant of the product (16 x 16 per
// workgroup, K over its wavefronts, eight groups of 16 in flight), the one a batch of the
// paper's sizes and a wide second layer take.
inline bool dz1_rides_with_tiles(unsigned int B, unsigned int H, unsigned int G) {
    return want_ksplit(B, H, G) && G >= 512u;
}

}  // namespace rp
