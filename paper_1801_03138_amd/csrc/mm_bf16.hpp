// Device code of the mixed-precision step's large products: bf16 operands, fp32 accumulation on
// 32x32x16 MFMA, one workgroup of eight wavefronts per output tile.
//
// At these sizes (17 GFLOP a launch) a launch spends some 8 us on its start, its first slice and its
// outputs and 12 us per 1,024 of contraction on 8192 x 1024 outputs, whatever the tiling; so the kernels
// that use these products do more per launch and write less, and the loop is built to need no second
// workgroup on the compute unit:
//  - slices of 64 of the contraction go from global memory straight into LDS (global_load_lds), NS of them
//    in flight; one barrier a slice, placed before the slice's last step, so that the
//    operands of the next slice's first step are read from LDS while that last step is multiplied;
//  - operands of step s + 1 are read before the MFMAs of step s issue, and requests of the slice
//    after next go out between MFMAs, one at a time;
//  - KG = 2: two groups of wavefronts share the tile's contraction, each for half of a slice's steps,
//    with twice as large a tile per wavefront (fewer LDS bytes per MFMA); they swap halves of
//    their accumulators through LDS at the end.
// Measured alone, 8192 x 1024 x 1024 with bias, ReLU and bf16 output: 128 x 128 tiles of four wavefronts,
// two slices deep and two workgroups a compute unit 21.4 us, 256 x 128 with KG = 2 19.8.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace rp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned short bf16_bits;
// 16 bytes in flight between a load and its use.  A native vector type: arrays of HIP's uint4
// struct are not promoted to registers by the compiler and end up in scratch memory.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) char* gchar;   // global memory, byte-addressed

#define RP_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

__device__ __forceinline__ bf16x8 as_bf16x8(const u32x4& v) { return __builtin_bit_cast(bf16x8, v); }

// Row (0..31 within the 32x32 tile) of accumulator element v held by `lane`; its column is lane % 32.
__device__ __forceinline__ unsigned int acc_row(unsigned int v, unsigned int lane) {
    return 8u * (v >> 2) + 4u * (lane >> 5) + (v & 3u);
}

// s_waitcnt vmcnt(N), nothing else
template <unsigned int N>
__device__ __forceinline__ void wait_loads() {
    __builtin_amdgcn_s_waitcnt((N & 0xFu) | ((N >> 4) << 14) | 0x0F70u);
}
// waits until at most `slices` (at most MAXS) slices of L loads each are in flight
template <int L, int MAXS, int K = 0>
__device__ __forceinline__ void wait_slices(unsigned int slices) {
    if constexpr (K >= MAXS) {
        wait_loads<K * L>();
    } else {
        if (slices == K) wait_loads<K * L>();
        else wait_slices<L, MAXS, K + 1>(slices);
    }
}

// This wavefront's LDS reads are in its registers, then everybody's are.
__device__ __forceinline__ void slice_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// One wavefront-wide request, 16 bytes a lane, to consecutive LDS addresses from dst on.  The row's address is
// pinned in scalar registers, the lane adds a 32-bit offset: no vector arithmetic per request.
__device__ __forceinline__ void request_lds(gchar row, unsigned int lane_off, unsigned char* dst) {
    asm volatile("" : "+s"(row));
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(row + lane_off), RP_LDS_PTR(dst), 16, 0, 0);
}

// 8 bytes to LDS.  Written out, because the compiler lets an LDS write of its own wait for every request in flight
// (it could be to the same place); slice_barrier waits for it.
__device__ __forceinline__ void write_lds8(unsigned char* at, unsigned int lo, unsigned int hi) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const unsigned int addr = (unsigned int)(size_t)RP_LDS_PTR(at);
    asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"((u32x2{lo, hi})) : "memory");
}

// A product's operands and how its tiles are numbered.
struct GemmArgs {
    const bf16_bits* A;
    unsigned int lda;
    const bf16_bits* Bt;
    const bf16_bits* Bt_hi;        // B operand of the tiles whose first row is m_split or beyond
    unsigned int m_split;
    unsigned int ldb;
    unsigned int M, N, K;          // K: length one workgroup contracts over
    unsigned int batch;            // products over the batch: rows of the operands
    unsigned int tiles_m, tiles_n, splits;
    unsigned int band;             // tiles are numbered band by band: `band` tile columns at a time, rows fastest after that
};

// Workgroups are dealt to the eight XCDs round-robin; each XCD gets a contiguous range of
// tile numbers, and tiles are numbered so that such a range is a compact block of the output
// (bands of `band` tile columns, within a band row by row): the workgroups that share an L2
// then share as few operand panels as possible, and each panel is fetched by few XCDs.  False: the
// workgroup has no tile.
template <int BM, int BN>
__device__ __forceinline__ bool tile_of(const GemmArgs& p, unsigned int block, unsigned int* m0, unsigned int* n0,
                                        unsigned int* split) {
    const unsigned int per_split = p.tiles_m * p.tiles_n, n_tiles = per_split * p.splits;
    const unsigned int per_xcd = (n_tiles + 7u) / 8u;
    const unsigned int tile_s = (block & 7u) * per_xcd + (block >> 3);
    if (tile_s >= n_tiles) return false;
    const unsigned int tile = tile_s % per_split;
    const unsigned int band_tiles = p.tiles_m * p.band, band_id = tile / band_tiles, in_band = tile % band_tiles;
    const unsigned int width = min(p.band, p.tiles_n - band_id * p.band);
    *m0 = (in_band / width) * BM;
    *n0 = (band_id * p.band + in_band % width) * BN;
    *split = tile_s / per_split;
    return true;
}

// A tile of BM x BN outputs, eight wavefronts as KG groups of WGM x WGN.
template <int BM_, int BN_, int WGM_, int WGN_, int KG_, int NS_>
struct MmTile {
    static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, KG = KG_, NS = NS_;
    static constexpr int NW = WGM * WGN * KG, kThreads = 64 * NW;
    static constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;   // 32 x 32 tiles a wavefront multiplies ...
    static constexpr int TK = TM / KG;                             // ... and tile rows it ends up with
    static constexpr int SP = 4 / KG;                              // 16-deep steps a group takes of a slice
    static constexpr unsigned int kStage = (BM + BN) * 128u;       // bytes of a slice
    static constexpr unsigned int kLds = NS * kStage > (KG == 2 ? BM * BN * 4u : 0u) ? NS * kStage : BM * BN * 4u;
    static_assert(NW == 8 && TM >= KG && TM % KG == 0 && TN >= 1 && NS >= 3 && SP % 2 == 0, "tile shape");
};

// The pipelined loop over nk slices, shared by both operand layouts.  fetch_one(u, buf, slice): request u
// (0 .. L - 1) of a slice into buffer buf; read(slice, buf, s, set): operands of step s; mfma(i, j, set); arrived(slice,
// buf): after one of the first slice and the last NS - 1 has arrived for everybody and before anybody reads it; before_tail(): once, when
// the last slice has arrived (loads of the epilogue's operands go there: no wait counts loads after it).
// make: for an operand that the workgroup works out itself, into LDS, a slice ahead: start(slice, buf) after the barrier
// that brought slice - 1 (to buf); multiply(slice); finish(slice, part, parts) for all parts, between the MFMAs of a step;
// after that and a barrier the slice is read, and done(slice) is called, and flush() a step later.  Loads and stores of its
// own only make the waits for the requests stricter: those complete in order.
struct MakeNothing {
    __device__ __forceinline__ void start(unsigned int, unsigned int) {}
    __device__ __forceinline__ void multiply(unsigned int) {}
    __device__ __forceinline__ void finish(unsigned int, int, int) {}
    __device__ __forceinline__ void done(unsigned int) {}
    __device__ __forceinline__ void flush() {}
};
template <class S, int L, class Fetch, class Read, class Mfma, class Arrived, class Tail, class Make>
__device__ __forceinline__ void mm_pipeline(unsigned int nk, Fetch&& fetch_one, Read&& read, Mfma&& mfma,
                                            Arrived&& arrived, Tail&& before_tail, Make&& make) {
    constexpr int NS = S::NS, SP = S::SP, NM = SP * S::TM * S::TN;
#pragma unroll
    for (unsigned int s0 = 0; s0 + 1 < (unsigned int)NS; ++s0)
        if (s0 < nk) {
#pragma unroll
            for (int u = 0; u < L; ++u) fetch_one(u, s0, s0);
        }
    if (nk < 2) before_tail();
    if (nk == 0) return;
    make.multiply(0u);
    make.finish(0u, 0, 1);
    wait_slices<L, NS - 2>(nk > 1 ? min(nk - 1u, (unsigned int)NS - 2u) : 0u);
    slice_barrier();
    arrived(0u, 0u);
    read(0u, 0u, 0, 0);
    make.done(0u);
    if (nk > 1) make.start(1u, 0u);
    auto step = [&](int s, auto fetch_flag, unsigned int fbuf, unsigned int fslice, bool making, unsigned int made) {
        constexpr bool FETCH = decltype(fetch_flag)::value;
#pragma unroll
        for (int i = 0; i < S::TM; ++i)
#pragma unroll
            for (int j = 0; j < S::TN; ++j) {
                mfma(i, j, s & 1);
                if (FETCH) {
                    const int m = (s * S::TM + i) * S::TN + j;   // this MFMA's number within the slice
#pragma unroll
                    for (int u = m * L / NM; u < (m + 1) * L / NM; ++u) fetch_one(u, fbuf, fslice);
                }
                if (s + 2 == SP && making) make.finish(made, i * S::TN + j, S::TM * S::TN);
                if (FETCH) __builtin_amdgcn_sched_barrier(0);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    // requests of a slice that are out before its last step: what may be in flight, beyond whole
    // slices, when the next slice is awaited there
    constexpr int SHARE = (SP - 1) * S::TM * S::TN * L / NM;
    unsigned int kt = 0, cur = 0, nxt = 1, fb = NS - 1;   // slice; buffers of this slice, the next one, the requested one
    // (two loops, so that each has one straight-line body: with both kinds of multiply in one loop
    // the compiler moved all accumulators between register files on every iteration)
    for (; kt + NS - 1 < nk; ++kt) {
#pragma unroll
        for (int s = 0; s < SP; ++s) {
            if (s + 1 < SP) {
                read(kt, cur, s + 1, (s + 1) & 1);
                if (s == 0) {
                    make.flush();
                    make.multiply(kt + 1u);
                }
            } else {
                // the next slice is here (its requests are a whole slice old); after the barrier nobody reads
                // this slice's buffer any more (its last operands are in registers), and the
                // next iteration's requests go there
                wait_loads<(NS - 3) * L + SHARE>();
                slice_barrier();
                read(kt + 1u, nxt, 0, 0);
                make.done(kt + 1u);
                make.start(kt + 2u, nxt);
            }
            __builtin_amdgcn_sched_barrier(0);
            step(s, std::true_type{}, fb, kt + NS - 1u, true, kt + 1u);
        }
        cur = nxt;
        nxt = nxt + 1 == NS ? 0 : nxt + 1;
        fb = fb + 1 == NS ? 0 : fb + 1;
    }
    for (; kt < nk; ++kt) {
#pragma unroll
        for (int s = 0; s < SP; ++s) {
            if (s + 1 < SP) {
                read(kt, cur, s + 1, (s + 1) & 1);
                if (s == 0) {
                    make.flush();
                    if (kt + 1 < nk) make.multiply(kt + 1u);
                }
            } else if (kt + 1 < nk) {
                wait_slices<L, NS - 2>(nk - 2u - kt);
                slice_barrier();
                arrived(kt + 1u, nxt);
                read(kt + 1u, nxt, 0, 0);
                make.done(kt + 1u);
                if (kt + 2 < nk) make.start(kt + 2u, nxt);
                if (kt + 2 == nk) before_tail();
            }
            __builtin_amdgcn_sched_barrier(0);
            step(s, std::false_type{}, 0u, 0u, kt + 1 < nk, kt + 1u);
        }
        cur = nxt;
        nxt = nxt + 1 == NS ? 0 : nxt + 1;
    }
}

// KG = 2: the groups swap accumulators, so that wavefronts of group g end with the sums of tile rows
// g TK .. + TK - 1 of their region in acc[0 .. TK - 1].  All of smem is overwritten.
template <class S>
__device__ __forceinline__ void mm_swap_groups(f32x16 (&acc)[S::TM][S::TN], unsigned char* smem, unsigned int wave,
                                               unsigned int lane) {
    __syncthreads();
    if constexpr (S::KG == 2) {
        constexpr int TK = S::TK, TN = S::TN;
        const unsigned int group = wave / (S::WGM * S::WGN), other = wave ^ (S::WGM * S::WGN);
        f32x4* const x = reinterpret_cast<f32x4*>(smem) + lane;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (group != (unsigned int)h) {
#pragma unroll
                for (int i = 0; i < TK; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x16& c = acc[h * TK + i][j];
                            x[((wave * TK + i) * TN + j) * 256u + q * 64u] = f32x4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
                        }
            }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (group == (unsigned int)h) {
#pragma unroll
                for (int i = 0; i < TK; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x4 v = x[((other * TK + i) * TN + j) * 256u + q * 64u];
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                // (group 0's half first on both sides)
                                const float mine = acc[h * TK + i][j][4 * q + e];
                                acc[i][j][4 * q + e] = h == 0 ? mine + v[e] : v[e] + mine;
                            }
                        }
                    }
            }
        __syncthreads();
    }
}

template <class S>
__device__ __forceinline__ void mm_clear(f32x16 (&acc)[S::TM][S::TN]) {
#pragma unroll
    for (int i = 0; i < S::TM; ++i)
#pragma unroll
        for (int j = 0; j < S::TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
}

// Where a wavefront's share of the finished tile begins (after mm_swap_groups): TK x TN tiles of 32.
template <class S>
__device__ __forceinline__ void mm_wave_at(unsigned int wave, unsigned int* m, unsigned int* n) {
    const unsigned int wi = wave % (S::WGM * S::WGN);
    *m = (wi / S::WGN) * (S::TM * 32u) + wave / (S::WGM * S::WGN) * (S::TK * 32u);
    *n = wi % S::WGN * (S::TN * 32u);
}

// C[m][n] = sum_k A[m][k] B[n][k], both operands K-contiguous; the MFMA operands are exchanged, so that
// element v of a lane's 32 x 32 accumulator is row lane % 32, column acc_row(v, lane).  p.K is a multiple of 64.
// Rows of an operand beyond its last repeat that one.  LDS rows are 128 bytes; the 16-byte piece at
// position c of row r holds piece c ^ (r / 2 mod 8), which spreads 16 rows' reads over all banks.
template <class S, class Tail>
__device__ __forceinline__ void mm_nt(const GemmArgs& p, unsigned int m0, unsigned int n0, unsigned char* smem,
                                      f32x16 (&acc)[S::TM][S::TN], Tail&& before_tail) {
    constexpr int NW = S::NW, GA = S::BM / 8 / NW, GB = S::BN / 8 / NW, L = GA + GB;   // eight rows a request
    static_assert(S::BM % (8 * NW) == 0 && S::BN % (8 * NW) == 0, "loader shape");
    const unsigned int lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned int group = wave / (S::WGM * S::WGN), wi = wave % (S::WGM * S::WGN);
    const unsigned int wn = wi % S::WGN, wm = wi / S::WGN, half = lane >> 5;
    auto swz = [](unsigned int r) { return (r >> 1) & 7u; };
    const unsigned int lr = lane >> 3, lc = lane & 7u;
    unsigned int a_off[GA], b_off[GB];
#pragma unroll
    for (int u = 0; u < GA; ++u) {
        const unsigned int r = (wave * GA + u) * 8u + lr;
        a_off[u] = (min(r, p.M - 1u - m0) * p.lda + (lc ^ swz(r)) * 8u) * 2u;
    }
#pragma unroll
    for (int u = 0; u < GB; ++u) {
        const unsigned int r = (wave * GB + u) * 8u + lr;
        b_off[u] = (min(r, p.N - 1u - n0) * p.ldb + (lc ^ swz(r)) * 8u) * 2u;
    }
    const gchar a_base = (gchar)reinterpret_cast<const char*>(p.A + (size_t)m0 * p.lda);
    const gchar b_base = (gchar)reinterpret_cast<const char*>((m0 >= p.m_split ? p.Bt_hi : p.Bt) + (size_t)n0 * p.ldb);
    auto fetch_one = [&](int u, unsigned int buf, unsigned int slice) {
        unsigned char* dst = smem + buf * S::kStage + (u < GA ? (wave * GA + u) * 1024u : S::BM * 128u + (wave * GB + u - GA) * 1024u);
        request_lds((u < GA ? a_base : b_base) + (size_t)slice * 128u,
                    u < GA ? a_off[u < GA ? u : 0] : b_off[u >= GA ? u - GA : 0], dst);
    };
    const unsigned int a_row = (wm * S::TM * 32u + (lane & 31u)) * 128u;
    const unsigned int b_row = S::BM * 128u + (wn * S::TN * 32u + (lane & 31u)) * 128u;
    const unsigned int sw = swz(lane & 31u);
    u32x4 a[2][S::TM], b[2][S::TN];
    auto read = [&](unsigned int, unsigned int buf, int s, int set) {
        const unsigned char* base = smem + buf * S::kStage + ((2u * (group * S::SP + s) + half) ^ sw) * 16u;
#pragma unroll
        for (int j = 0; j < S::TN; ++j) b[set][j] = *reinterpret_cast<const u32x4*>(base + b_row + j * 4096);
#pragma unroll
        for (int i = 0; i < S::TM; ++i) a[set][i] = *reinterpret_cast<const u32x4*>(base + a_row + i * 4096);
    };
    auto mfma = [&](int i, int j, int set) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(b[set][j]), as_bf16x8(a[set][i]), acc[i][j], 0, 0, 0);
    };
    mm_clear<S>(acc);
    mm_pipeline<S, L>(p.K / 64u, fetch_one, read, mfma, [](unsigned int, unsigned int) {}, before_tail, MakeNothing{});
}

// The transposing LDS read (ds_read_b64_tr_b16) hands a lane four consecutive rows of its column: within 16
// lanes, lane r points at 8 bytes of row r / 4, columns 4 (r mod 4).. of a 4 x 16 block and receives column r
// of its four rows.  Eight rows of a lane's column as an MFMA operand, from two of them:
__device__ __forceinline__ u32x4 tn_fragment(const unsigned char* smem, unsigned int at, unsigned int row_bytes) {
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)RP_LDS_PTR(smem + at));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)RP_LDS_PTR(smem + at + 4u * row_bytes));
    return __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// A lane's place in such an operand: its row of the 4-row blocks, its row within a 16-deep step and its 8 bytes
// of a 32-wide tile.
struct TnLane {
    unsigned int rr, row, col;
    __device__ __forceinline__ explicit TnLane(unsigned int lane)
        : rr((lane >> 2) & 3u), row(8u * (lane >> 5) + rr), col(32u * ((lane >> 4) & 1u) + 8u * (lane & 3u)) {}
};
// Byte of a row where its 32-wide tile t begins.  A 32-lane pass of that read covers 64 bytes of four rows: rows
// that are a multiple of 256 bytes would have all four on the same banks, so their 64-byte groups are rotated by
// XOR with the row number (ROT); rows of 64 or 192 bytes need none.
template <bool ROT>
__device__ __forceinline__ unsigned int tn_tile_at(unsigned int t, unsigned int row) {
    return 64u * (ROT ? t ^ (row & 3u) : t);
}

// C[m][n] = sum_i A[i][m] B[i][n] over the rows k_base .. of the batch: both operands one row per
// experience.  Element v of a lane's accumulator is row acc_row(v, lane), column lane % 32.  Slices are 64 batch rows;
// of one that the batch ends in, the rows beyond it are overwritten with zeros in LDS.  Columns beyond an
// operand's last are read from its first (their outputs are not stored).
template <class S>
__device__ __forceinline__ void mm_tn(const GemmArgs& p, unsigned int m0, unsigned int n0, unsigned int k_base,
                                      unsigned char* smem, f32x16 (&acc)[S::TM][S::TN]) {
    constexpr int NW = S::NW;
    constexpr unsigned int ROWA = S::BM * 2u, ROWB = S::BN * 2u, CPA = S::BM / 8, CPB = S::BN / 8;
    constexpr int GA = 64 * (int)CPA / 64 / NW, GB = 64 * (int)CPB / 64 / NW, L = GA + GB;
    constexpr unsigned int A_BYTES = 64u * ROWA;
    static_assert(CPA % 16 == 0 && CPB % 16 == 0, "rows of whole 256 bytes");
    const unsigned int tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned int group = wave / (S::WGM * S::WGN), wi = wave % (S::WGM * S::WGN);
    const unsigned int wn = wi % S::WGN, wm = wi / S::WGN;
    const unsigned int rows = p.batch > k_base ? min(p.K, p.batch - k_base) : 0u;
    const unsigned int nk = (rows + 63u) / 64u, left = rows & 63u;
    unsigned int a_off[GA], b_off[GB], a_last[GA], b_last[GB];   // ... of the slice the batch ends in: its last row repeats
#pragma unroll
    for (int u = 0; u < GA; ++u) {
        const unsigned int at = (wave * GA + u) * 64u + lane, r = at / CPA, col = m0 + 8u * ((at % CPA) ^ (4u * (r & 3u)));
        const unsigned int c = (col < p.M ? col : 0u) * 2u;
        a_off[u] = r * p.lda * 2u + c;
        a_last[u] = (left ? min(r, left - 1u) : r) * p.lda * 2u + c;
    }
#pragma unroll
    for (int u = 0; u < GB; ++u) {
        const unsigned int at = (wave * GB + u) * 64u + lane, r = at / CPB, col = n0 + 8u * ((at % CPB) ^ (4u * (r & 3u)));
        const unsigned int c = (col < p.N ? col : 0u) * 2u;
        b_off[u] = r * p.ldb * 2u + c;
        b_last[u] = (left ? min(r, left - 1u) : r) * p.ldb * 2u + c;
    }
    auto fetch_one = [&](int u, unsigned int buf, unsigned int slice) {
        const bool last = slice + 1u == nk;
        unsigned char* dst = smem + buf * S::kStage + (u < GA ? (wave * GA + u) * 1024u : A_BYTES + (wave * GB + u - GA) * 1024u);
        const size_t row = (size_t)k_base + slice * 64u;
        if (u < GA)
            request_lds((gchar)reinterpret_cast<const char*>(p.A + row * p.lda), last ? a_last[u < GA ? u : 0] : a_off[u < GA ? u : 0], dst);
        else
            request_lds((gchar)reinterpret_cast<const char*>(p.Bt + row * p.ldb),
                        last ? b_last[u >= GA ? u - GA : 0] : b_off[u >= GA ? u - GA : 0], dst);
    };
    const TnLane l(lane);
    const unsigned int lrow = group * S::SP * 16u + l.row;
    unsigned int a_at[S::TM], b_at[S::TN];
#pragma unroll
    for (int i = 0; i < S::TM; ++i) a_at[i] = lrow * ROWA + tn_tile_at<true>(wm * S::TM + i, l.rr) + l.col;
#pragma unroll
    for (int j = 0; j < S::TN; ++j) b_at[j] = A_BYTES + lrow * ROWB + tn_tile_at<true>(wn * S::TN + j, l.rr) + l.col;
    u32x4 a[2][S::TM], b[2][S::TN];
    auto read = [&](unsigned int, unsigned int buf, int s, int set) {
#pragma unroll
        for (int j = 0; j < S::TN; ++j) b[set][j] = tn_fragment(smem, buf * S::kStage + b_at[j] + 16u * s * ROWB, ROWB);
#pragma unroll
        for (int i = 0; i < S::TM; ++i) a[set][i] = tn_fragment(smem, buf * S::kStage + a_at[i] + 16u * s * ROWA, ROWA);
    };
    auto mfma = [&](int i, int j, int set) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a[set][i]), as_bf16x8(b[set][j]), acc[i][j], 0, 0, 0);
    };
    auto arrived = [&](unsigned int slice, unsigned int buf) {
        if (!left || slice + 1u != nk) return;
        const u32x4 zero = {0u, 0u, 0u, 0u};
        u32x4* sa = reinterpret_cast<u32x4*>(smem + buf * S::kStage);
        u32x4* sb = reinterpret_cast<u32x4*>(smem + buf * S::kStage + A_BYTES);
        for (unsigned int e = left * CPA + tid; e < 64u * CPA; e += S::kThreads) sa[e] = zero;
        for (unsigned int e = left * CPB + tid; e < 64u * CPB; e += S::kThreads) sb[e] = zero;
        slice_barrier();
    };
    mm_clear<S>(acc);
    mm_pipeline<S, L>(nk, fetch_one, read, mfma, arrived, []() {}, MakeNothing{});
}

}  // namespace rp
