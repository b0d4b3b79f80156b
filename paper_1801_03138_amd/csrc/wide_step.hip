// Mixed-precision train step for wide networks, where the step is bound by the dense products:
// bf16 operands, fp32 accumulation on 32x32x16 MFMA, fp32 master weights and Adam moments.
//
// The forward products and the error of the first layer have the form C[m][n] = sum_k A[m][k] *
// Bt[n][k] with both operands stored K-contiguous, which is the form the MFMA lane layout reads
// with 16-byte loads; the forward layers therefore read transposed bf16 copies of the weights.  The
// weight gradients contract over the batch, C[m][n] = sum_i A[i][m] * B[i][n], and read activations
// and errors as the other kernels leave them, one row per experience: the transposing LDS
// read turns a slice of batch rows into MFMA operands.  These products have a long contraction and small
// outputs: they are split along the batch over several workgroups per tile, and the optimizer kernel adds
// the fp32 partial products up.
//
// What follows the second layer has two forms (WidePlan).  Large steps have two launches: output layer, TD
// errors and the second layer's error (head_kernel), then the first layer's error and all gradients
// (grad_back_kernel); small ones a launch for each of output layer, TD errors, first layer's error and gradients.
//
// Paper: Integration with Reinforcement Learning Algorithm (train step with no host inputs),
// Deep Q-Network Model (update equation).
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <type_traits>
#include <vector>

#include "gather_block.hpp"
#include "mm_bf16.hpp"
#include "replay_kernels.hpp"
#include "trainer.hpp"

namespace rp {
namespace {

constexpr unsigned int kGemmThreads = 256;

__device__ __forceinline__ float bits_to_float(bf16_bits b) {
    return __uint_as_float((unsigned int)b << 16);
}

// ----------------------------------------------------------------------------------------
// Optimizer applied to one parameter from inside a product's epilogue.
// ----------------------------------------------------------------------------------------
struct OptState {
    float *w, *g, *m, *v;
    unsigned int opt;
    float lr, beta1, beta2, eps;
    const TrainCounters* ctr;
    float* wt;                  // frozen target network, or null
    unsigned int sync_every;    // the target takes the new weights when Adam's t is a multiple of this
};

// What every update of one step shares: Adam's bias corrections 1 - beta^t and whether the
// target network is due for a sync (t was advanced earlier in the step).
struct OptStep {
    float c1, c2;
    bool sync;
};
__device__ __forceinline__ OptStep opt_step(const OptState& o) {
    OptStep s;
    s.c1 = o.ctr->c1;
    s.c2 = o.ctr->c2;
    s.sync = o.wt && o.sync_every && o.ctr->adam_t % o.sync_every == 0;
    return s;
}

__device__ __forceinline__ float opt_update(const OptState& o, size_t k, float gk, const OptStep& st) {
    float wk = o.w[k];
    o.g[k] = gk;
    if (o.opt == RP_SGD) {
        wk -= o.lr * gk;
    } else {
        const float mk = o.beta1 * o.m[k] + (1.f - o.beta1) * gk;
        const float vk = o.beta2 * o.v[k] + (1.f - o.beta2) * gk * gk;
        o.m[k] = mk;
        o.v[k] = vk;
        wk -= o.lr * (mk / st.c1) / (sqrtf(vk / st.c2) + o.eps);
    }
    o.w[k] = wk;
    if (st.sync) o.wt[k] = wk;
    return wk;
}

// ----------------------------------------------------------------------------------------
// Epilogues of the tiled product.
// bf16 output (gemm_nt_block; pre() also gets the first row of the workgroup's tile): the product
// is formed with the MFMA operands exchanged, so a lane holds four consecutive columns of one
// output row; it passes each value through pre(), rounds to bf16 and parks the wavefront's tile in
// LDS, from where it leaves in 16-byte pieces -- eight lanes write one 128-byte run of a row --
// through store().  The gradients' epilogues (gemm_tn_block) get the raw 32x32 accumulator tiles.
// ----------------------------------------------------------------------------------------
// out[m][n] = bf16(relu(acc + bias[n]))
struct EpiForward {
    const float* bias;
    const float* bias_hi;     // bias for rows from m_split on (the target network's)
    unsigned int m_split;
    bf16_bits* out;
    unsigned int ldo;
    unsigned int M, N;
    __device__ __forceinline__ float pre(unsigned int m0, unsigned int n, float x) const {
        x += (m0 >= m_split ? bias_hi : bias)[n < N ? n : 0u];
        return x > 0.f ? x : 0.f;
    }
    // eight consecutive columns n..n+7 of row m (N is a multiple of 8)
    __device__ __forceinline__ void store(unsigned int m, unsigned int n, const u32x4& v) const {
        if (m < M && n < N) *reinterpret_cast<u32x4*>(out + (size_t)m * ldo + n) = v;
    }
};

// Two bf16 values, each kept where the bf16 beside it in k is positive: non-zero with the sign bit clear (NaN
// counts as not).
__device__ __forceinline__ unsigned int relu_mask(unsigned int v, unsigned int k) {
    const unsigned int lo = k & 0xFFFFu, hi = k >> 16;
    const bool lo_on = lo != 0u && lo <= 0x7F80u, hi_on = hi != 0u && hi <= 0x7F80u;
    return (lo_on ? v & 0xFFFFu : 0u) | (hi_on ? v & 0xFFFF0000u : 0u);
}

// out[m][n] = bf16(acc) where mask[m][n] > 0, else 0  (the ReLU derivative; both [M x ld])
struct EpiMask {
    const bf16_bits* mask;
    bf16_bits* out;
    unsigned int ld;
    unsigned int M, N;
    __device__ __forceinline__ float pre(unsigned int, unsigned int, float x) const { return x; }
    // eight consecutive columns n..n+7 of row m (N is a multiple of 8)
    __device__ __forceinline__ void store(unsigned int m, unsigned int n, const u32x4& v) const {
        if (m >= M || n >= N) return;
        const size_t at = (size_t)m * ld + n;
        const u32x4 k = *reinterpret_cast<const u32x4*>(mask + at);
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = relu_mask(v[e], k[e]);
        *reinterpret_cast<u32x4*>(out + at) = o;
    }
};

// Partial gradients of one K split, added up by the optimizer kernel.  M: rows of the weight
// matrix (of its transpose in EpiFirst); sums() gets the 32 column (row) sums of an error tile.
// part[split][m][n] = acc, row M the bias
struct EpiSquare {
    float* part;
    unsigned int M, N;
    template <int TN>
    __device__ __forceinline__ void tiles(unsigned int mb, unsigned int nb, const f32x16 (&c)[TN],
                                          unsigned int lane, unsigned int split) const {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (mb >= M || nb + j * 32u >= N) continue;   // (M and N are whole numbers of 32)
            float* at = part + ((size_t)split * (M + 1u) + mb + acc_row(0, lane)) * N + nb + j * 32u + (lane & 31u);
#pragma unroll
            for (unsigned int v = 0; v < 16; ++v) at[acc_row(v, 0) * N] = c[j][v];
        }
    }
    // every row of the accumulator holds the 32 sums
    __device__ __forceinline__ void sums(unsigned int nb, const f32x16 (&c)[1], unsigned int lane, unsigned int split) const {
        const unsigned int n = nb + lane;
        if (lane < 32u && n < N) part[((size_t)split * (M + 1u) + M) * N + n] = c[0][0];
    }
};

// The output layer's, whose error operand comes in three bf16 parts (see dq_col): the three 32-wide
// column tiles of a 96-wide tile are added.
struct EpiOutput {
    float* part;
    unsigned int M, Ap;
    template <int TN>
    __device__ __forceinline__ void tiles(unsigned int mb, unsigned int nb, const f32x16 (&c)[TN],
                                          unsigned int lane, unsigned int split) const {
        static_assert(TN == 3, "a tile is the three parts of 32 actions");
        if (mb >= M) return;                              // (a whole number of 32)
        float* at = part + ((size_t)split * (M + 1u) + mb + acc_row(0, lane)) * Ap + nb / 3u + (lane & 31u);
#pragma unroll
        for (unsigned int v = 0; v < 16; ++v) at[acc_row(v, 0) * Ap] = (c[2][v] + c[1][v]) + c[0][v];
    }
    __device__ __forceinline__ void sums(unsigned int nb, const f32x16 (&c)[3], unsigned int lane, unsigned int split) const {
        if (lane < 32u)
            part[((size_t)split * (M + 1u) + M) * Ap + nb / 3u + lane] = (c[2][0] + c[1][0]) + c[0][0];
    }
};

// The first layer's, transposed: part[split][j][d], d < D, column D the bias.
struct EpiFirst {
    float* part;
    unsigned int M, D, Dx;
    template <int TN>
    __device__ __forceinline__ void tiles(unsigned int mb, unsigned int nb, const f32x16 (&c)[TN],
                                          unsigned int lane, unsigned int split) const {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const unsigned int d = nb + j * 32u + (lane & 31u);
            if (mb >= M || d >= D) continue;              // (M is a whole number of 32)
            float* at = part + ((size_t)split * M + mb + acc_row(0, lane)) * Dx + d;
#pragma unroll
            for (unsigned int v = 0; v < 16; ++v) at[acc_row(v, 0) * Dx] = c[j][v];
        }
    }
    // every column of the accumulator holds the 32 sums
    __device__ __forceinline__ void sums(unsigned int mb, const f32x16 (&c)[1], unsigned int lane, unsigned int split) const {
        if (mb >= M || (lane & 31u) != 0u) return;
        float* at = part + ((size_t)split * M + mb + acc_row(0, lane)) * Dx + D;
#pragma unroll
        for (unsigned int v = 0; v < 16; ++v) at[acc_row(v, 0) * Dx] = c[0][v];
    }
};

// ----------------------------------------------------------------------------------------
// Tiled product C = A Bt^T: a workgroup of four wavefronts owns a BM x BN tile and keeps the
// accumulators in registers; the wavefronts split the tile WGM x WGN ways.  BK-wide slices of
// both operands go from global memory straight into LDS (global_load_lds, 16 bytes per lane, no
// trip through registers), two slices deep: the next slice is in flight while the current one
// is multiplied.  Such a load writes the wavefront's 64 pieces to consecutive LDS addresses,
// so LDS rows cannot be padded; instead the 16-byte piece at position c of row r holds piece
// c ^ swz(r) of that row's slice (the lanes fetch their global pieces in that order), which
// spreads the MFMA operand reads of 16 consecutive rows over all banks.
// K must be a multiple of BK.  Loads of rows beyond M / N are redirected to the last valid row:
// such rows only feed accumulator rows / columns that the epilogue never stores.
// ----------------------------------------------------------------------------------------
template <int BM, int BN, int BK, int WGM, int WGN, int NSTAGE = 2>
constexpr size_t gemm_lds_bytes() {
    const size_t slices = NSTAGE * (size_t)(BM + BN) * BK * 2;
    // the epilogue parks every wavefront's bf16 tile, rows padded by 16 bytes
    const size_t parked = 4 * (size_t)(BM / WGM) * ((BN / WGN) * 2 + 16);
    return slices > parked ? slices : parked;
}

template <int BM, int BN, int BK, int WGM, int WGN, int NSTAGE = 2, class Epi>
__device__ __forceinline__ void gemm_nt_block(const GemmArgs& p, const Epi& epi, unsigned int block) {
    static_assert(WGM * WGN == 4, "four wavefronts");
    static_assert(NSTAGE >= 2, "slices in flight");
    static_assert(BK == 32 || BK == 64, "slice width");
    constexpr int RB = BK * 2;                             // bytes per LDS row
    constexpr int CPR = RB / 16;                           // 16-byte pieces per row
    constexpr int RPI = 64 / CPR;                          // rows one wavefront-wide load covers
    constexpr int A_BYTES = BM * RB, STAGE = (BM + BN) * RB;
    constexpr int GA = BM / RPI / 4, GB = BN / RPI / 4;    // loads per wavefront, slice and operand
    static_assert(GA >= 1 && GB >= 1 && BM % (4 * RPI) == 0 && BN % (4 * RPI) == 0, "loader shape");
    constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;  // 32x32 tiles per wavefront
    static_assert(TM >= 1 && TN >= 1, "wavefront shape");

    extern __shared__ uint4 gemm_smem[];
    unsigned char* smem = reinterpret_cast<unsigned char*>(gemm_smem);

    unsigned int m0, n0, split;
    if (!tile_of<BM, BN>(p, block, &m0, &n0, &split)) return;

    const unsigned int tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const unsigned int wn = wave % WGN, wm = wave / WGN;
    // LDS has 64 four-byte banks: 16 lanes' 16-byte reads are conflict-free when they fall into 16
    // different slots of a 256-byte span.  256 / RB rows share such a span; successive groups of
    // that many rows get their pieces rotated by XOR with the group number.
    auto swz = [](unsigned int r) { return (r / (256u / RB)) & (CPR - 1u); };

    // loader: wavefront w moves row groups w*GA.. of A and w*GB.. of B; a lane's piece lands at
    // LDS position `lane` of the group, so the lane fetches the piece that belongs there
    // A request's address is a wavefront-uniform base (the tile's first row of the operand, advanced
    // by the slice's column: 64-bit, in scalar registers) plus a per-lane byte offset that never
    // changes (one 32-bit register per request, at most a tile's rows long, however large the
    // operand is), and its LDS destination is uniform as well: issuing a request then costs two
    // scalar instructions and the load itself, no vector arithmetic.
    const unsigned int lr = lane / CPR, lc = lane % CPR;
    const unsigned int wave_u = __builtin_amdgcn_readfirstlane(wave);
    unsigned int a_off[GA], b_off[GB];
#pragma unroll
    for (int u = 0; u < GA; ++u) {
        const unsigned int r = (wave * GA + u) * RPI + lr;
        a_off[u] = (min(r, p.M - 1u - m0) * p.lda + (lc ^ swz(r)) * 8u) * 2u;
    }
#pragma unroll
    for (int u = 0; u < GB; ++u) {
        const unsigned int r = (wave * GB + u) * RPI + lr;
        b_off[u] = (min(r, p.N - 1u - n0) * p.ldb + (lc ^ swz(r)) * 8u) * 2u;
    }
    typedef const __attribute__((address_space(1))) char* gchar;
    const gchar a_base = (gchar)reinterpret_cast<const char*>(p.A + (size_t)m0 * p.lda);
    const gchar b_base = (gchar)reinterpret_cast<const char*>((m0 >= p.m_split ? p.Bt_hi : p.Bt) + (size_t)n0 * p.ldb);
    // request u (0 .. GA + GB - 1) of a slice: one wavefront-wide 16-byte-per-lane load into LDS
    constexpr int L = GA + GB;                              // loads per wavefront and slice
    auto fetch_one = [&](int u, unsigned int buf, unsigned int k0) {
        gchar row = (u < GA ? a_base : b_base) + (size_t)k0 * 2u;
        const unsigned int off = u < GA ? a_off[u < GA ? u : 0] : b_off[u >= GA ? u - GA : 0];
        unsigned char* dst = smem + buf * STAGE + (u < GA ? (wave_u * GA + u) * 1024u : A_BYTES + (wave_u * GB + u - GA) * 1024u);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(row + off), RP_LDS_PTR(dst), 16, 0, 0);
    };
    auto fetch = [&](unsigned int buf, unsigned int k0) {
#pragma unroll
        for (int u = 0; u < L; ++u) fetch_one(u, buf, k0);
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const unsigned int a_row = (wm * TM * 32u + (lane & 31u)) * RB;
    const unsigned int b_row = (wn * TN * 32u + (lane & 31u)) * RB;
    const unsigned int sw = swz(lane & 31u), half = lane >> 5;
    // One slice's multiply.  A wavefront issues in order, and it is alone on its SIMD when the
    // workgroup has the compute unit to itself, so everything that has to happen during a
    // slice is interleaved with its MFMAs by hand: the LDS reads of step s + 1 are issued before
    // the MFMAs of step s (two sets of fragment registers), and the global -> LDS requests of a
    // later slice (FETCH) are spread out between the MFMAs, one at a time, instead of being
    // issued in a burst during which no MFMA could start.  The scheduling barriers keep the
    // compiler from regrouping them.
    auto multiply = [&](unsigned int buf, auto fetch_flag, unsigned int fbuf, unsigned int fk0) {
        constexpr bool FETCH = decltype(fetch_flag)::value;
        const unsigned char* as = smem + buf * STAGE + a_row;
        const unsigned char* bs = smem + buf * STAGE + A_BYTES + b_row;
        constexpr int STEPS = BK / 16, NM = STEPS * TM * TN;
        u32x4 a[2][TM], b[2][TN];
        auto request = [&](int s, int set) {
            const unsigned int ko = ((2u * s + half) ^ sw) * 16u;   // where this 16-deep step's piece sits
#pragma unroll
            for (int i = 0; i < TM; ++i) a[set][i] = *reinterpret_cast<const u32x4*>(as + i * 32 * RB + ko);
#pragma unroll
            for (int j = 0; j < TN; ++j) b[set][j] = *reinterpret_cast<const u32x4*>(bs + j * 32 * RB + ko);
        };
        request(0, 0);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            if (s + 1 < STEPS) request(s + 1, (s + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(b[s & 1][j]), as_bf16x8(a[s & 1][i]), acc[i][j], 0, 0, 0);
                    if (FETCH) {
                        const int m = (s * TM + i) * TN + j;          // this MFMA's number within the slice
#pragma unroll
                        for (int u = m * L / NM; u < (m + 1) * L / NM; ++u) fetch_one(u, fbuf, fk0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // NSTAGE slices deep: slice kt is awaited (every wavefront waits for its own loads, the barrier
    // covers the others'); after the barrier nobody reads the buffer of slice kt - 1 any more, so
    // slice kt + NSTAGE - 1 is requested into it and travels while slices kt .. are multiplied.
    // With two workgroups on a compute unit two slices are enough (the other workgroup computes
    // while this one waits); a workgroup that has a compute unit to itself needs its requests
    // further ahead than one slice's multiply time.
    const unsigned int nk = p.K / BK;
#pragma unroll
    for (unsigned int s0 = 0; s0 + 1 < (unsigned int)NSTAGE; ++s0)
        if (s0 < nk) fetch(s0, s0 * BK);
    // steady state: slices kt + 1 .. kt + NSTAGE - 2 may still be in flight while slice kt is awaited
    // (two loops, so that each has one straight-line body: with both kinds of multiply in one loop
    // the compiler moved all accumulators between register files on every iteration)
    unsigned int kt = 0;
    for (; kt + NSTAGE - 1 < nk; ++kt) {
        wait_loads<(NSTAGE - 2) * L>();
        __syncthreads();
        multiply(kt % NSTAGE, std::true_type{}, (kt + NSTAGE - 1) % NSTAGE, (kt + NSTAGE - 1) * BK);
    }
    // the last NSTAGE - 1 slices: nothing left to request
    for (; kt < nk; ++kt) {
        wait_slices<L, NSTAGE - 2>(nk - 1u - kt);
        __syncthreads();
        multiply(kt % NSTAGE, std::false_type{}, 0u, 0u);
    }

    // The accumulator of tile (i, j) is transposed: element v of a lane is output row
    // lane % 32, column acc_row(v, lane).  Park the wavefront's (TM*32) x (TN*32) tile as
    // bf16 in its own LDS region (the operand slices are no longer needed).
    constexpr int TSTRIDE = TN * 64 + 16;                // bytes per parked row
    constexpr int CR = TN * 4;                           // 16-byte pieces per row
    constexpr int RP = 64 / CR;                          // rows per pass of the wavefront
    static_assert(4 * TM * 32 * TSTRIDE <= (int)gemm_lds_bytes<BM, BN, BK, WGM, WGN, NSTAGE>(), "parked tiles fit");
    __syncthreads();
    unsigned char* park = smem + wave * (TM * 32 * TSTRIDE);
    const unsigned int wm0 = m0 + wm * TM * 32u, wn0 = n0 + wn * TN * 32u;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (unsigned int grp = 0; grp < 4; ++grp) {
                const unsigned int nl = j * 32u + 8u * grp + 4u * (lane >> 5);
                float x[4];
#pragma unroll
                for (unsigned int e = 0; e < 4; ++e) x[e] = epi.pre(m0, wn0 + nl + e, acc[i][j][4 * grp + e]);
                uint2 pk;
                pk.x = bf16_pair(x[0], x[1]);
                pk.y = bf16_pair(x[2], x[3]);
                *reinterpret_cast<uint2*>(park + (i * 32u + (lane & 31u)) * TSTRIDE + nl * 2u) = pk;
            }
    // same wavefront reads what it wrote: LDS operations of a wavefront complete in order
#pragma unroll
    for (int pass = 0; pass < TM * 32 / RP; ++pass) {
        const unsigned int row = pass * RP + lane / CR, piece = lane % CR;
        const u32x4 v = *reinterpret_cast<const u32x4*>(park + row * TSTRIDE + piece * 16u);
        epi.store(wm0 + row, wn0 + piece * 8u, v);
    }
}

// ----------------------------------------------------------------------------------------
// Tiled product over the batch, C[m][n] = sum_i A[i][m] * B[i][n]: both operands as the other kernels
// leave them, one row per experience, no transposed copies in memory.  A slice is 64 batch rows of
// the workgroup's BM and BN columns; it goes straight into LDS as in gemm_nt_block, and the
// transposing LDS read (ds_read_b64_tr_b16) hands a lane four consecutive batch rows of its column:
// within 16 lanes, lane r points at 8 bytes of row r / 4, columns 4 (r mod 4).. of a 4 x 16 block and
// receives column r of its four rows.  A 32-lane pass of that read covers 64 bytes of four rows: a row
// of 64 bytes, or of 192, puts those on different banks by itself, in rows of 256 bytes the
// 64-byte groups are rotated by XOR with the row number (the lanes fetch their global pieces in
// that order).  The contraction ends at row `batch`: of a slice that it ends in, the rows beyond are
// overwritten with zeros in LDS, and slices beyond are left out.
//
// A workgroup is eight wavefronts, two groups of four: both groups cover the whole tile, each for half
// of a slice's steps, and add their accumulators through LDS at the end.  The square layer's tiles
// have a compute unit to themselves, and with one wavefront per SIMD the transposing reads (twice
// the instructions of the 16-byte ones), the MFMAs and the requests hardly overlap.  (These choices were
// measured at batch 4096 and 1024 units, which take grad_back_kernel now: 23.9 us per launch with one group, 21.8 with
// two; deeper pipelines, four slices of 64 or 32 rows, 23.8, 24.4; two workgroups per compute unit 23.2.)
//
// Transposed copies of H1, H2 and both errors, with a row of ones for the biases, cost the launches that would
// write them more than they save here: batch 512, 512 units 49.1 us per step, 45.1 without.
//
// The bias gradients are sums over one operand's columns: the workgroups of the first tile row
// (SUM_ROWS: of the first tile column) multiply the fragments of B (of A) that they hold anyway
// with a register of ones, one more MFMA a wavefront and 16 rows (three for the three-part tile).
// ----------------------------------------------------------------------------------------
constexpr int kTnSlice = 64, kTnStages = 2;   // batch rows of a slice, slices in LDS

template <int BM, int BN>
constexpr size_t gemm_tn_lds_bytes() {
    // the slices, or the second group's accumulators and its sums
    return std::max(kTnStages * (size_t)kTnSlice * (BM + BN) * 2, (size_t)BM * BN * 4 + 4 * 4096);
}
constexpr unsigned int kTnThreads = 512;

template <int BM, int BN, int WGM, int WGN, bool SUM_ROWS, class Epi>
__device__ __forceinline__ void gemm_tn_block(const GemmArgs& p, const Epi& epi, unsigned int block) {
    unsigned int m0, n0, split;
    if (!tile_of<BM, BN>(p, block, &m0, &n0, &split)) return;
    const bool with_sums = (SUM_ROWS ? n0 : m0) == 0u;
    static_assert(WGM * WGN == 4, "four wavefronts a group");
    constexpr int ROWA = BM * 2, ROWB = BN * 2;            // bytes per LDS row
    constexpr int CPA = BM / 8, CPB = BN / 8;              // 16-byte pieces per row
    constexpr unsigned int A_BYTES = kTnSlice * ROWA, STAGE = kTnSlice * (ROWA + ROWB);
    // loads per slice, and per wavefront (where they do not divide evenly, some are made twice: every
    // wavefront then counts the same number in flight)
    constexpr int NA = kTnSlice * CPA / 64, NB = kTnSlice * CPB / 64;
    constexpr int GA = (NA + 7) / 8, GB = (NB + 7) / 8, L = GA + GB;
    constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;  // 32x32 tiles per wavefront
    static_assert(TM >= 1 && TN >= 1, "wavefront shape");
    // sums a wavefront forms: all three parts of a three-part tile, else one tile's, each wavefront another
    constexpr int NS = TN == 3 ? 3 : 1;
    static_assert(SUM_ROWS ? WGN >= TM && NS == 1 : (NS == 3 || WGM >= TN), "every tile's sums have a wavefront");

    extern __shared__ uint4 gemm_smem[];
    unsigned char* smem = reinterpret_cast<unsigned char*>(gemm_smem);
    const unsigned int tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const unsigned int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const unsigned int group = wave_u >> 2, wn = (wave_u & 3u) % WGN, wm = (wave_u & 3u) / WGN;
    const unsigned int k_base = split * p.K;

    // loader: the slice's pieces in LDS order, 64 a request.  Columns past the operand are redirected
    // to its first: such columns only feed accumulator elements that the epilogue never stores.
    auto a_load = [&](int u) { return min(wave_u * GA + u, (unsigned int)NA - 1u); };
    auto b_load = [&](int u) { return min(wave_u * GB + u, (unsigned int)NB - 1u); };
    unsigned int a_off[GA], b_off[GB];
#pragma unroll
    for (int u = 0; u < GA; ++u) {
        const unsigned int at = a_load(u) * 64u + lane, r = at / CPA;
        const unsigned int col = m0 + 8u * ((at % CPA) ^ (CPA == 16 ? 4u * (r & 3u) : 0u));
        a_off[u] = (r * p.lda + (col < p.M ? col : 0u)) * 2u;
    }
#pragma unroll
    for (int u = 0; u < GB; ++u) {
        const unsigned int at = b_load(u) * 64u + lane, r = at / CPB;
        const unsigned int col = n0 + 8u * ((at % CPB) ^ (CPB == 16 ? 4u * (r & 3u) : 0u));
        b_off[u] = (r * p.ldb + (col < p.N ? col : 0u)) * 2u;
    }
    // request u of the slice at row k: the slice's first row is kept in scalar registers (the empty asm
    // pins it there), the lane adds its 32-bit offset
    typedef const __attribute__((address_space(1))) char* gchar;
    auto request_at = [&](int u, unsigned int buf, gchar row, unsigned int off) {
        unsigned char* dst = smem + buf * STAGE + (u < GA ? a_load(u) * 1024u : A_BYTES + b_load(u - GA) * 1024u);
        asm volatile("" : "+s"(row));
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(row + off), RP_LDS_PTR(dst), 16, 0, 0);
    };
    auto fetch_one = [&](int u, unsigned int buf, unsigned int k) {
        if (u < GA) request_at(u, buf, (gchar)reinterpret_cast<const char*>(p.A + (size_t)k * p.lda), a_off[u < GA ? u : 0]);
        else request_at(u, buf, (gchar)reinterpret_cast<const char*>(p.Bt + (size_t)k * p.ldb), b_off[u >= GA ? u - GA : 0]);
    };

    f32x16 acc[TM][TN], sum[NS];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j][v] = 0.f;
#pragma unroll
        for (int j = 0; j < NS; ++j) sum[j][v] = 0.f;
    }
    const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};

    // where a lane reads in a slice: its row of the 4 x 16 blocks (batch rows 8 (lane / 32) + 0..3 of a
    // 16-deep step, 4..7 with the second read) and its 8 bytes of a 32-wide tile
    constexpr int STEPS = kTnSlice / 32;                   // 16-deep steps a group takes of a slice
    const unsigned int rr = (lane >> 2) & 3u, lrow = group * STEPS * 16u + 8u * (lane >> 5) + rr;
    const unsigned int lcol = 32u * ((lane >> 4) & 1u) + 8u * (lane & 3u);
    unsigned int a_at[TM], b_at[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const unsigned int t = wm * TM + i;
        a_at[i] = lrow * ROWA + 64u * (CPA == 16 ? t ^ rr : t) + lcol;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const unsigned int t = wn * TN + j;
        b_at[j] = A_BYTES + lrow * ROWB + 64u * (CPB == 16 ? t ^ rr : t) + lcol;
    }
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    auto fragment = [&](unsigned int at, unsigned int row_bytes) {   // batch rows 0..3 and 4..7 of the lane's eight
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)RP_LDS_PTR(smem + at));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)RP_LDS_PTR(smem + at + 4u * row_bytes));
        return __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // one slice's multiply, with the next one's requests between the MFMAs (as in gemm_nt_block)
    auto multiply = [&](unsigned int buf, auto fetch_flag, unsigned int fbuf, unsigned int fk0) {
        constexpr bool FETCH = decltype(fetch_flag)::value;
        constexpr int NM = STEPS * TM * TN;
        u32x4 a[2][TM], b[2][TN];
        auto request = [&](int s, int set) {
#pragma unroll
            for (int i = 0; i < TM; ++i) a[set][i] = fragment(buf * STAGE + a_at[i] + 16u * s * ROWA, ROWA);
#pragma unroll
            for (int j = 0; j < TN; ++j) b[set][j] = fragment(buf * STAGE + b_at[j] + 16u * s * ROWB, ROWB);
        };
        request(0, 0);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            if (s + 1 < STEPS) request(s + 1, (s + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            if (with_sums) {
#pragma unroll
                for (int j = 0; j < NS; ++j) {
                    if constexpr (SUM_ROWS) {
                        const u32x4 x = TM > 1 && wn ? a[s & 1][TM - 1] : a[s & 1][0];
                        sum[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(x), as_bf16x8(ones), sum[j], 0, 0, 0);
                    } else {
                        const u32x4 x = NS == 3 ? b[s & 1][j] : TN > 1 && wm ? b[s & 1][TN - 1] : b[s & 1][0];
                        sum[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ones), as_bf16x8(x), sum[j], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a[s & 1][i]), as_bf16x8(b[s & 1][j]), acc[i][j], 0, 0, 0);
                    if (FETCH) {
                        const int m = (s * TM + i) * TN + j;
#pragma unroll
                        for (int u = m * L / NM; u < (m + 1) * L / NM; ++u) fetch_one(u, fbuf, fk0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // (the pipeline of gemm_nt_block)  The last slice may end with the operands' rows: its requests
    // beyond them fetch the last row, and what they brought is overwritten with zeros.
    const unsigned int rows = p.batch > k_base ? min(p.K, p.batch - k_base) : 0u;
    const unsigned int nk = (rows + kTnSlice - 1u) / kTnSlice, left = rows % kTnSlice;
    auto last_offsets = [&]() {                              // before that slice's requests
#pragma unroll
        for (int u = 0; u < GA; ++u) {
            const unsigned int r = (a_load(u) * 64u + lane) / CPA;
            a_off[u] -= r < left ? 0u : (r - (left - 1u)) * p.lda * 2u;
        }
#pragma unroll
        for (int u = 0; u < GB; ++u) {
            const unsigned int r = (b_load(u) * 64u + lane) / CPB;
            b_off[u] -= r < left ? 0u : (r - (left - 1u)) * p.ldb * 2u;
        }
    };
#pragma unroll
    for (unsigned int s0 = 0; s0 + 1 < (unsigned int)kTnStages; ++s0)
        if (s0 < nk) {
            if (left && s0 + 1u == nk) last_offsets();
#pragma unroll
            for (int u = 0; u < L; ++u) fetch_one(u, s0, k_base + s0 * kTnSlice);
        }
    unsigned int kt = 0;
    for (; kt + kTnStages - 1 < nk; ++kt) {
        if (left && kt + kTnStages == nk) last_offsets();
        wait_loads<(kTnStages - 2) * L>();
        __syncthreads();
        multiply(kt % kTnStages, std::true_type{}, (kt + kTnStages - 1) % kTnStages, k_base + (kt + kTnStages - 1) * kTnSlice);
    }
    for (; kt < nk; ++kt) {
        wait_slices<L, kTnStages - 2>(nk - 1u - kt);
        __syncthreads();
        if (left && kt + 1u == nk) {
            const u32x4 zero = {0u, 0u, 0u, 0u};
            u32x4* sa = reinterpret_cast<u32x4*>(smem + (kt % kTnStages) * STAGE);
            u32x4* sb = reinterpret_cast<u32x4*>(smem + (kt % kTnStages) * STAGE + A_BYTES);
            for (unsigned int e = left * CPA + tid; e < (unsigned int)kTnSlice * CPA; e += kTnThreads) sa[e] = zero;
            for (unsigned int e = left * CPB + tid; e < (unsigned int)kTnSlice * CPB; e += kTnThreads) sb[e] = zero;
            __syncthreads();
        }
        multiply(kt % kTnStages, std::false_type{}, 0u, 0u);
    }

    // the second group hands its accumulators and sums to the first
    __syncthreads();
    f32x4* const give = reinterpret_cast<f32x4*>(smem) + (wave_u & 3u) * (TM * TN * 256u) + lane;
    f32x4* const give_sums = reinterpret_cast<f32x4*>(smem + (size_t)BM * BN * 4) + (wave_u & 3u) * 256u + lane;
    if (group) {
#pragma unroll
        for (int q = 0; q < TM * TN * 4; ++q) {
            const f32x16& c = acc[q / 4 / TN][q / 4 % TN];
            give[q * 64] = f32x4{c[q % 4 * 4], c[q % 4 * 4 + 1], c[q % 4 * 4 + 2], c[q % 4 * 4 + 3]};
        }
        if (with_sums) {
            // (a column sum is in every row: one element is enough)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                give_sums[q * 64] = SUM_ROWS ? f32x4{sum[0][q * 4], sum[0][q * 4 + 1], sum[0][q * 4 + 2], sum[0][q * 4 + 3]}
                                             : f32x4{sum[0][0], sum[NS > 1 ? 1 : 0][0], sum[NS > 2 ? 2 : 0][0], 0.f};
        }
    }
    __syncthreads();
    if (group) return;
#pragma unroll
    for (int q = 0; q < TM * TN * 4; ++q) {
        const f32x4 x = give[q * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[q / 4 / TN][q / 4 % TN][q % 4 * 4 + e] += x[e];
    }
    if (with_sums) {
#pragma unroll
        for (int q = 0; q < (SUM_ROWS ? 4 : 1); ++q) {
            const f32x4 x = give_sums[q * 64];
            if constexpr (SUM_ROWS) {
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[0][q * 4 + e] += x[e];
            } else {
#pragma unroll
                for (int e = 0; e < NS; ++e) sum[e][0] += x[e];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) epi.tiles(m0 + (wm * TM + i) * 32u, n0 + wn * TN * 32u, acc[i], lane, split);
    if (with_sums) {
        // (of the wavefronts that formed the same sums one stores them)
        if constexpr (SUM_ROWS) {
            if (wn < TM) epi.sums(m0 + (wm * TM + wn) * 32u, sum, lane, split);
        } else if constexpr (NS == 3) {
            if (wm == 0) epi.sums(n0, sum, lane, split);
        } else {
            if (wm < TN) epi.sums(n0 + (wn * TN + wm) * 32u, sum, lane, split);
        }
    }
}

template <int BM, int BN, int BK, int WGM, int WGN, int NSTAGE, class Epi>
__global__ __launch_bounds__(kGemmThreads) void gemm_nt_kernel(GemmArgs p, Epi epi) {
    gemm_nt_block<BM, BN, BK, WGM, WGN, NSTAGE>(p, epi, blockIdx.x);
}

// The three weight-gradient products of a step in one launch (each writes K-split partials):
// workgroups [0, n2) take the square layer's, [n2, n2 + n3) the output layer's, the rest the
// first layer's.  n2 and n3 are multiples of 8, which keeps a workgroup's index within its
// product congruent to its XCD.  The output layer's tiles are the three parts of 32 actions wide;
// NARROW1: the states are at most 32 wide and the first layer's gradient uses the matching tile.
template <bool NARROW1>
__global__ __launch_bounds__(kTnThreads) void grad_products_kernel(GemmArgs p2, EpiSquare e2, unsigned int n2,
                                                                     GemmArgs p3, EpiOutput e3, unsigned int n3,
                                                                     GemmArgs p1, EpiFirst e1) {
    const unsigned int b = blockIdx.x;
    if (b < n2) {
        gemm_tn_block<128, 128, 2, 2, false>(p2, e2, b);
    } else if (b < n2 + n3) {
        gemm_tn_block<128, 96, 4, 1, false>(p3, e3, b - n2);
    } else {
        if constexpr (NARROW1) gemm_tn_block<128, 32, 4, 1, true>(p1, e1, b - n2 - n3);
        else gemm_tn_block<128, 128, 2, 2, true>(p1, e1, b - n2 - n3);
    }
}

// The dynamic LDS size of each kernel is announced per kernel before the first launch (at trainer creation, outside any
// stream capture): up to 80 KB here (the gradients' launch), 144 KB in grad_back_kernel, 160 KB in forward_kernel.
template <int BM, int BN, int BK, int WGM, int WGN, class Epi, int NSTAGE = 2>
hipError_t configure_gemm() {
    auto kernel = gemm_nt_kernel<BM, BN, BK, WGM, WGN, NSTAGE, Epi>;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)gemm_lds_bytes<BM, BN, BK, WGM, WGN, NSTAGE>());
}

template <bool NARROW1>
hipError_t configure_grad_products() {
    auto kernel = grad_products_kernel<NARROW1>;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)gemm_tn_lds_bytes<128, 128>());
}

// Arguments and workgroup count (a multiple of 8) of one product with BM x BN tiles and BK-wide
// slices; false when the shape does not fit the kernel's assumptions.
template <int BM, int BN, int BK>
bool gemm_args(const bf16_bits* A, unsigned int lda, const bf16_bits* Bt, unsigned int ldb,
               unsigned int M, unsigned int N, unsigned int K, unsigned int splits,
               const bf16_bits* Bt_hi, unsigned int m_split, GemmArgs* a, unsigned int* blocks) {
    if (K == 0 || splits == 0 || K % (splits * BK) != 0 || lda % 8 != 0 || ldb % 8 != 0 || M == 0 || N == 0)
        return false;
    if (Bt_hi && m_split % BM != 0) return false;   // a tile takes one B operand
    a->A = A; a->lda = lda; a->Bt = Bt; a->ldb = ldb; a->M = M; a->N = N; a->K = K / splits;
    a->Bt_hi = Bt_hi ? Bt_hi : Bt;
    a->m_split = Bt_hi ? m_split : 0xFFFFFFFFu;
    a->tiles_m = (M + BM - 1) / BM;
    a->tiles_n = (N + BN - 1) / BN;
    a->splits = splits;
    a->batch = 0;
    const unsigned int n_tiles = a->tiles_m * a->tiles_n * splits;
    *blocks = 8u * ((n_tiles + 7u) / 8u);
    // band width: the one for which an XCD's share of the tiles (a block of about per_xcd / band
    // tile rows by `band` tile columns) touches the fewest operand rows
    const unsigned int per_xcd = std::min((n_tiles + 7u) / 8u, a->tiles_m * a->tiles_n);
    unsigned int best = a->tiles_n;
    size_t best_cost = ~(size_t)0;
    // (first among the widths whose bands line up with the XCDs' ranges, so that a range does not
    // straddle two bands; any width if there is none)
    for (int aligned = 1; aligned >= 0 && best_cost == ~(size_t)0; --aligned)
        for (unsigned int w = 1; w <= a->tiles_n; ++w) {
            const unsigned int band_tiles = a->tiles_m * w;
            if (aligned && band_tiles % per_xcd != 0 && per_xcd % band_tiles != 0) continue;
            // a range of per_xcd tile numbers covers whole bands when it is longer than one
            const unsigned int rows = per_xcd >= band_tiles ? a->tiles_m : std::min(a->tiles_m, (per_xcd + w - 1) / w);
            const unsigned int cols = per_xcd >= band_tiles
                                          ? std::min(a->tiles_n, w * ((per_xcd + band_tiles - 1) / band_tiles))
                                          : w;
            const size_t cost = (size_t)rows * BM + (size_t)cols * BN;
            if (cost < best_cost) {
                best_cost = cost;
                best = w;
            }
        }
    a->band = best;
    return true;
}

template <int BM, int BN, int BK, int WGM, int WGN, int NSTAGE = 2, class Epi>
hipError_t launch_gemm(hipStream_t st, const bf16_bits* A, unsigned int lda, const bf16_bits* Bt,
                       unsigned int ldb, unsigned int M, unsigned int N, unsigned int K,
                       const Epi& epi, unsigned int splits = 1, const bf16_bits* Bt_hi = nullptr,
                       unsigned int m_split = 0xFFFFFFFFu) {
    GemmArgs a;
    unsigned int blocks;
    if (!gemm_args<BM, BN, BK>(A, lda, Bt, ldb, M, N, K, splits, Bt_hi, m_split, &a, &blocks))
        return hipErrorInvalidValue;
    constexpr size_t lds = gemm_lds_bytes<BM, BN, BK, WGM, WGN, NSTAGE>();
    hipLaunchKernelGGL((gemm_nt_kernel<BM, BN, BK, WGM, WGN, NSTAGE, Epi>), dim3(blocks),
                       dim3(kGemmThreads), lds, st, a, epi);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------------------
// Product with few output tiles: the output layer, Q = H2 W3 + b3 (a few 32-wide column tiles, many
// rows), and others on small batches (few_tiles):
// one tile of 16 MT x 32 outputs per workgroup; the eight wavefronts split K, each loading its MFMA operands
// straight from global memory (four 32-deep steps requested before the first multiply), and
// add their accumulators through LDS.  K and N are multiples of 32.  Rows beyond M repeat the last one and are not
// stored.  What such a launch costs beyond its start is its loads: a wavefront's of 16 rows touches 16 runs of 64 bytes,
// where one of 32 rows (32x32x16 MFMA, tiles of 32 x 32) touched 32 of 32 bytes.  32 x 32 tiles of that kind -> this:
// output layer 1024 x 32 x 1024 6.6 -> 5.0 us, first layer's error 512 x 128 x 1024 7.0 -> 5.1; us per step, 27-128-1024-30
// at batch 512 42.9 -> 38.7, 1024-1024 at 64 43.3 -> 38.0, at 512 57.0 -> 53.9, 64-64 at 80 24.9 -> 23.6.
// ----------------------------------------------------------------------------------------
struct SkinnyArgs {
    const bf16_bits* A;
    unsigned int lda;
    const bf16_bits* Bt;
    unsigned int ldb;
    unsigned int M, N, K;
    // tiles whose first row is m_split (a multiple of 32) or beyond use these (the target network's)
    const bf16_bits* Bt_hi;
    unsigned int m_split;
};

// out[m][n] = acc + bias[n], fp32
struct SkinnyBias {
    const float* bias;   // [N]
    const float* bias_hi;
    unsigned int m_split;
    float* out;          // [M x ldo]
    unsigned int ldo;
    __device__ __forceinline__ void store(unsigned int m, unsigned int n, float x) const {
        out[(size_t)m * ldo + n] = x + (m >= m_split ? bias_hi : bias)[n];
    }
};

// out[m][n] = bf16(relu(acc + bias[n]))
struct SkinnyRelu {
    const float* bias;   // [N]
    const float* bias_hi;
    unsigned int m_split;
    bf16_bits* out;      // [M x ldo]
    unsigned int ldo;
    __device__ __forceinline__ void store(unsigned int m, unsigned int n, float x) const {
        x += (m >= m_split ? bias_hi : bias)[n];
        out[(size_t)m * ldo + n] = bf16_bits_rne(x > 0.f ? x : 0.f);
    }
};

// out[m][n] = bf16(acc) where mask[m][n] > 0, else 0  (both [M x ld])
struct SkinnyMask {
    const bf16_bits* mask;
    bf16_bits* out;
    unsigned int ld;
    __device__ __forceinline__ void store(unsigned int m, unsigned int n, float x) const {
        const size_t at = (size_t)m * ld + n;
        out[at] = bits_to_float(mask[at]) > 0.f ? bf16_bits_rne(x) : (bf16_bits)0;
    }
};

template <int MT, class Epi>
__global__ __launch_bounds__(512) void skinny_nt_kernel(SkinnyArgs p, Epi epi) {
    constexpr unsigned int NW = 8, LD = 36;
    __shared__ float red[NW][16 * MT][LD];
    const unsigned int tid = threadIdx.x, lane = tid & 63u, r16 = lane & 15u, q16 = lane >> 4;
    const unsigned int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned int m0 = blockIdx.x * (16u * MT), n0 = blockIdx.y * 32u;
    const bf16_bits* ap[MT];
#pragma unroll
    for (unsigned int i = 0; i < MT; ++i) ap[i] = p.A + (size_t)min(m0 + 16u * i + r16, p.M - 1u) * p.lda + 8u * q16;
    const bool hi = m0 >= p.m_split;
    const bf16_bits* bp = (hi ? p.Bt_hi : p.Bt) + (size_t)(n0 + r16) * p.ldb + 8u * q16;
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    f32x4 acc[MT][2];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (unsigned int kc = wave * 128u; kc < p.K; kc += NW * 128u) {
        u32x4 a[MT][4], b[2][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const unsigned int k = kc + s * 32u;
            const bool in = k < p.K;
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i][s] = in ? *reinterpret_cast<const u32x4*>(ap[i] + k) : zero4;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                b[j][s] = in ? *reinterpret_cast<const u32x4*>(bp + (size_t)(16u * j) * p.ldb + k) : zero4;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a[i][s]), as_bf16x8(b[j][s]), acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][16u * i + 4u * q16 + v][16u * j + r16] = acc[i][j][v];
    __syncthreads();
#pragma unroll
    for (unsigned int i = 0; i < MT; ++i) {
        const unsigned int r = 16u * i + (tid >> 5), c = tid & 31u;
        float s = 0.f;
#pragma unroll
        for (unsigned int w = 0; w < NW; ++w) s += red[w][r][c];
        if (m0 + r < p.M) epi.store(m0 + r, n0 + c, s);
    }
}

// 16 rows a tile while that leaves no more tiles than two a compute unit, 32 beyond (16 rows fetch the B operand twice
// as often: 64-512-512-64 at batch 500 41.3 us per step, 39.2 with 32; 1024-1024 at 256 49.7, 46.5).
template <class Epi>
hipError_t launch_skinny(hipStream_t st, const SkinnyArgs& a, const Epi& epi) {
    const dim3 g16((a.M + 15) / 16, a.N / 32), g32((a.M + 31) / 32, a.N / 32);
    if ((size_t)g16.x * g16.y <= 512u) hipLaunchKernelGGL((skinny_nt_kernel<1, Epi>), g16, dim3(512), 0, st, a, epi);
    else hipLaunchKernelGGL((skinny_nt_kernel<2, Epi>), g32, dim3(512), 0, st, a, epi);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------------------
// The first two layers of large steps in one launch: H2 = relu(relu(X W1 + b1) W2 + b2) for a tile of 128 rows x BN
// units.  The second layer's operand H1 is never read: the workgroup works its rows' H1 out, a slice of 64 units ahead of
// the product (each wavefront 32 rows x 32 units, from X in its registers and W1's rows), and leaves it in LDS.  The rows'
// H1 is needed again by the backward half: of the rows of S each of the row's tiles stores every so many'th slice.
// The bias is added in fp32 after the product, as in the launch of its own that smaller steps have, and H1 has the same
// bits.  With the bias as a step of the product, in three bf16 parts, the step was no faster (1024-1024 at batch 4096 76.9
// us, 76.3 like this), an infinite bias became NaN and so zero, and the gradients were twice as far from those worked out
// in 64 bits with the same bf16 roundings (dW1 there 5.6e-4, like this 2.9e-4).
// The workgroups of a row of tiles repeat the first layer (an eighth of the second's MFMAs in tiles 256 wide, 32 states);
// as a launch of its own it was bound by its start and by writing and reading H1 (17 MB each way at batch 4096 and
// 1024 units).  As long as the two launches there, some 28 us, but us per step 81.4 -> 79.6 (the S' half of H1 never goes to memory); at
// batch 1024 54.5 -> 52.7, 512-512 at 1100 40.8 -> 37.7, 192-192 at 4096 35.7 -> 33.5, 768-768 at 3000 unchanged.
// Without the first layer the launch takes 18.8 us there; its MFMAs add 2.7, ReLU, rounding and LDS writes 3.5 (as
// much when spread between the second layer's MFMAs), the stores of H1 1.9.
// ----------------------------------------------------------------------------------------
typedef MmTile<128, 256, 2, 4, 1, 3> FwLarge;
typedef MmTile<128, 128, 2, 2, 2, 4> FwSmall;

struct ForwardArgs {
    GemmArgs g;                          // Bt = W2T; K: the first layer's units
    const bf16_bits* X;                  // [. x Dp]
    unsigned int Dp;
    const bf16_bits *W1T, *W1T_hi;       // [K x Dp] (_hi: of the rows from g.m_split on)
    const float *b1, *b1_hi, *b2, *b2_hi;
    bf16_bits* H1;                       // rows below store_rows
    unsigned int store_rows;
    bf16_bits* H2;
};

// Dynamic LDS: the slices of W2T and W1T, two of H1, the first bias; then the epilogue's tile.  ND: 32-wide blocks of states.
constexpr unsigned int kFwMaxH = 2048;
template <class S, int ND>
constexpr size_t forward_lds() {
    return std::max<size_t>(S::NS * (S::BN * 128u + ND * 4096u) + 2u * S::BM * 128u + kFwMaxH * 4u,
                            std::max<size_t>(S::KG == 2 ? S::BM * S::BN * 4u : 0u, S::BM * (S::BN * 2u + 16u)));
}
static_assert(forward_lds<FwLarge, 2>() <= 160u * 1024u, "a compute unit's LDS: nothing left with 64 states");

// The slices of H1.  W1T's come with W2T's requests, one ahead, and the bias before them (their first from memory; a load in
// the loop would make the compiler wait for the requests in flight).
template <int ND>
struct MakeH1 {
    const ForwardArgs& p;
    const float* b1;                     // of this lane's first unit in a slice (in LDS)
    unsigned char *at, *lds, *w1;        // where this lane's first four units go; H1's slices; this lane's row of a slice of W1T
    unsigned int stage;                  // bytes between W1T's slices
    unsigned int m0, own, stride, half, g0, r, sw;   // own: the first slice this workgroup stores, then every stride-th
    u32x4 x[2 * ND], w[2 * ND];
    f32x4 b[4];
    f32x16 h;
    u32x4 v[2];
    bf16_bits* to;
    bool keep;
    __device__ __forceinline__ void start(unsigned int slice, unsigned int buf) {
#pragma unroll
        for (unsigned int g = 0; g < 4; ++g) b[g] = *reinterpret_cast<const f32x4*>(b1 + slice * 64u + 8u * g);
#pragma unroll
        for (unsigned int s = 0; s < 2 * ND; ++s)
            w[s] = *reinterpret_cast<const u32x4*>(w1 + buf * stage + 16u * ((2u * s + half) ^ sw));
    }
    __device__ __forceinline__ void multiply(unsigned int) {
#pragma unroll
        for (int v = 0; v < 16; ++v) h[v] = 0.f;
#pragma unroll
        for (int s = 0; s < 2 * ND; ++s)
            h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(w[s]), as_bf16x8(x[s]), h, 0, 0, 0);
    }
    __device__ __forceinline__ void finish(unsigned int slice, int part, int parts) {
        unsigned char* const to = at + (slice & 1u) * 16384u;
#pragma unroll
        for (int g = part * 4 / parts; g < (part + 1) * 4 / parts; ++g) {
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                y[e] = h[4 * g + e] + b[g][e];
                y[e] = y[e] > 0.f ? y[e] : 0.f;
            }
            write_lds8(to + 16u * ((g0 + g) ^ ((r >> 1) & 7u)), bf16_pair(y[0], y[1]), bf16_pair(y[2], y[3]));
        }
    }
    // (the slice is taken from LDS, 16 bytes a thread, and stored a step later: no wait for the reads)
    __device__ __forceinline__ void done(unsigned int slice) {
        keep = slice % stride == own && m0 < p.store_rows;
        if (!keep) return;
        const unsigned int row = threadIdx.x >> 3, c = threadIdx.x & 7u;
#pragma unroll
        for (unsigned int u = 0; u < 2; ++u)
            v[u] = *reinterpret_cast<const u32x4*>(lds + (slice & 1u) * 16384u + (row + 64u * u) * 128u + 16u * (c ^ ((row >> 1) & 7u)));
        to = p.H1 + (size_t)(m0 + row) * p.g.K + slice * 64u + c * 8u;
    }
    __device__ __forceinline__ void flush() {
        if (!keep) return;
        const unsigned int row = m0 + (threadIdx.x >> 3);
        if (row < p.store_rows) *reinterpret_cast<u32x4*>(to) = v[0];
        if (row + 64u < p.store_rows) *reinterpret_cast<u32x4*>(to + (size_t)64u * p.g.K) = v[1];
        keep = false;
    }
};

template <class S, int ND>
__global__ __launch_bounds__(S::kThreads) void forward_kernel(ForwardArgs p) {
    static_assert(S::BM == 128 && S::kThreads == 512, "a wavefront has 32 x 32 of a slice of H1");
    constexpr unsigned int BN = S::BN, LD = BN * 2u + 16u;
    constexpr unsigned int STAGE = BN * 128u + ND * 4096u, H1S = S::NS * STAGE;   // a slice of W2T and of W1T; H1's slices
    constexpr int GB = BN / 8 / S::NW, L = GB + 1;
    extern __shared__ uint4 gemm_smem[];
    unsigned char* smem = reinterpret_cast<unsigned char*>(gemm_smem);
    unsigned int m0, n0, split;
    if (!tile_of<S::BM, S::BN>(p.g, blockIdx.x, &m0, &n0, &split)) return;
    const unsigned int tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned int half = lane >> 5, N = p.g.N, nk = p.g.K / 64u;
    const bool hi = m0 >= p.g.m_split;
    const unsigned int group = wave / (S::WGM * S::WGN), wi = wave % (S::WGM * S::WGN), wn = wi % S::WGN, wm = wi / S::WGN;
    auto swz = [](unsigned int r) { return (r >> 1) & 7u; };
    unsigned int b_off[GB];
#pragma unroll
    for (int u = 0; u < GB; ++u) {
        const unsigned int r = (wave * GB + u) * 8u + (lane >> 3);
        b_off[u] = (min(r, N - 1u - n0) * p.g.ldb + ((lane & 7u) ^ swz(r)) * 8u) * 2u;
    }
    const gchar b_base = (gchar)reinterpret_cast<const char*>((hi ? p.g.Bt_hi : p.g.Bt) + (size_t)n0 * p.g.ldb);
    // W1T: 64 units of a slice, ND * 4 requests of 1 KB (ND = 1: two wavefronts make each, so that all count the same in
    // flight).  Rows of 64 ND bytes; their 16-byte pieces are rotated so that 16 rows' reads fall on all banks.
    constexpr unsigned int CP = 4u * ND, RR = 64u / CP;
    auto swz1 = [](unsigned int row) { return ND == 1 ? (row >> 2) & 3u : (row >> 1) & 7u; };
    const unsigned int w1_req = wave % (4u * ND), w1_row = w1_req * RR + lane / CP;
    const unsigned int w1_off = (w1_row * p.Dp + ((lane % CP) ^ swz1(w1_row)) * 8u) * 2u;
    const bf16_bits* const w1t = hi ? p.W1T_hi : p.W1T;
    auto fetch_one = [&](int u, unsigned int buf, unsigned int slice) {
        if (u < GB)
            request_lds(b_base + (size_t)slice * 128u, b_off[u < GB ? u : 0], smem + buf * STAGE + (wave * GB + u) * 1024u);
        else
            request_lds((gchar)reinterpret_cast<const char*>(w1t) + (size_t)min(slice + 1u, nk - 1u) * (64u * 64u * ND), w1_off,
                        smem + buf * STAGE + BN * 128u + w1_req * 1024u);
    };

    // the first layer: rows 32 (wave mod 4) .., units 32 (wave / 4) .. of a slice
    const unsigned int rb = wave & 3u, ub = wave >> 2, r = rb * 32u + (lane & 31u), unit = ub * 32u + (lane & 31u);
    const float* const b1 = hi ? p.b1_hi : p.b1;
    unsigned char* const b1s = smem + H1S + 2u * S::BM * 128u;
    for (unsigned int q = wave; q * 256u < p.g.K; q += S::NW)
        request_lds((gchar)reinterpret_cast<const char*>(b1), min(q * 256u + lane * 4u, p.g.K - 4u) * 4u, b1s + q * 1024u);
    const unsigned int unit0 = ub * 32u + 4u * half;         // units unit0 + 8 g .. + 3 are this lane's
    MakeH1<ND> make{p, reinterpret_cast<const float*>(b1s) + unit0, smem + H1S + r * 128u + 8u * half, smem + H1S,
                    smem + BN * 128u + unit * (64u * ND), STAGE, m0, n0 / BN, p.g.tiles_n, half, ub * 4u, r, swz1(unit), {}, {}, {}, {}, {}, nullptr, false};
    {
        const bf16_bits* x = p.X + (size_t)min(m0 + r, p.g.M - 1u) * p.Dp + 8u * half;
        const bf16_bits* w = w1t + (size_t)unit * p.Dp + 8u * half;
#pragma unroll
        for (int s = 0; s < 2 * ND; ++s) {
            make.x[s] = *reinterpret_cast<const u32x4*>(x + 16 * s);
            make.w[s] = *reinterpret_cast<const u32x4*>(w + 16 * s);
        }
#pragma unroll
        for (unsigned int g = 0; g < 4; ++g) make.b[g] = *reinterpret_cast<const f32x4*>(b1 + unit0 + 8u * g);
    }

    const unsigned int a_row = H1S + (wm * S::TM * 32u + (lane & 31u)) * 128u, b_row = (wn * S::TN * 32u + (lane & 31u)) * 128u;
    const unsigned int sw = swz(lane & 31u);
    u32x4 a[2][S::TM], b[2][S::TN];
    auto read = [&](unsigned int slice, unsigned int buf, int s, int set) {
        const unsigned int ko = ((2u * (group * S::SP + s) + half) ^ sw) * 16u;
#pragma unroll
        for (int j = 0; j < S::TN; ++j) b[set][j] = *reinterpret_cast<const u32x4*>(smem + buf * STAGE + b_row + ko + j * 4096);
#pragma unroll
        for (int i = 0; i < S::TM; ++i) a[set][i] = *reinterpret_cast<const u32x4*>(smem + (slice & 1u) * 16384u + a_row + ko + i * 4096);
    };
    f32x16 acc[S::TM][S::TN];
    auto mfma = [&](int i, int j, int set) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(b[set][j]), as_bf16x8(a[set][i]), acc[i][j], 0, 0, 0);
    };
    f32x4 bv[S::TN][4];
    unsigned int em, en;
    mm_wave_at<S>(wave, &em, &en);
    mm_clear<S>(acc);
    mm_pipeline<S, L>(nk, fetch_one, read, mfma, [](unsigned int, unsigned int) {}, [&]() {
        const float* b2 = hi ? p.b2_hi : p.b2;
#pragma unroll
        for (int j = 0; j < S::TN; ++j)
#pragma unroll
            for (unsigned int g = 0; g < 4; ++g) {
                const unsigned int n = n0 + en + j * 32u + 8u * g + 4u * half;
                bv[j][g] = *reinterpret_cast<const f32x4*>(b2 + (n < N ? n : 0u));
            }
    }, make);
    make.flush();
    mm_swap_groups<S>(acc, smem, wave, lane);
#pragma unroll
    for (int i = 0; i < S::TK; ++i)
#pragma unroll
        for (int j = 0; j < S::TN; ++j)
#pragma unroll
            for (unsigned int g = 0; g < 4; ++g) {
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = acc[i][j][4 * g + e] + bv[j][g][e];
                    x[e] = x[e] > 0.f ? x[e] : 0.f;
                }
                uint2 pk;
                pk.x = bf16_pair(x[0], x[1]);
                pk.y = bf16_pair(x[2], x[3]);
                *reinterpret_cast<uint2*>(smem + (em + i * 32u + (lane & 31u)) * LD + (en + j * 32u + 8u * g + 4u * half) * 2u) = pk;
            }
    // (a wavefront stores what it parked: its LDS operations complete in order)
    constexpr unsigned int CR = S::TN * 4u, RP = 64u / CR;
#pragma unroll
    for (unsigned int q = 0; q < S::TK * 32u / RP; ++q) {
        const unsigned int row = em + q * RP + lane / CR, c = en + lane % CR * 8u;
        const u32x4 v = *reinterpret_cast<const u32x4*>(smem + row * LD + c * 2u);
        if (m0 + row < p.g.M && n0 + c < N) *reinterpret_cast<u32x4*>(p.H2 + (size_t)(m0 + row) * N + n0 + c) = v;
    }
}

// ----------------------------------------------------------------------------------------
// TD target, loss and the gradient at the second hidden layer's pre-activation.
// A workgroup owns 16 batch rows x 256 hidden units, sixteen lanes to a row.  The lanes of a row
// work out y_i = r_i + gamma (1 - term_i) max_a Q(s'_i, a), delta_i = y_i - Q(s_i, a_i), the loss
// term and g_i = dL/dQ(s_i, a_i) among themselves, without LDS or a barrier, while their share of H2
// is on its way.  Workgroups of the first stripe of units store those and dL/dQ, split into three
// bf16 parts whose sum is the fp32 number, so that the output layer's weight gradient loses nothing
// to the split.  Then dZ2[i][k] = g_i * W3[k][a_i] * 1[H2[i][k] > 0] goes out, 16 bytes a lane.
// Bound by memory: H2 in, dZ2 out (8 MB each at batch 4096 and 1024 units).
// ----------------------------------------------------------------------------------------
// Column of dL/dQ that holds part s (0, 1, 2: from the highest bits down) of action a: the
// parts of 32 actions are neighbours, one tile of the product that contracts them with H2.
__device__ __forceinline__ unsigned int dq_col(unsigned int a, unsigned int s) {
    return (a >> 5) * 96u + s * 32u + (a & 31u);
}

struct TdArgs {
    unsigned int B, G, A, Ap;
    const float* Q;              // [2B x Ap]
    const int* act;
    const float* rew;
    const unsigned char* term;
    float gamma;
    unsigned int loss_kind;
    float beta1, beta2;
    float *y, *delta, *lossi;
    bf16_bits* dQ;               // [B x 3 Ap]
    const bf16_bits* W3T;        // [Ap x G]
    const bf16_bits* H2;         // [2B x G]
    bf16_bits* dZ2;              // [B x G]
    TrainCounters* ctr;
};

constexpr unsigned int kTdRows = 16, kTdCols = 256;

__global__ __launch_bounds__(256) void td_dz_kernel(TdArgs p) {
    const unsigned int tid = threadIdx.x, part = tid & 15u;
    const unsigned int i = blockIdx.x * kTdRows + (tid >> 4), k0 = blockIdx.y * kTdCols + part * 8u;
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {
        // (running products beta^t in double precision: no power function on the device)
        const double pw1 = p.ctr->pw1 * (double)p.beta1, pw2 = p.ctr->pw2 * (double)p.beta2;
        p.ctr->adam_t = p.ctr->adam_t + 1;
        p.ctr->pw1 = pw1;
        p.ctr->pw2 = pw2;
        p.ctr->c1 = (float)(1.0 - pw1);
        p.ctr->c2 = (float)(1.0 - pw2);
    }
    if (i >= p.B) return;                           // (the same for all lanes of a row)
    unsigned int ai = (unsigned int)p.act[i];
    if (ai >= p.A) ai = p.A - 1;                    // an out-of-range action must not turn into a wild address
    u32x4 hv[2] = {}, wv[2] = {};
#pragma unroll
    for (int e = 0; e < 2; ++e)
        if (k0 + 128u * e < p.G) {
            hv[e] = *reinterpret_cast<const u32x4*>(p.H2 + (size_t)i * p.G + k0 + 128u * e);
            wv[e] = *reinterpret_cast<const u32x4*>(p.W3T + (size_t)ai * p.G + k0 + 128u * e);
        }
    float best = -INFINITY;
    const float* qn = p.Q + (size_t)(p.B + i) * p.Ap;
    for (unsigned int a = part; a < p.A; a += 16u) best = fmaxf(best, qn[a]);
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) best = fmaxf(best, __shfl_xor(best, m, 64));
    const float q = p.Q[(size_t)i * p.Ap + ai];
    const float y = p.rew[i] + (p.term[i] ? 0.f : p.gamma * best);
    const float d = y - q;
    float li, slope;
    if (p.loss_kind == RP_MSE || fabsf(d) <= 1.f) {
        li = 0.5f * d * d;
        slope = d;
    } else {
        li = fabsf(d) - 0.5f;
        slope = d > 0.f ? 1.f : -1.f;
    }
    const float g = -slope / (float)p.B;
    if (blockIdx.y == 0) {
        if (part == 0) {
            p.y[i] = y;
            p.delta[i] = d;
            p.lossi[i] = li;
        }
        const bf16_bits hi = bf16_bits_rne(g);
        const float rest = g - bits_to_float(hi);
        const bf16_bits mid = bf16_bits_rne(rest);
        const bf16_bits lo = bf16_bits_rne(rest - bits_to_float(mid));
        bf16_bits* dq = p.dQ + (size_t)i * 3u * p.Ap;
        // two actions a lane: a row's 32-wide parts leave as 64-byte runs
        for (unsigned int a = 2u * part; a < p.Ap; a += 32u) {
            const unsigned int shift = a == ai ? 0u : 16u;
            const bool mine = (a ^ ai) < 2u;        // (a is even)
            *reinterpret_cast<unsigned int*>(dq + dq_col(a, 0)) = mine ? (unsigned int)hi << shift : 0u;
            *reinterpret_cast<unsigned int*>(dq + dq_col(a, 1)) = mine ? (unsigned int)mid << shift : 0u;
            *reinterpret_cast<unsigned int*>(dq + dq_col(a, 2)) = mine ? (unsigned int)lo << shift : 0u;
        }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        u32x4 out;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const float h_lo = __uint_as_float(hv[e][x] << 16), h_hi = __uint_as_float(hv[e][x] & 0xFFFF0000u);
            const float w_lo = __uint_as_float(wv[e][x] << 16), w_hi = __uint_as_float(wv[e][x] & 0xFFFF0000u);
            out[x] = bf16_pair(h_lo > 0.f ? g * w_lo : 0.f, h_hi > 0.f ? g * w_hi : 0.f);
        }
        if (k0 + 128u * e < p.G) *reinterpret_cast<u32x4*>(p.dZ2 + (size_t)i * p.G + k0 + 128u * e) = out;
    }
}

// ----------------------------------------------------------------------------------------
// The backward half of large steps, in two launches.
//
// head_kernel: the output layer, Q = H2 W3 + b3, targets, TD errors, loss terms, dL/dQ, dZ2 and db2.  A workgroup has
// whole rows, 16 of S and the same experiences' 16 of S' (and every gridDim.x-th such group), and its eight
// wavefronts split the hidden units, 32 at a time: a lane's share of H2 is the operand of the output layer's 16x16x32
// MFMA and afterwards the mask of dZ2.  H2 is read once, and every load of a group is requested before the first use:
// the launch is bound by memory (16.8 MB of H2 in, 8.4 MB of dZ2 out at batch 4096 and 1024 units).
//   y_i = r_i + gamma (1 - term_i) max_a Q(s'_i, a), delta_i = y_i - Q(s_i, a_i), g_i = dL/dQ(s_i, a_i),
//   dZ2[i][k] = g_i W3[k][a_i] 1[H2[i][k] > 0]
// dL/dQ is stored in three bf16 parts whose sum is the fp32 number, so that the output layer's weight gradient loses
// nothing to the split.
// As two launches, output layer and the rest, 7.5 + 9.5 us there (with the output layer's gradient in the second).
// ----------------------------------------------------------------------------------------
constexpr unsigned int kHeadThreads = 512, kHeadRows = 16, kHeadMaxGroups = 512;

struct HeadStepArgs {
    unsigned int B, G, A, Ap;
    const int* act;
    const float* rew;
    const unsigned char* term;
    float gamma;
    unsigned int loss_kind;
    float beta1, beta2;
    const float *b3, *b3_hi;             // of the rows of S and of S'
    const bf16_bits *W3T, *W3T_hi;       // [Ap x G], likewise
    const bf16_bits* H2;                 // [2B x G]
    float* Q;                            // [2B x Ap]
    float *y, *delta, *lossi;
    bf16_bits* dQ;                       // [B x 3 Ap]
    bf16_bits* dZ2;                      // [B x G]
    float* part2b;                       // [workgroups][G]: db2
    TrainCounters* ctr;
};

// v of another lane of the row of 16
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}

// SW: 32-unit steps a wavefront holds in registers; layers wider than 256 SW units go in several passes, which read H2
// once more.  TGT: the rows of S' have weights of their own.
template <int SW, bool TGT>
__global__ __launch_bounds__(kHeadThreads) void head_kernel(HeadStepArgs p) {
    constexpr unsigned int LD = 36, NB = TGT ? 2 : 1;
    __shared__ __attribute__((aligned(16))) float part[8][2][kHeadRows][LD];   // [wavefront][S, S'][row][action]
    __shared__ float best_s[kHeadRows], qa_s[kHeadRows], g_s[kHeadRows];
    const unsigned int tid = threadIdx.x, lane = tid & 63u, r16 = lane & 15u, q16 = lane >> 4;
    const unsigned int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x == 0 && tid == 0) {
        // (running products beta^t in double precision: no power function on the device)
        const double pw1 = p.ctr->pw1 * (double)p.beta1, pw2 = p.ctr->pw2 * (double)p.beta2;
        p.ctr->adam_t = p.ctr->adam_t + 1;
        p.ctr->pw1 = pw1;
        p.ctr->pw2 = pw2;
        p.ctr->c1 = (float)(1.0 - pw1);
        p.ctr->c2 = (float)(1.0 - pw2);
    }
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const unsigned int groups = (p.B + kHeadRows - 1u) / kHeadRows, passes = (p.G + 256u * SW - 1u) / (256u * SW);
    for (unsigned int grp = blockIdx.x; grp < groups; grp += gridDim.x) {
        // this lane's experience (the operands' row), and the same again for the rows beyond the batch
        const unsigned int row = grp * kHeadRows + r16, i = min(row, p.B - 1u);
        const unsigned int ai = min((unsigned int)p.act[i], p.A - 1u);   // an out-of-range action must not turn into a wild address
        const float rew = p.rew[i];
        const bool term = p.term[i] != 0;
        const bf16_bits* const h_s = p.H2 + (size_t)i * p.G + 8u * q16;
        const bf16_bits* const h_n = h_s + (size_t)p.B * p.G;
        auto at = [&](unsigned int pass, int s) { return pass * 256u * SW + (wave + 8u * s) * 32u; };   // a step's first unit
        u32x4 hs[SW];
        float best = -INFINITY;
        for (unsigned int ab = 0; ab < p.Ap; ab += 32u) {
            f32x4 c[2][2];
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int j = 0; j < 2; ++j) c[x][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (unsigned int pass = 0; pass < passes; ++pass) {
                u32x4 hn[SW], w[NB][2][SW];
#pragma unroll
                for (int s = 0; s < SW; ++s) {
                    const unsigned int k = at(pass, s), kc = k < p.G ? k : 0u;   // (G is a multiple of 32)
                    hs[s] = *reinterpret_cast<const u32x4*>(h_s + kc);
                    hn[s] = *reinterpret_cast<const u32x4*>(h_n + kc);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const size_t wa = (size_t)(ab + 16u * j + r16) * p.G + kc + 8u * q16;
                        w[0][j][s] = *reinterpret_cast<const u32x4*>(p.W3T + wa);
                        if constexpr (TGT) w[NB - 1][j][s] = *reinterpret_cast<const u32x4*>(p.W3T_hi + wa);
                    }
                }
#pragma unroll
                for (int s = 0; s < SW; ++s) {
                    const bool in = at(pass, s) < p.G;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        c[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(in ? hs[s] : zero), as_bf16x8(in ? w[0][j][s] : zero), c[0][j], 0, 0, 0);
                        c[1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(in ? hn[s] : zero), as_bf16x8(in ? w[NB - 1][j][s] : zero), c[1][j], 0, 0, 0);
                    }
                }
            }
            if (ab || grp != blockIdx.x) __syncthreads();    // (what is there has been read)
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) part[wave][x][4u * q16 + v][16u * j + r16] = c[x][j][v];
            __syncthreads();
            // sixteen threads a row, two actions each: first the rows of S, then those of S'
            const unsigned int x = tid >> 8, r = (tid >> 4) & 15u, a = ab + 2u * (tid & 15u);
            typedef float f32x2 __attribute__((ext_vector_type(2)));
            f32x2 qv = {0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 8; ++w) qv += *reinterpret_cast<const f32x2*>(&part[w][x][r][2u * (tid & 15u)]);
            qv += *reinterpret_cast<const f32x2*>((x ? p.b3_hi : p.b3) + a);
            const unsigned int m = grp * kHeadRows + r;
            if (m < p.B) *reinterpret_cast<f32x2*>(p.Q + ((x ? (size_t)p.B : 0u) + m) * p.Ap + a) = qv;
            if (a < p.A) best = fmaxf(best, qv[0]);
            if (a + 1u < p.A) best = fmaxf(best, qv[1]);
            if (x == 0) {
                const unsigned int am = min((unsigned int)p.act[min(m, p.B - 1u)], p.A - 1u);
                if ((a ^ am) < 2u) qa_s[r] = am == a ? qv[0] : qv[1];
            } else if (ab + 32u >= p.Ap) {
                best = fmaxf(best, dpp<0x128>(best));        // (rotations within the sixteen)
                best = fmaxf(best, dpp<0x124>(best));
                best = fmaxf(best, dpp<0x122>(best));
                best = fmaxf(best, dpp<0x121>(best));
                if ((tid & 15u) == 0) best_s[r] = best;
            }
        }
        __syncthreads();
        const float y = rew + (term ? 0.f : p.gamma * best_s[r16]);
        const float d = y - qa_s[r16];
        float li, slope;
        if (p.loss_kind == RP_MSE || fabsf(d) <= 1.f) {
            li = 0.5f * d * d;
            slope = d;
        } else {
            li = fabsf(d) - 0.5f;
            slope = d > 0.f ? 1.f : -1.f;
        }
        const float g = -slope / (float)p.B;
        if (tid < 16u) {
            g_s[r16] = g;
            if (row < p.B) {
                p.y[i] = y;
                p.delta[i] = d;
                p.lossi[i] = li;
            }
        }
        for (unsigned int pass = 0; pass < passes; ++pass) {
            u32x4 wv[SW];
#pragma unroll
            for (int s = 0; s < SW; ++s) {
                const unsigned int k = at(pass, s), kc = k < p.G ? k : 0u;
                wv[s] = *reinterpret_cast<const u32x4*>(p.W3T + (size_t)ai * p.G + kc + 8u * q16);
                if (passes > 1u) hs[s] = *reinterpret_cast<const u32x4*>(h_s + kc);
            }
#pragma unroll
            for (int s = 0; s < SW; ++s) {
                const unsigned int k = at(pass, s);
                u32x4 out;
                float cs[8];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const float h_lo = __uint_as_float(hs[s][x] << 16), h_hi = __uint_as_float(hs[s][x] & 0xFFFF0000u);
                    const float w_lo = __uint_as_float(wv[s][x] << 16), w_hi = __uint_as_float(wv[s][x] & 0xFFFF0000u);
                    out[x] = bf16_pair(h_lo > 0.f ? g * w_lo : 0.f, h_hi > 0.f ? g * w_hi : 0.f);
                    cs[2 * x] = row < p.B ? __uint_as_float(out[x] << 16) : 0.f;
                    cs[2 * x + 1] = row < p.B ? __uint_as_float(out[x] & 0xFFFF0000u) : 0.f;
                }
                if (row < p.B && k < p.G) *reinterpret_cast<u32x4*>(p.dZ2 + (size_t)i * p.G + k + 8u * q16) = out;
                // db2: the sixteen rows' sum of each column
                float* const sums = p.part2b + (size_t)blockIdx.x * p.G + k + 8u * q16;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    cs[e] += dpp<0x128>(cs[e]);
                    cs[e] += dpp<0x124>(cs[e]);
                    cs[e] += dpp<0x122>(cs[e]);
                    cs[e] += dpp<0x121>(cs[e]);
                }
                if (r16 == 0 && k < p.G) {
                    // (a later group adds to what the first one stored: the same thread did)
                    f32x4 lo = {cs[0], cs[1], cs[2], cs[3]}, up = {cs[4], cs[5], cs[6], cs[7]};
                    f32x4* const to = reinterpret_cast<f32x4*>(sums);
                    if (grp != blockIdx.x) {
                        lo += to[0];
                        up += to[1];
                    }
                    to[0] = lo;
                    to[1] = up;
                }
            }
        }
        __syncthreads();
        if (tid < 256u) {
            // dL/dQ: sixteen lanes a row, two actions a lane, so that a row's 32-wide parts leave as 64-byte runs
            const unsigned int r = tid >> 4, m = grp * kHeadRows + r, am = min((unsigned int)p.act[min(m, p.B - 1u)], p.A - 1u);
            const float gr = g_s[r];
            const bf16_bits hi = bf16_bits_rne(gr);
            const float rest = gr - bits_to_float(hi);
            const bf16_bits mid = bf16_bits_rne(rest);
            const bf16_bits lo = bf16_bits_rne(rest - bits_to_float(mid));
            bf16_bits* dq = p.dQ + (size_t)m * 3u * p.Ap;
            if (m < p.B)
                for (unsigned int a = 2u * (tid & 15u); a < p.Ap; a += 32u) {
                    const unsigned int shift = a == am ? 0u : 16u;
                    const bool mine = (a ^ am) < 2u;         // (a is even)
                    *reinterpret_cast<unsigned int*>(dq + dq_col(a, 0)) = mine ? (unsigned int)hi << shift : 0u;
                    *reinterpret_cast<unsigned int*>(dq + dq_col(a, 1)) = mine ? (unsigned int)mid << shift : 0u;
                    *reinterpret_cast<unsigned int*>(dq + dq_col(a, 2)) = mine ? (unsigned int)lo << shift : 0u;
                }
        }
    }
}

// grad_back_kernel: the step's two large backward products in one launch, side by side because neither
// needs the other, and the first layer's gradient with the first of them.
//  - workgroups [0, n_dz): dZ1 = (dZ2 W2^T) 1[H1 > 0], a tile of BM rows x 128 units.  dZ1 is needed for
//    [dW1^T | db1] = dZ1^T [X | 1] alone, so the tile stays in LDS as bf16, is contracted there with
//    its rows of X and never goes to memory: part1[split][j][d] (column D: db1), a split per row of tiles, or
//    per kGbMaxSplits-th one where there are more.
//  - the next n_dw: dW2 = H1^T dZ2, K-split partials part2[split][j][k].
//  - the rest: [dW3 ; db3], partials part3[split][k][a] (row G: db3).
// As launches of their own (dZ1 stored, then all gradients) 16.3 + 21.8 us at batch 4096 and 1024 units.
constexpr unsigned int kGbMaxSplits = 32;
typedef MmTile<256, 128, 2, 2, 2, 3> GbLarge;
typedef MmTile<128, 128, 2, 2, 2, 4> GbSmall;

struct GradBackArgs {
    GemmArgs dz;                 // A = dZ2, Bt = W2; tiles_m: rows of workgroups
    GemmArgs dw;                 // A = H1, Bt = dZ2
    unsigned int n_dz, n_dw;     // workgroups of the first two kinds, multiples of 8
    const bf16_bits* X;          // [B x Dp]
    const bf16_bits* H1;
    unsigned int D, Dp, Dx;
    const bf16_bits *H2, *dQ;    // dQ: [B x 3 Ap]
    unsigned int Ap, splits3;
    float *part1, *part2, *part3;
};

// Byte of element (r, col) of the dZ1 tile in LDS: rows of 256 bytes whose 64-byte groups are rotated by XOR
// with r mod 4 (for the transposing reads) and the 16-byte pieces of a group with r / 4 mod 4 (for the
// accumulators' stores, 32 rows of a column at a time).  col: of the first of some columns of one piece.
__device__ __forceinline__ unsigned int dz_at(unsigned int r, unsigned int col) {
    return r * 256u + 64u * ((col >> 5) ^ (r & 3u)) + 16u * (((col >> 3) & 3u) ^ ((r >> 2) & 3u)) + (col & 7u) * 2u;
}

template <class S>
__device__ __forceinline__ void dz1_block(const GradBackArgs& p, unsigned int block, unsigned char* smem) {
    static_assert(S::BN == 128 && S::KG == 2, "four tiles of 32 units, and the rows' halves");
    unsigned int m_first, n0, split;
    if (!tile_of<S::BM, S::BN>(p.dz, block, &m_first, &n0, &split)) return;
    const unsigned int tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned int row_split = m_first / S::BM, H = p.dz.N;
    constexpr unsigned int XT = S::BM * 256u, RED = XT + S::BM * 64u;   // places in LDS of X's rows and the halves' sums
    static_assert(RED + 4u * 8192u <= S::kLds, "the epilogue fits");
    unsigned int wm, wn;
    mm_wave_at<S>(wave, &wm, &wn);
    const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    for (unsigned int m0 = m_first; m0 < p.dz.M; m0 += p.dz.tiles_m * S::BM) {
        constexpr unsigned int CR = S::TN * 4u, RP = 64u / CR, PASSES = S::TK * 32u / RP, XN = S::BM * 4u / S::kThreads;
        u32x4 mk[PASSES], xv[XN];
        auto load_x = [&](unsigned int d0) {
#pragma unroll
            for (unsigned int u = 0; u < XN; ++u) {
                const unsigned int e = tid + u * S::kThreads, i = min(m0 + (e >> 2), p.dz.M - 1u);
                xv[u] = *reinterpret_cast<const u32x4*>(p.X + (size_t)i * p.Dp + d0 + (e & 3u) * 8u);
            }
        };
        auto load_mask = [&](unsigned int from, unsigned int to) {
#pragma unroll
            for (unsigned int q = 0; q < PASSES; ++q) {
                if (q < from || q >= to) continue;
                const unsigned int i = min(m0 + wm + q * RP + lane / CR, p.dz.M - 1u), n = n0 + wn + lane % CR * 8u;
                mk[q] = *reinterpret_cast<const u32x4*>(p.H1 + (size_t)i * H + (n < H ? n : 0u));
            }
        };
        f32x16 acc[S::TM][S::TN];
        if (m0 != m_first) __syncthreads();                   // (the last tile's epilogue still read LDS)
        mm_nt<S>(p.dz, m0, n0, smem, acc, [&]() {
            // half of the ReLU's mask and X's rows while the last slice is multiplied (no registers for more)
            load_mask(0, PASSES / 2);
            load_x(0u);
        });
        mm_swap_groups<S>(acc, smem, wave, lane);
        load_mask(PASSES / 2, PASSES);
        // (opaque from here on, so that the addresses below are not worked out ahead of the product, where
        // its registers are needed)
        unsigned int lane = threadIdx.x & 63u;
        asm volatile("" : "+v"(lane));
        const unsigned int tid = wave * 64u + lane;
        const TnLane l(lane);
#pragma unroll
        for (int i = 0; i < S::TK; ++i)
#pragma unroll
            for (int j = 0; j < S::TN; ++j)
#pragma unroll
                for (unsigned int g = 0; g < 4; ++g) {
                    uint2 pk;
                    pk.x = bf16_pair(acc[i][j][4 * g], acc[i][j][4 * g + 1]);
                    pk.y = bf16_pair(acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
                    *reinterpret_cast<uint2*>(smem + dz_at(wm + i * 32u + (lane & 31u), wn + j * 32u + 8u * g + 4u * (lane >> 5))) = pk;
                }
        // (the same wavefront reads what it wrote: LDS operations of a wavefront complete in order)
#pragma unroll
        for (unsigned int q = 0; q < PASSES; ++q) {
            const unsigned int r = wm + q * RP + lane / CR;
            u32x4* at = reinterpret_cast<u32x4*>(smem + dz_at(r, wn + lane % CR * 8u));
            u32x4 v = *at;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = m0 + r < p.dz.M ? relu_mask(v[e], mk[q][e]) : 0u;
            *at = v;
        }
        // [dW1^T | db1], 32 states at a time: wavefront (t, h) has units 32 t .. and half h of the rows
        const unsigned int t = wave & 3u, h = wave >> 2;
        for (unsigned int d0 = 0; d0 < p.Dp; d0 += 32u) {
#pragma unroll
            for (unsigned int u = 0; u < XN; ++u) {
                // (zeros for rows beyond the batch: their dZ1 is zero, and a factor that is not finite would make that NaN)
                const unsigned int e = tid + u * S::kThreads;
                *reinterpret_cast<u32x4*>(smem + XT + e * 16u) = m0 + (e >> 2) < p.dz.M ? xv[u] : u32x4{0u, 0u, 0u, 0u};
            }
            if (d0 + 32u < p.Dp) load_x(d0 + 32u);
            __syncthreads();
            f32x16 c, sum;
#pragma unroll
            for (int v = 0; v < 16; ++v) c[v] = sum[v] = 0.f;
#pragma unroll
            for (unsigned int s = 0; s < S::BM / 32u; ++s) {
                const unsigned int r = h * (S::BM / 2u) + 16u * s + l.row;
                typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
                const unsigned int col = t * 32u + (l.col >> 1);   // (the lane's first column of its 4 x 16 block)
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)RP_LDS_PTR(smem + dz_at(r, col)));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)RP_LDS_PTR(smem + dz_at(r + 4u, col)));
                const u32x4 a = __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                const u32x4 b = tn_fragment(smem, XT + r * 64u + l.col, 64u);
                c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
                if (d0 == 0) sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), as_bf16x8(ones), sum, 0, 0, 0);
            }
            float* const give = reinterpret_cast<float*>(smem + RED) + t * 2048u + lane;
            if (h) {
#pragma unroll
                for (unsigned int v = 0; v < 16; ++v) {
                    give[v * 64u] = c[v];
                    if (d0 == 0) give[1024u + v * 64u] = sum[v];
                }
            }
            __syncthreads();
            if (!h && n0 + t * 32u < H) {                     // (H is a whole number of 32)
                const unsigned int d = d0 + (lane & 31u);
                float* const at = p.part1 + ((size_t)row_split * H + n0 + t * 32u + acc_row(0, lane)) * p.Dx;
#pragma unroll
                for (unsigned int v = 0; v < 16; ++v) {
                    // (a later tile of this workgroup adds to what the first one stored: the same thread did)
                    if (d < p.D) {
                        float* const to = at + acc_row(v, 0) * p.Dx + d;
                        const float x = c[v] + give[v * 64u];
                        *to = m0 == m_first ? x : *to + x;
                    }
                    if (d0 == 0 && (lane & 31u) == 0u) {      // (every column holds the sums)
                        float* const to = at + acc_row(v, 0) * p.Dx + p.D;
                        const float x = sum[v] + give[1024u + v * 64u];
                        *to = m0 == m_first ? x : *to + x;
                    }
                }
            }
        }
    }
}

// [dW3 ; db3] = H2^T dL/dQ for 128 units and 32 actions, over every so many'th chunk of 256 batch rows: a chunk of both
// operands goes to LDS in one go (the sum of its 96 columns of dL/dQ, the three parts of the actions, is taken there).
constexpr unsigned int kW3Rows = 256, kW3MaxSplits = 32;

__device__ __forceinline__ void dw3_block(const GradBackArgs& p, unsigned int block, unsigned char* smem) {
    constexpr unsigned int DQ = kW3Rows * 256u, GA = kW3Rows * 16u / 512u, GB = kW3Rows * 12u / 512u;
    const unsigned int tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned int B = p.dz.M, G = p.dz.K, tiles = (G + 127u) / 128u, blocks_a = p.Ap / 32u;
    const unsigned int split = block / (tiles * blocks_a), m0 = block % tiles * 128u, a0 = block / tiles % blocks_a * 32u;
    const unsigned int t = wave & 3u, h = wave >> 2;
    const TnLane l(lane);
    f32x16 acc[3];
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[s][v] = 0.f;
    float dq_sum = 0.f;                       // db3: action tid % 32, rows 16 (tid / 32) .. of each chunk
    for (unsigned int r0 = split * kW3Rows; r0 < B; r0 += p.splits3 * kW3Rows) {
        if (r0 != split * kW3Rows) __syncthreads();
        const unsigned int rows = min(kW3Rows, B - r0);
        const gchar ha = (gchar)reinterpret_cast<const char*>(p.H2 + (size_t)r0 * G);
        const gchar qa = (gchar)reinterpret_cast<const char*>(p.dQ + (size_t)r0 * 3u * p.Ap + a0 * 3u);
#pragma unroll
        for (unsigned int u = 0; u < GA; ++u) {
            const unsigned int e = (wave * GA + u) * 64u + lane, r = e >> 4, col = m0 + 8u * ((e & 15u) ^ (4u * (r & 3u)));
            request_lds(ha, (min(r, rows - 1u) * G + (col < G ? col : 0u)) * 2u, smem + (wave * GA + u) * 1024u);
        }
#pragma unroll
        for (unsigned int u = 0; u < GB; ++u) {
            const unsigned int e = (wave * GB + u) * 64u + lane, r = e / 12u;
            request_lds(qa, (min(r, rows - 1u) * 3u * p.Ap + (e - r * 12u) * 8u) * 2u, smem + DQ + (wave * GB + u) * 1024u);
        }
        wait_loads<0>();
        __syncthreads();
        if (rows < kW3Rows) {                 // (whatever lies beyond the batch must not meet a factor of zero)
            const u32x4 zero = {0u, 0u, 0u, 0u};
            for (unsigned int e = rows * 16u + tid; e < kW3Rows * 16u; e += 512u) reinterpret_cast<u32x4*>(smem)[e] = zero;
            for (unsigned int e = rows * 12u + tid; e < kW3Rows * 12u; e += 512u) reinterpret_cast<u32x4*>(smem + DQ)[e] = zero;
            __syncthreads();
        }
        // wavefront (t, h): tile t of 32 units, half h of the rows
#pragma unroll
        for (unsigned int s = 0; s < kW3Rows / 32u; ++s) {
            const unsigned int r = h * (kW3Rows / 2u) + 16u * s + l.row;
            const u32x4 a = tn_fragment(smem, r * 256u + tn_tile_at<true>(t, l.rr) + l.col, 256u);
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                const u32x4 b = tn_fragment(smem, DQ + r * 192u + 64u * x + l.col, 192u);
                acc[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), as_bf16x8(b), acc[x], 0, 0, 0);
            }
        }
        if (m0 == 0) {
#pragma unroll
            for (unsigned int r = 0; r < 16; ++r) {
                const bf16_bits* dq = reinterpret_cast<const bf16_bits*>(smem + DQ + ((tid >> 5) * 16u + r) * 192u) + (tid & 31u);
                dq_sum += (bits_to_float(dq[64]) + bits_to_float(dq[32])) + bits_to_float(dq[0]);   // (exact: the fp32 number)
            }
        }
    }
    __syncthreads();
    float* const give = reinterpret_cast<float*>(smem) + t * 1024u + lane;
    float* const sums = reinterpret_cast<float*>(smem) + 4096u;
    if (h) {
#pragma unroll
        for (unsigned int v = 0; v < 16; ++v) give[v * 64u] = (acc[2][v] + acc[1][v]) + acc[0][v];
    }
    sums[tid] = dq_sum;
    __syncthreads();
    float* const out = p.part3 + (size_t)split * (G + 1u) * p.Ap + a0;
    if (m0 == 0 && tid < 32u) {
        float x = 0.f;
#pragma unroll
        for (unsigned int w = 0; w < 16; ++w) x += sums[w * 32u + tid];
        out[(size_t)G * p.Ap + tid] = x;
    }
    if (h || m0 + t * 32u >= G) return;       // (G is a whole number of 32)
#pragma unroll
    for (unsigned int v = 0; v < 16; ++v)
        out[(size_t)(m0 + t * 32u + acc_row(v, lane)) * p.Ap + (lane & 31u)] = ((acc[2][v] + acc[1][v]) + acc[0][v]) + give[v * 64u];
}

template <class S>
__global__ __launch_bounds__(S::kThreads) void grad_back_kernel(GradBackArgs p) {
    extern __shared__ uint4 gemm_smem[];
    unsigned char* smem = reinterpret_cast<unsigned char*>(gemm_smem);
    if (blockIdx.x < p.n_dz) {
        dz1_block<S>(p, blockIdx.x, smem);
        return;
    }
    static_assert(kW3Rows * 448u <= S::kLds, "a chunk of both operands");
    if (blockIdx.x >= p.n_dz + p.n_dw) {
        dw3_block(p, blockIdx.x - p.n_dz - p.n_dw, smem);
        return;
    }
    unsigned int m0, n0, split;
    if (!tile_of<S::BM, S::BN>(p.dw, blockIdx.x - p.n_dz, &m0, &n0, &split)) return;
    const unsigned int lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f32x16 acc[S::TM][S::TN];
    mm_tn<S>(p.dw, m0, n0, split * p.dw.K, smem, acc);
    mm_swap_groups<S>(acc, smem, wave, lane);
    unsigned int wm, wn;
    mm_wave_at<S>(wave, &wm, &wn);
    const EpiSquare epi{p.part2, p.dw.M, p.dw.N};
#pragma unroll
    for (int i = 0; i < S::TK; ++i) epi.tiles(m0 + wm + i * 32u, n0 + wn, acc[i], lane, split);
}

// The update of the two narrow layers and of the second layer's bias, from partial products of their gradients:
//   part3[z][m][a]: m <= G (row G = bias); gradient of W3[m][a] = sum_z part3[z][m][a]
//   part1[z][j][d]: j < H, d <= D (column D = bias); gradient of W1[d][j] = sum_z part1[z][j][d]
// One thread per parameter; splits are added in order, sixteen requested at a time.  Workgroup 0 also reduces the
// per-sample losses to their mean and advances the sampling step counter.
struct SmallOptArgs {
    OptState o;
    unsigned int splits3, splits1, splits_b2, H, G, D, Dp, Dx, Ap, B;
    const float* part3;
    const float* part1;
    const float* part_b2;       // [splits_b2] rows of G, b2_stride apart
    size_t b2_stride;
    size_t oW1, ob1, ob2, oW3, ob3;
    bf16_bits* W1T;   // [H x Dp]
    bf16_bits* W3T;   // [Ap x G]
    bf16_bits *W1T_target, *W3T_target;   // the target network's, or null
    TrainCounters* ctr;
    const float* lossi;
    unsigned int out_grad_only;   // dueling head: only store the output layer's gradient
};

__device__ __forceinline__ float sum_splits(const float* src, size_t stride, unsigned int splits) {
    float g = 0.f;
    for (unsigned int z0 = 0; z0 < splits; z0 += 16u) {
        float part[16];
#pragma unroll
        for (unsigned int z = 0; z < 16; ++z) part[z] = z0 + z < splits ? src[(z0 + z) * stride] : 0.f;
#pragma unroll
        for (unsigned int z = 0; z < 16; ++z) g += part[z];
    }
    return g;
}

// The second layer's bias, 16 columns a workgroup: sixteen threads a column share the partials, of which there may be hundreds.
__device__ __forceinline__ void bias_opt_block(const SmallOptArgs& p, unsigned int block) {
    __shared__ float share[16][17];
    const unsigned int c = threadIdx.x & 15u, z0 = threadIdx.x >> 4, k = block * 16u + c;
    share[z0][c] = sum_splits(p.part_b2 + z0 * p.b2_stride + k, 16u * p.b2_stride, z0 < p.splits_b2 ? (p.splits_b2 - z0 + 15u) / 16u : 0u);
    __syncthreads();
    if (z0) return;
    float g = 0.f;
#pragma unroll
    for (unsigned int z = 0; z < 16; ++z) g += share[z][c];
    opt_update(p.o, p.ob2 + k, g, opt_step(p.o));
}

__device__ __forceinline__ void small_opt_block(const SmallOptArgs& p, unsigned int block) {
    if (block < p.G / 16u) {
        bias_opt_block(p, block);
        return;
    }
    block -= p.G / 16u;
    const unsigned int n3 = (p.G + 1u) * p.Ap, n1 = p.H * (p.D + 1u);
    const unsigned int e = block * 256u + threadIdx.x;
    const OptStep st = opt_step(p.o);
    if (e < n3) {
        const unsigned int m = e / p.Ap, a = e - m * p.Ap;
        const size_t stride = (size_t)(p.G + 1u) * p.Ap;
        const float* src = p.part3 + e;
        const float g = sum_splits(src, stride, p.splits3);
        if (p.out_grad_only) {
            p.o.g[m < p.G ? p.oW3 + (size_t)m * p.Ap + a : p.ob3 + a] = g;
        } else if (m < p.G) {
            const bf16_bits h = bf16_bits_rne(opt_update(p.o, p.oW3 + (size_t)m * p.Ap + a, g, st));
            p.W3T[(size_t)a * p.G + m] = h;
            if (st.sync) p.W3T_target[(size_t)a * p.G + m] = h;
        } else {
            opt_update(p.o, p.ob3 + a, g, st);
        }
    } else if (e < n3 + n1) {
        const unsigned int f = e - n3, j = f / (p.D + 1u), d = f - j * (p.D + 1u);
        const size_t stride = (size_t)p.H * p.Dx;
        const float* src = p.part1 + (size_t)j * p.Dx + d;
        const float g = sum_splits(src, stride, p.splits1);
        if (d < p.D) {
            const bf16_bits h = bf16_bits_rne(opt_update(p.o, p.oW1 + (size_t)d * p.H + j, g, st));
            p.W1T[(size_t)j * p.Dp + d] = h;
            if (st.sync) p.W1T_target[(size_t)j * p.Dp + d] = h;
        } else {
            opt_update(p.o, p.ob1 + j, g, st);
        }
    }
    if (block == 0) {
        __shared__ float wsum[4];
        float acc = 0.f;
        for (unsigned int i = threadIdx.x; i < p.B; i += 256) acc += p.lossi[i];
        acc = wave_sum(acc);
        if ((threadIdx.x & 63u) == 0) wsum[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            p.ctr->loss = (wsum[0] + wsum[1] + wsum[2] + wsum[3]) / (float)p.B;
            p.ctr->step += 1;
        }
    }
}

// The square layer's update from the K-split partial products of [dW ; db]:
//   part[z][m][n], m <= R (row R, the bias, is not this kernel's part), n < N; the gradient is the sum
//   over z, splits added in order.
// A workgroup owns a kSqRows x 64 tile of W: a thread takes four consecutive columns of a row
// (16-byte accesses to the partials and to the fp32 weight, gradient and moments), writes the
// new weights' bf16 copy in the same orientation and parks it in LDS, from where the
// transposed copy (and the target network's, when a sync is due) leaves as 128-byte runs.
// R and N are multiples of 64.
struct SquareOptArgs {
    OptState o;
    unsigned int R, N, splits;
    const float* part;
    size_t w_off;
    bf16_bits* wb;              // [R x N]
    bf16_bits* wbT;             // [N x R]
    bf16_bits* wbT_target;      // [N x R] of the target network, or null
};

__device__ __forceinline__ f32x4 opt_update4(const OptState& o, size_t k, const f32x4& g, const OptStep& st) {
    f32x4 w = *reinterpret_cast<const f32x4*>(o.w + k);
    *reinterpret_cast<f32x4*>(o.g + k) = g;
    if (o.opt == RP_SGD) {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] -= o.lr * g[e];
    } else {
        f32x4 m = *reinterpret_cast<const f32x4*>(o.m + k);
        f32x4 v = *reinterpret_cast<const f32x4*>(o.v + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            m[e] = o.beta1 * m[e] + (1.f - o.beta1) * g[e];
            v[e] = o.beta2 * v[e] + (1.f - o.beta2) * g[e] * g[e];
            w[e] -= o.lr * (m[e] / st.c1) / (sqrtf(v[e] / st.c2) + o.eps);
        }
        *reinterpret_cast<f32x4*>(o.m + k) = m;
        *reinterpret_cast<f32x4*>(o.v + k) = v;
    }
    *reinterpret_cast<f32x4*>(o.w + k) = w;
    if (st.sync) *reinterpret_cast<f32x4*>(o.wt + k) = w;
    return w;
}

constexpr unsigned int kSqRows = 32;   // rows of W per workgroup of the square layer's update (columns: 64)

__device__ __forceinline__ void square_opt_block(const SquareOptArgs& p, unsigned int block_x, unsigned int block_y) {
    constexpr unsigned int TS = 68;                       // bf16 per parked row (64 + padding)
    __shared__ bf16_bits tile[kSqRows * TS];
    const unsigned int tid = threadIdx.x, c4 = (tid & 15u) * 4u, r0 = tid >> 4;
    const unsigned int m0 = block_y * kSqRows, n0 = block_x * 64u;
    const OptStep st = opt_step(p.o);
    const size_t zs = (size_t)(p.R + 1u) * p.N;           // one split's partials
    constexpr unsigned int Q = kSqRows / 16u;
    f32x4 g[Q];
#pragma unroll
    for (unsigned int q = 0; q < Q; ++q) {
        const float* src = p.part + (size_t)(m0 + q * 16u + r0) * p.N + n0 + c4;
        g[q] = *reinterpret_cast<const f32x4*>(src);
        for (unsigned int z = 1; z < p.splits; ++z) g[q] += *reinterpret_cast<const f32x4*>(src + z * zs);
    }
#pragma unroll
    for (unsigned int q = 0; q < Q; ++q) {
        const unsigned int r = q * 16u + r0;
        const size_t at = (size_t)(m0 + r) * p.N + n0 + c4;
        const f32x4 w = opt_update4(p.o, p.w_off + at, g[q], st);
        uint2 pk;
        pk.x = bf16_pair(w[0], w[1]);
        pk.y = bf16_pair(w[2], w[3]);
        *reinterpret_cast<uint2*>(p.wb + at) = pk;
        *reinterpret_cast<uint2*>(tile + r * TS + c4) = pk;
    }
    __syncthreads();
    // transposed copy: kSqRows / 2 lanes write one column of the tile as pairs of rows
    constexpr unsigned int LPC = kSqRows / 2u, CPP = 256u / LPC;   // lanes per column, columns per pass
    const unsigned int mp = (tid % LPC) * 2u;
#pragma unroll
    for (unsigned int pass = 0; pass < 64u / CPP; ++pass) {
        const unsigned int n = pass * CPP + tid / LPC;
        const unsigned int pair = (unsigned int)tile[mp * TS + n] | ((unsigned int)tile[(mp + 1u) * TS + n] << 16);
        const size_t at = (size_t)(n0 + n) * p.R + m0 + mp;
        *reinterpret_cast<unsigned int*>(p.wbT + at) = pair;
        if (st.sync) *reinterpret_cast<unsigned int*>(p.wbT_target + at) = pair;
    }
}

// One launch updates all three layers: the first (N / 64) (R / kSqRows) workgroups take the tiles
// of the square layer, the rest the two narrow layers.
__global__ __launch_bounds__(256) void opt_kernel(SquareOptArgs sq, SmallOptArgs sm) {
    const unsigned int tiles_n = sq.N / 64u, n_square = tiles_n * (sq.R / kSqRows);
    if (blockIdx.x < n_square)
        square_opt_block(sq, blockIdx.x % tiles_n, blockIdx.x / tiles_n);
    else
        small_opt_block(sm, blockIdx.x - n_square);
}

// The same launch with `next_blocks` more workgroups after its `own` ones, which append, sample and
// gather for the NEXT train step (inside a recorded run of steps): nothing the optimizer reads or
// writes is touched by them, and the next step then begins with its first layer.
__global__ __launch_bounds__(256) void opt_ahead_kernel(SquareOptArgs sq, SmallOptArgs sm, AppendGatherArgs next,
                                                        unsigned int own, unsigned int next_blocks) {
    if (blockIdx.x >= own) {
        append_gather_block<2, kDrawUniform>(next, blockIdx.x - own, next_blocks);
        return;
    }
    const unsigned int tiles_n = sq.N / 64u, n_square = tiles_n * (sq.R / kSqRows);
    if (blockIdx.x < n_square)
        square_opt_block(sq, blockIdx.x % tiles_n, blockIdx.x / tiles_n);
    else
        small_opt_block(sm, blockIdx.x - n_square);
}

// What a recorded opt_ahead_kernel node was launched with, apart from the next step's part.
struct OptRecorded {
    SquareOptArgs sq;
    SmallOptArgs sm;
    unsigned int own;
};

// K splits of the narrow layers' gradient products (contraction over the padded batch): as
// many as leave every workgroup at least 256 columns, in whole 64-wide slices, at most 16.
unsigned int batch_splits(unsigned int Bp) {
    unsigned int best = 1;
    for (unsigned int s = 2; s <= 16; ++s)
        if (Bp % (s * 64u) == 0 && Bp / s >= 256u) best = s;
    return best;
}

// K splits of the square layer's gradient product: doubled while its 128 x 128 tiles number
// fewer than the compute units, every split keeps at least 256 columns in whole 64-wide slices.
unsigned int square_splits_for(unsigned int Bp, unsigned int H, unsigned int G) {
    const unsigned int tiles = ((H + 127u) / 128u) * ((G + 127u) / 128u);
    unsigned int s = 1;
    while (tiles * s < 256u && s < 8u && Bp % (2u * s * 64u) == 0 && Bp / (2u * s) >= 256u) s *= 2u;
    return s;
}

// A product with M x N outputs that has few tiles of 128 x 64: those leave most of the chip idle, each
// a serial chain over the whole contraction, and the product in tiles of 16 or 32 rows x 32 columns, K split over eight
// wavefronts, is the faster one although it fetches its operands more often.  us per step in the small form, tiled -> this
// (27 inputs, 30 actions), for the first layer's error: 8 tiles (batch 512, 128-1024) 42.4 -> 34.9, 64 (batch 512, 1024-1024)
// 56.5 -> 53.9, 80 (batch 640) 56.2 -> 57.2, 128 (batch 1024) 62.8 -> 67.1; for the second layer, tiled in 128 x 128: 16
// (batch 64, 1024-1024) 46.1 -> 37.8, 64 (batch 256) 50.7 -> 46.4, 128 (batch 512) 53.9 -> 56.3; K = 64 (batch 100, 64-64) 25.1
// -> 23.4.  Of 130 shapes none of either product is more than 2 % faster on the other side of the line.
bool few_tiles(unsigned int M, unsigned int N) { return (size_t)((M + 127u) / 128u) * ((N + 63u) / 64u) <= 64u; }

// H2 = relu(H1 W2 + b2) for `rows` rows; with hi, rows from m_split on take those weights and biases.
hipError_t second_layer(hipStream_t st, const bf16_bits* H1, unsigned int rows, unsigned int H, unsigned int G,
                        const bf16_bits* W2T, const float* b2, bf16_bits* H2, const bf16_bits* hi, const float* b2_hi,
                        unsigned int m_split) {
    if (!hi) m_split = ~0u;
    if (few_tiles(rows, G)) {
        const SkinnyArgs a{H1, H, W2T, H, rows, G, H, hi ? hi : W2T, m_split};
        return launch_skinny(st, a, SkinnyRelu{b2, b2_hi, m_split, H2, G});
    }
    return launch_gemm<128, 128, 64, 2, 2>(st, H1, H, W2T, H, rows, G, H, EpiForward{b2, b2_hi, m_split, H2, G, rows, G},
                                           1, hi, m_split);
}

// (the narrowest variant that holds a row)
const void* head_func(unsigned int G, bool target) {
    if (G <= 256u) return target ? reinterpret_cast<const void*>(head_kernel<1, true>) : reinterpret_cast<const void*>(head_kernel<1, false>);
    if (G <= 512u) return target ? reinterpret_cast<const void*>(head_kernel<2, true>) : reinterpret_cast<const void*>(head_kernel<2, false>);
    return target ? reinterpret_cast<const void*>(head_kernel<4, true>) : reinterpret_cast<const void*>(head_kernel<4, false>);
}

template <class S>
hipError_t configure_forward() {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(forward_kernel<S, 1>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)forward_lds<S, 1>());
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(forward_kernel<S, 2>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)forward_lds<S, 2>());
}

template <class S>
hipError_t configure_grad_back() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(grad_back_kernel<S>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::kLds);
}

// How a step is launched.
WidePlan plan_for(unsigned int B, unsigned int H, unsigned int G, unsigned int Dp, unsigned int Ap) {
    WidePlan p;
    const unsigned int Bp = (B + 127u) / 128u * 128u;
    // The large form wherever the first layer's error has many tiles, and on large batches (below some 576 either may be
    // the faster, 1024-1024 at batch 64 37.7 us per step in the small form, 49.9 in the large one; before wide second layers
    // as well, 128-1024 at 512 35.0, 36.0, at 1280 42.6, 40.0), unless it is behind by this estimate of how much longer (us)
    // its step takes: it walks the states (grad_back_kernel) and the actions (head_kernel) 32 at a time within a workgroup,
    // where the small form has tiles for them, and the first layer (forward_kernel) in few workgroups where the second has
    // few tiles; the small form's dW2 walks longer shares of the batch, and it takes H1 and dZ1 through memory.  Fitted to
    // 4,900 shapes measured in both (64 to 2048 units, 4 to 1024 states, 2 to 1024 actions, batches of 64 to 8192): the form
    // taken is 0.6 % behind the other on average (3.3 % without the estimate).  Of 3,858 shapes 46 are slower than the step
    // was before it had a large form, by 13 % at most (without the estimate 713, the worst twice as long), and none with up
    // to 96 states, 65 actions, 1024 units and batch 4096; of 1,400 drawn there none.  us per step, small form, large one (30
    // actions and 27 states if not given): 256-256 at batch 1024 31.3, 28.7; with 256 states 38.7, 47.3; 1024 states 59.0, 107;
    // 128 actions 33.3, 34.5; 1024 actions 66.5, 91.2; 1024-1024 at 4096 86.5, 76.0; 1024 states 163, 187; 256 actions 132,
    // 120; 1024 actions 284, 288; 1024-128 at 640, 64 states and actions 39.6, 44.8.
    const unsigned int splits2 = square_splits_for(Bp, H, G);
    const bool fused = Dp <= 64u && H <= kFwMaxH;             // the first two layers in one launch
    const double states = Dp / 32u - 1u, actions = Ap / 32u - 1u, n = std::min(B, 4096u);
    const double behind = -0.81 + 0.53 * states + (0.17 + (1.27e-3 - 0.42e-6 * n) * G) * actions - 1.92e-3 * Bp / splits2 -
                          1.5e-9 * n * H * G +
                          (few_tiles(2u * B, G) ? 0.4 + (fused ? (0.58e-3 + 0.45e-3 * states) * H : 0.) : 0.);
    p.merged = (!few_tiles(B, H) || B >= 1536u || (B >= 576u && G <= 512u)) && behind < 0.;
    p.large = false;
    p.k2 = Bp;
    p.fw_cols = 0;
    if (!p.merged) {
        p.splits3 = p.splits1 = batch_splits(Bp);
        p.splits2 = p.splits_b2 = splits2;
        return p;
    }
    // The first two layers in one launch (up to 64 states; beyond, the first layer repeated in every tile is too much),
    // in tiles of 128 x 256 or 128 x 128: those that take less time in rounds of workgroups, 0.75 and 0.5 us a slice.
    // Over 370 shapes (64 to 2048 units, batches of 450 to 8192) the choice was nowhere more than 0.3 % of the step behind
    // the other; with 0.4 us for the narrow ones up to 9.2 %.
    if (fused) {
        const unsigned int rows = (2u * B + 127u) / 128u;
        const double large = (rows * ((G + 255u) / 256u) + 255u) / 256u * 0.75, small = (rows * ((G + 127u) / 128u) + 255u) / 256u * 0.5;
        p.fw_cols = large <= small ? 256u : 128u;
    }
    // The tiles' height and the splits of dW2's contraction: those whose launch ends first.  Workgroups are dealt to the
    // XCDs in turn, 32 compute units each, and a compute unit holds one: the first XCD's share is followed.  A workgroup of
    // dZ1's or dW2's takes so many us and so many more per slice of 64 of its contraction, one of dZ1's also for every 32
    // states beyond the first, one of dW3's per chunk; a split's partials are written and read at 10 TB/s (a launch apart:
    // in part from the caches).  The figures are those that tell the measured steps in all tiles and splits of 620 shapes
    // apart best (64 to 2048 units, batches of 450 to 8192, 27 to 96 states): the choice is 0.15 % behind the fastest on
    // average, 4 % at worst and more than 3 % in 6.  us per step, the best in tiles of 256 x 128, of 128 x 128 (27 states, 30
    // actions): 1024-1024 at batch 3000 69.3, 74.3; 896-896 at 2700 62.9, 66.1, at 2304 58.6, 55.5; 512-512 at 8192 62.2, 72.0.
    struct Cost { double dz, dz_slice, dz_states, dw, dw_slice; };
    static const Cost kCost[2] = {{7.1, 0.32, 1.3, 2., 0.65}, {10.1, 0.49, 1.3, 1., 0.9}};
    const unsigned int chunks = (B + kW3Rows - 1u) / kW3Rows;
    p.splits3 = std::min(chunks, kW3MaxSplits);
    const unsigned int n_w3 = p.splits3 * ((G + 127u) / 128u) * (Ap / 32u);
    const double t_w3 = 3.9 * ((chunks + p.splits3 - 1u) / p.splits3);
    double best = 0.;
    for (int large = 0; large < 2; ++large) {
        const Cost& c = kCost[large];
        const unsigned int bm = large ? 256u : 128u;
        auto tiles = [bm](unsigned int m, unsigned int n) { return ((m + bm - 1u) / bm) * ((n + 127u) / 128u); };
        const unsigned int rows = std::min((B + bm - 1u) / bm, kGbMaxSplits), rounds = ((B + bm - 1u) / bm + rows - 1u) / rows;
        for (unsigned int s = 1; s <= 16u && (s == 1 || B / s >= 256u); s *= 2u) {
            const unsigned int k = ((B + s - 1u) / s + 63u) / 64u * 64u, splits = (B + k - 1u) / k;
            const double t_dz = rounds * (c.dz + G / 64u * c.dz_slice + (Dp / 32u - 1u) * c.dz_states), t_dw = c.dw + k / 64u * c.dw_slice;
            double free_at[32] = {}, end = 0.;               // (a heap, the earliest at the front)
            const unsigned int n_dz = (rows * ((H + 127u) / 128u) + 7u) / 8u, n_dw = (tiles(H, G) * splits + 7u) / 8u;
            for (unsigned int i = 0; i < n_dz + n_dw + (n_w3 + 7u) / 8u; ++i) {
                std::pop_heap(free_at, free_at + 32, std::greater<double>());
                free_at[31] += i < n_dz ? t_dz : i < n_dz + n_dw ? t_dw : t_w3;
                end = std::max(end, free_at[31]);
                std::push_heap(free_at, free_at + 32, std::greater<double>());
            }
            end += 0.8e-6 * splits * H * G;
            if (best != 0. && end >= best) continue;
            best = end;
            p.large = large != 0;
            p.splits2 = splits;
            p.k2 = k;
        }
    }
    const unsigned int bm = p.large ? 256u : 128u;
    p.splits1 = std::min((B + bm - 1u) / bm, kGbMaxSplits);
    p.splits_b2 = std::min((B + kHeadRows - 1u) / kHeadRows, kHeadMaxGroups);
    return p;
}

bf16_bits host_bf16(float f) {
    unsigned int u;
    memcpy(&u, &f, 4);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (bf16_bits)((u >> 16) | 0x40u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_bits)(u >> 16);
}

}  // namespace

WidePlan wide_plan(unsigned int B, unsigned int H, unsigned int G, unsigned int Dp, unsigned int Ap) {
    return plan_for(B, H, G, Dp, Ap);
}

// Two hidden layers of one width, or of two.  This step is the faster one at every size measured (27
// inputs, 30 actions, one new experience a step, us per step layer by layer -> this: 64-256 at batch 8
// 104 -> 31, at batch 63 157 -> 34; 64-128 at batch 1 67 -> 24, at batch 40 107 -> 26; 128-1024 at batch
// 40 324 -> 45; with target network and dueling head at batch 512 929 -> 56), so that the layer-by-layer
// step is left to those who ask for it.
bool wide_step_supported(const train_config& cfg, const replay* rp_) {
    return cfg.param_dtype == RP_BF16 && rp_->cfg.state_dtype == RP_BF16 && rp_->cfg.layout == RP_PAIR &&
           cfg.hidden % 64 == 0 && cfg.hidden2 % 64 == 0;
}

// Allow the products' LDS sizes (once, at creation).
hipError_t wide_configure() {
    hipError_t ec = configure_gemm<128, 128, 32, 2, 2, EpiForward>();
    if (ec == hipSuccess) ec = configure_gemm<128, 128, 64, 2, 2, EpiForward>();
    if (ec == hipSuccess) ec = configure_gemm<128, 64, 64, 2, 2, EpiMask>();
    if (ec == hipSuccess) ec = configure_grad_products<true>();
    if (ec == hipSuccess) ec = configure_grad_products<false>();
    if (ec == hipSuccess) ec = configure_forward<FwLarge>();
    if (ec == hipSuccess) ec = configure_forward<FwSmall>();
    if (ec == hipSuccess) ec = configure_grad_back<GbLarge>();
    if (ec == hipSuccess) ec = configure_grad_back<GbSmall>();
    return ec;
}

// Refresh the bf16 operand copies of the weights from padded fp32 parameters (host array): all
// four of the trained network, or the three forward operands of the target network.
hipError_t wide_set_weights(trainer* t, const float* padded, bool target) {
    const size_t H = t->H, G = t->Hb, Dp = t->Dp, Ap = t->Ap;
    std::vector<bf16_bits> w1t(H * Dp), w2(H * G), w2t(H * G), w3t(Ap * G);
    for (size_t d = 0; d < Dp; ++d)
        for (size_t j = 0; j < H; ++j) w1t[j * Dp + d] = host_bf16(padded[t->oW1 + d * H + j]);
    for (size_t j = 0; j < H; ++j)
        for (size_t k = 0; k < G; ++k) {
            const bf16_bits h = host_bf16(padded[t->oW2 + j * G + k]);
            w2[j * G + k] = h;
            w2t[k * H + j] = h;
        }
    for (size_t k = 0; k < G; ++k)
        for (size_t a = 0; a < Ap; ++a) w3t[a * G + k] = host_bf16(padded[t->oW3 + k * Ap + a]);
    const WideBuffers& w = t->wd;
    hipError_t e = hipMemcpy(target ? w.W1T_t : w.W1T, w1t.data(), w1t.size() * 2, hipMemcpyHostToDevice);
    if (e == hipSuccess && !target) e = hipMemcpy(w.W2, w2.data(), w2.size() * 2, hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(target ? w.W2T_t : w.W2T, w2t.data(), w2t.size() * 2, hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(target ? w.W3T_t : w.W3T, w3t.data(), w3t.size() * 2, hipMemcpyHostToDevice);
    return e;
}

// Whether the rows of S' share the forward launches of those of S.
static bool rows_in_one_launch(const trainer* t) { return !t->wt || t->B % 128 == 0; }

// (gather, three forward products, TD errors, the first layer's error, the gradients, the update; what
// train_create adds itself: the dueling head's update, a draw in a launch of its own)
unsigned int wide_step_kernels(const trainer* t) {
    const unsigned int halves = rows_in_one_launch(t) ? 1u : 2u;   // launches of each layer's forward product
    return t->plan.merged ? 4u + (t->plan.fw_cols ? 1u : 2u) * halves : 5u + 3u * halves;
}

// The first two layers' products for `rows` rows from row `at` on; with m_split, rows from there on take the target
// network's weights, with target all of them.
template <class S>
static hipError_t launch_forward(trainer* t, hipStream_t st, const bf16_bits* X, unsigned int at, unsigned int rows,
                                 unsigned int m_split, bool target) {
    const unsigned int H = t->H, G = t->Hb, Dp = t->Dp;
    const WideBuffers& w = t->wd;
    const float* wt = t->wt ? t->wt : t->w;
    ForwardArgs a;
    unsigned int blocks;
    // (A is not read: the workgroups make it)
    if (!gemm_args<S::BM, S::BN, 64>(nullptr, H, target ? w.W2T_t : w.W2T, H, rows, G, H, 1,
                                     m_split != ~0u ? w.W2T_t : nullptr, m_split, &a.g, &blocks))
        return hipErrorInvalidValue;
    a.X = X + (size_t)at * Dp; a.Dp = Dp;
    a.W1T = target ? w.W1T_t : w.W1T; a.W1T_hi = t->wt ? w.W1T_t : w.W1T;
    a.b1 = (target ? wt : t->w) + t->ob1; a.b1_hi = wt + t->ob1;
    a.b2 = (target ? wt : t->w) + t->ob2; a.b2_hi = wt + t->ob2;
    a.H1 = static_cast<bf16_bits*>(t->H1); a.store_rows = at ? 0u : t->B;
    a.H2 = static_cast<bf16_bits*>(t->H2) + (size_t)at * G;
    constexpr size_t lds1 = forward_lds<S, 1>(), lds2 = forward_lds<S, 2>();
    if (Dp == 32u) hipLaunchKernelGGL((forward_kernel<S, 1>), dim3(blocks), dim3(S::kThreads), lds1, st, a);
    else hipLaunchKernelGGL((forward_kernel<S, 2>), dim3(blocks), dim3(S::kThreads), lds2, st, a);
    return hipGetLastError();
}

template <class S>
static hipError_t launch_grad_back(trainer* t, hipStream_t st, const WidePlan& plan, const bf16_bits* X, const bf16_bits* H1,
                                   const bf16_bits* dZ2) {
    const unsigned int B = t->B, H = t->H, G = t->Hb, D = t->cfg.state_dim;
    GradBackArgs a;
    // (rows of workgroups: at most plan.splits1, each with every so many'th tile)
    bool ok = gemm_args<S::BM, S::BN, 64>(dZ2, G, t->wd.W2, G, std::min(B, plan.splits1 * S::BM), H, G, 1, nullptr, 0, &a.dz, &a.n_dz);
    ok = ok && gemm_args<S::BM, S::BN, 64>(H1, H, dZ2, G, H, G, plan.splits2 * plan.k2, plan.splits2, nullptr, 0, &a.dw, &a.n_dw);
    if (!ok) return hipErrorInvalidValue;
    a.dz.M = B;
    a.dw.batch = B;
    a.X = X; a.H1 = H1; a.D = D; a.Dp = t->Dp; a.Dx = (D + 1 + 31) / 32 * 32;
    a.H2 = static_cast<const bf16_bits*>(t->H2); a.dQ = t->wd.dQ; a.Ap = t->Ap; a.splits3 = plan.splits3;
    a.part1 = t->wd.part1; a.part2 = t->wd.part2; a.part3 = t->wd.part3;
    const unsigned int n3 = plan.splits3 * ((G + 127) / 128) * (t->Ap / 32);
    hipLaunchKernelGGL(grad_back_kernel<S>, dim3(a.n_dz + a.n_dw + n3), dim3(S::kThreads), S::kLds, st, a);
    return hipGetLastError();
}

// Enqueue every kernel of one executed step after the append.
hipError_t enqueue_wide_step(trainer* t, hipStream_t st, unsigned int* count, bool sample) {
    // H, G: widths of the first and the second hidden layer
    const unsigned int B = t->B, Bp = t->Bp, H = t->H, G = t->Hb, Dp = t->Dp, Ap = t->Ap;
    const unsigned int D = t->cfg.state_dim, A = t->cfg.num_actions;
    WideBuffers& w = t->wd;
    bf16_bits* X = static_cast<bf16_bits*>(t->X);
    bf16_bits* H1 = static_cast<bf16_bits*>(t->H1);
    bf16_bits* H2 = static_cast<bf16_bits*>(t->H2);
    bf16_bits* dZ2 = static_cast<bf16_bits*>(t->dZ2);
    bf16_bits* dZ1 = static_cast<bf16_bits*>(t->dZ1);
    unsigned int n = 0;
    OptState o{t->w, t->g, t->m, t->v, t->cfg.opt, t->cfg.lr, t->cfg.beta1, t->cfg.beta2, t->cfg.eps,
               t->ctr, t->wt, t->cfg.target_sync};
    // With a frozen target network the rows of S' (B .. 2B-1) are multiplied by its weights: in
    // the same launch when tiles do not straddle row B, else in a launch of their own.
    const bool tgt = t->wt != nullptr;
    const bool one_launch = rows_in_one_launch(t);
    const float *b1t = tgt ? t->wt + t->ob1 : nullptr, *b2t = tgt ? t->wt + t->ob2 : nullptr;
    const float* b3t = tgt ? t->wt + t->ob3 : nullptr;
    const unsigned int rows = one_launch ? 2 * B : B;   // rows of the first forward launch

    // sample B slots and unpack into X = [S ; S']
    hipError_t e = hipSuccess;
    unsigned int launched = 0;
    if (sample) {
        e = launch_sample_gather(t->rp_->geom, t->rp_->cfg.seed, 0, &t->ctr->step, B, X,
                                 X + (size_t)B * Dp, Dp, t->act, t->rew, t->term, t->idx, st, 0, 0, t->rp_->draw_scratch, &launched);
        if (e != hipSuccess) return e;
        n += launched;
    }
    const WidePlan& plan = t->plan;
    if (plan.fw_cols) {
        auto forward = [&](unsigned int at, unsigned int n_rows, unsigned int split, bool target) {
            return plan.fw_cols == 256u ? launch_forward<FwLarge>(t, st, X, at, n_rows, split, target)
                                        : launch_forward<FwSmall>(t, st, X, at, n_rows, split, target);
        };
        e = forward(0, rows, tgt && one_launch ? B : ~0u, false);
        if (e != hipSuccess) return e;
        ++n;
        if (!one_launch) {
            e = forward(B, B, ~0u, true);
            if (e != hipSuccess) return e;
            ++n;
        }
    } else {
        // forward on the 2B rows
        e = launch_gemm<128, 128, 32, 2, 2>(st, X, Dp, w.W1T, Dp, rows, H, Dp,
                                               EpiForward{t->w + t->ob1, b1t, tgt ? B : ~0u, H1, H, rows, H},
                                               1, tgt && one_launch ? w.W1T_t : nullptr, B);
        if (e != hipSuccess) return e;
        ++n;
        if (!one_launch) {
            e = launch_gemm<128, 128, 32, 2, 2>(st, X + (size_t)B * Dp, Dp, w.W1T_t, Dp, B, H, Dp,
                                                   EpiForward{b1t, b1t, ~0u, H1 + (size_t)B * H, H, B, H});
            if (e != hipSuccess) return e;
            ++n;
        }
        const float* b2 = t->w + t->ob2;
        e = second_layer(st, H1, rows, H, G, w.W2T, b2, H2, tgt && one_launch ? w.W2T_t : nullptr, b2t, B);
        if (e != hipSuccess) return e;
        ++n;
        if (!one_launch) {
            e = second_layer(st, H1 + (size_t)B * H, B, H, G, w.W2T_t, b2t, H2 + (size_t)B * G, nullptr, nullptr, 0);
            if (e != hipSuccess) return e;
            ++n;
        }
    }
    if (!plan.merged) {
        SkinnyArgs a;
        a.A = H2; a.lda = G; a.Bt = w.W3T; a.ldb = G; a.M = rows; a.N = Ap; a.K = G;
        a.Bt_hi = tgt ? w.W3T_t : w.W3T; a.m_split = tgt ? B : ~0u;
        const float* b3 = t->w + t->ob3;
        e = launch_skinny(st, a, SkinnyBias{b3, tgt ? b3t : b3, a.m_split, t->Q, Ap});
        if (e != hipSuccess) return e;
        ++n;
        if (!one_launch) {
            a.A = H2 + (size_t)B * G; a.M = B; a.Bt = a.Bt_hi = w.W3T_t; a.m_split = ~0u;
            e = launch_skinny(st, a, SkinnyBias{b3t, b3t, ~0u, t->Q + (size_t)B * Ap, Ap});
        }
    }
    if (e != hipSuccess) return e;
    if (!plan.merged && !one_launch) ++n;
    const unsigned int Dx = (D + 1 + 31) / 32 * 32;
    if (plan.merged) {
        HeadStepArgs a;
        a.B = B; a.G = G; a.A = A; a.Ap = Ap;
        a.act = t->act; a.rew = t->rew; a.term = t->term;
        a.gamma = t->cfg.gamma; a.loss_kind = t->cfg.loss; a.beta1 = t->cfg.beta1; a.beta2 = t->cfg.beta2;
        a.b3 = t->w + t->ob3; a.b3_hi = tgt ? b3t : a.b3;
        a.W3T = w.W3T; a.W3T_hi = tgt ? w.W3T_t : w.W3T;
        a.H2 = H2; a.Q = t->Q; a.y = t->y; a.delta = t->delta; a.lossi = t->lossi;
        a.dQ = w.dQ; a.dZ2 = dZ2; a.part2b = w.part2b;
        a.ctr = t->ctr;
        void* kargs[] = {&a};
        e = hipLaunchKernel(head_func(G, tgt), dim3(plan.splits_b2), dim3(kHeadThreads), kargs, 0, st);
        if (e != hipSuccess) return e;
        ++n;
        e = plan.large ? launch_grad_back<GbLarge>(t, st, plan, X, H1, dZ2) : launch_grad_back<GbSmall>(t, st, plan, X, H1, dZ2);
        if (e != hipSuccess) return e;
        ++n;
    } else {
        // targets, TD errors, loss terms, dL/dQ and dZ2
        {
            TdArgs a;
            a.B = B; a.G = G; a.A = A; a.Ap = Ap;
            a.Q = t->Q; a.act = t->act; a.rew = t->rew; a.term = t->term;
            a.gamma = t->cfg.gamma; a.loss_kind = t->cfg.loss; a.beta1 = t->cfg.beta1; a.beta2 = t->cfg.beta2;
            a.y = t->y; a.delta = t->delta; a.lossi = t->lossi;
            a.dQ = w.dQ; a.W3T = w.W3T; a.H2 = H2; a.dZ2 = dZ2;
            a.ctr = t->ctr;
            hipLaunchKernelGGL(td_dz_kernel, dim3((B + kTdRows - 1) / kTdRows, (G + kTdCols - 1) / kTdCols), dim3(256),
                               0, st, a);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
            ++n;
        }
        // dZ1 = (dZ2 W2^T) masked by the first ReLU; uses W2 before its update
        if (few_tiles(B, H)) {
            const SkinnyArgs za{dZ2, G, w.W2, G, B, H, G, w.W2, ~0u};
            e = launch_skinny(st, za, SkinnyMask{H1, dZ1, H});
        } else {
            e = launch_gemm<128, 64, 64, 2, 2>(st, dZ2, G, w.W2, G, B, H, G, EpiMask{H1, dZ1, H, B, H});
        }
        if (e != hipSuccess) return e;
        ++n;
        // the three weight-gradient products, K-split partials each, in one launch:
        //   [dW2 ; db2] (row H);  [dW3 ; db3] (row G) with the three parts of dL/dQ side by side;
        //   [dW1^T | db1] (column D)
        const unsigned int splits = plan.splits1, splits2 = plan.splits2;
        {
            GemmArgs g2, g3, g1;
            unsigned int n2 = 0, n3 = 0, n1 = 0;
            const bool narrow1 = Dp == 32;
            bool ok = gemm_args<128, 128, 64>(H1, H, dZ2, G, H, G, Bp, splits2, nullptr, 0, &g2, &n2);
            ok = ok && gemm_args<128, 96, 64>(H2, G, w.dQ, 3 * Ap, G, 3 * Ap, Bp, splits, nullptr, 0, &g3, &n3);
            ok = ok && (narrow1 ? gemm_args<128, 32, 64>(dZ1, H, X, Dp, H, Dp, Bp, splits, nullptr, 0, &g1, &n1)
                                : gemm_args<128, 128, 64>(dZ1, H, X, Dp, H, Dp, Bp, splits, nullptr, 0, &g1, &n1));
            if (!ok) return hipErrorInvalidValue;
            g2.batch = g3.batch = g1.batch = B;
            const EpiSquare e2{w.part2, H, G};
            const EpiOutput e3{w.part3, G, Ap};
            const EpiFirst e1{w.part1, H, D, Dx};
            constexpr size_t lds = gemm_tn_lds_bytes<128, 128>();
            const dim3 grid(n2 + n3 + n1), block(kTnThreads);
            if (narrow1)
                hipLaunchKernelGGL(grad_products_kernel<true>, grid, block, lds, st, g2, e2, n2, g3, e3, n3, g1, e1);
            else
                hipLaunchKernelGGL(grad_products_kernel<false>, grid, block, lds, st, g2, e2, n2, g3, e3, n3, g1, e1);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
            ++n;
        }
    }
    // all three layers' update, mean loss, step counter
    {
        SquareOptArgs q;
        q.o = o; q.R = H; q.N = G; q.splits = plan.splits2; q.part = w.part2;
        q.w_off = t->oW2; q.wb = w.W2; q.wbT = w.W2T; q.wbT_target = w.W2T_t;
        SmallOptArgs a;
        a.o = o; a.splits3 = plan.splits3; a.splits1 = plan.splits1; a.H = H; a.G = G; a.D = D; a.Dp = Dp; a.Dx = Dx; a.Ap = Ap; a.B = B;
        a.part3 = w.part3; a.part1 = w.part1;
        // (the second layer's bias: row H of each split's partials, or rows of its own)
        a.part_b2 = plan.merged ? w.part2b : w.part2 + (size_t)H * G;
        a.splits_b2 = plan.splits_b2;
        a.b2_stride = plan.merged ? G : (size_t)(H + 1) * G;
        a.ob2 = t->ob2;
        a.oW1 = t->oW1; a.ob1 = t->ob1; a.oW3 = t->oW3; a.ob3 = t->ob3;
        a.W1T = w.W1T; a.W3T = w.W3T; a.W1T_target = w.W1T_t; a.W3T_target = w.W3T_t;
        a.ctr = t->ctr; a.lossi = t->lossi;
        a.out_grad_only = t->dueling ? 1u : 0u;
        const unsigned int elems = (G + 1) * Ap + H * (D + 1);
        const unsigned int own = (G / 64) * (H / kSqRows) + G / 16 + (elems + 255) / 256;
        if (t->rec_next) {
            // (recording a run of steps: this launch also gathers the next step's batch; the rest of
            // its arguments is kept for the launches that replace the next step's part)
            if (!t->w_args_host[0]) t->w_args_host[0] = malloc(sizeof(OptRecorded));
            if (!t->w_args_host[0]) return hipErrorOutOfMemory;
            const OptRecorded rec{q, a, own};
            memcpy(t->w_args_host[0], &rec, sizeof(rec));
            unsigned int nb = 0;
            size_t lds = 0;
            append_gather_shape(*t->rec_next, &nb, &lds);
            hipLaunchKernelGGL(opt_ahead_kernel, dim3(own + nb), dim3(256), lds, st, q, a, *t->rec_next, own, nb);
        } else {
            hipLaunchKernelGGL(opt_kernel, dim3(own), dim3(256), 0, st, q, a);
        }
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        ++n;
        unsigned int nh = 0;
        e = enqueue_head_update(t, st, &nh);
        if (e != hipSuccess) return e;
        n += nh;
    }
    if (count) *count = n;
    return hipGetLastError();
}

void* opt_ahead_func() { return reinterpret_cast<void*>(opt_ahead_kernel); }

hipError_t patch_opt_ahead_node(trainer* t, hipGraphExec_t exec, hipGraphNode_t node,
                                const hipKernelNodeParams& recorded, const AppendGatherArgs& next) {
    OptRecorded rec;
    memcpy(&rec, t->w_args_host[0], sizeof(rec));
    AppendGatherArgs nx = next;
    unsigned int nb = 0;
    size_t lds = 0;
    append_gather_shape(nx, &nb, &lds);
    void* kargs[] = {&rec.sq, &rec.sm, &nx, &rec.own, &nb};
    hipKernelNodeParams np = recorded;
    np.kernelParams = kargs;
    np.extra = nullptr;
    return hipGraphExecKernelNodeSetParams(exec, node, &np);
}

}  // namespace rp
