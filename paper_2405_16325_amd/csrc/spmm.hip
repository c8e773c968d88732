// 2:4 sparse x dense product on CDNA4's structured-sparse MFMA, shared by
// slope_spmm_fwd (Eq. 4, with the low-rank K-extension of Eq. 11) and slope_spmm_bwd_x (Eq. 6).
//
//     C[n, m] = sum_k B[n, k] * A[m, k]        A: packed 2:4 along k (vals + 4-bit metadata)
//             + sum_k2 B2[n, k2] * A2[m, k2]   dense bf16, K2 = adapter rank (optional)
//
// fwd  : A = W^R        (m = d_out, k = d_in ), B = X,  C = Y,  B2 = X L, A2 = R^T given as R (k-major)
// bwd_x: A = (W^{R,C})^T (m = d_in,  k = d_out), B = dY, C = dX (with adapters: B2 = dY R^T, A2 = L)
//
// The instruction is v_smfmac_f32_16x16x64_bf16 (D[16 x 16] += Asparse[16 x 64] * B[64 x 16]):
//   A   lane l holds row l%16 and the 8 packed values of logical k = 16*(l/16) .. +15
//   idx lane l holds the 4 metadata nibbles of those 16 k in bits 0..15 (idx0 | idx1 << 2 each)
//   B   lane l holds column l%16; registers 0-3 = k 8*(l/16) .. +7, registers 4-7 = 32 + the same
//   D   lane l holds column l%16, rows 4*(l/16) .. +3
// so the sparse operand is the weight, rows of D are output features, and a lane's four
// accumulators are four consecutive features of one token: an 8-byte store into row-major C.
//
// Four kernels here (launch_spmm picks; the forms for very few tokens are in spmm_stream.hip):
// spmm_split_kernel (the 256 x 256 tile), spmm_kernel<BM, BN> (the other large tiles) and spmm_ring_kernel<BM, BN>
// (the smaller ones) are the fast ones and need K % 64 == 0; spmm_generic_kernel takes any K % 8 == 0 with a plain
// register-staged pipeline.
//
// spmm_kernel.  What a compute unit can pull from L2 per unit of time matters as much as the matrix
// pipe (whose clock the power management lowers well below nominal under this load), so the data
// path is built around full 128-byte lines:
//   - every global -> LDS load instruction (global_load_lds_dwordx4, no registers in between)
//     fetches 8 rows x 128 contiguous bytes, 8 consecutive lanes per row;
//   - a row of the token operand has 128 bytes per k-step of 64, so B sits in a ring of three
//     k-step stages; a row of the packed weight has only 64, so A is fetched for two k-steps at
//     a time into two alternating pair buffers, and its metadata for eight k-steps at a time (four where LDS is short);
//   - inside a row the eight 16-byte chunks are rotated by (row / 2) % 8, which makes the
//     ds_read_b128 of the MFMA layout (16 lanes = 16 rows, same chunk) hit 16 different bank groups.
// A workgroup owns a BM x BN tile of C with 8 wavefronts, two per SIMD, all of which multiply (2 x 4) and load or four of which multiply
// (2 x 2) while the others load (tile_mult); one barrier per k-step: while a wavefront
// multiplies a k-step it reads the fragments of the next one, and the loads of the third after it are queued.  (Before, two groups of
// wavefronts took turns at reading and multiplying, two barriers per k-step, which made a k-step at least twice a group's
// LDS reads: the matrix pipes were busy a third of it.  us, operands in the last-level cache, before / now: 1000 tokens, 4352 x 4352 on
// 192 x 128 40.1 / 35.0, on 256 x 128 43.6 / 39.2; 2048 tokens, 4352 x 4352 on 256 x 192 57.3 / 52.7, on 192 x 192 51.3 / 50.3; 330
// tokens, 3328 x 13568, rank 64, in slabs 44.6 / 41.0.  From HBM, whose latency bounds them, 48.2 / 45.5, 52.1 / 52.2, 65.3 / 64.2,
// 59.0 / 59.0, 52.1 / 50.4.)
#include <type_traits>

#include "pipeline.h"
#include "skinny.h"

namespace {

template <int BMT> constexpr int FACTOR_PITCH = BMT * 2 + 32;  // pitch % 128 == 32: the four rows of a transposing read fall on distinct banks

// Rows kc .. kc + kn - 1 of a k-major factor, BMT columns, to LDS between two barriers, by THREADS threads.  Pieces of 16 bytes per thread: a
// compile-time count, so that all of a thread's global loads are in flight together (a loop of load, wait, LDS store per piece pays the L2 latency
// once per piece).  (A macro: as an inlined function the kernels with eight pieces per thread spill.)
#define STAGE_CHUNK                                                                                    \
    {                                                                                                  \
        constexpr int SEG = BMT / 8, PER = 128 * SEG / THREADS;                                        \
        static_assert(128 * SEG % THREADS == 0, "whole pieces per thread");                            \
        u32x4 piece[PER];                                                                              \
        _Pragma("unroll") for (int u = 0; u < PER; ++u) {                                              \
            const int idx = tid + u * THREADS, k = idx / SEG, col = tile_f0 + 8 * (idx % SEG);         \
            piece[u] = (u32x4){0u, 0u, 0u, 0u};                                                        \
            if (k < kn && col < m) piece[u] = *(const u32x4*)(A2 + (size_t)(kc + k) * m + col);        \
        }                                                                                              \
        __syncthreads();                                      /* the rings are drained / the last chunk is consumed */ \
        _Pragma("unroll") for (int u = 0; u < PER; ++u) {                                              \
            const int idx = tid + u * THREADS;                                                         \
            *(u32x4*)(smem + (idx / SEG) * FACTOR_PITCH<BMT> + (idx % SEG) * 16) = piece[u];           \
        }                                                                                              \
    }

// The factor's chunks by the wavefronts that only load, THREADS of them: the first is requested while the others multiply the last k-steps, the
// next ones while they multiply a chunk.  tid counts from the first of these wavefronts.  (us, from memory, eight wavefronts that stage / four that
// multiply / four that load: 2132 tokens, 3584 x 512, rank 160 on 256 x 128 23.0 / 23.5 / 22.6; 1239, 2816 x 256, rank 256 on 128 x 128 16.5 / 17.2 / 16.3.)
template <int BMT, int THREADS>
__device__ __forceinline__ void stage_factor(const bf16_t* __restrict__ A2, int K2, int m, uint8_t* smem, int tile_f0, int tid) {
    for (int kc = 0; kc < -K2; kc += 128) {
        const int kn = -K2 - kc < 128 ? -K2 - kc : 128;
        STAGE_CHUNK
        __syncthreads();
    }
}

// Tail shared by the tile kernels, for one wavefront whose acc[i][j] is the 16 x 16 fragment at
// features f0 + 16 i, tokens t0 + 16 j.
//  - dense K-extension: C += B2 * A2^T with v_mfma_f32_16x16x32_bf16.  K2 > 0: A2 is [m][K2],
//    k-contiguous like B2, and both operands come straight from global memory (lane l: row l%16,
//    k = 8*(l/16) .. +7).  K2 < 0: A2 is k-major, [-K2][m] (the adapter factor R as stored): the
//    workgroup stages the tile's BMT columns of 128 rows at a time in LDS (the rings are idle by
//    then) and the wavefronts read their fragments back with the transposing LDS read; every
//    thread of the workgroup must make the call (it contains barriers) or, STAGED, all others that of stage_factor;
//  - epilogue: store_rows. BNT = tokens of the workgroup's tile, tile_t0 its first token; every thread must make the call.
//  - with a slab buffer (a split over k, see launch_spmm_slabs): the fp32 accumulators go to
//    partial[token][feature] instead, 16 bytes per lane, and a reduction kernel finishes.
template <int MF, int NF, int BMT, int BNT, int THREADS, bool STAGED = false>
__device__ __forceinline__ void extend_and_store(f32x4 (&acc)[MF][NF], int f0, int t0, int m, int n, int l16, int lq,
                                                 const bf16_t* __restrict__ B2, const bf16_t* __restrict__ A2,
                                                 int K2, bf16_t* __restrict__ C, uint8_t* smem, int tile_f0,
                                                 int tile_t0, float* __restrict__ partial = nullptr) {
    if (K2 < 0) {
        constexpr int PITCH = FACTOR_PITCH<BMT>;
        const int KR = -K2, tid = (int)threadIdx.x;
        const bf16_t* b_row[NF];
#pragma unroll
        for (int j = 0; j < NF; ++j) b_row[j] = B2 + (size_t)wrap_row(t0 + j * 16 + l16, n) * KR + lq * 8;
        // lane (s = l16, q = lq) points at staged row 8 q + 4 h + s / 4, column 4 (s % 4) of a fragment
        const uint8_t* tr = smem + (8 * lq + (l16 >> 2)) * PITCH + 2 * (f0 - tile_f0 + 4 * (l16 & 3));
        // steps whose token-side fragments are requested before the pieces of the factor; where stage_factor brings those, all
        constexpr int FIRST = STAGED ? 4 : 2;
        for (int kc = 0; kc < KR; kc += 128) {
            const int kn = KR - kc < 128 ? KR - kc : 128;     // a multiple of 32
            // the token-side fragments of the whole chunk come straight from global memory: requested first
            // (steps past the chunk's end re-read the first, unused)
            AFrag b2[4][NF];
#pragma unroll
            for (int st = 0; st < FIRST; ++st)
#pragma unroll
                for (int j = 0; j < NF; ++j) b2[st][j].u = *(const u32x4*)(b_row[j] + kc + (32 * st < kn ? 32 * st : 0));
            if (STAGED) __syncthreads();                      // (the two of stage_factor)
            else STAGE_CHUNK
#pragma unroll
            for (int st = FIRST; st < 4; ++st)                // in the registers the staged pieces have left
#pragma unroll
                for (int j = 0; j < NF; ++j) b2[st][j].u = *(const u32x4*)(b_row[j] + kc + (32 * st < kn ? 32 * st : 0));
            __syncthreads();
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const int kk = 32 * st;
                if (kk >= kn) break;                          // uniform
#pragma unroll
                for (int i = 0; i < MF; ++i) {
                    union { s16x4 hh[2]; bf16x8 v; } a;
                    a.hh[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (s16x4 __attribute__((address_space(3)))*)(tr + kk * PITCH + 32 * i));
                    a.hh[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (s16x4 __attribute__((address_space(3)))*)(tr + (kk + 4) * PITCH + 32 * i));
#pragma unroll
                    for (int j = 0; j < NF; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b2[st][j].v, acc[i][j], 0, 0, 0);
                }
            }
        }
    }
    if (K2 > 0) {
        // operands of step k0 + 32 are requested before the MFMAs of step k0 are issued
        const bf16_t* a_row[MF];
        const bf16_t* b_row[NF];
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            int row = f0 + i * 16 + l16;
            a_row[i] = A2 + (size_t)wrap_row(row, m) * K2 + lq * 8;
        }
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            int row = t0 + j * 16 + l16;
            b_row[j] = B2 + (size_t)wrap_row(row, n) * K2 + lq * 8;
        }
        // Beside a large tile's sums there is no room for the features of two steps: a fragment of the next step is then loaded into
        // the registers of the same one as soon as its products are queued.  (us, from memory, each step's loads after the products before it / so: 5658
        // tokens, 768 x 256, rank 160 on 192 x 96 19.9 / 16.1; 11469, 512 x 256, rank 160 on 256 x 128 27.2 / 20.6; 664, 5888 x 3072, rank 160 47.3 / 40.9)
        constexpr bool IN_PLACE = THREADS < 512 && MF * NF > 16;
        constexpr int A_SETS = IN_PLACE ? 1 : 2;
        AFrag a2[A_SETS][MF], b2[2][NF];
#pragma unroll
        for (int j = 0; j < NF; ++j) b2[0][j].u = *(const u32x4*)(b_row[j]);
#pragma unroll
        for (int i = 0; i < MF; ++i) a2[0][i].u = *(const u32x4*)(a_row[i]);
        for (int k0 = 0; k0 < K2; k0 += 64) {                 // K2 % 32 == 0: two steps per trip, the second maybe absent
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int kk = k0 + 32 * h;                   // uniform
                if (kk >= K2) break;
                const int kn = kk + 32 < K2 ? kk + 32 : kk;   // the last step re-reads itself (unused)
                if (!IN_PLACE) {
#pragma unroll
                    for (int i = 0; i < MF; ++i) a2[(h ^ 1) % A_SETS][i].u = *(const u32x4*)(a_row[i] + kn);
                }
#pragma unroll
                for (int j = 0; j < NF; ++j) b2[h ^ 1][j].u = *(const u32x4*)(b_row[j] + kn);
                if (IN_PLACE) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < MF; ++i) {
#pragma unroll
                    for (int j = 0; j < NF; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2[h % A_SETS][i].v, b2[h][j].v, acc[i][j], 0, 0, 0);
                    if (IN_PLACE) {
                        a2[0][i].u = *(const u32x4*)(a_row[i] + kn);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        }
    }
    if (partial) {
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            int row = t0 + j * 16 + l16;                      // token
            if (row >= n) continue;
#pragma unroll
            for (int i = 0; i < MF; ++i) {
                int col = f0 + i * 16 + lq * 4;               // feature
                if (col < m) *(f32x4*)(partial + (size_t)row * m + col) = acc[i][j];
            }
        }
        return;
    }
    store_rows<MF, NF, BMT, BNT, THREADS>(acc, f0, t0, m, n, l16, lq, C, smem, tile_f0, tile_t0);
}

template <int BM, int BN>
struct SpmmSmem {
    static constexpr int A_PAIR = BM * 128;     // packed values of BM rows x 2 k-steps
    static constexpr int B_STAGE = BN * 128;    // BN token rows x 1 k-step
    static constexpr int B_OFF = 2 * A_PAIR;
    static constexpr int M_OFF = B_OFF + 3 * B_STAGE;
    // k-steps of a block of metadata, BM rows of 8 bytes per k-step; two blocks
    static constexpr int META_STEPS = M_OFF + 2 * BM * 64 + 1024 <= 160 * 1024 ? 8 : 4, M_BLOCK = BM * 8 * META_STEPS;
    static constexpr int DUMMY = M_OFF + 2 * M_BLOCK;  // landing zone for the metadata load of idle wavefronts
    static constexpr int TOTAL = DUMMY + 1024;
};

constexpr int SPMM_THREADS = 512;
// Wavefronts of a workgroup: RING_MULT that multiply and LOADERS that only load, in spmm_ring_kernel and on the tiles of spmm_kernel
// where four wavefronts have registers for the sums; elsewhere eight that do both.  Four have a quarter of the tile each and read a third
// fewer bytes from LDS in all, which with the loads' writes takes as long as the products (a k-step of 256 x 128: 105 KB read by eight
// wavefronts, 69 by four, at 240 bytes per cycle, 35 written at 128, against 512 cycles of products).  us, from memory, eight / four: 2048
// tokens, 4096 x 4096 on 256 x 128 42.0 / 38.7; 1500, 4352 x 4352 39.3 / 37.9; on 192 x 128 2040, 3000 x 6144 48.8 / 46.3, 3000 x 2048 21.1 / 20.0;
// 2048, 3072 x 768 12.3 / 11.9; the input gradient of 2048, 4096 x 4096 with rank 64 59.0 / 53.1.  (256 x 128 with leftover k-steps, TAIL,
// spills at the exits of its loop.)
constexpr int LOADERS = 4, RING_MULT = 4, RING_THREADS = 64 * (RING_MULT + LOADERS);
constexpr int tile_mult(int bm, int bn, bool tail) { return bm * bn <= (tail ? 192 : 256) * 128 ? RING_MULT : 8; }

// Where a row's loads of pair `pair` (of k-steps) start, in bytes of packed values.  Past the last k-step the last load of the row
// is repeated.
template <bool TAIL>
__device__ __forceinline__ int64_t pair_offset(int pair, int ksteps) {
    if (TAIL) return 2 * pair + 1 < ksteps ? (int64_t)pair * 128 : ((int64_t)ksteps - 2) * 64;
    return (int64_t)(2 * pair < ksteps ? pair : ksteps / 2 - 1) * 128;
}
// Metadata comes in blocks of STEPS k-steps, a row's 8 * STEPS bytes by as many neighbouring lanes as they have 16-byte pieces: a
// load is 64 contiguous bytes of 16 rows, or 32 of 32 rows.  One load of a wavefront (per part) is a block of 256 rows by 4 k-steps.
// The pieces of a row are exchanged by the row's upper bits, so that the sixteen rows of a 2-byte read of LDS fall on different banks.
// What loads cost is requests more than bytes, and these are a tenth of them: leaving the metadata out made the products 2 to 11 %
// faster.  us, blocks of four k-steps with a row's halves sixteen lanes apart / neighbouring lanes / blocks of eight: 2048 tokens, 4096 x
// 4096 on 256 x 128 44.0 / 43.8 / 42.7, weights from HBM 50.9 / 49.8 / 46.5; 16384, 5120 x 5120 on 256 x 256 405.5 / 404.0 / 399.1; 128
// tokens, 9216 x 9216, rank 128, in slabs 42.2 / - / 40.8.
template <int STEPS>
struct MetaLanes {
    static constexpr int PIECES = STEPS / 2, ROW = PIECES * 16, ROWS = 64 / PIECES, PARTS = STEPS / 4;
    // which piece of a row is in which place, both ways
    __device__ __forceinline__ static int swap(int row) { return row * PIECES / 16 % PIECES; }
    __device__ __forceinline__ static int piece(int lane) { return (lane % PIECES) ^ swap(lane / PIECES); }
};
#define LAST_STEP(S4) if (TAIL && ks0 + (S4) + 1 >= ksteps) break;

// TAIL: the number of k-steps is not a multiple of 4 (at least two of them).  The packed weight is fetched two k-steps at
// a time and its metadata eight or four, so at the end of a row those fetches would run past it.  They are moved back to end with
// the row instead: an odd last k-step then sits where the second step of its pair (the second 8 bytes of its 16 of
// metadata) belongs, and that is where it is read.  A template parameter, so that whole quads pay nothing for it.
//
// SplitJob: the k range is cut into slabs of slab_steps k-steps (whole quads), which leave fp32 partial sums in slabs[slab].
// The (tile, slab) pairs are dealt to the XCDs in equal shares, slab by slab (a slab's tiles share its tokens in L2): an
// eighth of every slab's tiles where that is a whole number, else eight equal runs of all pairs,
// the token tiles of a weight tile side by side.  A grid with the slabs in blockIdx.y gave 36 tiles per slab to seven of
// the XCDs, five each, and one to the last (128 tokens, 9216 x 9216: 33.6 -> 27.7 us).
// Such a launch may have workgroups of a second kind: they compute the sums of T = X L (see xl_split_kernel) that the
// kernel after this one needs, on compute units that the product leaves idle.
struct SplitJob {
    int nslabs, slab_steps;
    float* slabs;
    const bf16_t* L;                                          // or null
    float* Q;
    int r, k_per, xl_slabs;
};

// What a workgroup of a split launch does: its tile and slab, the slab that adds the dense extension, true; or a part of X L
// (done here) or nothing, false.
__device__ __forceinline__ bool split_item(const SplitJob& job, const bf16_t* __restrict__ B, int n, int K, int tiles_m, int tiles_n,
                                           uint8_t* smem, int& tm, int& tn, int& slab, int& extension_slab) {
    const int tiles = tiles_m * tiles_n, run = (tiles * job.nslabs + XCDS - 1) / XCDS;
    const int xcd = (int)blockIdx.x % XCDS, pos = (int)blockIdx.x / XCDS;
    if (pos >= run) {
        const int id = (pos - run) * XCDS + xcd;
        const int xl_tiles_r = (job.r + SK_BJ - 1) / SK_BJ, xl_tiles = xl_tiles_r * ((n + SK_BI - 1) / SK_BI);
        const int part = id / xl_tiles, tile = id % xl_tiles;
        if (part < job.xl_slabs)
            skinny_tile<false, true>(B, K, job.L, job.r, n, job.r, part * (uint32_t)job.k_per,
                                     min((uint32_t)K, (part + 1) * (uint32_t)job.k_per), tile / xl_tiles_r * SK_BI,
                                     tile % xl_tiles_r * SK_BJ, nullptr, job.Q + (size_t)part * n * job.r, smem);
        return false;
    }
    int tile;
    if (tiles % XCDS == 0) {
        slab = pos / (tiles / XCDS);
        tile = xcd * (tiles / XCDS) + pos % (tiles / XCDS);
    } else {
        const int item = xcd * run + pos;
        if (item >= tiles * job.nslabs) return false;
        slab = item / tiles;
        tile = item % tiles;
    }
    // the extension is added once: by the first slab if every XCD has its share of that (its workgroups start first), else
    // by a slab that depends on the tile
    extension_slab = tiles % XCDS == 0 ? 0 : tile % job.nslabs;
    tn = tile % tiles_n;
    tm = tile / tiles_n;
    return true;
}

// The 256 x 256 tiles left over after the whole rounds of a wide grid, positions first .. first + count - 1 of its order, as
// tiles of BM x BN that divide them.  An XCD gets an equal run of them, the parts of one side by side.
struct Leftover { int first, count, tiles_m, tiles_n; };
template <int BM, int BN>
__host__ __device__ inline bool leftover_tile(int block, const Leftover& left, int& tm, int& tn) {
    constexpr int PM = 256 / BM, PN = 256 / BN;
    const int run = (left.count + XCDS - 1) / XCDS, slot = block / XCDS, part = slot % (PM * PN);
    const int mine = slot / (PM * PN), tile = block % XCDS * run + mine;
    if (mine >= run || tile >= left.count) return false;
    tile_of_position(left.first + tile, left.tiles_m, left.tiles_n, tm, tn);
    tm = tm * PM + part % PM;
    tn = tn * PN + part / PM;
    return true;
}
template <int BM, int BN>
inline int leftover_grid(const Leftover& left) { return (left.count + XCDS - 1) / XCDS * XCDS * (256 / BM) * (256 / BN); }

// What a launch of a tile kernel is: a whole product, one split over k (SplitJob), or a wide grid's leftover tiles (Leftover).  Each
// has only its own arguments: with all of them in one kernel whole products of a few us took 0.2 us longer, for a further
// read of arguments before the first load (2 to 4 %: 447 tokens, 2168 x 128 4.46 us, 559, 3960 x 128 5.78 -> 6.04).
struct WholeJob {};
template <class Job> constexpr bool is_split = std::is_same<Job, SplitJob>::value;

// The workgroup's tile of a launch that is not split; false: none
template <int BM, int BN>
__device__ __forceinline__ bool tile_of(const WholeJob&, int m, int n, int tiles_m, int tiles_n, int& tm, int& tn) {
    return tile_of_block(tiles_m, tiles_n, tm, tn);
}
template <int BM, int BN>
__device__ __forceinline__ bool tile_of(const Leftover& left, int m, int n, int tiles_m, int tiles_n, int& tm, int& tn) {
    return leftover_tile<BM, BN>((int)blockIdx.x, left, tm, tn) && tm * BM < m && tn * BN < n;   // (parts past the edge of a ragged tile)
}

// The loads of spmm_kernel, by all eight wavefronts (ALL) or by LOADERS of them.
template <int BM, int BN, bool TAIL, bool ALL>
struct SpmmLoads {
    using S = SpmmSmem<BM, BN>;
    using ML = MetaLanes<S::META_STEPS>;
    static constexpr int LW = ALL ? 8 : LOADERS, A_LD = BM / (8 * LW), B_LD = BN / (8 * LW);   // 1 KiB loads per wavefront: per pair, per step
    static constexpr int M_LD = 8 / LW, M_ALL = ML::PARTS * M_LD;                             // per quad of k-steps, per block of metadata
    static constexpr int step_loads(int S4) { return B_LD + (S4 & 1) * A_LD + (S4 == 0) * M_LD; }
    const uint8_t* a_src[A_LD];
    const uint8_t* b_src[B_LD];
    const uint8_t* m_src[M_ALL];
    int m_dst[M_ALL], m_dst_step[M_ALL];                      // (rows the tile does not have land in the dummy, all from one place)
    int ksteps, loader, m_piece;
    uint8_t* smem;

    // loader lanes: 8 lanes per row, chunk rotated by (row / 2) % 8
    __device__ __forceinline__ void init(const bf16_t* B, int n, const bf16_t* Av, const uint8_t* Am, int m, int K, int m0, int n0,
                                         int k_first, int steps, int wave, int lane, uint8_t* lds) {
        ksteps = steps;
        loader = wave;
        smem = lds;
        m_piece = ML::piece(lane) * 16;
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            const int rl = (loader * A_LD + i) * 8 + (lane >> 3);     // row inside the tile
            a_src[i] = (const uint8_t*)Av + (size_t)wrap_row(m0 + rl, m) * K + (((lane & 7) ^ ((rl >> 1) & 7)) * 16) + (size_t)k_first * 64;
        }
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            const int rl = (loader * B_LD + i) * 8 + (lane >> 3);
            b_src[i] = (const uint8_t*)B + (size_t)wrap_row(n0 + rl, n) * K * 2 + (((lane & 7) ^ ((rl >> 1) & 7)) * 16) + (size_t)k_first * 128;
        }
#pragma unroll
        for (int p = 0; p < M_ALL; ++p) {
            const int rl = (p * LW + loader) * ML::ROWS;
            const bool has = rl < BM;                         // wave-uniform
            m_src[p] = Am + (size_t)(has ? wrap_row(m0 + rl + lane / ML::PIECES, m) : 0) * (K / 8) + (size_t)k_first * 8;
            m_dst[p] = has ? S::M_OFF + (p * LW + loader) * 1024 : S::DUMMY;
            m_dst_step[p] = has ? S::M_BLOCK : 0;
        }
    }
    __device__ __forceinline__ void tokens(int64_t off, int stage, int i) const {
        dma16(b_src[i] + off, smem + S::B_OFF + stage * S::B_STAGE + (loader * B_LD + i) * 1024);
    }
    __device__ __forceinline__ void weights(int64_t off, int buf, int i) const {
        dma16(a_src[i] + off, smem + buf * S::A_PAIR + (loader * A_LD + i) * 1024);
    }
    __device__ __forceinline__ void metadata(int block, int p) const {       // of k-steps META_STEPS * block ..
        const int off = block * ML::ROW + m_piece, last = ksteps * 8 - 16;
        dma16(m_src[p] + (off < last ? off : last), smem + m_dst[p] + (block & 1) * m_dst_step[p]);
    }
    // what the k-steps before the first would have queued; not by all: the tokens of the first two are left to the other wavefronts
    __device__ __forceinline__ void first() const {
#pragma unroll
        for (int p = 0; p < M_ALL; ++p) metadata(0, p);
        auto pair = [&](int p) {
#pragma unroll
            for (int i = 0; i < A_LD; ++i) weights(pair_offset<TAIL>(p, ksteps), p, i);
        };
        auto step = [&](int ks) {
#pragma unroll
            for (int i = 0; i < B_LD; ++i) tokens((int64_t)(ks < ksteps ? ks : ksteps - 1) * 128, ks, i);
        };
        pair(0);
        if (ALL) {
            step(0);
            step(1);
        }
        pair(1);
        step(2);
    }
    // Load x of step ks, S4 = ks % 4: what refills the buffers that it has left, `stage` of them the tokens', by k-step ks + 3 and the
    // pair after the next one, and a part of the next block of metadata.
    __device__ __forceinline__ int64_t b_offset(int ks) const { return (int64_t)(ks + 3 < ksteps ? ks + 3 : ksteps - 1) * 128; }
    __device__ __forceinline__ int64_t a_offset(int ks, int S4) const { return (S4 & 1) ? pair_offset<TAIL>((ks >> 1) + 2, ksteps) : 0; }
    __device__ __forceinline__ void one(int ks, int S4, int stage, int64_t b_off, int64_t a_off, int x) const {
        if (x < B_LD) tokens(b_off, stage, x);
        else if (S4 & 1) weights(a_off, S4 >> 1, x - B_LD);
        else if (ML::PARTS == 1 || (ks >> 2 & 1) == 0) metadata((ks >> 2) / ML::PARTS + 1, x - B_LD);
        else metadata((ks >> 2) / ML::PARTS + 1, M_ALL - M_LD + x - B_LD);
    }
};

template <int BM, int BN, bool TAIL, class Job>
__global__ void __launch_bounds__(SPMM_THREADS) spmm_kernel(const bf16_t* __restrict__ B, int n,
                                                            const bf16_t* __restrict__ Av,
                                                            const uint8_t* __restrict__ Am, int m, int K,
                                                            const bf16_t* __restrict__ B2,
                                                            const bf16_t* __restrict__ A2, int K2,
                                                            bf16_t* __restrict__ C, int tiles_m, int tiles_n,
                                                            Job job) {
    using S = SpmmSmem<BM, BN>;
    constexpr int MULT = tile_mult(BM, BN, TAIL);                // wavefronts that multiply
    constexpr bool OWN = MULT == 8;                          // all load as well, or LOADERS more do
    constexpr int MF = BM / 32, NF = BN / (8 * MULT);        // 16 x 16 fragments per wavefront
    using Loads = SpmmLoads<BM, BN, TAIL, OWN>;
    using ML = typename Loads::ML;
    extern __shared__ __align__(16) uint8_t smem[];
    fetch_arguments(B, n, Av, Am, m, K, tiles_m, tiles_n);

    int tm, tn, slab = 0, extension_slab = 0;
    if constexpr (is_split<Job>) {
        static_assert(SPMM_THREADS == SK_WAVES * 64 && RING_THREADS == SPMM_THREADS && SK_LDS <= S::TOTAL, "a skinny tile fits in the workgroup");
        if (!split_item(job, B, n, K, tiles_m, tiles_n, smem, tm, tn, slab, extension_slab)) return;
    } else {
        if (!tile_of<BM, BN>(job, m, n, tiles_m, tiles_n, tm, tn)) return;
    }
    const int m0 = tm * BM, n0 = tn * BN;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int l16 = lane & 15, lq = lane >> 4;

    int k_first = 0, slab_steps = K / 64;
    float* sums = nullptr;
    if constexpr (is_split<Job>) {
        slab_steps = job.slab_steps;
        k_first = slab * slab_steps;                          // a multiple of 4
        sums = job.slabs + (size_t)slab * (size_t)n * (size_t)m;
    }
    // a multiple of 4 unless TAIL
    const int ksteps = K / 64 - k_first > slab_steps ? slab_steps : K / 64 - k_first;

    // ---- reader lanes: fragment f = rows 16f .. 16f+15 = 2 KiB; lane (l16, lq) wants chunk 4h + lq
    const int sw = (l16 >> 1) & 7;
    const int rd0 = l16 * 128 + ((lq ^ sw) * 16);             // h = 0
    const int rd1 = l16 * 128 + (((4 + lq) ^ sw) * 16);       // h = 1
    const int a_rd = (wm * MF) * 2048;
    const int b_rd = S::B_OFF + (wn * NF) * 2048;
    const int m_rd = S::M_OFF + (wm * MF * 16 + l16) * ML::ROW + lq * 2, m_sw = ML::swap(l16) * 16;

    if constexpr (!OWN) {
        if (wave >= MULT) {                                   // (its barriers are those of the others)
            Loads load;
            load.init(B, n, Av, Am, m, K, m0, n0, k_first, ksteps, wave - MULT, lane, smem);
            load.first();
            WAIT_HERE(waitcnt_imm(Loads::A_LD + Loads::B_LD, 15));
            wg_barrier();
            wg_barrier();
            int stage = 0;
            auto step = [&](int ks, auto s4) {
                constexpr int S4 = decltype(s4)::value, LOADS = Loads::step_loads(S4);
                if (ks + 3 < ksteps) {
                    const int64_t b_off = load.b_offset(ks), a_off = load.a_offset(ks, S4);
#pragma unroll
                    for (int x = 0; x < LOADS; ++x) load.one(ks, S4, stage, b_off, a_off, x);
                    WAIT_HERE(waitcnt_imm(LOADS, 15));
                } else {                                      // nothing of what the last three k-steps would load is used
                    WAIT_HERE(waitcnt_imm(0, 15));
                }
                wg_barrier();
                stage = stage == 2 ? 0 : stage + 1;
            };
            for (int ks0 = 0; ks0 < ksteps; ks0 += 4) {
                step(ks0, std::integral_constant<int, 0>{});
                LAST_STEP(0)
                step(ks0 + 1, std::integral_constant<int, 1>{});
                LAST_STEP(1)
                step(ks0 + 2, std::integral_constant<int, 2>{});
                LAST_STEP(2)
                step(ks0 + 3, std::integral_constant<int, 3>{});
            }
            if (K2 < 0 && slab == extension_slab) stage_factor<BM, 64 * LOADERS>(A2, K2, m, smem, m0, t - 64 * MULT);
            return;
        }
    }
    Loads load;
    if constexpr (OWN) load.init(B, n, Av, Am, m, K, m0, n0, k_first, ksteps, wave, lane, smem);

    f32x4 acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

    struct Frags {                                            // of a k-step
        BFrag bf[NF];
        AFrag af[MF];
        int ai[MF];
    };
    // fragment x (the tokens' first) of k-step ks, with S4 = ks % 4 and its tokens in stage `bst`
    auto read_one = [&](Frags& f, int ks, int S4, int bst, int x) {
        if (x < NF) {
            const uint8_t* const pb = smem + b_rd + bst * S::B_STAGE + x * 2048;
            f.bf[x].u[0] = *(const u32x4*)(pb + rd0);
            f.bf[x].u[1] = *(const u32x4*)(pb + rd1);
        } else {
            const bool second = (S4 & 1) != 0 || (TAIL && ks == ksteps - 1);
            const int i = x - NF;
            f.af[i].u = *(const u32x4*)(smem + ((S4 >> 1) & 1) * S::A_PAIR + a_rd + i * 2048 + (second ? rd1 : rd0));
            const int piece = ((S4 >> 1) + (ML::PARTS == 2 ? (ks >> 2 & 1) * 2 : 0)) * 16;
            f.ai[i] = *(const uint16_t*)(smem + m_rd + (ks / S::META_STEPS & 1) * S::M_BLOCK + (piece ^ m_sw) + i * 16 * ML::ROW + (second ? 8 : 0));
        }
    };

    if constexpr (OWN) {
        load.first();
        WAIT_HERE(waitcnt_imm(Loads::A_LD + 2 * Loads::B_LD, 15));
    } else {                                                  // the tokens of the first two k-steps, which the loaders leave out
        constexpr int T_LD = BN / (8 * MULT);
#pragma unroll
        for (int i = 0; i < 2 * T_LD; ++i) {
            const int g = wave * T_LD + i % T_LD, rl = g * 8 + (lane >> 3), step = i / T_LD;
            const int kc = TAIL && step >= ksteps ? 0 : step;    // one k-step: again rather than past the row's end
            dma16((const uint8_t*)B + (size_t)wrap_row_near(n0 + rl, n) * K * 2 + (((lane & 7) ^ ((rl >> 1) & 7)) * 16) + (size_t)(k_first + kc) * 128,
                  smem + S::B_OFF + step * S::B_STAGE + g * 1024);
        }
        WAIT_HERE(waitcnt_imm(T_LD, 15));
    }
    wg_barrier();
    Frags f;
#pragma unroll
    for (int x = 0; x < MF + NF; ++x) read_one(f, 0, 0, 0, x);
    WAIT_HERE(waitcnt_imm(OWN ? Loads::A_LD + Loads::B_LD : 0, 0));
    wg_barrier();

    // One k-step, its fragments in registers: everybody has read it from LDS, the next one has landed.  Spread among its products
    // are the loads that refill the buffers it has left, first, since the k-step after the next one waits for them (last: up to 5 %
    // slower), and the reads of the next k-step's fragments: tokens, and a row of weights after the products of the same row, in
    // whose registers it can be.  S4 = ks % 4 is a literal so that the number of loads queued, which the wait at the end has to leave
    // outstanding, is a constant.
    int bst = 0;                                              // ring stage of the current k-step
    auto step = [&](int ks, auto s4) {
        constexpr int S4 = decltype(s4)::value, N4 = (S4 + 1) & 3;
        constexpr int LOADS = OWN ? Loads::step_loads(S4) : 0, EARLY = NF + LOADS, SLOTS = MF * NF, PER = (EARLY + SLOTS - 1) / SLOTS;
        const int next = bst == 2 ? 0 : bst + 1;
        const int64_t b_off = OWN ? load.b_offset(ks) : 0, a_off = OWN ? load.a_offset(ks, S4) : 0;
        Frags g;
#pragma unroll
        for (int i = 0; i < MF; ++i) {
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                acc[i][j] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(f.af[i].v, f.bf[j].v, acc[i][j], f.ai[i], 0, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int x = (i * NF + j) * PER; x < (i * NF + j + 1) * PER; ++x) {
                    if (x < LOADS) load.one(ks, S4, bst, b_off, a_off, x);
                    else if (x < EARLY) read_one(g, ks + 1, N4, next, x - LOADS);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            read_one(g, ks + 1, N4, next, NF + i);
            __builtin_amdgcn_sched_barrier(0);
        }
        WAIT_HERE(waitcnt_imm(OWN ? LOADS : 63, 0));
        wg_barrier();
        f = g;
        bst = next;
    };
    for (int ks0 = 0; ks0 < ksteps; ks0 += 4) {
        step(ks0, std::integral_constant<int, 0>{});
        LAST_STEP(0)
        step(ks0 + 1, std::integral_constant<int, 1>{});
        LAST_STEP(1)
        step(ks0 + 2, std::integral_constant<int, 2>{});
        LAST_STEP(2)
        step(ks0 + 3, std::integral_constant<int, 3>{});
    }
    if (OWN) WAIT_HERE(waitcnt_imm(0, 15));  // drain the clamped look-ahead loads

    static_assert(BN * (BM * 2 + 16) <= S::TOTAL, "the staged output tile fits in the rings");
    int te = threadIdx.x;                                    // (the lane's coordinates again rather than kept across the loop)
    if (!OWN) asm volatile("" : "+v"(te));
    const int we = __builtin_amdgcn_readfirstlane(te >> 6);
    extend_and_store<MF, NF, BM, BN, 64 * MULT, !OWN>(acc, m0 + (we & 1) * MF * 16, n0 + (we >> 1) * NF * 16, m, n, te & 15, te >> 4 & 3, B2, A2,
                                                slab == extension_slab ? K2 : 0, C, smem, m0, n0, sums);
}

// ------------------------------------------------------------------------------------------
// spmm_split_kernel: the 256 x 256 tile.  A fifth fewer operand bytes per flop than the
// 192 x 256 tile, but a ring of three B stages no longer fits beside it.  The two wavefront groups
// own the two token halves of the tile, so each half of a B stage is private to one group and free
// again as soon as that group has read it; two stages per half then give every load the same two
// to three phases (half k-steps) of flight that the shared ring of three gave:
//     A pair buffers 2 x 32 KiB | B half of group 0  2 x 16 KiB | of group 1  2 x 16 KiB | metadata 2 x 16 KiB
// Queued by every wavefront, k = k-step, phases 2k (group 0 reads step k) and 2k + 1 (group 1 does):
//     phase 2k     : B1(k+1);  lower half of A pair k/2 + 1 if k is even;  half of the metadata block of k/8 + 1 if k % 4 == 1
//     phase 2k + 1 : B0(k+2);  upper half of A pair k/2 + 1 if k is even
// and at the end of each phase a wavefront waits for everything it queued two or more phases ago,
// which covers all that the next phase reads.  Every buffer is rewritten in the first phase after
// the barrier that ends its last reader's phase.
struct SplitSmem {
    static constexpr int BM = 256, BN = 256;
    static constexpr int A_PAIR = BM * 128, B_HALF = BN / 2 * 128, M_BLOCK = BM * 64;   // metadata: 8 k-steps
    static constexpr int B_OFF = 2 * A_PAIR;                  // then [group][stage] halves of B
    static constexpr int M_OFF = B_OFF + 4 * B_HALF;
    static constexpr int TOTAL = M_OFF + 2 * M_BLOCK;
};

// loads one wavefront queues in the even / odd phase of k-step k (k taken mod 4)
constexpr int split_even(int k) { return 2 + ((k & 1) == 0 ? 2 : 0) + ((k & 3) == 1 ? 1 : 0); }
constexpr int split_odd(int k) { return 2 + ((k & 1) == 0 ? 2 : 0); }

template <bool PREFETCH, bool TAIL>
__global__ void __launch_bounds__(SPMM_THREADS) spmm_split_kernel(const bf16_t* __restrict__ B, int n,
                                                                  const bf16_t* __restrict__ Av,
                                                                  const uint8_t* __restrict__ Am, int m, int K,
                                                                  const bf16_t* __restrict__ B2,
                                                                  const bf16_t* __restrict__ A2, int K2,
                                                                  bf16_t* __restrict__ C, int tiles_m, int tiles_n) {
    using S = SplitSmem;
    constexpr int MF = 8, NF = 4;                            // wavefront tile 128 features x 64 tokens
    extern __shared__ __align__(16) uint8_t smem[];

    int tm, tn;
    if (!tile_of_block(tiles_m, tiles_n, tm, tn)) return;
    const int m0 = tm * S::BM, n0 = tn * S::BN;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int group = wave >> 2;                             // = token half of the tile
    const int wm = wave & 1, wn = wave >> 1;
    const int l16 = lane & 15, lq = lane >> 4;

    // ---- loader lanes: 8 lanes per row, chunk rotated by (row / 2) % 8.  A half of A and a half of
    //      B are 16 loads of 8 rows each: two per wavefront.
    const uint8_t* a_src[4];                                 // [half * 2 + i]
    const uint8_t* b_src[4];                                 // [group * 2 + i]
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int rl = ((q >> 1) * 16 + wave * 2 + (q & 1)) * 8 + (lane >> 3);     // row inside the tile
        int sw16 = ((lane & 7) ^ ((rl >> 1) & 7)) * 16;
        int ra = wrap_row(m0 + rl, m);
        int rb = wrap_row(n0 + rl, n);
        a_src[q] = (const uint8_t*)Av + (size_t)ra * K + sw16;
        b_src[q] = (const uint8_t*)B + (size_t)rb * K * 2 + sw16;
    }
    using ML = MetaLanes<8>;
    const uint8_t* m_src[2];                                 // 16 rows per wavefront and part
#pragma unroll
    for (int p = 0; p < 2; ++p)
        m_src[p] = Am + (size_t)wrap_row(m0 + (p * 8 + wave) * 16 + lane / ML::PIECES, m) * (K / 8);
    const int m_piece = ML::piece(lane) * 16;

    // ---- L2 prefetch of the token panel through the scalar cache.  A compute unit holds about 128 vector-memory
    //      requests of 128 bytes in flight, so its operand feed is that many lines per mean latency, and the
    //      latency is set by the lines that miss the XCD's L2 (a sixth of them, compulsory: each operand panel
    //      enters the L2 once per chunk of 8 x 4 tiles), on which all tiles that share the panel wait together.
    //      Scalar loads take another path into the same L2.  The 8 tiles of a chunk that share a token panel
    //      each touch an eighth of its rows PF_AHEAD k-steps ahead (4 rows per wavefront, both 64-byte halves of
    //      a row's 128 bytes: the L2 fills halves), so the vector loads of the token panel hit: 3-6 % on the
    //      whole product at OPT-66B sizes.  The scalar path takes about 70 such requests per microsecond and compute unit, which
    //      these 64 per k-step use up; touching only part of the panel, or the weight panels instead, gained
    //      nothing.  The loaded dwords are not used; they stay allocated until the wavefront's next
    //      s_waitcnt lgkmcnt(0), since a scalar load may return any time before that.
    constexpr int PF_AHEAD = 6, PF_ROWS = S::BN / CHUNK_M / 8;
    const uint8_t* pf_row[PF_ROWS];
#pragma unroll
    for (int r = 0; r < PF_ROWS; ++r) {
        int row = wrap_row(n0 + (tm % CHUNK_M) * (S::BN / CHUNK_M) + wave * PF_ROWS + r, n);
        pf_row[r] = (const uint8_t*)B + (size_t)row * K * 2;
    }
    // PREFETCH is the host's choice (launch_split): only for grids in the chunked order, and only if the tokens do
    // not fit into the last-level cache: lines that come from there rather than from HBM arrive soon enough anyway,
    // and the scalar loads then cost more than they gain (measured: 1-5 % faster with 16384 tokens of 9216 features
    // or more, 3-12 % slower with 8192 tokens or fewer).  It is a template parameter because a branch around the
    // loads inside the k-loop cost what they gain.  Tiles outside whole chunks, up to 11 rows and 7 columns of them, touch rows as if they
    // were in one, so that some rows of their panels are touched more than once and some not at all.  (us, without / with, grids with such strips: 16384 tokens,
    // 4352 x 10240 748 / 695; 16640, 4608 x 9216 714 / 667; 12544, 4352 x 16384 893 / 884; 44 products of 4096 to 10496 rows 1 to 10 % faster.)
    uint32_t pf[2 * PF_ROWS];
#pragma unroll
    for (int r = 0; r < 2 * PF_ROWS; ++r) pf[r] = 0;
    // to be placed right after an s_waitcnt lgkmcnt(0): retires the previous k-step's loads, issues the next
#define PF_ISSUE(ks)                                                                                   \
    {                                                                                                  \
        _Pragma("unroll") for (int r = 0; r < 2 * PF_ROWS; ++r) asm volatile("" ::"s"(pf[r]));         \
        const int kpf = (ks) + PF_AHEAD < ksteps ? (ks) + PF_AHEAD : ksteps - 1;                       \
        const uint32_t off = (uint32_t)kpf * 128u;            /* inside the row: K * 2 bytes, K < 2^31 */ \
        if (PREFETCH) {                                                                                \
            _Pragma("unroll") for (int r = 0; r < PF_ROWS; ++r) {                                      \
                asm volatile("s_load_dword %0, %1, %2" : "=s"(pf[2 * r]) : "s"(pf_row[r]), "s"(off));   \
                asm volatile("s_load_dword %0, %1, %2" : "=s"(pf[2 * r + 1]) : "s"(pf_row[r]), "s"(off + 64u)); \
            }                                                                                          \
        }                                                                                              \
    }
    // ---- reader lanes: fragment f = rows 16f .. 16f+15 = 2 KiB; lane (l16, lq) wants chunk 4h + lq
    const int sw = (l16 >> 1) & 7;
    const int rd0 = l16 * 128 + ((lq ^ sw) * 16);             // h = 0
    const int rd1 = l16 * 128 + (((4 + lq) ^ sw) * 16);       // h = 1
    const int a_rd = (wm * MF) * 2048;
    const int b_rd = S::B_OFF + group * 2 * S::B_HALF + ((wn & 1) * NF) * 2048;
    const int m_rd = S::M_OFF + (wm * MF * 16 + l16) * ML::ROW + lq * 2, m_sw = ML::swap(l16) * 16;

    const int ksteps = K / 64;                                // a multiple of 4 unless TAIL (see spmm_kernel)
    auto issue_b = [&](int g, int ks) {                       // token half g of k-step ks (clamped)
        int kc = ks < ksteps ? ks : ksteps - 1;
        uint8_t* st = smem + S::B_OFF + (g * 2 + (ks & 1)) * S::B_HALF + (wave * 2) * 1024;
        dma16(b_src[g * 2] + (size_t)kc * 128, st);
        dma16(b_src[g * 2 + 1] + (size_t)kc * 128, st + 1024);
    };
    auto issue_a = [&](int half, int pair) {                  // weight rows 128 half .. +127, k-steps 2 pair, 2 pair + 1
        const int64_t off = pair_offset<TAIL>(pair, ksteps);
        uint8_t* st = smem + (pair & 1) * S::A_PAIR + (half * 16 + wave * 2) * 1024;
        dma16(a_src[half * 2] + off, st);
        dma16(a_src[half * 2 + 1] + off, st + 1024);
    };
    auto issue_m = [&](int block, int part) {                 // metadata of k-steps 8 block .. 8 block + 7, half of the rows
        const int off = block * 64 + m_piece, last = ksteps * 8 - 16;
        dma16((part ? m_src[1] : m_src[0]) + (off < last ? off : last), smem + S::M_OFF + (block & 1) * S::M_BLOCK + (part * 8 + wave) * 1024);
    };

    f32x4 acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // S4 = k % 4 is a literal, so the number of loads a wait may leave in flight is a constant.
#define EVEN_LOADS(k, S4)                                                                              \
    {                                                                                                  \
        issue_b(1, (k) + 1);                                                                           \
        if (((S4) & 1) == 0) issue_a(0, ((k) >> 1) + 1);                                               \
        if (((S4) & 3) == 1) issue_m(((k) >> 3) + 1, ((k) >> 2) & 1);                                  \
    }
#define ODD_LOADS(k, S4)                                                                               \
    {                                                                                                  \
        issue_b(0, (k) + 2);                                                                           \
        if (((S4) & 1) == 0) issue_a(1, ((k) >> 1) + 1);                                               \
    }
#define SPLIT_READ(S4)                                                                                 \
        const bool second = ((S4) & 1) != 0 || (TAIL && ks == ksteps - 1);                             \
        const uint8_t* pa = smem + (((S4) >> 1) & 1) * S::A_PAIR + a_rd + (second ? rd1 : rd0);        \
        const uint8_t* pb = smem + b_rd + ((S4) & 1) * S::B_HALF;                                      \
        const uint8_t* pm = smem + m_rd + ((ks0 >> 3) & 1) * S::M_BLOCK + (((((S4) >> 1) + (ks0 >> 1 & 2)) * 16) ^ m_sw) + (second ? 8 : 0); \
        BFrag bf[NF];                                                                                  \
        AFrag af[MF];                                                                                  \
        int ai[MF];                                                                                    \
        _Pragma("unroll") for (int j = 0; j < NF; ++j) {                                               \
            bf[j].u[0] = *(const u32x4*)(pb + j * 2048 + rd0);                                         \
            bf[j].u[1] = *(const u32x4*)(pb + j * 2048 + rd1);                                         \
        }                                                                                              \
        _Pragma("unroll") for (int i = 0; i < MF; ++i) {                                               \
            af[i].u = *(const u32x4*)(pa + i * 2048);                                                  \
            ai[i] = *(const uint16_t*)(pm + i * 16 * ML::ROW);                                         \
        }
#define SPLIT_MFMA                                                                                     \
        _Pragma("unroll") for (int i = 0; i < MF; ++i) _Pragma("unroll") for (int j = 0; j < NF; ++j)  \
            acc[i][j] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(af[i].v, bf[j].v, acc[i][j], ai[i], 0, 0);
    // group 0: phase 2k reads step k, phase 2k + 1 multiplies it
#define SPLIT_STEP0(S4)                                                                                \
    {                                                                                                  \
        const int ks = ks0 + (S4);                                                                     \
        SPLIT_READ(S4)                                                                                 \
        EVEN_LOADS(ks, S4)                                                                             \
        WAIT_HERE(waitcnt_imm(split_even(S4) + split_odd((S4) + 3), 0));                               \
        PF_ISSUE(ks)                                                                                   \
        wg_barrier();                                                                                  \
        ODD_LOADS(ks, S4)                                                                              \
        SPLIT_MFMA                                                                                     \
        WAIT_HERE(waitcnt_imm(split_odd(S4) + split_even(S4), 15));                                    \
        wg_barrier();                                                                                  \
    }
    // group 1: phase 2k + 1 reads step k, phase 2k + 2 multiplies it
#define SPLIT_STEP1(S4)                                                                                \
    {                                                                                                  \
        const int ks = ks0 + (S4);                                                                     \
        SPLIT_READ(S4)                                                                                 \
        ODD_LOADS(ks, S4)                                                                              \
        WAIT_HERE(waitcnt_imm(split_odd(S4) + split_even(S4), 0));                                     \
        PF_ISSUE(ks)                                                                                   \
        wg_barrier();                                                                                  \
        EVEN_LOADS(ks + 1, (S4) + 1)                                                                   \
        SPLIT_MFMA                                                                                     \
        WAIT_HERE(waitcnt_imm(split_even((S4) + 1) + split_odd(S4), 15));                              \
        wg_barrier();                                                                                  \
    }

    // ---- prologue: what the schedule would have queued in the phases before phase 0
    issue_m(0, 0); issue_m(0, 1);
    issue_a(0, 0); issue_a(1, 0); issue_b(0, 0);
    issue_b(1, 0);
    issue_b(0, 1);                                            // = the odd phase of step -1
    WAIT_HERE(waitcnt_imm(4, 15));                            // metadata, A pair 0 and B0(0) have landed
    wg_barrier();
    if (group == 0) {
        for (int ks0 = 0; ks0 < ksteps; ks0 += 4) {
            SPLIT_STEP0(0) LAST_STEP(0) SPLIT_STEP0(1) LAST_STEP(1) SPLIT_STEP0(2) LAST_STEP(2) SPLIT_STEP0(3)
        }
        wg_barrier();                                         // group 1's last compute phase
    } else {
        EVEN_LOADS(0, 0)                                      // phase 0: nothing to multiply yet
        WAIT_HERE(waitcnt_imm(split_even(0) + split_odd(3), 15));
        wg_barrier();
        for (int ks0 = 0; ks0 < ksteps; ks0 += 4) {
            SPLIT_STEP1(0) LAST_STEP(0) SPLIT_STEP1(1) LAST_STEP(1) SPLIT_STEP1(2) LAST_STEP(2) SPLIT_STEP1(3)
        }
    }
#undef EVEN_LOADS
#undef ODD_LOADS
#undef SPLIT_READ
#undef SPLIT_MFMA
#undef SPLIT_STEP0
#undef SPLIT_STEP1
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // the last scalar prefetches have returned
#pragma unroll
    for (int r = 0; r < 2 * PF_ROWS; ++r) asm volatile("" ::"s"(pf[r]));
#undef PF_ISSUE
    WAIT_HERE(waitcnt_imm(0, 15));                            // drain the clamped look-ahead loads
    static_assert(S::BN * (S::BM * 2 + 16) <= S::TOTAL, "the staged output tile fits in the rings");
    extend_and_store<MF, NF, S::BM, S::BN, SPMM_THREADS>(acc, m0 + wm * MF * 16, n0 + wn * NF * 16, m, n, l16, lq, B2, A2, K2, C, smem,
                                           m0, n0);
}

// ------------------------------------------------------------------------------------------
// spmm_ring_kernel: the smaller tiles, one barrier per pair of k-steps.  A tile of 128 x 64 gives a wavefront four MFMAs
// per k-step, so a barrier per k-step, as above, would cost more than the k-step's loads (two of them took 0.35 us per
// k-step beside what its loads take).  Here a ring stage holds a pair of k-steps of both operands (the packed values come in
// pairs anyway, 128 bytes per row).  Four wavefronts, per pair, read the second k-step's fragments, multiply the first, pass the barrier,
// read the next pair's first k-step and multiply the second, so that no product waits for the reads of its own k-step.
// Four more, one per SIMD as well, only load: wait for their loads of the next pair, pass the barrier and queue the loads that refill the
// stage everybody has left.  Three to four stages keep two or three pairs (34 to 50 KB each) on the way, and the operand feed
// bounds the kernel.
// A wavefront that queues loads stands still until the address unit, 64 bytes per cycle for the whole compute unit, has taken them: where
// the multiplying ones did it, after the barrier, the last of them began their products some hundred cycles late (1000 tokens, 4352 x
// 4352: of 940 cycles per k-step four of the wavefronts spent 390 at the barrier, waiting for the other four; 50 for loads).  us, operands
// in the last-level cache and from HBM, eight that load and multiply / eight that multiply and four that load: 700 tokens, 4160 x 2112 on
// 192 x 64 17.0 / 15.1 and 17.1 / 15.3; 1000, 4352 x 4352 on 192 x 96 32.4 / 29.1 and 37.5 / 35.4; 1500, 2040 x 4096 on 128 x 96 22.2 / 20.1 and
// 22.3 / 20.3; 2048, 768 x 3072 on 128 x 64 13.2 / 12.5.  Two loaders: 2 to 7 % slower than four; four of higher priority: 0 to 4 %.  In the
// kernel above, whose loads are spread among its products, loaders beside eight that multiply gain nothing; see tile_mult for those beside four.
// Four that multiply have a quarter of the tile each, a third fewer bytes from LDS in all than eight, and the workgroup starts faster (us, from
// memory, eight / four and four loaders: 1000 tokens, 4352 x 4352 30.4 / 29.7; 1114, 704 x 1600 9.9 / 9.5; 875, 1536 x 768 6.8 / 6.6, without
// loaders 6.7; 2000, 1920 x 2048 15.4 / 15.1; 424, 1792 x 3584 in slabs 14.4 / 14.2; 300, 9216 x 4096 20.9 / 21.5).
// (Reads a k-step ahead of their products, against products that follow their reads: 2048 tokens, 768 x 3072 on 128 x 64 16.9
// -> 15.7 us, on 128 x 128 23.3 -> 20.8; 300, 9216 x 4096 on 192 x 64 26.7 -> 23.8.)
// Metadata: META_PAIRS pairs (16 bytes each) per row at a time, as many neighbouring lanes per row, the pieces of a row
// rotated so that the sixteen rows of a 2-byte read fall on different banks.
// Weights from HBM, us, the two-phase kernel / here: 2048 tokens, 768 x 3072 on 128 x 64 20.4 / 15.8; 512 tokens, 4096 x 4096
// 26.7 / 20.8; 300 tokens, 9216 x 4096 on 128 x 128 39.6 / 33.0, on 192 x 64 39.9 / 29.5; on 192 x 128 and larger tiles, where
// a stage of this ring would leave room for two only, a barrier per k-step with as many stages took 42 against 45 on
// 192 x 128 and 53 against 49 on 256 x 128 (1000 tokens, 4352 x 4352): those stay with the kernel above.
template <int BM, int BN>
struct RingSmem {
    static constexpr int A_STAGE = BM * 128, B_STEP = BN * 128;   // packed values of BM rows x 2 k-steps; BN tokens x 1
    static constexpr int STAGE = A_STAGE + 2 * B_STEP;
    static constexpr int META_PAIRS = 3 * STAGE + 2 * BM * 64 <= 160 * 1024 ? 4 : 2;
    static constexpr int M_ROW = META_PAIRS * 16, M_BLOCK = BM * M_ROW;   // two blocks of metadata
    static constexpr int FIT = (160 * 1024 - 2 * M_BLOCK) / STAGE;
    static constexpr int STAGES = FIT < META_PAIRS + 1 ? FIT : META_PAIRS + 1;   // a block is rewritten when the pair
                                                                                  // before its successor's first has been read
    static constexpr int M_OFF = STAGES * STAGE, TOTAL = M_OFF + 2 * M_BLOCK;
    static_assert(STAGES >= 3 && M_BLOCK % 1024 == 0, "a ring");
};

// Loads of the `pairs` pairs after the pair with index u in its block of metadata: what may be in flight while that pair is read
template <class S>
constexpr int ring_leave(int u, int pairs, int each, int meta) {
    int c = 0;
    for (int q = 1; q <= pairs; ++q) c += each + ((u + q) % S::META_PAIRS == 0 ? meta : 0);
    return c;
}

// TAIL: an odd number of k-steps; the values and metadata of the last one are then fetched as the second half of a pair that
// ends with the row (see spmm_kernel).
template <int BM, int BN, bool TAIL, class Job>
__global__ void __launch_bounds__(RING_THREADS) spmm_ring_kernel(const bf16_t* __restrict__ B, int n,
                                                                 const bf16_t* __restrict__ Av,
                                                                 const uint8_t* __restrict__ Am, int m, int K,
                                                                 const bf16_t* __restrict__ B2,
                                                                 const bf16_t* __restrict__ A2, int K2,
                                                                 bf16_t* __restrict__ C, int tiles_m, int tiles_n,
                                                                 Job job) {
    using S = RingSmem<BM, BN>;
    constexpr int META_PAIRS = S::META_PAIRS;
    constexpr int WM = 2, WN = RING_MULT / WM;                // wavefronts over the tile
    constexpr int MF = BM / (16 * WM), NF = BN / (16 * WN);
    constexpr int A_LD = BM / (8 * LOADERS), B_LD = BN / (8 * LOADERS);   // 1 KiB loads per loading wavefront: of a pair, of a k-step
    constexpr int M_LOADS = S::M_BLOCK / 1024, M_LD = (M_LOADS + LOADERS - 1) / LOADERS;   // per block; some twice where need be
    static_assert(BM % 64 == 0 && BN % 32 == 0 && BM % (16 * WM) == 0 && BN % (16 * WN) == 0, "whole loads and fragments");
    extern __shared__ __align__(16) uint8_t smem[];
    fetch_arguments(B, n, Av, Am, m, K, tiles_m, tiles_n);

    int tm, tn, slab = 0, extension_slab = 0;
    if constexpr (is_split<Job>) {
        static_assert(SPMM_THREADS == SK_WAVES * 64 && RING_THREADS == SPMM_THREADS && SK_LDS <= S::TOTAL, "a skinny tile fits in the workgroup");
        if (!split_item(job, B, n, K, tiles_m, tiles_n, smem, tm, tn, slab, extension_slab)) return;
    } else {
        if (!tile_of<BM, BN>(job, m, n, tiles_m, tiles_n, tm, tn)) return;
    }
    const int m0 = tm * BM, n0 = tn * BN;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int l16 = lane & 15, lq = lane >> 4;
    int k_first = 0, slab_steps = K / 64;
    float* sums = nullptr;
    if constexpr (is_split<Job>) {
        slab_steps = job.slab_steps;
        k_first = slab * slab_steps;                          // a multiple of 4
        sums = job.slabs + (size_t)slab * (size_t)n * (size_t)m;
    }
    const int ksteps = K / 64 - k_first > slab_steps ? slab_steps : K / 64 - k_first;
    const int pairs = (ksteps + 1) / 2;

    if (wave >= RING_MULT) {                                  // (a wavefront that has ended does not count at barriers)
        const int loader = wave - RING_MULT;
        // ---- loader lanes: 8 lanes per row of 128 bytes, chunk rotated by (row / 2) % 8; the tokens' two k-steps are the same rows
        const uint8_t* a_src[A_LD];
        const uint8_t* b_src[B_LD];
        const uint8_t* m_src[M_LD];
        int m_pair[M_LD], m_dst[M_LD];                        // pair inside the block; LDS offset inside it
        auto load_a = [&](int i, int p, uint8_t* st) { dma16(a_src[i] + pair_offset<TAIL>(p, ksteps), st + (loader * A_LD + i) * 1024); };
        auto load_b = [&](int i, int p, uint8_t* st) {
            uint8_t* const dst = st + S::A_STAGE + (loader * B_LD + i) * 1024;
            dma16(b_src[i] + (size_t)p * 256, dst);
            dma16(b_src[i] + (size_t)p * 256 + (!TAIL || 2 * p + 1 < ksteps ? 128 : 0), dst + S::B_STEP);
        };
        auto load_m = [&](int i, int p) {
            const int64_t off = (int64_t)(p + m_pair[i]) * 16, last = (int64_t)ksteps * 8 - 16;
            dma16(m_src[i] + (off < last ? off : last), smem + m_dst[i] + (p / META_PAIRS & 1) * S::M_BLOCK);
        };
        // Each address is followed by its load of the first pair, so that those are on their way while the next ones are made (us, from
        // memory, all addresses first / so: 46 tokens, 8256 x 8448 in five slabs of 192 x 64 21.4 / 20.2; 700, 4160 x 2112 16.0 / 15.3; 1114, 1600
        // x 704 7.5 / 7.2)
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            const int rl = (loader * A_LD + i) * 8 + (lane >> 3);
            a_src[i] = (const uint8_t*)Av + (size_t)wrap_row_near(m0 + rl, m) * K + (((lane & 7) ^ ((rl >> 1) & 7)) * 16) + (size_t)k_first * 64;
            load_a(i, 0, smem);
        }
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            const int rl = (loader * B_LD + i) * 8 + (lane >> 3);
            b_src[i] = (const uint8_t*)B + (size_t)wrap_row_near(n0 + rl, n) * K * 2 + (((lane & 7) ^ ((rl >> 1) & 7)) * 16) + (size_t)k_first * 128;
        }
#pragma unroll
        for (int i = 0; i < M_LD; ++i) {
            const int idx = (loader * M_LD + i) % M_LOADS, rl = (idx * 64 + lane) / META_PAIRS;
            m_src[i] = Am + (size_t)wrap_row_near(m0 + rl, m) * (K / 8) + (size_t)k_first * 8;
            m_pair[i] = (lane % META_PAIRS) ^ (rl * META_PAIRS / 16 % META_PAIRS);
            m_dst[i] = S::M_OFF + idx * 1024;
            load_m(i, 0);
        }
        auto issue = [&](int p, int stage, bool new_block) {  // loads of pair p (inside the contraction, at least in part)
            uint8_t* const st = smem + stage * S::STAGE;
            if (new_block) {
#pragma unroll
                for (int i = 0; i < M_LD; ++i) load_m(i, p);
            }
#pragma unroll
            for (int i = 0; i < A_LD; ++i) load_a(i, p, st);
#pragma unroll
            for (int i = 0; i < B_LD; ++i) load_b(i, p, st);
        };
#pragma unroll
        for (int p = 1; p < S::STAGES - 1; ++p)
            if (p < pairs) issue(p, p, p % META_PAIRS == 0);
        int stage = S::STAGES - 1;
        // pair p, with index u in its block of metadata, has landed, with up to STAGES - 2 pairs still behind it, and everybody has read the
        // one before it, whose stage is filled again.  (Where fewer than STAGES - 2 follow, waiting for all of them, with one wavefront per
        // SIMD left to multiply, made contractions of 256 slower than with eight: us, eight / four, all / four, so: 1889 tokens, 768 x 256 on 128 x
        // 64 4.7 / 5.1 / 4.7; over 61 products of contractions up to 1024 on that tile 2 % slower, now 2 % faster in the mean.)
        auto pair = [&](int p, auto index) {
            constexpr int u = decltype(index)::value, EACH = A_LD + 2 * B_LD, BEHIND = S::STAGES - 2;
            static_assert(BEHIND >= 1 && BEHIND <= 3, "each number of pairs has its wait");
            if (p + BEHIND < pairs) WAIT_HERE(waitcnt_imm(ring_leave<S>(u, BEHIND, EACH, M_LD), 15));
            else if (BEHIND > 2 && p + 2 < pairs) WAIT_HERE(waitcnt_imm(ring_leave<S>(u, 2, EACH, M_LD), 15));
            else if (BEHIND > 1 && p + 1 < pairs) WAIT_HERE(waitcnt_imm(ring_leave<S>(u, 1, EACH, M_LD), 15));
            else WAIT_HERE(waitcnt_imm(0, 15));
            wg_barrier();
            if (p + S::STAGES - 1 < pairs) issue(p + S::STAGES - 1, stage, (u + S::STAGES - 1) % META_PAIRS == 0);
            stage = stage == S::STAGES - 1 ? 0 : stage + 1;
        };
        for (int p = 0; p < pairs; p += META_PAIRS) {
            pair(p, std::integral_constant<int, 0>{});
            if (p + 1 >= pairs) break;
            pair(p + 1, std::integral_constant<int, 1>{});
            if constexpr (META_PAIRS == 4) {
                if (p + 2 >= pairs) break;
                pair(p + 2, std::integral_constant<int, 2>{});
                if (p + 3 >= pairs) break;
                pair(p + 3, std::integral_constant<int, 3>{});
            }
        }
        if (K2 < 0 && slab == extension_slab) stage_factor<BM, 64 * LOADERS>(A2, K2, m, smem, m0, t - 64 * RING_MULT);
        return;
    }

    f32x4 acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // ---- reader lanes: fragment f = rows 16f .. 16f+15 = 2 KiB; lane (l16, lq) wants chunk 4h + lq
    const int sw = (l16 >> 1) & 7;
    const int rd0 = l16 * 128 + ((lq ^ sw) * 16), rd1 = l16 * 128 + (((4 + lq) ^ sw) * 16);
    const int a_rd = wm * MF * 2048, b_rd = S::A_STAGE + wn * NF * 2048;
    const int m_rd = S::M_OFF + (wm * MF * 16 + l16) * S::M_ROW + lq * 2, m_sw = l16 * META_PAIRS / 16 % META_PAIRS;
    struct Frags {                                            // of a k-step
        BFrag bf[NF];
        AFrag af[MF];
        int ai[MF];
    };
    // second: the second half of the pair's rows of values and metadata
    auto read = [&](Frags& f, int stage, int p, int u, int e, bool second) {
        const uint8_t* const st = smem + stage * S::STAGE;
        const uint8_t* const pm = smem + m_rd + (p / META_PAIRS & 1) * S::M_BLOCK + (u ^ m_sw) * 16 + (second ? 8 : 0);
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            f.bf[j].u[0] = *(const u32x4*)(st + b_rd + e * S::B_STEP + j * 2048 + rd0);
            f.bf[j].u[1] = *(const u32x4*)(st + b_rd + e * S::B_STEP + j * 2048 + rd1);
        }
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            f.af[i].u = *(const u32x4*)(st + a_rd + i * 2048 + (second ? rd1 : rd0));
            f.ai[i] = *(const uint16_t*)(pm + i * 16 * S::M_ROW);
        }
    };
    auto multiply = [&](const Frags& f) {
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j)
                acc[i][j] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(f.af[i].v, f.bf[j].v, acc[i][j], f.ai[i], 0, 0);
    };
    // The tokens of the first pair, which the loaders leave out: theirs are the weights (0.3 % less than all by the loaders in the mean)
#pragma unroll
    for (int i = 0; i < BN / (4 * RING_MULT); ++i) {
        const int j = wave * (BN / (4 * RING_MULT)) + i, step = j / (BN / 8), rl = j % (BN / 8) * 8 + (lane >> 3);   // step: wave-uniform
        dma16((const uint8_t*)B + (size_t)wrap_row_near(n0 + rl, n) * K * 2 + (((lane & 7) ^ ((rl >> 1) & 7)) * 16) + (size_t)k_first * 128 +
                  (step && (!TAIL || ksteps > 1) ? 128 : 0), smem + S::A_STAGE + j * 1024);
    }
    WAIT_HERE(waitcnt_imm(0, 15));
    // the loaders pass this when pair p has landed, the others when they have read what came before it
    auto landed = [&]() {
        WAIT_HERE(waitcnt_imm(63, 0));
        wg_barrier();
    };
    landed();
    Frags f0, f1;
    read(f0, 0, 0, 0, 0, TAIL && ksteps == 1);
    int stage = 0;
    auto pair = [&](int p, auto index) {                      // index = p % META_PAIRS; f0 holds the pair's first k-step
        constexpr int u = decltype(index)::value, next = (u + 1) % META_PAIRS;
        const bool odd_end = TAIL && 2 * p + 1 >= ksteps;
        if (!odd_end) read(f1, stage, p, u, 1, true);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f0);
        if (p + 1 < pairs) {
            landed();
            const int after = stage == S::STAGES - 1 ? 0 : stage + 1;
            read(f0, after, p + 1, next, 0, TAIL && 2 * p + 3 >= ksteps);
            __builtin_amdgcn_sched_barrier(0);
            stage = after;
        }
        if (!odd_end) multiply(f1);
    };
    for (int p = 0; p < pairs; p += META_PAIRS) {
        pair(p, std::integral_constant<int, 0>{});
        if (p + 1 >= pairs) break;
        pair(p + 1, std::integral_constant<int, 1>{});
        if constexpr (META_PAIRS == 4) {
            if (p + 2 >= pairs) break;
            pair(p + 2, std::integral_constant<int, 2>{});
            if (p + 3 >= pairs) break;
            pair(p + 3, std::integral_constant<int, 3>{});
        }
    }
    static_assert(BN * (BM * 2 + 16) <= S::TOTAL && 128 * (BM * 2 + 32) <= S::TOTAL, "the staged output tile and factor fit in the ring");
    extend_and_store<MF, NF, BM, BN, 64 * RING_MULT, true>(acc, m0 + wm * MF * 16, n0 + wn * NF * 16, m, n, l16, lq, B2, A2,
                                                   slab == extension_slab ? K2 : 0, C, smem, m0, n0, sums);
}

// ------------------------------------------------------------------------------------------
// Generic kernel (any K % 8 == 0): a tile of 32 F x 32 F, G groups of 4 wavefronts (2 x 2), operands staged
// through registers, two k-steps (a pair) per trip.  What a compute unit can keep in flight is a number of requests, not
// of bytes, so all loads are of whole 128-byte lines: 8 lanes per row of packed values, 16 per row of tokens (half as
// many requests as with a k-step per trip and 64 bytes per row: 1000 tokens, 1000 x 1000, 14.4 -> 10.5 us).
// LDS holds rows of 128 bytes, the 16-byte chunks rotated by (row / 2) % 8 as in the kernels above.
// With one group (F = 4: 128 x 128) every trip is a memory latency, which several workgroups per compute unit hide from
// each other.  Few tiles get F = 2 (64 x 64) and four groups that take the pairs in turn and add their partial tiles
// through LDS in a fixed order: four times as many workgroups, a quarter of the trips in a row (20.1 -> 10.5 us there; the
// form before this one, 128 x 128 with a k-step of byte-wise metadata loads per trip, took 35).
// RAGGED (K not a multiple of 64): rows of the packed weight are only 8-byte, rows of the metadata only
// 1-byte aligned (the hardware takes 16-byte loads at such addresses).
// The last pair may be partly past the end of the rows.  Its loads come in pieces of 8 logical k (8 bytes of packed
// values, 16 bytes of tokens, 1 byte of metadata), each either wholly inside the row or replaced: zeros for
// values and tokens, the nibble pair 0x44 (positions 0, 1: a legal encoding) for metadata, so the tail contributes
// exact zeros.
enum { GEN_WHOLE = 0, GEN_PARTIAL = 1, GEN_RAGGED = 2 };      // K % 128 == 0; whole k-steps (K % 64 == 0); any K % 8 == 0
template <int F, int G>
struct GenSmem {
    static constexpr int BM = 32 * F, BN = 32 * F;            // the tile
    static constexpr int A_BYTES = BM * 128, B_STEP = BN * 128, M_BYTES = BM * 16;
    static constexpr int M_OFF = A_BYTES + 2 * B_STEP;
    static constexpr int STAGE = M_OFF + M_BYTES;
    static constexpr int SUM_PITCH = BM + 4;                  // floats per token row of a partial tile
    static constexpr int SUMS = G > 1 ? G * BN * SUM_PITCH * 4 : 0;
    static constexpr int TOTAL = G * STAGE > SUMS ? G * STAGE : SUMS;
};

template <int FORM, int F, int G>
__global__ void __launch_bounds__(256 * G) spmm_generic_kernel(const bf16_t* __restrict__ B, int n,
                                                           const bf16_t* __restrict__ Av,
                                                           const uint8_t* __restrict__ Am, int m, int K,
                                                           const bf16_t* __restrict__ B2,
                                                           const bf16_t* __restrict__ A2, int K2,
                                                           bf16_t* __restrict__ C, int tiles_m) {
    using S = GenSmem<F, G>;
    constexpr int MF = F, NF = F, A_LD = F, B_LD = 2 * F;         // 16-byte pieces per lane and pair
    __shared__ __align__(16) uint8_t smem[S::TOTAL];
    const int m0 = (blockIdx.x % tiles_m) * S::BM, n0 = (blockIdx.x / tiles_m) * S::BN;
    const int group = (int)threadIdx.x >> 8;
    const int t = threadIdx.x & 255, lane = t & 63, wave = t >> 6;   // inside the group
    uint8_t* const stage = smem + group * S::STAGE;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, lq = lane >> 4;
    // loader lanes: piece u of the packed values is row (t + 256 u) / 8, chunk t % 8; of the tokens row
    // (t + 256 u) / 16, k-step (t % 16) / 8, chunk t % 8
    const uint8_t* a_src[A_LD];
    const bf16_t* b_src[B_LD];
    const int a_dst = (t >> 3) * 128 + (((t & 7) ^ ((t >> 4) & 7)) * 16);   // piece i: 32 rows further on
    const int b_dst = S::A_BYTES + ((t >> 3) & 1) * S::B_STEP + (t >> 4) * 128 + (((t & 7) ^ ((t >> 5) & 7)) * 16);   // 16 rows
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
        const int rl = (t + 256 * i) >> 3;
        a_src[i] = (const uint8_t*)Av + (size_t)wrap_row(m0 + rl, m) * K + (t & 7) * 16;
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        const int rl = (t + 256 * i) >> 4;
        b_src[i] = B + (size_t)wrap_row(n0 + rl, n) * K + (t & 15) * 8;
    }
    const int mrow = t % S::BM;
    const uint8_t* const m_src = Am + (size_t)wrap_row(m0 + mrow, m) * (K / 8);
    f32x4 acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

    u32x4 a_reg[A_LD], b_reg[B_LD], m_reg;
    auto load = [&](int p) {                                  // pair p (uniform, inside the contraction at least in part)
        const int k0 = p * 128;
        if (FORM == GEN_WHOLE || k0 + 128 <= K) {
#pragma unroll
            for (int i = 0; i < A_LD; ++i) {
                if (FORM == GEN_RAGGED) a_reg[i] = *(const u32x4_a8*)(a_src[i] + k0);
                else a_reg[i] = *(const u32x4*)(a_src[i] + k0);
            }
#pragma unroll
            for (int i = 0; i < B_LD; ++i) b_reg[i] = *(const u32x4*)(b_src[i] + k0);
            if (t < S::BM) __builtin_memcpy(&m_reg, m_src + p * 16, 16);
            return;
        }
        const int ak = k0 + (t & 7) * 16, bk = k0 + (t & 15) * 8;
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            u32x2 lo = {0u, 0u}, hi = {0u, 0u};
            if (ak < K) lo = *(const u32x2*)(a_src[i] + k0);
            if (ak + 8 < K) hi = *(const u32x2*)(a_src[i] + k0 + 8);
            a_reg[i] = (u32x4){lo[0], lo[1], hi[0], hi[1]};
        }
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            b_reg[i] = (u32x4){0u, 0u, 0u, 0u};
            if (bk < K) b_reg[i] = *(const u32x4*)(b_src[i] + k0);
        }
        const int have = K / 8 - p * 16;                      // metadata bytes of this pair inside the row: 1 .. 15
        uint8_t byte[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) byte[e] = m_src[p * 16 + (e < have ? e : have - 1)];   // past the end the last again
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (e >= have) byte[e] = 0x44;
        __builtin_memcpy(&m_reg, byte, 16);
    };

    // group g takes pairs g, g + G, ...; on the last trip some groups may have none
    const int pairs = (K + 127) / 128, trips = (pairs + G - 1) / G, sw = (l16 >> 1) & 7;
    if (group < pairs) load(group);
    for (int tr = 0; tr < trips; ++tr) {
        const int p = tr * G + group;
        if (tr > 0) __syncthreads();                          // everybody has read the last pair
#pragma unroll
        for (int i = 0; i < A_LD; ++i) *(u32x4*)(stage + a_dst + i * 4096) = a_reg[i];
#pragma unroll
        for (int i = 0; i < B_LD; ++i) *(u32x4*)(stage + b_dst + i * 2048) = b_reg[i];
        if (t < S::BM) *(u32x4*)(stage + S::M_OFF + t * 16) = m_reg;
        if (p + G < pairs) load(p + G);
        __syncthreads();
        if (p >= pairs) continue;                             // uniform per wavefront (the barriers are above)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint8_t* sb = stage + S::A_BYTES + e * S::B_STEP + (wn * NF * 16 + l16) * 128;
            const uint8_t* sa = stage + (wm * MF * 16 + l16) * 128 + (((4 * e + lq) ^ sw) * 16);
            const uint8_t* sm = stage + S::M_OFF + (wm * MF * 16 + l16) * 16 + 8 * e + 2 * lq;
            BFrag bf[NF];
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                bf[j].u[0] = *(const u32x4*)(sb + j * 2048 + ((lq ^ sw) * 16));
                bf[j].u[1] = *(const u32x4*)(sb + j * 2048 + (((4 + lq) ^ sw) * 16));
            }
#pragma unroll
            for (int i = 0; i < MF; ++i) {
                AFrag a;
                a.u = *(const u32x4*)(sa + i * 2048);
                const int idx = *(const uint16_t*)(sm + i * 256);
#pragma unroll
                for (int j = 0; j < NF; ++j)
                    acc[i][j] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(a.v, bf[j].v, acc[i][j], idx, 0, 0);
            }
        }
    }
    __syncthreads();                                          // the stages are free
    if constexpr (G == 1) {
        static_assert(S::BN * (S::BM * 2 + 16) <= S::TOTAL, "the staged output tile fits in the stages");
        extend_and_store<MF, NF, S::BM, S::BN, 256>(acc, m0 + wm * MF * 16, n0 + wn * NF * 16, m, n, l16, lq, B2, A2, K2, C,
                                                    smem, m0, n0);
    } else {
        // adapter extension from global memory, its steps of 32 dealt to the groups (A2 k-contiguous or k-major)
        const int KR = K2 < 0 ? -K2 : K2;
        for (int k0 = 32 * group; k0 < KR; k0 += 32 * G) {
            AFrag a2[MF], b2[NF];
#pragma unroll
            for (int j = 0; j < NF; ++j)
                b2[j].u = *(const u32x4*)(B2 + (size_t)wrap_row(n0 + (wn * NF + j) * 16 + l16, n) * KR + k0 + lq * 8);
#pragma unroll
            for (int i = 0; i < MF; ++i) {
                const int row = wrap_row(m0 + (wm * MF + i) * 16 + l16, m);
                if (K2 > 0) {
                    a2[i].u = *(const u32x4*)(A2 + (size_t)row * KR + k0 + lq * 8);
                } else {
                    const bf16_t* p = A2 + (size_t)(k0 + lq * 8) * m + row;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        a2[i].u[e] = (uint32_t)p[(size_t)(2 * e) * m] | ((uint32_t)p[(size_t)(2 * e + 1) * m] << 16);
                }
            }
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
                for (int j = 0; j < NF; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2[i].v, b2[j].v, acc[i][j], 0, 0, 0);
        }
        // the groups' partial tiles, [group][token][SUM_PITCH]; the stages are idle
        float* const part = (float*)smem;
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j)
                *(f32x4*)(part + ((group * S::BN + (wn * NF + j) * 16 + l16) * S::SUM_PITCH + (wm * MF + i) * 16 + lq * 4)) = acc[i][j];
        __syncthreads();
        for (int idx = (int)threadIdx.x; idx < S::BM * S::BN / 4; idx += 256 * G) {
            const int tok = idx / (S::BM / 4), col = (idx % (S::BM / 4)) * 4;
            f32x4 v = *(const f32x4*)(part + tok * S::SUM_PITCH + col);
#pragma unroll
            for (int q = 1; q < G; ++q) {
                const f32x4 x = *(const f32x4*)(part + (q * S::BN + tok) * S::SUM_PITCH + col);
                v[0] += x[0]; v[1] += x[1]; v[2] += x[2]; v[3] += x[3];
            }
            if (n0 + tok < n && m0 + col < m) {               // m % 8 == 0
                union { __bf16 h[4]; u32x2 u; } o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o.h[e] = (__bf16)v[e];
                *(u32x2*)(C + (size_t)(n0 + tok) * m + m0 + col) = o.u;
            }
        }
    }
}

// The form with four groups on 64 x 64 tiles, while those tiles are at most two rounds of one workgroup per compute unit
// (1000 tokens, 1000 x 1000, 256 tiles: 10.5 us against 20.1 for 128 x 128; 2000 tokens, 512 tiles: 18.9 against 21.1; but
// 2048 tokens, 2056 x 2056, 1056 tiles: 79 against 43).  Where whole k-steps let the tile kernels compete it is the better
// one in a single round only (spmm_tile_choice).  Register-staged tiles of 128 x 64 to 256 x 128 with two to four groups
// were measured too: never better than both this and the tile kernels' rings.
inline int64_t tiles_of_64(int64_t n, int64_t m) { return ((m + 63) / 64) * ((n + 63) / 64); }

template <int F, int G>
hipError_t launch_generic_as(const bf16_t* B, int64_t n, const bf16_t* Av, const uint8_t* Am, int64_t m, int64_t K,
                             const bf16_t* B2, const bf16_t* A2, int64_t K2, bf16_t* C, hipStream_t s) {
    using S = GenSmem<F, G>;
    static_assert(S::TOTAL <= 160 * 1024, "LDS budget");
    const int tiles_m = (int)((m + S::BM - 1) / S::BM), tiles_n = (int)((n + S::BN - 1) / S::BN);
    auto kern = K % 128 == 0 ? spmm_generic_kernel<GEN_WHOLE, F, G>
                : K % 64 == 0 ? spmm_generic_kernel<GEN_PARTIAL, F, G> : spmm_generic_kernel<GEN_RAGGED, F, G>;
    kern<<<dim3((unsigned)(tiles_m * tiles_n)), dim3(256 * G), 0, s>>>(B, (int)n, Av, Am, (int)m, (int)K, B2, A2, (int)K2,
                                                                       C, tiles_m);
    return hipGetLastError();
}

hipError_t launch_generic(const bf16_t* B, int64_t n, const bf16_t* Av, const uint8_t* Am, int64_t m, int64_t K,
                          const bf16_t* B2, const bf16_t* A2, int64_t K2, bf16_t* C, hipStream_t s) {
    if (spmm_generic_edge(n, m) == 64) return launch_generic_as<2, 4>(B, n, Av, Am, m, K, B2, A2, K2, C, s);
    return launch_generic_as<4, 1>(B, n, Av, Am, m, K, B2, A2, K2, C, s);
}

// workgroups of a launch over the tiles, or over the tiles of every slab and the parts of X L beside them
template <int BM, int BN>
int tile_grid(int tiles_m, int tiles_n, int64_t, const WholeJob&) { return super_grid(tiles_m, tiles_n); }
template <int BM, int BN>
int tile_grid(int, int, int64_t, const Leftover& left) { return leftover_grid<BM, BN>(left); }
template <int BM, int BN>
int tile_grid(int tiles_m, int tiles_n, int64_t n, const SplitJob& job) {
    const int xl = job.L ? job.xl_slabs * ((job.r + SK_BJ - 1) / SK_BJ) * (int)((n + SK_BI - 1) / SK_BI) : 0;
    return ((tiles_m * tiles_n * job.nslabs + XCDS - 1) / XCDS + (xl + XCDS - 1) / XCDS) * XCDS;
}

template <int BM, int BN, bool TAIL, class Job>
hipError_t launch_tile_as(const bf16_t* B, int64_t n, const bf16_t* Av, const uint8_t* Am, int64_t m, int64_t K,
                          const bf16_t* B2, const bf16_t* A2, int64_t K2, bf16_t* C, hipStream_t s, const Job& job) {
    using S = SpmmSmem<BM, BN>;
    static_assert(S::TOTAL <= 160 * 1024, "LDS budget");
    int tiles_m = (int)((m + BM - 1) / BM), tiles_n = (int)((n + BN - 1) / BN);
    hipError_t e = allow_dynamic_lds<spmm_kernel<BM, BN, TAIL, Job>>(S::TOTAL);
    if (e != hipSuccess) return e;
    const int grid = tile_grid<BM, BN>(tiles_m, tiles_n, n, job);
    spmm_kernel<BM, BN, TAIL, Job><<<dim3((unsigned)grid), dim3(SPMM_THREADS), S::TOTAL, s>>>(
        B, (int)n, Av, Am, (int)m, (int)K, B2, A2, (int)K2, C, tiles_m, tiles_n, job);
    return hipGetLastError();
}

template <int BM, int BN, bool TAIL, class Job>
hipError_t launch_ring_as(const bf16_t* B, int64_t n, const bf16_t* Av, const uint8_t* Am, int64_t m, int64_t K,
                          const bf16_t* B2, const bf16_t* A2, int64_t K2, bf16_t* C, hipStream_t s, const Job& job) {
    using S = RingSmem<BM, BN>;
    static_assert(S::TOTAL <= 160 * 1024, "LDS budget");
    int tiles_m = (int)((m + BM - 1) / BM), tiles_n = (int)((n + BN - 1) / BN);
    hipError_t e = allow_dynamic_lds<spmm_ring_kernel<BM, BN, TAIL, Job>>(S::TOTAL);
    if (e != hipSuccess) return e;
    const int grid = tile_grid<BM, BN>(tiles_m, tiles_n, n, job);
    spmm_ring_kernel<BM, BN, TAIL, Job><<<dim3((unsigned)grid), dim3(RING_THREADS), S::TOTAL, s>>>(
        B, (int)n, Av, Am, (int)m, (int)K, B2, A2, (int)K2, C, tiles_m, tiles_n, job);
    return hipGetLastError();
}

// a whole product, or one split over k
template <int BM, int BN, class Job = WholeJob>
hipError_t launch_tile(const bf16_t* B, int64_t n, const bf16_t* Av, const uint8_t* Am, int64_t m, int64_t K,
                       const bf16_t* B2, const bf16_t* A2, int64_t K2, bf16_t* C, hipStream_t s, const Job& job = {}) {
    auto launch = K % 256 == 0 ? launch_tile_as<BM, BN, false, Job> : launch_tile_as<BM, BN, true, Job>;
    return launch(B, n, Av, Am, m, K, B2, A2, K2, C, s, job);
}

template <int BM, int BN, class Job = WholeJob>
hipError_t launch_ring(const bf16_t* B, int64_t n, const bf16_t* Av, const uint8_t* Am, int64_t m, int64_t K,
                       const bf16_t* B2, const bf16_t* A2, int64_t K2, bf16_t* C, hipStream_t s, const Job& job = {}) {
    auto launch = K % 128 == 0 ? launch_ring_as<BM, BN, false, Job> : launch_ring_as<BM, BN, true, Job>;
    return launch(B, n, Av, Am, m, K, B2, A2, K2, C, s, job);
}

// C[idx] = bf16( sum over slabs, in order, of P[s][idx] ), four elements per thread
__global__ void __launch_bounds__(256) slab_reduce_kernel(const f32x4* __restrict__ P, int nslabs, size_t count4,
                                                          u32x2* __restrict__ C) {
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= count4) return;
    f32x4 v = P[idx];
    for (int sl = 1; sl < nslabs; ++sl) {
        f32x4 w = P[(size_t)sl * count4 + idx];
        v[0] += w[0]; v[1] += w[1]; v[2] += w[2]; v[3] += w[3];
    }
    union { __bf16 h[4]; u32x2 u; } o;
    o.h[0] = (__bf16)v[0]; o.h[1] = (__bf16)v[1]; o.h[2] = (__bf16)v[2]; o.h[3] = (__bf16)v[3];
    C[idx] = o.u;
}

template <bool PREFETCH, bool TAIL>
hipError_t launch_split_as(const bf16_t* B, int64_t n, const bf16_t* Av, const uint8_t* Am, int64_t m, int64_t K,
                           const bf16_t* B2, const bf16_t* A2, int64_t K2, bf16_t* C, int tiles_m, int tiles_n, int grid,
                           hipStream_t s) {
    using S = SplitSmem;
    static_assert(S::TOTAL <= 160 * 1024, "LDS budget");
    hipError_t e = allow_dynamic_lds<spmm_split_kernel<PREFETCH, TAIL>>(S::TOTAL);
    if (e != hipSuccess) return e;
    spmm_split_kernel<PREFETCH, TAIL><<<dim3((unsigned)grid), dim3(SPMM_THREADS), S::TOTAL, s>>>(
        B, (int)n, Av, Am, (int)m, (int)K, B2, A2, (int)K2, C, tiles_m, tiles_n);
    return hipGetLastError();
}

// A last round of 256 x 256 tiles that at most half of the compute units would have a tile of: its tiles as one round of
// tiles of a half, 256 x 128, or up to a quarter of a round of 128 x 128, in a launch of their own.  The first launch is whole rounds
// then: its workgroups 0 .. first - 1 are exactly the positions 0 .. first - 1 of the order.  Half a round's own compute units
// pull their operands faster than a full round's, so that halving the tiles pays on long contractions only (us, from the last-level
// cache and from HBM, one launch / two: 64 tiles left, 16384 tokens, 4352 x 4352 309 / 289 and 379 / 345; 48, 4096, 4864 x 2048 58.6 /
// 54.8 and 58.5 / 53.4; 16, 4096, 4352 x 2048 58.7 / 52.8 and 59.8 / 53.7; 64, 16384, 4352 x 1024 97.3 / 96.4 and 109.7 / 108.3, x 512 64.7
// / 64.6 and 80.1 / 83.4; 128 left, 16384, 2560 x 10240 469 / 451 and 542 / 521, x 6144 267 / 266 and 315 / 297, x 4096 171 / 175 and 208
// / 197, x 2048 94.6 / 97.8 and 110.8 / 114.0; 12288, 6144 x 4160 303 / 311 and 356 / 367).
inline Leftover leftover_tiles(int tiles_m, int tiles_n, int64_t K) {
    const int64_t tiles = (int64_t)tiles_m * tiles_n, rem = tiles % RESIDENT;
    const int64_t shortest = rem <= RESIDENT / 4 ? 2048 : 6144;
    if (!wide_grid(tiles_m, tiles_n) || tiles > (1 << 30) || rem == 0 || rem > RESIDENT / 2 || K < shortest) return {0, 0, 0, 0};
    return {(int)(tiles - rem), (int)rem, tiles_m, tiles_n};
}

hipError_t launch_split(const bf16_t* B, int64_t n, const bf16_t* Av, const uint8_t* Am, int64_t m, int64_t K,
                        const bf16_t* B2, const bf16_t* A2, int64_t K2, bf16_t* C, hipStream_t s) {
    using S = SplitSmem;
    int tiles_m = (int)((m + S::BM - 1) / S::BM), tiles_n = (int)((n + S::BN - 1) / S::BN);
    const bool prefetch = wide_grid(tiles_m, tiles_n) && (size_t)n * (size_t)K * 2 > LAST_LEVEL_CACHE_BYTES;
    auto launch = K % 256 == 0 ? (prefetch ? launch_split_as<true, false> : launch_split_as<false, false>)
                               : (prefetch ? launch_split_as<true, true> : launch_split_as<false, true>);
    const Leftover left = leftover_tiles(tiles_m, tiles_n, K);
    const hipError_t e = launch(B, n, Av, Am, m, K, B2, A2, K2, C, tiles_m, tiles_n, left.count ? left.first : super_grid(tiles_m, tiles_n), s);
    if (e != hipSuccess || !left.count) return e;
    if (left.count > RESIDENT / 4) return launch_tile<256, 128>(B, n, Av, Am, m, K, B2, A2, K2, C, s, left);
    return launch_ring<128, 128>(B, n, Av, Am, m, K, B2, A2, K2, C, s, left);
}

}  // namespace

// Products of too few tiles to fill the chip, a few dozen tokens on any weight or some thousand on a small one: narrow
// token tiles on small weight tiles would re-read the tokens from L2 for every few weight rows (the tile kernels run at the
// L2 -> LDS rate), and tall weight tiles alone are too few.  So the k range is cut into slabs that run
// as separate workgroups and leave fp32 partial sums in `slabs`, and a short second kernel (fixed order: bit-identical
// runs) rounds to bf16.  SLAB_MAX_TOKENS is the reach of the estimate for long weights on tiles of 256 rows below.
constexpr int64_t SLAB_MAX_TOKENS = 1024;

// The tile kernels take whole k-steps of 64, at least two of them (700 tokens: 4160 x 2112 54 -> 25 us, 2112 x 4160
// 96 -> 35 us against the generic kernel).
static bool tile_kernel_fits(int64_t K) { return K % 64 == 0 && K >= 128; }
// One round of 64 x 64 tiles: the generic kernel's four groups are the best form without a split where twice as large
// tiles would leave half of the compute units idle (300 tokens, 1536 x 1536 8.6 us, on 128 x 64 9.5; 1024 tokens, 1024 x
// 1024 8.7): all of a compute unit's 16 wavefronts load, and each k-step waits for its own quarter of them only.  (777
// tokens, 1280 x 5120, 260 tiles in two rounds: 34 -> 50 us.)
static bool one_round_of_64(int64_t n, int64_t m) { return tiles_of_64(n, m) <= RESIDENT; }

static int64_t slab_steps_of(int64_t K, int want) {           // k-steps per slab, whole quads
    const int64_t quads = (K + 255) / 256;
    return (quads + want - 1) / want * 4;
}

// ---- The room for slabs: how many of them a call's scratch holds.  Sizes of scratch are part of the interface (programs keep
// buffers, and slope_spmm_fwd takes its buffer on trust), so a split may never want more than the two rules below name,
// whatever the estimate that chooses it (launch_us, further down) prefers: they stay as they are, with the times of earlier
// kernels in them, while that one follows the kernels.
static int slabs_of_a_long_weight(int64_t n, int64_t m, int64_t K) {
    if (n <= STREAM_MAX_TOKENS || n > SLAB_MAX_TOKENS || !tile_kernel_fits(K)) return 0;
    const int64_t tiles = ((m + 255) / 256) * ((n + 127) / 128);
    if (tiles >= RESIDENT) return 0;                          // the chip is full without a split (measured: slabs lose)
    const int64_t quads = (K + 255) / 256;                    // slabs are whole quads of k-steps (the last may be shorter)
    // Estimate per slab count: the rounds of 256 workgroups, each pulling its share of the packed
    // weight at what one compute unit sustains with this tile (about 24 B/ns of weight bytes), plus
    // writing and re-reading the partial sums at HBM speed.  One slab means: not worth it.
    const double weight = 1.125 * (double)m * (double)K, cu = 24.0, hbm = 5.0e3;   // bytes, bytes per ns
    int best = 1;
    double best_ns = 1e300;
    // (a round is counted full at 7/8 of the compute units, which leaves room for X L beside the tiles.  9216 x 36864 at 128
    // tokens, us: 6 slabs, 216 workgroups, 112, with an adapter of rank 128 117; 7 slabs, 252 workgroups, 107 and 123)
    const int64_t fit = RESIDENT - RESIDENT / 8;
    for (int sl = 1; sl <= 16 && sl * 4 <= quads; ++sl) {
        const double rounds = (double)((tiles * sl + fit - 1) / fit);
        const double ns = rounds * weight / (double)(tiles * sl) / cu
                          + (sl > 1 ? 2.0 * sl * (double)n * (double)m * 4.0 / hbm : 0.0);
        if (ns < best_ns) { best_ns = ns; best = sl; }
    }
    // One round of 64 x 64 tiles with four groups takes about 2 us and 2.6 us per 512 of the contraction on weights that come
    // from HBM, slabs the estimate and 8 us, or the weight at 3.4 TB/s (us, 64 x 64 / slabs: 64 tokens, 4096 x 2048
    // 12.8 / 18.8, 4096 x 4096 20.9 / 19.8, 16384 x 4096 25.1 / 28.4, 9984 x 7168 38.2 / 30.7, 12544 x 12288 67.3 / 52.8;
    // 128 tokens, 4096 x 4096 20.5 / 23.9, 7168 x 7168 36.3 / 30.1; 39 tokens, 16384 x 9216 with rank 32 55.3 / 60.3).
    const double slabs_ns = 8e3 + best_ns > weight / 3.4e3 ? 8e3 + best_ns : weight / 3.4e3;
    if (one_round_of_64(n, m) && 2e3 + 2.6e3 * (double)K / 512.0 <= slabs_ns) return 0;
    return best < 2 ? 0 : best;
}

// More than 128 tokens on up to half a round of 256 x 128 tiles: slabs on those where they were once estimated a tenth faster
// than whole tiles of the shape with the fewest rounds x operand bytes.
static int slabs_of_a_partial_round(int64_t n, int64_t m, int64_t K) {
    const int64_t tiles = ((m + 255) / 256) * ((n + 127) / 128), quads = (K + 255) / 256;
    if (n <= 128 || !tile_kernel_fits(K) || tiles > RESIDENT / 2) return 0;
    auto step_us = [](int64_t bm, int64_t bn) { return 0.35 + (double)(72 * bm + 128 * bn) / 1e5; };
    double whole = 3.0 + 2.05 * (double)K / 512.0;
    if (!one_round_of_64(n, m)) {
        constexpr int bms[6] = {256, 192, 256, 128, 128, 64}, bns[6] = {256, 256, 128, 128, 64, 128};
        int64_t least = INT64_MAX;
        for (int c = 0; c < 6; ++c) {
            const int64_t rounds = (((m + bms[c] - 1) / bms[c]) * ((n + bns[c] - 1) / bns[c]) + RESIDENT - 1) / RESIDENT;
            if (rounds * (72 * bms[c] + 128 * bns[c]) >= least) continue;
            least = rounds * (72 * bms[c] + 128 * bns[c]);
            whole = (double)rounds * (3.0 + (double)K / 64.0 * step_us(bms[c], bns[c]));
        }
    }
    double least = 0.9 * whole;
    int best = 0;
    for (int64_t sl = 2; sl <= 16 && sl * 4 <= quads && sl * tiles <= RESIDENT; ++sl) {
        const double us = 10.0 + (double)((quads + sl - 1) / sl * 4) * step_us(256, 128) + 8.0 * (double)sl * (double)n * (double)m / 6e6;
        if (us < least) { least = us; best = (int)sl; }
    }
    return best;
}

// Slabs there is room for, 0: none.  The room of a long weight in whole quads of k-steps is always there, any other only where
// the call's scratch with it fits that of slope_spmm_fwd_static (`optional`).
SlabRoom spmm_slab_room(int64_t n, int64_t m, int64_t K) {
    const int slabs = slabs_of_a_long_weight(n, m, K);
    if (slabs) return {slabs, K % 256 != 0, true};
    return {slabs_of_a_partial_round(n, m, K), true, false};
}

// Tiles of the product without a split; of two that take as long the first.  64 x 64 stands for the generic kernel's four groups.
struct SpmmTile { int bm, bn; };
constexpr SpmmTile SPMM_TILES[] = {{256, 256}, {256, 192}, {192, 256}, {192, 192}, {256, 128}, {192, 128},
                                   {128, 128}, {192, 96}, {192, 64}, {128, 96}, {128, 64}};
static bool ring_tile(int bm, int bn) { return bn <= 96 || (bm == 128 && bn == 128); }

// Time of a product on bm x bn tiles, in us: rounds of 256 resident tiles, each of 3.3 us and its k-steps.  A k-step is the
// operand feed of a compute unit, 53 bytes per ns (a little more on the smaller tiles of the ring kernel; up to a fifth more
// with few compute units at work), and takes longer for weight bytes that come from HBM: those that few token tiles share.
// With slabs: the k-steps of one, and the second launch, which reads what the first has written.
// The constants were fitted on weights from HBM and on tiles that read a k-step before they multiplied it, and before wavefronts that
// only load, which take up to 15 % off the tiles up to 256 x 128 (over 70 shapes, most of them in the last-level cache, the whole tile chosen
// is 2.5 % longer than the best in the mean, 21.8 % at most, mostly where that is 64 x 64: see spmm_tile_choice).  Before those, against them the kernels
// took 1.02 (128 x 128) to 1.18 (256 x 192) of the estimate on such weights, 0.91 to 1.12 on those from the cache: over 110
// shapes of 33 to 6000 tokens (512 to 36864 rows, contractions of 128 to 20000), each on five whole tiles and four splits of low
// estimate, the form chosen takes 1.2 % longer than the best one in the mean, more than 10 % in one (65 tokens, 21888 x 7232),
// 1.5 % on weights from the cache.
// Few tokens on many rows are no exception (us, from HBM: 64 tokens, 20480 x 1024 11.2 on 128 x 64, 15.8 on 64 x 64 tiles, several
// to a compute unit; 36864 x 1024 14.6 on 192 x 64, 18.3 and 23.6).
struct TileCost { int64_t tiles; double start, step, less, stream; };   // what does not depend on the slabs
static TileCost tile_cost(int64_t n, int64_t m, int64_t K, int bm, int bn) {
    const int64_t tiles_n = (n + bn - 1) / bn, tiles = ((m + bm - 1) / bm) * tiles_n;
    if (bm == 64)                                             // (half of the last pair's loads go by where K % 128 is not 0)
        return {tiles, 3.0, 0.248 * (1.0 + 0.25 / (double)tiles_n) * (K % 128 ? 1.12 : 1.0), 0.0, 0.0};
    return {tiles, 3.3, (72.0 * bm * (1.0 + 0.54 / (double)tiles_n) + 128.0 * bn) / 53e3,
            ring_tile(bm, bn) && bm * bn != 192 * 96 ? 0.057 : 0.0,
            3.3 + 1.125 * (double)m * (double)K / 6.2e6};                   // one pass over the weight
}
static double launch_us(const TileCost& c, double ksteps, int slabs) {
    const int64_t groups = c.tiles * slabs, rounds = (groups + RESIDENT - 1) / RESIDENT;
    const double idle = 1.0 - 0.2 * (1.0 - (double)groups / (double)(rounds * RESIDENT));
    const double us = (double)rounds * (c.start + ksteps * (c.step * idle - c.less));
    return us < c.stream ? c.stream : us;
}

// the tile of least time and that time
static double best_tile_us(int64_t n, int64_t m, int64_t K, int& bm, int& bn) {
    bm = bn = 64;
    const double ksteps = (double)K / 64.0;
    double least = one_round_of_64(n, m) ? launch_us(tile_cost(n, m, K, 64, 64), ksteps, 1) : 1e300;
    for (const SpmmTile& t : SPMM_TILES) {
        const TileCost cost = tile_cost(n, m, K, t.bm, t.bn);
        double us = launch_us(cost, ksteps, 1);
        if (t.bm == 256 && t.bn == 256) {                     // whole rounds, and a round of 128 x 128 or 256 x 128 tiles with its launch
            const Leftover left = leftover_tiles((int)((m + 255) / 256), (int)((n + 255) / 256), K);
            const bool halves = left.count > RESIDENT / 4;
            TileCost part = tile_cost(n, m, K, halves ? 256 : 128, 128);
            part.tiles = left.count * (halves ? 2 : 4);
            part.stream = 0.0;
            if (left.count) us = launch_us({left.first, cost.start, cost.step, 0.0, cost.stream}, ksteps, 1) + launch_us(part, ksteps, 1) + 3.0;
        }
        if (us < least) { least = us; bm = t.bm; bn = t.bn; }
    }
    return least;
}

// Split of T = X L into workgroups beside the slabs' tiles: on the compute units that their single round leaves idle, and
// not longer than a slab (a chunk of 32 rows of L takes a wavefront about as long as a k-step takes a tile).  The second
// kernel then adds up the sums of T = X L itself, for every 64 features: two launches fewer, as long as its workgroups
// together read at most XL_BESIDE_BYTES of them, about 6 TB/s (128 tokens, rank 128: 28 MB at 9216 x 9216, 10 us; but
// 600 MB at 36864 x 9216 with 16 slabs, 54 us against 15 with T).  With X L in a launch of its own that never pays: 37
// tokens, 9728 x 17664, rank 32 76.5 us, 67.3 with T; 60 tokens, 20480 x 8192 73.1 / 68.5.
constexpr int64_t XL_BESIDE_BYTES = (int64_t)40 << 20;
bool slab_xl_split(int64_t n, int64_t m, int64_t K, int64_t r, const SpmmSplit& split, XlSplit& x) {
    const int64_t groups = ((m + split.bm - 1) / split.bm) * ((n + split.bn - 1) / split.bn) * split.slabs;
    const int64_t tiles = ((n + SK_BI - 1) / SK_BI) * ((r + SK_BJ - 1) / SK_BJ);
    // (each XCD gets its share of both, rounded up: one workgroup too many on one would only start after the round)
    const int64_t idle = (RESIDENT / XCDS - (groups + XCDS - 1) / XCDS) * XCDS;
    if (tiles > idle) return false;
    const int64_t slab_read = (m + 63) / 64 * ((n + 31) / 32 * 32) * r * 4;
    int64_t max_floats = XL_BESIDE_BYTES / slab_read * n * r;
    if (max_floats > (int64_t)(xl_small_scratch_bytes(n, K, r) / 4)) max_floats = (int64_t)(xl_small_scratch_bytes(n, K, r) / 4);
    if (max_floats <= 0) return false;
    // the fewest slabs that take half as long as the product: the kernel after it reads them all for every 64 features
    const int64_t most = slab_steps_of(K, split.slabs) / 2;
    for (int64_t held = n * r; held <= max_floats; held += n * r) {
        x = xl_split(n, K, r, held, idle);
        if (x.steps <= most) return true;
        if (x.slabs * tiles + tiles > idle) break;
    }
    return x.slabs > 0 && x.steps <= 2 * most;
}

// Without T's launches to save, a product that one launch is estimated to take less than this for is left whole: a call of
// two launches takes the host 12.2 us and more whatever the card does in them, one of one launch 8.5 (us a call, whole and
// split: estimate 14.0, 358 tokens, 256 x 3328 14.0, 12.2; 14.3, 767, 896 x 3008 15.8, 14.4; 15.7, 399, 256 x 3840 15.7, 12.9; but
// 10.7, 742, 512 x 2112 12.0, 13.0; 11.0, 487, 1216 x 2176 12.1, 12.9; 12.1, 239, 5760 x 2048 12.8, 17.9).
constexpr double SPLIT_MIN_US = 13.5;
// Split of the product over k within that room, {0, 0, 0}: none.  With an adapter and up to XL_SMALL_MAX_TOKENS tokens a split
// whose launch has room for X L beside its tiles saves the launches of X L: about 8 us and their operands at 4.4 TB/s,
// against 3 for the larger second kernel, or the time of X L, 0.8 us per chunk of 32 rows of L and wavefront, where that is the
// longer.  (70 shapes of 33 to 512 tokens with adapters on up to 14 forms: the one chosen takes 2.2 % longer than the best from HBM,
// 18 % at most.  us: 166 tokens, 1280 x 27008, rank 32 52 in 8 slabs of 128 x 64, X L 53 chunks; 34 in 9 of 192 x 64, 37 in the 11
// that are taken; 264 tokens, 2048 x 14272, rank 64 53 in three of 128 x 64 and 38; 330 tokens, 3328 x 13568, rank 64 64 in three of
// 256 x 128 and 49.)
SpmmSplit spmm_split(int64_t n, int64_t m, int64_t K, int64_t r, const SlabRoom& room) {
    SpmmSplit best = {0, 0, 0};
    if (room.slabs < 2) return best;
    const bool xl = r > 0 && n <= XL_SMALL_MAX_TOKENS;
    int bm, bn;
    double least = best_tile_us(n, m, K, bm, bn);
    if (!xl && least < SPLIT_MIN_US) return best;
    // Whole products of 64 k-steps and more take an eighth longer than estimated beside split ones, on weights from HBM: over 44
    // shapes of 129 to 1024 tokens, k of 4096 to 10000, the form chosen takes 0.4 % longer than the best measured one in the
    // mean, 8.5 % at most, on weights from the last-level cache 2.4 % and 13 %.  us, whole / two or three slabs from
    // HBM and from the cache: 512 tokens, 4096 x 4096 22.3 / 25.0 and 19.5 / 24.0; 700, 2112 x 4160 25.4 / 27.2 and 22.0 / 24.5;
    // 518, 2240 x 4928 29.2 / 27.2 and 24.5 / 23.9; 530, 1792 x 4864 25.2 / 19.7 and 20.5 / 17.9.
    const double xl_first = xl ? 8.0 + 2.0 * (double)(n + r) * (double)K / 4.4e6 : 0.0;
    least = (K >= 4096 ? 1.125 : 1.0) * least + xl_first;
    // On tiles of bm rows, into all numbers of slabs that leave none empty.  (X L is looked at only where it decides.)
    auto consider = [&](const SpmmTile& t, bool one_round) {
        const TileCost cost = tile_cost(n, m, K, t.bm, t.bn);
        const double finish = 0.12 + 8.0 * (double)n * (double)m / 4.84e6;  // the second launch, per slab
        const int most = one_round && cost.tiles * room.slabs > RESIDENT ? (int)(RESIDENT / cost.tiles) : room.slabs;
        for (int sl = 2; sl <= most; ++sl) {
            const int64_t steps = slab_steps_of(K, sl);
            double us = launch_us(cost, (double)steps, sl) + 1.7 + finish * sl;
            if (us + (xl ? 3.0 : 0.0) >= least || (K / 64 + steps - 1) / steps != sl) continue;
            const SpmmSplit c = {t.bm, t.bn, sl};
            XlSplit x;
            if (xl && slab_xl_split(n, m, K, r, c, x)) us = (us > 5.0 + 0.8 * x.steps ? us : 5.0 + 0.8 * x.steps) + 3.0;
            else us += xl_first;
            if (us < least) { least = us; best = c; }
        }
    };
    const SpmmTile tall = {256, n <= 64 ? 64 : 128};
    // A long weight on enough rows: tiles of 256, which ask least often for the tokens, in any number of rounds.  Where all the
    // slabs there is room for fill less than 13/16 of a round of them, the smaller tiles fill it up (us from HBM, 256 x 128 /
    // the smaller tile, workgroups of the former: 134 tokens, 8064 x 7808 48.5 / 38.4, 192; 482, 4096 x 8192 47.0 / 40.2, 192;
    // 327, 3328 x 8960 36.0 / 33.4, 195; 217, 512 x 19456 30.2 / 18.0, 32; from there on the former are as fast on the widest, 256,
    // 9216 x 9216 56.9 / 68, and behind by less: 128, 9216 x 9216 41.6 / 39.9, 216; 100, 5632 x 13056 37.8 / 34.9, 220; 114, 5376 x 16384
    // 46.0 / 40.5, 210).
    if (room.long_weight && K >= 7168 && 16 * ((m + 255) / 256) * ((n + 127) / 128) * room.slabs >= 13 * RESIDENT) {
        least = 1e300;
        consider(tall, false);
        return best;
    }
    consider({128, 64}, true);
    consider({192, 64}, true);
    consider({128, 128}, true);
    if (n > 64 || K >= 7168) consider(tall, false);
    return best;
}

hipError_t launch_spmm_slabs(const bf16_t* B, int64_t n, const bf16_t* A_vals, const uint8_t* A_meta, int64_t m,
                             int64_t K, const SlabAdapter& ad, const SpmmSplit& split, bf16_t* C, float* slabs, hipStream_t s) {
    const int slab_steps = (int)slab_steps_of(K, split.slabs);
    const int nslabs = (int)((K / 64 + slab_steps - 1) / slab_steps);       // <= split.slabs
    const SplitJob job = {nslabs, slab_steps, slabs, ad.T ? nullptr : ad.L, ad.Q, (int)ad.r, ad.x.k_per, ad.x.slabs};
    const bf16_t* A2 = ad.T ? ad.R : nullptr;                 // as stored, k-major
    const int64_t K2 = ad.T ? -ad.r : 0;
    hipError_t e;
    switch (split.bm * 1000 + split.bn) {
        case 128064: e = launch_ring<128, 64>(B, n, A_vals, A_meta, m, K, ad.T, A2, K2, nullptr, s, job); break;
        case 192064: e = launch_ring<192, 64>(B, n, A_vals, A_meta, m, K, ad.T, A2, K2, nullptr, s, job); break;
        case 256064: e = launch_ring<256, 64>(B, n, A_vals, A_meta, m, K, ad.T, A2, K2, nullptr, s, job); break;
        case 128128: e = launch_ring<128, 128>(B, n, A_vals, A_meta, m, K, ad.T, A2, K2, nullptr, s, job); break;
        default: e = launch_tile<256, 128>(B, n, A_vals, A_meta, m, K, ad.T, A2, K2, nullptr, s, job); break;
    }
    if (e != hipSuccess) return e;
    if (ad.r && !ad.T) return launch_adapter_finish(slabs, nslabs, n, m, ad.Q, ad.x.slabs, ad.R, ad.r, C, s);
    const size_t count4 = (size_t)n * (size_t)m / 4;
    slab_reduce_kernel<<<dim3((unsigned)((count4 + 255) / 256)), dim3(256), 0, s>>>((const f32x4*)slabs, nslabs, count4,
                                                                                   (u32x2*)C);
    return hipGetLastError();
}

int spmm_generic_edge(int64_t n, int64_t m) { return tiles_of_64(n, m) <= 2 * RESIDENT ? 64 : 128; }

// Where the estimate prefers 64 x 64 tiles on a contraction of more k-steps than this, the ring kernel on 128 x 64, with half as many workgroups, is the
// faster one
//  - where an odd last k-step leaves the generic kernel (us, generic / 128 x 64: 43 tokens, 4160 x 1728 15.2 / 12.3 on operands from the last-level
//    cache, 15.3 / 13.2 from HBM; 37 products without an adapter are 17 and 13 % faster in the mean, 42 with one 6 and 3 %);
//  - on operands from the last-level cache, more so the longer they are, while from HBM it is 5 % slower without an adapter, 7 to 10 % with one: so from the
//    bytes of operands on where it gains more than it loses.  us, 64 x 64 / 128 x 64 cached and from HBM: 112 tokens, 512 x 1280 10.8 / 11.2 and
//    9.2 / 10.3; 231, 1272 x 2432 15.0 / 14.1 and 14.0 / 15.5; 1214, 424 x 2432 16.1 / 14.1 and 14.7 / 15.4; 1019, 576 x 3328 20.4 / 16.8 and 18.9
//    / 19.6; with an adapter 68, 4864 x 2560, rank 128, a call, cached 20.0 / 19.5.  Mean over 150 products without an adapter below / above the line: 0 / 11 %
//    faster cached, 8 / 5 % slower from HBM; over 179 with one 1 % slower / 3 % faster cached, 9 / 8 % slower from HBM.
constexpr int64_t LONGEST_OF_64 = 16 * 64;
constexpr double FEWEST_BYTES = 2.5e6, FEWEST_BYTES_WITH_ADAPTER = 5e6;

// Tile of the product for n tokens, m sparse rows, contraction K: bm = bn = 0 means the generic kernel, whose whole pairs of
// k-steps on a round of 64 x 64 tiles count as a tile shape of their own.
void spmm_tile_choice(int64_t n, int64_t m, int64_t K, bool adapter, int& bm, int& bn) {
    bm = bn = 0;
    if (!tile_kernel_fits(K)) return;
    best_tile_us(n, m, K, bm, bn);
    if (bm != 64) return;
    // (whether a product is split is decided by the estimate as it stands; not up to 64 rows, where half of the taller tile is nothing)
    const double bytes = (double)K * (1.125 * (double)m + 2.0 * (double)n);
    if (K > LONGEST_OF_64 && m > 64 && (K % 128 != 0 || bytes >= (adapter ? FEWEST_BYTES_WITH_ADAPTER : FEWEST_BYTES))) { bm = 128; bn = 64; }
    else if (K % 128 != 0 && one_round_of_64(n, m)) bm = bn = 0;
}

// Tokens at the end of a batch that a pass of the small-batch kernel over the packed weight (5 TB/s, 6 us for its launch and
// the drained chip before it) takes for less than the round of tiles that they begin (0: none): up to 32 beyond a multiple
// of the tile kernels' 256 or 128 (777 tokens, 20480 x 5120: 139 us in two rounds of tiles, 80 + 25 for 768 and 9 tokens).
int64_t spmm_rest_tokens(int64_t n, int64_t m, int64_t K) {
    if (n <= 128 || !tile_kernel_fits(K) || one_round_of_64(n, m)) return 0;
    int bm, bn;
    double least = best_tile_us(n, m, K, bm, bn);
    int64_t best = 0;
    for (int64_t edge = 256; edge >= 128; edge /= 2) {
        const int64_t rest = n % edge;
        if (rest == 0 || rest > STREAM_MAX_TOKENS || rest == n) continue;
        const double us = best_tile_us(n - rest, m, K, bm, bn) + 1.125 * (double)m * (double)K / 5e6 + 6.0;
        if (us < 0.95 * least) { least = us / 0.95; best = rest; }
    }
    return best;
}

static hipError_t launch_tiles(const bf16_t* B, int64_t n, const bf16_t* A_vals, const uint8_t* A_meta, int64_t m, int64_t K,
                               const bf16_t* B2, const bf16_t* A2, int64_t K2, bf16_t* C, hipStream_t s) {
    int bm, bn;
    spmm_tile_choice(n, m, K, K2 != 0, bm, bn);
    if (bm == 0) {
        return launch_generic(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
    }
    switch (bm * 1000 + bn) {
        case 256256: return launch_split(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        case 256192: return launch_tile<256, 192>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        case 192256: return launch_tile<192, 256>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        case 192192: return launch_tile<192, 192>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        case 256128: return launch_tile<256, 128>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        case 192128: return launch_tile<192, 128>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        case 128128: return launch_ring<128, 128>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        case 192096: return launch_ring<192, 96>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        case 192064: return launch_ring<192, 64>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        case 128096: return launch_ring<128, 96>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        case 128064: return launch_ring<128, 64>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
        default: return launch_generic_as<2, 4>(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);     // 64 x 64
    }
}

hipError_t launch_spmm(const bf16_t* B, int64_t n, const bf16_t* A_vals, const uint8_t* A_meta, int64_t m, int64_t K,
                       const bf16_t* B2, const bf16_t* A2, int64_t K2, bf16_t* C, hipStream_t s) {
    const int64_t rest = K2 <= 0 ? spmm_rest_tokens(n, m, K) : 0;  // (the small-batch kernel takes A2 k-major)
    n -= rest;
    hipError_t e = launch_tiles(B, n, A_vals, A_meta, m, K, B2, A2, K2, C, s);
    if (e != hipSuccess || rest == 0) return e;
    // second, so that it finds the packed weight in the last-level cache (777 tokens: the other way round 6 us slower)
    return launch_spmm_stream(B + n * K, rest, A_vals, A_meta, m, K, B2 ? B2 - n * K2 : nullptr, A2, -K2, C + n * m, nullptr, s);
}
