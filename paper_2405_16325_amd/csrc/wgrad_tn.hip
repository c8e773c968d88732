// Dense products on MFMA tiles: the weight gradient dW = dY^T X (Eq. 5) with the prune-and-compress step of Algorithm 1
// line 13 folded into the epilogue, the skinny products of the adapters, products of masked dense weights.
//
// The contraction of the gradients runs over the b tokens, the slow index of both operands in memory, and the tiles read
// them as they are stored: [token][feature] panels in LDS, fragments through the transposing LDS read (dense.h).  Only
// where the matrix pipes would wait for those reads are operands copied into token-contiguous form first (wgrad_copies),
// and callers that share an operand between layers may make such copies themselves:
//     Xt [d_in ][ld],  dYt[d_out][ld],   bp = b rounded up to 64, the tail zero-filled,
//     ld = row pitch: bp, plus one 128-byte line where bp * 2 is a multiple of 4 KiB (rows that
//     far apart crowd the same L2 channels: the padded pitch is 2-3 % faster at b = 16384)
// The product
//     D[i, j] = sum_t X[t, i] * dY[t, j]
// runs with the same machinery as the sparse kernels: 8 wavefronts, all of which load and multiply or, up to 256 x 128, four multiply and
// four load, with one barrier per k-step or in two groups half a k-step apart (dense_tn_sums), global -> LDS loads of full 128-byte lines, conflict-free LDS reads in MFMA order, v_mfma_f32_16x16x32_bf16.
// D rows are d_in and D columns d_out, so a lane's four accumulators (column l%16, rows
// 4*(l/16) .. +3) are exactly one group of four of W^R's row: the epilogue picks two of them with
// the group's metadata nibble and stores one 4-byte pair of the packed gradient.
#include <cmath>
#include <numeric>
#include <type_traits>

#include "dense.h"

namespace {

// out[c][r] = in[r][c] for r < rows, zero for rows <= r < rows_pad; in is [rows][cols] bf16 with
// cols % 8 == 0, out is [cols] rows of pitch ld >= rows_pad, rows_pad % 64 == 0, ld % 8 == 0.
// Tiles of TP_ROWS rows x 64 columns through LDS, 16-byte global accesses on both sides, non-temporal (116.9 -> 99.4 us
// for 16384 x 9216 alone, 8 % inside a training step); consecutive workgroups go down the rows, so that every output
// row is written front to back.  One launch takes one or two matrices one after the other (the operands of a product).
constexpr int TP_ROWS = 64;                                   // 128 and 256 measured the same
struct TransposeJob {
    const bf16_t* in;
    bf16_t* out;
    int cols, rows, rows_pad, ld, tiles;                      // no tiles: no matrix
};
inline TransposeJob transpose_job(const bf16_t* in, int64_t rows, int64_t cols, int64_t rows_pad, int64_t ld, bf16_t* out) {
    return {in, out, (int)cols, (int)rows, (int)rows_pad, (int)ld, (int)(((rows_pad + TP_ROWS - 1) / TP_ROWS) * ((cols + 63) / 64))};
}

__global__ void __launch_bounds__(256) transpose_pad_kernel(TransposeJob j0, TransposeJob j1) {
    __shared__ bf16_t tile[64][TP_ROWS + 2];
    int64_t w = flat_block();
    const bool first = w < j0.tiles;
    const TransposeJob j = first ? j0 : j1;
    w -= first ? 0 : j0.tiles;
    if (w >= j.tiles) return;
    const bf16_t* __restrict__ in = j.in;
    bf16_t* __restrict__ out = j.out;
    const int row_tiles = (j.rows_pad + TP_ROWS - 1) / TP_ROWS, r0 = (int)w % row_tiles * TP_ROWS, c0 = (int)w / row_tiles * 64;
    const int t = threadIdx.x;
#pragma unroll
    for (int p = 0; p < TP_ROWS / 32; ++p) {
        int r = (t >> 3) + 32 * p, c8 = (t & 7) * 8;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (r0 + r < j.rows && c0 + c8 < j.cols) v = __builtin_nontemporal_load((const u32x4*)(in + (size_t)(r0 + r) * j.cols + c0 + c8));
#pragma unroll
        for (int e = 0; e < 8; ++e) tile[c8 + e][r] = (bf16_t)(v[e >> 1] >> (16 * (e & 1)));
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < TP_ROWS / 32; ++p) {
        int idx = t + 256 * p, c = idx / (TP_ROWS / 8), r8 = (idx % (TP_ROWS / 8)) * 8;
        if (c0 + c >= j.cols || r0 + r8 >= j.rows_pad) continue;
        const uint32_t* src = (const uint32_t*)&tile[c][r8];
        u32x4 v = {src[0], src[1], src[2], src[3]};
        __builtin_nontemporal_store(v, (u32x4*)(out + (size_t)(c0 + c) * j.ld + r0 + r8));
    }
}

inline hipError_t launch_transposes(const TransposeJob& j0, const TransposeJob& j1, hipStream_t s) {
    const int64_t tiles = (int64_t)j0.tiles + j1.tiles;
    transpose_pad_kernel<<<grid_of(tiles), dim3(256), 0, s>>>(j0, j1);
    return hipGetLastError();
}

// pitch (elements) of a token-contiguous copy with bp tokens per row
inline int64_t token_pitch(int64_t bp) { return (bp * 2) % 4096 == 0 ? bp + 64 : bp; }

template <int BM, int BN, int NS>
struct TnSmem {
    static constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128;   // one k-step of 64
    static constexpr int STAGE = A_BYTES + B_BYTES;
    static constexpr int TOTAL = NS * STAGE;                       // ring of NS stages
};

constexpr int TN_THREADS = 512;
// Wavefronts of a tile.  Up to 256 x 128 four of them only load (why: spmm_ring_kernel) and load nothing past the end, and four multiply,
// with a quarter of the tile each: a third fewer bytes from LDS in all than eight, which on operands as stored, by the transposing reads, take
// longer than the products.  us, from memory, eight that do both / four and four: dW of 1024 x 1024 over 4096 tokens on 64 x 64 19.4 / 16.9,
// 3072 x 768 over 2048 on 128 x 128 18.7 / 17.0, 4096 x 2048 over 4096 on 256 x 128 59.5 / 56.6, 2816 x 2816 59.9 / 56.0; masked dense 704 x 768 over
// 518 5.1 / 4.8, 3072 x 2048 over 2048 on 192 x 128 24.6 / 22.9; the gradients of 3136 x 896, rank 64 over 14376 tokens 187 / 182.  On 192 x
// 192, where their registers just suffice: 2112 x 4160 over 700 15.9 / 17.3.
constexpr int TN_LOADERS = 4;
constexpr int tn_loaders(int bm, int bn) { return bm * bn <= 256 * 128 ? TN_LOADERS : 0; }
constexpr int tn_mult(int bm, int bn) { return tn_loaders(bm, bn) ? 4 : 8; }
constexpr int tn_threads(int bm, int bn) { return 64 * (tn_mult(bm, bn) + tn_loaders(bm, bn)); }
enum { EPI_MASKED_PACKED = 0, EPI_PLAIN = 1 };

// Metadata of the 32 Q columns of W^R from c (a multiple of 32) of rows o, o + 16, .. of N, by dwords; columns outside the matrix: any.  The
// dwords of rows that are not a multiple of 32 columns may lie at any byte, and the last of such a row, which ends inside it, is read by
// bytes.  All rows' loads leave together: row after row each costs a trip to memory.
template <int N, int Q>
__device__ __forceinline__ void load_meta(const uint8_t* __restrict__ meta, int o, int c, int m, int n, uint32_t (&w)[N][Q]) {
    typedef uint32_t __attribute__((aligned(1))) u32_a1;
    const uint8_t* const p = meta + (size_t)o * (m / 8) + c / 8;
    const size_t next = (size_t)16 * (m / 8);
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int q = 0; q < Q; ++q) w[j][q] = o + 16 * j < n && c + 32 * q + 32 <= m ? *(const u32_a1*)(p + j * next + 4 * q) : 0u;
    if (m % 32 != 0 && c < m && c + 32 * Q > m) {             // uniform
        const int bytes = m / 8 % 4;
        uint32_t v[N][3];
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int e = 0; e < 3; ++e) v[j][e] = e < bytes && o + 16 * j < n ? p[j * next + (m - c) / 32 * 4 + e] : 0u;
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int q = 0; q < Q; ++q) w[j][q] = q == (m - c) / 32 ? v[j][0] | v[j][1] << 8 | v[j][2] << 16 : w[j][q];
    }
}

// Masked, packed epilogue: acc[i][j] of a wavefront is the 16 x 16 fragment at D rows c0 + 16 i (d_in) and D
// columns o0 + 16 j (d_out).  A lane's four accumulators are one group of four along d_in of row o: the
// group's metadata nibble picks the two that W^R keeps.  Stored straight from the registers a pair is a
// 4-byte piece and an instruction touches sixteen rows; so the workgroup's tile of pairs goes through LDS
// (the rings are idle) as [d_out row][pair] and leaves in whole rows, 16 bytes per lane.
// BMT x BNT = the workgroup's tile (d_in x d_out) at (tile_c0, tile_o0); every thread must make the call.
template <int MF, int NF, int BMT, int BNT, int THREADS>
__device__ __forceinline__ void store_masked_packed(const f32x4 (&acc)[MF][NF], int m, int n, int c0, int o0,
                                                    int tile_c0, int tile_o0, int l16, int lq,
                                                    const uint8_t* __restrict__ meta, bf16_t* __restrict__ out,
                                                    uint8_t* smem) {
    constexpr int WM = MF * 16;
    constexpr int CP = BMT + 16;                              // bytes per staged row of pairs: 16 rows x 4 lanes x 4 B
                                                              // of one store fall on 64 different banks
    const size_t gpitch = (size_t)m / 2;
    __syncthreads();                                          // every wavefront is done with the rings
    // Columns whose metadata is loaded together.  With four wavefronts a wavefront has twice the columns, and column after column each
    // paid a trip to memory; with eight, all together are slower.  (163 gradients of up to 1e10 products, from memory, time one by one over all
    // together, up to 8 k-steps and beyond 40: 64 x 128 1.08 and 1.03, 128 x 128 1.06 and 1.02, 192 x 128 1.04 and 1.02, 256 x 128 1.03 and
    // 1.02, 64 x 64 1.03 and 1.02; the tiles of eight, 123 gradients, 256 x 256 0.98 and 0.99, 256 x 192 0.99 and 1.00, 192 x 192 1.00.  us: 281 tokens,
    // 768 x 8960 11.6 / 11.3; 533, 1360 x 856 9.8 / 9.5.)
    constexpr int TOGETHER = THREADS < 512 ? NF : 1;
#pragma unroll
    for (int j0 = 0; j0 < NF; j0 += TOGETHER) {
        // of the wavefront's WM d_in columns of each row: WM / 4 groups = WM / 8 bytes
        uint32_t mw[TOGETHER][WM / 32];
        load_meta(meta, o0 + j0 * 16 + l16, c0, m, n, mw);
#pragma unroll
        for (int jj = 0; jj < TOGETHER; ++jj) {
            const int j = j0 + jj, o = o0 + j * 16 + l16;
#pragma unroll
            for (int i = 0; i < MF; ++i) {
                int gl = i * 4 + lq;                          // group index inside the WM columns
                uint32_t nib = (mw[jj][i >> 1] >> (4 * (gl & 7))) & 0xFu;
                uint32_t a = nib & 3u, c = nib >> 2;
                f32x4 v = acc[i][j];
                float v0 = a == 0 ? v[0] : (a == 1 ? v[1] : v[2]);
                float v1 = c == 1 ? v[1] : (c == 2 ? v[2] : v[3]);
                union { __bf16 h[2]; uint32_t u; } pr;
                pr.h[0] = (__bf16)v0;
                pr.h[1] = (__bf16)v1;
                *(uint32_t*)(smem + (o - tile_o0) * CP + ((c0 - tile_c0) / 4 + gl) * 4) = pr.u;
            }
        }
    }
    __syncthreads();
    // 16-byte pieces (four pairs = sixteen columns of W), all read from LDS before the first is stored; the last of a row that is not
    // a multiple of 16 columns is a half one
    constexpr int PPR = BMT / 16, PIECES = BNT * PPR, PER_THREAD = (PIECES + THREADS - 1) / THREADS;
    constexpr bool EVEN = PIECES % THREADS == 0;           // else the last round of pieces is for the first threads only
    u32x4 piece[PER_THREAD];
#pragma unroll
    for (int u = 0; u < PER_THREAD; ++u) {
        const int idx = (int)threadIdx.x + u * THREADS;
        if (EVEN || idx < PIECES) piece[u] = *(const u32x4*)(smem + (idx / PPR) * CP + (idx % PPR) * 16);
    }
#pragma unroll
    for (int u = 0; u < PER_THREAD; ++u) {
        const int idx = (int)threadIdx.x + u * THREADS;
        const int o = tile_o0 + idx / PPR, col = tile_c0 + (idx % PPR) * 16;
        if ((EVEN || idx < PIECES) && o < n && col + 16 <= m) *(u32x4_a8*)(out + (size_t)o * gpitch + (col >> 1)) = piece[u];
    }
    if (m % 16 == 0) return;                                  // uniform
#pragma unroll
    for (int u = 0; u < PER_THREAD; ++u) {
        const int idx = (int)threadIdx.x + u * THREADS;
        const int o = tile_o0 + idx / PPR, col = tile_c0 + (idx % PPR) * 16;
        if ((EVEN || idx < PIECES) && o < n && col + 8 == m) *(u32x2*)(out + (size_t)o * gpitch + (col >> 1)) = (u32x2){piece[u][0], piece[u][1]};
    }
}

// The fp32 accumulators into partial[n][m] for a later reduction.
template <int MF, int NF>
__device__ __forceinline__ void store_sums(const f32x4 (&acc)[MF][NF], int m, int n, int c0, int o0, int l16, int lq,
                                           float* __restrict__ partial) {
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        int row = o0 + j * 16 + l16;
        if (row >= n) continue;
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            int col = c0 + i * 16 + lq * 4;
            if (col < m) *(f32x4*)(partial + (size_t)row * m + col) = acc[i][j];
        }
    }
}

// acc = the tile at (m0, n0) of D[i, j] = sum_k At[i, k] * Bt[j, k] over the k-steps [k_begin, k_end), of ksteps k-steps of 64 in
// all (the look-ahead past a slab's end reads real, unused data).  AKM, BKM: the operand is k-major.
// NS = ring depth: loads run NS - 1 k-steps ahead.  Two stages are all that fits beside a 256 x 256
// tile; small tiles (memory-bound skinny products) take a deeper ring to cover the HBM latency.
// Every thread of the workgroup must make the call; wavefront w holds the fragments at rows w % 2 * BM / 2, columns w / 2 * WROWS.
// False: a wavefront that has only loaded, and is done.
template <int BM, int BN, int NS, bool AKM, bool BKM>
__device__ __forceinline__ bool dense_tn_sums(const DenseOperand& At, const DenseOperand& Bt, int ksteps, int k_begin, int k_end, int m0,
                                              int n0, uint8_t* smem, f32x4 (&acc)[BM / 32][BN / (8 * tn_mult(BM, BN))]) {
    using S = TnSmem<BM, BN, NS>;
    constexpr int MULT = tn_mult(BM, BN), WROWS = BN / (MULT / 2);
    constexpr int MF = BM / 32, NF = WROWS / 16;             // 16 x 16 fragments per wavefront (2 x 4 or 2 x 2 waves)
    constexpr int LD_A = BM / 64, LD_B = BN / 64;            // 1 KiB loads per wavefront per step
    constexpr int AHEAD = (NS - 2) * (LD_A + LD_B);          // loads that may stay in flight at a wait
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    constexpr bool LOADERS = tn_loaders(BM, BN) != 0;
    // The first k-steps' loads are shared out to eight as they would be without loaders, of whom the multiplying wavefronts are the first: four
    // loaders alone took long to fill the ring (us, from memory, by themselves / so: masked dense 768 x 704 over 518 5.0 / 4.7, 576 x 1408 over
    // 1625 7.8 / 7.5; dW of 1000 x 1000 over 1000 9.5 / 9.3, 1024 x 1024 over 4096 17.3 / 17.0; eight, no loaders: 5.0, 7.7, 9.3, 19.0).  No more
    // steps than the ring holds ahead: a third one on 256 x 128 was loaded twice, which took 0.3 to 1.8 % more on 8 to 20 k-steps.
    constexpr int PRE = NS - 1 < 3 ? NS - 1 : 3;              // (what `behind` is asked for knows)
    static_assert(PRE <= NS - 1, "the steps that are shared out are among those loaded before the loop, so that each is loaded once");
    constexpr int LAST = (NS - 1) * S::STAGE;
    if (LOADERS && wave >= MULT) {
        constexpr int EACH = 8 / TN_LOADERS;                  // a loader has the loads of so many of the eight
        // loads behind step k_begin + s, those of the NS - 2 steps after it
        constexpr auto behind = [](int s) {
            int c = 0;
            for (int p = s + 1; p <= s + NS - 2; ++p) c += (LD_A + LD_B) * (p < PRE ? EACH - MULT / TN_LOADERS : EACH);
            return c;
        };
        DenseLoader<AKM, BKM, BM, BM / 2> la[EACH];
        DenseLoader<BKM, AKM, BN, WROWS> lb[EACH];
        auto load_a = [&](int v, int ks, int at) {
#pragma unroll
            for (int i = 0; i < LD_A; ++i) la[v].load(ks, i, smem, at, wave - MULT + v * TN_LOADERS);
        };
        auto load_b = [&](int v, int ks, int at) {
#pragma unroll
            for (int i = 0; i < LD_B; ++i) lb[v].load(ks, i, smem, at + S::A_BYTES, wave - MULT + v * TN_LOADERS);
        };
        auto issue = [&](int ks, int at, int from) {          // the loads of the eight from `from` on
#pragma unroll
            for (int v = 0; v < EACH; ++v)
                if (v * TN_LOADERS >= from) {
                    load_a(v, ks, at);
                    load_b(v, ks, at);
                }
        };
#pragma unroll
        for (int v = 0; v < EACH; ++v) {
            la[v].init(At, m0, 0, wave - MULT + v * TN_LOADERS, lane, 0, ksteps, smem);
            lb[v].init(Bt, n0, 0, wave - MULT + v * TN_LOADERS, lane, 0, ksteps, smem);
        }
#pragma unroll
        for (int p = 0; p < NS - 1; ++p)
            if (k_begin + p < k_end) issue(k_begin + p, p * S::STAGE, p < PRE ? MULT : 0);
        int at = LAST;
        for (int ks = k_begin; ks < k_end; ++ks) {
            // step ks has landed (in the last NS - 2 steps there are fewer loads behind it: then all are waited for) and everybody has
            // read the one before it, whose stage is filled again
            if (ks + NS - 2 >= k_end) WAIT_HERE(waitcnt_imm(0, 15));
            else if (ks == k_begin) WAIT_HERE(waitcnt_imm(behind(0), 15));
            else if (ks == k_begin + 1) WAIT_HERE(waitcnt_imm(behind(1), 15));
            else WAIT_HERE(waitcnt_imm(behind(2), 15));
            wg_barrier();
            if (ks + NS - 1 < k_end) issue(ks + NS - 1, at, 0);
            at = at == LAST ? 0 : at + S::STAGE;
        }
        return false;
    }
    DenseLoader<AKM, BKM, BM, BM / 2> opa;
    DenseLoader<BKM, AKM, BN, WROWS> opb;
    opa.init(At, m0, (wave & 1) * (BM / 2), wave, lane, 0, ksteps, smem);
    opb.init(Bt, n0, (wave >> 1) * WROWS, wave, lane, 0, ksteps, smem);
    auto issue = [&](int ks, int at) {                       // k-step ks (clamped) into the stage at byte `at`
#pragma unroll
        for (int i = 0; i < LD_A; ++i) opa.load(ks, i, smem, at, wave);
#pragma unroll
        for (int i = 0; i < LD_B; ++i) opb.load(ks, i, smem, at + S::A_BYTES, wave);
    };

#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // The stage that is read, as a byte offset that wraps.  As (ks % NS) * STAGE it became a multiply-high and subtractions per
    // lane before every step's LDS reads (us, from HBM: 2048 x 1024 over 4096 on 64 x 128 30.5 -> 26.0, 704 x 2112 over 4160
    // 27.0 -> 22.2, 2048 x 1024 over 8192 51.8 -> 41.8); the 256 x 256 kernel, where registers are short, is 1 % slower this way.
    int at = 0;
    if (LOADERS) {
#pragma unroll
        for (int p = 0; p < PRE; ++p)
            if (k_begin + p < k_end) issue(k_begin + p, p * S::STAGE);
        if (k_begin + PRE - 1 < k_end) WAIT_HERE(waitcnt_imm((PRE - 1) * (LD_A + LD_B), 15));
        else WAIT_HERE(waitcnt_imm(0, 15));
    } else {
#pragma unroll
        for (int p = 0; p < NS - 1; ++p) issue(k_begin + p, p * S::STAGE);
        WAIT_HERE(waitcnt_imm(AHEAD, 15));                    // the first step has landed (this wave's share)
    }
    wg_barrier();
    // Two schedules of a k-step.  One barrier, the fragments of a half of the k-step read while the other half is multiplied (us, operands in
    // the last-level cache, in two phases / so: 64 x 64, 1024 x 1024 over 4096 tokens 23.9 / 21.0; 128 x 128, 3072 x 768 over 2048 tokens 22.4 / 20.6;
    // 192 x 192, 1024 x 2048 over 4096 47.9 / 42.7; 256 x 128, 4096 x 4096 over 4096 tokens 129 / 120).  Where the ring has two stages two
    // phases, as in the 256 x 256 kernel, so that loads are queued later (256 x 192, 5120 x 6464 over 752 tokens: 62.7 against 65.3).
    if constexpr (!LOADERS && NS == 2) {
        const int group = wave >> 2;
        // One k-step.  Loads of step s + NS - 1 are queued in the even phase in which their stage, last
        // read for step s - 1, has just been released: group 0 is then in its memory phase of step s,
        // group 1 in its compute phase of step s - 1.  One phase later every wavefront waits until only
        // the loads of steps beyond s + 1 are outstanding, before the barrier after which group 0 reads
        // step s + 1.
#define TN_STEP(G)                                                                                         \
        {                                                                                                  \
            const auto sa = opa.stage(smem, at);                                                           \
            const auto sb = opb.stage(smem, at + S::A_BYTES);                                              \
            BFrag af[MF], bf[NF];                                                                          \
            _Pragma("unroll") for (int i = 0; i < MF; ++i) af[i] = opa.frag(sa, i);                        \
            _Pragma("unroll") for (int j = 0; j < NF; ++j) bf[j] = opb.frag(sb, j);                        \
            if (G == 0) issue(ks + NS - 1, at == 0 ? LAST : at - S::STAGE);                                \
            /* all LDS reads of this stage have returned before anybody may overwrite it */                \
            WAIT_HERE(waitcnt_imm(G == 1 ? AHEAD : 63, 0));                                                \
            wg_barrier();                                                                                  \
            if (G == 1) issue(ks + NS, at);                                                                \
            /* before the MFMAs: among them, where the compiler may put these loads, they land 5 to 8 % later */\
            if (G == 1) __builtin_amdgcn_sched_barrier(0);                                                 \
            _Pragma("unroll") for (int h = 0; h < 2; ++h)                                                  \
            _Pragma("unroll") for (int i = 0; i < MF; ++i) _Pragma("unroll") for (int jj = 0; jj < NF; ++jj) {\
                const int j = (i & 1) ? NF - 1 - jj : jj;         /* back and forth: one operand changes per MFMA */\
                AFrag a, b;                                                                                \
                a.u = af[i].u[h]; b.u = bf[j].u[h];                                                        \
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, acc[i][j], 0, 0, 0);         \
            }                                                                                              \
            if (G == 0) WAIT_HERE(waitcnt_imm(AHEAD, 15));                                                 \
            wg_barrier();                                                                                  \
            at = at == LAST ? 0 : at + S::STAGE;                                                           \
        }
        if (group == 0) {
            for (int ks = k_begin; ks < k_end; ++ks) TN_STEP(0)
            wg_barrier();
        } else {
            issue(k_begin + NS - 1, LAST);
            wg_barrier();
            for (int ks = k_begin; ks < k_end; ++ks) TN_STEP(1)
        }
#undef TN_STEP
    } else {
        struct Half { u32x4 a[MF], b[NF]; };                  // fragments of half a k-step
        constexpr int READS = MF + NF, LOADS = LOADERS ? 0 : LD_A + LD_B, MFMAS = MF * NF;
        auto read_one = [&](Half& f, const auto& sa, const auto& sb, int h, int x) {
            if (x < NF) f.b[x] = opb.half(sb, x, h);
            else f.a[x - NF] = opa.half(sa, x - NF, h);
        };
        auto load_one = [&](int ks, int x) {                  // into the stage at `at`
            if (x < LD_A) opa.load(ks, x, smem, at, wave);
            else opb.load(ks, x - LD_A, smem, at + S::A_BYTES, wave);
        };
        // The products of f and P pieces of other work: spread among them, or before them where they are few (64 x 64 tiles, spread:
        // 22.7 us for 21.0; 256 x 128, not spread: 60.5 for 48.7)
        constexpr bool SPREAD = MFMAS > 8;
        auto multiply = [&](const Half& f, auto pieces, auto piece) {
            constexpr int P = decltype(pieces)::value, PER = (P + MFMAS - 1) / MFMAS;
            if (!SPREAD) {
#pragma unroll
                for (int x = 0; x < P; ++x) {
                    if (x == READS) __builtin_amdgcn_sched_barrier(0);
                    piece(x);
                }
                if (P <= READS) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int q = 0; q < MFMAS; ++q) {
                const int i = q / NF, j = (i & 1) ? NF - 1 - q % NF : q % NF;   // back and forth: one operand changes per MFMA
                AFrag a, b;
                a.u = f.a[i]; b.u = f.b[j];
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, acc[i][j], 0, 0, 0);
                if (!SPREAD) continue;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int x = q * PER; x < (q + 1) * PER; ++x)
                    if (x < P) piece(x);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        Half f0, f1;
        {
            const auto sa = opa.stage(smem, 0);
            const auto sb = opb.stage(smem, S::A_BYTES);
#pragma unroll
            for (int x = 0; x < READS; ++x) read_one(f0, sa, sb, 0, x);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!LOADERS) issue(k_begin + NS - 1, LAST);
        WAIT_HERE(waitcnt_imm(63, 0));                        // (else the compiler waits for all reads at the head of the loop)
        auto first_half = [&] {
            const auto sa = opa.stage(smem, at);
            const auto sb = opb.stage(smem, at + S::A_BYTES);
            multiply(f0, std::integral_constant<int, READS>{}, [&](int x) { read_one(f1, sa, sb, 1, x); });
        };
        // With loaders nothing follows the last k-step, which comes after the loop.  (On up to 64 x 128 it stays inside: 1024 x 4096 over
        // 2048 20.2 / 21.4 after it, while leaving the loop from inside costs larger tiles copies of their sums: 3072 x 768 over 2048 17.6 / 17.0)
        constexpr bool AFTER = LOADERS && BM * BN > 64 * 128;
        const int full = AFTER ? k_end - 1 : k_end;
        for (int ks = k_begin; ks < full; ++ks) {
            first_half();
            if (LOADERS && !AFTER && ks + 1 == k_end) {
                multiply(f1, std::integral_constant<int, 0>{}, [](int) {});
                break;
            }
            // this wavefront has read the stage, and its loads of the next one (with loaders: of the first ones) have landed
            WAIT_HERE(waitcnt_imm(LOADERS ? 0 : AHEAD, 0));
            wg_barrier();
            const int next = at == LAST ? 0 : at + S::STAGE;
            const auto sa = opa.stage(smem, next);            // (after the last k-step read and not used)
            const auto sb = opb.stage(smem, next + S::A_BYTES);
            multiply(f1, std::integral_constant<int, READS + LOADS>{}, [&](int x) {
                if (x < READS) read_one(f0, sa, sb, 0, x);
                else load_one(ks + NS, x - READS);            // into the stage that everybody has read
            });
            at = next;
        }
        if (AFTER) {
            first_half();
            multiply(f1, std::integral_constant<int, 0>{}, [](int) {});
        }
    }
    if (!LOADERS) WAIT_HERE(waitcnt_imm(0, 15));              // drain the clamped look-ahead loads
    return true;
}

// D[i, j] = sum_k At[i, k] * Bt[j, k] over ksteps k-steps of 64;  At: m rows, Bt: n rows.
//   EPI_MASKED_PACKED: out = packed gradient [n][m/2] selected by meta (u8[n][m/8])
//   EPI_PLAIN        : out = bf16 [n][m]  (row j, four consecutive i per lane)
template <int BM, int BN, int EPI, int NS, bool AKM, bool BKM>
__global__ void __launch_bounds__(tn_threads(BM, BN)) dense_tn_kernel(DenseOperand At, DenseOperand Bt, int ksteps, const uint8_t* __restrict__ meta,
                                                              bf16_t* __restrict__ out, int tiles_m, int tiles_n) {
    using S = TnSmem<BM, BN, NS>;
    constexpr int MULT = tn_mult(BM, BN), MF = BM / 32, NF = BN / (8 * MULT);
    extern __shared__ __align__(16) uint8_t smem[];
    fetch_arguments(At.p, At.rows, At.ld, At.k, Bt.p, Bt.rows, Bt.ld, Bt.k, ksteps, meta, out, tiles_m, tiles_n);
    int tm, tn;
    if (!tile_of_block(tiles_m, tiles_n, tm, tn)) return;
    const int m0 = tm * BM, n0 = tn * BN, lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), mw = m0 + (wave & 1) * (BM / 2), nw = n0 + (wave >> 1) * (BN / (MULT / 2));
    const int m = At.rows, n = Bt.rows;
    f32x4 acc[MF][NF];
    if (!dense_tn_sums<BM, BN, NS, AKM, BKM>(At, Bt, ksteps, 0, ksteps, m0, n0, smem, acc)) return;
    if constexpr (EPI == EPI_PLAIN) {
        static_assert(BN * (BM * 2 + 16) <= S::TOTAL, "the staged output tile fits in the ring");
        store_rows<MF, NF, BM, BN, 64 * MULT>(acc, mw, nw, m, n, l16, lq, out, smem, m0, n0);
    } else {
        static_assert(BN * (BM + 16) <= S::TOTAL, "the staged tile of pairs fits in the ring");
        store_masked_packed<MF, NF, BM, BN, 64 * MULT>(acc, m, n, mw, nw, m0, n0, l16, lq, meta, out, smem);
    }
}

// The skinny products of the adapters, one or two in a launch (no workgroups: none): D as above, bf16 [n][m], or fp32 sums of
// slabs of the contraction for skinny_sum_kernel.  One of the sides is the rank, in tiles of RANK rows, the other in tiles of
// LONG.  grid: workgroups per slab, a multiple of 8.  Operands are read as they are stored:
//   the factors   (GRADIENTS false): T = X L with L k-major, T2 = dY R^T, both operands k-contiguous; the rank is m in both;
//   the gradients (GRADIENTS true):  dL = X^T T2 (rank m) and dR = T^T dY (rank n), contractions over the tokens, all k-major.
struct SkinnyJob {
    DenseOperand A, B;
    int ksteps;
    bf16_t* out;
    float* sums;
    int tiles_m, tiles_n, grid, slabs, slab_steps;
};

template <int BM, int BN, int NS, bool AKM, bool BKM>
__device__ __forceinline__ void skinny_tn_tile(const SkinnyJob& j, int w, uint8_t* smem) {
    using S = TnSmem<BM, BN, NS>;
    constexpr int MULT = tn_mult(BM, BN), MF = BM / 32, NF = BN / (8 * MULT);
    const int slab = w / j.grid, m = j.A.rows, n = j.B.rows;
    int tm, tn;
    if (!tile_of_index(w % j.grid, j.tiles_m, j.tiles_n, tm, tn)) return;
    const int m0 = tm * BM, n0 = tn * BN, lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), mw = m0 + (wave & 1) * (BM / 2), nw = n0 + (wave >> 1) * (BN / (MULT / 2));
    const int k_begin = slab * j.slab_steps, k_end = min(k_begin + j.slab_steps, j.ksteps);
    f32x4 acc[MF][NF];
    if (!dense_tn_sums<BM, BN, NS, AKM, BKM>(j.A, j.B, j.ksteps, k_begin, k_end, m0, n0, smem, acc)) return;
    static_assert(BN * (BM * 2 + 16) <= S::TOTAL, "the staged output tile fits in the ring");
    if (j.slabs > 1) store_sums<MF, NF>(acc, m, n, mw, nw, l16, lq, j.sums + (size_t)slab * n * m);
    else store_rows<MF, NF, BM, BN, 64 * MULT>(acc, mw, nw, m, n, l16, lq, j.out, smem, m0, n0);
}

template <int LONG, int RANK, int NS, bool GRADIENTS>
__global__ void __launch_bounds__(tn_threads(LONG, RANK)) skinny_tn_kernel(SkinnyJob j0, SkinnyJob j1) {
    extern __shared__ __align__(16) uint8_t smem[];
    const int w = (int)blockIdx.x, first = j0.grid * j0.slabs;
    if (w < first) skinny_tn_tile<RANK, LONG, NS, true, GRADIENTS>(j0, w, smem);
    else if (GRADIENTS) skinny_tn_tile<LONG, RANK, NS, true, true>(j1, w - first, smem);
    else skinny_tn_tile<RANK, LONG, NS, false, false>(j1, w - first, smem);
}

// out = sum over the slabs (in slab order: runs are bit-identical), rounded to bf16; four elements per lane, one or two outputs
struct SkinnySum { const f32x4* P; int slabs; int64_t count4; u32x2* out; };
__global__ void __launch_bounds__(256) skinny_sum_kernel(SkinnySum a, SkinnySum b) {
    int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool first = idx < a.count4;
    const SkinnySum s = first ? a : b;
    if (!first) idx -= a.count4;
    if (idx >= s.count4) return;
    f32x4 v = s.P[idx];
#pragma unroll 4
    for (int sl = 1; sl < s.slabs; ++sl) {
        f32x4 w = s.P[(size_t)sl * s.count4 + idx];
        v[0] += w[0]; v[1] += w[1]; v[2] += w[2]; v[3] += w[3];
    }
    union { __bf16 h[4]; u32x2 u; } o;
    o.h[0] = (__bf16)v[0]; o.h[1] = (__bf16)v[1]; o.h[2] = (__bf16)v[2]; o.h[3] = (__bf16)v[3];
    s.out[idx] = o.u;
}

// The 256 x 256 tile of the weight gradient with split rings.  A plain two-stage ring (all that
// fits beside such a tile) makes every k-step a burst: nothing may be queued for a stage before
// both groups have read it, and everything queued must have landed one k-step later, so the load
// path runs dry at every step.  Here the two groups take the two column halves of the tile, which
// makes each half of the B panel private to one group, free again as soon as that group has read
// it, while the A panel, read by both, gets a ring of three:
//     A ring  3 x 32 KiB | B half of group 0  2 x 16 KiB | B half of group 1  2 x 16 KiB  = 160 KiB
// Every phase (half a k-step) each wavefront queues four 1 KiB loads
//     even phase 2k  :  B1(k+1), lower half of A(k+2)        odd phase 2k+1 :  upper half of A(k+2), B0(k+2)
// and at the end of every phase waits only for what it queued two or more phases ago (at most
// eight loads stay in flight), which is what the next phase reads.  A stage is always rewritten in
// the first phase after its last reader's barrier.
struct SplitSmem {
    static constexpr int BM = 256, BN = 256;
    static constexpr int A_STAGE = BM * 128, B_HALF = BN / 2 * 128;
    static constexpr int B_OFF = 3 * A_STAGE;                 // then [group][stage] halves of B
    static constexpr int TOTAL = 3 * A_STAGE + 4 * B_HALF;
};

// TAIL: the tiles left over after the last full round of 256.  Run as a round of their own they would
// keep some compute units busy for a whole tile's time while the rest of the chip idles.  Instead they (positions
// first_tile .. of the tile order) are taken in bundles of consecutive tiles, the bundles' k-steps are laid end to end and
// cut into equal shares, one for each lane: as many workgroups of one XCD as a bundle has tiles, which walk the share in
// step, one tile each, and so find each other's operand panels in the XCD's L2 (shares per workgroup instead, laid along
// the tiles: 2.2 to 2.4 us per k-step, from HBM; a whole round 1.36).  A share lies in one bundle or in a few; a workgroup
// leaves fp32 accumulators in register order for each tile it touches, and tail_finish_kernel adds a tile's parts and
// stores.  Lane w's part of bundle c is number w + c, less the bundle boundaries up to c that are share boundaries too
// (every aligned-th): no gaps, a bundle's parts one after the other.
// 400 tiles (5120 x 5120, 16384 tokens): 617 us as two rounds, 359 + 217 + 25 with the 144 leftover ones cut; 36864 x 9216,
// 64 leftover tiles in shares per workgroup before: 122 + 24, now 104 + 17.
// Short contractions have whole numbers of shares per bundle instead (row > ksteps: the last one is cut short): no share
// then has a second part to start.
struct TailPlan { int first_tile, tiles, bundle, lanes_per_xcd, lanes, share, row, aligned, parts; double steps; };
constexpr TailPlan NO_TAIL = {0, 0, 1, 1, 0, 1, 1, 1, 0, 0.0};

template <int EPI, bool TAIL, bool AKM, bool BKM>
__global__ void __launch_bounds__(TN_THREADS) dense_tn_split_kernel(DenseOperand At, DenseOperand Bt, int all_steps,
                                                                    const uint8_t* __restrict__ meta,
                                                                    bf16_t* __restrict__ out, int tiles_m,
                                                                    int tiles_n, TailPlan tail,
                                                                    f32x4* __restrict__ partial) {
    using S = SplitSmem;
    constexpr int MF = 8, NF = 4, WM = 128;                  // wavefront tile 128 x 64, 2 x 4 wavefronts
    extern __shared__ __align__(16) uint8_t smem[];

    const int m = At.rows, n = Bt.rows;
    int tm, tn, k_first = 0, ksteps = all_steps;
    // TAIL: this workgroup's lane and its tile in a bundle; [at, at_end) the k-steps of the lane's share that are left
    const int slot = (int)blockIdx.x / XCDS, member = slot % tail.bundle;
    const int lane_id = ((int)blockIdx.x % XCDS) * tail.lanes_per_xcd + slot / tail.bundle;
    if (TAIL && (slot / tail.bundle >= tail.lanes_per_xcd || lane_id >= tail.lanes)) return;
    int at = lane_id * tail.share, at_end = at + tail.share;
next_part:
    if (TAIL) {
        const int c = at / tail.row, tile = c * tail.bundle + member;
        k_first = at - c * tail.row;
        if (tile >= tail.tiles || k_first >= all_steps) return; // the end of the row, or a member the last bundle does not have
        ksteps = at_end - at < all_steps - k_first ? at_end - at : all_steps - k_first;
        tile_of_position(tail.first_tile + tile, tiles_m, tiles_n, tm, tn);
    } else if (!tile_of_block(tiles_m, tiles_n, tm, tn)) {
        return;
    }
    const int m0 = tm * S::BM, n0 = tn * S::BN;
    int t = threadIdx.x;
    if (TAIL) asm volatile("" : "+v"(t));                     // the lane's coordinates are derived again per part (no spills)
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int group = wave >> 2;                             // = column half of the tile
    const int wm = wave & 1, wn = wave >> 1;
    const int l16 = lane & 15, lq = lane >> 4;

    // Each load set (half of A, half of B) is 16 loads: two per wavefront, one at a time (look-ahead past the last step: unused).
    // Where both operands are k-contiguous their accesses are written out here: the same ones through DenseLoader are scheduled so
    // that the kernel takes 2 % longer (us, 16384 tokens, 8192 x 8192 1372 / 1403, 36864 x 9216 7043 / 7188; a fifth more fetched into
    // the L2s).
    constexpr bool CONTIGUOUS = !AKM && !BKM;
    DenseLoader<AKM, BKM, S::BM, WM> opa;
    DenseLoader<BKM, AKM, S::BN, NF * 16> opb;
    const uint8_t* a_src[4];                                 // [half * 2 + i]: 8 lanes per row, chunk rotated by (row / 2) % 8
    const uint8_t* b_src[4];                                 // [group * 2 + i]
    if (CONTIGUOUS) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int rl = ((q >> 1) * 16 + wave * 2 + (q & 1)) * 8 + (lane >> 3), sw16 = ((lane & 7) ^ ((rl >> 1) & 7)) * 16;
            a_src[q] = (const uint8_t*)At.p + (size_t)wrap_row(m0 + rl, m) * At.ld * 2 + sw16 + (size_t)k_first * 128;
            b_src[q] = (const uint8_t*)Bt.p + (size_t)wrap_row(n0 + rl, n) * Bt.ld * 2 + sw16 + (size_t)k_first * 128;
        }
    } else {
        opa.init(At, m0, wm * WM, wave, lane, k_first, ksteps, smem);
        opb.init(Bt, n0, wn * (NF * 16), wave, lane, k_first, ksteps, smem);
    }
    const int sw = (l16 >> 1) & 7, rd0 = l16 * 128 + ((lq ^ sw) * 16), rd1 = l16 * 128 + (((4 + lq) ^ sw) * 16);
    const int a_rd = (wm * MF) * 2048, b_rd = S::B_OFF + group * 2 * S::B_HALF + ((wn & 1) * NF) * 2048;
    auto issue_a = [&](int half, int ks, int i) {
        const int kc = ks < ksteps ? ks : ksteps - 1;
        if (CONTIGUOUS) dma16(a_src[half * 2 + i] + (size_t)kc * 128, smem + (ks % 3) * S::A_STAGE + (half * 16 + wave * 2 + i) * 1024);
        else opa.load(ks, half * 2 + i, smem, (ks % 3) * S::A_STAGE, wave);
    };
    // (B half g of step ks lies at (g * 2 + ks % 2) * B_HALF; the loader numbers its pieces from the tile's first column)
    auto issue_b = [&](int g, int ks, int i) {
        const int kc = ks < ksteps ? ks : ksteps - 1;
        if (CONTIGUOUS) dma16(b_src[g * 2 + i] + (size_t)kc * 128, smem + S::B_OFF + (g * 2 + (ks & 1)) * S::B_HALF + (wave * 2 + i) * 1024);
        else opb.load(ks, g * 2 + i, smem, S::B_OFF + (g + (ks & 1)) * S::B_HALF, wave);
    };
    auto even_load = [&](int k, int idx) { if (idx < 2) issue_b(1, k + 1, idx); else issue_a(0, k + 2, idx - 2); };
    auto odd_load = [&](int k, int idx) { if (idx < 2) issue_a(1, k + 2, idx); else issue_b(0, k + 2, idx - 2); };

    f32x4 acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

    constexpr int KEEP = 8;                                  // loads of the last two phases
#define SPLIT_READ(ks)                                                                                 \
        const auto sa = opa.stage(smem, ((ks) % 3) * S::A_STAGE);                                      \
        const auto sb = opb.stage(smem, S::B_OFF + (group + ((ks) & 1)) * S::B_HALF);                  \
        const uint8_t* const pa = smem + ((ks) % 3) * S::A_STAGE + a_rd;                               \
        const uint8_t* const pb = smem + b_rd + ((ks) & 1) * S::B_HALF;                                \
        BFrag af[MF], bf[NF];                                                                          \
        _Pragma("unroll") for (int i = 0; i < MF; ++i) {                                               \
            if (!CONTIGUOUS) { af[i] = opa.frag(sa, i); continue; }                                    \
            af[i].u[0] = *(const u32x4*)(pa + i * 2048 + rd0);                                         \
            af[i].u[1] = *(const u32x4*)(pa + i * 2048 + rd1);                                         \
        }                                                                                              \
        _Pragma("unroll") for (int j = 0; j < NF; ++j) {                                               \
            if (!CONTIGUOUS) { bf[j] = opb.frag(sb, j); continue; }                                    \
            bf[j].u[0] = *(const u32x4*)(pb + j * 2048 + rd0);                                         \
            bf[j].u[1] = *(const u32x4*)(pb + j * 2048 + rd1);                                         \
        }
// the compute phase: 64 MFMAs with the phase's four loads spread between them (queued in one burst
// at the start of the phase they cost 2 % more).  The B fragments are taken back and forth, so that only
// one operand changes from one MFMA to the next: the kernel runs at the clock the chip's power limit
// allows, and that order draws measurably less (1.7 % faster than always restarting at fragment 0).
#define SPLIT_MFMA(LOAD, k)                                                                            \
        _Pragma("unroll") for (int h = 0; h < 2; ++h)                                                  \
        _Pragma("unroll") for (int i = 0; i < MF; ++i) {                                               \
            _Pragma("unroll") for (int jj = 0; jj < NF; ++jj) {                                        \
                const int j = (i & 1) ? NF - 1 - jj : jj;                                              \
                AFrag a, b;                                                                            \
                a.u = af[i].u[h]; b.u = bf[j].u[h];                                                    \
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, acc[i][j], 0, 0, 0);     \
            }                                                                                          \
            if (h == 0 && (i & 1) == 1) LOAD(k, i >> 1);                                               \
            __builtin_amdgcn_sched_barrier(0);                                                         \
        }
#define EVEN_LOADS(k) { even_load(k, 0); even_load(k, 1); even_load(k, 2); even_load(k, 3); }
#define ODD_LOADS(k)  { odd_load(k, 0); odd_load(k, 1); odd_load(k, 2); odd_load(k, 3); }

    // steps 0 and 1 as far as the schedule would have queued them before phase 0
    issue_a(0, 0, 0); issue_a(0, 0, 1); issue_a(1, 0, 0); issue_a(1, 0, 1); issue_b(0, 0, 0); issue_b(0, 0, 1);
    issue_b(1, 0, 0); issue_b(1, 0, 1); issue_a(0, 1, 0); issue_a(0, 1, 1);
    issue_a(1, 1, 0); issue_a(1, 1, 1); issue_b(0, 1, 0); issue_b(0, 1, 1);
    WAIT_HERE(waitcnt_imm(KEEP, 15));                         // A(0) and B0(0) have landed
    wg_barrier();
    if (group == 0) {
        for (int ks = 0; ks < ksteps; ++ks) {
            SPLIT_READ(ks)                                    // phase 2 ks
            EVEN_LOADS(ks)
            WAIT_HERE(waitcnt_imm(KEEP, 0));
            wg_barrier();
            SPLIT_MFMA(odd_load, ks)                          // phase 2 ks + 1
            WAIT_HERE(waitcnt_imm(KEEP, 15));
            wg_barrier();
        }
        wg_barrier();                                         // group 1's last compute phase
    } else {
        EVEN_LOADS(0)                                         // phase 0: nothing to compute yet
        WAIT_HERE(waitcnt_imm(KEEP, 15));
        wg_barrier();
        for (int ks = 0; ks < ksteps; ++ks) {
            SPLIT_READ(ks)                                    // phase 2 ks + 1
            ODD_LOADS(ks)
            WAIT_HERE(waitcnt_imm(KEEP, 0));
            wg_barrier();
            SPLIT_MFMA(even_load, ks + 1)                     // phase 2 ks + 2
            WAIT_HERE(waitcnt_imm(KEEP, 15));
            wg_barrier();
        }
    }
#undef SPLIT_READ
#undef SPLIT_MFMA
#undef EVEN_LOADS
#undef ODD_LOADS
    WAIT_HERE(waitcnt_imm(0, 15));                            // drain the clamped look-ahead loads
    if (TAIL) {
        const int c = at / tail.row;
        f32x4* dst = partial + (int64_t)((lane_id + c - c / tail.aligned) * tail.bundle + member) * (MF * NF * TN_THREADS) + t;
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j) dst[(i * NF + j) * TN_THREADS] = acc[i][j];
        at += ksteps;
        if (at >= at_end) return;
        wg_barrier();                                         // every wavefront's reads and look-ahead loads are over
        goto next_part;
    }
    static_assert(S::BN * (S::BM * 2 + 16) <= S::TOTAL, "the staged output tile fits in the rings");
    if (EPI == EPI_PLAIN)
        store_rows<MF, NF, S::BM, S::BN, TN_THREADS>(acc, m0 + wm * WM, n0 + wn * NF * 16, m, n, l16, lq, out, smem, m0, n0);
    else store_masked_packed<MF, NF, S::BM, S::BN, TN_THREADS>(acc, m, n, m0 + wm * WM, n0 + wn * NF * 16, m0, n0, l16, lq, meta, out,
                                                   smem);
}

// Second pass of the tail: workgroup (leftover tile i, fragment column j) adds the tile's parts, in order, for one of the
// four fragment columns of every wavefront of the kernel above, and stores the pairs that W^R keeps: 64 rows (d_out) of
// the tile through LDS, as store_masked_packed does.  (Two kernels before, a sum and a store by one workgroup per tile:
// 24 us for 64 tiles in four parts each, now 17.)
__global__ void __launch_bounds__(TN_THREADS) tail_finish_kernel(const f32x4* __restrict__ partial, int m, int n, int ksteps,
                                                                 const uint8_t* __restrict__ meta,
                                                                 bf16_t* __restrict__ out, int tiles_m, int tiles_n,
                                                                 TailPlan tail) {
    using S = SplitSmem;
    constexpr int MF = 8, NF = 4, WM = 128, CP = S::BM + 16, ROWS = 64;
    __shared__ __align__(16) uint8_t smem[ROWS * CP];
    const int tile = (int)blockIdx.x / NF, j = (int)blockIdx.x % NF;
    int tm, tn;
    tile_of_position(tail.first_tile + tile, tiles_m, tiles_n, tm, tn);
    const int m0 = tm * S::BM, n0 = tn * S::BN;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave & 1, wn = wave >> 1, l16 = lane & 15, lq = lane >> 4;
    const int c = tile / tail.bundle, first = c * tail.row / tail.share, last = (c * tail.row + ksteps - 1) / tail.share;
    constexpr int PART = MF * NF * TN_THREADS;
    const f32x4* src = partial + (int64_t)((first + c - c / tail.aligned) * tail.bundle + tile % tail.bundle) * PART + j * TN_THREADS + t;
    f32x4 acc[MF];
#pragma unroll
    for (int i = 0; i < MF; ++i) acc[i] = src[i * NF * TN_THREADS];
    for (int w = first + 1; w <= last; ++w) {
        src += (int64_t)tail.bundle * PART;
        f32x4 x[MF];
#pragma unroll
        for (int i = 0; i < MF; ++i) x[i] = src[i * NF * TN_THREADS];
#pragma unroll
        for (int i = 0; i < MF; ++i) { acc[i][0] += x[i][0]; acc[i][1] += x[i][1]; acc[i][2] += x[i][2]; acc[i][3] += x[i][3]; }
    }
    const int o = n0 + wn * 64 + j * 16 + l16, c0 = m0 + wm * WM;
    uint32_t mw[WM / 32];
#pragma unroll
    for (int q = 0; q < WM / 32; ++q)
        mw[q] = o < n && c0 + 32 * q < m ? *(const uint32_t*)(meta + (size_t)o * (m / 8) + c0 / 8 + 4 * q) : 0u;
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int gl = i * 4 + lq;
        const uint32_t nib = (mw[i >> 1] >> (4 * (gl & 7))) & 0xFu, a = nib & 3u, c = nib >> 2;
        union { __bf16 h[2]; uint32_t u; } pr;
        pr.h[0] = (__bf16)(a == 0 ? acc[i][0] : (a == 1 ? acc[i][1] : acc[i][2]));
        pr.h[1] = (__bf16)(c == 1 ? acc[i][1] : (c == 2 ? acc[i][2] : acc[i][3]));
        *(uint32_t*)(smem + (wn * 16 + l16) * CP + (wm * (WM / 4) + gl) * 4) = pr.u;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < ROWS * (S::BM / 16) / TN_THREADS; ++u) {
        const int idx = t + u * TN_THREADS, row = idx / (S::BM / 16), pc = idx % (S::BM / 16);
        const int orow = n0 + (row >> 4) * 64 + j * 16 + (row & 15), col = m0 + pc * 16;
        if (orow < n && col < m) *(u32x4*)(out + (size_t)orow * (m / 2) + (col >> 1)) = *(const u32x4*)(smem + row * CP + pc * 16);
    }
}

template <int BM, int BN, int EPI, int NS, bool AKM, bool BKM>
hipError_t launch_dense_tn(const DenseOperand& A, const DenseOperand& B, int64_t ksteps, const uint8_t* meta, bf16_t* out, hipStream_t s) {
    using S = TnSmem<BM, BN, NS>;
    static_assert(S::TOTAL <= 160 * 1024, "LDS budget");
    const int tiles_m = (A.rows + BM - 1) / BM, tiles_n = (B.rows + BN - 1) / BN;
    hipError_t e = allow_dynamic_lds<dense_tn_kernel<BM, BN, EPI, NS, AKM, BKM>>(S::TOTAL);
    if (e != hipSuccess) return e;
    dense_tn_kernel<BM, BN, EPI, NS, AKM, BKM><<<dim3((unsigned)super_grid(tiles_m, tiles_n)), dim3(tn_threads(BM, BN)), S::TOTAL, s>>>(
        A, B, (int)ksteps, meta, out, tiles_m, tiles_n);
    return hipGetLastError();
}

// How the tiles left over after the last full round are cut (tiles == 0: not worth cutting).  Only wide grids (the tile
// order has positions there).  An XCD's 32 compute units hold 32 / bundle lanes; the bundle is the largest (its tiles share
// panels) whose shares are within 1/16 of the shortest.  In units of a k-step (1.36 us) a share costs its k-steps, about 6
// for every part, the parts' way through memory (256 KiB each, written and read at 6 TB/s: 0.065 per part) and a launch
// (5); a round of whole tiles costs ksteps + 6.  Where a bundle can be cut into whole shares, its lanes have a part each and
// its tiles fewer of them to add: then the cheaper of the two.  (19 k-steps, us: 4096 x 5120 uneven shares 77.8, whole
// ones 72.1; 3328 x 6656 83.1 / 76.8; 128 k-steps: 3328 x 6656 282 / 266.  More than half a round left: 5120 x 5120, 128
// k-steps, where the rule begins to cut: 316 not cut, 321 cut; 256 k-steps: 627 / 597; 11 x 37 tiles, 128 k-steps: 311 / 333, 192:
// 471 / 471, 256: 632 / 611.)
inline TailPlan tail_plan(int64_t tiles_m, int64_t tiles_n, int64_t ksteps) {
    const TailPlan p = NO_TAIL;
    const int64_t tiles = tiles_m * tiles_n;
    if (!wide_grid((int)tiles_m, (int)tiles_n) || tiles < RESIDENT || tiles > (1 << 30) || ksteps > (1 << 20)) return p;
    const int64_t rem = tiles % RESIDENT;
    if (rem == 0) return p;
    constexpr int64_t PER_XCD = RESIDENT / XCDS;
    int64_t shortest = INT64_MAX, bundle = 0, share = 0, lanes_per_xcd = 0;
    for (int pass = 0; pass < 2; ++pass)
        for (int64_t e = rem < PER_XCD ? rem : PER_XCD; e >= 1; --e) {
            const int64_t per = PER_XCD / e, row = (rem + e - 1) / e * ksteps;
            int64_t sh = (row + XCDS * per - 1) / (XCDS * per);
            if (sh < 8) sh = 8;
            if (pass == 0) { if (sh < shortest) shortest = sh; }
            else if (!bundle && sh * 16 <= shortest * 17) { bundle = e; share = sh; lanes_per_xcd = per; }
        }
    const int64_t bundles = (rem + bundle - 1) / bundle;
    int64_t lanes = (bundles * ksteps + share - 1) / share;
    int64_t aligned = share / std::gcd(share, ksteps), parts = lanes + bundles - 1 - (bundles - 1) / aligned, row = ksteps;
    const double shares = (double)share + 6.0 * (1.0 + (double)((share + ksteps - 1) / ksteps)) + 0.065 * (double)(parts * bundle) + 5.0;
    // (in the strips beside whole chunks of a narrow grid a bundle's tiles share few panels)
    const bool narrow = (tiles_m < tiles_n ? tiles_m : tiles_n) < 13;
    double cost = shares + (narrow ? 0.2 * (double)share : 0.0);
    if (rem <= RESIDENT / 2 && ksteps >= 16) {                // measured: the cut never lost here; a share of the round + 1/4
        const int64_t slabs = RESIDENT / rem < ksteps / 8 ? RESIDENT / rem : ksteps / 8;
        cost = ((double)ksteps + 6.0) * (1.0 / (double)slabs + 0.25);
    } else if (cost > 0.95 * ((double)ksteps + 6.0)) {
        return p;
    }
    // whole shares: as many per bundle as an XCD's lanes and eight k-steps each allow
    double least = shares;
    for (int64_t e = rem < PER_XCD ? rem : PER_XCD; e >= 1; --e) {
        const int64_t count = (rem + e - 1) / e;
        int64_t cut = XCDS * (PER_XCD / e) / count;
        if (cut > ksteps / 8) cut = ksteps / 8;
        if (cut < 2) continue;
        const int64_t sh = (ksteps + cut - 1) / cut;
        cut = (ksteps + sh - 1) / sh;
        const double whole = (double)sh + 6.0 + 0.065 * (double)(cut * rem) + 5.0;
        if (whole >= least) continue;
        least = whole;
        bundle = e;
        lanes_per_xcd = PER_XCD / e;
        share = sh;
        row = cut * sh;
        lanes = parts = cut * count;
        aligned = 1;
    }
    return {(int)(tiles - rem), (int)rem, (int)bundle, (int)lanes_per_xcd, (int)lanes, (int)share, (int)row, (int)aligned, (int)parts, cost};
}

// tail: scratch for the parts of the leftover tiles (masked packed results only), or null
template <int EPI, bool AKM, bool BKM>
hipError_t launch_dense_tn_split(const DenseOperand& A, const DenseOperand& B, int64_t ksteps, const uint8_t* meta, bf16_t* out,
                                 hipStream_t s, float* tail) {
    using S = SplitSmem;
    static_assert(S::TOTAL <= 160 * 1024, "LDS budget");
    const int tiles_m = (A.rows + S::BM - 1) / S::BM, tiles_n = (B.rows + S::BN - 1) / S::BN;
    hipError_t e = allow_dynamic_lds<dense_tn_split_kernel<EPI, false, AKM, BKM>>(S::TOTAL);
    if (e != hipSuccess) return e;
    const TailPlan p = tail ? tail_plan(tiles_m, tiles_n, ksteps) : NO_TAIL;
    // with a tail the first launch is whole rounds only: workgroups 0 .. first_tile - 1 are exactly the
    // positions 0 .. first_tile - 1 of the order
    const int grid = p.tiles ? p.first_tile : super_grid(tiles_m, tiles_n);
    dense_tn_split_kernel<EPI, false, AKM, BKM><<<dim3((unsigned)grid), dim3(TN_THREADS), S::TOTAL, s>>>(
        A, B, (int)ksteps, meta, out, tiles_m, tiles_n, NO_TAIL, nullptr);
    if ((e = hipGetLastError()) != hipSuccess || !p.tiles) return e;
    if constexpr (EPI == EPI_MASKED_PACKED) {
        if ((e = allow_dynamic_lds<dense_tn_split_kernel<EPI, true, AKM, BKM>>(S::TOTAL)) != hipSuccess) return e;
        dense_tn_split_kernel<EPI, true, AKM, BKM><<<dim3(RESIDENT), dim3(TN_THREADS), S::TOTAL, s>>>(
            A, B, (int)ksteps, meta, out, tiles_m, tiles_n, p, (f32x4*)tail);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        tail_finish_kernel<<<dim3((unsigned)(p.tiles * 4)), dim3(TN_THREADS), 0, s>>>(
            (const f32x4*)tail, A.rows, B.rows, (int)ksteps, meta, out, tiles_m, tiles_n, p);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace

namespace {
inline size_t round256(size_t v) { return (v + 255) & ~(size_t)255; }
}  // namespace

// Token-contiguous copy of a [b][d] activation: d rows of token_pitch(b rounded up to 64) elements.
size_t token_copy_bytes(int64_t b, int64_t d) { return (size_t)d * (size_t)token_pitch((b + 63) / 64 * 64) * 2; }

// One or two copies (in1 == nullptr: one) of matrices with b rows in one launch.
hipError_t launch_token_copies(const bf16_t* in0, int64_t cols0, bf16_t* out0, const bf16_t* in1, int64_t cols1,
                               bf16_t* out1, int64_t b, hipStream_t s) {
    const int64_t bp = (b + 63) / 64 * 64, ld = token_pitch(bp);
    return launch_transposes(transpose_job(in0, b, cols0, bp, ld, out0), in1 ? transpose_job(in1, b, cols1, bp, ld, out1) : TransposeJob{}, s);
}

// Layers that the forms with token-contiguous copies in their interface take.
bool wgrad_tn_fits(int64_t d_in) { return d_in % 32 == 0; }

// Tiles (m x n) of the dense products, the weight gradient's and those of masked dense weights; of two that take as long the
// first.  [0] is the kernel with split rings, which with scratch memory cuts the tiles left over after its last full
// round along the tokens (launch_dense_tn_split).
struct DenseTile { int bm, bn; };
constexpr DenseTile DENSE_TILES[] = {{256, 256}, {256, 192}, {192, 192}, {256, 128}, {192, 128}, {128, 128}, {64, 128}, {64, 64}};

// The kernels run at the rate their compute units pull operands from L2, 53 bytes per ns (up to a fifth more with few of them
// at work, a little less on 192 x 192, a seventh less on 256 x 192, whose ring has two stages): a launch takes rounds
// of 256 resident tiles, each its k-steps, 3 us, and up to 6 for the way of its results.  The tiles up to 256 x 128 are up to 15 % faster
// than that by now; the order of the estimates, which is all that counts, has held.
// `start` and `slower`: what a round of the 256 x 256 kernel takes beside its k-steps, and the factor on these.
static double dense_tile_us(int c, int64_t m, int64_t n, int64_t ksteps, double start = 9.0, double slower = 1.0) {
    const int bm = DENSE_TILES[c].bm, bn = DENSE_TILES[c].bn;
    const int64_t tiles = ((m + bm - 1) / bm) * ((n + bn - 1) / bn), rounds = (tiles + RESIDENT - 1) / RESIDENT;
    const double step = 128.0 * (double)(bm + bn) / 53e3 * (bn != 192 ? 1.0 : bm == 256 ? 1.15 : 1.04), busy = (double)tiles / (double)(rounds * RESIDENT);
    if (c != 0) { start = 3.0 + 6.0 * (double)(bm * bn) / 65536.0; slower = 1.0; }
    return (double)rounds * (start + (double)ksteps * step * slower * (1.0 - 0.22 * (1.0 - busy)));
}

// Tile of a product of whole tiles.  Where 256 x 256 and 256 x 192 have as many rounds, the former is the faster one on operands from HBM and the latter
// on operands from the last-level cache, by 5 to 18 % each (us, 256 x 192 / 256 x 256: gradient of 12606 tokens, 5120 x 2048 240 / 285 cached, 253 /
// 231 from HBM; masked dense 4674 tokens, 5120 x 8192 292 / 323, 332 / 312).
//  - k-contiguous operands, masked dense weights: as from HBM.  Also right behind the kernel that makes the weights other traffic has passed through the
//    cache (16 steps of 1000 to 16000 tokens 0 to 15 % faster than with 256 x 192: 3613 tokens, 5632 x 5888 524 / 457; 1232, 8000 x 5184 295 / 276).
//  - operands as stored, gradients: dY has just been read for the input gradient, and X is still there if it is not more than half of the cache.
//    Then a twelfth more for the k-steps of 256 x 256 (`cached`; us, forward and both gradients of one layer: 11959 tokens, 3072 x 3328 502 / 543; 3867, 4608 x 2048 169 /
//    182; of 400 steps of 512 to 16384 tokens the 22 that it concerns are up to 8 % faster, one 1 % slower; with X from HBM the gradient alone loses: 4068, 2560 x 3840 87 / 80).  Else a round takes 2 us
//    longer than from k-contiguous ones from the fourth k-step on (over 1332 gradients from memory the tile chosen so is 0.3 % longer than the
//    best in the mean, 21 % at most; us, forward and both gradients: 15599, 2048 x 5120 696 / 669).
enum DenseFrom { K_CONTIGUOUS, AS_STORED, AS_STORED_CACHED };
static int dense_tile_choice(int64_t m, int64_t n, int64_t ksteps, DenseFrom from) {
    int best = 0;
    if (ksteps <= 3) from = K_CONTIGUOUS;                     // results take most of the time
    double least = dense_tile_us(0, m, n, ksteps, from == AS_STORED ? 11.0 : 9.0, from == AS_STORED_CACHED ? 1.08 : 1.0);
    for (int c = 1; c < (int)(sizeof(DENSE_TILES) / sizeof(DENSE_TILES[0])); ++c) {
        const double us = dense_tile_us(c, m, n, ksteps);
        if (us < least) { least = us; best = c; }
    }
    return best;
}
static DenseFrom gradient_operands(int64_t b, int64_t d_in, int64_t d_out) {
    const bool cached = (size_t)(2 * b * d_in) <= LAST_LEVEL_CACHE_BYTES / 2 && (size_t)(2 * b * (d_in + d_out)) <= LAST_LEVEL_CACHE_BYTES;
    return cached ? AS_STORED_CACHED : AS_STORED;
}

// Cutting what is left over after the whole rounds is estimated to be no longer than whole tiles of another shape.  Scratch of the calls follows
// from it, so that this estimate stays as it is, whatever becomes of the kernels.
static bool cutting_pays(int64_t m, int64_t n, int64_t ksteps, const TailPlan& p) {
    const int64_t rounds = ((m + 255) / 256) * ((n + 255) / 256) / RESIDENT;
    const double cut = (double)rounds * (9.0 + (double)ksteps * (128.0 * 512.0 / 53e3)) + 1.3 * p.steps + 16.0;
    for (int c = 1; c < (int)(sizeof(DENSE_TILES) / sizeof(DENSE_TILES[0])); ++c)
        if (dense_tile_us(c, m, n, ksteps) < cut) return false;
    return true;
}

template <int EPI, bool AKM, bool BKM>
static hipError_t launch_dense_tile(int tile, const DenseOperand& A, const DenseOperand& B, int64_t ksteps, const uint8_t* meta,
                                    bf16_t* out, hipStream_t s, float* tail = nullptr) {
    switch (tile) {
        case 0: return launch_dense_tn_split<EPI, AKM, BKM>(A, B, ksteps, meta, out, s, tail);
        case 1: return launch_dense_tn<256, 192, EPI, 2, AKM, BKM>(A, B, ksteps, meta, out, s);
        case 2: return launch_dense_tn<192, 192, EPI, 3, AKM, BKM>(A, B, ksteps, meta, out, s);
        case 3: return launch_dense_tn<256, 128, EPI, 3, AKM, BKM>(A, B, ksteps, meta, out, s);
        case 4: return launch_dense_tn<192, 128, EPI, 4, AKM, BKM>(A, B, ksteps, meta, out, s);
        case 5: return launch_dense_tn<128, 128, EPI, 4, AKM, BKM>(A, B, ksteps, meta, out, s);
        case 6: return launch_dense_tn<64, 128, EPI, 6, AKM, BKM>(A, B, ksteps, meta, out, s);
        default: return launch_dense_tn<64, 64, EPI, 8, AKM, BKM>(A, B, ksteps, meta, out, s);
    }
}

// Scratch bytes of launch_wgrad_masked_t's tail pass, 0 where it does not cut: where the estimate above takes whole tiles, of
// this or another shape (1153 tokens, 5120 x 4096: 78 us cut, 58 on 256 x 192; 1640, 19840 x 1000: 89 cut, 80 whole), and where a rule of fewest rounds x
// rows among four of the tiles would not cut, which is as much scratch as this call ever asks for: programs keep buffers.
size_t wgrad_tail_bytes(int64_t b, int64_t d_in, int64_t d_out) {
    const int64_t ksteps = (b + 63) / 64;
    const TailPlan p = tail_plan((d_in + 255) / 256, (d_out + 255) / 256, ksteps);
    if (!p.tiles) return 0;
    auto rows = [&](int64_t bm, int64_t bn) { return (((d_in + bm - 1) / bm) * ((d_out + bn - 1) / bn) + RESIDENT - 1) / RESIDENT * (bm + bn) * 100; };
    const int64_t whole = ((d_in + 255) / 256) * ((d_out + 255) / 256) / RESIDENT * 512 * 100;
    const int64_t cut = whole + (int64_t)(512.0 * 100.0 * p.steps / (double)(ksteps + 6));
    if (cut > rows(256, 128) || cut > rows(128, 128) || cut > rows(128, 64)) return 0;
    if (!cutting_pays(d_in, d_out, ksteps, p)) return 0;
    return (size_t)p.parts * (size_t)p.bundle * (256 * 256 * 4);
}

// dW (masked, packed) from token-contiguous copies Xt [d_in][ld], dYt [d_out][ld]; tail_or_null: scratch of
// wgrad_tail_bytes(b, d_in, d_out) bytes, or nullptr (then a last partial round of tiles runs as it is)
hipError_t launch_wgrad_masked_t(const bf16_t* dYt, const bf16_t* Xt, int64_t b, const uint8_t* meta, int64_t d_out,
                                 int64_t d_in, bf16_t* gvals, float* tail_or_null, hipStream_t s) {
    const int64_t bp = (b + 63) / 64 * 64, ld = token_pitch(bp);
    const int tile = tail_or_null ? 0 : dense_tile_choice(d_in, d_out, bp / 64, K_CONTIGUOUS);
    return launch_dense_tile<EPI_MASKED_PACKED, false, false>(tile, {Xt, (int)d_in, (int)ld, (int)bp}, {dYt, (int)d_out, (int)ld, (int)bp}, bp / 64, meta, gvals, s, tail_or_null);
}

// The same product from the operands as stored, token after token.  The tiles that pull their operands from L2 as fast as they can
// lose nothing by it, and the copies are saved (us, copies and product / as stored: 2048 tokens, 3072 x 768 33.0 / 20.2; 700, 4160 x
// 2112 26.6 / 18.7; 4096, 4096 x 4096 134 / 117; 16384, 2560 x 10240 793 / 682).  The 256 x 256 kernel on many rounds
// keeps its matrix pipes busy, and there the transposing LDS reads, half as many bytes per cycle as plain ones, make it 4 % slower
// with X as stored, 3 % with dY, 9 % with both, while a copy is a stream of its operand at 5.9 TB/s.  So an operand is copied, where
// there is room, when the other one is wide: X from about 9000 rows, dY from about 11000 columns on (16384 tokens, us, the call with
// neither copied, X, dY, both: 8192 x 8192 1486, 1513, 1537, 1605; 36864 x 9216 7700, 7287, 7691, 7522; 9216 x 36864 7802, 7713, 7539,
// 7610; 16384 x 16384 6022, 5926, 6014, 6057: the rule loses 2 % there, elsewhere nothing).
enum { COPY_X = 1, COPY_DY = 2 };
static int wgrad_copies(int64_t d_in, int64_t d_out, int tile) {
    if (d_in % 32 != 0 || tile != 0) return 0;
    const double product = 2.0 * (double)d_out * (double)d_in / 1.5e9, x = 4.0 * (double)d_in / 5.9e6, dy = 4.0 * (double)d_out / 5.9e6;   // us per token
    const double cost[4] = {0.088 * product, x + 0.032 * product, dy + 0.042 * product, x + dy};
    int best = 0;
    for (int c = 1; c < 4; ++c)
        if (cost[c] < cost[best]) best = c;
    return best;
}

// Layers that the tiles cannot read as stored.  (Not from copies: us, 500 tokens, 64 x (2^24 + 64), copies and tiles 10580, the kernel
// with 64-bit addresses 4910.)
static bool too_wide(int64_t d_in, int64_t d_out) { return d_in >= KMAJOR_EXTENT_MAX || d_out >= KMAJOR_EXTENT_MAX; }

// dW (masked, packed) from dY [b][d_out] and X [b][d_in].  Xt, dYt: room for their copies (launch_token_copies), or null; tail as above.
hipError_t launch_wgrad_masked(const bf16_t* dY, const bf16_t* X, int64_t b, const uint8_t* meta, int64_t d_out, int64_t d_in, bf16_t* gvals,
                               bf16_t* Xt, bf16_t* dYt, float* tail_or_null, hipStream_t s) {
    if (too_wide(d_in, d_out)) return launch_wgrad_wide(dY, X, b, meta, d_out, d_in, gvals, s);
    if (wgrad_in_groups(b, d_in, d_out)) return launch_wgrad_groups(dY, X, b, meta, d_out, d_in, gvals, s);
    const int64_t bp = (b + 63) / 64 * 64, ld = token_pitch(bp);
    const int tile = tail_or_null ? 0 : dense_tile_choice(d_in, d_out, bp / 64, gradient_operands(b, d_in, d_out));
    const int copies = Xt && dYt ? wgrad_copies(d_in, d_out, tile) : 0;
    const DenseOperand x = copies & COPY_X ? DenseOperand{Xt, (int)d_in, (int)ld, (int)bp} : DenseOperand{X, (int)d_in, (int)d_in, (int)b};
    const DenseOperand dy = copies & COPY_DY ? DenseOperand{dYt, (int)d_out, (int)ld, (int)bp} : DenseOperand{dY, (int)d_out, (int)d_out, (int)b};
    if (copies) {
        const hipError_t e = launch_transposes(copies & COPY_X ? transpose_job(X, b, d_in, bp, ld, Xt) : TransposeJob{},
                                               copies & COPY_DY ? transpose_job(dY, b, d_out, bp, ld, dYt) : TransposeJob{}, s);
        if (e != hipSuccess) return e;
    }
    constexpr int EPI = EPI_MASKED_PACKED;
    switch (copies) {                                         // (tile 0 only where there are any)
        case COPY_X: return launch_dense_tn_split<EPI, false, true>(x, dy, bp / 64, meta, gvals, s, tail_or_null);
        case COPY_DY: return launch_dense_tn_split<EPI, true, false>(x, dy, bp / 64, meta, gvals, s, tail_or_null);
        case COPY_X | COPY_DY: return launch_dense_tn_split<EPI, false, false>(x, dy, bp / 64, meta, gvals, s, tail_or_null);
        default: return launch_dense_tile<EPI, true, true>(tile, x, dy, bp / 64, meta, gvals, s, tail_or_null);
    }
}

// C[n, m] = B[n, K] * A[m, K]^T for the skinny products of the adapters (T = X L, dY R^T, and over the tokens dL and
// dR): one side is the rank, the other a layer extent or the tokens.  Both operands bf16 of row pitch ld, K % 64 == 0.
// The product is bound by streaming the long operand once, so what counts is that a single round of workgroups (one per
// compute unit, the ring fills the LDS) covers it: with too few tiles the contraction is cut into slabs that leave fp32
// sums for a second kernel, at most as many as fit beside each other, since a thin second round costs as much as the
// first (5120 x 64 over 16384 tokens in tiles of 64 x 64: 1 slab 95 us, 3 slabs 44.7, 4 slabs 61.7).
// The rule takes the least of an estimate: the long operand at 4.6 TB/s, or what a compute unit pulls for its tiles
// at 41 B/ns; slabs cost 3 us for the second launch, 0.4 us each and their traffic.  With few tokens there is room for more
// slabs than pay: the best number is where a further one adds as much to the second kernel as it takes from the first
// (dY R^T of 127 x 17664, rank 32: 69 slabs 11.4 + 20.8 us, the call with its product 121.6; 17 slabs 103.2).
// 5120 x 64 / 9216 x 128 / 2560 x 64 over 16384 / 16384 / 4096 tokens: estimates 41 / 75 / 12 us, measured 44.7 / 76 / 11.8;
// before, in tiles of 128 x 64 without slabs, 108 / 133 / 31.
constexpr int SKINNY_LONG[5] = {64, 64, 128, 128, 64}, SKINNY_RANK[5] = {128, 64, 64, 128, 256};   // tiles of the two sides
struct SkinnyPlan { int tile, slabs, slab_steps; };
static SkinnyPlan skinny_plan(int64_t longer, int64_t rank, int64_t K, size_t partial_bytes) {
    const int64_t ksteps = K / 64;
    SkinnyPlan best = {0, 1, (int)ksteps};
    double best_us = 1e300;
    for (int c = 0; c < 5; ++c) {
        const int64_t tiles = ((longer + SKINNY_LONG[c] - 1) / SKINNY_LONG[c]) * ((rank + SKINNY_RANK[c] - 1) / SKINNY_RANK[c]);
        const double pull = 128.0 * (double)(SKINNY_LONG[c] + SKINNY_RANK[c]) / 41e3;   // per k-step
        const double per_slab = 0.4 + 8.0 * (double)longer * (double)rank / 10e6;
        int64_t slabs = RESIDENT / tiles;
        if (slabs > ksteps / 4) slabs = ksteps / 4;          // at least four k-steps per slab
        const int64_t room = (int64_t)(partial_bytes / ((size_t)longer * (size_t)rank * 4));
        if (slabs > room) slabs = room;
        const double least = sqrt((double)ksteps * pull / per_slab);             // more slabs cost more than they save
        if ((double)slabs > least) slabs = (int64_t)(least + 0.5);
        for (const int64_t want : {slabs, (int64_t)1}) {
            if (want < 1) continue;
            const int64_t steps = (ksteps + want - 1) / want, cut = (ksteps + steps - 1) / steps;
            const double rounds = (double)((tiles * cut + RESIDENT - 1) / RESIDENT);
            const double pulled = rounds * (double)steps * pull, stream = 2.0 * (double)longer * (double)K / 4.6e6;
            const double us = (pulled > stream ? pulled : stream) + (cut > 1 ? 3.0 + per_slab * (double)cut : 0.0);
            if (us < best_us) { best_us = us; best = {c, (int)cut, (int)steps}; }
        }
    }
    return best;
}

// Two products of the same rank in one launch: tile and k-steps per slab (of either) by the same estimate.  Their workgroups
// share the one round, so each gets fewer slabs than it would by itself.
struct SkinnyPair { int tile; int64_t slab_steps; };
static SkinnyPair skinny_pair_plan(int64_t long0, int64_t K0, int64_t long1, int64_t K1, int64_t rank, size_t partial_bytes) {
    const int64_t ks0 = K0 / 64, ks1 = K1 / 64, most = ks0 > ks1 ? ks0 : ks1;
    SkinnyPair best = {1, most};
    double best_us = 1e300;
    for (int c = 0; c < 5; ++c) {
        const int64_t across = (rank + SKINNY_RANK[c] - 1) / SKINNY_RANK[c];
        const int64_t t0 = (long0 + SKINNY_LONG[c] - 1) / SKINNY_LONG[c] * across, t1 = (long1 + SKINNY_LONG[c] - 1) / SKINNY_LONG[c] * across;
        const double pull = 128.0 * (double)(SKINNY_LONG[c] + SKINNY_RANK[c]) / 41e3;
        const double stream = 2.0 * ((double)long0 * (double)K0 + (double)long1 * (double)K1) / 4.6e6;
        int64_t last = 0;
        for (int64_t cut = 1; cut <= 64; ++cut) {
            const int64_t steps = (most + cut - 1) / cut, s0 = (ks0 + steps - 1) / steps, s1 = (ks1 + steps - 1) / steps;
            if (steps == last) continue;
            last = steps;
            const size_t sums = ((s0 > 1 ? (size_t)(s0 * long0) : 0) + (s1 > 1 ? (size_t)(s1 * long1) : 0)) * (size_t)rank * 4;
            if (cut > 1 && (s0 * t0 + s1 * t1 > RESIDENT || steps < 4 || sums > partial_bytes)) break;
            const double chain = (double)steps * pull, all = (double)(t0 * ks0 + t1 * ks1) * pull / (double)RESIDENT;
            double us = chain > all ? chain : all;
            if (us < stream) us = stream;
            if (sums) us += 3.0 + 0.4 * (double)(s0 > s1 ? s0 : s1) + 2.0 * (double)sums / 10e6;
            if (us < best_us) { best_us = us; best = {c, steps}; }
        }
    }
    return best;
}

// scratch of the calls that compute T or dY R^T and know no contraction length: slabs for fewer than 128 tiles
size_t dense_tn_plain_partial_bytes(int64_t n, int64_t m) {
    const int64_t tiles = ((m + 127) / 128) * ((n + 63) / 64);
    if (tiles >= RESIDENT / 2) return 0;
    return (size_t)((RESIDENT + tiles - 1) / tiles) * (size_t)n * (size_t)m * 4;
}

int dense_tn_plain_slabs(int64_t n, int64_t m, int64_t K, size_t partial_bytes) { return skinny_plan(n, m, K, partial_bytes).slabs; }

static SkinnyJob skinny_job(const DenseOperand& A, const DenseOperand& B, int64_t K, bf16_t* out, int64_t slab_steps) {
    SkinnyJob j = {A, B, (int)((K + 63) / 64), out, nullptr, 0, 0, 0, 1, (int)slab_steps};
    j.slabs = (j.ksteps + j.slab_steps - 1) / j.slab_steps;
    return j;
}
constexpr SkinnyJob NO_JOB = {{}, {}, 0, nullptr, nullptr, 0, 0, 0, 1, 1};

template <int LONG, int RANK, int NS, bool GRADIENTS>
static hipError_t launch_skinny_as(SkinnyJob j0, SkinnyJob j1, hipStream_t s) {
    using S = TnSmem<LONG, RANK, NS>;
    static_assert(S::TOTAL <= 160 * 1024, "LDS budget");
    auto place = [](SkinnyJob& j, bool flip) {
        const int bm = flip ? RANK : LONG, bn = flip ? LONG : RANK;
        j.tiles_m = (j.A.rows + bm - 1) / bm;
        j.tiles_n = (j.B.rows + bn - 1) / bn;
        j.grid = j.A.p ? super_grid(j.tiles_m, j.tiles_n) : 0;
    };
    place(j0, true);
    place(j1, !GRADIENTS);
    hipError_t e = allow_dynamic_lds<skinny_tn_kernel<LONG, RANK, NS, GRADIENTS>>(S::TOTAL);
    if (e != hipSuccess) return e;
    skinny_tn_kernel<LONG, RANK, NS, GRADIENTS><<<dim3((unsigned)(j0.grid * j0.slabs + j1.grid * j1.slabs)), dim3(tn_threads(LONG, RANK)), S::TOTAL, s>>>(j0, j1);
    if ((e = hipGetLastError()) != hipSuccess || (j0.slabs <= 1 && j1.slabs <= 1)) return e;
    auto sum = [](const SkinnyJob& j) {
        return j.slabs > 1 ? SkinnySum{(const f32x4*)j.sums, j.slabs, (int64_t)j.A.rows * j.B.rows / 4, (u32x2*)j.out} : SkinnySum{};
    };
    const SkinnySum a = sum(j0), b = sum(j1);
    skinny_sum_kernel<<<dim3((unsigned)((a.count4 + b.count4 + 255) / 256)), dim3(256), 0, s>>>(a, b);
    return hipGetLastError();
}

// sums: scratch for the slabs of both
template <bool GRADIENTS>
static hipError_t launch_skinny_tn(int tile, SkinnyJob j0, SkinnyJob j1, float* sums, hipStream_t s) {
    j0.sums = sums;
    j1.sums = sums + (j0.slabs > 1 ? (size_t)j0.slabs * j0.A.rows * j0.B.rows : 0);
    switch (tile) {
        case 0: return launch_skinny_as<64, 128, 6, GRADIENTS>(j0, j1, s);
        case 1: return launch_skinny_as<64, 64, 8, GRADIENTS>(j0, j1, s);
        case 2: return launch_skinny_as<128, 64, 6, GRADIENTS>(j0, j1, s);
        case 3: return launch_skinny_as<128, 128, 4, GRADIENTS>(j0, j1, s);
        default: return launch_skinny_as<64, 256, 4, GRADIENTS>(j0, j1, s);
    }
}

// T[n, r] = X[n, K] L[K, r] (k-major) or dY R^T with R [r][K]; partial_bytes of scratch at `partial` (none: no slabs)
hipError_t launch_skinny_factor(const bf16_t* B, int64_t n, int64_t K, const bf16_t* A, bool a_kmajor, int64_t r, bf16_t* T,
                                float* partial, size_t partial_bytes, hipStream_t s) {
    const SkinnyPlan p = skinny_plan(n, r, K, partial ? partial_bytes : 0);
    const SkinnyJob j = skinny_job({A, (int)r, (int)(a_kmajor ? r : K), (int)K}, {B, (int)n, (int)K, (int)K}, K, T, p.slab_steps);
    return launch_skinny_tn<false>(p.tile, a_kmajor ? j : NO_JOB, a_kmajor ? NO_JOB : j, partial, s);
}

// The same product for any shape (dense weights with a general N:M mask, where no sparse MFMA applies)
hipError_t launch_dense_tn_any(const bf16_t* B, int64_t n, const bf16_t* A, int64_t m, int64_t K, bf16_t* C,
                               hipStream_t s) {
    return launch_dense_tile<EPI_PLAIN, false, false>(dense_tile_choice(m, n, K / 64, K_CONTIGUOUS), {A, (int)m, (int)K, (int)K}, {B, (int)n, (int)K, (int)K}, K / 64, nullptr, C, s);
}

// ------------------------------------------------------------------------------------------
// Weight gradient of a layer with adapters: the packed dW as above plus the adapter gradients
// (chain rule of Eq. 11)   dL = X^T (dY R^T)  [d_in, r],   dR = (X L)^T dY  [r, d_out],
// all three contractions over the tokens.
// Workspace: Xt | dYt | r x d_in values (a size that is part of the interface, not used) | T = X L [b][r] | T2 = dY R^T [b][r] (r rows of a token-contiguous copy's pitch
// each) | scratch that launch_wgrad_masked and the skinny products use one after the other, for these with room for T and T2 once more.
// Xt and dYt are written where launch_wgrad_masked wants copies.
static size_t wgrad_adapter_shared_bytes(int64_t b, int64_t d_in, int64_t d_out, int64_t r) {
    if (d_in % 64 != 0 || d_out % 64 != 0) return wgrad_tail_bytes(b, d_in, d_out);   // no tile kernel for the skinny products
    const size_t tail = wgrad_tail_bytes(b, d_in, d_out);
    auto slabs = [r](int64_t n, int64_t K) {                  // of one of the four products, n the side that is not the rank
        const int sl = skinny_plan(n, r, K, ~(size_t)0).slabs;
        return sl > 1 ? (size_t)sl * (size_t)n * (size_t)r * 4 : 0;
    };
    const int64_t bp = (b + 63) / 64 * 64;
    size_t sums = 0;
    for (const size_t s : {slabs(b, d_in), slabs(b, d_out), slabs(d_in, bp), slabs(d_out, bp)}) sums = s > sums ? s : sums;
    return tail > sums ? tail : sums;
}

size_t wgrad_adapter_workspace_bytes(int64_t b, int64_t d_in, int64_t d_out, int64_t r) {
    size_t ld = (size_t)token_pitch((b + 63) / 64 * 64);
    return round256(token_copy_bytes(b, d_in)) + round256(token_copy_bytes(b, d_out)) + round256((size_t)r * d_in * 2) +
           2 * round256((size_t)b * r * 2) + 2 * round256((size_t)r * ld * 2) + wgrad_adapter_shared_bytes(b, d_in, d_out, r);
}

hipError_t launch_wgrad_adapter(const bf16_t* dY, const bf16_t* X, int64_t b, const uint8_t* meta, int64_t d_out,
                                int64_t d_in, const bf16_t* L, const bf16_t* R, int64_t r, bf16_t* gvals, bf16_t* dL,
                                bf16_t* dR, void* workspace, hipStream_t s) {
    const int64_t bp = (b + 63) / 64 * 64, ld = token_pitch(bp);
    uint8_t* w = (uint8_t*)workspace;
    bf16_t* Xt = (bf16_t*)w;   w += round256(token_copy_bytes(b, d_in));
    bf16_t* dYt = (bf16_t*)w;  w += round256(token_copy_bytes(b, d_out));
    w += round256((size_t)r * d_in * 2);
    bf16_t* T = (bf16_t*)w;    w += round256((size_t)r * ld * 2);
    bf16_t* T2 = (bf16_t*)w;   w += round256((size_t)r * ld * 2);
    float* const sums = (float*)w;
    w += 2 * round256((size_t)b * r * 2);
    float* tail = wgrad_tail_bytes(b, d_in, d_out) ? (float*)w : nullptr;
    const size_t room = 2 * round256((size_t)b * r * 2) + wgrad_adapter_shared_bytes(b, d_in, d_out, r);

    hipError_t e = launch_wgrad_masked(dY, X, b, meta, d_out, d_in, gvals, Xt, dYt, d_in % 32 == 0 ? tail : nullptr, s);
    if (e != hipSuccess) return e;
    // Extents that are not whole k-steps of the tile kernels, and short products: the kernel for ragged extents
    if (d_in % 64 != 0 || d_out % 64 != 0 || skinny_pair_is_short(b, d_in, d_out, r)) {
        if ((e = launch_skinny_factors({X, d_in, L, r, true, b, r, d_in, T}, {dY, d_out, R, d_out, false, b, r, d_out, T2}, s)) != hipSuccess) return e;
        return launch_skinny_gradients({X, d_in, T2, r, true, d_in, r, b, dL}, {T, r, dY, d_out, true, r, d_out, b, dR}, s);
    }
    // T and T2 in one launch, then dL and dR in another, each with one kernel for the sums of its slabs (2048 tokens, 4352 x
    // 4352, rank 128: ten launches, 71 us, before)
    const int ir = (int)r, ib = (int)b, in = (int)d_in, out = (int)d_out;
    const SkinnyPair f = skinny_pair_plan(b, d_in, b, d_out, r, room);
    if ((e = launch_skinny_tn<false>(f.tile, skinny_job({L, ir, ir, in}, {X, ib, in, in}, d_in, T, f.slab_steps),
                                     skinny_job({R, ir, out, out}, {dY, ib, out, out}, d_out, T2, f.slab_steps), sums, s)) != hipSuccess)
        return e;
    // Wide layers: T and T2, whose long contraction wants slabs, are the tiles' in any case (us, the call, 64 tokens, 64 x (2^24 + 64),
    // rank 64: 71880 with all four products on the kernel for ragged extents, 7800 so)
    if (too_wide(d_in, d_out)) return launch_skinny_gradients({X, d_in, T2, r, true, d_in, r, b, dL}, {T, r, dY, d_out, true, r, d_out, b, dR}, s);
    const SkinnyPair g = skinny_pair_plan(d_in, bp, d_out, bp, r, room);
    return launch_skinny_tn<true>(g.tile, skinny_job({T2, ir, ir, ib}, {X, in, in, ib}, b, dL, g.slab_steps),
                                  skinny_job({dY, out, out, ib}, {T, ir, ir, ib}, b, dR, g.slab_steps), sums, s);
}
