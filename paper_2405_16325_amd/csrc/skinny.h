// One tile of a skinny adapter product (one side as short as an adapter's rank) per workgroup, shared by the kernel for
// ragged layers, the product T = X L of a few hundred tokens and the workgroups that compute it beside a sparse product.
#pragma once
#include "common.h"

namespace {

// C[i][j] = sum_k B(i, k) * A(j, k) for rows of any multiple of 8 elements and any number of tokens, bf16 operands, fp32
// accumulation.
// An operand is either k-contiguous, [rows][ld] with K % 8 == 0 (KMAJOR false: the 16 bytes an MFMA lane wants are
// loaded straight into its registers), or k-major, [K][ld] with rows % 8 == 0 (KMAJOR true: 32 x rows pieces staged in
// LDS as stored and read back with the transposing LDS read).  Pieces of 16 bytes are inside an operand or outside
// as a whole; outside they are zeros.
//
// With one side as short as an adapter's rank the product has a few dozen tiles, so what bounds it is the chain of
// memory latencies along k.  A workgroup therefore takes a small tile, 32 x 64, and its wavefronts (eight) take the
// chunks of 32 k in turn (wavefront w: chunks w, w + 8, ...), each with the next chunk's loads in flight (four
// chunks' were 10 % slower) and a private stage in LDS: no barrier before the sum of the eight partial tiles, which is in a fixed order.
// 1000 tokens, 1000 x 1000, rank 64: 94 us with plain fp32 multiply-adds on 32 x 32 tiles, 6 us here, per product.
constexpr int SK_WAVES = 8, SK_BI = 32, SK_BJ = 64;
constexpr int SK_PA = SK_BJ * 2 + 32, SK_PB = SK_BI * 2 + 32;   // bytes per staged k: the four rows of a transposing
                                                                // read fall on distinct banks
constexpr int SK_STAGE = 32 * (SK_PA + SK_PB);
constexpr int SK_SUM_PITCH = SK_BJ + 4;                         // floats per token row of a partial tile
// bytes of LDS that a tile of WAVES wavefronts takes
constexpr int skinny_lds(int waves) { return waves * (SK_STAGE > SK_BI * SK_SUM_PITCH * 4 ? SK_STAGE : SK_BI * SK_SUM_PITCH * 4); }
constexpr int SK_LDS = skinny_lds(SK_WAVES);

template <bool KMAJOR, int F>                                   // F fragments of 16 rows
struct SkinnyOperand {
    static constexpr int PITCH = F * 32 + 32;
    const bf16_t* base;
    int64_t ld;
    int rows;
    uint32_t K;
    int row0;
    __device__ __forceinline__ void load(uint32_t k0, int lane, u32x4 (&v)[F]) const {
#pragma unroll
        for (int u = 0; u < F; ++u) {
            v[u] = (u32x4){0u, 0u, 0u, 0u};
            if (KMAJOR) {
                const int p = lane + 64 * u, row = row0 + 8 * (p % (2 * F));
                const uint32_t k = k0 + (uint32_t)p / (2 * F);
                if (k < K && row < rows) v[u] = *(const u32x4*)(base + (int64_t)k * ld + row);
            } else {
                const int row = row0 + 16 * u + (lane & 15);
                const uint32_t k = k0 + 8 * (lane >> 4);
                if (k < K && row < rows) v[u] = *(const u32x4*)(base + (int64_t)row * ld + k);
            }
        }
    }
    // the loaded pieces -> MFMA fragments (through the wavefront's stage if k-major)
    __device__ __forceinline__ void fragments(const u32x4 (&v)[F], int lane, uint8_t* stage, bf16x8 (&f)[F]) const {
        if (KMAJOR) {
#pragma unroll
            for (int u = 0; u < F; ++u) {
                const int p = lane + 64 * u;
                *(u32x4*)(stage + (p / (2 * F)) * PITCH + (p % (2 * F)) * 16) = v[u];
            }
            asm volatile("" ::: "memory");                      // one wavefront's LDS accesses complete in order
            const int l16 = lane & 15, lq = lane >> 4;
            const uint8_t* tr = stage + (8 * lq + (l16 >> 2)) * PITCH + 8 * (l16 & 3);
#pragma unroll
            for (int u = 0; u < F; ++u) {
                union { s16x4 h[2]; bf16x8 v; } x;
                x.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(tr + 32 * u));
                x.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (s16x4 __attribute__((address_space(3)))*)(tr + 4 * PITCH + 32 * u));
                f[u] = x.v;
            }
            asm volatile("" ::: "memory");
        } else {
#pragma unroll
            for (int u = 0; u < F; ++u) {
                union { u32x4 u4; bf16x8 v; } x;
                x.u4 = v[u];
                f[u] = x.v;
            }
        }
    }
};

// The tile at rows i0 of B and j0 of A, contraction [k_begin, K) (k_begin a multiple of 32; K bounds the operands too):
// store(i, j, four sums of columns j .. j + 3 of the tile's row i).  smem: skinny_lds(WAVES) bytes, 16-byte aligned.  Every
// thread of a workgroup of WAVES wavefronts must make the call (it contains barriers).
template <bool BKMAJOR, bool AKMAJOR, int WAVES, class Store>
__device__ __forceinline__ void skinny_sums(const bf16_t* __restrict__ B, int64_t ldb, const bf16_t* __restrict__ A, int64_t lda,
                                            int n, int m, uint32_t k_begin, uint32_t K, int i0, int j0, uint8_t* smem, const Store& store) {
    constexpr int FA = SK_BJ / 16, FB = SK_BI / 16;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const SkinnyOperand<BKMAJOR, FB> ob = {B, ldb, n, K, i0};
    const SkinnyOperand<AKMAJOR, FA> oa = {A, lda, m, K, j0};
    uint8_t* const stage = smem + wave * SK_STAGE;
    f32x4 acc[FA][FB];
#pragma unroll
    for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int j = 0; j < FB; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    u32x4 va[FA], vb[FB];
    constexpr uint32_t step = 32 * WAVES;                       // K < 2^31: a look-ahead past it does not wrap in 32 bits
    static_assert(0x7FFFFFFFu + 2 * step + 32 > 0x7FFFFFFFu, "k0 + step and the chunk after it");
    oa.load(k_begin + wave * 32, lane, va);
    ob.load(k_begin + wave * 32, lane, vb);
    for (uint32_t k0 = k_begin + wave * 32; k0 < K; k0 += step) {    // uniform per wavefront
        u32x4 na[FA], nb[FB];
        oa.load(k0 + step, lane, na);                           // past the end: zeros, no access
        ob.load(k0 + step, lane, nb);
        bf16x8 fa[FA], fb[FB];
        oa.fragments(va, lane, stage, fa);
        ob.fragments(vb, lane, stage + 32 * SK_PA, fb);
#pragma unroll
        for (int i = 0; i < FA; ++i)
#pragma unroll
            for (int j = 0; j < FB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < FA; ++u) va[u] = na[u];
#pragma unroll
        for (int u = 0; u < FB; ++u) vb[u] = nb[u];
    }
    // partial tiles to LDS (lane: column i = l16, rows j = 4 lq .. + 3), summed in wavefront order
    __syncthreads();
    float* const part = (float*)smem;
    const int l16 = lane & 15, lq = lane >> 4;
#pragma unroll
    for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int j = 0; j < FB; ++j)
            *(f32x4*)(part + (wave * SK_BI + 16 * j + l16) * SK_SUM_PITCH + 16 * i + 4 * lq) = acc[i][j];
    __syncthreads();
#pragma unroll
    for (int idx = t; idx < SK_BI * SK_BJ / 4; idx += WAVES * 64) {  // 32 rows x 16 groups of four
        const int row = idx / (SK_BJ / 4), col = (idx % (SK_BJ / 4)) * 4;
        f32x4 v = *(const f32x4*)(part + row * SK_SUM_PITCH + col);
#pragma unroll
        for (int w = 1; w < WAVES; ++w) {
            const f32x4 x = *(const f32x4*)(part + (w * SK_BI + row) * SK_SUM_PITCH + col);
            v[0] += x[0]; v[1] += x[1]; v[2] += x[2]; v[3] += x[3];
        }
        store(row, col, v);
    }
}

// The same with the results in memory: bf16 in C[n][m], or the fp32 sums in sums[n][m] if that is given (m % 8 == 0).
template <bool BKMAJOR, bool AKMAJOR, int WAVES = SK_WAVES>
__device__ __forceinline__ void skinny_tile(const bf16_t* __restrict__ B, int64_t ldb, const bf16_t* __restrict__ A, int64_t lda,
                                            int n, int m, uint32_t k_begin, uint32_t K, int i0, int j0, bf16_t* __restrict__ C,
                                            float* __restrict__ sums, uint8_t* smem) {
    skinny_sums<BKMAJOR, AKMAJOR, WAVES>(B, ldb, A, lda, n, m, k_begin, K, i0, j0, smem, [&](int row, int col, const f32x4& v) {
        if (i0 + row >= n || j0 + col >= m) return;
        if (sums) {
            *(f32x4*)(sums + (int64_t)(i0 + row) * m + j0 + col) = v;
            return;
        }
        union { __bf16 h[4]; u32x2 u; } o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o.h[e] = (__bf16)v[e];
        *(u32x2*)(C + (int64_t)(i0 + row) * m + j0 + col) = o.u;
    });
}

}  // namespace
