// Operands of the dense MFMA tiles: global memory -> LDS stages -> fragments, for both layouts in memory.
#pragma once
#include "pipeline.h"

namespace {

// 64 lanes x 16 bytes from `offset` + AT (per lane) inside the `bytes` bytes at `from` (uniform), zeros outside them; lane l's land at
// lds_dst + 16 l.  Written as instructions because behind the builtin the compiler waits for every such load (vmcnt(0)) before a
// transposing LDS read, which empties the load ring at each k-step; the kernels wait where they must.  The s_nop are the wait
// states between a vector instruction that writes a scalar register (v_readfirstlane) and a vector memory instruction that reads
// it (5), and between a write of m0 and its use (1), which the compiler does not insert in front of inline instructions.
// The immediate offset counts for the LDS address too.
template <int AT>
__device__ __forceinline__ void dma16_bounded(uint64_t from, uint32_t bytes, uint32_t offset, uint32_t lds_dst) {
    auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    const u32x4 rsrc = {uniform((uint32_t)from), uniform((uint32_t)(from >> 32)), uniform(bytes), 0x00020000u};
    asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen offset:%3 lds" ::"{m0}"(uniform(lds_dst - AT)), "v"(offset), "s"(rsrc),
                 "n"(AT)
                 : "memory");
}
// dma16 as an instruction, for kernels that mix both kinds of operands
__device__ __forceinline__ void dma16_quiet(const void* gsrc, uint32_t lds_dst) {
    const uint32_t dst = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_dst);
    asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %1, off" ::"{m0}"(dst), "v"(gsrc) : "memory");
}

// An operand of a dense product, in one of two layouts:
//   k-contiguous, [rows][ld]: whole k-steps of 64;
//   k-major, [k][ld] (activations as stored: k = tokens, rows = features): any number of k, rows % 8 == 0.
struct DenseOperand { const bf16_t* p; int rows, ld, k; };
constexpr int64_t KMAJOR_EXTENT_MAX = (int64_t)1 << 24;       // rows of a k-major operand: 32-bit offsets into a k-step of 64

// E rows of it by a k-step of 64, as a stage of E * 128 bytes in LDS.
//   k-contiguous: 8 rows x 128 bytes per load, 16-byte chunks rotated by (row / 2) % 8, fragments read with ds_read_b128.  Rows past
//     the end are other rows (wrap_row), never stored.
//   k-major: panels of 64 rows, [64 k][128 bytes] each; a load brings 8 k x 128 bytes, a wavefront the same 8 k of every panel.
//     Fragments (16 rows = 32 bytes of a k) are read with the transposing LDS read, sixteen k at a time (8 q + 4 h + 0 .. 3 for
//     quarter q of the wavefront): the 32-byte units of a k are exchanged by bits 1 and 3 of k, so that those of eight k fall
//     on all 64 banks.  Loads go through a buffer descriptor of the k-step's own: k past the last, and rows past the end of the
//     last k, read as zeros; rows past the end of another k are the next one's, never stored.
// KM: k-major; MIXED: the product's other operand is.  WAVE_ROWS: rows of a wavefront's fragments.
template <bool KM, bool MIXED, int E, int WAVE_ROWS>
struct DenseLoader {
    static constexpr int LD = E / 64;                         // 1 KiB loads per wavefront and k-step
    static constexpr int UNITS = !KM ? 2 : WAVE_ROWS % 64 ? WAVE_ROWS / 16 : 4;   // fragments less than a panel apart
    static_assert(LD <= 4, "immediate offsets of the k-major loads");
    const uint8_t* src[KM ? 1 : LD];
    uint64_t from;                                            // k-major: the first k-step
    uint32_t row_bytes, lds, lane_off;
    int whole, rest, ksteps;                                  // k-major: whole k-steps, positions in the one after them
    int frag_off[UNITS];

    // row0: first row of the tile; wave_row0: first of the wavefront's rows in the tile; steps: where look-ahead is clamped
    __device__ __forceinline__ void init(const DenseOperand& o, int row0, int wave_row0, int wave, int lane, int k_first, int steps,
                                         uint8_t* smem) {
        const int l16 = lane & 15, lq = lane >> 4;
        ksteps = steps;
        lds = (uint32_t)(uintptr_t)(uint8_t __attribute__((address_space(3)))*)smem;
        if constexpr (KM) {
            row_bytes = (uint32_t)o.ld * 2;
            from = (uint64_t)o.p + (uint64_t)(uint32_t)k_first * ((uint64_t)row_bytes * 64);
            from = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)from) |
                   (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(from >> 32)) << 32;
            whole = o.k / 64 - k_first;
            rest = o.k % 64;
            lane_off = (uint32_t)row0 * 2 + (uint32_t)(8 * wave + (lane >> 3)) * row_bytes +
                       (uint32_t)(((lane & 7) ^ ((((lane >> 4) & 1) | ((wave & 1) << 1)) * 2)) * 16);
            const int sw = ((l16 >> 3) & 1) | ((lq & 1) << 1);
#pragma unroll
            for (int i = 0; i < UNITS; ++i) {
                const int f = wave_row0 / 16 + i;
                frag_off[i] = (f >> 2) * 8192 + (8 * lq + (l16 >> 2)) * 128 + (((f & 3) ^ sw) * 32) + (l16 & 3) * 8;
            }
        } else {
#pragma unroll
            for (int i = 0; i < LD; ++i) {
                const int rl = slot(i, wave) * 8 + (lane >> 3);
                src[i] = (const uint8_t*)o.p + (size_t)wrap_row(row0 + rl, o.rows) * o.ld * 2 + (((lane & 7) ^ ((rl >> 1) & 7)) * 16) +
                         (size_t)k_first * 128;
            }
            const int sw = (l16 >> 1) & 7;                    // a fragment is 2 KiB; lane (l16, lq) wants chunks lq and 4 + lq
            frag_off[0] = wave_row0 * 128 + l16 * 128 + ((lq ^ sw) * 16);
            frag_off[1] = wave_row0 * 128 + l16 * 128 + (((4 + lq) ^ sw) * 16);
        }
    }
    // 1 KiB piece of the stage that load i of the wavefront fills; loads 2 j and 2 j + 1 of all wavefronts are rows 128 j .. + 127
    __device__ __forceinline__ static int slot(int i, int wave) {
        return KM ? i * 8 + wave : LD % 2 ? wave * LD + i : i / 2 * 16 + wave * 2 + (i & 1);
    }
    __device__ __forceinline__ void load(int ks, int i, uint8_t* smem, int stage, int wave) const {   // stage: its offset in smem
        const int dst = stage + slot(i, wave) * 1024;
        if constexpr (KM) {
            const uint32_t bytes = (ks < whole ? 64u : ks == whole ? (uint32_t)rest : 0u) * row_bytes;
            const uint64_t at = from + (uint64_t)(uint32_t)ks * ((uint64_t)row_bytes * 64);
            if (i == 0) dma16_bounded<0>(at, bytes, lane_off, lds + dst);
            else if (i == 1) dma16_bounded<128>(at, bytes, lane_off, lds + dst);
            else if (i == 2) dma16_bounded<256>(at, bytes, lane_off, lds + dst);
            else dma16_bounded<384>(at, bytes, lane_off, lds + dst);
        } else {
            const int kc = ks < ksteps ? ks : ksteps - 1;
            if (MIXED) dma16_quiet(src[i] + (size_t)kc * 128, lds + dst);
            else dma16(src[i] + (size_t)kc * 128, smem + dst);
        }
    }
    // the wavefront's fragments in a stage
    struct Stage { const uint8_t* p; uint32_t at[UNITS]; };
    __device__ __forceinline__ Stage stage(uint8_t* smem, int offset) const {
        Stage st;
        st.p = smem + offset;
        if constexpr (KM)
#pragma unroll
            for (int u = 0; u < UNITS; ++u) {
                st.at[u] = lds + (uint32_t)(offset + frag_off[u]);
                asm("" : "+v"(st.at[u]));                     // one address for all of the unit's reads: the rest is in their offsets
            }
        return st;
    }
    // fragment i, half h of the k-step: 16 rows x 32 k
    __device__ __forceinline__ u32x4 half(const Stage& st, int i, int h) const {
        if constexpr (KM) {
            typedef s16x4 __attribute__((address_space(3)))* lds_t;
            const uint32_t at = st.at[i % UNITS] + i / UNITS * 8192 + h * 4096;
            union { s16x4 q[2]; u32x4 u; } x;
            x.q[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(uintptr_t)at);
            x.q[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(uintptr_t)(at + 512));
            return x.u;
        }
        return *(const u32x4*)(st.p + frag_off[h] + i * 2048);
    }
    __device__ __forceinline__ BFrag frag(const Stage& st, int i) const {
        BFrag f;
        f.u[0] = half(st, i, 0);
        f.u[1] = half(st, i, 1);
        return f;
    }
};

}  // namespace
