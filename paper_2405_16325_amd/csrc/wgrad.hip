// slope_wgrad_masked for few tokens on small layers, and for layers of 2^24 rows or columns and more, which the 32-bit offsets of
// the dense tiles do not reach (wgrad_tn.hip): dW = dY^T X (Eq. 5) on dense MFMA, with the prune-and-compress step of
// Algorithm 1 line 13 folded into the epilogue, 64-bit addresses and plain register-staged pipelines.
//
// The contraction runs over the b tokens, which is the slow index of both operands, so both are
// staged in LDS as [token][feature] slabs (the same order as in memory: fully coalesced loads) and
// read back with ds_read_b64_tr_b16, CDNA4's transposing LDS read: inside each block of 16 lanes,
// lane r receives element r of four consecutive slab rows, i.e. four consecutive k of one feature.
//
// The MFMA is v_mfma_f32_16x16x32_bf16 with D rows = d_in and D columns = d_out:
//   D lane l holds column (d_out) l%16 and rows (d_in) 4*(l/16) .. +3 = exactly one group of four
//   of W^R's row, so the epilogue picks two of a lane's four accumulators with the group's
//   metadata nibble and stores them as one 4-byte pair of the packed gradient.
#include "pipeline.h"

namespace {

constexpr int WG_KS = 32;                      // tokens per LDS stage

__device__ __forceinline__ void wgrad_tile_of_block(int nblocks, int tiles_m, int tiles_n, int& tm, int& tn) {
    int b = blockIdx.x;
    int xcd = b % XCDS, pos = b / XCDS;
    int q = nblocks / XCDS, rem = nblocks % XCDS;
    int id = xcd * q + (xcd < rem ? xcd : rem) + pos;
    constexpr int GM = 4;
    int per_group = GM * tiles_n;
    int g = id / per_group, first_m = g * GM;
    int gsize = tiles_m - first_m < GM ? tiles_m - first_m : GM;
    int in_group = id - g * per_group;
    tm = first_m + in_group % gsize;
    tn = in_group / gsize;
}

// BM: tile extent along d_in (MFMA rows), BN: along d_out (MFMA columns).
template <int BM, int BN>
struct WgSmem {
    static constexpr int PITCH_A = BM * 2 + 32;     // bytes per token row; pitch % 128 == 32 keeps the
    static constexpr int PITCH_B = BN * 2 + 32;     // four rows of a transposing read on distinct banks
    static constexpr int A_BYTES = WG_KS * PITCH_A;
    static constexpr int B_BYTES = WG_KS * PITCH_B;
    static constexpr int STAGE = A_BYTES + B_BYTES;
};

__device__ __forceinline__ s16x4 lds_read_tr(const uint8_t* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p);
}

template <int BM, int BN>
__global__ void __launch_bounds__(256) wgrad_kernel(const bf16_t* __restrict__ dY, const bf16_t* __restrict__ X, int b,
                                                    const uint8_t* __restrict__ meta, int d_out, int d_in,
                                                    bf16_t* __restrict__ G, int tiles_m, int tiles_n) {
    using S = WgSmem<BM, BN>;
    constexpr int MF = BM / 32, NF = BN / 32;           // 16 x 16 fragments per wavefront (2 x 2 waves)
    constexpr int A_LD = BM / 64, B_LD = BN / 64;       // 16-byte loads per lane per stage (32 rows)
    extern __shared__ __align__(16) uint8_t smem[];

    int tm, tn;
    wgrad_tile_of_block(tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
    const int i0 = tm * BM, o0 = tn * BN;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, lq = lane >> 4;

    // global -> register staging: lane owns 16-byte pieces (8 features) of token rows
    constexpr int A_PER_ROW = BM / 8, B_PER_ROW = BN / 8;
    uint4 a_reg[A_LD], b_reg[B_LD];
    auto load_global = [&](int t0) {
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            int idx = t + 256 * i, row = idx / A_PER_ROW, c = idx % A_PER_ROW;
            int tok = t0 + row, col = i0 + 8 * c;
            a_reg[i] = (tok < b && col < d_in) ? *(const uint4*)(X + (size_t)tok * d_in + col) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            int idx = t + 256 * i, row = idx / B_PER_ROW, c = idx % B_PER_ROW;
            int tok = t0 + row, col = o0 + 8 * c;
            b_reg[i] = (tok < b && col < d_out) ? *(const uint4*)(dY + (size_t)tok * d_out + col) : make_uint4(0, 0, 0, 0);
        }
    };
    auto store_lds = [&](int stage) {
        uint8_t* base = smem + stage * S::STAGE;
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            int idx = t + 256 * i, row = idx / A_PER_ROW, c = idx % A_PER_ROW;
            *(uint4*)(base + row * S::PITCH_A + 16 * c) = a_reg[i];
        }
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            int idx = t + 256 * i, row = idx / B_PER_ROW, c = idx % B_PER_ROW;
            *(uint4*)(base + S::A_BYTES + row * S::PITCH_B + 16 * c) = b_reg[i];
        }
    };

    f32x4 acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // transposing-read addresses: lane (s = l%16, q = l/16) points at slab row 8q + 4h + s/4,
    // feature 4*(s%4); it receives k = 8q + 4h .. +3 of feature s
    const int tr_row = 8 * lq + (l16 >> 2), tr_col = 4 * (l16 & 3);
    const int a_off = tr_row * S::PITCH_A + 2 * (wm * (BM / 2) + tr_col);
    const int b_off = tr_row * S::PITCH_B + 2 * (wn * (BN / 2) + tr_col);

    const int ksteps = (b + WG_KS - 1) / WG_KS;
    load_global(0);
    store_lds(0);
    __syncthreads();
    for (int ks = 0; ks < ksteps; ++ks) {
        const int stage = ks & 1;
        if (ks + 1 < ksteps) load_global((ks + 1) * WG_KS);
        const uint8_t* sa = smem + stage * S::STAGE + a_off;
        const uint8_t* sb = smem + stage * S::STAGE + S::A_BYTES + b_off;
        bf16x8 bf[NF];
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            union { s16x4 h[2]; bf16x8 v; } x;
            x.h[0] = lds_read_tr(sb + 32 * j);
            x.h[1] = lds_read_tr(sb + 32 * j + 4 * S::PITCH_B);
            bf[j] = x.v;
        }
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            union { s16x4 h[2]; bf16x8 v; } a;
            a.h[0] = lds_read_tr(sa + 32 * i);
            a.h[1] = lds_read_tr(sa + 32 * i + 4 * S::PITCH_A);
#pragma unroll
            for (int j = 0; j < NF; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, bf[j], acc[i][j], 0, 0, 0);
        }
        if (ks + 1 < ksteps) store_lds(stage ^ 1);
        __syncthreads();
    }

    // epilogue: a lane's four accumulators are one group of four along d_in of row o
    const size_t mpitch = (size_t)d_in / 8, gpitch = (size_t)d_in / 2;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        int o = o0 + (wn * NF + j) * 16 + l16;
        if (o >= d_out) continue;
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            int col = i0 + (wm * MF + i) * 16 + lq * 4;   // first d_in index of the group
            if (col >= d_in) continue;
            int g = col >> 2;
            uint32_t nib = (meta[(size_t)o * mpitch + (g >> 1)] >> (4 * (g & 1))) & 0xFu;
            uint32_t a = nib & 3u, c = nib >> 2;
            f32x4 v = acc[i][j];
            float v0 = a == 0 ? v[0] : (a == 1 ? v[1] : v[2]);
            float v1 = c == 1 ? v[1] : (c == 2 ? v[2] : v[3]);
            union { __bf16 h[2]; uint32_t u; } out;
            out.h[0] = (__bf16)v0;
            out.h[1] = (__bf16)v1;
            *(uint32_t*)(G + (size_t)o * gpitch + 2 * g) = out.u;
        }
    }
}

// Few tokens on few tiles: 64 x 64 of them, and four groups of four wavefronts that take the slabs of 32 tokens in turn, each with LDS
// stages of its own; the groups' partial tiles are added through LDS in group order.  Such a layer is bound by the chain of
// latencies along its few k-steps, and here a quarter of them follow one another.
constexpr int WGS_GROUPS = 4, WGS_EDGE = 64, WGS_SUM_PITCH = WGS_EDGE + 4;   // floats per d_out row of a partial tile
struct WgsSmem {
    using S = WgSmem<WGS_EDGE, WGS_EDGE>;
    static constexpr int RING = WGS_GROUPS * 2 * S::STAGE, SUMS = WGS_GROUPS * WGS_EDGE * WGS_SUM_PITCH * 4;
    static constexpr int TOTAL = RING > SUMS ? RING : SUMS;
};
__global__ void __launch_bounds__(256 * WGS_GROUPS) wgrad_groups_kernel(const bf16_t* __restrict__ dY,
                                                                        const bf16_t* __restrict__ X, int b,
                                                                        const uint8_t* __restrict__ meta, int d_out,
                                                                        int d_in, bf16_t* __restrict__ G, int tiles_m,
                                                                        int tiles_n) {
    using S = WgSmem<WGS_EDGE, WGS_EDGE>;
    __shared__ __align__(16) uint8_t smem[WgsSmem::TOTAL];
    int tm, tn;
    wgrad_tile_of_block(tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
    const int i0 = tm * WGS_EDGE, o0 = tn * WGS_EDGE;
    const int group = (int)threadIdx.x >> 8, t = threadIdx.x & 255, lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, lq = lane >> 4;
    uint8_t* const ring = smem + group * 2 * S::STAGE;

    // a lane brings one 16-byte piece of either operand per slab: token row t / 8, features 8 (t % 8) .. + 7
    const int row = t >> 3, c = t & 7;
    const bool a_in = i0 + 8 * c < d_in, b_in = o0 + 8 * c < d_out;      // extents are multiples of 8: whole pieces
    uint4 a_reg, b_reg;
    auto load_global = [&](int slab) {
        const uint32_t tok = (uint32_t)slab * WG_KS + row;     // b < 2^31: past the last token, not around it
        a_reg = tok < (uint32_t)b && a_in ? *(const uint4*)(X + (size_t)tok * d_in + i0 + 8 * c) : make_uint4(0, 0, 0, 0);
        b_reg = tok < (uint32_t)b && b_in ? *(const uint4*)(dY + (size_t)tok * d_out + o0 + 8 * c) : make_uint4(0, 0, 0, 0);
    };
    auto store_lds = [&](int stage) {
        uint8_t* base = ring + stage * S::STAGE;
        *(uint4*)(base + row * S::PITCH_A + 16 * c) = a_reg;
        *(uint4*)(base + S::A_BYTES + row * S::PITCH_B + 16 * c) = b_reg;
    };
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const int tr_row = 8 * lq + (l16 >> 2), tr_col = 4 * (l16 & 3);
    const int a_off = tr_row * S::PITCH_A + 2 * (wm * 32 + tr_col), b_off = tr_row * S::PITCH_B + 2 * (wn * 32 + tr_col);

    // group g takes slabs g, g + 4, ...; slabs past the last token are zeros
    const int trips = (int)((((uint32_t)b + WG_KS - 1) / WG_KS + WGS_GROUPS - 1) / WGS_GROUPS);
    load_global(group);
    store_lds(0);
    __syncthreads();
    for (int tr = 0; tr < trips; ++tr) {
        const int stage = tr & 1;
        if (tr + 1 < trips) load_global((tr + 1) * WGS_GROUPS + group);
        const uint8_t* sa = ring + stage * S::STAGE + a_off;
        const uint8_t* sb = ring + stage * S::STAGE + S::A_BYTES + b_off;
        bf16x8 af[2], bf[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            union { s16x4 h[2]; bf16x8 v; } x, y;
            x.h[0] = lds_read_tr(sb + 32 * j);
            x.h[1] = lds_read_tr(sb + 32 * j + 4 * S::PITCH_B);
            y.h[0] = lds_read_tr(sa + 32 * j);
            y.h[1] = lds_read_tr(sa + 32 * j + 4 * S::PITCH_A);
            bf[j] = x.v;
            af[j] = y.v;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
        if (tr + 1 < trips) store_lds(stage ^ 1);
        __syncthreads();
    }
    // partial tiles [group][d_out row][d_in column]; the stages are idle
    float* const part = (float*)smem;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            *(f32x4*)(part + (group * WGS_EDGE + (wn * 2 + j) * 16 + l16) * WGS_SUM_PITCH + (wm * 2 + i) * 16 + lq * 4) = acc[i][j];
    __syncthreads();
    // one group of four columns per thread: 64 rows x 16 groups
    const int orow = (int)threadIdx.x >> 4, g = threadIdx.x & 15;
    f32x4 v = *(const f32x4*)(part + orow * WGS_SUM_PITCH + 4 * g);
#pragma unroll
    for (int q = 1; q < WGS_GROUPS; ++q) {
        const f32x4 x = *(const f32x4*)(part + (q * WGS_EDGE + orow) * WGS_SUM_PITCH + 4 * g);
        v[0] += x[0]; v[1] += x[1]; v[2] += x[2]; v[3] += x[3];
    }
    const int o = o0 + orow, col = i0 + 4 * g;
    if (o >= d_out || col >= d_in) return;
    const uint32_t nib = (meta[(size_t)o * (d_in / 8) + (col >> 3)] >> (col & 4)) & 0xFu;
    const uint32_t ka = nib & 3u, kc = nib >> 2;
    union { __bf16 h[2]; uint32_t u; } out;
    out.h[0] = (__bf16)(ka == 0 ? v[0] : (ka == 1 ? v[1] : v[2]));
    out.h[1] = (__bf16)(kc == 1 ? v[1] : (kc == 2 ? v[2] : v[3]));
    *(uint32_t*)(G + (size_t)o * (d_in / 2) + (col >> 1)) = out.u;
}

template <int BM, int BN>
hipError_t launch_tile(const bf16_t* dY, const bf16_t* X, int64_t b, const uint8_t* meta, int64_t d_out, int64_t d_in,
                       bf16_t* G, hipStream_t s) {
    using S = WgSmem<BM, BN>;
    int tiles_m = (int)((d_in + BM - 1) / BM), tiles_n = (int)((d_out + BN - 1) / BN);
    size_t smem = 2 * S::STAGE;
    auto kern = wgrad_kernel<BM, BN>;
    hipError_t e = allow_dynamic_lds<wgrad_kernel<BM, BN>>((int)smem);
    if (e != hipSuccess) return e;
    kern<<<dim3((unsigned)(tiles_m * tiles_n)), dim3(256), smem, s>>>(dY, X, (int)b, meta, (int)d_out, (int)d_in, G,
                                                                       tiles_m, tiles_n);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_wgrad_wide(const bf16_t* dY, const bf16_t* X, int64_t b, const uint8_t* meta, int64_t d_out, int64_t d_in,
                             bf16_t* gvals, hipStream_t s) {
    return launch_tile<128, 128>(dY, X, b, meta, d_out, d_in, gvals, s);
}

// Up to four trips of the groups through one round of tiles, one trip (up to 128 tokens) through two.  us, the dense tiles / here:
// 1000 x 1000, 1 token 4.9 / 4.35, 128 5.4 / 4.75, 300 6.7 / 6.45, 512 7.75 / 7.7, 600 8.5 / 8.7; 264 x 272, 128 4.7 / 4.1; 1024 x
// 1024, 128 5.3 / 4.8; two rounds, 2264 x 696, 64 tokens 5.45 / 5.7, 65 5.9 / 5.7, 128 6.5 / 6.0, 300 8.0 / 8.4.
bool wgrad_in_groups(int64_t b, int64_t d_in, int64_t d_out) {
    const int64_t tiles = ((d_in + WGS_EDGE - 1) / WGS_EDGE) * ((d_out + WGS_EDGE - 1) / WGS_EDGE);
    constexpr int64_t TRIP = WGS_GROUPS * WG_KS;
    return tiles <= RESIDENT ? b <= 4 * TRIP : tiles <= 2 * RESIDENT && b > TRIP / 2 && b <= TRIP;
}
hipError_t launch_wgrad_groups(const bf16_t* dY, const bf16_t* X, int64_t b, const uint8_t* meta, int64_t d_out, int64_t d_in,
                               bf16_t* gvals, hipStream_t s) {
    const int64_t tm = (d_in + WGS_EDGE - 1) / WGS_EDGE, tn = (d_out + WGS_EDGE - 1) / WGS_EDGE;
    wgrad_groups_kernel<<<dim3((unsigned)(tm * tn)), dim3(256 * WGS_GROUPS), 0, s>>>(dY, X, (int)b, meta, (int)d_out, (int)d_in, gvals,
                                                                                     (int)tm, (int)tn);
    return hipGetLastError();
}
