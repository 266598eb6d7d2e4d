// Network kernels of the large levels on matrix cores in float (levels 1 to 3
// above 32768 cells), one work item (a 64 x 4 column footprint over 4 or 2
// z-planes) at a time (Alg. 2: CConv_1 + pool down, interpolation + CConv_2 +
// combine up; at level 1 also the mask, the scaling and the dots).
//
// These kernels are bound by issue and by latency together, not by memory
// (their traffic is 1 TB/s).  On the benchmark's 128^3 scene the waves of
// level 1 issue in 28 % of their cycles, wait for a turn in 28 to 32 % and for
// LDS, memory or a barrier in 39 to 44 %; the matrix cores are busy in 7 to
// 11 %.  So the item is staged and evaluated with as few instructions per cell
// as possible.  All planes of the item, with their one-cell border, are staged in
// LDS in one go, as one 8-byte record per cell: the CConv input (float) and the
// cell's two MFMA features (fluid and air counts as a bf16 / fp16 pair).  One
// barrier separates staging from the CConv, and every LDS address of the CConv
// is a per-lane base plus a constant.
//
// Wave w covers x = 16 w .. 16 w + 15 of the footprint and its four rows; lane
// (g, n) (g = lane / 16, n = lane % 16) owns cell (x = 16 w + n, y = g) of each
// plane, and row q of a plane is one 16-cell group.  Groups are classified once
// per solve (k_march_modes; the labels do not change during a solve):
//   zero     every output is zero;
//   pure     every cell that matters has an all-fluid window, i.e. the constant
//            fluid kernel (on coarser levels also all-air and all-solid windows,
//            each with its own).  A wave with any pure group applies that kernel to
//            all its cells: the 9 inputs of a plane around the lane's column
//            are read once and enter the sums of the three output planes that
//            see them (27 multiply-adds and 13 reads per cell of a 4-plane
//            item, the kernel in scalar registers);
//   general  matrix cores.  The per-cell kernels K^T[tap][cell] = A[tap][feature]
//            B[feature][cell] come out with lane (g, n) holding the taps of
//            window positions {4g + i, 16 + 4g + i : i < 4} of cell n; the lane
//            reads the records at exactly those positions (the feature and tap
//            enumerations coincide), so they give both its B fragment and its
//            eight input values.  The four partial sums of a cell (one per lane
//            group) are combined for the four groups together with a
//            reduce-scatter over the lane groups (two gfx950 permlane swaps).
#pragma once

#include "nps_kernels.hpp"

namespace nps {

enum GroupMode : uint32_t { kGZero = 0, kGPure = 1, kGGeneral = 2, kGPureAir = 4, kGPureSolid = 8 };
constexpr uint32_t kAnyGeneral = 0x02020202u;   // over a wave's four modes

// One mode byte per 16-cell group, the four rows of a wave in one aligned word: word
// (z ncy + cy) nwx + (16-cell column).  nwx counts the columns that hold cells (words
// for whole footprints take up to four times as much: for the coarser levels of a grid
// 4 cells wide and 375936 long, 118 MB more).
__host__ __device__ inline int wave_columns(Grid g) { return (int)((unsigned)(g.nx + 15) / 16u); }
__host__ __device__ inline size_t group_mode_bytes(Grid g) {
    return (size_t)wave_columns(g) * ((g.ny + PY - 1) / PY) * g.nz * 4;
}

// Group modes of the level-1 down (CConv_1, input zero off fluid) and up
// (CConv_2, output restricted to fluid) kernels, and one byte per item and
// kernel that is set when all its groups are zero.  One block per item
// (CH planes).
//   down: zero when no window of the group holds fluid; pure when every
//         window that holds fluid is all fluid (a window without fluid
//         outputs zero under any kernel);
//   up:   zero when no cell of the group is fluid; pure when every fluid
//         cell's window is all fluid (other outputs are masked).
// A row of 64 labels becomes a 64-bit mask (one ballot), so the windows are
// shifts and a few ANDs and ORs of row masks: one label load per cell and halo
// cell, where one thread per cell read its 27 window labels (128^3: 9.9 us;
// before, 30.5 us and 4.5 us for the item flags in a launch of their own).
template <int CH>
__global__ __launch_bounds__(kBlock) void k_march_modes(const uint8_t* __restrict__ lab, Grid g,
                                                        uint8_t* __restrict__ mdown, uint8_t* __restrict__ mup,
                                                        uint8_t* __restrict__ zdown, uint8_t* __restrict__ zup) {
    constexpr int R = (CH + 2) * PHY;
    __shared__ uint64_t own_s[R];   // fluid cells of a row
    __shared__ uint32_t edge_s[R];  // and of the cells beside it (bits 0, 1)
    const Columns cl = march_columns(g);
    const int per = cl.ncx * cl.ncy, rest = (int)blockIdx.x % per, zc = (int)blockIdx.x / per;
    const int cx = rest % cl.ncx, cy = rest / cl.ncx, x0 = cx * PX, y0 = cy * PY, z0 = zc * CH;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t own[R / 4], edge[R / 4];
    static_assert(R % 4 == 0, "whole rounds of four waves");
#pragma unroll
    for (int k = 0; k < R / 4; ++k) {
        const int r = wv + 4 * k, z = z0 + r / PHY - 1, y = y0 + r % PHY - 1;
        const bool row = z >= 0 && z < g.nz && y >= 0 && y < g.ny;
        const int x = x0 + lane, xe = lane == 0 ? x0 - 1 : x0 + PX;   // lanes 0, 1: the cells beside the row
        const bool in = row && x < g.nx, ine = row && lane < 2 && xe >= 0 && xe < g.nx;
        own[k] = *at_or(lab, in ? cell_index(g, z, y, x) : 0, in, g_pad_solid);
        edge[k] = *at_or(lab, ine ? cell_index(g, z, y, xe) : 0, ine, g_pad_solid);
    }
#pragma unroll
    for (int k = 0; k < R / 4; ++k) {
        const uint64_t f = __ballot(own[k] == kFluid), e = __ballot(edge[k] == kFluid);
        if (lane == 0) {
            own_s[wv + 4 * k] = f;
            edge_s[wv + 4 * k] = (uint32_t)e;
        }
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    // thread (i, q, w): plane i, row q, wave w (threads past CH planes idle)
    const int w = threadIdx.x & 3, q = (threadIdx.x >> 2) & 3, i = threadIdx.x >> 4;
    uint32_t md = kGZero, mu = kGZero;
    if (i < CH && z0 + i < g.nz) {   // a row outside the grid is zero
        uint64_t any = 0u, all = ~(uint64_t)0;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const uint64_t f = own_s[(i + a) * PHY + q + b];
                const uint32_t e = edge_s[(i + a) * PHY + q + b];
                const uint64_t lo = (f << 1) | (e & 1u), hi = (f >> 1) | ((uint64_t)(e >> 1) << 63);
                any |= f | lo | hi;
                all &= f & lo & hi;
            }
        const uint64_t own_f = own_s[(i + 1) * PHY + q + 1];
        const int left = g.nx - x0;   // columns of the footprint inside the grid
        const uint64_t valid = y0 + q >= g.ny ? 0u : left >= 64 ? ~(uint64_t)0 : (((uint64_t)1 << left) - 1u);
        auto mode = [&](uint64_t need) -> uint32_t {   // need: the cells that matter
            need &= valid;
            if (((need >> (16 * w)) & 0xffffu) == 0) return kGZero;
            return (((need & ~all) >> (16 * w)) & 0xffffu) ? kGGeneral : kGPure;
        };
        md = mode(any);
        mu = mode(own_f);
        const int nwx = wave_columns(g), wx = 4 * cx + w;
        if (wx < nwx) {   // the others hold no cell
            const size_t at = (((size_t)(z0 + i) * cl.ncy + cy) * nwx + wx) * 4 + q;
            mdown[at] = (uint8_t)md;
            mup[at] = (uint8_t)mu;
        }
    }
    const uint64_t nd = __ballot(md != kGZero), nu = __ballot(mu != kGZero);
    if (threadIdx.x == 0) {
        zdown[blockIdx.x] = nd == 0u;
        zup[blockIdx.x] = nu == 0u;
    }
}

// Group modes of a coarser level: pure when all windows of a wave's four whole
// groups in a plane are pure cells of one label, general otherwise (zero only
// where the row lies outside the grid; no output is masked there).  Four groups at
// once, as every precision has it: in the mixed modes the constant kernel is the
// float one and the others are rounded, so the choice is part of the results.
template <int CH>
__global__ __launch_bounds__(kBlock) void k_coarse_modes(const uint32_t* __restrict__ cnt, Grid g, uint32_t full,
                                                         uint8_t* __restrict__ mode) {
    constexpr int R = (CH + 2) * PHY;
    __shared__ uint64_t own_s[R][3];   // a row's pure cells of each label
    __shared__ uint32_t edge_s[R][3];  // and the cells beside it (bits 0, 1)
    const Columns cl = march_columns(g);
    const int per = cl.ncx * cl.ncy, rest = (int)blockIdx.x % per, zc = (int)blockIdx.x / per;
    const int cx = rest % cl.ncx, cy = rest / cl.ncx, x0 = cx * PX, y0 = cy * PY, z0 = zc * CH;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t own[R / 4], edge[R / 4];
#pragma unroll
    for (int k = 0; k < R / 4; ++k) {
        const int r = wv + 4 * k, z = z0 + r / PHY - 1, y = y0 + r % PHY - 1;
        const bool row = z >= 0 && z < g.nz && y >= 0 && y < g.ny;
        const int x = x0 + lane, xe = lane == 0 ? x0 - 1 : x0 + PX;
        const bool in = row && x < g.nx, ine = row && lane < 2 && xe >= 0 && xe < g.nx;
        own[k] = *at_or(cnt, in ? cell_index(g, z, y, x) : 0, in, pad_zero<uint32_t>());
        edge[k] = *at_or(cnt, ine ? cell_index(g, z, y, xe) : 0, ine, pad_zero<uint32_t>());
    }
    const uint32_t pure[3] = {full, full << 16, 0u};   // packed counts of a pure cell
#pragma unroll
    for (int k = 0; k < R / 4; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const uint64_t f = __ballot(own[k] == pure[c]), e = __ballot(edge[k] == pure[c]);
            if (lane == 0) {
                own_s[wv + 4 * k][c] = f;
                edge_s[wv + 4 * k][c] = (uint32_t)e;
            }
        }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const int w = threadIdx.x & 3, q = (threadIdx.x >> 2) & 3, i = threadIdx.x >> 4;   // thread (i, q, w)
    const bool on = i < CH && z0 + i < g.nz;
    const int left = g.nx - x0;
    uint64_t valid = left >= 64 ? ~(uint64_t)0 : (((uint64_t)1 << left) - 1u);
    if (!on || y0 + q >= g.ny) valid = 0u;
    const uint32_t need = (uint32_t)(valid >> (16 * w)) & 0xffffu;
    int m = need ? (int)kGGeneral : (int)kGZero;
    if (on) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            uint64_t all = ~(uint64_t)0;
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    const uint64_t f = own_s[(i + a) * PHY + q + b][c];
                    const uint32_t e = edge_s[(i + a) * PHY + q + b][c];
                    all &= f & ((f << 1) | (e & 1u)) & ((f >> 1) | ((uint64_t)(e >> 1) << 63));
                }
            if (((uint32_t)(all >> (16 * w)) & need) == 0xffffu)
                m = c == 0 ? kGPure : c == 1 ? kGPureAir : kGPureSolid;
        }
    }
    // the wave's four rows: one kernel for all 64 cells, or the matrix cores
    // (all three exchanges before any test: every lane takes part in each)
    const int m1 = __shfl_xor(m, 4, 64), m2 = __shfl_xor(m, 8, 64), m3 = __shfl_xor(m, 12, 64);
    if (need && (m != m1 || m != m2 || m != m3)) m = kGGeneral;
    const int nwx = wave_columns(g), wx = 4 * cx + w;
    if (on && wx < nwx) mode[(((size_t)(z0 + i) * cl.ncy + cy) * nwx + wx) * 4 + q] = (uint8_t)m;
}

// The staged item: (CH + 2) planes of PHY rows of kRS records.  The cell at x
// offset ix (-1 .. 64) from the footprint is record ix + XO of its row: XO = 2
// for the down kernel, whose staging writes four cells from ix = 4k at once,
// 1 for the up kernel, whose staging writes the pair (2j - 1, 2j).
constexpr int kRS = 68;
template <int CH>
constexpr int kRecords = (CH + 2) * PHY * kRS;

// A wave's MFMA operands for all its groups.
template <int KM>
struct MarchCtx {
    static constexpr int P = KM == kMfmaBf16x3 ? kPieces : 1;
    u16x8 a[P][2][2];
    int lofs[8];    // record of window position j of output plane 0, row 0
    bool one;       // lane group 2: position 27 carries the constant feature
};

template <int KM, int XO>
__device__ __forceinline__ MarchCtx<KM> march_ctx(const MfmaW* __restrict__ wm) {
    MarchCtx<KM> c;
    const int lane = threadIdx.x & 63, g = lane >> 4, n = lane & 15, wv = threadIdx.x >> 6;
#pragma unroll
    for (int p = 0; p < MarchCtx<KM>::P; ++p)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const uint16_t* src = KM == kMfmaF16 ? &wm->f16[mb][ks][lane][0] : &wm->bf16[p][mb][ks][lane][0];
                c.a[p][mb][ks] = *reinterpret_cast<const u16x8*>(src);
            }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int o = min(16 * (j >> 2) + 4 * g + (j & 3), kTaps - 1);
        c.lofs[j] = (o / 9 * PHY + o / 3 % 3) * kRS + 16 * wv + n + XO + o % 3 - 1;
        // one register per position (the compiler re-formed the sums for every group)
        __asm__ volatile("" : "+v"(c.lofs[j]));
    }
    c.one = g == 2;
    return c;
}

__device__ __forceinline__ uint32_t bits(float v) { return __float_as_uint(v); }
__device__ __forceinline__ float fbits(uint32_t v) { return __uint_as_float(v); }

// The partial CConv sum of the lane for a general group (at: the group's
// record offset, a constant): sum over its eight window positions of
// K_t(cell) r(cell + t).
template <int KM>
__device__ __forceinline__ float march_group(const uint2* rec, int at, const MarchCtx<KM>& c) {
    uint2 rv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) rv[j] = rec[c.lofs[j] + at];
    float pa = 0.0f, pb2 = 0.0f;   // two chains of four
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u16x8 B[2];
    B[0] = __builtin_bit_cast(u16x8, (u32x4){rv[0].y, rv[1].y, rv[2].y, rv[3].y});
    B[1] = __builtin_bit_cast(u16x8, (u32x4){rv[4].y, rv[5].y, rv[6].y, c.one ? feat_one<KM>() : rv[7].y});
    f32x4 acc[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        acc[mb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int p = 0; p < MarchCtx<KM>::P; ++p)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                if (KM == kMfmaF16)
                    acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, c.a[p][mb][ks]),
                                                                     __builtin_bit_cast(f16x8, B[ks]), acc[mb], 0, 0, 0);
                else
                    acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, c.a[p][mb][ks]),
                                                                      __builtin_bit_cast(bf16x8, B[ks]), acc[mb], 0, 0, 0);
            }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        pa = fmaf(acc[0][j], fbits(rv[j].x), pa);
        pb2 = fmaf(acc[1][j], fbits(rv[j + 4].x), pb2);
    }
    return pa + pb2;
}

// Sum of a value over the lane pairs (l, l ^ 32) and (l, l ^ 16), given per
// lane for four groups: returns for lane (g, n) the total over the four lane
// groups of group g's value at n.  v_permlane32_swap exchanges the upper half
// of its first operand with the lower half of its second, v_permlane16_swap
// the odd 16-lane rows of the first with the even rows of the second.
__device__ __forceinline__ float reduce_scatter4(const float (&p)[4]) {
    const auto s0 = __builtin_amdgcn_permlane32_swap(bits(p[0]), bits(p[2]), false, false);
    const auto s1 = __builtin_amdgcn_permlane32_swap(bits(p[1]), bits(p[3]), false, false);
    const float a0 = fbits(s0[0]) + fbits(s0[1]);   // lanes < 32: group 0, else group 2
    const float a1 = fbits(s1[0]) + fbits(s1[1]);   // lanes < 32: group 1, else group 3
    const auto t = __builtin_amdgcn_permlane16_swap(bits(a0), bits(a1), false, false);
    return fbits(t[0]) + fbits(t[1]);
}

// The CConv of the lane's cell in every plane of the item.  modes[i]: the
// wave's four group modes in plane i (one byte each, uniform).
template <int KM, int XO, int CH, bool L1>
__device__ __forceinline__ void march_cconv(const uint2* rec, const uint32_t (&modes)[CH], const MarchCtx<KM>& mc,
                                            const CConvW<float>* __restrict__ w, float (&out)[CH]) {
    const int lane = threadIdx.x & 63, gq = lane >> 4;
    uint32_t any = 0u;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        out[i] = 0.0f;
        any |= modes[i];
    }
    // the constant kernels of the wave's pure groups (level 1: fluid only)
#pragma unroll 1
    for (int c = 0; c < (L1 ? 1 : 3); ++c) {
        const uint32_t bit = c == 0 ? kGPure : c == 1 ? kGPureAir : kGPureSolid;
        if (!(any & (0x01010101u * bit))) continue;
        // in scalar registers, loaded per item: kept across the item loop, the 27 of them spilled
        const float* kc = w->Kpure[c];
        __asm__ volatile("" : "+s"(kc));
        float kp[kTaps], acc[CH];
#pragma unroll
        for (int t = 0; t < kTaps; ++t) kp[t] = kc[t];
#pragma unroll
        for (int i = 0; i < CH; ++i) acc[i] = 0.0f;
        const uint2* corner = rec + gq * kRS + 16 * (int)(threadIdx.x >> 6) + (lane & 15) + XO - 1;
#pragma unroll
        for (int k = 0; k < CH + 2; ++k) {
            float s[3][2];   // the plane is at z offset a - 1 from output plane k - a; short sums round less
#pragma unroll
            for (int d = 0; d < 9; ++d) {
                const float v = fbits(corner[(k * PHY + d / 3) * kRS + d % 3].x);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    float& t = s[a][d >= 5];
                    t = d == 0 || d == 5 ? kp[9 * a + d] * v : fmaf(kp[9 * a + d], v, t);
                }
            }
#pragma unroll
            for (int a = 0; a < 3; ++a)
                if (k - a >= 0 && k - a < CH) acc[k - a] += s[a][0] + s[a][1];
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) out[i] = L1 || ((modes[i] >> (8 * gq)) & bit) ? acc[i] : out[i];
    }
    if (any & kAnyGeneral) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const uint32_t m = modes[i];
            if (!(m & kAnyGeneral)) continue;
            float part[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                part[q] = ((m >> (8 * q)) & kGGeneral) ? march_group<KM>(rec, (i * PHY + q) * kRS, mc) : 0.0f;
            const float red = reduce_scatter4(part);
            out[i] = ((m >> (8 * gq)) & kGGeneral) ? red : out[i];
        }
    }
}

// The wave's modes of the item's planes (zero past the grid).
template <int CH>
__device__ __forceinline__ void load_modes(const uint32_t* __restrict__ gmode, Columns cl, const MarchItem& it, Grid g,
                                           uint32_t (&modes)[CH]) {
    const int wx = 4 * it.cx + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwx = wave_columns(g);
    const int nz = wx < nwx ? g.nz : 0;   // a wave past the columns has no plane
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int z = it.zc * CH + i;
        modes[i] = z < nz ? __builtin_amdgcn_readfirstlane(gmode[((size_t)z * cl.ncy + it.cy) * nwx + wx]) : 0u;
    }
}

// The thread index as a value of its own in every item: what staging derives
// from it is then formed per item instead of staying in registers (30 of them,
// which spilled) across the item loop, of which a block runs one or two rounds.
__device__ __forceinline__ int item_thread() {
    int t = (int)threadIdx.x;
    __asm__ volatile("" : "+v"(t));
    return t;
}

// Staging tasks of an item's rows: quads of four cells (a float4 and a word of
// labels where the rows are aligned), then the two cells beside every row.
// Whole waves hold one kind (kQuads is a multiple of 64), so the kind of a
// wave's round k is uniform.
template <int CH>
struct StageTasks {
    static constexpr int kRows = (CH + 2) * PHY;
    static constexpr int kQuads = kRows * (PX / 4), kAll = kQuads + 2 * kRows;
    static constexpr int K = (kAll + kBlock - 1) / kBlock;
    static_assert(kQuads % 64 == 0, "uniform kind of a wave's round");
    __device__ static __forceinline__ bool quads(int wv, int k) {
        return (k + 1) * kBlock <= kQuads || 64 * wv + k * kBlock < kQuads;
    }
    __device__ static __forceinline__ bool edges(int wv, int k) {
        return !quads(wv, k) && 64 * wv + k * kBlock < kAll;
    }
};

struct StagePos {
    int rec;              // first record of the task
    uint32_t base;        // cell index of the first cell
    int cells;            // cells inside the grid (quads 0 .. 4, edges 0 or 1)
};

template <int CH, int XO, bool QUAD>
__device__ __forceinline__ StagePos stage_pos(Grid g, int x0, int y0, int z0, int t) {
    using S = StageTasks<CH>;
    const int e = min(t, S::kAll - 1) - S::kQuads;
    const int row = QUAD ? t / (PX / 4) : e >> 1, ix = QUAD ? 4 * (t % (PX / 4)) : (e & 1) ? PX : -1;
    const int z = z0 + row / PHY - 1, y = y0 + row % PHY - 1, x = x0 + ix;
    const bool in = z >= 0 && z < g.nz && y >= 0 && y < g.ny && x >= 0 && x < g.nx;
    return StagePos{row * kRS + ix + XO, in ? (uint32_t)cell_index(g, z, y, x) : 0u,
                    in ? (QUAD ? min(4, g.nx - x) : 1) : 0};
}

// The labels of a task, one byte each (solid outside the grid).  wide: rows of
// four labels are aligned words, and nx is a multiple of 4.
template <bool QUAD>
__device__ __forceinline__ uint32_t stage_labels(const uint8_t* __restrict__ lab, const StagePos& s, int wide) {
    if constexpr (!QUAD) return *at_or(lab, s.base, s.cells > 0, g_pad_solid);
    if (wide) return *reinterpret_cast<const uint32_t*>(at_or(lab, s.base, s.cells > 0, g_pad_solid));
    uint32_t v = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) v |= (uint32_t)*at_or(lab, s.base + j, j < s.cells, g_pad_solid) << (8 * j);
    return v;
}

template <bool QUAD>
__device__ __forceinline__ float4 stage_values(const float* __restrict__ r, const StagePos& s, int wide) {
    if constexpr (!QUAD) return float4{*at_or(r, s.base, s.cells > 0, pad_zero<float>()), 0.0f, 0.0f, 0.0f};
    if (wide) return *reinterpret_cast<const float4*>(at_or(r, s.base, s.cells > 0, pad_zero<float>()));
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = *at_or(r, s.base + j, j < s.cells, pad_zero<float>());
    return float4{v[0], v[1], v[2], v[3]};
}

// The image of a staging task: four labels in a word (level 1), or four counts.
template <bool L1>
struct ImgQuad {
    uint32_t v[L1 ? 1 : 4];
    __device__ __forceinline__ uint32_t cell(int j) const {
        if constexpr (L1) return (v[0] >> (8 * j)) & 255u;
        else return v[j];
    }
};

template <bool L1, bool QUAD>
__device__ __forceinline__ ImgQuad<L1> stage_image_quad(const void* __restrict__ img, const StagePos& s, int wide) {
    ImgQuad<L1> q{};
    if constexpr (L1) {
        q.v[0] = stage_labels<QUAD>(static_cast<const uint8_t*>(img), s, wide);
    } else {
        const uint32_t* cnt = static_cast<const uint32_t*>(img);
        if constexpr (!QUAD) {
            q.v[0] = *at_or(cnt, s.base, s.cells > 0, pad_zero<uint32_t>());
        } else if (wide) {
            const uint4 u = *reinterpret_cast<const uint4*>(at_or(cnt, s.base, s.cells > 0, pad_zero<uint32_t>()));
            q.v[0] = u.x;
            q.v[1] = u.y;
            q.v[2] = u.z;
            q.v[3] = u.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) q.v[j] = *at_or(cnt, s.base + j, j < s.cells, pad_zero<uint32_t>());
        }
    }
    return q;
}

// Waves per SIMD of the level-1 kernels: one more hides more of the staging's
// latency (network evaluations in bf16 on scenes of spheres under a flat surface,
// 128^3: up 21.1 -> 18.8 us, down 16.1 -> 14.8 us; 256^3: up 98 -> 86 us, down 78 -> 67
// us), yet another one spills (up 26.0 us).  The
// three-piece weights of FP32 and the operands of more than two dots take
// registers of one wave each.
constexpr int march_waves(int km, int nd) { return 5 - (km == kMfmaBf16x3 ? 1 : 0) - (nd > 2 ? 1 : 0); }

// x1 = CConv_1(r) and, below the coarsest level (rnext), r_next = Pool(x1); at
// level 1 (L1) the input is masked to fluid and izero names the items that only
// write zeros.  Levels 2 and 3 ran tile kernels with a full 3-D halo before (16 x
// 4 x 4 cells a block; 128^3 level of a 256^3 grid: 32 us down, 40 us up).  The 2x2x2
// pool sums x pairs with a DPP quad permutation, y pairs with a permlane swap
// and z pairs in a register (items start on even planes).
template <int KM, int CH, bool L1>
__global__ __launch_bounds__(kBlock) NPS_WAVES_PER_EU(march_waves(KM, 0)) void k_down_m(
    const void* __restrict__ img, Grid g, const float* __restrict__ r, float* __restrict__ x1,
    float* __restrict__ rnext, const CConvW<float>* __restrict__ w, const MfmaW* __restrict__ wm, const State* st,
    const uint32_t* __restrict__ gmode, const uint8_t* __restrict__ izero, int flags) {
    const int wide = flags & kWideRows;
    constexpr int XO = 2;
    using S = StageTasks<CH>;
    __shared__ __attribute__((aligned(16))) uint2 rec[kRecords<CH>];
    const int done = st->done;   // tested once the first loads are out
    const MarchCtx<KM> mc = march_ctx<KM, XO>(wm);
    const Columns cl = march_columns(g);
    const Grid gc = coarser(g);
    const int lane = threadIdx.x & 63, gq = lane >> 4, n = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t pstride = (uint32_t)g.ny * (uint32_t)g.nx;
    const MarchItems mi = march_items(cl, (int)gridDim.x, (int)blockIdx.x, flags & kSlabs);
    bool first = true;
    for (int li = mi.li; li < mi.count; li += mi.step) {
        const MarchItem it = march_item(mi, li, cl);
        const int x0 = it.cx * PX, y0 = it.cy * PY, z0 = it.zc * CH;
        const int xx = x0 + 16 * wv + n, yy = y0 + gq;
        const bool col = xx < g.nx && yy < g.ny;
        if (L1 && izero[it.zc * mi.per + it.rest]) {   // no window holds fluid: x1 is zero (read nowhere), and so is the pool
            if (done) return;
#pragma unroll
            for (int i = 1; i < CH; i += 2)
                if (((n | gq) & 1) == 0 && col && z0 + i < g.nz)
                    rnext[cell_index(gc, (z0 + i) >> 1, yy >> 1, xx >> 1)] = 0.0f;
            continue;
        }
        const int tid = item_thread();
        uint32_t modes[CH];
        load_modes<CH>(gmode, cl, it, g, modes);
        ImgQuad<L1> lw[S::K];
        float4 rw[S::K];
#pragma unroll
        for (int k = 0; k < S::K; ++k) {
            if (S::quads(wv, k)) {
                const StagePos s = stage_pos<CH, XO, true>(g, x0, y0, z0, tid + k * kBlock);
                rw[k] = stage_values<true>(r, s, wide);
                lw[k] = stage_image_quad<L1, true>(img, s, wide);
            } else if (S::edges(wv, k)) {
                const StagePos s = stage_pos<CH, XO, false>(g, x0, y0, z0, tid + k * kBlock);
                rw[k] = stage_values<false>(r, s, wide);
                lw[k] = stage_image_quad<L1, false>(img, s, wide);
            }
        }
        if (first) {
            __asm__ volatile("" ::: "memory");   // the loads stay above the test
            if (done) return;
            first = false;
        } else {
            __syncthreads();   // the previous item's reads of the records are done
        }
#pragma unroll
        for (int k = 0; k < S::K; ++k) {
            const float v[4] = {rw[k].x, rw[k].y, rw[k].z, rw[k].w};
            auto record = [&](int j) {
                const uint32_t l = lw[k].cell(j);
                return uint2{bits(!L1 || l == kFluid ? v[j] : 0.0f), feat_word<KM, L1>(l)};
            };
            if (S::quads(wv, k)) {
                const uint2 e0 = record(0), e1 = record(1), e2 = record(2), e3 = record(3);
                uint4* dst = reinterpret_cast<uint4*>(rec + stage_pos<CH, XO, true>(g, x0, y0, z0, tid + k * kBlock).rec);
                dst[0] = uint4{e0.x, e0.y, e1.x, e1.y};
                dst[1] = uint4{e2.x, e2.y, e3.x, e3.y};
            } else if (S::edges(wv, k)) {   // lanes past the last task repeat it
                rec[stage_pos<CH, XO, false>(g, x0, y0, z0, tid + k * kBlock).rec] = record(0);
            }
        }
        __syncthreads();   // the item is staged
        float out[CH];
        march_cconv<KM, XO, CH, L1>(rec, modes, mc, w, out);
        const uint32_t own = col ? (uint32_t)z0 * pstride + (uint32_t)yy * g.nx + xx : 0u;
        float pool = 0.0f;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const bool zin = z0 + i < g.nz;
            if (col && zin) x1[(size_t)own + (size_t)i * pstride] = out[i];
            // 2x2x2 pool: x pair (DPP quad_perm [1,0,3,2]), y pair (rows 2k, 2k+1)
            auto right = [](float v) {
                return fbits(__builtin_amdgcn_update_dpp(0u, bits(v), 0xB1, 0xF, 0xF, false));
            };
            if constexpr (L1) {
                const float px = out[i] + right(out[i]);
                const auto t = __builtin_amdgcn_permlane16_swap(bits(px), bits(px), false, false);
                pool += fbits(t[0]) + fbits(t[1]);
            } else {   // in the order of the other levels' pool: x, then y, then z (valid on the storing lanes)
                const auto t = __builtin_amdgcn_permlane16_swap(bits(out[i]), bits(out[i]), false, false);
                const float below = fbits(t[1]);
                pool = (((pool + out[i]) + right(out[i])) + below) + right(below);
            }
            if (i & 1) {
                if (((n | gq) & 1) == 0 && col && zin && rnext)
                    rnext[cell_index(gc, (z0 + i) >> 1, yy >> 1, xx >> 1)] = pool * 0.125f;
                pool = 0.0f;
            }
        }
    }
}

// Level-1 up: dhat = (c1 x1 + c2 CConv_2^1(Interp(x^2))) / ||r|| on fluid
// cells (0 elsewhere) and the state's ndots partial dots of dhat with ad0..
// The coarse cells the item interpolates from (coordinates clamped into the
// coarse grid, which is the interpolation's edge rule) are staged first, with
// the labels' features.  The trilinear interpolation (cell-centred, edges
// clamped) then runs per octet: the 2x2x2 coarse cells (j - 1, j) along each
// axis give the 2x2x2 fine cells (2j - 1, 2j), whose weights along an axis are
// (3/4, 1/4) and (1/4, 3/4); shared along x, y and z that is 4.5 operations
// and one LDS read per fine cell (formed cell by cell: 14 and 8).
constexpr int kCX = PX / 2 + 2, kCY = PY / 2 + 2, kCPlane = kCX * kCY;
template <int CH>
constexpr int kCoarseCells = (CH / 2 + 2) * kCPlane;
template <int CH>
constexpr int kOctets = (CH / 2 + 1) * (PY / 2 + 1) * (PX / 2 + 1);

// The pair of fine values between coarse values lo and hi: 3/4 lo + 1/4 hi, 1/4 lo
// + 3/4 hi (rounded as the tile kernels of the other levels do off level 1).
template <bool L1>
__device__ __forceinline__ void interp_pair(float lo, float hi, float& a, float& b) {
    const float d = hi - lo;
    a = fmaf(0.25f, d, lo);
    b = L1 ? fmaf(-0.25f, d, hi) : fmaf(0.75f, d, lo);
}

// ND: the most dots the state can ask for (NPSDO: n_ortho; PCG 1; flexible
// PCG 2; 0 for the hook and the symmetric variant); HOOK: the parity hook and
// training's forward (no scaling, no dots; x2out, when given, receives the
// CConv's output on the live items, for the backward).
// L1 false: a coarser level, x = c1 x1 + c2 CConv_2(Interp(xc)) on all cells
// (written to dhat), lvl the index of its c1, c2.
template <int KM, bool HOOK, int ND, int CH, bool L1>
__global__ __launch_bounds__(kBlock) NPS_WAVES_PER_EU(march_waves(KM, ND)) void k_up_m(
    const void* __restrict__ img, Grid g, const float* __restrict__ xc, const float* __restrict__ x1,
    float* __restrict__ dhat, const CConvW<float>* __restrict__ w, const MfmaW* __restrict__ wm, const State* st,
    double* __restrict__ partials, const float* __restrict__ ad0, const float* __restrict__ ad1,
    const float* __restrict__ ad2, const float* __restrict__ ad3, const uint32_t* __restrict__ gmode,
    const uint8_t* __restrict__ izero, int flags, float* __restrict__ x2out, int lvl) {
    const int wide = flags & kWideRows;
    static_assert((!HOOK || ND == 0) && (L1 || HOOK), "the hook and the coarser levels form no dots");
    constexpr int XO = 1;
    using S = StageTasks<CH>;
    constexpr int KC = (kCoarseCells<CH> + kBlock - 1) / kBlock, KO = (kOctets<CH> + kBlock - 1) / kBlock;
    __shared__ __attribute__((aligned(16))) uint2 rec[kRecords<CH>];
    __shared__ float csh[KC * kBlock];
    const int done = st->done;
    const float c1 = (float)st->c1[L1 ? 0 : lvl], c2 = (float)st->c2[L1 ? 0 : lvl];
    const float scale = HOOK ? 1.0f : (float)st->scale;
    const int ndots = HOOK || st->sym ? 0 : min(st->ndots, ND);   // the symmetric variant dots after P^T
    const MarchCtx<KM> mc = march_ctx<KM, XO>(wm);
    const Columns cl = march_columns(g);
    const Grid gc = coarser(g);
    const int lane = threadIdx.x & 63, gq = lane >> 4, n = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float* adp[kMaxOrtho] = {ad0, ad1, ad2, ad3};
    const uint32_t fluid_word = feat_word<KM, true>(kFluid);
    double v[kRedWidth] = {0.0, 0.0, 0.0, 0.0};
    const uint32_t pstride = (uint32_t)g.ny * (uint32_t)g.nx;
    const MarchItems mi = march_items(cl, (int)gridDim.x, (int)blockIdx.x, flags & kSlabs);
    bool first = true;
    for (int li = mi.li; li < mi.count; li += mi.step) {
        const MarchItem it = march_item(mi, li, cl);
        const int x0 = it.cx * PX, y0 = it.cy * PY, z0 = it.zc * CH;
        const int xx = x0 + 16 * wv + n, yy = y0 + gq;
        const bool col = xx < g.nx && yy < g.ny;
        const uint32_t own = col ? (uint32_t)z0 * pstride + (uint32_t)yy * g.nx + xx : 0u;
        if (L1 && izero[it.zc * mi.per + it.rest]) {   // no fluid cell: the output is zero, the dots get nothing
            if (done) return;
#pragma unroll
            for (int i = 0; i < CH; ++i)
                if (col && z0 + i < g.nz) dhat[(size_t)own + (size_t)i * pstride] = 0.0f;
            continue;
        }
        const int tid = item_thread();
        uint32_t modes[CH];
        load_modes<CH>(gmode, cl, it, g, modes);
        float cw[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const int i = min(tid + k * kBlock, kCoarseCells<CH> - 1);
            const int jz = min(max(z0 / 2 - 1 + i / kCPlane, 0), gc.nz - 1),
                      jy = min(max(y0 / 2 - 1 + i / kCX % kCY, 0), gc.ny - 1),
                      jx = min(max(x0 / 2 - 1 + i % kCX, 0), gc.nx - 1);
            cw[k] = xc[cell_index(gc, jz, jy, jx)];
        }
        ImgQuad<L1> lw[S::K];
#pragma unroll
        for (int k = 0; k < S::K; ++k) {
            if (S::quads(wv, k))
                lw[k] = stage_image_quad<L1, true>(img, stage_pos<CH, XO, true>(g, x0, y0, z0, tid + k * kBlock), wide);
            else if (S::edges(wv, k))
                lw[k] = stage_image_quad<L1, false>(img, stage_pos<CH, XO, false>(g, x0, y0, z0, tid + k * kBlock), wide);
        }
        if (first) {
            __asm__ volatile("" ::: "memory");
            if (done) return;
            first = false;
        } else {
            __syncthreads();   // the previous item's reads of the records are done
        }
#pragma unroll
        for (int k = 0; k < KC; ++k) csh[tid + k * kBlock] = cw[k];
#pragma unroll
        for (int k = 0; k < S::K; ++k) {
            if (S::quads(wv, k)) {
                uint2* dst = rec + stage_pos<CH, XO, true>(g, x0, y0, z0, tid + k * kBlock).rec;
#pragma unroll
                for (int j = 0; j < 4; ++j) dst[j].y = feat_word<KM, L1>(lw[k].cell(j));
            } else if (S::edges(wv, k)) {   // lanes past the last task repeat it
                rec[stage_pos<CH, XO, false>(g, x0, y0, z0, tid + k * kBlock).rec].y = feat_word<KM, L1>(lw[k].cell(0));
            }
        }
        __syncthreads();   // coarse cells and features staged
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            const int o = tid + k * kBlock;
            if (o < kOctets<CH>) {
                constexpr int OX = PX / 2 + 1, OY = PY / 2 + 1;
                const int ox = o % OX, oy = o / OX % OY, oz = o / (OX * OY);
                const float* c = csh + (oz * kCY + oy) * kCX + ox;   // coarse cell (j - 1) of each axis
                float f[2][2][2], fy[2][2][2];
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        interp_pair<L1>(c[(a * kCY + b) * kCX], c[(a * kCY + b) * kCX + 1], f[a][b][0], f[a][b][1]);
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int x = 0; x < 2; ++x) interp_pair<L1>(f[a][0][x], f[a][1][x], fy[a][0][x], fy[a][1][x]);
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int x = 0; x < 2; ++x) interp_pair<L1>(fy[0][b][x], fy[1][b][x], f[0][b][x], f[1][b][x]);
                // the CConv_2 input is zero outside the grid and not masked inside (only the level's output is)
                const int fz = z0 + 2 * oz - 1, fyy = y0 + 2 * oy - 1, fx = x0 + 2 * ox - 1;
                const bool xin[2] = {fx >= 0 && fx < g.nx, fx + 1 < g.nx};
                uint2* dst = rec + (2 * oz * PHY + 2 * oy) * kRS + 2 * ox;
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const bool yz = fz + a >= 0 && fz + a < g.nz && fyy + b >= 0 && fyy + b < g.ny;
#pragma unroll
                        for (int x = 0; x < 2; ++x)
                            dst[(a * PHY + b) * kRS + x].x = bits(yz && xin[x] ? f[a][b][x] : 0.0f);
                    }
            }
        }
        // the lane cell's operands (an unused dot slot reads x1; planes past the grid read the first)
        float x1v[CH], adv[CH][ND > 0 ? ND : 1];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const size_t q = (size_t)own + (z0 + i < g.nz ? (size_t)i * pstride : 0);
            x1v[i] = x1[q];
#pragma unroll
            for (int j = 0; j < ND; ++j) adv[i][j] = (j < ndots ? adp[j] : x1)[q];
        }
        __syncthreads();   // the item is staged
        float x2[CH];
        march_cconv<KM, XO, CH, L1>(rec, modes, mc, w, x2);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const bool fl = !L1 || rec[((i + 1) * PHY + gq + 1) * kRS + 16 * wv + n + XO].y == fluid_word;
            const float out = fl ? (c1 * x1v[i] + c2 * x2[i]) * scale : 0.0f;
            if (col && z0 + i < g.nz) {
                dhat[(size_t)own + (size_t)i * pstride] = out;
                if (HOOK && x2out) x2out[(size_t)own + (size_t)i * pstride] = x2[i];
#pragma unroll
                for (int j = 0; j < ND; ++j)
                    if (j < ndots) v[j] = fma((double)out, (double)adv[i][j], v[j]);
            }
        }
    }
    if (!HOOK && !done) block_partials<kBlock>(v, partials);
}

}  // namespace nps
