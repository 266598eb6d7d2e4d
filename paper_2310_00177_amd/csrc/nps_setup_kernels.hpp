// Per-call set-up kernels: everything of a network evaluation or a solve that
// depends on the labels and the weights only.
//
// Set-up is a chain of short kernels, so what bounds it is how many launches
// the chain has (3-5 us each from the host, and 1-2 us of ramp on the GPU), not
// the few megabytes it reads.  It therefore runs as few, wide kernels:
//   state_init / validate + live_list   the state (a solve also validates its inputs)
//   pyramid     the counts of every level >= 2 and the boundary sums of every level
//   finish      the Aff scalars and the stored kernels of all levels but the largest in double
// One launch per level and block before (26 launches, 100 us of a 154 us
// 32^3 evaluation in FP32).
#pragma once

#include "nps_kernels.hpp"

namespace nps {

// ---------------------------------------------------------------------------
// image pyramid and boundary sums
// ---------------------------------------------------------------------------
// The image-window sums of an Aff block need, per level, the fluid and air
// counts summed over the cells of each boundary class: the class of a cell is
// one bit per face of the grid it touches (a cell of an axis with one cell
// touches both).  Integers, so their order does not matter.
constexpr int kClasses = 64;
constexpr uint32_t kZLo = 1, kZHi = 2, kYLo = 4, kYHi = 8, kXLo = 16, kXHi = 32;

__host__ __device__ inline uint32_t cell_class(Grid g, int z, int y, int x) {
    return (z == 0 ? kZLo : 0u) | (z == g.nz - 1 ? kZHi : 0u) | (y == 0 ? kYLo : 0u) | (y == g.ny - 1 ? kYHi : 0u) |
           (x == 0 ? kXLo : 0u) | (x == g.nx - 1 ? kXHi : 0u);
}

// Sums per level (row l - 1) and class: [level][class][fluid, air].  The class
// of no face is not accumulated: it is the rest of the grid's total.
struct ClassSums {
    uint32_t n[kMaxLevels][kClasses][2];
};

constexpr int kPyrSide = 32;       // cells per side of a block's cube: 2^(kMaxLevels - 1)
constexpr int kPyrThreads = 1024;  // one row of 32 labels per thread

__host__ __device__ inline int pyramid_blocks(Grid g) {
    auto up = [](int n) { return (n + kPyrSide - 1) / kPyrSide; };
    return up(g.nz) * up(g.ny) * up(g.nx);
}

struct PyramidOut {
    uint32_t* cnt[kMaxLevels + 1];   // counts of levels 2 .. L
};

// Counts of every level below a 32^3 cube of labels in one pass: the rows of
// two y and two z neighbours are added across lanes (y in the lane's low bit, z
// in its high bit), the levels from 3 on are summed in LDS.  tot receives the
// block's fluid and air totals.  wide: rows of 16 labels are 16-byte aligned.
// 128^3: 10.5 us (12.5 us with the rows added by lane shuffles through LDS and written
// by a quarter of the lanes).
__global__ __launch_bounds__(kPyrThreads) void k_pyramid(const uint8_t* __restrict__ lab, Grid g, int L, PyramidOut out,
                                                         ClassSums* __restrict__ cls, uint2* __restrict__ tot,
                                                         int wide) {
    constexpr int H = kPyrSide / 2;
    __shared__ uint32_t sum[2][H * H * H];
    __shared__ uint32_t cs[kMaxLevels][kClasses][2];
    const int t = threadIdx.x, cube = block_unit<kPyrThreads>();
    if (cube >= pyramid_blocks(g)) return;
    for (int i = t; i < kMaxLevels * kClasses * 2; i += kPyrThreads) (&cs[0][0][0])[i] = 0u;
    const int bx = (g.nx + kPyrSide - 1) / kPyrSide, by = (g.ny + kPyrSide - 1) / kPyrSide;
    const int x0 = cube % bx * kPyrSide, y0 = cube / bx % by * kPyrSide, z0 = cube / (bx * by) * kPyrSide;
    // a wave holds two z-planes of 32 rows: lane bit 0 = y & 1, lane bit 5 = z & 1
    const int y = y0 + (t & 31), z = z0 + (t >> 5);
    const bool row = y < g.ny && z < g.nz;
    uint32_t w[kPyrSide / 4];
    if (wide) {   // then nx is a multiple of 16: each half of the row is all in the grid or all out
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint4 v = {0x02020202u, 0x02020202u, 0x02020202u, 0x02020202u};
            if (row && x0 + 16 * h < g.nx) v = *reinterpret_cast<const uint4*>(lab + cell_index(g, z, y, x0 + 16 * h));
            w[4 * h] = v.x;
            w[4 * h + 1] = v.y;
            w[4 * h + 2] = v.z;
            w[4 * h + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kPyrSide / 4; ++i) {
            w[i] = 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int x = x0 + 4 * i + k;
                const uint32_t l = row && x < g.nx ? lab[cell_index(g, z, y, x)] : (uint32_t)kSolid;
                w[i] |= l << (8 * k);
            }
        }
    }
    // one packed count (fluid | air << 16) per label, added over the row and in x pairs
    uint32_t pair[H], mid = 0u, lo = 0u, hi = 0u;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        pair[i] = 0u;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int xi = 2 * i + k;
            const uint32_t l = (w[xi >> 2] >> (8 * (xi & 3))) & 255u;
            const uint32_t c = l == kFluid ? 1u : l == kAir ? 0x10000u : 0u;
            pair[i] += c;
            const int x = x0 + xi;
            if (x == 0) lo += c;
            else if (x == g.nx - 1) hi += c;
            else mid += c;
        }
    }
    __syncthreads();   // cs is cleared
    auto add = [&](int l, uint32_t c, uint32_t v) {
        if (v & 0xffffu) atomicAdd(&cs[l - 1][c][0], v & 0xffffu);
        if (v >> 16) atomicAdd(&cs[l - 1][c][1], v >> 16);
    };
    if (row) {
        const uint32_t yz = cell_class(g, z, y, -1);
        if (yz) add(1, yz, mid);
        if (lo) add(1, yz | kXLo | (g.nx == 1 ? kXHi : 0u), lo);
        if (hi) add(1, yz | kXHi, hi);
    }
    // level 2: add the row of y ^ 1 (DPP quad_perm [1,0,3,2]) and the rows of z ^ 1;
    // the four lanes that then hold a row's sums write a quarter of it each
    const Grid g2 = coarser(g);
    const int y2 = (t & 31) >> 1, z2 = t >> 6, sub = (t & 1) | (t >> 4 & 2);
    uint32_t own[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < H; ++i) {
        uint32_t v = pair[i];
        v += (uint32_t)__builtin_amdgcn_update_dpp(0u, v, 0xB1, 0xF, 0xF, false);
        const auto sw = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = sw[0] + sw[1];
        own[i & 3] = (i >> 2) == sub ? v : own[i & 3];
    }
    {
        const int yy = (y0 >> 1) + y2, zz = (z0 >> 1) + z2;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = 4 * sub + j, xx = (x0 >> 1) + i;
            sum[0][(z2 * H + y2) * H + i] = own[j];
            if (in_grid(g2, zz, yy, xx)) {
                out.cnt[2][cell_index(g2, zz, yy, xx)] = own[j];
                const uint32_t c = cell_class(g2, zz, yy, xx);
                if (c) add(2, c, own[j]);
            }
        }
    }
    __syncthreads();
    // levels 3 and on; past level L only the block's total is of interest
    Grid gl = g2;
    int side = H, cur = 0;
    for (int l = 3; side > 1; ++l) {
        const int s2 = side / 2;
        gl = coarser(gl);
        if (t < s2 * s2 * s2) {
            const int cx = t % s2, cy = t / s2 % s2, cz = t / (s2 * s2);
            uint32_t v = 0u;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                v += sum[cur][((2 * cz + (k >> 2)) * side + 2 * cy + ((k >> 1) & 1)) * side + 2 * cx + (k & 1)];
            sum[cur ^ 1][t] = v;
            const int xx = (x0 >> (l - 1)) + cx, yy = (y0 >> (l - 1)) + cy, zz = (z0 >> (l - 1)) + cz;
            if (l <= L && in_grid(gl, zz, yy, xx)) {
                out.cnt[l][cell_index(gl, zz, yy, xx)] = v;
                const uint32_t c = cell_class(gl, zz, yy, xx);
                if (c) add(l, c, v);
            }
        }
        side = s2;
        cur ^= 1;
        __syncthreads();
    }
    if (t == 0) tot[cube] = uint2{sum[cur][0] & 0xffffu, sum[cur][0] >> 16};
    for (int i = t; i < kMaxLevels * kClasses * 2; i += kPyrThreads) {
        const uint32_t v = (&cs[0][0][0])[i];
        if (v) atomicAdd(&(&cls->n[0][0][0])[i], v);
    }
}

// The boundary classes' cells along one axis: class bits 0, lo, hi, lo | hi.
__device__ __forceinline__ int axis_cells(int n, uint32_t bits) {
    if (n == 1) return bits == 3u ? 1 : 0;
    return bits == 0u ? n - 2 : bits == 3u ? 0 : 1;
}

// Cells of class c of a grid.
__device__ __forceinline__ double class_cells(Grid g, uint32_t c) {
    return (double)axis_cells(g.nz, c & 3u) * (double)axis_cells(g.ny, (c >> 2) & 3u) *
           (double)axis_cells(g.nx, (c >> 4) & 3u);
}

// Whether q - o lies in the grid for a cell q of class c.
__device__ __forceinline__ bool class_sees(uint32_t c, int o) {
    const int oz = o / 9 - 1, oy = (o / 3) % 3 - 1, ox = o % 3 - 1;
    const bool out = (oz > 0 && (c & kZLo)) || (oz < 0 && (c & kZHi)) || (oy > 0 && (c & kYLo)) ||
                     (oy < 0 && (c & kYHi)) || (ox > 0 && (c & kXLo)) || (ox < 0 && (c & kXHi));
    return !out;
}

// ---------------------------------------------------------------------------
// Aff scalars and stored kernels
// ---------------------------------------------------------------------------
// K[t][cell] of one CConv block on one level (see k_setup_finish).
enum KgenKind : int { kGenTap = 0, kGenTap9 = 1, kGenMfma = 2 };

struct KgenSeg {
    const void* img;           // labels (level 1) or counts
    Grid g;
    const CConvW<double>* w;
    const MfmaW* wm;
    void* out;
    int kind, l1, blocks;      // blocks of this segment
};

constexpr int kMaxSegs = 2 * kMaxLevels;

struct FinishArgs {
    Grid g;                    // level 1
    int L, pyr;                // levels, pyramid blocks
    const ClassSums* cls;
    const uint2* tot;
    const AffW* aff;           // [level][Aff_1, Aff_2]
    double aff_b[2 * kMaxLevels];
    State* st;
    int nseg;
    KgenSeg seg[kMaxSegs];
};

// The image-window sums of Aff_1^l and Aff_2^l (global means), one block per
// level, one wave per sum, one lane per boundary class: S = sum_p sum_o sum_c
// w[c][o] i_c(p + o), the image solid outside the grid.  With q = p + o the
// in-grid part is sum over classes of (class sum of i_c) times W_c(class) = sum
// of w[c][o] over the o with q - o in the grid; the out-of-grid part is sum_o
// w[solid][o] (n - #{p : p + o in the grid}).  The weights go through LDS: read
// one by one from memory by a single block for all levels, their latencies were
// the length of the whole kernel (22 us).
__device__ __forceinline__ void aff_scalars(const FinishArgs& a, int s) {
    __shared__ double tsh[2][kBlock / 64], w_s[2][3 * kTaps];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const Grid g{a.g.nz >> s, a.g.ny >> s, a.g.nx >> s};
    const uint32_t c = (uint32_t)lane;
    const uint32_t k0 = c ? a.cls->n[s][c][0] : 0u, k1 = c ? a.cls->n[s][c][1] : 0u;
    if (threadIdx.x < 2 * 3 * kTaps) {
        const int k = (int)threadIdx.x / (3 * kTaps), e = (int)threadIdx.x % (3 * kTaps);
        w_s[k][e] = (&a.aff[2 * s + k].w[0][0])[e];
    }
    double tf = 0.0, ta = 0.0;   // fluid and air cells of the grid (exact integers)
    for (int b0 = 0; b0 < a.pyr; b0 += 4 * kBlock) {
        uint2 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = b0 + u * kBlock + (int)threadIdx.x;
            t[u] = b < a.pyr ? a.tot[b] : uint2{0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            tf += (double)t[u].x;
            ta += (double)t[u].y;
        }
    }
    tf = wave_sum(tf);
    ta = wave_sum(ta);
    if (lane == 0) {
        tsh[0][wv] = tf;
        tsh[1][wv] = ta;
    }
    __syncthreads();
    if (wv >= 2) return;
    tf = ta = 0.0;
#pragma unroll
    for (int i = 0; i < kBlock / 64; ++i) {
        tf += tsh[0][i];
        ta += tsh[1][i];
    }
    const double full = (double)(1u << (3 * s)), n = (double)ncells(g);
    double n0 = (double)k0, n1 = (double)k1;
    const double b0 = wave_sum(n0), b1 = wave_sum(n1);
    if (c == 0) {
        n0 = tf - b0;
        n1 = ta - b1;
    }
    const double inv = 1.0 / full, i0 = n0 * inv, i1 = n1 * inv, i2 = (class_cells(g, c) * full - n0 - n1) * inv;
    const double* w = w_s[wv];
    double W0 = 0.0, W1 = 0.0, W2 = 0.0;
#pragma unroll 9
    for (int o = 0; o < kTaps; ++o) {
        const bool in = class_sees(c, o);
        W0 += in ? w[o] : 0.0;
        W1 += in ? w[kTaps + o] : 0.0;
        W2 += in ? w[2 * kTaps + o] : 0.0;
    }
    double v = i0 * W0 + i1 * W1 + i2 * W2;
    if (lane < kTaps) {   // the solid padding, one offset per lane
        const int o = lane;
        const double in = (double)max(g.nz - abs(o / 9 - 1), 0) * (double)max(g.ny - abs((o / 3) % 3 - 1), 0) *
                          (double)max(g.nx - abs(o % 3 - 1), 0);
        v += w[2 * kTaps + o] * (n - in);
    }
    const double S = wave_sum(v);
    if (lane == 0) (wv == 0 ? a.st->c1 : a.st->c2)[s] = a.aff_b[2 * s + wv] + S / (27.0 * n);
}

// Taps t0 .. t0 + TG of the cells of block b of a segment, in double: a thread
// reads the 27 window cells of its cell once for the TG taps.  TG = 1 spreads a
// level of few cells over 27 times as many threads.  The block's weights go
// through LDS (w_s): as scalar loads, 500 doubles of them for TG = 9, each
// waited for in turn (40 x 56 x 72 in FP64: 38 us).
constexpr int kGenTaps = 9;

template <class T, bool L1, int TG>
__device__ __forceinline__ void kgen_taps(const KgenSeg& sg, int b, double2* w_s) {
    static_assert(kTaps % TG == 0 && TG <= kGenTaps, "whole tap groups");
    const Grid g = sg.g;
    const int n = (int)ncells(g), nb = (n + kBlock - 1) / kBlock;
    const int t0 = (b / nb) * TG, p = min((b % nb) * kBlock + (int)threadIdx.x, n - 1);
    const CConvW<double>* __restrict__ w = sg.w;
    const int x = p % g.nx, y = p / g.nx % g.ny, z = p / (g.nx * g.ny);
    uint32_t v[kTaps];
#pragma unroll
    for (int o = 0; o < kTaps; ++o) {   // outside the grid: solid (no counts)
        const int qz = z + o / 9 - 1, qy = y + (o / 3) % 3 - 1, qx = x + o % 3 - 1;
        const bool in = in_grid(g, qz, qy, qx);
        const size_t q = in ? cell_index(g, qz, qy, qx) : 0;
        if (L1) v[o] = *at_or(static_cast<const uint8_t*>(sg.img), q, in, g_pad_solid);
        else v[o] = *at_or(static_cast<const uint32_t*>(sg.img), q, in, pad_zero<uint32_t>());
    }
    for (int i = threadIdx.x; i < kTaps * TG; i += kBlock) {
        const int o = i / TG, u = i % TG;
        w_s[i] = double2{w->D[o][t0 + u][0], w->D[o][t0 + u][1]};
    }
    double K[TG];
#pragma unroll
    for (int u = 0; u < TG; ++u) K[u] = w->C[t0 + u];
    __syncthreads();
#pragma unroll
    for (int o = 0; o < kTaps; ++o) {
        uint32_t c0, c1;
        counts_of<L1>(v[o], c0, c1);
        const double n0 = (double)c0, n1 = (double)c1;
#pragma unroll
        for (int u = 0; u < TG; ++u) {
            const double2 d = w_s[o * TG + u];
            K[u] = fma(d.x, n0, fma(d.y, n1, K[u]));
        }
    }
    T* out = static_cast<T*>(sg.out);
    if ((b % nb) * kBlock + (int)threadIdx.x < n) {
#pragma unroll
        for (int u = 0; u < TG; ++u) out[(size_t)(t0 + u) * n + p] = (T)K[u];
    }
}

// Blocks 0 .. L - 2: the Aff scalars of a level.  The others: the stored kernels,
// segment by segment, so that all of them overlap.  KM: the matrix-core form of
// the float segments of kind kGenMfma.
template <class T, int KM>
__global__ __launch_bounds__(kBlock) NPS_WAVES_PER_EU(4) void k_setup_finish(FinishArgs a) {
    int b = (int)blockIdx.x - (a.L - 1);
    if (b < 0) {
        aff_scalars(a, (int)blockIdx.x);
        return;
    }
    __shared__ double2 w_s[kTaps * kGenTaps];
    int i = 0;
    while (i < a.nseg - 1 && b >= a.seg[i].blocks) b -= a.seg[i++].blocks;
    const KgenSeg sg = a.seg[i];
    if (sg.kind == kGenMfma) {
        if constexpr (sizeof(T) == 4) {
            if (sg.l1) kgen_mfma<KM, true>(sg.img, sg.g, sg.wm, static_cast<float*>(sg.out), b, sg.blocks);
            else kgen_mfma<KM, false>(sg.img, sg.g, sg.wm, static_cast<float*>(sg.out), b, sg.blocks);
        }
    } else if (sg.kind == kGenTap9) {
        if (sg.l1) kgen_taps<T, true, kGenTaps>(sg, b, w_s);
        else kgen_taps<T, false, kGenTaps>(sg, b, w_s);
    } else {
        if (sg.l1) kgen_taps<T, true, 1>(sg, b, w_s);
        else kgen_taps<T, false, 1>(sg, b, w_s);
    }
}

// ---------------------------------------------------------------------------
// state, validation and the live items of a solve
// ---------------------------------------------------------------------------
__device__ __forceinline__ void clear_classes(ClassSums* cls) {
    for (int i = threadIdx.x; i < kMaxLevels * kClasses * 2; i += (int)blockDim.x) (&cls->n[0][0][0])[i] = 0u;
}

// The state of a network evaluation on its own (one block).
__global__ __launch_bounds__(kBlock) void k_state_init(State* st, ClassSums* cls) {
    clear_classes(cls);
    if (threadIdx.x == 0) {
        State s = {};
        s.scale = 1.0;
        *st = s;
    }
}

// Buffers zeroed on the 7-point items without fluid (4 or 8 B elements).
struct ZeroBufs {
    void* p[2 * kRing + 3];
    int bytes[2 * kRing + 3];
    int n;
};

// One pass over the items of the 7-point kernels (columns_of order; a thread
// per column): validates labels and b, sums ||b||^2 and the fluid cells, sets
// x0 = 0, flags the items that hold fluid, and zeroes the cells of the others
// in every buffer of zb: on such an item r = 0 and A d = 0, and it adds nothing
// to any dot, so the 7-point kernels need not visit it.
template <class X>
__global__ __launch_bounds__(kBlock) void k_validate(const uint8_t* __restrict__ lab, Grid g,
                                                     const double* __restrict__ b, X* __restrict__ x0,
                                                     uint8_t* __restrict__ live, ZeroBufs zb, double* partials) {
    constexpr int kMaxChunk = 8;
    const Columns cl = columns_of(g);   // chunk <= kMaxChunk
    double v[kRedWidth] = {0.0, 0.0, 0.0, 0.0};   // bb, n_fluid, bad labels, non-finite
    for (int w = blockIdx.x; w < cl.count(); w += gridDim.x) {
        const int xx = (w % cl.ncx) * PX + (int)threadIdx.x % PX,
                  yy = ((w / cl.ncx) % cl.ncy) * PY + (int)threadIdx.x / PX, z0 = (w / (cl.ncx * cl.ncy)) * cl.chunk;
        const int z1 = min(z0 + cl.chunk, g.nz);
        const bool col = xx < g.nx && yy < g.ny;
        uint8_t l[kMaxChunk];
        double bv[kMaxChunk];
#pragma unroll
        for (int k = 0; k < kMaxChunk; ++k) {   // b is read with the label (used on fluid cells only)
            const bool in = col && z0 + k < z1;
            const size_t q = in ? cell_index(g, z0 + k, yy, xx) : 0;
            l[k] = *at_or(lab, q, in, g_pad_solid);
            bv[k] = *at_or(b, q, in, pad_zero<double>());
        }
        int f = 0;
#pragma unroll
        for (int k = 0; k < kMaxChunk; ++k) {
            if (l[k] > kSolid) v[2] += 1.0;
            if (l[k] == kFluid) {
                f = 1;
                v[1] += 1.0;
                if (!isfinite(bv[k])) v[3] += 1.0;
                else v[0] += bv[k] * bv[k];
            }
        }
        if (col)
            for (int z = z0; z < z1; ++z) x0[cell_index(g, z, yy, xx)] = X(0);
        const int any = __syncthreads_or(f);
        if (threadIdx.x == 0) live[w] = any ? 1 : 0;
        if (any || !col) continue;
        for (int i = 0; i < zb.n; ++i)
            for (int z = z0; z < z1; ++z) {
                const size_t q = cell_index(g, z, yy, xx);
                if (zb.bytes[i] == 8) static_cast<double*>(zb.p[i])[q] = 0.0;
                else static_cast<float*>(zb.p[i])[q] = 0.0f;
            }
    }
    block_partials<kBlock>(v, partials);
}

struct SolveParams {
    double tol;
    int max_iter, fixed, n_ortho, method, sym;
};

// One block: the state of a solve from the nparts validation partials, and
// items[0 .. nlive) = the live items in increasing order (z-major, so each
// XCD's contiguous share of the list is a z-range).  A thread owns 16
// consecutive flags per round.
__global__ __launch_bounds__(kCtlBlock) void k_live_list(const uint8_t* __restrict__ live, int count,
                                                         uint32_t* __restrict__ items,
                                                         const double* __restrict__ partials, int nparts, State* st,
                                                         ClassSums* cls, SolveParams p) {
    constexpr int W = kCtlBlock / 64, U = 16;
    __shared__ uint32_t wsum[W];
    double head[4][kSumU];
    head_partials<4, kCtlBlock>(partials, nparts, head);
    clear_classes(cls);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t base = 0;
    for (int i0 = 0; i0 < count; i0 += U * kCtlBlock) {
        const int i = i0 + U * (int)threadIdx.x;
        uint32_t m = 0u;
        if (i < count) {   // the flags are padded to a multiple of 256 bytes
            const uint4 f = *reinterpret_cast<const uint4*>(live + i);
            const uint32_t w[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (i + k < count && ((w[k >> 2] >> (8 * (k & 3))) & 255u)) m |= 1u << k;
        }
        const uint32_t mine = (uint32_t)__popc(m);
        uint32_t incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)incl, d, 64);
            if (lane >= d) incl += o;
        }
        if (lane == 63) wsum[wv] = incl;
        __syncthreads();
        uint32_t off = base + incl - mine, tot = 0;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            off += k < wv ? wsum[k] : 0u;
            tot += wsum[k];
        }
        while (m) {
            items[off++] = (uint32_t)(i + __ffs((int)m) - 1);
            m &= m - 1u;
        }
        base += tot;
        __syncthreads();   // wsum is rewritten by the next round
    }
    double v[4];
    finish_partials<4, kCtlBlock>(head, partials, nparts, 4, v);
    if (threadIdx.x == 0) {
        State s = {};
        s.bb = v[0];
        s.tol2bb = p.tol * p.tol * v[0];
        s.n_fluid = (int)v[1];
        s.bad_label = (int)v[2];
        s.nonfinite = (int)v[3];
        s.scale = 1.0;
        s.max_iter = p.max_iter;
        s.fixed = p.fixed;
        s.n_ortho = p.n_ortho;
        s.method = p.method;
        s.sym = p.sym;
        s.nlive = (int)base;
        *st = s;
    }
}

}  // namespace nps
