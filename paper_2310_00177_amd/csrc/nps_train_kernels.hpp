// Backward kernels of the network (training loss of Sec. "Training").
//
// With g the gradient of a CConv block's output, r its input, I the image:
//   dL/dB_t      = sum_p g(p) r(p + a_t)                        (= U_t)
//   dL/dW[t,c,o] = sum_p g(p) r(p + a_t) I_c(p + o)
//   dL/dr(q)     = sum_t K_t(q - a_t) g(q - a_t)                 (transposed apply)
// In count form I_c = n_c / 8^(l-1) for fluid and air, and the solid channel
// follows from sum_c I_c = 1 (also for the solid padding):
//   dL/dW[t,solid,o] = U_t - dL/dW[t,fluid,o] - dL/dW[t,air,o].
// Only the transposed applies form a chain (k_adj, level by level, on kernels K
// formed at setup).  The 27 x 55 sums of every block (54 counts and the
// constant 1) need just the gradients the chain leaves behind, so in float one
// launch (k_wgrad) contracts all blocks of all levels once the chain is done,
// and its per-block partials are added up once per step.
#pragma once

#include "nps_kernels.hpp"
#include "nps_march_kernels.hpp"
#include "nps_setup_kernels.hpp"

#include <type_traits>

namespace nps {

constexpr int kFeat = 2 * kTaps + 1;            // 54 counts + the constant
constexpr int kWGrad = kTaps * kFeat;           // 1485 sums per CConv block
constexpr int kWPart = kWGrad + 3;              // a row of partial sums, padded
constexpr int kWRows = 1024;                    // rows (blocks) of all CConv blocks together

// ---------------------------------------------------------------------------
// the adjoint chain
// ---------------------------------------------------------------------------
// Block sums of the partials of dL/dc1 and dL/dc2: part[b] and part[grid + b].
__device__ __forceinline__ void dc_partials(const double (&v)[2], double* __restrict__ part) {
    __shared__ double sh[2][kBlock / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const double s0 = wave_sum(v[0]), s1 = wave_sum(v[1]);
    if (lane == 0) {
        sh[0][wid] = s0;
        sh[1][wid] = s1;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < kBlock / 64; ++i) t += sh[threadIdx.x][i];
        part[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

// The transposed apply of one CConv block on stored kernels.  UP, the up block
// x = c1 x1 + c2 CConv_2(Interp(xc)): out = CConv_2^T(c2 gx), and with x1 also
// the block's partials of dL/dc1 = gx.x1 and dL/dc2 = gx.x2 (part[b], part[grid
// + b]).  Down block x1 = CConv_1(r): out = CConv_1^T(g) with g = coef gx + the
// pool adjoint of the next level's input gradient (gnext / 8 of the parent
// cell), coef = c1, or 1 on the coarsest level (lvl < 0); at level 1 the output
// is restricted to fluid, where the input was.  At level 1 (L1) gx counts on
// fluid cells only.
// The gather reads K_t at 27 neighbours: all 27 loads go out ahead of the
// staging, at the cell itself where a neighbour lies outside (its g is zero).
// Tests around the loads had serialised them (16^3 level: 10 -> 4 us).
template <class T, bool L1, bool UP>
__global__ __launch_bounds__(kBlock) void k_adj(const uint8_t* __restrict__ lab, Grid g, const T* __restrict__ gx,
                                                const T* __restrict__ gnext, const T* __restrict__ kst,
                                                const State* st, int lvl, const T* __restrict__ x1,
                                                const T* __restrict__ x2, T* __restrict__ out,
                                                double* __restrict__ part) {
    __shared__ T g_s[kHaloP];
    const T coef = UP ? (T)st->c2[lvl] : lvl >= 0 ? (T)st->c1[lvl] : T(1);
    const Tiles tl = tiles_of(g);
    const int n = (int)ncells(g);
    const Grid gc = coarser(g);
    const int lx = threadIdx.x % TX, ly = (threadIdx.x / TX) % TY, lz = threadIdx.x / (TX * TY);
    const int base = halo_base(lx, ly, lz);
    double v[2] = {0.0, 0.0};
    struct E {
        T gx, gn;
        uint8_t l;
    };
    for (TileSpan sp = tile_span(tl.count()); sp.t0 < sp.t1; sp.t0 += sp.step) {
        const TileOrigin o = tile_origin(sp.t0, tl);
        const int xx = o.x0 + lx, yy = o.y0 + ly, zz = o.z0 + lz;
        const bool active = in_grid(g, zz, yy, xx);
        const int idx = active ? (int)cell_index(g, zz, yy, xx) : 0;
        T kv[kTaps];
#pragma unroll
        for (int t = 0; t < kTaps; ++t) {
            const int dz = t / 9 - 1, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
            const bool in = active && in_grid(g, zz - dz, yy - dy, xx - dx);
            kv[t] = kst[(size_t)t * n + (in ? idx - ((dz * g.ny + dy) * g.nx + dx) : idx)];
        }
        const auto e = load_batch<kHalo, E>([&](int i) {
            int x, y, z;
            halo_coords(i, o, x, y, z);
            const bool in = in_grid(g, z, y, x);
            const size_t q = in ? cell_index(g, z, y, x) : 0;
            E r{*at_or(gx, q, in, pad_zero<T>()), T(0), (uint8_t)kFluid};
            if constexpr (L1) r.l = *at_or(lab, q, in, g_pad_solid);
            if constexpr (!UP)
                if (gnext) r.gn = *at_or(gnext, in ? cell_index(gc, z >> 1, y >> 1, x >> 1) : 0, in, pad_zero<T>());
            return r;
        });
        uint8_t own = kFluid;
        if constexpr (L1) own = active ? lab[idx] : (uint8_t)kSolid;
        T x1v = T(0), x2v = T(0);
        if (UP && x1) {
            x1v = x1[idx];
            x2v = x2[idx];
        }
        __syncthreads();   // the previous tile's reads are done
        put_batch(e, [&](int i, E r) {
            const T m = r.l == kFluid ? r.gx : T(0);
            g_s[i] = UP ? m : coef * m + r.gn * T(0.125);
        });
        __syncthreads();
        T s = T(0);
#pragma unroll
        for (int t = 0; t < kTaps; ++t) s = fma(kv[t], g_s[base - halo_off(t)], s);
        if constexpr (UP) s *= coef;
        if (L1 && !UP && own != kFluid) s = T(0);
        if (active) out[idx] = s;
        if (UP && active && own == kFluid) {   // x1, x2 may hold anything where the output is masked
            v[0] += (double)g_s[base] * (double)x1v;
            v[1] += (double)g_s[base] * (double)x2v;
        }
    }
    if (UP && x1) dc_partials(v, part);
}

// The same at level 1 in float without stored kernels (108 bytes a cell, which
// took 107 us to form and two passes to read at 128^3): K is formed on matrix
// cores as in the forward.  A work item is that of the level-1 network kernels.
// Plane by plane, the waves form V_t(p) = K_t(p) g(p) for the plane's cells with
// a one-cell border, 16 cells at a time, into a table of 27 rows in LDS; then
// each thread gathers V_t(q - a_t) for its column: 9 taps for each of the three
// output planes that see the plane.  UP: groups without fluid have V = 0 and
// groups whose fluid cells have all-fluid windows (g is zero on the others) take
// the constant fluid kernel, by the modes of the forward's up kernel; an item
// that no group reaches is zero.  The table bounds the occupancy (two blocks a
// CU); per plane a wave writes 8 values a lane and group and reads 27 a cell.  128^3:
// 65 us, against 107 us to form and store K and 70 us to gather it.
constexpr int kAF = 72, kAFRows = PHY + 2;      // feature rows: x offsets -4 .. 67, y offsets -2 .. 5
constexpr int kAG = 72;                         // g rows: x offsets -4 .. 67 (-1 .. 64 used)
constexpr int kAVRow = 68, kAV = 420;           // V rows: x offsets -1 .. 64; 4 kAV = 16 mod 64 banks between lane groups

template <int KM, bool UP, int CH>
__global__ __launch_bounds__(kBlock) NPS_WAVES_PER_EU(2) void k_adj_l1m(
    const uint8_t* __restrict__ lab, Grid g, const float* __restrict__ gx, const float* __restrict__ gnext,
    const CConvW<float>* __restrict__ w, const MfmaW* __restrict__ wm, const State* st, const float* __restrict__ x1,
    const float* __restrict__ x2, float* __restrict__ out, double* __restrict__ part,
    const uint32_t* __restrict__ gmode, int flags) {
    const int wide = flags & kWideRows;
    constexpr int P = MarchCtx<KM>::P, NPL = CH + 2;
    using S = StageTasks<CH>;
    __shared__ __attribute__((aligned(16))) uint32_t f_s[(CH + 4) * kAFRows * kAF];
    __shared__ __attribute__((aligned(16))) float g_s[NPL * PHY * kAG];
    __shared__ float v_s[(kTaps + 1) * kAV];
    __shared__ uint32_t m_s[NPL * 3 * 4];
    const float coef = UP ? (float)st->c2[0] : (float)st->c1[0];
    const Columns cl = march_columns(g);
    const Grid gc = coarser(g);
    const int nwx = wave_columns(g);
    const int lane = threadIdx.x & 63, lg = lane >> 4, n = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t fluid_word = feat_word<KM, true>(kFluid), pstride = (uint32_t)g.ny * (uint32_t)g.nx;
    u16x8 A[P][2][2];
    int fofs[8], vofs[8];   // feature offset of window position j; V row of the tap in slot j (past 26: a spare row)
    float kp[8];            // the all-fluid kernel at those taps
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) A[p][mb][ks] = *reinterpret_cast<const u16x8*>(&wm->bf16[p][mb][ks][lane][0]);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int t = 16 * (j >> 2) + 4 * lg + (j & 3), o = min(t, kTaps - 1);
        fofs[j] = ((o / 9 - 1) * kAFRows + o / 3 % 3 - 1) * kAF + o % 3 - 1;
        vofs[j] = min(t, kTaps) * kAV;
        kp[j] = t < kTaps ? w->Kpure[kFluid][o] : 0.0f;
    }
    const bool one = lg == 2;
    // V of 16 cells: fb the lane's cell in f_s, gi in g_s, vi in a row of v_s
    auto group = [&](int fb, int gi, int vi, uint32_t mode) {
        const float gv = g_s[gi];
        float K[8];
        if (mode == kGZero) {
#pragma unroll
            for (int j = 0; j < 8; ++j) v_s[vofs[j] + vi] = 0.0f;
            return;
        }
        if (mode == kGPure) {
#pragma unroll
            for (int j = 0; j < 8; ++j) K[j] = kp[j];
        } else {
            uint32_t fw[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) fw[j] = f_s[fb + fofs[j]];
            fw[7] = one ? feat_one<KM>() : fw[7];
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const u16x8 B[2] = {__builtin_bit_cast(u16x8, (u32x4){fw[0], fw[1], fw[2], fw[3]}),
                                __builtin_bit_cast(u16x8, (u32x4){fw[4], fw[5], fw[6], fw[7]})};
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[p][mb][ks]),
                                                                      __builtin_bit_cast(bf16x8, B[ks]), acc, 0, 0, 0);
#pragma unroll
                for (int j = 0; j < 4; ++j) K[4 * mb + j] = acc[j];
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) v_s[vofs[j] + vi] = K[j] * gv;
    };
    // the edge group: the 12 cells beside the footprint's rows (lanes past them
    // repeat the last into spare columns)
    const int en = min(n, 2 * PHY - 1), erow = en >> 1, eix = (en & 1) ? PX : -1;
    const int evi = n < 2 * PHY ? erow * kAVRow + eix + 1 : PHY * kAVRow + n - 2 * PHY;
    static_assert(PHY * kAVRow + 16 - 2 * PHY <= kAV, "spare columns");
    double v[2] = {0.0, 0.0};
    const MarchItems mi = march_items(cl, (int)gridDim.x, (int)blockIdx.x, flags & kSlabs);
    for (int li = mi.li; li < mi.count; li += mi.step) {
        const MarchItem it = march_item(mi, li, cl);
        const int x0 = it.cx * PX, y0 = it.cy * PY, z0 = it.zc * CH;
        const int tid = item_thread();
        const int xx = x0 + lane, yy = y0 + wv;   // the thread's column
        const bool col = xx < g.nx && yy < g.ny;
        const uint32_t own = col ? (uint32_t)z0 * pstride + (uint32_t)yy * g.nx + xx : 0u;
        // modes of the planes' groups: the footprint's rows and its y neighbours' (four waves each)
        uint32_t mw = 0u;
        if (tid < NPL * 12) {
            const int z = z0 - 1 + tid / 12, cy = it.cy - 1 + tid / 4 % 3, wx = 4 * it.cx + tid % 4;
            const bool in = z >= 0 && z < g.nz && cy >= 0 && cy < cl.ncy && wx < nwx;
            if (in) mw = UP ? gmode[((size_t)z * cl.ncy + cy) * nwx + wx] : kAnyGeneral;
        }
        float4 gw[S::K];
        uint32_t lw[S::K];
        float2 nw[S::K];
#pragma unroll
        for (int k = 0; k < S::K; ++k) {
            auto load = [&](auto quad) {
                constexpr bool Q = decltype(quad)::value;
                const int t = tid + k * kBlock;
                const StagePos s = stage_pos<CH, 0, Q>(g, x0, y0, z0, t);
                gw[k] = stage_values<Q>(gx, s, wide);
                lw[k] = stage_labels<Q>(lab, s, wide);
                nw[k] = float2{0.0f, 0.0f};
                if (!UP && s.cells > 0) {   // the parents of the task's x pairs (quads start on even x)
                    const int e = min(t, S::kAll - 1) - S::kQuads, row = Q ? t / (PX / 4) : e >> 1;
                    const int ix = Q ? 4 * (t % (PX / 4)) : (e & 1) ? PX : -1;
                    const int z = z0 + row / PHY - 1, y = y0 + row % PHY - 1, x = x0 + ix;
                    const size_t q = cell_index(gc, z >> 1, y >> 1, x >> 1);
                    nw[k].x = gnext[q];
                    nw[k].y = s.cells > 2 ? gnext[q + 1] : 0.0f;
                }
            };
            if (S::quads(wv, k)) load(std::true_type{});
            else if (S::edges(wv, k)) load(std::false_type{});
        }
        // features: rows of 18 words of four labels
        constexpr int FT = (CH + 4) * kAFRows * (kAF / 4), KF = (FT + kBlock - 1) / kBlock;
        uint32_t fw[KF];
#pragma unroll
        for (int k = 0; k < KF; ++k) {
            const int t = min(tid + k * kBlock, FT - 1), row = t / (kAF / 4), x = x0 - 4 + 4 * (t % (kAF / 4));
            const int z = z0 - 2 + row / kAFRows, y = y0 - 2 + row % kAFRows;
            const bool in = z >= 0 && z < g.nz && y >= 0 && y < g.ny && x >= 0 && x < g.nx;
            fw[k] = stage_labels<true>(lab, StagePos{0, in ? (uint32_t)cell_index(g, z, y, x) : 0u,
                                                     in ? min(4, g.nx - x) : 0}, wide);
        }
        bool some = mw != 0u;
        __syncthreads();   // the previous item's reads are done
        if (tid < NPL * 12) m_s[tid] = mw;
#pragma unroll
        for (int k = 0; k < S::K; ++k) {
            auto put = [&](auto quad) {
                constexpr bool Q = decltype(quad)::value;
                const int t = tid + k * kBlock, e = min(t, S::kAll - 1) - S::kQuads;
                const int at = Q ? t / (PX / 4) * kAG + 4 * (t % (PX / 4)) + 4 : (e >> 1) * kAG + ((e & 1) ? PX : -1) + 4;
                const float r[4] = {gw[k].x, gw[k].y, gw[k].z, gw[k].w};
                float q[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float m = ((lw[k] >> (8 * j)) & 255u) == kFluid ? r[j] : 0.0f;
                    q[j] = UP ? m : fmaf(0.125f, j < 2 ? nw[k].x : nw[k].y, coef * m);
                }
                if constexpr (Q) *reinterpret_cast<float4*>(g_s + at) = float4{q[0], q[1], q[2], q[3]};
                else g_s[at] = q[0];
                if constexpr (!Q) some = some || q[0] != 0.0f;   // fluid beside the footprint
            };
            if (S::quads(wv, k)) put(std::true_type{});
            else if (S::edges(wv, k)) put(std::false_type{});
        }
#pragma unroll
        for (int k = 0; k < KF; ++k) {
            const int t = min(tid + k * kBlock, FT - 1);
            uint32_t e[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) e[j] = feat_word<KM, true>((fw[k] >> (8 * j)) & 255u);
            *reinterpret_cast<uint4*>(f_s + 4 * t) = uint4{e[0], e[1], e[2], e[3]};
        }
        if (!__syncthreads_or(some)) {   // no cell of the item's border or inside contributes
#pragma unroll
            for (int i = 0; i < CH; ++i)
                if (col && z0 + i < g.nz) out[(size_t)own + (size_t)i * pstride] = 0.0f;
            continue;
        }
        float a2 = 0.0f, a1 = 0.0f;   // output planes k - 2 and k - 1 so far
        for (int k = 0; k < NPL; ++k) {
            // the wave's words of the rows above, inside and below the footprint
            const uint32_t mlo = __builtin_amdgcn_readfirstlane(m_s[k * 12 + wv]),
                           min_ = __builtin_amdgcn_readfirstlane(m_s[k * 12 + 4 + wv]),
                           mhi = __builtin_amdgcn_readfirstlane(m_s[k * 12 + 8 + wv]);
            const uint32_t mode[PHY] = {mlo >> 24, min_ & 255u, (min_ >> 8) & 255u, (min_ >> 16) & 255u, min_ >> 24,
                                        mhi & 255u};
            const int fb = ((k + 1) * kAFRows + 1) * kAF + 16 * wv + n + 4, gi = k * PHY * kAG + 16 * wv + n + 4;
#pragma unroll
            for (int r = 0; r < PHY; ++r) group(fb + r * kAF, gi + r * kAG, r * kAVRow + 16 * wv + n + 1, mode[r]);
            if (wv == (k & 3))   // the edge cells, in turn
                group(((k + 1) * kAFRows + 1 + erow) * kAF + eix + 4, (k * PHY + erow) * kAG + eix + 4, evi, kGGeneral);
            __syncthreads();   // V of the plane
            // sums of nine as trees: with the products rounded on their own, they keep the
            // rounding of a chain of fused multiply-adds
            auto nine = [&](int az) {
                float q[9];
#pragma unroll
                for (int d = 0; d < 9; ++d)
                    q[d] = v_s[(9 * az + d) * kAV + (wv + 2 - d / 3) * kAVRow + lane + 2 - d % 3];
                return (((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]))) + q[8];
            };
            a2 += nine(0);                 // a_z = -1: output plane k - 2
            a1 += nine(1);                 // a_z = 0: output plane k - 1
            const float a0 = nine(2);      // a_z = 1: output plane k
            const int i = k - 2;
            if (i >= 0 && z0 + i < g.nz && col) {
                const bool fl = f_s[((i + 2) * kAFRows + wv + 2) * kAF + lane + 4] == fluid_word;
                const size_t q = (size_t)own + (size_t)i * pstride;
                out[q] = UP ? coef * a2 : fl ? a2 : 0.0f;
                if (UP && x1 && fl) {   // x1, x2 may hold anything where the output is masked
                    const double gv = (double)g_s[((i + 1) * PHY + wv + 1) * kAG + lane + 4];
                    v[0] += gv * (double)x1[q];
                    v[1] += gv * (double)x2[q];
                }
            }
            a2 = a1;
            a1 = a0;
            __syncthreads();   // the gather is done
        }
    }
    if (UP && x1) dc_partials(v, part);
}

// A copy of the adjoint's input, for a caller whose output overlaps it: level 1
// reads g in the up sweep's first step and again, a window at a time, in the last
// step, which writes y.
template <class T>
__global__ __launch_bounds__(kBlock) void k_copy(size_t n, const T* __restrict__ src, T* __restrict__ dst) {
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) dst[i] = src[i];
}

// Adjoint of the 2x trilinear upsampling: gc(j) = sum over fine cells f of
// w(f -> j) gf(f).  Along one axis a fine cell f feeds f/2 with 3/4 and its
// neighbour on f's side (clamped) with 1/4, so coarse j collects f = 2j, 2j+1
// (3/4), 2j-1, 2j+2 (1/4), and at the ends the clamped quarter of f = 0 or
// f = 2n-1 once more: always four terms, with the outer two clamped.  Axis by
// axis in double; the 64 loads are independent.
template <class T>
__global__ __launch_bounds__(kBlock) void k_adj_interp(Grid gcoarse, const T* __restrict__ gf, T* __restrict__ gcout) {
    const Grid gfine{2 * gcoarse.nz, 2 * gcoarse.ny, 2 * gcoarse.nx};
    const int n = (int)ncells(gcoarse);
    auto cells = [](int j, int nf, int (&f)[4]) {
        f[0] = max(2 * j - 1, 0);
        f[1] = 2 * j;
        f[2] = 2 * j + 1;
        f[3] = min(2 * j + 2, nf - 1);
    };
    auto sum4 = [](double a, double b, double c, double d) { return 0.75 * (b + c) + 0.25 * (a + d); };
    for (int q = (int)(blockIdx.x * kBlock + threadIdx.x); q < n; q += (int)(gridDim.x * kBlock)) {
        const int x = q % gcoarse.nx, y = q / gcoarse.nx % gcoarse.ny, z = q / (gcoarse.nx * gcoarse.ny);
        int fx[4], fy[4], fz[4];
        cells(x, gfine.nx, fx);
        cells(y, gfine.ny, fy);
        cells(z, gfine.nz, fz);
        T v[4][4][4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int c = 0; c < 4; ++c) v[a][b][c] = gf[cell_index(gfine, fz[a], fy[b], fx[c])];
        double sz[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            double sy[4];
#pragma unroll
            for (int b = 0; b < 4; ++b)
                sy[b] = sum4((double)v[a][b][0], (double)v[a][b][1], (double)v[a][b][2], (double)v[a][b][3]);
            sz[a] = sum4(sy[0], sy[1], sy[2], sy[3]);
        }
        gcout[q] = (T)sum4(sz[0], sz[1], sz[2], sz[3]);
    }
}

// ---------------------------------------------------------------------------
// parameter sums
// ---------------------------------------------------------------------------
// One CConv block: G[t][f] = sum_p g(p) r(p + a_t) F_f(p) over the level's
// cells, F the 54 window counts and the constant 1.
struct WgradSeg {
    const void* img;                  // labels (level 1) or counts
    Grid g;
    const void *gx, *gnext, *r;       // as in k_adj; r: the block's input (up: the coarse x it interpolates)
    int l1, up, lvl;                  // lvl: index of the coefficient of gx (< 0: 1)
    int pieces;                       // pieces of a count: 1 up to level 3 (exact in bf16), else 2
    int row0, rows;                   // blocks (rows of partial sums) of this CConv block
    double scale;                     // 8^-(l-1)
    size_t gw;                        // W of the block in the gradient blob
};

constexpr int kMaxWSegs = 2 * kMaxLevels;

struct WgradArgs {
    int nseg, add;                    // add: to the rows of the systems before (a batch)
    WgradSeg seg[kMaxWSegs];
};

typedef float f32x2 __attribute__((ext_vector_type(2)));

// bf16 of a pair, rounded to nearest even, as one word; and its values.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a, b}, bf16x2));
}
__device__ __forceinline__ float pair_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float pair_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// LDS of a block: the staged tile, then the waves' sums of one tap block.
template <class T>
struct WgradLds {
    static constexpr int kR = 2 * kHaloP * 4, kG = kR + kHaloP * (int)sizeof(T), kC = kG + kBlock * (int)sizeof(T);
    static constexpr int kTile = kC + kCoarseTileP * (int)sizeof(T);
    static constexpr int kSums = 4 * 16 * 64 * (int)sizeof(T);
    static constexpr int kBytes = kTile > kSums ? kTile : kSums;
};

// The sums of one block's tiles on the matrix cores: G is a 27 x 55 matrix
// product contracted over the cells, U[t][p] = g(p) r(p + a_t) times F[f][p].
// A wave owns the 64 cells of its z-plane of the tile and all of G (2 x 4 blocks
// of 16 x 16); lane (k, n) supplies tap 16 mb + n and feature 16 fb + n.
//   float   v_mfma_f32_16x16x32_bf16, 32 cells at a time (lane k: 8 cells along
//           x): U is split into PU = 3 bf16 pieces whose sum is the float
//           exactly, the counts are exact in one piece up to level 3 and in two
//           beyond, so all products are exact and the sums are fp32, as on the
//           fp32 matrix cores, at 3/16 of their time.  PU = 1: the bf16 leg.
//   double  v_mfma_f64_16x16x4_f64.
// What bounds it is forming U (16 products and their pieces per lane and 32
// cells) beside 24 matrix instructions.  A wave whose g is all zero skips its
// cells, a level-1 down tile without fluid in reach the tile.  All blocks of a
// 128^3 system: 88.5 us in float.  (On fp32 matrix cores, and per thread on the vector
// ALU in double, inside the transposed applies: 230 us for level 1 up, 140 us down, 25
// us and more for every other block.)
template <class T, int PU, int NF, bool L1, bool UP>
__device__ __forceinline__ void wgrad_block(const WgradSeg& sg, const State* st, int add, char* lds,
                                            double* __restrict__ row) {
    constexpr bool F64 = sizeof(T) == 8;
    using M = WgradLds<T>;
    uint32_t* f_s = reinterpret_cast<uint32_t*>(lds);                  // float: bf16 count pairs; double: image words
    uint32_t* f2_s = f_s + kHaloP;                                     // their second pieces
    T* r_s = reinterpret_cast<T*>(lds + M::kR);
    T* g_s = reinterpret_cast<T*>(lds + M::kG);
    T* c_s = reinterpret_cast<T*>(lds + M::kC);
    const Grid g = sg.g, gc = coarser(g);
    const T coef = sg.lvl < 0 ? T(1) : UP ? (T)st->c2[sg.lvl] : (T)st->c1[sg.lvl];
    const T* gx = static_cast<const T*>(sg.gx);
    const T* gnext = static_cast<const T*>(sg.gnext);
    const T* r = static_cast<const T*>(sg.r);
    const Tiles tl = tiles_of(g);
    const int lx = threadIdx.x % TX, ly = (threadIdx.x / TX) % TY, lz = threadIdx.x / (TX * TY);
    const int lane = threadIdx.x & 63, n = lane & 15, k = lane >> 4;
    int toff[2], foff[4];   // LDS offsets of the lane's taps and window positions
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) toff[mb] = halo_off_rt(min(16 * mb + n, kTaps - 1));
#pragma unroll
    for (int fb = 0; fb < 4; ++fb) foff[fb] = halo_off_rt(min(8 * fb + (n >> 1), kTaps - 1));
    const bool air = n & 1, one = n == 2 * kTaps - 48;   // feature 54 = 48 + n
    using Acc = typename std::conditional<F64, f64x4, f32x4>::type;
    Acc acc[2][4];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int fb = 0; fb < 4; ++fb) acc[mb][fb] = Acc{0, 0, 0, 0};
    InterpSlots isl;
    if constexpr (UP) isl = interp_slots();
    for (int tile = (int)blockIdx.x - sg.row0; tile < tl.count(); tile += sg.rows) {
        const TileOrigin o = tile_origin(tile, tl);
        const int xx = o.x0 + lx, yy = o.y0 + ly, zz = o.z0 + lz;
        const bool active = in_grid(g, zz, yy, xx);
        const size_t idx = active ? cell_index(g, zz, yy, xx) : 0;
        // loads
        T gv = active ? gx[idx] : T(0);
        const T gn = !UP && gnext && active ? gnext[cell_index(gc, zz >> 1, yy >> 1, xx >> 1)] : T(0);
        uint8_t own = kFluid;
        if constexpr (L1) own = active ? static_cast<const uint8_t*>(sg.img)[idx] : (uint8_t)kSolid;
        UpLoads<T> ul;
        Batch<kHalo, T> rl;
        if constexpr (UP) {
            ul = load_image_interp<L1, T>(sg.img, r, g, o);
        } else {
            ul.img = load_batch<kHalo, uint32_t>([&](int i) { return image_load<L1>(sg.img, g, o, i); });
            rl = load_batch<kHalo, T>([&](int i) {
                const HaloCell c = halo_cell(g, o, i);
                return *at_or(r, c.q, c.in, pad_zero<T>());
            });
        }
        __syncthreads();   // the previous tile's reads are done
        put_batch(ul.img, [&](int i, uint32_t v) {
            if constexpr (F64) {
                f_s[i] = v;
            } else {
                uint32_t c0, c1;
                counts_of<L1>(v, c0, c1);
                const float a = (float)c0, b = (float)c1;
                const uint32_t h = (__float_as_uint(a) >> 16) | (__float_as_uint(b) & 0xffff0000u);
                f_s[i] = h;
                if constexpr (NF == 2) {
                    const float a2 = a - pair_lo(h), b2 = b - pair_hi(h);
                    f2_s[i] = (__float_as_uint(a2) >> 16) | (__float_as_uint(b2) & 0xffff0000u);
                }
            }
        });
        if (L1 && own != kFluid) gv = T(0);
        gv = UP ? coef * gv : coef * gv + gn * T(0.125);
        g_s[threadIdx.x] = gv;
        const bool work = __any(gv != T(0));   // the wave's cells are its z-plane's (a NaN differs from zero)
        if constexpr (UP) {
            put_batch(ul.c, [&](int i, T v) { c_s[i] = v; });
            __syncthreads();
            interp_tile<T>(r_s, c_s, g, o, isl);
            __syncthreads();
        } else {
            bool any = false;
#pragma unroll
            for (int j = 0; j < Batch<kHalo, T>::K; ++j) {
                const T v = !L1 || ul.img.v[j] == (uint32_t)kFluid ? rl.v[j] : T(0);   // the input is padded with zeros
                r_s[threadIdx.x + j * kBlock] = v;
                any = any || v != T(0);
            }
            if (L1) {
                if (!__syncthreads_or(any)) continue;
            } else {
                __syncthreads();
            }
        }
        if (!work) continue;
        if constexpr (F64) {
#pragma unroll 4
            for (int s = 0; s < 16; ++s) {   // cells 4 s + k of the wave's plane
                const int x = 4 * (s & 3) + k, y = s >> 2, hb = halo_base(x, y, lz);
                const T gp = g_s[(lz * TY + y) * TX + x];
                T u[2];
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) u[mb] = gp * r_s[hb + toff[mb]];
#pragma unroll
                for (int fb = 0; fb < 4; ++fb) {
                    uint32_t c0, c1;
                    counts_of<L1>(f_s[hb + foff[fb]], c0, c1);
                    T b = (T)(air ? c1 : c0);
                    if (fb == 3) b = one ? T(1) : b;
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb)
                        acc[mb][fb] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[mb], b, acc[mb][fb], 0, 0, 0);
                }
            }
        } else {
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const uint32_t sel = air ? 0x07060302u : 0x05040100u;   // the lane's channel of two words
#pragma unroll
            for (int s = 0; s < 2; ++s) {    // rows 2 s + (k >> 1), cells 8 (k & 1) + 0 .. 7
                const int x = 8 * (k & 1), y = 2 * s + (k >> 1), hb = halo_base(x, y, lz);
                const float4* gp = reinterpret_cast<const float4*>(g_s + (lz * TY + y) * TX + x);
                const float4 g0 = gp[0], g1 = gp[1];
                const float gq[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
                u32x4 U[PU][2];
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float a = gq[2 * j] * r_s[hb + toff[mb] + 2 * j], b = gq[2 * j + 1] * r_s[hb + toff[mb] + 2 * j + 1];
#pragma unroll
                        for (int p = 0; p < PU; ++p) {
                            const uint32_t w = bf16_pair(a, b);
                            U[p][mb][j] = w;
                            a -= pair_lo(w);
                            b -= pair_hi(w);
                        }
                    }
#pragma unroll
                for (int fb = 0; fb < 4; ++fb)
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        const uint32_t* src = (f ? f2_s : f_s) + hb + foff[fb];
                        u32x4 F;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            F[j] = __builtin_amdgcn_perm(src[2 * j + 1], src[2 * j], sel);
                            if (fb == 3) F[j] = one ? (f ? 0u : 0x3f803f80u) : F[j];
                        }
#pragma unroll
                        for (int p = 0; p < PU; ++p)
#pragma unroll
                            for (int mb = 0; mb < 2; ++mb)
                                acc[mb][fb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    __builtin_bit_cast(bf16x8, U[p][mb]), __builtin_bit_cast(bf16x8, F), acc[mb][fb], 0,
                                    0, 0);
                    }
            }
        }
    }
    // the four waves' sums, one tap block at a time, added in wave order; lane
    // (k, n) holds rows 4 k + i (float) or 4 i + k (double) of column n
    T* sum_s = reinterpret_cast<T*>(lds);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        __syncthreads();
#pragma unroll
        for (int fb = 0; fb < 4; ++fb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m = F64 ? 4 * i + k : 4 * k + i;
                sum_s[(lz * 16 + m) * 64 + 16 * fb + n] = acc[mb][fb][i];
            }
        __syncthreads();
        for (int e = threadIdx.x; e < 16 * 64; e += kBlock) {
            const int t = 16 * mb + (e >> 6), f = e & 63;
            if (t >= kTaps || f >= kFeat) continue;
            double v = 0.0;
#pragma unroll
            for (int w = 0; w < kBlock / 64; ++w) v += (double)sum_s[w * 1024 + e];
            double* dst = row + t * kFeat + f;
            *dst = add ? *dst + v : v;
        }
    }
}

// All CConv blocks of a system; block b's sums go to row b of part.
template <class T, int PU>
__global__ __launch_bounds__(kBlock) NPS_WAVES_PER_EU(sizeof(T) == 8 ? 2 : 4) void k_wgrad(WgradArgs a, const State* st,
                                                                                          double* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) char lds[WgradLds<T>::kBytes];
    int i = 0;
    while (i < a.nseg - 1 && (int)blockIdx.x >= a.seg[i + 1].row0) ++i;
    const WgradSeg sg = a.seg[i];
    double* row = part + (size_t)blockIdx.x * kWPart;
    constexpr int N2 = sizeof(T) == 8 ? 1 : 2;   // doubles hold every count
    if (sg.l1) {
        if (sg.up) wgrad_block<T, PU, 1, true, true>(sg, st, a.add, lds, row);
        else wgrad_block<T, PU, 1, true, false>(sg, st, a.add, lds, row);
    } else if (sg.pieces == 1) {
        if (sg.up) wgrad_block<T, PU, 1, false, true>(sg, st, a.add, lds, row);
        else wgrad_block<T, PU, 1, false, false>(sg, st, a.add, lds, row);
    } else {
        if (sg.up) wgrad_block<T, PU, N2, false, true>(sg, st, a.add, lds, row);
        else wgrad_block<T, PU, N2, false, false>(sg, st, a.add, lds, row);
    }
}

// The rows are added up in two passes of fixed order: k_wgrad_chunks sums
// each chunk of kWChunk consecutive rows of a CConv block into the chunk's
// first row (in place: no other block reads that chunk), then k_wgrad_reduce
// sums the first rows in chunk order.
constexpr int kWChunk = 32;

__global__ __launch_bounds__(kBlock) void k_wgrad_chunks(WgradArgs a, double* __restrict__ part) {
    const WgradSeg& sg = a.seg[blockIdx.z];
    const int idx = blockIdx.y * kBlock + threadIdx.x;   // column
    const int c0 = (int)blockIdx.x * kWChunk;
    if (idx >= kWGrad || c0 >= sg.rows) return;
    const int b0 = sg.row0 + c0, b1 = sg.row0 + min(c0 + kWChunk, sg.rows);
    constexpr int U = 8;
    double s = 0.0;
    for (int b = b0; b < b1; b += U) {
        double t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) t[u] = b + u < b1 ? part[(size_t)(b + u) * kWPart + idx] : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) s += t[u];
    }
    part[(size_t)b0 * kWPart + idx] = s;
}

// One block per CConv block: its sums into the gradient blob: W[t][c][o] (c =
// fluid, air scaled by 1/8^(l-1); solid from U_t), B[t] = U_t.
__global__ __launch_bounds__(kBlock) void k_wgrad_reduce(WgradArgs a, const double* __restrict__ part,
                                                         double* __restrict__ grad) {
    __shared__ double sums[kWGrad];
    const WgradSeg& sg = a.seg[blockIdx.x];
    double* gW = grad + sg.gw;
    double* gB = gW + kTaps * 3 * kTaps;
    for (int idx = threadIdx.x; idx < kWGrad; idx += kBlock) {
        constexpr int U = 8;
        double s = 0.0;
        for (int c = 0; c < sg.rows; c += U * kWChunk) {
            double t[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                t[u] = c + u * kWChunk < sg.rows ? part[(size_t)(sg.row0 + c + u * kWChunk) * kWPart + idx] : 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) s += t[u];
        }
        sums[idx] = s;
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < kTaps * kTaps; idx += kBlock) {   // (t, o)
        const int t = idx / kTaps, o = idx % kTaps;
        const double u = sums[t * kFeat + kFeat - 1];
        const double gf = sg.scale * sums[t * kFeat + 2 * o], ga = sg.scale * sums[t * kFeat + 2 * o + 1];
        gW[(t * 3 + kFluid) * kTaps + o] += gf;
        gW[(t * 3 + kAir) * kTaps + o] += ga;
        gW[(t * 3 + kSolid) * kTaps + o] += u - gf - ga;
    }
    for (int t = threadIdx.x; t < kTaps; t += kBlock) gB[t] += sums[t * kFeat + kFeat - 1];
}

// Aff gradients: dL/dWbar = dL/dc * S / (27 n_l), dL/dBbar = dL/dc, for Aff_1
// and Aff_2 of every level (one block each), with the image-window sums
// S[c][o] = sum_p I_c(p + o) (solid padding), the derivative of an Aff scalar
// with respect to its weights times 27 n_l.  They come from the set-up's
// boundary sums: S[c][o] adds the classes whose cells q have q - o in the grid,
// and the solid channel follows from sum_c I_c = 1.  Integers, exact in double.
// (A pass over the image per level before: 115 us of a 128^3 system.)
struct AffGradArgs {
    Grid g;                                // level 1
    int pyr;                               // pyramid blocks
    const ClassSums* cls;
    const uint2* tot;
    const double* dc[kMaxLevels];          // dL/dc1, dL/dc2 partials of a level ([2][nparts])
    int nparts[kMaxLevels];
    size_t ga[kMaxLevels];                 // Aff_1 of the level in the gradient blob (Aff_2 follows)
};

__global__ __launch_bounds__(kBlock) void k_aff_grad(AffGradArgs a, double* __restrict__ grad) {
    __shared__ double sh[4][kBlock / 64], dc_s[2];
    __shared__ double n_s[2][kClasses];
    const int s = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // every load that needs no sum goes out first
    const int o = min((int)threadIdx.x, kTaps - 1);
    const uint32_t cl = (uint32_t)lane;
    const uint32_t k0 = cl ? a.cls->n[s][cl][0] : 0u, k1 = cl ? a.cls->n[s][cl][1] : 0u;
    double* g1 = grad + a.ga[s];
    double* g2 = g1 + 3 * kTaps + 1;
    double old1[4], old2[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        old1[c] = g1[c < 3 ? c * kTaps + o : 3 * kTaps];
        old2[c] = g2[c < 3 ? c * kTaps + o : 3 * kTaps];
    }
    double v[4] = {0.0, 0.0, 0.0, 0.0};    // dL/dc1, dL/dc2, fluid and air cells of the grid
    const int np = a.nparts[s];
    for (int b0 = 0; b0 < max(np, a.pyr); b0 += 2 * kBlock) {
        double d0[2], d1[2];
        uint2 t[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int b = b0 + u * kBlock + (int)threadIdx.x;
            d0[u] = b < np ? a.dc[s][b] : 0.0;
            d1[u] = b < np ? a.dc[s][np + b] : 0.0;
            t[u] = b < a.pyr ? a.tot[b] : uint2{0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            v[0] += d0[u];
            v[1] += d1[u];
            v[2] += (double)t[u].x;
            v[3] += (double)t[u].y;
        }
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        v[w] = wave_sum(v[w]);
        if (lane == 0) sh[w][wv] = v[w];
    }
    __syncthreads();
    if (threadIdx.x < kClasses) {          // wave 0: the class sums, class 0 the rest of the grid
        double t[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            t[w] = 0.0;
#pragma unroll
            for (int i = 0; i < kBlock / 64; ++i) t[w] += sh[w][i];
        }
        const double n0 = (double)k0, n1 = (double)k1;
        const double b0 = wave_sum(n0), b1 = wave_sum(n1);
        n_s[0][cl] = cl ? n0 : t[2] - b0;
        n_s[1][cl] = cl ? n1 : t[3] - b1;
        if (cl < 2) dc_s[cl] = t[cl];
    }
    __syncthreads();
    if (threadIdx.x >= kTaps) return;
    const Grid g{a.g.nz >> s, a.g.ny >> s, a.g.nx >> s};
    const double n = (double)ncells(g), inv = 1.0 / (double)(1u << (3 * s)), n27 = 27.0 * n;
    double S[3] = {0.0, 0.0, 0.0};
#pragma unroll 16
    for (uint32_t c = 0; c < kClasses; ++c) {
        const bool in = class_sees(c, o);
        S[0] += in ? n_s[0][c] : 0.0;
        S[1] += in ? n_s[1][c] : 0.0;
    }
    S[0] *= inv;
    S[1] *= inv;
    S[2] = n - S[0] - S[1];
    const double d0 = dc_s[0], d1 = dc_s[1];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        g1[c * kTaps + o] = old1[c] + d0 * S[c] / n27;
        g2[c * kTaps + o] = old2[c] + d1 * S[c] / n27;
    }
    if (o == 0) {   // Bbar
        g1[3 * kTaps] = old1[3] + d0;
        g2[3 * kTaps] = old2[3] + d1;
    }
}

// ---------------------------------------------------------------------------
// the loss
// ---------------------------------------------------------------------------
// The mixed-BC 7-point rows (Sec. "Spatial Discretization") of kZRun cells of one
// column each: row(z, v, A v) for z = z0 .. z0 + kZRun - 1 inside the grid, v
// the cell's value and label l.  A thread reads a cell and its four x/y
// neighbours straight from memory (the neighbours' lines are in the caches; the
// z neighbours are the column's own cells), all loads in flight: staged tiles
// with a full halo read 2.5 cells per cell behind two barriers (128^3: 22 and
// 18.5 us for the two kernels below).
constexpr int kZRun = 4;

template <class T, class Row>
__device__ __forceinline__ void seven_point_run(const uint8_t* __restrict__ lab, const T* __restrict__ v, Grid g, int x,
                                                int y, int z0, Row row) {
    constexpr int N = kZRun + 2;
    T c[N], nb[kZRun][4];
    uint8_t lc[N], ln[kZRun][4];
    const bool col = x < g.nx && y < g.ny;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int z = z0 - 1 + i;
        const bool in = col && z >= 0 && z < g.nz;
        const size_t q = in ? cell_index(g, z, y, x) : 0;
        c[i] = *at_or(v, q, in, pad_zero<T>());
        lc[i] = *at_or(lab, q, in, g_pad_solid);
    }
#pragma unroll
    for (int i = 0; i < kZRun; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int yy = y + (k == 0 ? -1 : k == 1 ? 1 : 0), xx = x + (k == 2 ? -1 : k == 3 ? 1 : 0);
            const bool in = col && in_grid(g, z0 + i, yy, xx);
            const size_t q = in ? cell_index(g, z0 + i, yy, xx) : 0;
            nb[i][k] = *at_or(v, q, in, pad_zero<T>());
            ln[i][k] = *at_or(lab, q, in, g_pad_solid);
        }
#pragma unroll
    for (int i = 0; i < kZRun; ++i) {
        if (!col || z0 + i >= g.nz) continue;
        T a = T(0);
        if (lc[i + 1] == kFluid) {   // neighbours in the order z-, z+, y-, y+, x-, x+
            const uint8_t l[6] = {lc[i], lc[i + 2], ln[i][0], ln[i][1], ln[i][2], ln[i][3]};
            const T n[6] = {c[i], c[i + 2], nb[i][0], nb[i][1], nb[i][2], nb[i][3]};
            int cnt = 0;
            T s = T(0);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                cnt += l[k] != kSolid;
                if (l[k] == kFluid) s += n[k];
            }
            a = (T)cnt * c[i + 1] - s;
        }
        row(z0 + i, lc[i + 1], a);
    }
}

// Runs of a grid: 64 x 4 columns by kZRun planes per block.
__host__ __device__ inline int seven_point_blocks(Grid g) {
    return ((g.nx + PX - 1) / PX) * ((g.ny + PY - 1) / PY) * ((g.nz + kZRun - 1) / kZRun);
}

template <class F>
__device__ __forceinline__ void seven_point_items(Grid g, F f) {
    const int ncx = (g.nx + PX - 1) / PX, ncy = (g.ny + PY - 1) / PY, n = seven_point_blocks(g);
    for (TileSpan sp = tile_span(n); sp.t0 < sp.t1; sp.t0 += sp.step)
        f(sp.t0 % ncx * PX + (int)threadIdx.x % PX, sp.t0 / ncx % ncy * PY + (int)threadIdx.x / PX,
          sp.t0 / (ncx * ncy) * kZRun);
}

// Training loss of one system: res = b - A y on fluid cells; partial ||res||^2.
template <class T>
__global__ __launch_bounds__(kBlock) void k_train_residual(const uint8_t* __restrict__ lab, Grid g,
                                                           const T* __restrict__ b, const T* __restrict__ y,
                                                           T* __restrict__ res, double* partials) {
    double v[kRedWidth] = {0.0, 0.0, 0.0, 0.0};
    seven_point_items(g, [&](int x, int yy, int z0) {
        T bv[kZRun];
#pragma unroll
        for (int i = 0; i < kZRun; ++i) {
            const bool in = x < g.nx && yy < g.ny && z0 + i < g.nz;
            bv[i] = *at_or(b, in ? cell_index(g, z0 + i, yy, x) : 0, in, pad_zero<T>());
        }
        seven_point_run<T>(lab, y, g, x, yy, z0, [&](int z, uint8_t l, T a) {
            T bz = bv[0];
#pragma unroll
            for (int i = 1; i < kZRun; ++i) bz = z == z0 + i ? bv[i] : bz;
            const T rv = l == kFluid ? bz - a : T(0);
            res[cell_index(g, z, yy, x)] = rv;
            v[0] += (double)rv * (double)rv;
        });
    });
    block_partials<kBlock>(v, partials);
}

// dL/dy = -w A res / ||res|| (A is symmetric), from the residual and its
// norm in st->rr; w weighs the system in a batch mean (1 alone).
template <class T>
__global__ __launch_bounds__(kBlock) void k_train_gy(const uint8_t* __restrict__ lab, Grid g, const T* __restrict__ res,
                                                     const State* st, T* __restrict__ gy, double w) {
    const T inv = (T)(-w / sqrt(st->rr));
    seven_point_items(g, [&](int x, int y, int z0) {
        seven_point_run<T>(lab, res, g, x, y, z0,
                           [&](int z, uint8_t, T a) { gy[cell_index(g, z, y, x)] = inv * a; });
    });
}

}  // namespace nps
