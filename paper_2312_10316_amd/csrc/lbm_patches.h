// lbm_patches.h -- several time steps of the D2Q9 TRT-R update per launch on small lattices (temporal
// blocking over a block's waves, gfx950); launched by lbm_kernels3d.hip, a translation unit that leaves the
// build time for it.
#pragma once

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "lbm_internal.h"
#include "lbm_kernel_common.h"

namespace lbm {
namespace {

// A strip's wave (lbm_strips.h) computes its rows one after the other, which a small lattice cannot hide: at
// 256^2 the chip holds one wave per SIMD, and a lone wave issues an instruction every 7.7 cycles.  Here a block
// of NW waves takes a patch of NW R rows at once (R rows per wave, lane = column, R nodes per lane for all T steps, so u, u .
// grad u, D and S are read once): H = NW R - 2 (T - 1) output rows of 64 - 2 T columns.  Between two steps the
// populations moving along y go to the neighbouring waves through LDS (two buffers, one barrier per step), those
// moving along x only come from the neighbouring lanes.  A step takes one row and one column off the patch's
// edges; waves whose rows are no longer needed only keep the barrier.  The same work per output row as a strip
// of H rows.  Two rows per wave halve the exchange and recompute less (24 rows for 18, not 16 for 10), at one
// block per CU instead of two.  What bounds it: the launch (about 2 us in a replayed graph) and T times the
// latency of a node update and the exchange.  Us per step, strips / patches: FP64 64^2 1.96 / 1.17, FP32 128^2
// 1.80 / 0.99, 256^2 2.11 / 1.33, 512^2 3.73 / 2.62, 1000^2 7.15 / 5.79, FP16 with
// stochastic rounding 300^2 3.96 / 2.14.
// Bitwise T single steps, as the strips.
// IMG: every step's state is stored, image_bytes apart from buf[parity ^ 1] on (the adjoint's recomputation).
template <int MODE, int AUX, bool HAS_K, bool HAS_S, int T, int NW, int R, int BC, bool IMG = false>
__global__ __launch_bounds__(64 * NW) void patch_kernel(const StepArgs sa, const int64_t image_bytes)
{
    using St = typename ModeTraits<MODE>::St;
    using M = typename ModeTraits<MODE>::M;
    using E = typename St::T;
    using C = Codec<St, M>;
    using X = std::conditional_t<sizeof(E) == 2, E, M>;  // a value in LDS: the code, or what it decodes to
    constexpr int V = strip_width(T, 1), H = NW * R - 2 * (T - 1);
    static_assert(H >= 1, "no output row");
    __shared__ X xch[2][6 * NW * 64 + 2];  // one spare element at either end (lanes without a neighbour)
    const InstDesc &d = sa.d;
    const int nx = d.L.nx, ny = d.L.ny;
    const int64_t pitch = d.L.pitch;
    const int ns = (nx + V - 1) / V;
    const int t = tile_of_block(blockIdx.x, gridDim.x, 1, 0, 0);
    const int tr = t / ns, xs = (t - tr * ns) * V;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63u);
    int xi = (xs - T + lane) % nx;
    xi = xi < 0 ? xi + nx : xi;
    const bool live = lane >= T && lane < T + V && xs + lane - T < nx;
    const unsigned xm = xi == 0 ? (unsigned)nx - 1 : (unsigned)xi - 1, xp = xi == nx - 1 ? 0u : (unsigned)xi + 1;
    const unsigned bc = (unsigned)xi * (unsigned)sizeof(E), bm = xm * (unsigned)sizeof(E), bp = xp * (unsigned)sizeof(E);
    const unsigned fc = (unsigned)xi * (unsigned)sizeof(M);
    const E *__restrict__ src = static_cast<const E *>(d.buf[sa.parity]);
    const M *__restrict__ u = static_cast<const M *>(d.u);
    const int64_t level = launch_level<C>(d, sa.parity);
    advance_level<C>(d, sa.parity, level, T, t == 0 && threadIdx.x == 0);
    const F16Params &f = d.f16;

    // row k of the wave is row w R + k of the patch, lattice row y[k]
    int y[R];
    M g[R][9], P[R][9], ux[R], uy[R], bx[R], by[R], s[R], phiw[R];  // (bx, by): u_b d_b u_a
    Relax<M> r[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int yr = (tr * H - (T - 1) + w * R + k) % ny;
        y[k] = __builtin_amdgcn_readfirstlane(yr < 0 ? yr + ny : yr);
        const int ym = wrap_dec(y[k], ny), yp = wrap_inc(y[k], ny);
        const E *__restrict__ pm = src + (int64_t)ym * 9 * pitch, *__restrict__ pc = src + (int64_t)y[k] * 9 * pitch,
                *__restrict__ pp = src + (int64_t)yp * 9 * pitch;
        g[k][0] = C::dec(ld_at(pc, bc), 0, f);
        g[k][1] = C::dec(ld_at(pc + pitch, bm), 1, f);
        g[k][2] = C::dec(ld_at(pm + 2 * pitch, bc), 2, f);
        g[k][3] = C::dec(ld_at(pc + 3 * pitch, bp), 3, f);
        g[k][4] = C::dec(ld_at(pp + 4 * pitch, bc), 4, f);
        g[k][5] = C::dec(ld_at(pm + 5 * pitch, bm), 5, f);
        g[k][6] = C::dec(ld_at(pm + 6 * pitch, bp), 6, f);
        g[k][7] = C::dec(ld_at(pp + 7 * pitch, bp), 7, f);
        g[k][8] = C::dec(ld_at(pp + 8 * pitch, bm), 8, f);
        if constexpr (BC == 2)
#pragma unroll
            for (int i = 2; i < 9; ++i) P[k][i] = C::dec(ld_at(pc + i * pitch, bc), i, f);
        const M *__restrict__ uc = u + (int64_t)y[k] * 2 * pitch;
        ux[k] = ld_at(uc, fc);
        uy[k] = ld_at(uc + pitch, fc);
        if (AUX == 0) {
            const bool bot = BC == 2 && y[k] == 0, top = BC == 2 && y[k] == ny - 1;  // one-sided next to a wall
            const M *__restrict__ un = u + (int64_t)(top ? y[k] : yp) * 2 * pitch, *__restrict__ us = u + (int64_t)(bot ? y[k] : ym) * 2 * pitch;
            const M hy = bot || top ? M(1) : M(0.5);
            const M dxux = (lane_e(ux[k]) - lane_w(ux[k])) * M(0.5);
            const M dxuy = (lane_e(uy[k]) - lane_w(uy[k])) * M(0.5);
            const M dyux = (ld_at(un, fc) - ld_at(us, fc)) * hy;
            const M dyuy = (ld_at(un + pitch, fc) - ld_at(us + pitch, fc)) * hy;
            bx[k] = ux[k] * dxux + uy[k] * dyux;
            by[k] = ux[k] * dxuy + uy[k] * dyuy;
        }
        r[k].w1 = (M)d.w1;
        r[k].w2 = (M)d.w2;
        r[k].beta = (M)d.beta;
        r[k].w3 = (M)d.w3;
        if (HAS_K) r[k] = relax_from_k<M>(ld_at(static_cast<const M *>(d.k) + (int64_t)y[k] * pitch, fc), (M)d.lambda, (M)d.w3);
        s[k] = HAS_S ? ld_at(static_cast<const M *>(d.s) + (int64_t)y[k] * pitch, fc) : M(0);
        phiw[k] = BC == 2 && (y[k] == 0 || y[k] == ny - 1) ? ld_at(static_cast<const M *>(d.bc) + (int64_t)y[k] * pitch, fc) : M(0);
    }
    // the exchange: plane p, wave v, lane
    auto at = [&](int p, int v) { return 1 + (p * NW + v) * 64 + lane; };
    const int wm = max(w - 1, 0), wp = min(w + 1, NW - 1);
#pragma unroll
    for (int n = 1; n <= T; ++n) {
        if (w * R + R - 1 >= n - 1 && w * R <= NW * R - n) {
            X c[R][9];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                if constexpr (BC == 2)
                    if (y[k] == 0 || y[k] == ny - 1) {
                        const bool bottom = y[k] == 0;
                        wall_reflect<M>(phiw[k], ux[k], uy[k], bottom, bottom ? P[k][4] : P[k][2], bottom ? P[k][7] : P[k][5],
                                        bottom ? P[k][8] : P[k][6], g[k]);
                    }
                M Ax = M(0), Ay = M(0);
                if (AUX == 0) {
                    const M phi = g[k][0] + g[k][1] + g[k][2] + g[k][3] + g[k][4] + g[k][5] + g[k][6] + g[k][7] + g[k][8];
                    Ax = phi * bx[k];
                    Ay = phi * by[k];
                }
                collide<M, false>(g[k], ux[k], uy[k], r[k], Ax, Ay, s[k], P[k]);
                const auto rb = C::bits(f, level + n, (int64_t)y[k] * nx, (unsigned)xi);
                if (IMG || n == T) {
                    const int v = w * R + k - (T - 1);  // output row of the patch
                    if (live && v >= 0 && v < H && tr * H + v < ny) {
                        E *__restrict__ o = reinterpret_cast<E *>(static_cast<char *>(d.buf[sa.parity ^ 1]) + (IMG ? n - 1 : 0) * image_bytes) + (int64_t)y[k] * 9 * pitch;
#pragma unroll
                        for (int i = 0; i < 9; ++i) st_at(o + i * pitch, bc, C::enc(P[k][i], i, f, rb));
                    }
                }
                if (n < T)
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        const E e = C::enc(P[k][i], i, f, rb);
                        P[k][i] = C::dec(e, i, f);
                        if constexpr (sizeof(E) == 2) c[k][i] = e;
                        else c[k][i] = P[k][i];
                    }
            }
            if (n < T) {
                X *x = xch[n & 1];
                x[at(0, w)] = c[R - 1][2];
                x[at(1, w)] = c[R - 1][5];
                x[at(2, w)] = c[R - 1][6];
                x[at(3, w)] = c[0][4];
                x[at(4, w)] = c[0][7];
                x[at(5, w)] = c[0][8];
            }
        }
        if (n == T) break;
        __syncthreads();
        if (w * R + R - 1 >= n && w * R <= NW * R - 1 - n) {
            const X *x = xch[n & 1];
            auto val = [&](int i, int p, int v, int dx) {
                if constexpr (sizeof(E) == 2) return C::dec(x[at(p, v) + dx], i, f);
                else return x[at(p, v) + dx];
            };
#pragma unroll
            for (int k = 0; k < R; ++k) {
                g[k][0] = P[k][0];
                g[k][1] = lane_w(P[k][1]);
                g[k][3] = lane_e(P[k][3]);
                if (k == 0) {
                    g[k][2] = val(2, 0, wm, 0);
                    g[k][5] = val(5, 1, wm, -1);
                    g[k][6] = val(6, 2, wm, 1);
                } else {
                    g[k][2] = P[k - 1][2];
                    g[k][5] = lane_w(P[k - 1][5]);
                    g[k][6] = lane_e(P[k - 1][6]);
                }
                if (k == R - 1) {
                    g[k][4] = val(4, 3, wp, 0);
                    g[k][7] = val(7, 4, wp, 1);
                    g[k][8] = val(8, 5, wp, -1);
                } else {
                    g[k][4] = P[k + 1][4];
                    g[k][7] = lane_e(P[k + 1][7]);
                    g[k][8] = lane_w(P[k + 1][8]);
                }
            }
        }
    }
}

template <int MODE, int AUX, int T, int NW, int R, int BC, bool IMG = false>
hipError_t launch_patches_st(const StepArgs &a, hipStream_t st, int64_t image_bytes = 0)
{
    constexpr int V = strip_width(T, 1), H = NW * R - 2 * (T - 1);
    const int64_t nb = (int64_t)((a.d.L.nx + V - 1) / V) * ((a.d.L.ny + H - 1) / H);
    if (nb > INT32_MAX / 16) return hipErrorInvalidValue;
    const bool hk = a.d.has_k, hs = a.d.has_s;
    if (hk && hs) patch_kernel<MODE, AUX, true, true, T, NW, R, BC, IMG><<<(int)nb, 64 * NW, 0, st>>>(a, image_bytes);
    else if (hk) patch_kernel<MODE, AUX, true, false, T, NW, R, BC, IMG><<<(int)nb, 64 * NW, 0, st>>>(a, image_bytes);
    else if (hs) patch_kernel<MODE, AUX, false, true, T, NW, R, BC, IMG><<<(int)nb, 64 * NW, 0, st>>>(a, image_bytes);
    else patch_kernel<MODE, AUX, false, false, T, NW, R, BC, IMG><<<(int)nb, 64 * NW, 0, st>>>(a, image_bytes);
    return hipGetLastError();
}

template <int MODE, int AUX, int BC>
hipError_t launch_patches_kind(const StepArgs &a, const StripLaunch &s, hipStream_t st)
{
    if (s.steps == 8 && s.patch == 16 && s.rows == 1) return launch_patches_st<MODE, AUX, 8, 16, 1, BC>(a, st);
    if (s.steps == 4 && s.patch == 12 && s.rows == 1) return launch_patches_st<MODE, AUX, 4, 12, 1, BC>(a, st);
    if (s.steps == 4 && s.patch == 16 && s.rows == 1) return launch_patches_st<MODE, AUX, 4, 16, 1, BC>(a, st);
    if constexpr (BC == 0) {
        if (s.steps == 4 && s.patch == 12 && s.rows == 2) return launch_patches_st<MODE, AUX, 4, 12, 2, BC>(a, st);
        if (s.steps == 4 && s.patch == 16 && s.rows == 2) return launch_patches_st<MODE, AUX, 4, 16, 2, BC>(a, st);
    }
    return hipErrorInvalidValue;
}

template <int MODE>
hipError_t launch_patches_mode(int aux, const StepArgs &a, const StripLaunch &s, hipStream_t st)
{
    if (a.d.bckind == 2) return aux == 0 ? launch_patches_kind<MODE, 0, 2>(a, s, st) : launch_patches_kind<MODE, 2, 2>(a, s, st);
    return aux == 0 ? launch_patches_kind<MODE, 0, 0>(a, s, st) : launch_patches_kind<MODE, 2, 0>(a, s, st);
}

template <int MODE, int AUX>
hipError_t launch_patch_images_kind(const StepArgs &a, int waves, int64_t image_bytes, hipStream_t st)
{
    if (waves == 12) return launch_patches_st<MODE, AUX, kPatchImages, 12, 1, 0, true>(a, st, image_bytes);
    if (waves == 16) return launch_patches_st<MODE, AUX, kPatchImages, 16, 1, 0, true>(a, st, image_bytes);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_patches(int mode, int aux, const StepArgs &a, const StripLaunch &s, hipStream_t st)
{
    if (a.d.L.q != 9 || a.d.bckind == 1 || a.d.w3 != 0.0 || aux == 1 || a.d.buf[0] == a.d.buf[1]) return hipErrorInvalidValue;
    switch (mode) {
    case MODE_F64_F64: return launch_patches_mode<MODE_F64_F64>(aux, a, s, st);
    case MODE_F64_F32: return launch_patches_mode<MODE_F64_F32>(aux, a, s, st);
    case MODE_F32_F32: return launch_patches_mode<MODE_F32_F32>(aux, a, s, st);
    case MODE_F16S_F32: return launch_patches_mode<MODE_F16S_F32>(aux, a, s, st);
    case MODE_F16SR_F32: return launch_patches_mode<MODE_F16SR_F32>(aux, a, s, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_patch_images(int mode, int aux, const StepArgs &a, int waves, int64_t image_bytes, hipStream_t st)
{
    if (a.d.L.q != 9 || a.d.bckind != 0 || a.d.w3 != 0.0 || aux == 1 || a.d.buf[0] == a.d.buf[1]) return hipErrorInvalidValue;
    switch (mode) {
    case MODE_F64_F64: return aux == 0 ? launch_patch_images_kind<MODE_F64_F64, 0>(a, waves, image_bytes, st) : launch_patch_images_kind<MODE_F64_F64, 2>(a, waves, image_bytes, st);
    case MODE_F64_F32: return aux == 0 ? launch_patch_images_kind<MODE_F64_F32, 0>(a, waves, image_bytes, st) : launch_patch_images_kind<MODE_F64_F32, 2>(a, waves, image_bytes, st);
    case MODE_F32_F32: return aux == 0 ? launch_patch_images_kind<MODE_F32_F32, 0>(a, waves, image_bytes, st) : launch_patch_images_kind<MODE_F32_F32, 2>(a, waves, image_bytes, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
