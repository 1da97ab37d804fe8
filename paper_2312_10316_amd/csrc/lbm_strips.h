// lbm_strips.h -- four time steps of the D2Q9 TRT-R update per launch on strips that one wave owns
// (temporal blocking in registers, gfx950); included by lbm_fused.hip.
//
// A wave walks a strip of 64 columns row by row (lane = column) and carries T steps at once: iteration
// r computes step 1 of row r from the state in memory, step 2 of row r - 1 from the step-1 values of
// rows r - 2 .. r, ..., step T of row r - T + 1, which it stores.  Everything between the steps stays in
// the wave's registers: the populations of one step that the next one pulls from rows already passed
// (9 values per step), and u, u . grad u, the relaxation and the source of the last T rows.  Values from
// the neighbouring columns come from the neighbouring lanes (DPP wave shifts), so there is no LDS ring,
// no barrier and no frame wave, and waves do not wait for each other.  The price is lanes and rows:
// each step takes one lane off either end of the wave (strips of 64 - 2 T output columns), and a strip
// of H rows computes T H + T (T - 1) node rows.
//
// Every node runs the one-step kernel's arithmetic (the same pulls, sums, collide; u_b d_b u_a of
// Eq. (16) is one subexpression there and is computed once per row here) and each step's populations
// go through the storage codec, so T steps are bitwise T single steps.
//
// What bounds it: VALU issue for FP32 (2048^2: 97 vector instructions per node and step, issued 90 % of
// the time with three resident waves per SIMD at 140 VGPRs), memory and VALU about equally for FP64
// (256 VGPRs, two waves).  Against two steps per launch through an LDS ring (lbm_fused.hip): FP32
// 2048^2 131k -> 215k MLUPS, 8192^2 140k -> 221k, 256^2 24k -> 33k, FP64 2048^2 64k -> 119k, 8192^2 69k ->
// 126k.  Why T = 4: 56 columns start every strip on a 32-byte boundary; three steps need 58 (or waste
// two lanes) and measured 135k at 2048^2 FP32, because the stores of neighbouring strips then share
// 32-byte sectors; with six the carried values no longer fit the registers of FP64.
// Capping the registers for a fourth resident wave spills (2048^2 FP32 215k -> 168k).
#pragma once

#include <type_traits>

#include "lbm_internal.h"
#include "lbm_kernel_common.h"

namespace lbm {
namespace {

// The neighbouring lane's value: of lane - 1 (the node to the west) and lane + 1 (east); the lanes at
// the wave's ends, which have no such neighbour, get 0.
template <class M>
__device__ __forceinline__ M lane_west(M v)
{
    if constexpr (sizeof(M) == 8) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x138, 0xf, 0xf, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x138, 0xf, 0xf, true);
        return __builtin_bit_cast(M, ((uint64_t)hi << 32) | lo);
    } else {
        return __builtin_bit_cast(M, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
    }
}
template <class M>
__device__ __forceinline__ M lane_east(M v)
{
    if constexpr (sizeof(M) == 8) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x130, 0xf, 0xf, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x130, 0xf, 0xf, true);
        return __builtin_bit_cast(M, ((uint64_t)hi << 32) | lo);
    } else {
        return __builtin_bit_cast(M, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
    }
}

// T steps of the output columns xs .. and rows y0 .. y1 - 1, reading buf[parity] and writing
// buf[parity ^ 1]; called by every lane of the wave.  UP: walks bottom to top (odd tile rows), so that
// vertically adjacent strips read the rows they share at about the same time, from L2.
// The loads of each row are issued one row ahead.
template <int MODE, int AUX, bool HAS_K, bool HAS_S, int T, bool CST, bool UP>
__device__ __forceinline__ void strip_walk(const InstDesc &d, int parity, int xs, int y0, int y1, bool first)
{
    using St = typename ModeTraits<MODE>::St;
    using M = typename ModeTraits<MODE>::M;
    using E = typename St::T;
    using C = Codec<St, M>;
    constexpr int V = strip_width(T);
    constexpr int dir = UP ? -1 : 1;
    const int nx = d.L.nx, ny = d.L.ny;
    const int64_t pitch = d.L.pitch;
    const int lane = (int)(threadIdx.x & 63u);
    int xi = (xs - T + lane) % nx;
    xi = xi < 0 ? xi + nx : xi;
    const bool live = lane >= T && lane < T + V && xs + lane - T < nx;
    const unsigned xm = xi == 0 ? (unsigned)nx - 1 : (unsigned)xi - 1;
    const unsigned xp = xi == nx - 1 ? 0u : (unsigned)xi + 1;
    unsigned bc = (unsigned)xi * (unsigned)sizeof(E), bm = xm * (unsigned)sizeof(E), bp = xp * (unsigned)sizeof(E);
    unsigned fc = (unsigned)xi * (unsigned)sizeof(M);
    const E *__restrict__ src = static_cast<const E *>(d.buf[parity]);
    E *__restrict__ dst = static_cast<E *>(d.buf[parity ^ 1]);
    const M *__restrict__ u = static_cast<const M *>(d.u);
    const M *__restrict__ kf = static_cast<const M *>(d.k);
    const M *__restrict__ sf = static_cast<const M *>(d.s);
    const M lam = (M)d.lambda;
    Relax<M> rconst;
    rconst.w1 = (M)d.w1;
    rconst.w2 = (M)d.w2;
    rconst.beta = (M)d.beta;
    rconst.w3 = (M)d.w3;
    const int64_t level = launch_level<C>(d, parity);
    advance_level<C>(d, parity, level, T, first && lane == 0);

    auto next_row = [ny](int r) { return UP ? wrap_dec(r, ny) : wrap_inc(r, ny); };
    // wrapped rows of the walk: behind, current, ahead
    int rb = (UP ? y1 - 1 + T : y0 - T) % ny;
    rb = rb < 0 ? rb + ny : rb;
    int rc = next_row(rb), ra = next_row(rc);
    int hist[T];  // wrapped rows r, r - dir, ... (stochastic rounding)

    struct Loads {
        E g[9];
        M ux, uy, k, s;
    };
    // row rc's pulls, k and s, and u of row ra
    auto fetch = [&](Loads &o) {
        asm volatile("" : "+v"(bc), "+v"(bm), "+v"(bp), "+v"(fc));
        const int b = __builtin_amdgcn_readfirstlane(rb), c = __builtin_amdgcn_readfirstlane(rc),
                  a = __builtin_amdgcn_readfirstlane(ra);
        const E *__restrict__ pm = src + (int64_t)(UP ? a : b) * 9 * pitch;
        const E *__restrict__ pc = src + (int64_t)c * 9 * pitch;
        const E *__restrict__ pp = src + (int64_t)(UP ? b : a) * 9 * pitch;
        o.g[0] = ld_at(pc, bc);
        o.g[1] = ld_at(pc + pitch, bm);
        o.g[2] = ld_at(pm + 2 * pitch, bc);
        o.g[3] = ld_at(pc + 3 * pitch, bp);
        o.g[4] = ld_at(pp + 4 * pitch, bc);
        o.g[5] = ld_at(pm + 5 * pitch, bm);
        o.g[6] = ld_at(pm + 6 * pitch, bp);
        o.g[7] = ld_at(pp + 7 * pitch, bp);
        o.g[8] = ld_at(pp + 8 * pitch, bm);
        const M *__restrict__ ua = u + (int64_t)a * 2 * pitch;
        o.ux = ld_at(ua, fc);
        o.uy = ld_at(ua + pitch, fc);
        if (HAS_K) o.k = ld_at(kf + (int64_t)c * pitch, fc);
        if (HAS_S) o.s = ld_at(sf + (int64_t)c * pitch, fc);
    };

    // of one row: u, u_b d_b u_a, the source and the relaxation (R[j]: row r - j dir)
    struct RowData {
        M ux, uy, bx, by, s;
        Relax<M> r;
    };
    // of one step, as its reader pulls them: c from the last computed row (i = 0, 1, 3), b and o the
    // populations moving with the walk (vertical, from the west, from the east) of the last two rows
    struct Carry {
        M c0, c1, c3, b0, bw, be, o0, ow, oe;
    };
    RowData R[T];
    Carry L[T > 1 ? T - 1 : 1];
    M uxa, uya;  // u of the row ahead of the last one taken
    {
        const M *__restrict__ ub = u + (int64_t)__builtin_amdgcn_readfirstlane(rb) * 2 * pitch;
        const M *__restrict__ uc = u + (int64_t)__builtin_amdgcn_readfirstlane(rc) * 2 * pitch;
        R[0].ux = ld_at(ub, fc);
        R[0].uy = ld_at(ub + pitch, fc);
        uxa = ld_at(uc, fc);
        uya = ld_at(uc + pitch, fc);
    }
    Loads nxt;
    fetch(nxt);

    auto row = [&](auto stages, const int y) __attribute__((always_inline)) {
        constexpr int NS = decltype(stages)::value;
#pragma unroll
        for (int j = T - 1; j > 0; --j) {
            R[j] = R[j - 1];
            hist[j] = hist[j - 1];
        }
        hist[0] = rc;
        const Loads cur = nxt;
        rb = rc;
        rc = ra;
        ra = next_row(ra);
        fetch(nxt);
        RowData &q = R[0];
        q.ux = uxa;
        q.uy = uya;
        uxa = cur.ux;
        uya = cur.uy;
        if (AUX == 0) {
            const M dxux = (lane_east(q.ux) - lane_west(q.ux)) * M(0.5);
            const M dxuy = (lane_east(q.uy) - lane_west(q.uy)) * M(0.5);
            const M dyux = ((UP ? R[1].ux : uxa) - (UP ? uxa : R[1].ux)) * M(0.5);
            const M dyuy = ((UP ? R[1].uy : uya) - (UP ? uya : R[1].uy)) * M(0.5);
            q.bx = q.ux * dxux + q.uy * dyux;
            q.by = q.ux * dxuy + q.uy * dyuy;
        }
        q.r = HAS_K ? relax_from_k<M>(cur.k, lam, rconst.w3) : rconst;
        q.s = HAS_S ? cur.s : M(0);
        M g[9], P[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) g[i] = C::dec(cur.g[i], i, d.f16);
#pragma unroll
        for (int s = 1; s <= NS; ++s) {
            const RowData &n = R[s - 1];
            M Ax = M(0), Ay = M(0);
            if (AUX == 0) {
                const M phi = g[0] + g[1] + g[2] + g[3] + g[4] + g[5] + g[6] + g[7] + g[8];
                Ax = phi * n.bx;
                Ay = phi * n.by;
            }
            collide<M, false>(g, n.ux, n.uy, n.r, Ax, Ay, n.s, P);
            const auto rbits = C::bits(d.f16, level + s, (int64_t)hist[s - 1] * nx, (unsigned)xi);
            if (s == T) {
                if (live) {
                    E *__restrict__ out = dst + (int64_t)__builtin_amdgcn_readfirstlane(y) * 9 * pitch;
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        if constexpr (CST) st_at(out + i * pitch, bc, C::enc(P[i], i, d.f16, rbits));
                        else st_nt_at(out + i * pitch, bc, C::enc(P[i], i, d.f16, rbits));
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < 9; ++i) P[i] = C::dec(C::enc(P[i], i, d.f16, rbits), i, d.f16);
                Carry &l = L[s - 1];
                const M n1 = lane_west(P[1]), n3 = lane_east(P[3]), n5 = lane_west(P[5]), n6 = lane_east(P[6]),
                        n7 = lane_east(P[7]), n8 = lane_west(P[8]);
                if (s < NS) {
                    g[0] = l.c0;
                    g[1] = l.c1;
                    g[3] = l.c3;
                    g[2] = UP ? P[2] : l.o0;
                    g[5] = UP ? n5 : l.ow;
                    g[6] = UP ? n6 : l.oe;
                    g[4] = UP ? l.o0 : P[4];
                    g[8] = UP ? l.ow : n8;
                    g[7] = UP ? l.oe : n7;
                }
                l.o0 = l.b0;
                l.ow = l.bw;
                l.oe = l.be;
                l.b0 = UP ? P[4] : P[2];
                l.bw = UP ? n8 : n5;
                l.be = UP ? n7 : n6;
                l.c0 = P[0];
                l.c1 = n1;
                l.c3 = n3;
            }
        }
    };
    // rows of the walk before the first output row: two more for each step
    const auto none = 0;
    row(std::integral_constant<int, 1>{}, none);
    if constexpr (T > 1) row(std::integral_constant<int, 1>{}, none);
    if constexpr (T > 2) {
        row(std::integral_constant<int, 2>{}, none);
        row(std::integral_constant<int, 2>{}, none);
    }
    if constexpr (T > 3) {
        row(std::integral_constant<int, 3>{}, none);
        row(std::integral_constant<int, 3>{}, none);
    }
    if constexpr (T > 4) {
        row(std::integral_constant<int, 4>{}, none);
        row(std::integral_constant<int, 4>{}, none);
    }
    constexpr std::integral_constant<int, T> all{};
    int y = UP ? y1 - 1 : y0;
    int left = y1 - y0;
    for (; left > 1; left -= 2) {
        row(all, y);
        row(all, y + dir);
        y += 2 * dir;
    }
    if (left) row(all, y);
}

// One instance: wave w of block b owns strip t % ns of tile row t / ns, t = 4 b + w in XCD row bands.
template <int MODE, int AUX, bool HAS_K, bool HAS_S, int T, bool CST>
__global__ __launch_bounds__(256) void strip_kernel(const StepArgs a, const int rows)
{
    const InstDesc &d = a.d;
    const int ns = (d.L.nx + strip_width(T) - 1) / strip_width(T);
    const int t = tile_of_block(blockIdx.x, gridDim.x, 1, 0, 0) * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int tr = t / ns, y0 = tr * rows, xs = (t - tr * ns) * strip_width(T);
    if (y0 >= d.L.ny) return;
    const int y1 = min(y0 + rows, d.L.ny);
    if (tr & 1) strip_walk<MODE, AUX, HAS_K, HAS_S, T, CST, true>(d, a.parity, xs, y0, y1, t == 0);
    else strip_walk<MODE, AUX, HAS_K, HAS_S, T, CST, false>(d, a.parity, xs, y0, y1, t == 0);
}

}  // namespace
}  // namespace lbm
