// lbm_strips.h -- four time steps of the D2Q9 TRT-R update per launch on strips that one wave owns
// (temporal blocking in registers, gfx950); launched by lbm_adjoint.hip, the translation unit that leaves
// the build time for it.
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
// FP16 storage on large lattices gives each lane two adjacent columns (strips of 120 columns: fewer
// lanes lost at the ends, half the lane shifts, one 4-byte access where 2-byte ones were).
//
// What bounds it: VALU issue for FP32 (2048^2: 97 vector instructions per node and step, issued 90 % of
// the time with three resident waves per SIMD at 140 VGPRs), memory and VALU about equally for FP64
// (256 VGPRs, two waves).  Against two steps per launch through an LDS ring (lbm_fused.hip): FP32
// 2048^2 131k -> 215k MLUPS, 8192^2 140k -> 221k, 256^2 24k -> 33k, FP64 2048^2 64k -> 119k, 8192^2 69k ->
// 126k; FP16 (VALU issue both ways) 8192^2 with D 180k -> 210k, with stochastic rounding 141k -> 150k,
// 1024^2 118k -> 139k.  Why T = 4: 56 columns start every strip on a 32-byte boundary; three steps need 58 (or waste
// two lanes) and measured 135k at 2048^2 FP32, because the stores of neighbouring strips then share
// 32-byte sectors; with six the carried values no longer fit the registers of FP64.
// Capping the registers for a fourth resident wave spills (2048^2 FP32 215k -> 168k).
#pragma once

#include <type_traits>

#include "lbm_internal.h"
#include "lbm_kernel_common.h"

namespace lbm {
namespace {

// The neighbouring lane's value: of lane - 1 (the columns to the west) and lane + 1 (east); the lanes at
// the wave's ends, which have no such neighbour, get 0.
template <int CTRL>
__device__ __forceinline__ uint32_t lane_shift(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int kFromWest = 0x138, kFromEast = 0x130;  // wave_shr:1, wave_shl:1

// The values of NC adjacent columns, which one lane owns.
template <class E, int NC>
struct Cols {
    E v[NC];
};
template <int CTRL, class E, int NC>
__device__ __forceinline__ Cols<E, NC> shift_words(Cols<E, NC> p)
{
    if constexpr (sizeof(Cols<E, NC>) == 8) {
        const uint64_t b = __builtin_bit_cast(uint64_t, p);
        return __builtin_bit_cast(Cols<E, NC>, (uint64_t)lane_shift<CTRL>((uint32_t)(b >> 32)) << 32 | lane_shift<CTRL>((uint32_t)b));
    } else if constexpr (sizeof(Cols<E, NC>) == 4) {
        return __builtin_bit_cast(Cols<E, NC>, lane_shift<CTRL>(__builtin_bit_cast(uint32_t, p)));
    } else {
        return __builtin_bit_cast(Cols<E, NC>, (uint16_t)lane_shift<CTRL>(__builtin_bit_cast(uint16_t, p)));
    }
}
// The values one column to the west and to the east.
template <class E, int NC>
__device__ __forceinline__ Cols<E, NC> west_of(Cols<E, NC> p)
{
    if constexpr (NC == 1) return shift_words<kFromWest>(p);
    else if constexpr (sizeof(E) == 4) return {__builtin_bit_cast(E, lane_shift<kFromWest>(__builtin_bit_cast(uint32_t, p.v[1]))), p.v[0]};
    else return {shift_words<kFromWest>(p).v[1], p.v[0]};
}
template <class E, int NC>
__device__ __forceinline__ Cols<E, NC> east_of(Cols<E, NC> p)
{
    if constexpr (NC == 1) return shift_words<kFromEast>(p);
    else if constexpr (sizeof(E) == 4) return {p.v[1], __builtin_bit_cast(E, lane_shift<kFromEast>(__builtin_bit_cast(uint32_t, p.v[0])))};
    else return {p.v[1], shift_words<kFromEast>(p).v[0]};
}
template <class E, int NC>
__device__ __forceinline__ Cols<E, NC> ld_cols(const E *base, unsigned byte_off)
{
    if constexpr (NC == 1) {
        return {ld_at(base, byte_off)};
    } else {
        typedef E vec __attribute__((ext_vector_type(NC)));
        return __builtin_bit_cast(Cols<E, NC>, *reinterpret_cast<const vec *>(reinterpret_cast<const char *>(base) + byte_off));
    }
}
template <bool CST, class E, int NC>
__device__ __forceinline__ void st_cols(E *base, unsigned byte_off, Cols<E, NC> p)
{
    if constexpr (NC == 1) {
        if constexpr (CST) st_at(base, byte_off, p.v[0]);
        else st_nt_at(base, byte_off, p.v[0]);
    } else {
        typedef E vec __attribute__((ext_vector_type(NC)));
        vec *to = reinterpret_cast<vec *>(reinterpret_cast<char *>(base) + byte_off);
        const vec v = __builtin_bit_cast(vec, p);
        if constexpr (CST) *to = v;
        else __builtin_nontemporal_store(v, to);
    }
}

// T steps of the output columns xs .. and rows y0 .. y1 - 1, reading buf[parity] and writing
// buf[parity ^ 1]; called by every lane of the wave.  UP: walks bottom to top (odd tile rows), so that
// vertically adjacent strips read the rows they share at about the same time, from L2.
// The loads of each row are issued one row ahead.  NC: columns per lane (2 needs an even nx, so that no
// lane's pair lies across the periodic seam and every pair is aligned).
template <int MODE, int AUX, bool HAS_K, bool HAS_S, int T, int NC, bool CST, bool UP>
__device__ __forceinline__ void strip_walk(const InstDesc &d, int parity, int xs, int y0, int y1, bool first)
{
    using St = typename ModeTraits<MODE>::St;
    using M = typename ModeTraits<MODE>::M;
    using E = typename St::T;
    using C = Codec<St, M>;
    using EC = Cols<E, NC>;
    using MC = Cols<M, NC>;
    constexpr int V = strip_width(T, NC);
    constexpr int dir = UP ? -1 : 1;
    constexpr bool kShiftPulls = NC > 1;  // the pulls' x-neighbours from the lanes, not from memory
    // populations moving along x are shifted to their reader's column when they are made, or, for FP16
    // codes, when they are read (1024^2 one column per lane: 129k -> 139k MLUPS)
    constexpr bool kLate = NC > 1 || is_f16_mode(MODE);
    const int nx = d.L.nx, ny = d.L.ny;
    const int64_t pitch = d.L.pitch;
    const int lane = (int)(threadIdx.x & 63u);
    int xi = (xs - T + lane * NC) % nx;  // the lane's first column
    xi = xi < 0 ? xi + nx : xi;
    const bool live = lane * NC >= T && lane * NC < T + V && xs + lane * NC - T < nx;
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
        EC g[9];
        MC ux, uy, k, s;
    };
    // row rc's pulls, k and s, and u of row ra
    auto fetch = [&](Loads &o) {
        // offsets re-read each row (an empty asm that claims to update them) keep every access a scalar
        // row base plus a 32-bit lane offset
        asm volatile("" : "+v"(bc), "+v"(bm), "+v"(bp), "+v"(fc));
        const int b = __builtin_amdgcn_readfirstlane(rb), c = __builtin_amdgcn_readfirstlane(rc),
                  a = __builtin_amdgcn_readfirstlane(ra);
        const E *__restrict__ pm = src + (int64_t)(UP ? a : b) * 9 * pitch;
        const E *__restrict__ pc = src + (int64_t)c * 9 * pitch;
        const E *__restrict__ pp = src + (int64_t)(UP ? b : a) * 9 * pitch;
        const unsigned ow = kShiftPulls ? bc : bm, oe = kShiftPulls ? bc : bp;
        o.g[0] = ld_cols<E, NC>(pc, bc);
        o.g[1] = ld_cols<E, NC>(pc + pitch, ow);
        o.g[2] = ld_cols<E, NC>(pm + 2 * pitch, bc);
        o.g[3] = ld_cols<E, NC>(pc + 3 * pitch, oe);
        o.g[4] = ld_cols<E, NC>(pp + 4 * pitch, bc);
        o.g[5] = ld_cols<E, NC>(pm + 5 * pitch, ow);
        o.g[6] = ld_cols<E, NC>(pm + 6 * pitch, oe);
        o.g[7] = ld_cols<E, NC>(pp + 7 * pitch, oe);
        o.g[8] = ld_cols<E, NC>(pp + 8 * pitch, ow);
        const M *__restrict__ ua = u + (int64_t)a * 2 * pitch;
        o.ux = ld_cols<M, NC>(ua, fc);
        o.uy = ld_cols<M, NC>(ua + pitch, fc);
        if (HAS_K) o.k = ld_cols<M, NC>(kf + (int64_t)c * pitch, fc);
        if (HAS_S) o.s = ld_cols<M, NC>(sf + (int64_t)c * pitch, fc);
    };

    // of one row: u, u_b d_b u_a, the source and the relaxation (R[j]: row r - j dir)
    struct RowData {
        MC ux, uy, bx, by, s;
        Relax<M> r[NC];
    };
    // of one step, codes at the lane's own columns: c from the last computed row (i = 0, 1, 3), b and o the
    // populations moving with the walk (vertical, from the west, from the east) of the last two rows
    struct Carry {
        EC c0, c1, c3, b0, bw, be, o0, ow, oe;
    };
    RowData R[T];
    Carry L[T > 1 ? T - 1 : 1];
    MC uxa, uya;  // u of the row ahead of the last one taken
    {
        const M *__restrict__ ub = u + (int64_t)__builtin_amdgcn_readfirstlane(rb) * 2 * pitch;
        const M *__restrict__ uc = u + (int64_t)__builtin_amdgcn_readfirstlane(rc) * 2 * pitch;
        R[0].ux = ld_cols<M, NC>(ub, fc);
        R[0].uy = ld_cols<M, NC>(ub + pitch, fc);
        uxa = ld_cols<M, NC>(uc, fc);
        uya = ld_cols<M, NC>(uc + pitch, fc);
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
            const MC xe = east_of(q.ux), xw = west_of(q.ux), ye = east_of(q.uy), yw = west_of(q.uy);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const M dxux = (xe.v[c] - xw.v[c]) * M(0.5);
                const M dxuy = (ye.v[c] - yw.v[c]) * M(0.5);
                const M dyux = ((UP ? R[1].ux : uxa).v[c] - (UP ? uxa : R[1].ux).v[c]) * M(0.5);
                const M dyuy = ((UP ? R[1].uy : uya).v[c] - (UP ? uya : R[1].uy).v[c]) * M(0.5);
                q.bx.v[c] = q.ux.v[c] * dxux + q.uy.v[c] * dyux;
                q.by.v[c] = q.ux.v[c] * dxuy + q.uy.v[c] * dyuy;
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            q.r[c] = HAS_K ? relax_from_k<M>(cur.k.v[c], lam, rconst.w3) : rconst;
            q.s.v[c] = HAS_S ? cur.s.v[c] : M(0);
        }
        EC p[9];  // what the step pulls (step 1: from memory)
#pragma unroll
        for (int i = 0; i < 9; ++i) p[i] = !kShiftPulls || kEx[i] == 0 ? cur.g[i] : (kEx[i] > 0 ? west_of(cur.g[i]) : east_of(cur.g[i]));
#pragma unroll
        for (int s = 1; s <= NS; ++s) {
            const RowData &n = R[s - 1];
            EC o[9];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                M g[9], P[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) g[i] = C::dec(p[i].v[c], i, d.f16);
                M Ax = M(0), Ay = M(0);
                if (AUX == 0) {
                    const M phi = g[0] + g[1] + g[2] + g[3] + g[4] + g[5] + g[6] + g[7] + g[8];
                    Ax = phi * n.bx.v[c];
                    Ay = phi * n.by.v[c];
                }
                collide<M, false>(g, n.ux.v[c], n.uy.v[c], n.r[c], Ax, Ay, n.s.v[c], P);
                const auto rbits = C::bits(d.f16, level + s, (int64_t)hist[s - 1] * nx, (unsigned)(xi + c));
#pragma unroll
                for (int i = 0; i < 9; ++i) o[i].v[c] = C::enc(P[i], i, d.f16, rbits);
            }
            if (s == T) {
                if (live) {
                    E *__restrict__ out = dst + (int64_t)__builtin_amdgcn_readfirstlane(y) * 9 * pitch;
#pragma unroll
                    for (int i = 0; i < 9; ++i) st_cols<CST>(out + i * pitch, bc, o[i]);
                }
            } else {
                const EC n1 = kLate ? o[1] : west_of(o[1]), n3 = kLate ? o[3] : east_of(o[3]);
                const EC n5 = kLate ? o[5] : west_of(o[5]), n6 = kLate ? o[6] : east_of(o[6]);
                const EC n8 = kLate ? o[8] : west_of(o[8]), n7 = kLate ? o[7] : east_of(o[7]);
                Carry &l = L[s - 1];
                if (s < NS) {  // step s + 1 pulls row r - s dir
                    const EC w5 = UP ? n5 : l.ow, e6 = UP ? n6 : l.oe, w8 = UP ? l.ow : n8, e7 = UP ? l.oe : n7;
                    p[0] = l.c0;
                    p[1] = kLate ? west_of(l.c1) : l.c1;
                    p[3] = kLate ? east_of(l.c3) : l.c3;
                    p[2] = UP ? o[2] : l.o0;
                    p[4] = UP ? l.o0 : o[4];
                    p[5] = kLate ? west_of(w5) : w5;
                    p[6] = kLate ? east_of(e6) : e6;
                    p[7] = kLate ? east_of(e7) : e7;
                    p[8] = kLate ? west_of(w8) : w8;
                }
                l.o0 = l.b0;
                l.ow = l.bw;
                l.oe = l.be;
                l.b0 = UP ? o[4] : o[2];
                l.bw = UP ? n8 : n5;
                l.be = UP ? n7 : n6;
                l.c0 = o[0];
                l.c1 = n1;
                l.c3 = n3;
            }
        }
    };
    // rows of the walk before the first output row: two more for each step
    const auto none = 0;
    row(std::integral_constant<int, 1>{}, none);
    row(std::integral_constant<int, 1>{}, none);
    row(std::integral_constant<int, 2>{}, none);
    row(std::integral_constant<int, 2>{}, none);
    row(std::integral_constant<int, 3>{}, none);
    row(std::integral_constant<int, 3>{}, none);
    static_assert(T == 4, "the rows before the first output row");
    constexpr std::integral_constant<int, T> all{};
    int y = UP ? y1 - 1 : y0;
    if constexpr (NC == 1) {  // unrolled by two: the rolled values are renamed, not copied
        int left = y1 - y0;
        for (; left > 1; left -= 2) {
            row(all, y);
            row(all, y + dir);
            y += 2 * dir;
        }
        if (left) row(all, y);
    } else {  // unrolled, two columns per lane would not fit 256 registers
#pragma unroll 1
        for (int left = y1 - y0; left > 0; --left, y += dir) row(all, y);
    }
}

// One instance: wave w of block b owns strip t % ns of tile row t / ns, t = 4 b + w in XCD row bands.
template <int MODE, int AUX, bool HAS_K, bool HAS_S, int T, int NC, bool CST>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NC == 2 ? 2 : 1)))
void strip_kernel(const StepArgs a, const int rows)
{
    const InstDesc &d = a.d;
    const int ns = (d.L.nx + strip_width(T, NC) - 1) / strip_width(T, NC);
    const int t = tile_of_block(blockIdx.x, gridDim.x, 1, 0, 0) * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int tr = t / ns, y0 = tr * rows, xs = (t - tr * ns) * strip_width(T, NC);
    if (y0 >= d.L.ny) return;
    const int y1 = min(y0 + rows, d.L.ny);
    if (tr & 1) strip_walk<MODE, AUX, HAS_K, HAS_S, T, NC, CST, true>(d, a.parity, xs, y0, y1, t == 0);
    else strip_walk<MODE, AUX, HAS_K, HAS_S, T, NC, CST, false>(d, a.parity, xs, y0, y1, t == 0);
}

template <int MODE, int AUX, int NC, bool CST>
hipError_t launch_strips_st(const StepArgs &a, int rows, hipStream_t st)
{
    constexpr int T = kStripSteps;
    const int64_t ns = (a.d.L.nx + strip_width(T, NC) - 1) / strip_width(T, NC);
    const int64_t nb = (ns * ((a.d.L.ny + rows - 1) / rows) + 3) / 4;
    if (nb > INT32_MAX / 4 || (NC == 2 && a.d.L.nx % 2 != 0)) return hipErrorInvalidValue;
    const bool hk = a.d.has_k, hs = a.d.has_s;
    if (hk && hs) strip_kernel<MODE, AUX, true, true, T, NC, CST><<<(int)nb, 256, 0, st>>>(a, rows);
    else if (hk) strip_kernel<MODE, AUX, true, false, T, NC, CST><<<(int)nb, 256, 0, st>>>(a, rows);
    else if (hs) strip_kernel<MODE, AUX, false, true, T, NC, CST><<<(int)nb, 256, 0, st>>>(a, rows);
    else strip_kernel<MODE, AUX, false, false, T, NC, CST><<<(int)nb, 256, 0, st>>>(a, rows);
    return hipGetLastError();
}

template <int MODE, int NC>
hipError_t launch_strips_mode(int aux, const StepArgs &a, const StripLaunch &s, hipStream_t st)
{
    switch (aux) {
    case 0: return s.cached ? launch_strips_st<MODE, 0, NC, true>(a, s.rows, st) : launch_strips_st<MODE, 0, NC, false>(a, s.rows, st);
    case 2: return s.cached ? launch_strips_st<MODE, 2, NC, true>(a, s.rows, st) : launch_strips_st<MODE, 2, NC, false>(a, s.rows, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_strips(int mode, int aux, const StepArgs &a, const StripLaunch &s, hipStream_t st)
{
    if (a.d.L.q != 9 || a.d.bckind != 0 || a.d.w3 != 0.0 || s.rows < 1 || a.d.buf[0] == a.d.buf[1])
        return hipErrorInvalidValue;
    if (s.cols == 2) {
        switch (mode) {
        case MODE_F16S_F32: return launch_strips_mode<MODE_F16S_F32, 2>(aux, a, s, st);
        case MODE_F16SR_F32: return launch_strips_mode<MODE_F16SR_F32, 2>(aux, a, s, st);
        default: return hipErrorInvalidValue;
        }
    }
    switch (mode) {
    case MODE_F64_F64: return launch_strips_mode<MODE_F64_F64, 1>(aux, a, s, st);
    case MODE_F64_F32: return launch_strips_mode<MODE_F64_F32, 1>(aux, a, s, st);
    case MODE_F32_F32: return launch_strips_mode<MODE_F32_F32, 1>(aux, a, s, st);
    case MODE_F16S_F32: return launch_strips_mode<MODE_F16S_F32, 1>(aux, a, s, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
