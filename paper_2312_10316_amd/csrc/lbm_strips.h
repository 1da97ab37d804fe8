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
// What bounds it: VALU issue for FP32 (2048^2: 133 vector instructions per node and step, the recomputed rows and
// lanes included, busy on 0.67 of the launch's cycles; the flux form 232 and 0.90) and FP16 (two columns per lane,
// 8192^2: 157 and all cycles), memory and the latency of two waves per SIMD for FP64 (188 VGPRs; VALU on 0.45 of the
// cycles, 4.6 TB/s).  The rows before the
// first output row run in a loop of their own with the steps that have no row yet skipped by uniform
// branches; as straight code they had cost 40 VGPRs (FP32 140 -> 100).
// Against two steps per launch through an LDS ring (lbm_fused.hip), in MLUPS of long runs of the rotating pulse (one
// card and day differs from another by up to 10 %, a dense field of FP16 codes from the pulse by 7 %): FP32 2048^2
// 131k -> 200k, 8192^2 140k -> 218k, FP64 2048^2 64k -> 116k, 8192^2 69k -> 125k; flux form FP32 2048^2 99k -> 153k,
// 8192^2 114k -> 194k, FP64 2048^2 55k -> 80k (T = 2, 56 columns, 4096^2: 63k, 83k with four); FP16 (VALU issue both
// ways) 8192^2 204k -> 248k, with D 180k -> 219k and, with stochastic rounding, 141k -> 152k (without D tiles are the
// faster).  Lattices up to about 1200^2 run on patches (lbm_patches.h).
// Why T = 4: 56 columns start every strip of FP32 and FP64 on a 32-byte boundary; three steps need 58 (or waste two
// lanes) and measured 135k at 2048^2 FP32, because the stores of neighbouring strips then share 32-byte sectors; with
// six the carried values no longer fit the registers of FP64.  FP16 strips share sectors all the same (56 columns are
// 112 bytes, 120 are 240): they are bound by issue, and whole sectors (48 or 112 columns) would cost lanes.
#pragma once

#include <type_traits>

#include "lbm_internal.h"
#include "lbm_kernel_common.h"

namespace lbm {
namespace {

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
// lane's pair lies across the periodic seam and every pair is aligned).  BC: 0 periodic, 2 walls.
//
// Flux form (AUX 1): a step's collision at row y needs phi of its pulls at rows y - 1 and y + 1 and in the
// two neighbouring columns, so each step pulls one row ahead of the row it collides (two rows of lag and
// two columns off either end of the wave per step instead of one).
//
// Walls (BC 2): the rows beyond a wall wrap to the other side of the lattice and are computed for
// nothing; the rows next to a wall replace what would come from there by the reflection (wall_reflect).
template <int MODE, int AUX, bool HAS_K, bool HAS_S, int T, int NC, bool CST, bool UP, int BC = 0>
__device__ __forceinline__ void strip_walk(const InstDesc &d, int parity, int xs, int y0, int y1, bool first)
{
    using St = typename ModeTraits<MODE>::St;
    using M = typename ModeTraits<MODE>::M;
    using E = typename St::T;
    using C = Codec<St, M>;
    using EC = Cols<E, NC>;
    using MC = Cols<M, NC>;
    constexpr bool kFlux = AUX == 1;
    static_assert(NC == 1 || (!kFlux && BC == 0), "two columns per lane: local or no aux term, periodic");
    constexpr int G = kFlux ? 2 * T : T;     // columns lost at either end; also the rows the walk starts before y0
    constexpr int V = strip_width(G, NC);
    constexpr int dir = UP ? -1 : 1;
    constexpr int ND = kFlux ? 2 * T + 1 : T;  // rows of per-row data kept
    constexpr bool kShiftPulls = NC > 1;     // the pulls' x-neighbours from the lanes, not from memory
    // populations moving along x are shifted to their reader's column when they are made, or, for FP16
    // codes, when they are read (1024^2 one column per lane: 129k -> 139k MLUPS); walls need them unshifted
    constexpr bool kLate = NC > 1 || is_f16_mode(MODE) || BC == 2;
    const int nx = d.L.nx, ny = d.L.ny;
    const int64_t pitch = d.L.pitch;
    const int lane = (int)(threadIdx.x & 63u);
    int xi = (xs - G + lane * NC) % nx;  // the lane's first column
    xi = xi < 0 ? xi + nx : xi;
    const bool live = lane * NC >= G && lane * NC < G + V && xs + lane * NC - G < nx;
    const unsigned xm = xi == 0 ? (unsigned)nx - 1 : (unsigned)xi - 1;
    const unsigned xp = xi == nx - 1 ? 0u : (unsigned)xi + 1;
    unsigned bc = (unsigned)xi * (unsigned)sizeof(E), bm = xm * (unsigned)sizeof(E), bp = xp * (unsigned)sizeof(E);
    unsigned fc = (unsigned)xi * (unsigned)sizeof(M);
    const E *__restrict__ src = static_cast<const E *>(d.buf[parity]);
    E *__restrict__ dst = static_cast<E *>(d.buf[parity ^ 1]);
    const M *__restrict__ u = static_cast<const M *>(d.u);
    const M *__restrict__ kf = static_cast<const M *>(d.k);
    const M *__restrict__ sf = static_cast<const M *>(d.s);
    const M *__restrict__ wall = static_cast<const M *>(d.bc);
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
    int rb = (UP ? y1 - 1 + G : y0 - G) % ny;
    rb = rb < 0 ? rb + ny : rb;
    int rc = next_row(rb), ra = next_row(rc);
    int hist[ND];  // wrapped rows r, r - dir, ...

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

    // of one row (R[j]: row r - j dir): u, u_b d_b u_a (local aux term), the source and the relaxation (the
    // flux form keeps twice the rows and only k, from which each step computes it)
    struct RowData {
        MC ux, uy, bx, by, s, k;
        Relax<M> r[NC];
    };
    // of one step: c from the last computed row (i = 0, 1, 3), b and o the populations moving with the walk
    // (vertical, from the west, from the east) of the last two rows, a (walls) those moving against it
    struct Carry {
        EC c0, c1, c3, b0, bw, be, o0, ow, oe, a0, aw, ae;
    };
    // of one step in the flux form: the last pulled row's populations, phi of it and of the row before
    struct Ahead {
        M g[9], phi, phi_b;
    };
    RowData R[ND];
    Carry L[T > 1 ? T - 1 : 1];
    Ahead F[kFlux ? T : 1];
    MC uxa, uya;  // u of the row ahead of the last one taken
    {
        const M *__restrict__ ub = u + (int64_t)__builtin_amdgcn_readfirstlane(rb) * 2 * pitch;
        const M *__restrict__ uc = u + (int64_t)__builtin_amdgcn_readfirstlane(rc) * 2 * pitch;
        R[0].ux = ld_cols<M, NC>(ub, fc);
        R[0].uy = ld_cols<M, NC>(ub + pitch, fc);
        uxa = ld_cols<M, NC>(uc, fc);
        uya = ld_cols<M, NC>(uc + pitch, fc);
        hist[0] = rb;
    }
    Loads nxt;
    fetch(nxt);

    // One iteration.  `all`: every step has its rows (the walk's first rows run fewer steps: step s pulls
    // from iteration `lag` (s - 1) on; the flux form collides two iterations later); y: the output row.
    constexpr int lag = kFlux ? 4 : 2;
    auto row = [&](auto all, const int k, const int y) __attribute__((always_inline)) {
        constexpr bool ALL = decltype(all)::value;
#pragma unroll
        for (int j = ND - 1; j > 0; --j) {
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
            MC un = UP ? R[1].ux : uxa, us = UP ? uxa : R[1].ux, vn = UP ? R[1].uy : uya, vs = UP ? uya : R[1].uy;
            M hy = M(0.5);
            if constexpr (BC == 2) {  // one-sided next to a wall
                if (hist[0] == 0) { us = q.ux; vs = q.uy; hy = M(1); }
                else if (hist[0] == ny - 1) { un = q.ux; vn = q.uy; hy = M(1); }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const M dxux = (xe.v[c] - xw.v[c]) * M(0.5);
                const M dxuy = (ye.v[c] - yw.v[c]) * M(0.5);
                const M dyux = (un.v[c] - us.v[c]) * hy;
                const M dyuy = (vn.v[c] - vs.v[c]) * hy;
                q.bx.v[c] = q.ux.v[c] * dxux + q.uy.v[c] * dyux;
                q.by.v[c] = q.ux.v[c] * dxuy + q.uy.v[c] * dyuy;
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (HAS_K && kFlux) q.k.v[c] = cur.k.v[c];
            else q.r[c] = HAS_K ? relax_from_k<M>(cur.k.v[c], lam, rconst.w3) : rconst;
            q.s.v[c] = HAS_S ? cur.s.v[c] : M(0);
        }
        EC p[9];  // what the step pulls (step 1: from memory)
#pragma unroll
        for (int i = 0; i < 9; ++i) p[i] = !kShiftPulls || kEx[i] == 0 ? cur.g[i] : (kEx[i] > 0 ? west_of(cur.g[i]) : east_of(cur.g[i]));
        EC own[9];  // walls: the node's own values of the step before (i = 2, 4, 5, 6, 7, 8)
        if constexpr (BC == 2) {
            if (hist[0] == 0 || hist[0] == ny - 1) {
                const E *__restrict__ pc = src + (int64_t)__builtin_amdgcn_readfirstlane(hist[0]) * 9 * pitch;
#pragma unroll
                for (int i = 2; i < 9; ++i) own[i] = ld_cols<E, NC>(pc + i * pitch, bc);
            }
        }
        // step s of its rows, from what it pulls (p); leaves what step s + 1 pulls in p
        auto step = [&](auto which) __attribute__((always_inline)) {
            constexpr int s = decltype(which)::value;
            constexpr int jc = kFlux ? 2 * s - 1 : s - 1;  // the row it collides is r - jc dir
            EC o[9];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const RowData &n = R[jc];
                M g[9], P[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) g[i] = C::dec(p[i].v[c], i, d.f16);
                if constexpr (BC == 2) {
                    const int yr = hist[s - 1];
                    if (yr == 0 || yr == ny - 1) {
                        const bool bottom = yr == 0;
                        const M p2 = bottom ? C::dec(own[4].v[c], 4, d.f16) : C::dec(own[2].v[c], 2, d.f16);
                        const M p5 = bottom ? C::dec(own[7].v[c], 7, d.f16) : C::dec(own[5].v[c], 5, d.f16);
                        const M p6 = bottom ? C::dec(own[8].v[c], 8, d.f16) : C::dec(own[6].v[c], 6, d.f16);
                        wall_reflect<M>(ld_at(wall + (int64_t)__builtin_amdgcn_readfirstlane(yr) * pitch, fc), n.ux.v[c],
                                        n.uy.v[c], bottom, p2, p5, p6, g);
                    }
                }
                M Ax = M(0), Ay = M(0);
                if constexpr (AUX != 2) {
                    const M phi = g[0] + g[1] + g[2] + g[3] + g[4] + g[5] + g[6] + g[7] + g[8];
                    if constexpr (AUX == 0) {
                        Ax = phi * n.bx.v[c];
                        Ay = phi * n.by.v[c];
                    } else {  // collide the row pulled last, then take this one
                        Ahead &f = F[s - 1];
                        const RowData &nb = R[jc + 1], &na = R[jc - 1];  // behind and ahead
                        const M uxw = lane_w(n.ux.v[0]), uyw = lane_w(n.uy.v[0]), uxe = lane_e(n.ux.v[0]), uye = lane_e(n.uy.v[0]);
                        const M pw = lane_w(f.phi), pe = lane_e(f.phi);
                        const RowData &ns = UP ? na : nb, &nn = UP ? nb : na;
                        flux_aux<M>(pw, pe, UP ? phi : f.phi_b, UP ? f.phi_b : phi, uxw, uyw, uxe, uye, ns.ux.v[0], ns.uy.v[0],
                                    nn.ux.v[0], nn.uy.v[0], n.ux.v[0], n.uy.v[0], Ax, Ay);
#pragma unroll
                        for (int i = 0; i < 9; ++i) {
                            const M t = g[i];
                            g[i] = f.g[i];
                            f.g[i] = t;
                        }
                        f.phi_b = f.phi;
                        f.phi = phi;
                    }
                }
                if (!kFlux || ALL || k >= lag * (s - 1) + 2) {
                    const Relax<M> rr = HAS_K && kFlux ? relax_from_k<M>(n.k.v[c], lam, rconst.w3) : n.r[c];
                    collide<M, false>(g, n.ux.v[c], n.uy.v[c], rr, Ax, Ay, n.s.v[c], P);
                    const auto rbits = C::bits(d.f16, level + s, (int64_t)hist[jc] * nx, (unsigned)(xi + c));
#pragma unroll
                    for (int i = 0; i < 9; ++i) o[i].v[c] = C::enc(P[i], i, d.f16, rbits);
                }
            }
            if constexpr (s == T) {
                if (live && ALL) {
                    E *__restrict__ out = dst + (int64_t)__builtin_amdgcn_readfirstlane(y) * 9 * pitch;
#pragma unroll
                    for (int i = 0; i < 9; ++i) st_cols<CST>(out + i * pitch, bc, o[i]);
                }
            } else {
                const EC n1 = kLate ? o[1] : west_of(o[1]), n3 = kLate ? o[3] : east_of(o[3]);
                const EC n5 = kLate ? o[5] : west_of(o[5]), n6 = kLate ? o[6] : east_of(o[6]);
                const EC n8 = kLate ? o[8] : west_of(o[8]), n7 = kLate ? o[7] : east_of(o[7]);
                Carry &l = L[s - 1];
                // step s + 1 pulls the row before the one just collided
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
                if constexpr (BC == 2) {
                    own[2] = UP ? l.a0 : l.b0;
                    own[4] = UP ? l.b0 : l.a0;
                    own[5] = UP ? l.aw : l.bw;
                    own[8] = UP ? l.bw : l.aw;
                    own[6] = UP ? l.ae : l.be;
                    own[7] = UP ? l.be : l.ae;
                    l.a0 = UP ? o[2] : o[4];
                    l.aw = UP ? o[5] : o[8];
                    l.ae = UP ? o[6] : o[7];
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
        };
        step(std::integral_constant<int, 1>{});
        if constexpr (T > 1) if (ALL || k >= lag) {
            step(std::integral_constant<int, 2>{});
            if constexpr (T > 2) if (ALL || k >= 2 * lag) {
                step(std::integral_constant<int, 3>{});
                if constexpr (T > 3) if (ALL || k >= 3 * lag) step(std::integral_constant<int, 4>{});
            }
        }
    };
    static_assert(T <= 4, "steps of one walk");
    constexpr int nk = kFlux ? 4 * T - 2 : 2 * (T - 1);  // iterations before the first output row
#pragma unroll 1
    for (int k = 0; k < nk; ++k) row(std::false_type{}, k, 0);
    constexpr std::true_type all{};
    int y = UP ? y1 - 1 : y0;
    if constexpr (MODE != MODE_F16SR_F32) {  // unrolled by two: the rolled values are renamed, not copied
        int left = y1 - y0;
        for (; left > 1; left -= 2) {
            row(all, nk, y);
            row(all, nk, y + dir);
            y += 2 * dir;
        }
        if (left) row(all, nk, y);
    } else {  // the rounding's values spill when unrolled (8192^2 with D 149k -> 130k MLUPS)
#pragma unroll 1
        for (int left = y1 - y0; left > 0; --left, y += dir) row(all, nk, y);
    }
}

// One instance: wave w of block b owns strip t % ns of tile row t / ns, t = 4 b + w in XCD row bands.
template <int MODE, int AUX, bool HAS_K, bool HAS_S, int T, int NC, bool CST, int BC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NC == 2 ? 2 : 1)))
void strip_kernel(const StepArgs a, const int rows)
{
    constexpr int V = strip_width(AUX == 1 ? 2 * T : T, NC);
    const InstDesc &d = a.d;
    const int ns = (d.L.nx + V - 1) / V;
    const int t = tile_of_block(blockIdx.x, gridDim.x, 1, 0, 0) * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int tr = t / ns, y0 = tr * rows, xs = (t - tr * ns) * V;
    if (y0 >= d.L.ny) return;
    const int y1 = min(y0 + rows, d.L.ny);
    if (tr & 1) strip_walk<MODE, AUX, HAS_K, HAS_S, T, NC, CST, true, BC>(d, a.parity, xs, y0, y1, t == 0);
    else strip_walk<MODE, AUX, HAS_K, HAS_S, T, NC, CST, false, BC>(d, a.parity, xs, y0, y1, t == 0);
}

// Many instances (periodic D2Q9 TRT-R, one storage form, local or no aux term): wave w of block b runs work
// item 4 b + w in XCD order, strip `tile` of instance `inst`; the descriptor is wave-uniform.
template <int MODE, int AUX>
__global__ __launch_bounds__(256) void batched_strip_kernel(const BatchArgs a, const int rows, const int items)
{
    constexpr int T = kStripSteps, V = strip_width(T, 1);
    const int it = tile_of_block(blockIdx.x, gridDim.x, 1, 0, 0) * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (it >= items) return;
    const WorkItem w = a.items[it];
    const InstDesc &d = a.inst[w.inst];
    const int ns = (d.L.nx + V - 1) / V, tr = w.tile / ns, y0 = tr * rows, xs = (w.tile - tr * ns) * V;
    const int y1 = min(y0 + rows, d.L.ny);
    if (d.has_k) {
        if (d.has_s) strip_walk<MODE, AUX, true, true, T, 1, true, false>(d, a.parity, xs, y0, y1, w.tile == 0);
        else strip_walk<MODE, AUX, true, false, T, 1, true, false>(d, a.parity, xs, y0, y1, w.tile == 0);
    } else {
        if (d.has_s) strip_walk<MODE, AUX, false, true, T, 1, true, false>(d, a.parity, xs, y0, y1, w.tile == 0);
        else strip_walk<MODE, AUX, false, false, T, 1, true, false>(d, a.parity, xs, y0, y1, w.tile == 0);
    }
}

template <int MODE, int AUX, int T, int NC, bool CST, int BC = 0>
hipError_t launch_strips_st(const StepArgs &a, const StripLaunch &s, hipStream_t st)
{
    const int rows = s.rows;
    const size_t lds = (size_t)s.lds_reserve;  // unused LDS that caps the resident waves
    constexpr int V = strip_width(AUX == 1 ? 2 * T : T, NC);
    const int64_t ns = (a.d.L.nx + V - 1) / V;
    const int64_t nb = (ns * ((a.d.L.ny + rows - 1) / rows) + 3) / 4;
    if (nb > INT32_MAX / 4 || (NC == 2 && a.d.L.nx % 2 != 0)) return hipErrorInvalidValue;
    const bool hk = a.d.has_k, hs = a.d.has_s;
    if (hk && hs) strip_kernel<MODE, AUX, true, true, T, NC, CST, BC><<<(int)nb, 256, lds, st>>>(a, rows);
    else if (hk) strip_kernel<MODE, AUX, true, false, T, NC, CST, BC><<<(int)nb, 256, lds, st>>>(a, rows);
    else if (hs) strip_kernel<MODE, AUX, false, true, T, NC, CST, BC><<<(int)nb, 256, lds, st>>>(a, rows);
    else strip_kernel<MODE, AUX, false, false, T, NC, CST, BC><<<(int)nb, 256, lds, st>>>(a, rows);
    return hipGetLastError();
}

template <int MODE, int AUX, int T, int NC, int BC = 0>
hipError_t launch_strips_kind(const StepArgs &a, const StripLaunch &s, hipStream_t st)
{
    return s.cached ? launch_strips_st<MODE, AUX, T, NC, true, BC>(a, s, st)
                    : launch_strips_st<MODE, AUX, T, NC, false, BC>(a, s, st);
}

template <int MODE>
hipError_t launch_strips_mode(int aux, const StepArgs &a, const StripLaunch &s, hipStream_t st)
{
    if (a.d.bckind == 2) {
        if constexpr (MODE == MODE_F64_F64 || MODE == MODE_F32_F32 || MODE == MODE_F16S_F32) {
            switch (aux) {
            case 0: return launch_strips_kind<MODE, 0, kStripSteps, 1, 2>(a, s, st);
            case 2: return launch_strips_kind<MODE, 2, kStripSteps, 1, 2>(a, s, st);
            default: return hipErrorInvalidValue;
            }
        }
        return hipErrorInvalidValue;
    }
    if (s.cols == 2) {
        if constexpr (is_f16_mode(MODE)) {
            switch (aux) {
            case 0: return launch_strips_kind<MODE, 0, kStripSteps, 2>(a, s, st);
            case 2: return launch_strips_kind<MODE, 2, kStripSteps, 2>(a, s, st);
            default: return hipErrorInvalidValue;
            }
        }
        return hipErrorInvalidValue;
    }
    if constexpr (MODE != MODE_F16SR_F32) {
        switch (aux) {
        case 0: return launch_strips_kind<MODE, 0, kStripSteps, 1>(a, s, st);
        case 1: return launch_strips_kind<MODE, 1, kFluxStripSteps, 1>(a, s, st);
        case 2: return launch_strips_kind<MODE, 2, kStripSteps, 1>(a, s, st);
        default: return hipErrorInvalidValue;
        }
    }
    return hipErrorInvalidValue;
}

template <int MODE>
hipError_t launch_batched_strips_mode(int aux, const BatchArgs &a, int rows, int items, hipStream_t st)
{
    const int nb = (items + 3) / 4;
    switch (aux) {
    case 0: batched_strip_kernel<MODE, 0><<<nb, 256, 0, st>>>(a, rows, items); break;
    case 2: batched_strip_kernel<MODE, 2><<<nb, 256, 0, st>>>(a, rows, items); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_strips(int mode, int aux, const StepArgs &a, const StripLaunch &s, hipStream_t st)
{
    if (a.d.L.q != 9 || a.d.bckind == 1 || a.d.w3 != 0.0 || s.rows < 1 || s.lds_reserve < 0 || s.lds_reserve > 98304 || a.d.buf[0] == a.d.buf[1])
        return hipErrorInvalidValue;
    switch (mode) {
    case MODE_F64_F64: return launch_strips_mode<MODE_F64_F64>(aux, a, s, st);
    case MODE_F64_F32: return launch_strips_mode<MODE_F64_F32>(aux, a, s, st);
    case MODE_F32_F32: return launch_strips_mode<MODE_F32_F32>(aux, a, s, st);
    case MODE_F16S_F32: return launch_strips_mode<MODE_F16S_F32>(aux, a, s, st);
    case MODE_F16SR_F32: return launch_strips_mode<MODE_F16SR_F32>(aux, a, s, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_batched_strips(int mode, int aux, const BatchArgs &a, int rows, int items, hipStream_t st)
{
    if (rows < 1 || items < 1) return hipErrorInvalidValue;
    switch (mode) {
    case MODE_F64_F64: return launch_batched_strips_mode<MODE_F64_F64>(aux, a, rows, items, st);
    case MODE_F64_F32: return launch_batched_strips_mode<MODE_F64_F32>(aux, a, rows, items, st);
    case MODE_F32_F32: return launch_batched_strips_mode<MODE_F32_F32>(aux, a, rows, items, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
