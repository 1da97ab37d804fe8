// lbm_adjoint.hip -- adjoint (reverse-mode) kernels of the TRT-R D2Q9 step for gfx950.
//
// With u, D and S fixed, one step of Sec. 2.2, Eq. (14) is affine in the pre-collision populations:
//   g^{n+1}_i(x + e_i) = sum_j M_ij(x) g^n_j(x) + c_i(x),   M(x) = dP(x)/dg(x),
// because the equilibrium (Eq. (6)) and the auxiliary term (Eq. (16), with phi at the node) are linear
// in phi = sum_j g_j, and the non-equilibrium projections (Eqs. (8), (13)) are linear in g.  The
// adjoint step is therefore
//   lam^n_j(x) = sum_i M_ij(x) mu_i(x),   mu_i(x) = lam^{n+1}_i(x + e_i),
// and, since D(x) enters only the collision at x (through tau1, tau2 and beta, Sec. 2.4),
//   dL/dD(x) += sum_i mu_i(x) dP_i(x)/dD(x) |_{g^n(x)}.
// M = H C R factorises through moments (R: raw moments phi, j, Pi of g; C: the post-collision Hermite
// coefficients a0..a3 as functions of those moments; H: the reconstruction w_i h_m(e_i)), so M^T mu
// is computed as R^T C^T H^T mu without forming M.  All in lattice units, like the forward kernel.
#include "lbm_internal.h"
#include "lbm_kernel_common.h"
#include "lbm_strips.h"

namespace lbm {
namespace {

template <int MODE>
struct AdjTraits;
template <>
struct AdjTraits<MODE_F64_F64> {
    using St = StoreF64;
    using M = double;
};
template <>
struct AdjTraits<MODE_F64_F32> {
    using St = StoreF64;
    using M = float;
};
template <>
struct AdjTraits<MODE_F32_F32> {
    using St = StoreF32;
    using M = float;
};

__device__ __forceinline__ int wdec(int v, int n) { return v == 0 ? n - 1 : v - 1; }
__device__ __forceinline__ int winc(int v, int n) { return v == n - 1 ? 0 : v + 1; }

// The relaxation at a node and its derivatives with respect to k: tau1 = 1/2 + k, tau2 = 1/2 + Lambda/k.
template <class M>
struct AdjRelax {
    M w1, w2, beta, dw1, dw2, dbeta;
};
template <class M>
__device__ __forceinline__ AdjRelax<M> adj_relax(M k, M lam)
{
    const M tau1 = M(0.5) + k, tau2 = M(0.5) + lam / k;
    return {M(1) - M(1) / tau1,   M(1) - M(1) / tau2,
            M(1) - M(0.5) / tau1, M(1) / (tau1 * tau1),
            -lam / (k * k * tau2 * tau2), M(0.5) / (tau1 * tau1)};
}

// q = H^T mu: the Hermite "moments" of mu weighted as in the reconstruction
template <class M>
struct AdjMoments {
    M q0, q1x, q1y, q2xx, q2yy, q2xy, q3xxy, q3xyy;
};
template <class M>
__device__ __forceinline__ AdjMoments<M> adj_moments(const M mu[9])
{
    M q0 = 0, q1x = 0, q1y = 0, q2xx = 0, q2yy = 0, q2xy = 0, q3xxy = 0, q3xyy = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const M wm = M(kW[i]) * mu[i];
        const int ex = kEx[i], ey = kEy[i];
        q0 += wm;
        if (ex) q1x += M(3 * ex) * wm;
        if (ey) q1y += M(3 * ey) * wm;
        q2xx += M(4.5 * (ex * ex - 1.0 / 3.0)) * wm;
        q2yy += M(4.5 * (ey * ey - 1.0 / 3.0)) * wm;
        if (ex * ey) q2xy += M(9 * ex * ey) * wm;
        if (ey) q3xxy += M(13.5 * (ex * ex * ey - ey / 3.0)) * wm;
        if (ex) q3xyy += M(13.5 * (ex * ey * ey - ex / 3.0)) * wm;
    }
    return {q0, q1x, q1y, q2xx, q2yy, q2xy, q3xxy, q3xyy};
}

// lam^n = R^T t with t = C^T q (derivatives of the Hermite coefficients with respect to phi, j, Pi);
// (ahx, ahy) = u_b d_b u_a
template <class M>
__device__ __forceinline__ void adj_lambda(const AdjMoments<M> &q, const AdjRelax<M> &r, M ux, M uy, M ahx, M ahy, M lam[9])
{
    const M uxx = ux * ux, uyy = uy * uy, uxy = ux * uy;
    const M tphi = q.q0 + q.q1x * (ux * (M(1) - r.w1) + r.beta * ahx) + q.q1y * (uy * (M(1) - r.w1) + r.beta * ahy) +
                   q.q2xx * (uxx * (M(1) - r.w2) - r.w2 * M(1.0 / 3.0)) + q.q2yy * (uyy * (M(1) - r.w2) - r.w2 * M(1.0 / 3.0)) +
                   q.q2xy * uxy * (M(1) - r.w2) + q.q3xxy * uxx * uy + q.q3xyy * ux * uyy;
    const M tjx = r.w1 * q.q1x, tjy = r.w1 * q.q1y, tpxx = r.w2 * q.q2xx, tpyy = r.w2 * q.q2yy, tpxy = r.w2 * q.q2xy;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int ex = kEx[j], ey = kEy[j];
        M v = tphi;
        if (ex) v += M(ex) * tjx + tpxx;
        if (ey) v += M(ey) * tjy + tpyy;
        if (ex * ey) v += M(ex * ey) * tpxy;
        lam[j] = v;
    }
}

// mu . dP/dk at g^n(x)
template <class M>
__device__ __forceinline__ M adj_dk(const AdjMoments<M> &q, const AdjRelax<M> &r, const M g[9], M ux, M uy, M ahx, M ahy, M s)
{
    const M uxx = ux * ux, uyy = uy * uy, uxy = ux * uy;
    const M phi = g[0] + g[1] + g[2] + g[3] + g[4] + g[5] + g[6] + g[7] + g[8];
    const M jx = (g[1] - g[3]) + (g[5] - g[6]) + (g[8] - g[7]);
    const M jy = (g[2] - g[4]) + (g[5] + g[6]) - (g[7] + g[8]);
    const M sd = (g[5] + g[6]) + (g[7] + g[8]);
    const M nxx = g[1] + g[3] + sd - phi * M(1.0 / 3.0) - phi * uxx;
    const M nyy = g[2] + g[4] + sd - phi * M(1.0 / 3.0) - phi * uyy;
    const M nxy = (g[5] + g[7]) - (g[6] + g[8]) - phi * uxy;
    return q.q1x * (r.dw1 * (jx - phi * ux) + r.dbeta * (phi * ahx + ux * s)) +
           q.q1y * (r.dw1 * (jy - phi * uy) + r.dbeta * (phi * ahy + uy * s)) +
           r.dw2 * (q.q2xx * nxx + q.q2yy * nyy + q.q2xy * nxy);
}

// Block (64, 4): lane = column, wave = row.
template <int MODE, bool HAS_K, bool HAS_S, bool LOCAL>
__global__ __launch_bounds__(256) void adjoint_kernel(const AdjArgs a)
{
    using St = typename AdjTraits<MODE>::St;
    using M = typename AdjTraits<MODE>::M;
    using T = typename St::T;
    using C = Codec<St, M>;
    // Tiles of 256 columns (the block's four waves side by side, lane = column) by one row, in row bands
    // over the XCDs (each XCD's rows and their neighbours in one L2); the row is uniform, so every
    // access is a scalar row base plus a 32-bit lane offset.
    const int nx = a.L.nx, ny = a.L.ny;
    const int64_t pitch = a.L.pitch;
    const int ntx = (nx + 255) / 256;
    const int t = tile_of_block(blockIdx.x, gridDim.x, 1, ntx, 0);
    const int y = __builtin_amdgcn_readfirstlane(t / ntx);
    const int x = (t % ntx) * 256 + __builtin_amdgcn_readfirstlane((int)threadIdx.y) * 64 + (int)threadIdx.x;
    if (x >= nx) return;
    const unsigned xc = (unsigned)x, xm = (unsigned)wdec(x, nx), xp = (unsigned)winc(x, nx);
    const int ym = __builtin_amdgcn_readfirstlane(wdec(y, ny)), yp = __builtin_amdgcn_readfirstlane(winc(y, ny));
    const unsigned bc = xc * (unsigned)sizeof(T), bm = xm * (unsigned)sizeof(T), bp = xp * (unsigned)sizeof(T);
    const unsigned fc = xc * (unsigned)sizeof(M), fm = xm * (unsigned)sizeof(M), fp = xp * (unsigned)sizeof(M);
    const T *st = static_cast<const T *>(a.state);
    const M *lin = static_cast<const M *>(a.lam_in);
    M *lout = static_cast<M *>(a.lam_out);
    const M *u = static_cast<const M *>(a.u);

    // forward pre-collision state g^n(x) = buf_i(x - e_i)
    M g[9];
    {
        const T *rm = st + (int64_t)ym * 9 * pitch, *rc = st + (int64_t)y * 9 * pitch, *rp = st + (int64_t)yp * 9 * pitch;
        g[0] = C::dec(ld_at(rc, bc), 0, a.f16);
        g[1] = C::dec(ld_at(rc + 1 * pitch, bm), 1, a.f16);
        g[2] = C::dec(ld_at(rm + 2 * pitch, bc), 2, a.f16);
        g[3] = C::dec(ld_at(rc + 3 * pitch, bp), 3, a.f16);
        g[4] = C::dec(ld_at(rp + 4 * pitch, bc), 4, a.f16);
        g[5] = C::dec(ld_at(rm + 5 * pitch, bm), 5, a.f16);
        g[6] = C::dec(ld_at(rm + 6 * pitch, bp), 6, a.f16);
        g[7] = C::dec(ld_at(rp + 7 * pitch, bp), 7, a.f16);
        g[8] = C::dec(ld_at(rp + 8 * pitch, bm), 8, a.f16);
    }
    // mu_i(x) = lam^{n+1}_i(x + e_i)
    M mu[9];
    {
        const M *lm = lin + (int64_t)ym * 9 * pitch, *lc = lin + (int64_t)y * 9 * pitch, *lp = lin + (int64_t)yp * 9 * pitch;
        mu[0] = ld_at(lc, fc);
        mu[1] = ld_at(lc + 1 * pitch, fp);
        mu[2] = ld_at(lp + 2 * pitch, fc);
        mu[3] = ld_at(lc + 3 * pitch, fm);
        mu[4] = ld_at(lm + 4 * pitch, fc);
        mu[5] = ld_at(lp + 5 * pitch, fp);
        mu[6] = ld_at(lp + 6 * pitch, fm);
        mu[7] = ld_at(lm + 7 * pitch, fm);
        mu[8] = ld_at(lm + 8 * pitch, fp);
    }
    const M *uc = u + (int64_t)y * 2 * pitch;
    const M ux = ld_at(uc, fc), uy = ld_at(uc + pitch, fc);
    M ahx = M(0), ahy = M(0);  // u_b d_b u_a (central differences), Eq. (16) without phi
    if (LOCAL) {
        const M *um = u + (int64_t)ym * 2 * pitch, *up = u + (int64_t)yp * 2 * pitch;
        ahx = ux * (ld_at(uc, fp) - ld_at(uc, fm)) * M(0.5) + uy * (ld_at(up, fc) - ld_at(um, fc)) * M(0.5);
        ahy = ux * (ld_at(uc + pitch, fp) - ld_at(uc + pitch, fm)) * M(0.5) +
              uy * (ld_at(up + pitch, fc) - ld_at(um + pitch, fc)) * M(0.5);
    }
    const M k = HAS_K ? ld_at(static_cast<const M *>(a.k) + (int64_t)y * pitch, fc) : (M)a.k_const;
    const M s = HAS_S ? ld_at(static_cast<const M *>(a.s) + (int64_t)y * pitch, fc) : M(0);
    const AdjRelax<M> r = adj_relax<M>(k, (M)a.lambda);
    const AdjMoments<M> q = adj_moments<M>(mu);
    M lam[9];
    adj_lambda<M>(q, r, ux, uy, ahx, ahy, lam);
    M *lo = lout + (int64_t)y * 9 * pitch;
#pragma unroll
    for (int j = 0; j < 9; ++j) st_at(lo + j * pitch, fc, lam[j]);
    const M dk = adj_dk<M>(q, r, g, ux, uy, ahx, ahy, s);
    double *gr = a.grad + (int64_t)y * nx;
    gr[x] += a.dk_dD * (double)dk;
}

// kAdjointPatchSteps steps of adjoint_kernel in one launch, on patches of NW rows (wave = row, lane = column) as
// in lbm_patches.h: lam stays in registers between the steps, its components that move along y change rows
// through LDS (two buffers, one barrier per step), and u . grad u, the relaxation and its derivatives are computed
// once.  Only the H = NW - 2 (T - 1) rows that the block writes read the forward states.  Same arithmetic, so
// bitwise equal to the single steps (dL/dD is summed in the same order).  What bounds it: instructions, 205 per
// node and step against 284, of 1.8 times the nodes at 16 waves (FP32 64 VGPRs: two blocks per CU), and below
// 300^2 the launch.  Us per segment of 9 steps (recomputation by single steps), single / patches: FP32 512^2 102 /
// 89, 1000^2 371 / 283, 2048^2 1450 / 1046; FP64 512^2 174 / 146, 2048^2 2856 / 2164.
template <int MODE, bool HAS_K, bool HAS_S, bool LOCAL, int NW>
__global__ __launch_bounds__(64 * NW) void adjoint_patch_kernel(const AdjArgs a, const int64_t image_bytes)
{
    using St = typename AdjTraits<MODE>::St;
    using M = typename AdjTraits<MODE>::M;
    using E = typename St::T;
    using C = Codec<St, M>;
    constexpr int T = kAdjointPatchSteps, V = strip_width(T, 1), H = NW - 2 * (T - 1);
    __shared__ M xch[2][6 * NW * 64 + 2];  // one spare element at either end (lanes without a neighbour)
    const int nx = a.L.nx, ny = a.L.ny;
    const int64_t pitch = a.L.pitch;
    const int ns = (nx + V - 1) / V;
    const int t = tile_of_block(blockIdx.x, gridDim.x, 1, 0, 0);
    const int tr = t / ns, xs = (t - tr * ns) * V;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63u);
    int xi = (xs - T + lane) % nx;
    xi = xi < 0 ? xi + nx : xi;
    int y = (tr * H - (T - 1) + w) % ny;
    y = __builtin_amdgcn_readfirstlane(y < 0 ? y + ny : y);
    const bool out = w >= T - 1 && w < T - 1 + H && tr * H + w - (T - 1) < ny;
    const bool live = lane >= T && lane < T + V && xs + lane - T < nx;
    const int ym = wdec(y, ny), yp = winc(y, ny);
    const unsigned xc = (unsigned)xi, xm = (unsigned)wdec(xi, nx), xp = (unsigned)winc(xi, nx);
    const unsigned bc = xc * (unsigned)sizeof(E), bm = xm * (unsigned)sizeof(E), bp = xp * (unsigned)sizeof(E);
    const unsigned fc = xc * (unsigned)sizeof(M), fm = xm * (unsigned)sizeof(M), fp = xp * (unsigned)sizeof(M);
    const M *__restrict__ u = static_cast<const M *>(a.u);
    M mu[9];
    {
        const M *__restrict__ lin = static_cast<const M *>(a.lam_in);
        const M *__restrict__ lm = lin + (int64_t)ym * 9 * pitch, *__restrict__ lc = lin + (int64_t)y * 9 * pitch,
                *__restrict__ lp = lin + (int64_t)yp * 9 * pitch;
        mu[0] = ld_at(lc, fc);
        mu[1] = ld_at(lc + 1 * pitch, fp);
        mu[2] = ld_at(lp + 2 * pitch, fc);
        mu[3] = ld_at(lc + 3 * pitch, fm);
        mu[4] = ld_at(lm + 4 * pitch, fc);
        mu[5] = ld_at(lp + 5 * pitch, fp);
        mu[6] = ld_at(lp + 6 * pitch, fm);
        mu[7] = ld_at(lm + 7 * pitch, fm);
        mu[8] = ld_at(lm + 8 * pitch, fp);
    }
    const M *__restrict__ uc = u + (int64_t)y * 2 * pitch;
    const M ux = ld_at(uc, fc), uy = ld_at(uc + pitch, fc);
    M ahx = M(0), ahy = M(0);
    if (LOCAL) {
        const M *__restrict__ um = u + (int64_t)ym * 2 * pitch, *__restrict__ up = u + (int64_t)yp * 2 * pitch;
        ahx = ux * (lane_e(ux) - lane_w(ux)) * M(0.5) + uy * (ld_at(up, fc) - ld_at(um, fc)) * M(0.5);
        ahy = ux * (lane_e(uy) - lane_w(uy)) * M(0.5) + uy * (ld_at(up + pitch, fc) - ld_at(um + pitch, fc)) * M(0.5);
    }
    const M k = HAS_K ? ld_at(static_cast<const M *>(a.k) + (int64_t)y * pitch, fc) : (M)a.k_const;
    const M s = HAS_S ? ld_at(static_cast<const M *>(a.s) + (int64_t)y * pitch, fc) : M(0);
    double *gr = a.grad + (int64_t)y * nx + xi;
    double sum = out && live ? *gr : 0.0;
    const AdjRelax<M> r = adj_relax<M>(k, (M)a.lambda);
    auto at = [&](int p, int v) { return 1 + (p * NW + v) * 64 + lane; };
    const int wm = max(w - 1, 0), wp = min(w + 1, NW - 1);
#pragma unroll
    for (int n = 1; n <= T; ++n) {
        if (w >= n - 1 && w <= NW - n) {
            M g[9];
            if (out) {
                const E *__restrict__ st = reinterpret_cast<const E *>(static_cast<const char *>(a.state) - (n - 1) * image_bytes);
                const E *__restrict__ rm = st + (int64_t)ym * 9 * pitch, *__restrict__ rc = st + (int64_t)y * 9 * pitch,
                        *__restrict__ rp = st + (int64_t)yp * 9 * pitch;
                g[0] = C::dec(ld_at(rc, bc), 0, a.f16);
                g[1] = C::dec(ld_at(rc + 1 * pitch, bm), 1, a.f16);
                g[2] = C::dec(ld_at(rm + 2 * pitch, bc), 2, a.f16);
                g[3] = C::dec(ld_at(rc + 3 * pitch, bp), 3, a.f16);
                g[4] = C::dec(ld_at(rp + 4 * pitch, bc), 4, a.f16);
                g[5] = C::dec(ld_at(rm + 5 * pitch, bm), 5, a.f16);
                g[6] = C::dec(ld_at(rm + 6 * pitch, bp), 6, a.f16);
                g[7] = C::dec(ld_at(rp + 7 * pitch, bp), 7, a.f16);
                g[8] = C::dec(ld_at(rp + 8 * pitch, bm), 8, a.f16);
            }
            const AdjMoments<M> q = adj_moments<M>(mu);
            M lam[9];
            adj_lambda<M>(q, r, ux, uy, ahx, ahy, lam);
            if (n == T) {
                if (out && live) {
                    M *__restrict__ lo = static_cast<M *>(a.lam_out) + (int64_t)y * 9 * pitch;
#pragma unroll
                    for (int j = 0; j < 9; ++j) st_at(lo + j * pitch, fc, lam[j]);
                }
            } else {
                M *x = xch[n & 1];
                x[at(0, w)] = lam[2];
                x[at(1, w)] = lam[4];
#pragma unroll
                for (int i = 5; i < 9; ++i) x[at(i - 3, w)] = lam[i];
                mu[0] = lam[0];
                mu[1] = lane_e(lam[1]);
                mu[3] = lane_w(lam[3]);
            }
            if (out) sum += a.dk_dD * (double)adj_dk<M>(q, r, g, ux, uy, ahx, ahy, s);
        }
        if (n == T) break;
        __syncthreads();
        if (w >= n && w <= NW - 1 - n) {
            const M *x = xch[n & 1];
            mu[2] = x[at(0, wp)];
            mu[4] = x[at(1, wm)];
            mu[5] = x[at(2, wp) + 1];
            mu[6] = x[at(3, wp) - 1];
            mu[7] = x[at(4, wm) - 1];
            mu[8] = x[at(5, wm) + 1];
        }
    }
    if (out && live) *gr = sum;
}

// lam_i(x) = dL/dphi(x) for every i (adjoint of phi = sum_i g_i)
template <class M>
__global__ __launch_bounds__(256) void adjoint_seed_kernel(const double *dphi, M *lam, Layout L)
{
    const int64_t N = (int64_t)L.nx * L.ny;
    for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n < N; n += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(n % L.nx), y = (int)(n / L.nx);
        const M v = (M)dphi[n];
#pragma unroll
        for (int i = 0; i < 9; ++i) lam[((int64_t)y * 9 + i) * L.pitch + x] = v;
    }
}

// dL/dphi0(x) = sum_i lam0_i(x) dg_eq_i/dphi0(x) (adjoint of the initial condition g = g_eq(phi0, u))
template <class M>
__global__ __launch_bounds__(256) void adjoint_init_kernel(const M *lam, const M *u, double *dphi0, Layout L)
{
    const int64_t N = (int64_t)L.nx * L.ny;
    for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n < N; n += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(n % L.nx), y = (int)(n / L.nx);
        M e[9];
        equilibrium<M>(M(1), u[(int64_t)y * 2 * L.pitch + x], u[((int64_t)y * 2 + 1) * L.pitch + x], e);
        double acc = 0;
#pragma unroll
        for (int i = 0; i < 9; ++i) acc += (double)(e[i] * lam[((int64_t)y * 9 + i) * L.pitch + x]);
        dphi0[n] = acc;
    }
}

template <int MODE, bool LOCAL>
hipError_t launch_adj_aux(const AdjArgs &a, hipStream_t st)
{
    dim3 block(64, 4);
    const int grid = ((a.L.nx + 255) / 256) * a.L.ny;  // 256-column tiles of one row
    const bool hk = a.k != nullptr, hs = a.s != nullptr;
    if (hk && hs) adjoint_kernel<MODE, true, true, LOCAL><<<grid, block, 0, st>>>(a);
    else if (hk) adjoint_kernel<MODE, true, false, LOCAL><<<grid, block, 0, st>>>(a);
    else if (hs) adjoint_kernel<MODE, false, true, LOCAL><<<grid, block, 0, st>>>(a);
    else adjoint_kernel<MODE, false, false, LOCAL><<<grid, block, 0, st>>>(a);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_adj_mode(int aux, const AdjArgs &a, hipStream_t st)
{
    return aux == 0 ? launch_adj_aux<MODE, true>(a, st) : launch_adj_aux<MODE, false>(a, st);
}

template <int MODE, bool LOCAL, int NW>
hipError_t launch_adj_patches_aux(const AdjArgs &a, int64_t image_bytes, hipStream_t st)
{
    constexpr int V = strip_width(kAdjointPatchSteps, 1), H = NW - 2 * (kAdjointPatchSteps - 1);
    const int64_t nb = (int64_t)((a.L.nx + V - 1) / V) * ((a.L.ny + H - 1) / H);
    if (nb > INT32_MAX / 16) return hipErrorInvalidValue;
    const bool hk = a.k != nullptr, hs = a.s != nullptr;
    if (hk && hs) adjoint_patch_kernel<MODE, true, true, LOCAL, NW><<<(int)nb, 64 * NW, 0, st>>>(a, image_bytes);
    else if (hk) adjoint_patch_kernel<MODE, true, false, LOCAL, NW><<<(int)nb, 64 * NW, 0, st>>>(a, image_bytes);
    else if (hs) adjoint_patch_kernel<MODE, false, true, LOCAL, NW><<<(int)nb, 64 * NW, 0, st>>>(a, image_bytes);
    else adjoint_patch_kernel<MODE, false, false, LOCAL, NW><<<(int)nb, 64 * NW, 0, st>>>(a, image_bytes);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_adj_patches_mode(int aux, const AdjArgs &a, int waves, int64_t image_bytes, hipStream_t st)
{
    if (waves == 12)
        return aux == 0 ? launch_adj_patches_aux<MODE, true, 12>(a, image_bytes, st) : launch_adj_patches_aux<MODE, false, 12>(a, image_bytes, st);
    if (waves == 16)
        return aux == 0 ? launch_adj_patches_aux<MODE, true, 16>(a, image_bytes, st) : launch_adj_patches_aux<MODE, false, 16>(a, image_bytes, st);
    return hipErrorInvalidValue;
}

int adj_grid(const Layout &L)
{
    int64_t g = ((int64_t)L.nx * L.ny + 255) / 256;
    return (int)(g > 8192 ? 8192 : (g < 1 ? 1 : g));
}

}  // namespace

hipError_t launch_adjoint(int mode, int aux, const AdjArgs &a, hipStream_t st)
{
    switch (mode) {
    case MODE_F64_F64: return launch_adj_mode<MODE_F64_F64>(aux, a, st);
    case MODE_F64_F32: return launch_adj_mode<MODE_F64_F32>(aux, a, st);
    case MODE_F32_F32: return launch_adj_mode<MODE_F32_F32>(aux, a, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_adjoint_patches(int mode, int aux, const AdjArgs &a, int waves, int64_t image_bytes, hipStream_t st)
{
    switch (mode) {
    case MODE_F64_F64: return launch_adj_patches_mode<MODE_F64_F64>(aux, a, waves, image_bytes, st);
    case MODE_F64_F32: return launch_adj_patches_mode<MODE_F64_F32>(aux, a, waves, image_bytes, st);
    case MODE_F32_F32: return launch_adj_patches_mode<MODE_F32_F32>(aux, a, waves, image_bytes, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_adjoint_seed(int mode, const double *dphi, void *lam, const Layout &L, hipStream_t st)
{
    if (mode == MODE_F64_F64) adjoint_seed_kernel<double><<<adj_grid(L), 256, 0, st>>>(dphi, static_cast<double *>(lam), L);
    else adjoint_seed_kernel<float><<<adj_grid(L), 256, 0, st>>>(dphi, static_cast<float *>(lam), L);
    return hipGetLastError();
}

hipError_t launch_adjoint_init(int mode, const void *lam, const void *u, double *dphi0, const Layout &L, hipStream_t st)
{
    if (mode == MODE_F64_F64)
        adjoint_init_kernel<double><<<adj_grid(L), 256, 0, st>>>(static_cast<const double *>(lam), static_cast<const double *>(u), dphi0, L);
    else
        adjoint_init_kernel<float><<<adj_grid(L), 256, 0, st>>>(static_cast<const float *>(lam), static_cast<const float *>(u), dphi0, L);
    return hipGetLastError();
}

}  // namespace lbm
