// Newtonian ideal MHD (Sec. IV.B, eight-field core: rho, S, E, B) in the
// conservative finite-difference form (eq. conservative_discretization):
//   L = - sum_d (F_{i+1/2} - F_{i-1/2}) / dx_d,
// with the evolved fields reconstructed at every interface by WENO5-Z
// (App. B; q = 2, eps = dx^4 unless set), WENO5-JS (App. B) or WENO3 (App. A,
// eps = dx^2 unless set), and the local Lax-Friedrichs flux (eq. LLF)
// F = (F(U^L) + F(U^R) - S (U^R - U^L)) / 2, S the larger of |v_d| + c_f over
// the two states (fast magnetosonic speed c_f), or the HLL flux
// F = (S^R F^L - S^L F^R + S^R S^L (U^R - U^L)) / (S^R - S^L) with
// S^L = min(v_d - c_f, 0), S^R = max(v_d + c_f, 0) over the two states.  With
// the divergence-cleaning scalar psi (nine fields) the B^i flux along d gains
// delta^{di} psi, psi has the flux c_h^2 B^d and the source -kappa_psi psi, and
// the cleaning speeds -c_h, +c_h join the signal speeds.  Fused with the
// Runge-Kutta stage update.
#include "k_common.h"

namespace mol {

namespace {

struct MhdConst {
    double gam;
    double eps;
    double q;
    double ih;  // 1 / dx
    double ch2, ch, kpsi;  // cleaning: c_h^2, c_h, kappa_psi
};

// WENO5-Z value at the interface to the right of v[2] reconstructed from the
// left, using one division: alpha_r = d_r (e_r^2 + tau^2) / e_r^2 with
// e_r = eps + beta_r, scaled by e_0^2 e_1^2 e_2^2.  The right state at the
// interface to the left of a cell is the same formula on mirrored values.
template <bool Q2>
__device__ __forceinline__ double weno5z(double v0, double v1, double v2, double v3, double v4,
                                         double eps, double q)
{
    const double p0 = (2.0 * v2 + 5.0 * v3 - v4) * (1.0 / 6.0);
    const double p1 = (-v1 + 5.0 * v2 + 2.0 * v3) * (1.0 / 6.0);
    const double p2 = (2.0 * v0 - 7.0 * v1 + 11.0 * v2) * (1.0 / 6.0);
    const double a0 = v2 - 2.0 * v3 + v4, b0 = 3.0 * v2 - 4.0 * v3 + v4;
    const double a1 = v1 - 2.0 * v2 + v3, b1 = v1 - v3;
    const double a2 = v0 - 2.0 * v1 + v2, b2 = v0 - 4.0 * v1 + 3.0 * v2;
    const double be0 = (13.0 / 12.0) * a0 * a0 + 0.25 * b0 * b0;
    const double be1 = (13.0 / 12.0) * a1 * a1 + 0.25 * b1 * b1;
    const double be2 = (13.0 / 12.0) * a2 * a2 + 0.25 * b2 * b2;
    const double tau = fabs(be0 - be2);
    const double e0 = eps + be0, e1 = eps + be1, e2 = eps + be2;
    double w0, w1, w2;
    if constexpr (Q2) {
        const double s0 = e0 * e0, s1 = e1 * e1, s2 = e2 * e2, t2 = tau * tau;
        w0 = 0.3 * (s0 + t2) * (s1 * s2);
        w1 = 0.6 * (s1 + t2) * (s0 * s2);
        w2 = 0.1 * (s2 + t2) * (s0 * s1);
    } else {
        w0 = 0.3 * (1.0 + pow(tau / e0, q));
        w1 = 0.6 * (1.0 + pow(tau / e1, q));
        w2 = 0.1 * (1.0 + pow(tau / e2, q));
    }
    return (w0 * p0 + w1 * p1 + w2 * p2) / (w0 + w1 + w2);
}

// WENO5-JS value at the interface to the right of v[2] from the left:
// alpha_r = d_r / e_r^2, e_r = eps + beta_r, scaled by e_0^2 e_1^2 e_2^2.
__device__ __forceinline__ double weno5js(double v0, double v1, double v2, double v3, double v4, double eps)
{
    const double p0 = (2.0 * v2 + 5.0 * v3 - v4) * (1.0 / 6.0);
    const double p1 = (-v1 + 5.0 * v2 + 2.0 * v3) * (1.0 / 6.0);
    const double p2 = (2.0 * v0 - 7.0 * v1 + 11.0 * v2) * (1.0 / 6.0);
    const double a0 = v2 - 2.0 * v3 + v4, b0 = 3.0 * v2 - 4.0 * v3 + v4;
    const double a1 = v1 - 2.0 * v2 + v3, b1 = v1 - v3;
    const double a2 = v0 - 2.0 * v1 + v2, b2 = v0 - 4.0 * v1 + 3.0 * v2;
    const double e0 = eps + ((13.0 / 12.0) * a0 * a0 + 0.25 * b0 * b0);
    const double e1 = eps + ((13.0 / 12.0) * a1 * a1 + 0.25 * b1 * b1);
    const double e2 = eps + ((13.0 / 12.0) * a2 * a2 + 0.25 * b2 * b2);
    const double s0 = e0 * e0, s1 = e1 * e1, s2 = e2 * e2;
    const double w0 = 0.3 * (s1 * s2), w1 = 0.6 * (s0 * s2), w2 = 0.1 * (s0 * s1);
    return (w0 * p0 + w1 * p1 + w2 * p2) / (w0 + w1 + w2);
}

// WENO3 value at the interface to the right of v2 from the left (cells v1,
// v2, v3): alpha_0 = (2/3) / e_0^2, alpha_1 = (1/3) / e_1^2, scaled by e_0^2 e_1^2.
__device__ __forceinline__ double weno3(double v1, double v2, double v3, double eps)
{
    const double p0 = 0.5 * (v2 + v3), p1 = 1.5 * v2 - 0.5 * v1;
    const double d0 = v3 - v2, d1 = v2 - v1;
    const double e0 = eps + d0 * d0, e1 = eps + d1 * d1;
    const double w0 = (2.0 / 3.0) * (e1 * e1), w1 = (1.0 / 3.0) * (e0 * e0);
    return (w0 * p0 + w1 * p1) / (w0 + w1);
}

enum { REC_W5Z = 0, REC_W5JS = 1, REC_W3 = 2 };
enum { RS_LLF = 0, RS_HLL = 1, RS_SPLIT = 2 };

// reconstructed value at the interface to the right of v2 from the left
template <int REC, bool Q2>
__device__ __forceinline__ double recon(double v0, double v1, double v2, double v3, double v4, double eps, double q)
{
    if constexpr (REC == REC_W3)
        return weno3(v1, v2, v3, eps);
    else if constexpr (REC == REC_W5JS)
        return weno5js(v0, v1, v2, v3, v4, eps);
    else
        return weno5z<Q2>(v0, v1, v2, v3, v4, eps, q);
}

// physical flux along d, the normal velocity v_d and the fast speed c_f
__device__ __forceinline__ void flux(const double U[8], int d, double gam, double F[8], double& vdo, double& cf)
{
    const double rho = U[0], ir = 1.0 / rho;
    const double vx = U[1] * ir, vy = U[2] * ir, vz = U[3] * ir;
    const double Bx = U[5], By = U[6], Bz = U[7];
    const double B2 = Bx * Bx + By * By + Bz * Bz;
    const double S2 = U[1] * U[1] + U[2] * U[2] + U[3] * U[3];
    const double p = (gam - 1.0) * (U[4] - 0.5 * S2 * ir - 0.5 * B2);
    const double pt = p + 0.5 * B2;
    const double vB = vx * Bx + vy * By + vz * Bz;
    const double vd = d == 0 ? vx : d == 1 ? vy : vz;
    const double Bd = d == 0 ? Bx : d == 1 ? By : Bz;
    F[0] = U[1 + d];
    F[1] = U[1] * vd - Bd * Bx + (d == 0 ? pt : 0.0);
    F[2] = U[2] * vd - Bd * By + (d == 1 ? pt : 0.0);
    F[3] = U[3] * vd - Bd * Bz + (d == 2 ? pt : 0.0);
    F[4] = (U[4] + pt) * vd - vB * Bd;
    F[5] = vd * Bx - vx * Bd;
    F[6] = vd * By - vy * Bd;
    F[7] = vd * Bz - vz * Bd;
    // (a^2 + b^2)^2 - 4 a^2 b_d^2 as (a^2 - b^2)^2 + 4 a^2 b_t^2: no cancellation
    // where the sound and Alfven speeds meet with B nearly along d
    const double Bt2 = d == 0 ? By * By + Bz * Bz : d == 1 ? Bx * Bx + Bz * Bz : Bx * Bx + By * By;
    const double a2 = gam * p * ir, b2 = B2 * ir, bt2 = Bt2 * ir;
    const double dab = a2 - b2;
    const double cf2 = 0.5 * (a2 + b2 + sqrt(dab * dab + 4.0 * a2 * bt2));
    vdo = vd;
    cf = sqrt(cf2);
}

// Interface flux by flux splitting between cells 2 and 3 of a six-cell line;
// get(f, m) returns cell m (0..5) of field f.
template <int NF, int REC, bool Q2, class Get>
__device__ __forceinline__ void split_flux(Get get, int d, const MhdConst& C, double Fh[NF])
{
    // (F +- alpha U)/2 of the six cells, alpha the largest signal speed
    // among them; left-biased reconstruction of the + part around cell 2,
    // right-biased (mirrored) of the - part around cell 3
    double gp[NF][6], gm[NF][6], alpha = 0.0;
#pragma unroll
    for (int m = 0; m < 6; ++m) {
        double U[NF], F[NF], vd, cf;
#pragma unroll
        for (int f = 0; f < NF; ++f) U[f] = get(f, m);
        flux(U, d, C.gam, F, vd, cf);
        double sp = fabs(vd) + cf;
        if constexpr (NF == 9) {
            F[5 + d] += U[8];
            F[8] = C.ch2 * U[5 + d];
            sp = fmax(sp, C.ch);
        }
        alpha = fmax(alpha, sp);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            gp[f][m] = F[f];
            gm[f][m] = U[f];
        }
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        double p[6], q[6];
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            p[m] = 0.5 * (gp[f][m] + alpha * gm[f][m]);
            q[m] = 0.5 * (gp[f][m] - alpha * gm[f][m]);
        }
        Fh[f] = recon<REC, Q2>(p[0], p[1], p[2], p[3], p[4], C.eps, C.q) +
                recon<REC, Q2>(q[5], q[4], q[3], q[2], q[1], C.eps, C.q);
    }
}

// Both states that a cell v2 of the line v0 .. v4 contributes: left, at the
// interface to its right, and right (the left formula on mirrored cells), at
// the interface to its left.  They share the smoothness indicators and the
// unnormalised weights: with d_ij = v_j - v_i, 4 beta_r from the second
// differences a_r and b_r, e_r = 4 (eps + beta_r) and X_r = (e_r^2 + tau^2)
// e_s^2 e_t^2 (WENO5-Z; the factor 4 cancels between them), the left value is
// v2 plus the weighted mean (3 X_0, 6 X_1, X_2) of the candidates' distances
// from v2, the right value the same with X_0 and X_2 exchanged.  The weights
// carry a common factor K, so that the products with the distances stay finite
// for all values for which those of d_r / (eps + beta_r)^p times the other
// denominators with the candidates do (WENO5-Z at jumps of any shape: from
// 10^22.3 without K to 10^22.8); K costs no operation.  eps4 = 4 eps (WENO3: eps).
template <int REC, bool Q2>
__device__ __forceinline__ void cell_states(double v0, double v1, double v2, double v3, double v4, double eps4,
                                            double q, double& left, double& right)
{
    const double d12 = v2 - v1, d23 = v3 - v2;
    if constexpr (REC == REC_W3) {
        const double e0 = fma(d23, d23, eps4), e1 = fma(d12, d12, eps4), s0 = e0 * e0, s1 = e1 * e1;
        left = v2 + 0.5 * (fma(2.0 * s1, d23, s0 * d12) / fma(2.0, s1, s0));
        right = v2 - 0.5 * (fma(2.0 * s0, d12, s1 * d23) / fma(2.0, s0, s1));
        return;
    }
    const double d01 = v1 - v0, d34 = v4 - v3;
    const double a0 = d34 - d23, a1 = d23 - d12, a2 = d12 - d01;
    const double b0 = fma(-3.0, d23, d34), b1 = d12 + d23, b2 = fma(3.0, d12, -d01);
    const double c = 13.0 / 3.0;
    const double be0 = fma(c * a0, a0, b0 * b0), be1 = fma(c * a1, a1, b1 * b1), be2 = fma(c * a2, a2, b2 * b2);
    const double e0 = eps4 + be0, e1 = eps4 + be1, e2 = eps4 + be2;
    double X0, X1, X2;
    if constexpr (REC == REC_W5Z && !Q2) {
        const double tau = fabs(be0 - be2);
        X0 = 1.0 + pow(tau / e0, q);
        X1 = 1.0 + pow(tau / e1, q);
        X2 = 1.0 + pow(tau / e2, q);
    } else {
        const double s0 = e0 * e0, s1 = e1 * e1, s2 = e2 * e2;
        X0 = s1 * s2;
        X1 = s0 * s2;
        X2 = s0 * s1;
        if constexpr (REC == REC_W5Z) {
            const double tau = be0 - be2;
            X0 *= fma(tau, tau, s0);
            X1 *= fma(tau, tau, s1);
            X2 *= fma(tau, tau, s2);
        }
    }
    constexpr double K = 0x1p-20;
    const double t0 = 3.0 * K * X0, t1 = 6.0 * K * X1, t2 = 3.0 * K * X2;
    const double nl = fma(t0, fma(4.0, d23, -d34), fma(t1, fma(2.0, d23, d12), X2 * fma(5.0 * K, d12, -2.0 * K * d01)));
    const double nr = fma(t2, fma(4.0, d12, -d01), fma(t1, fma(2.0, d12, d23), X0 * fma(5.0 * K, d23, -2.0 * K * d34)));
    left = fma(1.0 / 6.0, nl / fma(K, X2, t0 + t1), v2);
    right = fma(-1.0 / 6.0, nr / fma(K, X0, t2 + t1), v2);
}

// interface flux (LLF or HLL) from the two states
template <int NF, int RS>
__device__ __forceinline__ void interface_flux(const double UL[NF], const double UR[NF], int d, const MhdConst& C,
                                               double Fh[NF])
{
    double FL[NF], FR[NF], vL, cL, vR, cR;
    flux(UL, d, C.gam, FL, vL, cL);
    flux(UR, d, C.gam, FR, vR, cR);
    if constexpr (NF == 9) {
        FL[5 + d] += UL[8];
        FR[5 + d] += UR[8];
        FL[8] = C.ch2 * UL[5 + d];
        FR[8] = C.ch2 * UR[5 + d];
    }
    if constexpr (RS == RS_HLL) {
        double SL = fmin(vL - cL, vR - cR), SR = fmax(vL + cL, vR + cR);
        if constexpr (NF == 9) {
            SL = fmin(SL, -C.ch);
            SR = fmax(SR, C.ch);
        }
        SL = fmin(SL, 0.0);
        SR = fmax(SR, 0.0);
        // (an explicit last fma: neither kernel fuses the flux into a difference)
        const double id = 1.0 / (SR - SL), aL = SR * id, aR = -SL * id, aU = SR * SL * id;
#pragma unroll
        for (int f = 0; f < NF; ++f) Fh[f] = fma(aL, FL[f], fma(aR, FR[f], aU * (UR[f] - UL[f])));
    } else {
        double S = fmax(fabs(vL) + cL, fabs(vR) + cR);
        if constexpr (NF == 9) S = fmax(S, C.ch);
#pragma unroll
        for (int f = 0; f < 8; ++f) Fh[f] = 0.5 * (FL[f] + FR[f] - S * (UR[f] - UL[f]));
        // (one rounding order: of ch2 U^L + ch2 U^R either product could be fused)
        if constexpr (NF == 9) Fh[8] = 0.5 * fma(-S, UR[8] - UL[8], C.ch2 * (UL[5 + d] + UR[5 + d]));
    }
}

// Interface flux between cells 2 and 3 of a six-cell line: get(f, m) is cell m
// of field f.  LLF and HLL take the states that cell_states gives each of the
// two cells, so that both kernels below give the same bits.
template <int NF, int REC, int RS, bool Q2, class Get>
__device__ __forceinline__ void face_flux(Get get, int d, const MhdConst& C, double Fh[NF])
{
    if constexpr (RS == RS_SPLIT) {
        split_flux<NF, REC, Q2>(get, d, C, Fh);
    } else {
        const double es = REC == REC_W3 ? C.eps : 4.0 * C.eps;
        double UL[NF], UR[NF], unused;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const double c0 = get(f, 0), c1 = get(f, 1), c2 = get(f, 2), c3 = get(f, 3), c4 = get(f, 4), c5 = get(f, 5);
            cell_states<REC, Q2>(c0, c1, c2, c3, c4, es, C.q, UL[f], unused);
            cell_states<REC, Q2>(c1, c2, c3, c4, c5, es, C.q, unused, UR[f]);
        }
        interface_flux<NF, RS>(UL, UR, d, C, Fh);
    }
}

// The value of the lane one above (below) in the row of 16 lanes.
template <int CTRL>
__device__ __forceinline__ double row_dpp(double v)
{
    const int2 u = __builtin_bit_cast(int2, v);
    int2 r;
    r.x = __builtin_amdgcn_update_dpp(0, u.x, CTRL, 0xf, 0xf, true);
    r.y = __builtin_amdgcn_update_dpp(0, u.y, CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, r);
}
constexpr int DPP_FROM_NEXT = 0x101, DPP_FROM_PREV = 0x111;  // row_shl:1, row_shr:1

// LLF and HLL fluxes.  One workgroup of 16 x 16 threads owns a tile of 14 x 16
// columns and marches along z over zc planes; thread (tx, ty) stands for the
// cell (tx - 1, ty) of each plane, and along every axis it reconstructs both
// states of its cell at once (cell_states) and evaluates the flux on the far
// side of the cell with the near state of the next cell:
//   z: from a 5-cell register window of the column, the left state and the
//      flux below carried from the plane before;
//   x: the next cell is the next lane of the row of 16, so states and fluxes
//      pass through DPP moves (lanes 0 and 15 are the cells beyond the tile);
//   y: through LDS; the threads of lanes 0 and 15, which own no column, take
//      the cells of the rows below and above the tile.
// The plane with its x/y halo comes into LDS by 16-byte LDS-DMA loads, one
// plane ahead.  Why cells instead of interfaces: the kernel is bound by FP64
// issue, and the indicators, most of the reconstruction's arithmetic, are the
// same for both states of a cell.  Interface by interface before, this after
// (128^3, rough data, LLF; HLL within 2%): SSP-RK3 stage WENO5-Z 0.597 -> 0.397
// ms, WENO5-JS 0.565 -> 0.385, WENO3 0.433 -> 0.276; RK4 stage, five arrays
// instead of three, 0.641 -> 0.433, 0.614 -> 0.421 and 0.484 -> 0.301.  A sixth
// of it came from requesting a point's stage inputs together and a further 4%
// from two barriers per plane instead of four.
// The scheduling barriers keep two fields' reconstructions in flight at a
// time: without them the kernel spills.  The WENO5 instances take more than
// 256 registers and run one wave per SIMD without scratch (held to two waves
// they spill 300 bytes per lane: 0.58 against 0.41 ms at 128^3); WENO3 fits
// two waves, and two workgroups in a CU's LDS if the exchange along y uses
// one array and two barriers more (0.25 against 0.30 ms).
constexpr int CX = MHD_CX, CY = MHD_CY;

template <int NF, int REC, int RS, bool Q2>
__global__ __launch_bounds__(256, REC == REC_W3 ? 2 : 1) void mhd_cells_kernel(StageArgs a, MhdConst C, int zc)
{
    constexpr int H = REC == REC_W3 ? 2 : 3;  // halo: reach of the states of the cells beyond the tile
    constexpr int CHX = CX + 2 * H, CHY = CY + 2 * H;
    constexpr bool TWO = REC != REC_W3;
    __shared__ double pl[2][NF][CHY][CHX];
    // y exchange, rows -1 .. CY of cells: near states and fluxes.  With two
    // arrays, two barriers per plane order all uses of LDS: states written |
    // states read, fluxes written, next plane arrived | fluxes read.
    __shared__ double ey[NF][CY + 2][CX];
    __shared__ double fy_[TWO ? NF : 1][CY + 2][CX];
    auto fy = [&](int f) __attribute__((always_inline)) { return TWO ? fy_[f] : ey[f]; };
    const Tile tile = a.tiles[xcd_tile(blockIdx.x, gridDim.x)];
    const PatchDev P = a.patches[tile.patch];
    const int tx = threadIdx.x, ty = threadIdx.y, tid = tx + 16 * ty;
    const int x0 = tile.o[0], y0 = tile.o[1], z0 = tile.o[2];
    const int z1 = min(z0 + zc, P.n[2]);
    const int64_t fs = P.fs;
    const int sz = P.pitch_z;
    const int cx = x0 + tx - 1, cy = y0 + ty;  // this thread's cell
    const bool col = tx >= 1 && tx <= CX && cx < P.n[0] && cy < P.n[1];
    // its column (the ghosted box's last one for cells beyond it, which feed
    // no column of the patch)
    const double* __restrict__ Us = a.Us;
    const int64_t colbase = P.off + (int64_t)(min(cy, P.n[1] + G - 1) + G) * P.pitch_y + (min(cx, P.n[0] + G - 1) + G);
    // cell of the y sweep: its column and row in the tile (rows -1 .. CY)
    const int yc = tx == 0 || tx == 15 ? min(ty, CX - 1) : tx - 1;
    const int yr = tx == 0 ? -1 : (tx == 15 ? CY : ty);
    // LDS-DMA of a plane: one load per field, thread tid the tid-th 16-byte
    // chunk of the CHY x CHX doubles
    constexpr int NCH = CHY * CHX / 2;
    static_assert(NCH <= 256 && CHX % 2 == 0, "one chunk per thread and field");
    const int hy = tid / (CHX / 2) + G - H, hx = 2 * (tid % (CHX / 2)) + G - H;  // in the ghosted box
    // (a chunk of the narrower halo starts at an odd column: one that would end
    // beyond the box holds nothing that is needed)
    const int doff = x0 + hx + (G - H) % 2 < P.n[0] + 2 * G && y0 + hy < P.n[1] + 2 * G ? hy * P.pitch_y + hx : 0;
    const int64_t tbase = P.off + (int64_t)y0 * P.pitch_y + x0;
    auto dma = [&](int k, int b) __attribute__((always_inline)) {
        const double* src = Us + tbase + (int64_t)(k + G) * sz;
        if (tid < NCH)
#pragma unroll
            for (int f = 0; f < NF; ++f)
                __builtin_amdgcn_global_load_lds((const void*)(src + f * fs + doff),
                                                 (lds_void*)(&pl[b][f][0][0] + 2 * (tid & ~63)), 16, 0, 0);
    };
    const double es = REC == REC_W3 ? C.eps : 4.0 * C.eps;

    const StageCoef sc = stage_coef(a);
    dma(z0, 0);
    double w[NF][5];             // cells k-1 .. k+3 of the column
    double ULz[NF], Fz[NF];      // left state of cell k, z flux below cell k
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int m = 0; m < 5; ++m) w[f][m] = Us[colbase + f * fs + (int64_t)(z0 - 3 + m + G) * sz];
    // two lead-in steps bring the left state of cell z0 and the flux below it
    for (int k = z0 - 2; k < z1; ++k) {
        const int b = (k - z0) & 1;
        if (k >= z0 && k + 1 < z1) dma(k + 1, b ^ 1);
        // ---- z: states of cell k + 1, flux between cells k and k + 1
        double r[NF];
        {
            double UL[NF], UR[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                cell_states<REC, Q2>(w[f][0], w[f][1], w[f][2], w[f][3], w[f][4], es, C.q, UL[f], UR[f]);
                if (f % 2) __builtin_amdgcn_sched_barrier(0);
            }
            if (k >= z0 - 1) {
                double F[NF];
                interface_flux<NF, RS>(ULz, UR, 2, C, F);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    r[f] = F[f] - Fz[f];
                    Fz[f] = F[f];
                }
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                ULz[f] = UL[f];
#pragma unroll
                for (int m = 0; m < 4; ++m) w[f][m] = w[f][m + 1];
                w[f][4] = k + 1 < z1 ? Us[colbase + f * fs + (int64_t)(k + 4 + G) * sz] : 0.0;
            }
        }
        if (k < z0) continue;
        if (k == z0) {
            __builtin_amdgcn_s_waitcnt(VM_WAIT);  // the first plane
            lds_barrier();
        }
        // ---- x
        {
            double UL[NF], UR[NF], F[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const double* p = &pl[b][f][ty + H][tx + H - 1];
                cell_states<REC, Q2>(TWO ? p[-2] : 0.0, p[-1], p[0], p[1], TWO ? p[2] : 0.0, es, C.q, UL[f], UR[f]);
                UR[f] = row_dpp<DPP_FROM_NEXT>(UR[f]);
                if (f % 2) __builtin_amdgcn_sched_barrier(0);
            }
            interface_flux<NF, RS>(UL, UR, 0, C, F);
#pragma unroll
            for (int f = 0; f < NF; ++f) r[f] += F[f] - row_dpp<DPP_FROM_PREV>(F[f]);
        }
        // ---- y; the stage update's inputs are requested together before the
        // last exchange (one latency instead of one per field)
        double pu[NF], pw[NF], psi = 0.0;
        const int64_t cidx = colbase + (int64_t)(k + G) * sz;
        {
            double UL[NF], UR[NF], F[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const double* p = &pl[b][f][yr + H][yc + H];
                cell_states<REC, Q2>(TWO ? p[-2 * CHX] : 0.0, p[-CHX], p[0], p[CHX], TWO ? p[2 * CHX] : 0.0, es, C.q,
                                     UL[f], UR[f]);
                ey[f][yr + 1][yc] = UR[f];
                if (f % 2) __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (NF == 9) psi = pl[b][8][ty + H][tx + H - 1];
            lds_barrier();
            const int up = min(yr + 2, CY + 1);
#pragma unroll
            for (int f = 0; f < NF; ++f) UR[f] = ey[f][up][yc];
            if constexpr (!TWO) lds_barrier();
            interface_flux<NF, RS>(UL, UR, 1, C, F);
#pragma unroll
            for (int f = 0; f < NF; ++f) fy(f)[yr + 1][yc] = F[f];
            __builtin_amdgcn_s_waitcnt(VM_WAIT);  // the next plane
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                pu[f] = sc.pun[cidx + f * fs];
                pw[f] = sc.pw[cidx + f * fs];
            }
            lds_barrier();
#pragma unroll
            for (int f = 0; f < NF; ++f) r[f] += F[f] - fy(f)[max(yr, 0)][yc];
        }
        if (col) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                // psi: the damping source at the cell
                const double rhs = f == 8 ? -r[f] * C.ih - C.kpsi * psi : -r[f] * C.ih;
                a.out[cidx + f * fs] = stage_update(a, sc, cidx + f * fs, rhs, pu[f], pw[f]);
            }
        }
        if constexpr (!TWO) lds_barrier();
    }
}

// Interface by interface: flux splitting (its reconstruction depends on the
// interface, so nothing is shared between the states of a cell), and LLF and HLL
// on levels whose patches its 15 x 15 columns fit so much better than 14 x 16
// that twice the reconstructions cost less (125 patches of 15^3, where the cell
// kernel needs two tiles per patch: WENO5-Z 147 -> 111 us).
// One workgroup of 16 x 16 threads owns a tile of 15 x 15 columns and marches
// along z over ZC planes.  Per plane: the plane (with a 3-cell halo in x and
// y) is staged in LDS; thread (tx, ty) computes the x-interface flux to the
// left of column (tx, ty) and the y-interface flux below it (the extra row and
// column of threads supply the fluxes on the far side of the tile), so every
// interface flux is computed once; the z-interface flux above the plane comes
// from a 6-cell register window carried along the column, the one below from
// the previous plane.  Then the flux differences form the right-hand side and
// the RK stage update is applied.
constexpr int MT = 15;           // columns per tile edge
constexpr int MB = MT + 1;       // threads per tile edge
constexpr int MH = MT + 6;       // plane width with halo
constexpr int MP = MH + 1;       // LDS row pitch

template <int NF, int REC, int RS, bool Q2>
__global__ __launch_bounds__(MB * MB) void mhd_faces_kernel(StageArgs a, MhdConst C, int zc)
{
    __shared__ double pl[NF][MH][MP];
    __shared__ double fx[NF][MT][MB];
    __shared__ double fy[NF][MB][MT];
    const Tile tile = a.tiles[xcd_tile(blockIdx.x, gridDim.x)];
    const PatchDev P = a.patches[tile.patch];
    const int tx = threadIdx.x, ty = threadIdx.y, tid = tx + MB * ty;
    const int x0 = tile.o[0], y0 = tile.o[1], z0 = tile.o[2];
    const int z1 = min(z0 + zc, P.n[2]);
    const int64_t fs = P.fs;
    const int sz = P.pitch_z;
    const bool col = tx < MT && ty < MT && x0 + tx < P.n[0] && y0 + ty < P.n[1];
    // ghosted-box coordinates of this thread's column
    const int64_t colbase = P.off + (int64_t)(y0 + ty + G) * P.pitch_y + (x0 + tx + G);
    const double* __restrict__ Us = a.Us;

    [[maybe_unused]] const StageCoef sc = stage_coef(a);
    double w[NF][6];  // cells k-2 .. k+3 of the own column
    double Fm[NF];    // z-flux below the current plane
    if (col) {
        double c7[NF][7];
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int m = 0; m < 7; ++m) c7[f][m] = Us[colbase + f * fs + (int64_t)(z0 - 3 + m + G) * sz];
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int m = 0; m < 6; ++m) w[f][m] = c7[f][m + 1];
        face_flux<NF, REC, RS, Q2>([&](int f, int m) { return c7[f][m]; }, 2, C, Fm);
    }
    for (int k = z0; k < z1; ++k) {
        // stage plane k with its x/y halo
        const int64_t pbase = P.off + (int64_t)(k + G) * sz + (int64_t)y0 * P.pitch_y + x0;
        for (int e = tid; e < NF * MH * MH; e += MB * MB) {
            const int f = e / (MH * MH), r = e - f * MH * MH, hy = r / MH, hx = r - hy * MH;
            const bool ok = x0 + hx < P.n[0] + 2 * G && y0 + hy < P.n[1] + 2 * G;
            pl[f][hy][hx] = ok ? Us[pbase + f * fs + (int64_t)hy * P.pitch_y + hx] : 0.0;
        }
        __syncthreads();
        // x-interface to the left of column (tx, ty): cells tx-3 .. tx+2 of row ty
        double Fp[NF];
        if (col) face_flux<NF, REC, RS, Q2>([&](int f, int m) { return w[f][m]; }, 2, C, Fp);
        if (ty < MT && x0 + tx <= P.n[0] && y0 + ty < P.n[1]) {
            double F[NF];
            face_flux<NF, REC, RS, Q2>([&](int f, int m) { return pl[f][ty + G][tx + m]; }, 0, C, F);
#pragma unroll
            for (int f = 0; f < NF; ++f) fx[f][ty][tx] = F[f];
        }
        // y-interface below column (tx, ty)
        if (tx < MT && y0 + ty <= P.n[1] && x0 + tx < P.n[0]) {
            double F[NF];
            face_flux<NF, REC, RS, Q2>([&](int f, int m) { return pl[f][ty + m][tx + G]; }, 1, C, F);
#pragma unroll
            for (int f = 0; f < NF; ++f) fy[f][ty][tx] = F[f];
        }
        __syncthreads();
        if (col) {
            const int64_t cidx = colbase + (int64_t)(k + G) * sz;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const double dx = fx[f][ty][tx + 1] - fx[f][ty][tx], dy = fy[f][ty + 1][tx] - fy[f][ty][tx];
                // (LLF, HLL: in the cell kernel's order)
                const double div = RS == RS_SPLIT ? dx + dy + (Fp[f] - Fm[f]) : (Fp[f] - Fm[f]) + dx + dy;
                // psi: the damping source at the cell (w[8][2] is plane k of the column)
                const double rhs = f == 8 ? -div * C.ih - C.kpsi * w[f][2] : -div * C.ih;
                const int64_t i = cidx + f * fs;
                if constexpr (RS == RS_SPLIT)
                    stage_store(a, i, rhs);
                else
                    a.out[i] = stage_update(a, sc, i, rhs, sc.pun[i], sc.pw[i]);
            }
            if (k + 1 < z1) {
#pragma unroll
                for (int f = 0; f < NF; ++f) {
#pragma unroll
                    for (int m = 0; m < 5; ++m) w[f][m] = w[f][m + 1];
                    w[f][5] = Us[colbase + f * fs + (int64_t)(k + 4 + G) * sz];
                    Fm[f] = Fp[f];
                }
            }
        }
        __syncthreads();
    }
}

template <int NF, int REC, bool Q2>
void launch(const SysParams& sp, const StageArgs& a, const MhdConst& C, int zc, hipStream_t s)
{
    auto go = [&](auto kernel) { kernel<<<a.ntiles, dim3(16, 16, 1), 0, s>>>(a, C, zc); };
    const bool hll = sp.mhd_flux == MOL_FLUX_HLL;
    if (sp.mhd_flux == MOL_FLUX_SPLIT)
        go(mhd_faces_kernel<NF, REC, RS_SPLIT, Q2>);
    else if (sp.mhd_cells)
        hll ? go(mhd_cells_kernel<NF, REC, RS_HLL, Q2>) : go(mhd_cells_kernel<NF, REC, RS_LLF, Q2>);
    else if constexpr ((NF == 8 || REC == REC_W3) && Q2)
        hll ? go(mhd_faces_kernel<NF, REC, RS_HLL, Q2>) : go(mhd_faces_kernel<NF, REC, RS_LLF, Q2>);
}

template <int NF>
hipError_t dispatch(const SysParams& sp, const StageArgs& a, const MhdConst& C, int zc, hipStream_t s)
{
    switch (sp.mhd_recon) {
    case MOL_RECON_WENO3: launch<NF, REC_W3, true>(sp, a, C, zc, s); break;
    case MOL_RECON_WENO5JS: launch<NF, REC_W5JS, true>(sp, a, C, zc, s); break;
    default: C.q == 2.0 ? launch<NF, REC_W5Z, true>(sp, a, C, zc, s) : launch<NF, REC_W5Z, false>(sp, a, C, zc, s);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_stage_mhd(const SysParams& sp, const StageArgs& a, const int td[3], hipStream_t s)
{
    if (a.ntiles <= 0) return hipSuccess;
    MhdConst C;
    C.gam = sp.gamma_ad;
    const double h2 = sp.h * sp.h;
    const double e = sp.weno_eps > 0.0 ? sp.weno_eps : (sp.mhd_recon == MOL_RECON_WENO3 ? h2 : h2 * h2);
    C.eps = e;
    C.q = sp.weno_q;
    C.ih = 1.0 / sp.h;
    if (td[0] != MT || td[1] != MT) return hipErrorInvalidConfiguration;
    C.ch = sp.mhd_ch;
    C.ch2 = sp.mhd_ch * sp.mhd_ch;
    C.kpsi = sp.mhd_kpsi;
    if (sp.system == MOL_MHD_GLM) return dispatch<9>(sp, a, C, td[2], s);
    return dispatch<8>(sp, a, C, td[2], s);
}

}  // namespace mol
