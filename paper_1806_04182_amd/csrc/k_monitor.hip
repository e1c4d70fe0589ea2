// Constraint and dissipation monitors of a level (Sec. V: Theta, Z^i,
// the bracket H_Z of the Theta equation, the conformal constraints
// ln det gt = 0 and tr At = 0; Sec. II.B.1: the size of the KO term),
// reduced deterministically (fixed tile walk, fixed fold of the block's waves,
// one final block) like the norms.  Here: the point-wise ones, the KO term and,
// where that is faster, |Z|, one thread per interior point; other masks with
// |Z| or H_Z, which need the metric's geometry, go to the CCZ4 stage kernel's
// monitor form.
#include <algorithm>

#include "k_common.h"

namespace mol {

namespace {

constexpr int RB = 256;
constexpr int NQ = MON_VALUES;

// 4th-order stencils of Sec. II.B.1 along stride s: first derivative, dissipation
__device__ __forceinline__ double d1(const double* u, int64_t s, double i12h)
{
    return (8.0 * (u[s] - u[-s]) - (u[2 * s] - u[-2 * s])) * i12h;
}
__device__ __forceinline__ double ko(const double* u, int64_t s, double kc)
{
    const double c = u[0];
    const double a1 = (u[s] - c) + (u[-s] - c), a2 = (u[2 * s] - c) + (u[-2 * s] - c),
                 a3 = (u[3 * s] - c) + (u[-3 * s] - c);
    return (a3 - 6.0 * a2 + 15.0 * a1) * kc;
}

// CCZ4 field order
enum { F_CHI = 0, F_GT = 1, F_AT = 8, F_GH = 14, F_TH = 17 };
__device__ __forceinline__ int sym(int i, int j)
{
    // xx xy xz yy yz zz
    return i == j ? (i == 0 ? 0 : (i == 1 ? 3 : 5)) : (i + j == 1 ? 1 : (i + j == 2 ? 2 : 4));
}

struct MonArgs {
    const PatchDev* patches;
    const Tile* tiles;
    int ntiles;
    int nf;
    int ccz4;
    unsigned which;
    double h, sigma;
    const double* U;
    double* point;  // nullable: requested monitors at interior points, field k = k-th requested
    double* partial;
};

// ZED: with |Z|, without the KO term (|Z|'s registers would cost the other
// masks three waves per SIMD)
template <bool ZED>
__global__ __launch_bounds__(RB) void monitor_kernel(MonArgs a)
{
    __shared__ double sh[NQ * 4];
    double r[NQ];
    for (int q = 0; q < NQ; ++q) r[q] = 0.0;
    const double h = a.h, dV = h * h * h;
    const double i12h = 1.0 / (12.0 * h), kcoef = a.sigma / (64.0 * h);
    for (int tt = blockIdx.x; tt < a.ntiles; tt += gridDim.x) {
        const Tile t = a.tiles[tt];
        const PatchDev P = a.patches[t.patch];
        const int i = t.o[0] + threadIdx.x, j = t.o[1] + threadIdx.y, k = t.o[2] + threadIdx.z;
        if (i >= P.n[0] || j >= P.n[1] || k >= P.n[2]) continue;
        const int64_t c = P.off + (int64_t)(k + G) * P.pitch_z + (int64_t)(j + G) * P.pitch_y + i + G;
        const int64_t st[3] = {1, P.pitch_y, P.pitch_z};
        const double* U = a.U + c;
        for (int f = 0; f < a.nf; ++f)
            if (!isfinite(U[f * P.fs])) r[3 * MOL_MON_COUNT] += 1.0;
        double mon[MOL_MON_COUNT];
        if (!ZED && (a.which & MOL_MON_KO)) {
            double s = 0.0;
            for (int f = 0; f < a.nf; ++f) {
                const double* u = U + f * P.fs;
                const double q = ko(u, st[0], kcoef) + ko(u, st[1], kcoef) + ko(u, st[2], kcoef);
                s += q * q;
            }
            mon[5] = sqrt(s);
        }
        if (!ZED && a.ccz4 && (a.which & (MOL_MON_THETA | MOL_MON_LNDET | MOL_MON_TRA))) {
            const int64_t fs = P.fs;
            double g[3][3], A[3][3];
            for (int p = 0; p < 3; ++p)
                for (int q = 0; q < 3; ++q) {
                    g[p][q] = U[(F_GT + sym(p, q)) * fs];
                    A[p][q] = U[(F_AT + sym(p, q)) * fs];
                }
            // ln det gt from h = gt - I (no cancellation), and the inverse
            const double hx = g[0][0] - 1.0, hy = g[1][1] - 1.0, hz = g[2][2] - 1.0;
            const double cxx = g[1][1] * g[2][2] - g[1][2] * g[1][2], cxy = g[0][2] * g[1][2] - g[0][1] * g[2][2],
                         cxz = g[0][1] * g[1][2] - g[0][2] * g[1][1], cyy = g[0][0] * g[2][2] - g[0][2] * g[0][2],
                         cyz = g[0][1] * g[0][2] - g[0][0] * g[1][2], czz = g[0][0] * g[1][1] - g[0][1] * g[0][1];
            const double dm = (hx + hy + hz) +
                              ((hx * hy - g[0][1] * g[0][1]) + (hx * hz - g[0][2] * g[0][2]) +
                               (hy * hz - g[1][2] * g[1][2])) +
                              (hx * (hy * hz - g[1][2] * g[1][2]) - g[0][1] * (g[0][1] * hz - g[1][2] * g[0][2]) +
                               g[0][2] * (g[0][1] * g[1][2] - hy * g[0][2]));
            const double idet = 1.0 / (1.0 + dm);
            double gi[3][3];
            gi[0][0] = cxx * idet;
            gi[0][1] = gi[1][0] = cxy * idet;
            gi[0][2] = gi[2][0] = cxz * idet;
            gi[1][1] = cyy * idet;
            gi[1][2] = gi[2][1] = cyz * idet;
            gi[2][2] = czz * idet;
            mon[0] = U[F_TH * fs];
            mon[3] = log1p(dm);
            double trA = 0.0;
            for (int p = 0; p < 3; ++p)
                for (int q = 0; q < 3; ++q) trA += gi[p][q] * A[p][q];
            mon[4] = trA;
        }
        if constexpr (ZED) {
            // the streamed form's operations in its order (asm and sym_trace keep
            // the compiler from fusing them in another way; the same bits):
            // dg[m] = d_m gt, Gu[i] = Gt^i_jk
            const int64_t fs = P.fs;
            const double chi = U[F_CHI * fs];
            double g[6], gu[6], A[6], dg[3][6], Gl[3][6], Gu[3][6], Z[3], zz = 0.0, trA = 0.0;
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                g[q] = U[(F_GT + q) * fs];
                A[q] = U[(F_AT + q) * fs];
            }
            const double dm = metric_inverse(g, gu);
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    dg[m][q] = d1(U + (F_GT + q) * fs, st[m], i12h);
                    asm("" : "+v"(dg[m][q]));
                }
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int r = q; r < 3; ++r)
                        Gl[p][sym(q, r)] = 0.5 * (dg[q][sym(p, r)] + dg[r][sym(p, q)] - dg[p][sym(q, r)]);
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int m = 0; m < 6; ++m)
                    Gu[p][m] = gu[sym(p, 0)] * Gl[0][m] + gu[sym(p, 1)] * Gl[1][m] + gu[sym(p, 2)] * Gl[2][m];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const double Gc = sym_trace(gu, Gu[p]);
                Z[p] = 0.5 * chi * (U[(F_GH + p) * fs] - Gc);
            }
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    zz += g[sym(p, q)] * Z[p] * Z[q];
                    trA += gu[sym(p, q)] * A[sym(p, q)];
                }
            mon[0] = U[F_TH * fs];
            mon[1] = sqrt(zz / chi);
            mon[3] = log1p(dm);
            mon[4] = trA;
        }
        int rank = 0;
        for (int q = 0; q < MOL_MON_COUNT; ++q) {
            if (!(a.which >> q & 1u)) continue;
            const double v = mon[q];
            if (a.point) a.point[c + rank * P.fs] = v;
            ++rank;
            if (!isfinite(v)) continue;
            r[3 * q] += fabs(v) * dV;
            r[3 * q + 1] += v * v * dV;
            r[3 * q + 2] = fmax(r[3 * q + 2], fabs(v));
        }
    }
    mon_block_reduce(r, sh);
    if (threadIdx.x == 0 && threadIdx.y == 0 && threadIdx.z == 0)
        for (int q = 0; q < NQ; ++q) a.partial[blockIdx.x * NQ + q] = r[q];
}

__global__ __launch_bounds__(RB) void monitor_final_kernel(const double* __restrict__ partial, int nb,
                                                           double* __restrict__ out)
{
    __shared__ double sh[NQ * 4];
    double r[NQ];
    for (int q = 0; q < NQ; ++q) r[q] = 0.0;
    const int t = threadIdx.x;
    for (int b = t; b < nb; b += RB)
        for (int q = 0; q < NQ; ++q) {
            const double v = partial[b * NQ + q];
            r[q] = mon_is_max(q) ? fmax(r[q], v) : r[q] + v;
        }
    mon_block_reduce(r, sh);
    if (t == 0)
        for (int q = 0; q < NQ; ++q) out[q] = r[q];
}

}  // namespace

int monitor_partials() { return NQ; }

hipError_t launch_monitor(const PatchDev* patches, const Tile* tiles, int ntiles, const int td[3], const Tile* ctiles,
                          int nctiles, int nf, int ccz4,
                          unsigned which, double h, double sigma, const double* U, double* point, double* partial,
                          int nblocks, double* out, hipStream_t s)
{
    hipError_t e;
    const bool z = ccz4 && (which & MOL_MON_Z);
    // |Z| without H_Z and the KO term reads six fields' first derivatives, but
    // the streamed form passes all 25 fields: point-wise on levels of at most
    // one streamed tile per two compute units, which wait for the passes (8^3
    // to 32^3 points 20 against 32 us, 40^3 41 and 33), and where the point-wise
    // tiles are no more (whole rows of 32: 64^3 57 and 67 us, 96^3 153 and 182;
    // elsewhere, 80^3: 124 and 115, 64 patches of 16^3: 102 and 67)
    const bool direct = z && !(which & (MOL_MON_HZ | MOL_MON_KO)) && (nctiles <= 128 || ntiles <= nctiles);
    const bool stream = ccz4 && (which & (MOL_MON_Z | MOL_MON_HZ)) && !direct;
    // one block per tile up to nblocks, two per compute unit (|Z| point-wise
    // takes a compute unit: half as many; the streamed form walks the tiles by
    // XCD: a block for each of the eight).  More blocks than tiles cost the
    // final fold: wave 8^3 17.3 -> 15.7 us with 8 instead of 512
    nblocks = stream ? std::clamp(nctiles, 8, nblocks) : std::clamp(ntiles, 1, direct ? nblocks / 2 : nblocks);
    if (stream) {
        e = launch_ccz4_monitor(patches, ctiles, nctiles, which, h, sigma, U, point, partial, nblocks, s);
    } else {
        MonArgs a{patches, tiles, ntiles, nf, ccz4, which, h, sigma, U, point, partial};
        const dim3 b(td[0], td[1], td[2]);
        z ? monitor_kernel<true><<<nblocks, b, 0, s>>>(a) : monitor_kernel<false><<<nblocks, b, 0, s>>>(a);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    monitor_final_kernel<<<1, RB, 0, s>>>(partial, nblocks, out);
    return hipGetLastError();
}

}  // namespace mol
