// Ghost fill, its transpose, coarse-fine prolongation and injection kernels
// (the data movement of the Sec. III skeleton), plus a vector update used
// by the RK4 adjoint.
#include <algorithm>

#include "k_common.h"

namespace mol {

namespace {

constexpr int BLK = 256;

int grid_for(int64_t n)
{
    int64_t b = (n + BLK - 1) / BLK;
    return (int)(b < 1 ? 1 : (b > 65535 * 8 ? 65535 * 8 : b));
}

// Launches of one thread per (point, field or group of fields): points along
// x, fields along y, so that no thread divides 64-bit indices to find its
// point (the channel's coarse step of 14 fills and 8 band launches: 178 ->
// 172 us; large launches do not change)
dim3 grid_for(int64_t n, int nf) { return dim3(grid_for(n), nf, 1); }
__device__ __forceinline__ int64_t first_point() { return blockIdx.x * (int64_t)BLK + threadIdx.x; }
__device__ __forceinline__ int64_t next_point() { return (int64_t)gridDim.x * BLK; }

// Copies of nf fields between two points: the loads of up to FC fields are
// issued together before their stores.
constexpr int FC = 8;
__device__ __forceinline__ void copy_fields(const double* __restrict__ src, int64_t sfs, double* __restrict__ dst,
                                            int64_t dfs, int nf)
{
    for (int f0 = 0; f0 < nf; f0 += FC) {
        double v[FC];
#pragma unroll
        for (int j = 0; j < FC; ++j)
            if (f0 + j < nf) v[j] = src[(f0 + j) * sfs];
#pragma unroll
        for (int j = 0; j < FC; ++j)
            if (f0 + j < nf) dst[(f0 + j) * dfs] = v[j];
    }
}

// same-level / periodic copy: ghost <- interior point of the owning patch.
// One thread per (ghost point, group of FC fields), the group in the grid's y,
// so that a launch has ceil(nf / FC) times as many threads, each with one
// batch of loads in flight, and consecutive threads still copy consecutive
// points.
__global__ __launch_bounds__(BLK) void fill_kernel(const GhostCopy* __restrict__ e, int64_t n, int nf,
                                                   double* __restrict__ U)
{
    const int f0 = blockIdx.y * FC;
    for (int64_t t = first_point(); t < n; t += next_point()) {
        const GhostCopy c = e[t];
        copy_fields(U + c.src + f0 * c.sfs, c.sfs, U + c.dst + f0 * c.dfs, c.dfs, min(FC, nf - f0));
    }
}

// transpose of the copy: source += its images, images <- 0; one thread per
// (source point, field), the field the slow index (every address is touched
// by exactly one thread)
__global__ __launch_bounds__(BLK) void fill_adjoint_kernel(const GhostSource* __restrict__ src, int64_t n,
                                                           const GhostImage* __restrict__ img, int nf,
                                                           double* __restrict__ A)
{
    const int64_t f = blockIdx.y;
    for (int64_t t = first_point(); t < n; t += next_point()) {
        const GhostSource s = src[t];
        double acc = A[s.src + f * s.sfs];
        for (int q = s.beg; q < s.end; ++q) {
            const int64_t d = img[q].dst + f * img[q].dfs;
            acc += A[d];
            A[d] = 0.0;
        }
        A[s.src + f * s.sfs] = acc;
    }
}

constexpr int PROLONG_FPW = 9;  // fields per workgroup of the prolongation at most
struct BorW {
    double w[4];
};

// parent BOR stage state (App. D) T = U^n + sum_j w_j k_j on the band of
// parent points that the prolongation stencils read.  A band entry writes T at
// its position in some parent patch's ghosted box (dst) from the interior
// point that owns it (src), so the parent's k arrays need no ghost fill.
// One thread per (point, field).
__global__ __launch_bounds__(BLK) void bor_band_kernel(const GhostCopy* __restrict__ band, int64_t n, int nf,
                                                       BorW W, const double* __restrict__ Un,
                                                       const double* __restrict__ k0,
                                                       const double* __restrict__ k1,
                                                       const double* __restrict__ k2,
                                                       const double* __restrict__ k3, double* __restrict__ T)
{
    const int f = blockIdx.y;
    for (int64_t t = first_point(); t < n; t += next_point()) {
        const GhostCopy b = band[t];
        const int64_t q = b.src + f * b.sfs;
        T[b.dst + f * b.dfs] = Un[q] + W.w[0] * k0[q] + W.w[1] * k1[q] + W.w[2] * k2[q] + W.w[3] * k3[q];
    }
}

// Lagrange weights at xi = m / R, m = 0 .. R-1
struct LagW {
    double w[4][6];
};

// Coarse-fine ghost points: tensor-product quintic Lagrange interpolation
// (Sec. III.A) of the parent's BOR stage state.  One workgroup per (brick of
// parent cells, group of fields): per field, the brick's nodes are loaded into
// LDS once and interpolated axis by axis (x, then y, then z), each stage
// through LDS, the last one storing the brick's present fine points; the next
// field's nodes are in flight meanwhile.  A point with m = 0 on an axis takes
// the node i0 itself (selected, not weighted), so only the nodes of its own
// stencil enter its value; nodes and points of the brick outside the band
// hold whatever the buffer does and reach no present point.
// Why: a cell's stencil is 216 nodes, and neighbouring cells share nearly all
// of them (a brick of 8 x 8 x 2 cells loads 9 nodes per cell).  What is left
// is bound by the index arithmetic of the stages, so the offsets of a
// thread's items are computed once for all fields of the group.  One thread
// per (cell, field) before, this after: 25 fields on the shell of a 32^3 level
// 18.2 -> 10.1 us, ratio 2 around 128^3 points 321 -> 133 us, ratio 3 around
// 192 x 132 x 96 points 110 -> 75 us, two fields on a channel 12.1 -> 3.8 us.
// (Eight lanes per cell: 37, 550, 199, 6.3 us; one field per workgroup: 11.5,
// 228, 132, 3.5 us; U^n + sum w k formed here instead of by bor_band_kernel:
// 21 us on the 32^3 shell against 10 and 8 us apart.)
template <int R>
__global__ __launch_bounds__(BLK) void prolong_kernel(const ProlongBrick* __restrict__ e, int nb, int nf, int fpw,
                                                      const uint32_t* __restrict__ rows, LagW L,
                                                      const double* __restrict__ T, double* __restrict__ U)
{
    constexpr int N0 = brick_items(R, 0), N1 = brick_items(R, 1), N2 = brick_items(R, 2), N3 = brick_items(R, 3);
    constexpr int I0 = (N0 + BLK - 1) / BLK, I1 = (N1 + BLK - 1) / BLK, I2 = (N2 + BLK - 1) / BLK,
                  I3 = (N3 + BLK - 1) / BLK;
    __shared__ double A[N0 > N2 * R ? N0 : N2 * R];  // nodes [z][y][x]; then values [z][fine y][fine x]
    __shared__ double B[N1 * R];                     // values [z][y][fine x]
    static_assert(N1 * R < 65536 && N2 * R < 65536, "packed LDS offsets");
    const int tid = threadIdx.x, grp = blockIdx.x / nb;
    const ProlongBrick c = e[blockIdx.x - grp * nb];
    const int f0 = grp * fpw, f1 = min(f0 + fpw, nf);
    const int nx = c.n[0], ny = c.n[1], nz = c.n[2], ax = nx + 5, ay = ny + 5, az = nz + 5, fx = nx * R, fy = ny * R;
    const int n0 = ax * ay * az, n1 = nx * ay * az, n2 = fx * ny * az, n3 = fx * fy * nz;
    // t / n for small non-negative t, with i = 1 / n: the half keeps the product
    // clear of the integers (t < 4096, n <= 64)
    auto quot = [](int t, float i) __attribute__((always_inline)) { return (int)(((float)t + 0.5f) * i); };
    const float iax = 1.0f / ax, iay = 1.0f / ay, inx = 1.0f / nx, ifx = 1.0f / fx, iny = 1.0f / ny, ify = 1.0f / fy;
    // offsets of this thread's items: nodes in the parent; LDS source and
    // result (packed) of the x and y stages; fine point and its presence bits
    int g0[I0], l1[I1], l2[I2], g3[I3], b3[I3];
#pragma unroll
    for (int i = 0; i < I0; ++i) {
        const int t = tid + i * BLK, r = quot(t, iax), x = t - r * ax, z = quot(r, iay), y = r - z * ay;
        g0[i] = t < n0 ? z * c.cpz + y * c.cpy + x : 0;
    }
#pragma unroll
    for (int i = 0; i < I1; ++i) {
        const int t = tid + i * BLK, r = quot(t, inx), x = t - r * nx;
        l1[i] = (r * ax + x) | (r * fx + x * R) << 16;
    }
#pragma unroll
    for (int i = 0; i < I2; ++i) {
        const int t = tid + i * BLK, r = quot(t, ifx), x = t - r * fx, z = quot(r, iny), y = r - z * ny;
        l2[i] = ((z * ay + y) * fx + x) | ((z * fy + y * R) * fx + x) << 16;
    }
#pragma unroll
    for (int i = 0; i < I3; ++i) {
        const int t = tid + i * BLK, r = quot(t, ifx), x = t - r * fx, z = quot(r, ify), y = r - z * fy;
        g3[i] = z * R * c.dpz + y * c.dpy + x;
        b3[i] = 0;
        if (t < n3)
#pragma unroll
            for (int m = 0; m < R; ++m) b3[i] |= (int)(rows[c.rows + (z * R + m) * fy + y] >> x & 1) << m;
    }
    // sum over the six nodes at stride s, in order
    auto lag = [&](const double* p, int s, int m) __attribute__((always_inline)) {
        double v = 0.0;
#pragma unroll
        for (int a = 0; a < 6; ++a) v += L.w[m][a] * p[a * s];
        return v;
    };
    const double* __restrict__ src = T + c.cbase;
    double v[I0];
#pragma unroll
    for (int i = 0; i < I0; ++i) v[i] = src[f0 * c.cfs + g0[i]];
    for (int f = f0; f < f1; ++f) {
#pragma unroll
        for (int i = 0; i < I0; ++i)
            if (tid + i * BLK < n0) A[tid + i * BLK] = v[i];
        if (f + 1 < f1)
#pragma unroll
            for (int i = 0; i < I0; ++i) v[i] = src[(f + 1) * c.cfs + g0[i]];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < I1; ++i)
            if (tid + i * BLK < n1) {
                const double* p = A + (l1[i] & 0xffff);
                double* o = B + (l1[i] >> 16);
                o[0] = p[2];
#pragma unroll
                for (int m = 1; m < R; ++m) o[m] = lag(p, 1, m);
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < I2; ++i)
            if (tid + i * BLK < n2) {
                const double* p = B + (l2[i] & 0xffff);
                double* o = A + (l2[i] >> 16);
                o[0] = p[2 * fx];
#pragma unroll
                for (int m = 1; m < R; ++m) o[m * fx] = lag(p, fx, m);
            }
        __syncthreads();
        double* __restrict__ dst = U + c.dbase + f * c.dfs;
#pragma unroll
        for (int i = 0; i < I3; ++i)
            if (b3[i]) {
                const double* p = A + tid + i * BLK;
#pragma unroll
                for (int m = 0; m < R; ++m)
                    if (b3[i] >> m & 1)
                        dst[(int64_t)g3[i] + (int64_t)m * c.dpz] = m == 0 ? p[2 * fx * fy] : lag(p, fx * fy, m);
            }
        __syncthreads();  // before the next field's nodes
    }
}

__global__ __launch_bounds__(BLK) void restrict_kernel(const RestrictPt* __restrict__ e, int64_t n, int nf,
                                                       const double* __restrict__ Uf, double* __restrict__ Uc)
{
    const int f0 = blockIdx.y * FC;
    for (int64_t t = first_point(); t < n; t += next_point()) {
        const RestrictPt r = e[t];
        copy_fields(Uf + r.f + f0 * r.ffs, r.ffs, Uc + r.c + f0 * r.cfs, r.cfs, min(FC, nf - f0));
    }
}

__global__ __launch_bounds__(BLK) void axpby_kernel(int64_t n, double a, const double* x,
                                                    double b, const double* y, double* z)
{
    for (int64_t t = blockIdx.x * (int64_t)BLK + threadIdx.x; t < n; t += (int64_t)gridDim.x * BLK)
        z[t] = a * x[t] + b * y[t];
}

}  // namespace

hipError_t launch_fill(const GhostCopy* e, int64_t n, int nf, double* U, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    fill_kernel<<<grid_for(n, (nf + FC - 1) / FC), BLK, 0, s>>>(e, n, nf, U);
    return hipGetLastError();
}

hipError_t launch_fill_adjoint(const GhostSource* src, int64_t n, const GhostImage* img, int nf, double* A,
                               hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    fill_adjoint_kernel<<<grid_for(n, nf), BLK, 0, s>>>(src, n, img, nf, A);
    return hipGetLastError();
}

// Radiative outer boundary (open domain): one thread per (boundary point,
// field); the right-hand side -v (x^i/r) d_i U - v (U - U_inf)/r with 2nd-order
// differences (centred inside the ghosted array, one-sided at its edge), then
// the same Runge-Kutta stage update as the interior.
__global__ __launch_bounds__(BLK) void radiative_kernel(StageArgs a, PatchDev P, const RadPt* __restrict__ pts,
                                                        int64_t n, int nf, RadParams rp, double x0, double y0,
                                                        double z0, double h)
{
    const int N[3] = {P.n[0] + 2 * G, P.n[1] + 2 * G, P.n[2] + 2 * G};
    const int64_t S[3] = {1, P.pitch_y, P.pitch_z};
    const double xl[3] = {x0, y0, z0}, i2h = 0.5 / h;
    const int f = blockIdx.y;
    for (int64_t t = first_point(); t < n; t += next_point()) {
        const RadPt q = pts[t];
        const int64_t idx = P.off + f * P.fs + q.a[2] * S[2] + q.a[1] * S[1] + q.a[0];
        const double* u = a.Us + idx;
        double x[3], r2 = 0.0;
        for (int d = 0; d < 3; ++d) {
            x[d] = xl[d] + (P.lo[d] + q.a[d] - G) * h;
            r2 += x[d] * x[d];
        }
        const double ir = 1.0 / sqrt(r2);
        double adv = 0.0;
        for (int d = 0; d < 3; ++d) {
            const int64_t s = S[d];
            double du;
            if (q.a[d] == 0)
                du = (-3.0 * u[0] + 4.0 * u[s] - u[2 * s]) * i2h;
            else if (q.a[d] == N[d] - 1)
                du = (3.0 * u[0] - 4.0 * u[-s] + u[-2 * s]) * i2h;
            else
                du = (u[s] - u[-s]) * i2h;
            adv += x[d] * ir * du;
        }
        const double rhs = -rp.v[f] * adv - rp.v[f] * (u[0] - rp.uinf[f]) * ir;
        stage_apply(a, idx, rhs, stage_load(a, idx));
    }
}

// copy between two level buffers (regrid): dst[e.dst + f dfs] = src[e.src + f sfs]
__global__ __launch_bounds__(BLK) void copy2_kernel(const GhostCopy* __restrict__ e, int64_t n, int nf,
                                                    const double* __restrict__ src, double* __restrict__ dst)
{
    const int64_t f = blockIdx.y;
    for (int64_t t = first_point(); t < n; t += next_point()) {
        const GhostCopy c = e[t];
        dst[c.dst + f * c.dfs] = src[c.src + f * c.sfs];
    }
}

hipError_t launch_copy2(const GhostCopy* e, int64_t n, int nf, const double* src, double* dst, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    copy2_kernel<<<grid_for(n, nf), BLK, 0, s>>>(e, n, nf, src, dst);
    return hipGetLastError();
}

hipError_t launch_radiative(const StageArgs& a, const PatchDev& P, const RadPt* pts, int64_t n, int nf,
                            const RadParams& rp, const double xlo[3], double h, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    radiative_kernel<<<grid_for(n, nf), BLK, 0, s>>>(a, P, pts, n, nf, rp, xlo[0], xlo[1], xlo[2], h);
    return hipGetLastError();
}

hipError_t launch_bor_band(const GhostCopy* band, int64_t n, int nf, const double w[4], const double* Un,
                           const double* k0, const double* k1, const double* k2, const double* k3, double* T,
                           hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    BorW W;
    for (int j = 0; j < 4; ++j) W.w[j] = w[j];
    bor_band_kernel<<<grid_for(n, nf), BLK, 0, s>>>(band, n, nf, W, Un, k0, k1, k2, k3, T);
    return hipGetLastError();
}

hipError_t launch_prolong(const ProlongBrick* e, int64_t n, const uint32_t* rows, int nf, int R,
                          const double* lw_host, const double* T, double* U, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    LagW L{};
    if (R < 2 || R > 4) return hipErrorInvalidValue;
    for (int m = 0; m < R; ++m)
        for (int j = 0; j < 6; ++j) L.w[m][j] = lw_host[m * 6 + j];
    // fields per workgroup: the more, the less index arithmetic, as long as
    // four workgroups per compute unit are left
    const int fpw = (int)std::clamp<int64_t>(n * nf / 1024, 1, PROLONG_FPW);
    const int64_t grid = n * ((nf + fpw - 1) / fpw);
    if (grid > INT32_MAX) return hipErrorInvalidConfiguration;
    switch (R) {
    case 2: prolong_kernel<2><<<(int)grid, BLK, 0, s>>>(e, (int)n, nf, fpw, rows, L, T, U); break;
    case 3: prolong_kernel<3><<<(int)grid, BLK, 0, s>>>(e, (int)n, nf, fpw, rows, L, T, U); break;
    default: prolong_kernel<4><<<(int)grid, BLK, 0, s>>>(e, (int)n, nf, fpw, rows, L, T, U); break;
    }
    return hipGetLastError();
}

hipError_t launch_restrict(const RestrictPt* e, int64_t n, int nf, const double* Uf, double* Uc, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    restrict_kernel<<<grid_for(n, (nf + FC - 1) / FC), BLK, 0, s>>>(e, n, nf, Uf, Uc);
    return hipGetLastError();
}

hipError_t launch_axpby(int64_t n, double a, const double* x, double b, const double* y, double* z,
                        hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    axpby_kernel<<<grid_for(n), BLK, 0, s>>>(n, a, x, b, y, z);
    return hipGetLastError();
}

}  // namespace mol
