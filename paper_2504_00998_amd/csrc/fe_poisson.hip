// Electrostatics on the same finite-element space (paper Sec. 2.2, Eq. for the
// Poisson problem, -lap(phi) / 4 pi = rho + b).
//
// The Galerkin system is K phi = 4 pi M s for the nodal charge density s
// (GLL-collocated right-hand side, M the lumped mass).  With phi = M^-1/2 x it
// reads  H0 x = 2 pi M^1/2 s,  H0 = M^-1/2 (1/2 K) M^-1/2,  which is the
// filter's operator H~ with a zero diagonal term, so the filter's step kernel
// serves as the matrix-vector product.  Dirichlet axes of the mesh give
// phi = 0 on those faces; with none (periodic / zero-Neumann only, the
// constant-field setup of Sec. 2.2.1) H0 has the null vector M^1/2 1, which is
// projected out of the right-hand side and of every search direction, so the
// solution has zero mean (integral of phi = 0).  Conjugate gradients with a
// Jacobi preconditioner (the assembled diagonal of H0); the product is the
// single-vector tensor-product kernel, which leaves the partial sums of p.Hp.
// The iteration runs on the device: its dot products are fixed-order two-pass reductions whose
// results, and the CG scalars computed from them, stay in device memory; the
// host reads the convergence state once per batch of iterations, and
// iterations queued after convergence leave the iterate untouched.
//
// The constrained-potential-difference setup (Sec. 2.2.2) prescribes phi in
// the two conductor regions, Omega_0 = {z <= z_lo} and Omega_1 = {z >= z_hi}:
// phi = -w there, plus dV in Omega_1 (w = V_loc - V_sm at the nodes), so the
// total potential phi + w is 0 and dV inside the conductors.  The same CG runs
// on the free block: the constrained entries of x start at M^1/2 g, the
// initial residual b - H0 x0 is taken on the free nodes only, and the Jacobi
// preconditioner is zero on constrained nodes, which keeps every search
// direction and the residual zero there; the constrained phi are written as
// the data themselves at the end.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "fe_internal.h"

namespace fe {

namespace {

__global__ void mass_sqrt_kernel(const double *massax, int maxf, int nfx, int nfy, int64_t n, double *out) {
    const int64_t I = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (I >= n) return;
    const int tx = (int)(I % nfx), ty = (int)((I / nfx) % nfy), tz = (int)(I / ((int64_t)nfx * nfy));
    out[I] = std::sqrt((massax[tx] * massax[maxf + ty]) * massax[2 * maxf + tz]);
}

// out_I = x_I M_I^-1/2 (per-axis factors, multiplied in the order the step
// kernels use)
__global__ void dscale_kernel(const double *axisD, int maxf, int nfx, int nfy, int64_t n, const double *x,
                              double *out) {
    const int64_t I = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (I >= n) return;
    const int tx = (int)(I % nfx), ty = (int)((I / nfx) % nfy), tz = (int)(I / ((int64_t)nfx * nfy));
    out[I] = x[I] * ((axisD[tx] * axisD[maxf + ty]) * axisD[2 * maxf + tz]);
}

__global__ void vmul_kernel(double *z, const double *a, const double *b, int64_t n) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) z[i] = a[i] * b[i];
}

__global__ void xpby_kernel(double *p, const double *z, double beta, int64_t n) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) p[i] = z[i] + beta * p[i];
}

inline unsigned blocks(int64_t n) { return (unsigned)((n + 255) / 256); }

// ---------------------------------------------------------------- device CG
// Scalars of the device iteration (doubles in the work buffer).
enum : int {
    S_RZ0 = 0,    // r.z of the current iterate (z = projected P r), even iterations
    S_RZ1,        // the same, odd iterations
    S_ALPHA,      // rz / p.Hp
    S_BNRM,       // |b|
    S_REL,        // |r| / |b| after the last update
    S_DONE,       // 1 once converged (or broken down): later products and updates do nothing
    S_IT,         // updates made
    S_TOL,
    S_BREAK,      // 1 when p.Hp <= 0 was met
    S_STOP,       // the same for the direction
    S_COUNT
};
constexpr int kRedThreads = 256, kRedWaves = kRedThreads / 64;
constexpr int kRedBlocks = 1024;  // partial sums per reduction (fixed: the summation order does not depend on timing)

// Fixed-order sums of the block's per-thread values for C components, in every
// thread: across the wavefront, then over the wavefronts through lds (one use per
// launch, or a barrier between).
template <int C> __device__ __forceinline__ void block_sum(double (&v)[C], double *lds) {
    const int wave = threadIdx.x / 64;
#pragma unroll
    for (int c = 0; c < C; ++c) {
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) v[c] += __shfl_xor(v[c], w);
        if ((threadIdx.x & 63) == 0) lds[c * kRedWaves + wave] = v[c];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C; ++c) {
        v[c] = lds[c * kRedWaves];
#pragma unroll
        for (int w = 1; w < kRedWaves; ++w) v[c] += lds[c * kRedWaves + w];
    }
}

// part[blk] = sum over the block's grid-stride elements of p_i q_i (where the
// product does not leave these sums itself)
__global__ __launch_bounds__(kRedThreads) void cg_pq_kernel(const double *p, const double *q, int64_t n,
                                                            const double *sc, double *part) {
    __shared__ double lds[kRedWaves];
    if (sc[S_DONE] != 0.0) return;
    double v[1] = {0.0};
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kRedThreads)
        v[0] += p[i] * q[i];
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

// The two passes over the vectors of an iteration are bound by the streams they
// read and write (the vectors stay in the last-level cache at a few million
// nodes).  A wavefront walks a range of z at one y and 64 x positions, so that
// e = M^1/2 1 / |M^1/2 1| and the Jacobi inverse come from the per-axis tables
// (tab: x and y factors in registers, z ones wave-uniform) instead of being two
// more streams in each pass; x is updated where p is read anyway.  1.78 M nodes,
// us per iteration: update 21.2 -> 12.7, direction 14.4 -> 17.0 with the update
// of x in it; with the product 67 -> 56 (139 before the products' partial sums
// and the scalars of the iteration came out of the same three launches).  512 or
// 2048 blocks, or 4 or 8 nodes at a time, are slower.
struct CgWalk {
    int maxf, nfx, nfy, nfz, ntx, nzr;  // 64-wide x tiles, nodes of a range of z
    int tasks;                          // wavefronts with work: ntx nfy ceil(nfz / nzr)
    double s, ie;                       // h / 4, 1 / |M^1/2 1|
    int singular, cpd;
    double z_lo, z_hi;
};

// load(u, i) for U nodes i of the range, then use(u, i, valid, Jacobi inverse, e)
// for them.  tab: 15 rows of maxf (0-2 M^-1/2, 6-8 M, 9-11 diag K, 12-14 diag M per axis).
template <int U, class Load, class Use>
__device__ __forceinline__ void cg_walk(const CgWalk &t, const double *__restrict__ tab, const double *__restrict__ zcoord,
                                        Load load, Use use) {
    int task = __builtin_amdgcn_readfirstlane((int)blockIdx.x * kRedWaves + (int)threadIdx.x / 64);
    for (; task < t.tasks; task += (int)gridDim.x * kRedWaves) {
        const int ty = task / t.ntx % t.nfy, z0 = task / t.ntx / t.nfy * t.nzr, z1 = min(z0 + t.nzr, t.nfz);
        const int x = task % t.ntx * 64 + (int)(threadIdx.x & 63), tx = min(x, t.nfx - 1), F = t.maxf;
        const double my = tab[7 * F + ty], ky = tab[10 * F + ty], dy = tab[13 * F + ty];
        const double mx = tab[6 * F + tx], kx = tab[9 * F + tx], dx = tab[12 * F + tx];
        const double mxy = mx * my, a = t.s * (kx * dy + dx * ky), b = t.s * (dx * dy);
        const double exy = t.singular ? (mx * tab[tx]) * (my * tab[F + ty]) * t.ie : 0.0;
        const int64_t plane = (int64_t)t.nfx * t.nfy, i0 = (int64_t)ty * t.nfx + tx;
        for (int z = z0; z < z1; z += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) load(u, i0 + plane * min(z + u, z1 - 1));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int tz = min(z + u, z1 - 1);
                const double mz = tab[8 * F + tz], kz = tab[11 * F + tz], dz = tab[14 * F + tz], zc = zcoord[tz];
                const bool fixed = t.cpd && (zc <= t.z_lo || zc >= t.z_hi);
                const double pinv = fixed ? 0.0 : mxy * mz / __builtin_fma(a, dz, b * kz);
                use(u, i0 + plane * tz, x < t.nfx && z + u < z1, pinv, exy * (mz * tab[2 * F + tz]));
            }
        }
    }
}

// alpha = rz / p.q from the product's npq partial sums (each block adds them up,
// in the same order); r -= alpha q, and the partial sums r.r, r.z, e.z, r.e with
// z = pinv r (before the null-space projection).  p.q <= 0 stops the iteration.
__global__ __launch_bounds__(kRedThreads) void cg_update_kernel(double *__restrict__ r, const double *__restrict__ q,
                                                                CgWalk t, const double *__restrict__ tab,
                                                                const double *__restrict__ zcoord, double *sc, int rzi,
                                                                const double *pq, int npq, double *part) {
    __shared__ double lds[4 * kRedWaves], lds1[kRedWaves];
    if (sc[S_DONE] != 0.0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) sc[S_STOP] = 1.0;
        return;
    }
    double a[1] = {0.0};
    for (int b = threadIdx.x; b < npq; b += kRedThreads) a[0] += pq[b];
    block_sum<1>(a, lds1);
    if (!(a[0] > 0.0)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) sc[S_BREAK] = sc[S_STOP] = 1.0;
        return;
    }
    const double al = sc[rzi] / a[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) sc[S_ALPHA] = al;
    double v[4] = {0.0, 0.0, 0.0, 0.0}, rr[2], qq[2];
    cg_walk<2>(
        t, tab, zcoord,
        [&](int u, int64_t i) {
            rr[u] = r[i];
            qq[u] = q[i];
        },
        [&](int u, int64_t i, bool valid, double pinv, double e) {
            // a zero preconditioner entry marks a constrained node: no equation there
            const double ri = valid && pinv != 0.0 ? rr[u] - al * qq[u] : 0.0;
            if (valid) r[i] = ri;
            const double zi = pinv * ri;
            v[0] += ri * ri;
            v[1] += ri * zi;
            v[2] += e * zi;
            v[3] += ri * e;
        });
    block_sum<4>(v, lds);
    if (threadIdx.x == 0)
        for (int c = 0; c < 4; ++c) part[c * kRedBlocks + blockIdx.x] = v[c];
}

// x += alpha p; |r| / |b|, convergence, and with the projected z
// (z' = z - (e.z) e, r.z' = r.z - (e.z)(r.e)) beta and p = z' + beta p.
// Each of the two flags is read by one kind of launch and set by the other (S_DONE
// here, S_STOP by the update), so all threads of a launch see the same value.
__global__ __launch_bounds__(kRedThreads) void cg_direction_kernel(double *__restrict__ x, double *__restrict__ p,
                                                                   const double *__restrict__ r, CgWalk t,
                                                                   const double *__restrict__ tab,
                                                                   const double *__restrict__ zcoord,
                                                                   const double *part, int nb, double *sc, int rzi) {
    __shared__ double lds[4 * kRedWaves];
    if (sc[S_STOP] != 0.0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) sc[S_DONE] = 1.0;
        return;
    }
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nb; b += kRedThreads)
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] += part[c * kRedBlocks + b];
    block_sum<4>(v, lds);
    const double al = sc[S_ALPHA], rel = sqrt(v[0]) / sc[S_BNRM];
    const double ez = v[2], rz = v[1] - ez * v[3], beta = rz / sc[rzi];
    const bool done = rel <= sc[S_TOL];
    double pp[2], xx[2], rr[2];
    cg_walk<2>(
        t, tab, zcoord,
        [&](int u, int64_t i) {
            pp[u] = p[i];
            xx[u] = x[i];
            rr[u] = r[i];
        },
        [&](int u, int64_t i, bool valid, double pinv, double e) {
            if (valid) x[i] = xx[u] + al * pp[u];
            if (valid && !done) p[i] = (pinv * rr[u] - ez * e) + beta * pp[u];
        });
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc[S_IT] += 1.0;
        sc[S_REL] = rel;
        sc[S_RZ0 + S_RZ1 - rzi] = rz;  // the other slot: this one is still being read
        if (done) sc[S_DONE] = 1.0;
    }
}

// 1 / diag(H0) = M / diag(1/2 K): the assembled diagonal of the stiffness is the
// sum of three products of one-dimensional ones (kd, md: the assembled
// diagonals of each axis' stiffness and mass; s = h / 4), M the lumped mass; zero
// on the nodes of a conductor region.
__global__ void jacobi_inverse_kernel(double *pinv, const double *massax, const double *kd, const double *md, int maxf,
                                      double s, int nfx, int nfy, int64_t n, const double *zcoord, int cpd, double z_lo,
                                      double z_hi) {
    const int64_t I = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (I >= n) return;
    const int tx = (int)(I % nfx), ty = (int)((I / nfx) % nfy), tz = (int)(I / ((int64_t)nfx * nfy));
    const double M = massax[tx] * massax[maxf + ty] * massax[2 * maxf + tz];
    const double kx = kd[tx], ky = kd[maxf + ty], kz = kd[2 * maxf + tz];
    const double mx = md[tx], my = md[maxf + ty], mz = md[2 * maxf + tz];
    const bool fixed = cpd && (zcoord[tz] <= z_lo || zcoord[tz] >= z_hi);
    pinv[I] = fixed ? 0.0 : M / (s * (kx * my * mz + mx * ky * mz + mx * my * kz));
}

// Region of a node for the constrained setup: 0 free, 1 Omega_0, 2 Omega_1.
__device__ __forceinline__ int cpd_region(double z, double z_lo, double z_hi) {
    return z <= z_lo ? 1 : (z >= z_hi ? 2 : 0);
}

// x = M^1/2 g on constrained nodes (g = -w, plus dV in Omega_1), 0 elsewhere
__global__ void cpd_start_kernel(double *x, const double *msqrt, const double *w, const double *zcoord, int nfx,
                                 int nfy, int64_t n, double z_lo, double z_hi, double dV) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int reg = cpd_region(zcoord[i / ((int64_t)nfx * nfy)], z_lo, z_hi);
    const double g = (reg == 2 ? dV : 0.0) - (w ? w[i] : 0.0);
    x[i] = reg ? msqrt[i] * g : 0.0;
}

// r = b - q on free nodes, 0 on constrained ones
__global__ void cpd_residual_kernel(double *r, const double *q, const double *pinv, int64_t n) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    r[i] = pinv[i] != 0.0 ? r[i] - q[i] : 0.0;
}

// phi = g on constrained nodes (the data, exactly)
__global__ void cpd_fix_kernel(double *phi, const double *w, const double *zcoord, int nfx, int nfy, int64_t n,
                               double z_lo, double z_hi, double dV) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int reg = cpd_region(zcoord[i / ((int64_t)nfx * nfy)], z_lo, z_hi);
    if (reg) phi[i] = (reg == 2 ? dV : 0.0) - (w ? w[i] : 0.0);
}

#define FE_HIPP(call, what)                                                                          \
    do {                                                                                             \
        hipError_t _e = (call);                                                                      \
        if (_e != hipSuccess) return fail(FE_EDEVICE, std::string(what) + ": " + hipGetErrorString(_e)); \
    } while (0)
#define FE_BLASP(call, what)                                                                         \
    do {                                                                                             \
        rocblas_status _b = (call);                                                                  \
        if (_b != rocblas_status_success)                                                            \
            return fail(FE_EDEVICE, std::string(what) + ": " + rocblas_status_to_string(_b));         \
    } while (0)

}  // namespace

hipError_t launch_mass_sqrt(const fe_mesh *m, double *out, hipStream_t s) {
    hipLaunchKernelGGL(mass_sqrt_kernel, dim3(blocks(m->n)), dim3(256), 0, s, m->d_axis + 6 * m->maxf, m->maxf,
                       (int)m->nf[0], (int)m->nf[1], m->n, out);
    return hipGetLastError();
}

hipError_t launch_vmul(double *z, const double *a, const double *b, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(vmul_kernel, dim3(blocks(n)), dim3(256), 0, s, z, a, b, n);
    return hipGetLastError();
}

hipError_t launch_xpby(double *p, const double *z, double beta, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(xpby_kernel, dim3(blocks(n)), dim3(256), 0, s, p, z, beta, n);
    return hipGetLastError();
}

}  // namespace fe

using namespace fe;

extern "C" size_t fe_poisson_work_bytes(const fe_mesh *m) {
    if (!m) return 0;
    return ((size_t)8 * (size_t)m->n + 4 * (size_t)kRedBlocks + 16) * sizeof(double);
}

namespace fe {

// The conductor regions of the constrained setup (null: the mesh's own
// boundary conditions only).
struct CpdSpec {
    const double *w;
    double z_lo, z_hi, dV;
};

fe_status poisson_solve(fe_mesh *m, const double *charge, double *phi, double tol, int32_t maxit, double *work,
                        size_t work_bytes, int32_t *iters_host, double *relres_host, hipStream_t st,
                        const CpdSpec *cpd) {
    if (!m || !charge || !phi || !work) return fail(FE_EINVAL, "NULL argument");
    if (!(tol > 0.0) || !std::isfinite(tol)) return fail(FE_EINVAL, "tol must be positive");
    if (maxit < 1) return fail(FE_EINVAL, "maxit must be >= 1");
    if (work_bytes < fe_poisson_work_bytes(m))
        return fail(FE_ENOMEM, "work smaller than fe_poisson_work_bytes");
    FE_HIPP(hipSetDevice(m->device), "hipSetDevice");
    const int64_t n = m->n;
    const int ni = (int)n;
    double *x = work, *r = x + n, *z = r + n, *p = z + n, *q = p + n, *e = q + n, *pinv = e + n, *zero = pinv + n;
    const bool singular =
        !cpd && m->bc[0] != FE_BC_DIRICHLET && m->bc[1] != FE_BC_DIRICHLET && m->bc[2] != FE_BC_DIRICHLET;

    void *hv = nullptr;
    fe_status stt = blas_handle(m, st, &hv);
    if (stt != FE_OK) return stt;
    rocblas_handle h = static_cast<rocblas_handle>(hv);

    if (cpd) {
        // no equation on constrained nodes: a zero preconditioner entry marks them
        int64_t nc = 0;
        for (int64_t tz = 0; tz < m->nf[2]; ++tz) {
            const double zz = m->axis_coord[2][(size_t)tz];
            if (zz <= cpd->z_lo || zz >= cpd->z_hi) nc += m->nf[0] * m->nf[1];
        }
        if (nc == 0) return fail(FE_EINVAL, "no node lies in a conductor region (z <= z_lo or z >= z_hi)");
        if (nc == n) return fail(FE_EINVAL, "every node lies in a conductor region: nothing to solve");
    }
    hipLaunchKernelGGL(jacobi_inverse_kernel, dim3(blocks(n)), dim3(256), 0, st, pinv, m->d_axis + 6 * m->maxf,
                       m->d_axis + 9 * m->maxf, m->d_axis + 12 * m->maxf, m->maxf, 0.25 * m->h, (int)m->nf[0],
                       (int)m->nf[1], n, m->d_zcoord, cpd ? 1 : 0, cpd ? cpd->z_lo : 0.0, cpd ? cpd->z_hi : 0.0);
    FE_HIPP(hipGetLastError(), "jacobi inverse");
    FE_HIPP(launch_fill(zero, n, 0.0, st), "fill");
    // e = M^1/2 1 / |M^1/2 1| (the null vector when no axis is Dirichlet)
    FE_HIPP(launch_mass_sqrt(m, e, st), "mass sqrt");
    if (cpd) {
        hipLaunchKernelGGL(cpd_start_kernel, dim3(blocks(n)), dim3(256), 0, st, x, e, cpd->w, m->d_zcoord,
                           (int)m->nf[0], (int)m->nf[1], n, cpd->z_lo, cpd->z_hi, cpd->dV);
        FE_HIPP(hipGetLastError(), "cpd start");
    } else {
        FE_HIPP(launch_fill(x, n, 0.0, st), "fill");
    }
    // r = b = 2 pi M^1/2 s
    FE_HIPP(launch_vmul(r, e, charge, n, st), "rhs");
    const double twopi = 2.0 * M_PI;
    FE_BLASP(rocblas_dscal(h, ni, &twopi, r, 1), "dscal");
    if (cpd) {
        // r = b - H0 x0 on the free nodes (the prescribed values moved to the right-hand side)
        StepArgs a{x, 1, q, 1, nullptr, 0, 1.0, 0.0, 0.0, 1, zero};
        FE_HIPP(tensor_vec_applies(m, a) ? launch_tensor_vec(m, a, st) : launch_step(m, a, FE_F64, st), "product");
        hipLaunchKernelGGL(cpd_residual_kernel, dim3(blocks(n)), dim3(256), 0, st, r, q, pinv, n);
        FE_HIPP(hipGetLastError(), "cpd residual");
    }
    double enrm = 0.0;
    FE_BLASP(rocblas_dnrm2(h, ni, e, 1, &enrm), "dnrm2");
    const double ie = 1.0 / enrm;
    FE_BLASP(rocblas_dscal(h, ni, &ie, e, 1), "dscal");
    auto project = [&](double *v) -> fe_status {
        if (!singular) return FE_OK;
        double c = 0.0;
        FE_BLASP(rocblas_ddot(h, ni, e, 1, v, 1, &c), "ddot");
        c = -c;
        FE_BLASP(rocblas_daxpy(h, ni, &c, e, 1, v, 1), "daxpy");
        return FE_OK;
    };
    if ((stt = project(r)) != FE_OK) return stt;
    double bnrm = 0.0;
    FE_BLASP(rocblas_dnrm2(h, ni, r, 1, &bnrm), "dnrm2");
    int it = 0;
    double rel = 0.0;
    if (bnrm > 0.0) {
        FE_HIPP(launch_vmul(z, pinv, r, n, st), "precondition");
        if ((stt = project(z)) != FE_OK) return stt;
        FE_HIPP(hipMemcpyAsync(p, z, n * sizeof(double), hipMemcpyDeviceToDevice, st), "copy");
        double rz = 0.0;
        FE_BLASP(rocblas_ddot(h, ni, r, 1, z, 1, &rz), "ddot");
        // the iteration itself on the device; the host looks at its state
        // once per batch
        double *part = zero + n, *sc = part + 4 * kRedBlocks;
        const double sc0[S_COUNT] = {rz, 0.0, 0.0, bnrm, 1.0, 0.0, 0.0, tol, 0.0, 0.0};
        FE_HIPP(hipMemcpyAsync(sc, sc0, sizeof(sc0), hipMemcpyHostToDevice, st), "copy scalars");
        const int nb = (int)std::min<int64_t>(kRedBlocks, (n + kRedThreads - 1) / kRedThreads);
        CgWalk t{m->maxf, (int)m->nf[0], (int)m->nf[1], (int)m->nf[2], (int)((m->nf[0] + 63) / 64), 0, 0, 0.25 * m->h, ie,
                 singular ? 1 : 0, cpd ? 1 : 0, cpd ? cpd->z_lo : 0.0, cpd ? cpd->z_hi : 0.0};
        const int64_t cols = (int64_t)t.ntx * t.nfy;
        t.nzr = (int)std::min<int64_t>(t.nfz, (cols * t.nfz + kRedBlocks * kRedWaves - 1) / (kRedBlocks * kRedWaves));
        while (cols * ((t.nfz + t.nzr - 1) / t.nzr) > kRedBlocks * kRedWaves && t.nzr < t.nfz) ++t.nzr;
        t.tasks = (int)(cols * ((t.nfz + t.nzr - 1) / t.nzr));
        const int nr = std::min(kRedBlocks, (t.tasks + kRedWaves - 1) / kRedWaves);
        constexpr int kBatch = 8;
        // iteration j of a batch: three launches on fixed buffers, where the
        // product leaves the partial sums of p.q (in z, free by now)
        auto iteration = [&](hipStream_t ss, int j) -> hipError_t {
            const int rzi = j % 2 ? S_RZ1 : S_RZ0;
            StepArgs a{p, 1, q, 1, nullptr, 0, 1.0, 0.0, 0.0, 1, zero};
            int nq = 0;
            const int most = (int)std::min<int64_t>(n, kRedBlocks);
            hipError_t e2 = tensor_vec_applies(m, a) ? launch_tensor_vec(m, a, ss, sc + S_DONE, z, most, &nq) : hipSuccess;
            if (e2 != hipSuccess) return e2;
            if (nq == 0) {
                // planes out of the kernel's range, or more tiles than partial sums
                if ((e2 = launch_step(m, a, FE_F64, ss)) != hipSuccess) return e2;
                nq = nb;
                hipLaunchKernelGGL(cg_pq_kernel, dim3(nb), dim3(kRedThreads), 0, ss, p, q, n, sc, z);
            }
            hipLaunchKernelGGL(cg_update_kernel, dim3(nr), dim3(kRedThreads), 0, ss, r, q, t, m->d_axis,
                               m->d_zcoord, sc, rzi, z, nq, part);
            hipLaunchKernelGGL(cg_direction_kernel, dim3(nr), dim3(kRedThreads), 0, ss, x, p, r, t, m->d_axis,
                               m->d_zcoord, part, nr, sc, rzi);
            return hipGetLastError();
        };
        // After the first batch (direct launches, which also set the kernels'
        // launch attributes) a full batch is captured once, on a private
        // stream so that the caller's stream may be the null stream, into a
        // HIP graph of kernel nodes only, and replayed on the caller's stream:
        // the same launches in the same order, without the per-launch host
        // overhead of 24 short kernels.  If the capture or instantiation
        // fails the batches stay direct launches.
        hipGraphExec_t exec = nullptr;
        bool graph_tried = false;
        auto capture = [&]() {
            graph_tried = true;
            hipStream_t cs = nullptr;
            if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) return;
            hipGraph_t graph = nullptr;
            bool ok = hipStreamBeginCapture(cs, hipStreamCaptureModeRelaxed) == hipSuccess;
            if (ok) {
                for (int j = 0; j < kBatch && ok; ++j) ok = iteration(cs, j) == hipSuccess;
                ok = (hipStreamEndCapture(cs, &graph) == hipSuccess) && ok && graph;
            }
            if (ok && hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) exec = nullptr;
            if (graph) (void)hipGraphDestroy(graph);
            (void)hipStreamDestroy(cs);
            (void)hipGetLastError();  // a failed capture leaves no error behind
        };
        double sh[S_COUNT] = {};
        int queued = 0;
        fe_status loop_st = FE_OK;
        while (queued < maxit) {
            const int nbatch = std::min(kBatch, maxit - queued);
            if (queued > 0 && nbatch == kBatch && !graph_tried) capture();
            if (exec && nbatch == kBatch) {
                if (hipGraphLaunch(exec, st) != hipSuccess) { loop_st = fail(FE_EDEVICE, "CG graph launch"); break; }
            } else {
                for (int j = 0; j < nbatch; ++j)
                    if (iteration(st, j) != hipSuccess) { loop_st = fail(FE_EDEVICE, "CG kernel launch"); break; }
                if (loop_st != FE_OK) break;
            }
            queued += nbatch;
            if (hipMemcpyAsync(sh, sc, sizeof(sh), hipMemcpyDeviceToHost, st) != hipSuccess ||
                hipStreamSynchronize(st) != hipSuccess) {
                loop_st = fail(FE_EDEVICE, "read CG state");
                break;
            }
            if (sh[S_DONE] != 0.0) break;
        }
        if (exec) (void)hipGraphExecDestroy(exec);
        if (loop_st != FE_OK) return loop_st;
        if (sh[S_BREAK] != 0.0) return fail(FE_EDEVICE, "CG breakdown: p^T H0 p <= 0");
        it = (int)sh[S_IT];
        rel = sh[S_REL];
        if ((stt = project(x)) != FE_OK) return stt;
    }
    // phi = M^-1/2 x
    hipLaunchKernelGGL(dscale_kernel, dim3(blocks(n)), dim3(256), 0, st, m->d_axis, m->maxf, (int)m->nf[0],
                       (int)m->nf[1], n, x, phi);
    FE_HIPP(hipGetLastError(), "scale");
    if (cpd) {
        hipLaunchKernelGGL(cpd_fix_kernel, dim3(blocks(n)), dim3(256), 0, st, phi, cpd->w, m->d_zcoord,
                           (int)m->nf[0], (int)m->nf[1], n, cpd->z_lo, cpd->z_hi, cpd->dV);
        FE_HIPP(hipGetLastError(), "cpd data");
    }
    if (iters_host) *iters_host = it;
    if (relres_host) *relres_host = rel;
    return FE_OK;
}

}  // namespace fe

extern "C" {

fe_status fe_poisson_solve(fe_mesh *m, const double *charge, double *phi, double tol, int32_t maxit,
                           double *work, size_t work_bytes, int32_t *iters_host, double *relres_host,
                           hipStream_t st) {
    return fe::poisson_solve(m, charge, phi, tol, maxit, work, work_bytes, iters_host, relres_host, st, nullptr);
}

fe_status fe_poisson_solve_cpd(fe_mesh *m, const double *charge, const double *w, double z_lo, double z_hi,
                               double dV, double *phi, double tol, int32_t maxit, double *work, size_t work_bytes,
                               int32_t *iters_host, double *relres_host, hipStream_t st) {
    if (!m) return fail(FE_EINVAL, "NULL argument");
    if (!std::isfinite(z_lo) || !std::isfinite(z_hi) || !std::isfinite(dV) || !(z_lo < z_hi))
        return fail(FE_EINVAL, "z_lo < z_hi and dV must be finite");
    if (m->bc[2] == FE_BC_PERIODIC) return fail(FE_EINVAL, "the z axis of a CPD mesh cannot be periodic");
    if (phi && ((charge && fe::overlap(phi, m->n, 1, 1, charge, m->n, 1, 1)) ||
                (w && fe::overlap(phi, m->n, 1, 1, w, m->n, 1, 1))))
        return fail(FE_EINVAL, "phi overlaps charge or w");
    const fe::CpdSpec cpd{w, z_lo, z_hi, dV};
    return fe::poisson_solve(m, charge, phi, tol, maxit, work, work_bytes, iters_host, relres_host, st, &cpd);
}

}  // extern "C"
