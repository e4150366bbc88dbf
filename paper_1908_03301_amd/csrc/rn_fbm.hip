// rn_fbm.hip -- correlated conductance fields on the GPU (Sec. II, Eqs. 1-2):
// fractional Brownian motion by Fourier filtering of caller-drawn white noise,
// and the bond conductances built from the node field, with optional bond
// dilution by caller-drawn uniforms. This replaces, on one GPU, the paper's
// distributed generator; the flow solve does not depend on it.
//
// Transforms are hipFFT's double-precision real-to-complex and back; the
// spectral filter, which also standardises, and the bonds are kernels here.
#include "rn_runtime.hpp"

#include <hipfft/hipfft.h>

#include <cmath>
#include <cstring>

namespace rn {
namespace {

// Amplitude of the spectral filter on the half spectrum of a real nz x ny x nx
// grid (x fastest, nxh = nx/2 + 1 modes along x): (sum_k beta_k f_k^2)^expo /
// N, with f the mode's frequency in cycles per node, N the inverse transform's
// norm, and 0 at k = 0. It is the same for +-f along y and z, so one power
// serves up to four modes: computed for each, the powers took twice as long as
// the filter's bytes.
struct FbmGrid {
    int nx, ny, nz, nxh, nyh, nzh;        // nyh = ny/2 + 1 and nzh = nz/2 + 1 frequencies up to sign
    double b[3], expo, inv_n;
};

__device__ __forceinline__ double fbm_amplitude(const FbmGrid &F, int jx, int jy, int jz)
{
    const double fx = (double)jx / F.nx, fy = (double)jy / F.ny, fz = (double)jz / F.nz;
    const double k2 = F.b[0] * fx * fx + F.b[1] * fy * fy + F.b[2] * fz * fz;
    return k2 > 0.0 ? pow(k2, F.expo) * F.inv_n : 0.0;
}

// The rows of one (|f_y|, |f_z|): visit(row offset) for each of the one, two
// or four sign pairs.
template <typename V>
__device__ __forceinline__ void fbm_rows(const FbmGrid &F, int jy, int jz, V &&visit)
{
    const bool my = jy > 0 && 2 * jy != F.ny, mz = jz > 0 && 2 * jz != F.nz;
    for (int s = 0; s < 4; ++s) {
        if (((s & 1) && !my) || ((s & 2) && !mz)) continue;
        const int y = (s & 1) ? F.ny - jy : jy, z = (s & 2) ? F.nz - jz : jz;
        visit(((int64_t)z * F.ny + y) * F.nxh);
    }
}

constexpr int kRedThreads = 256, kRedBlocks = 1024;

__device__ __forceinline__ double fbm_block_sum(double acc)
{
    __shared__ double sh[kRedThreads];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kRedThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    return sh[0];
}

// Variance of the filtered field from its spectrum (Parseval; its mean is 0):
// block sums in a fixed order, then one block adds them and stores 1 / sd (0
// for a field of zeros). The field is then standardised by the filter itself,
// in place of two sums over it, a read-back of its mean and a pass that
// divides (0.25 of 1.09 ms at 256^3).
__global__ void fbm_power_kernel(const hipfftDoubleComplex *spec, FbmGrid F, double *partial)
{
    double acc = 0.0;
    const int64_t total = (int64_t)F.nzh * F.nyh * F.nxh;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const unsigned u = (unsigned)i, t = u / (unsigned)F.nxh;
        const int jx = (int)(u - t * (unsigned)F.nxh), jz = (int)(t / (unsigned)F.nyh), jy = (int)(t - (unsigned)jz * (unsigned)F.nyh);
        const double a = fbm_amplitude(F, jx, jy, jz);
        double p = 0.0;
        fbm_rows(F, jy, jz, [&](int64_t row) {
            const hipfftDoubleComplex v = spec[row + jx];
            p += (a * v.x) * (a * v.x) + (a * v.y) * (a * v.y);
        });
        acc += jx > 0 && 2 * jx != F.nx ? 2.0 * p : p;      // the conjugate half
    }
    acc = fbm_block_sum(acc);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

__global__ void fbm_scale_kernel(const double *partial, double *scale)
{
    double acc = 0.0;
    for (int b = threadIdx.x; b < kRedBlocks; b += kRedThreads) acc += partial[b];
    acc = fbm_block_sum(acc);
    if (threadIdx.x == 0) *scale = acc > 0.0 ? 1.0 / sqrt(acc) : 0.0;
}

__global__ void fbm_filter_kernel(hipfftDoubleComplex *spec, FbmGrid F, const double *scale)
{
    const double sc = *scale;
    const int64_t total = (int64_t)F.nzh * F.nyh * F.nxh;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const unsigned u = (unsigned)i, t = u / (unsigned)F.nxh;
        const int jx = (int)(u - t * (unsigned)F.nxh), jz = (int)(t / (unsigned)F.nyh), jy = (int)(t - (unsigned)jz * (unsigned)F.nyh);
        const double a = fbm_amplitude(F, jx, jy, jz) * sc;
        fbm_rows(F, jy, jz, [&](int64_t row) {
            hipfftDoubleComplex v = spec[row + jx];
            v.x = sc != 0.0 ? v.x * a : 0.0;                // zeros also where the noise is not finite
            v.y = sc != 0.0 ? v.y * a : 0.0;
            spec[row + jx] = v;
        });
    }
}

// g_k[i] = exp(sigma (phi_i + phi_{i+e_k}) / 2) on the periodic grid; 0 on the
// last plane along k unless periodic; 0 where u_k[i] >= occupancy (u_k given)
__global__ void fbm_bonds_kernel(const double *phi, int nx, int ny, int nz, int dim, double sigma, int periodic,
                                 const double *u0, const double *u1, const double *u2, double occ, double *g0,
                                 double *g1, double *g2)
{
    // n < 2^31: 32-bit index arithmetic (64-bit divisions took longer than the
    // exponentials); a node's loads go out together
    const unsigned n = (unsigned)((int64_t)nx * ny * nz);
    const int st[3] = {1, nx, nx * ny};
    const int ext[3] = {nx, ny, nz};
    const double *u[3] = {u0, u1, u2};
    double *g[3] = {g0, g1, g2};
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const unsigned row = i / (unsigned)nx, z = row / (unsigned)ny;
        const int c[3] = {(int)(i - row * (unsigned)nx), (int)(row - z * (unsigned)ny), (int)z};
        const double here = phi[i];
        double there[3], draw[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (k >= dim) break;
            const int j = c[k] == ext[k] - 1 ? (int)i - (ext[k] - 1) * st[k] : (int)i + st[k];
            there[k] = phi[j];
            draw[k] = u[k] ? u[k][i] : -1.0;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (k >= dim) break;
            double v = exp(sigma * 0.5 * (here + there[k]));
            if (c[k] == ext[k] - 1 && !periodic) v = 0.0;
            if (u[k] && !(draw[k] < occ)) v = 0.0;
            g[k][i] = v;
        }
    }
}

int grid_of(int64_t n)
{
    const int64_t b = (n + 255) / 256;
    return (int)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

bool shape_ok(int dim, int64_t nx, int64_t ny, int64_t nz)
{
    if (dim != 2 && dim != 3) return false;
    if (nx < 1 || ny < 1 || nz < 1 || (dim == 2 && nz != 1)) return false;
    if (nx > INT32_MAX || ny > INT32_MAX || nz > INT32_MAX) return false;
    return (double)nx * (double)ny * (double)nz < 2147483647.0;
}

// The forward and inverse plans of the last grid, kept on the context: plan
// creation costs milliseconds, more than the transforms of a 2048^2 grid.
struct FbmPlans {
    int dim = 0, nx = 0, ny = 0, nz = 0;
    hipfftHandle fwd = 0, inv = 0;
    ~FbmPlans()
    {
        if (fwd) (void)hipfftDestroy(fwd);
        if (inv) (void)hipfftDestroy(inv);
    }
};

struct Scratch {
    rn_ctx *ctx;
    char *base = nullptr;
    explicit Scratch(rn_ctx *c) : ctx(c) {}
    ~Scratch()
    {
        if (base) {
            (void)hipStreamSynchronize(ctx->stream);
            ctx->pool.free(base);
        }
    }
};

}  // namespace

void fbm_release(rn_ctx *ctx)
{
    delete static_cast<FbmPlans *>(ctx->fbm_plans);
    ctx->fbm_plans = nullptr;
}

}  // namespace rn

using namespace rn;

#define FBM_TRY(expr)                                                                 \
    do {                                                                              \
        hipError_t e_ = (expr);                                                       \
        if (e_ != hipSuccess) {                                                       \
            ctx->err = std::string(#expr) + ": " + hipGetErrorString(e_);            \
            return RN_EDEVICE;                                                        \
        }                                                                             \
    } while (0)

#define FFT_TRY(expr)                                                                 \
    do {                                                                              \
        hipfftResult r_ = (expr);                                                     \
        if (r_ != HIPFFT_SUCCESS) {                                                   \
            ctx->err = std::string(#expr) + ": hipfft status " + std::to_string((int)r_); \
            return RN_EDEVICE;                                                        \
        }                                                                             \
    } while (0)

extern "C" int rn_fbm_field(rn_ctx *ctx, int32_t dim, int64_t nx, int64_t ny, int64_t nz, double H,
                            const double *beta, const double *noise, double *field_out, int32_t mem)
{
    if (!ctx || !noise || !field_out || !shape_ok(dim, nx, ny, nz) || !std::isfinite(H)) return RN_EINVAL;
    if (mem != RN_MEM_HOST && mem != RN_MEM_DEVICE) return RN_EINVAL;
    double b[3] = {1.0, 1.0, 1.0};
    for (int k = 0; beta && k < dim; ++k) {
        if (!(beta[k] > 0.0) || !std::isfinite(beta[k])) return RN_EINVAL;
        b[k] = beta[k];
    }
    std::lock_guard<std::mutex> lk(ctx->call_mu);
    if (ctx->server) return RN_EINVAL;        // the server owns the stream once started
    FBM_TRY(hipSetDevice(ctx->device));
    const int64_t n = nx * ny * nz;
    const int64_t nspec = nz * ny * (nx / 2 + 1);
    auto a256 = [](size_t v) { return (v + 255) & ~(size_t)255; };
    // device callers: the field's own buffer takes the copy of the noise that
    // the transforms work on, if it is aligned for their 16-byte accesses and
    // shares no memory with the noise
    const uintptr_t fa = reinterpret_cast<uintptr_t>(field_out), na = reinterpret_cast<uintptr_t>(noise);
    const bool direct = mem == RN_MEM_DEVICE && (fa & 15) == 0 && (fa + 8 * n <= na || na + 8 * n <= fa);
    const size_t off_x = 0, off_s = direct ? 0 : a256(8 * n), off_p = off_s + a256(16 * nspec),
                 off_sum = off_p + a256(8 * kRedBlocks), total = off_sum + 256;
    Scratch sc(ctx);
    hipError_t he;
    sc.base = (char *)ctx->pool.alloc(total, &he);
    if (!sc.base) return RN_ENOMEM;
    double *x = direct ? field_out : (double *)(sc.base + off_x);
    hipfftDoubleComplex *spec = (hipfftDoubleComplex *)(sc.base + off_s);
    double *partial = (double *)(sc.base + off_p), *sums = (double *)(sc.base + off_sum);
    const hipStream_t st = ctx->stream;
    FBM_TRY(hipMemcpyAsync(x, noise, 8 * n, mem == RN_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice, st));
    FbmPlans *pl = static_cast<FbmPlans *>(ctx->fbm_plans);
    if (!pl || pl->dim != dim || pl->nx != nx || pl->ny != ny || pl->nz != nz) {
        fbm_release(ctx);
        pl = new FbmPlans();
        ctx->fbm_plans = pl;
        // hipFFT's first extent is the slowest: (ny, nx) and (nz, ny, nx)
        if (dim == 2) {
            FFT_TRY(hipfftPlan2d(&pl->fwd, (int)ny, (int)nx, HIPFFT_D2Z));
            FFT_TRY(hipfftPlan2d(&pl->inv, (int)ny, (int)nx, HIPFFT_Z2D));
        } else {
            FFT_TRY(hipfftPlan3d(&pl->fwd, (int)nz, (int)ny, (int)nx, HIPFFT_D2Z));
            FFT_TRY(hipfftPlan3d(&pl->inv, (int)nz, (int)ny, (int)nx, HIPFFT_Z2D));
        }
        pl->dim = dim;
        pl->nx = (int)nx;
        pl->ny = (int)ny;
        pl->nz = (int)nz;
    }
    const hipfftHandle fwd = pl->fwd, inv = pl->inv;
    FFT_TRY(hipfftSetStream(fwd, st));
    FFT_TRY(hipfftSetStream(inv, st));
    FFT_TRY(hipfftExecD2Z(fwd, x, spec));
    FbmGrid F;
    F.nx = (int)nx;
    F.ny = (int)ny;
    F.nz = (int)nz;
    F.nxh = F.nx / 2 + 1;
    F.nyh = F.ny / 2 + 1;
    F.nzh = F.nz / 2 + 1;
    for (int k = 0; k < 3; ++k) F.b[k] = k < dim ? b[k] : 0.0;
    F.expo = -(H + 0.5 * dim) / 2.0;
    F.inv_n = 1.0 / (double)n;
    fbm_power_kernel<<<kRedBlocks, kRedThreads, 0, st>>>(spec, F, partial);
    fbm_scale_kernel<<<1, kRedThreads, 0, st>>>(partial, sums);
    fbm_filter_kernel<<<grid_of((int64_t)F.nzh * F.nyh * F.nxh), 256, 0, st>>>(spec, F, sums);
    FBM_TRY(hipGetLastError());
    FFT_TRY(hipfftExecZ2D(inv, spec, x));
    if (!direct)
        FBM_TRY(hipMemcpyAsync(field_out, x, 8 * n,
                               mem == RN_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice, st));
    FBM_TRY(hipStreamSynchronize(st));
    return RN_OK;
}

extern "C" int rn_fbm_bonds(rn_ctx *ctx, int32_t dim, int64_t nx, int64_t ny, int64_t nz, const double *field,
                            double sigma, int32_t periodic, const double *const u[3], double occupancy,
                            double *const g_out[3], int32_t mem)
{
    if (!ctx || !field || !g_out || !shape_ok(dim, nx, ny, nz) || !std::isfinite(sigma)) return RN_EINVAL;
    if (mem != RN_MEM_HOST && mem != RN_MEM_DEVICE) return RN_EINVAL;
    if (periodic != 0 && periodic != 1) return RN_EINVAL;
    for (int k = 0; k < dim; ++k)
        if (!g_out[k]) return RN_EINVAL;
    const bool dilute = u && u[0];
    if (dilute) {
        for (int k = 0; k < dim; ++k)
            if (!u[k]) return RN_EINVAL;
        if (!std::isfinite(occupancy)) return RN_EINVAL;
    }
    std::lock_guard<std::mutex> lk(ctx->call_mu);
    if (ctx->server) return RN_EINVAL;
    FBM_TRY(hipSetDevice(ctx->device));
    const int64_t n = nx * ny * nz;
    const hipStream_t st = ctx->stream;
    const double *phi = field;
    const double *ud[3] = {nullptr, nullptr, nullptr};
    double *gd[3] = {nullptr, nullptr, nullptr};
    Scratch sc(ctx);
    if (mem == RN_MEM_HOST) {
        // stage: field, the uniforms and the bond arrays
        const size_t a = (8 * (size_t)n + 255) & ~(size_t)255;
        const size_t total = a * (1 + (dilute ? dim : 0) + dim);
        hipError_t he;
        sc.base = (char *)ctx->pool.alloc(total, &he);
        if (!sc.base) return RN_ENOMEM;
        char *p = sc.base;
        FBM_TRY(hipMemcpyAsync(p, field, 8 * n, hipMemcpyHostToDevice, st));
        phi = (const double *)p;
        p += a;
        for (int k = 0; dilute && k < dim; ++k, p += a) {
            FBM_TRY(hipMemcpyAsync(p, u[k], 8 * n, hipMemcpyHostToDevice, st));
            ud[k] = (const double *)p;
        }
        for (int k = 0; k < dim; ++k, p += a) gd[k] = (double *)p;
    } else {
        for (int k = 0; k < dim; ++k) {
            gd[k] = g_out[k];
            if (dilute) ud[k] = u[k];
        }
    }
    fbm_bonds_kernel<<<grid_of(n), 256, 0, st>>>(phi, (int)nx, (int)ny, (int)nz, dim, sigma, periodic, ud[0], ud[1],
                                                 ud[2], occupancy, gd[0], gd[1], gd[2]);
    FBM_TRY(hipGetLastError());
    if (mem == RN_MEM_HOST)
        for (int k = 0; k < dim; ++k) FBM_TRY(hipMemcpyAsync(g_out[k], gd[k], 8 * n, hipMemcpyDeviceToHost, st));
    FBM_TRY(hipStreamSynchronize(st));
    return RN_OK;
}
