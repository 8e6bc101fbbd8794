// Molecular-dynamics kernels for the potential's main application (Sec. IV.C:
// equilibrium and driven MD of diamond Si): velocity-Verlet kicks and drifts,
// the homogeneous non-equilibrium driving force built from the per-atom
// virial, and deterministic kinetic-energy / momentum sums.
//
// Units: positions A, velocities A/fs, forces eV/A, masses u, time fs; a force
// F on a mass m accelerates by F / (m * 103.642691) A/fs^2 (1 u A^2/fs^2 =
// 103.642691 eV).  Arrays are SoA [3][N] float64 in the caller's atom order.
#include <hip/hip_runtime.h>

#include "mt_host.h"

namespace mt {
namespace {

constexpr double kAccel = 1.0 / 103.642691;

int blocks_for(int n) { return (n + 255) / 256; }

// dt_half (F_i + F_ext,i - <F_ext>) / m_i, with F_ext,i = W_i^T F_e
// (W_i row-major [9][N]) and <F_ext> = W^T F_e / N from the symmetric total
// virial (xx yy zz yz zx xy), so that the driving force adds no momentum.
struct KickArgs {
    const double* force;
    const double* atom_virial;
    const double* virial6;
    double fe[3];
    const double* inv_mass;
    double dt_half;
};

__device__ __forceinline__ void kicked(const KickArgs& K, int N, int i, double* __restrict__ vel, double (&v)[3]) {
    double f[3] = {K.force[i], K.force[(size_t)N + i], K.force[(size_t)2 * N + i]};
    if (K.atom_virial) {
        double W[3][3];
        const double* w = K.virial6;
        W[0][0] = w[0]; W[1][1] = w[1]; W[2][2] = w[2];
        W[1][2] = W[2][1] = w[3]; W[2][0] = W[0][2] = w[4]; W[0][1] = W[1][0] = w[5];
        for (int b = 0; b < 3; ++b) {
            double ext = 0.0, mean = 0.0;
            for (int a = 0; a < 3; ++a) {
                ext += K.fe[a] * K.atom_virial[(size_t)(3 * a + b) * N + i];
                mean += K.fe[a] * W[a][b];
            }
            f[b] += ext - mean / N;
        }
    }
    const double s = K.dt_half * kAccel * K.inv_mass[i];
    for (int k = 0; k < 3; ++k) {
        v[k] = vel[(size_t)k * N + i] + s * f[k];
        vel[(size_t)k * N + i] = v[k];
    }
}

__global__ __launch_bounds__(256) void k_kick(int N, double* __restrict__ vel, KickArgs K) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    double v[3];
    if (i < N) kicked(K, N, i, vel, v);
}

__global__ __launch_bounds__(256) void k_drift(int N, double* __restrict__ pos,
                                               const double* __restrict__ vel, double dt) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    for (int k = 0; k < 3; ++k) pos[(size_t)k * N + i] += dt * vel[(size_t)k * N + i];
}

__global__ __launch_bounds__(256) void k_scale(int N, double* __restrict__ vel, double lambda) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    for (int k = 0; k < 3; ++k) vel[(size_t)k * N + i] *= lambda;
}

// Atoms per thread whose loads are issued together in the single-block
// reductions below (one memory latency per round instead of one per atom).
constexpr int kBatch = 8;

// One block: each thread sums a fixed strided subset (atoms t, t + 1024, ...
// in ascending order), then butterflies over a wavefront and one barrier; the
// result depends only on N.  Bound by the latency of one block's loads (8,000
// atoms: 6.5 us with a barrier per level of a tree over 1,024 threads, 5.6 now).
// out = [sum m v^2, sum m v_x, sum m v_y, sum m v_z].
__global__ __launch_bounds__(1024) void k_kinetic(int N, const double* __restrict__ vel,
                                                  const double* __restrict__ mass,
                                                  double* __restrict__ out) {
    __shared__ double sh[4][16];
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i0 = threadIdx.x; i0 < N; i0 += kBatch * blockDim.x) {
        double m[kBatch], vx[kBatch], vy[kBatch], vz[kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const int i = i0 + b * blockDim.x;
            const bool in = i < N;
            m[b] = in ? mass[i] : 0.0;
            vx[b] = in ? vel[i] : 0.0;
            vy[b] = in ? vel[(size_t)N + i] : 0.0;
            vz[b] = in ? vel[(size_t)2 * N + i] : 0.0;
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            if (i0 + b * (int)blockDim.x >= N) break;
            a[0] += m[b] * (vx[b] * vx[b] + vy[b] * vy[b] + vz[b] * vz[b]);
            a[1] += m[b] * vx[b];
            a[2] += m[b] * vy[b];
            a[3] += m[b] * vz[b];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int k = 0; k < 4; ++k) a[k] += __shfl_xor(a[k], o, 64);
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < 4; ++k) sh[k][threadIdx.x >> 6] = a[k];
    __syncthreads();
    if (threadIdx.x < 4) {
        double t = 0.0;
        for (int w = 0; w < 16; ++w) t += sh[threadIdx.x][w];
        out[threadIdx.x] = t;
    }
}

// out[0] = max_i |r_i - r0_i|^2 (exact: max is order independent), atoms whose
// displacement is not a number left out.  The blocks meet in an atomic maximum of
// the bit patterns, which order like the values of doubles that are not negative;
// k_clear sets out to zero first.  One block for all atoms is bound by a single
// compute unit's loads: 8,000 atoms 9.6 us, 3.9 us with the clear.
__global__ void k_clear(unsigned long long* out) { *out = 0ull; }
__device__ __forceinline__ void block_max(double a, unsigned long long* __restrict__ out) {
    __shared__ double sh[4];
    a = __builtin_fmax(a, 0.0);
    for (int o = 32; o > 0; o >>= 1) a = __builtin_fmax(a, __shfl_xor(a, o, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) a = __builtin_fmax(a, sh[w]);
        atomicMax(out, (unsigned long long)__double_as_longlong(a));
    }
}
__global__ __launch_bounds__(256) void k_max_disp(int N, const double* __restrict__ pos,
                                                  const double* __restrict__ ref,
                                                  unsigned long long* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    double a = 0.0;
    if (i < N)
        for (int k = 0; k < 3; ++k) {
            const double d = pos[(size_t)k * N + i] - ref[(size_t)k * N + i];
            a += d * d;
        }
    block_max(a, out);
}

// The first half of a velocity-Verlet step in one pass: k_kick, k_drift and,
// with out, k_max_disp, to the same bits.  Each of the three is little more than
// a launch and the latency of its loads (8,000 atoms: 3.0 + 2.4 + 2.6 us, 4.2 us
// in one).
__global__ __launch_bounds__(256) void k_first_half(int N, double* __restrict__ vel, KickArgs K,
                                                    double* __restrict__ pos, double dt,
                                                    const double* __restrict__ ref,
                                                    unsigned long long* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    double a = 0.0;
    if (i < N) {
        double v[3];
        kicked(K, N, i, vel, v);
        for (int k = 0; k < 3; ++k) {
            const double p = pos[(size_t)k * N + i] + dt * v[k];
            pos[(size_t)k * N + i] = p;
            if (out) {
                const double d = p - ref[(size_t)k * N + i];
                a += d * d;
            }
        }
    }
    if (out) block_max(a, out);
}

int kick_args(int N, const double* vel, const double* force, const double* atom_virial, const double* virial,
              const double* fe, const double* inv_mass, double dt_half, KickArgs& K) {
    if (N <= 0) { set_error("N must be positive"); return MT_EINVAL; }
    if (!vel || !force || !inv_mass) { set_error("vel, force and inv_mass must not be NULL"); return MT_EINVAL; }
    if ((atom_virial != nullptr) != (fe != nullptr) || (atom_virial && !virial)) {
        set_error("the driving force needs fe, atom_virial and virial together");
        return MT_EINVAL;
    }
    K = KickArgs{force, atom_virial, virial, {fe ? fe[0] : 0.0, fe ? fe[1] : 0.0, fe ? fe[2] : 0.0}, inv_mass, dt_half};
    return MT_OK;
}

}  // namespace
}  // namespace mt

using namespace mt;

extern "C" {

int mt_md_kick(int N, double* vel, const double* force, const double* atom_virial,
               const double* virial, const double* fe, const double* inv_mass, double dt_half,
               void* stream) {
    KickArgs K;
    const int rc = kick_args(N, vel, force, atom_virial, virial, fe, inv_mass, dt_half, K);
    if (rc != MT_OK) return rc;
    hipLaunchKernelGGL(k_kick, dim3(blocks_for(N)), dim3(256), 0, (hipStream_t)stream, N, vel, K);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? MT_OK : hip_fail(e, "k_kick");
}

int mt_md_first_half(int N, double* vel, const double* force, const double* atom_virial,
                     const double* virial, const double* fe, const double* inv_mass, double dt_half,
                     double* pos, double dt, const double* ref, double* out, void* stream) {
    KickArgs K;
    const int rc = kick_args(N, vel, force, atom_virial, virial, fe, inv_mass, dt_half, K);
    if (rc != MT_OK) return rc;
    if (!pos || (ref != nullptr) != (out != nullptr)) {
        set_error("pos must not be NULL; ref and out go together");
        return MT_EINVAL;
    }
    auto bits = reinterpret_cast<unsigned long long*>(out);
    if (bits) hipLaunchKernelGGL(k_clear, dim3(1), dim3(1), 0, (hipStream_t)stream, bits);
    hipLaunchKernelGGL(k_first_half, dim3(blocks_for(N)), dim3(256), 0, (hipStream_t)stream, N, vel, K, pos, dt,
                       ref, bits);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? MT_OK : hip_fail(e, "k_first_half");
}

int mt_md_drift(int N, double* pos, const double* vel, double dt, void* stream) {
    if (N <= 0 || !pos || !vel) { set_error("N must be positive, pos and vel not NULL"); return MT_EINVAL; }
    hipLaunchKernelGGL(k_drift, dim3(blocks_for(N)), dim3(256), 0, (hipStream_t)stream, N, pos, vel, dt);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? MT_OK : hip_fail(e, "k_drift");
}

int mt_md_scale(int N, double* vel, double lambda, void* stream) {
    if (N <= 0 || !vel) { set_error("N must be positive, vel not NULL"); return MT_EINVAL; }
    hipLaunchKernelGGL(k_scale, dim3(blocks_for(N)), dim3(256), 0, (hipStream_t)stream, N, vel, lambda);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? MT_OK : hip_fail(e, "k_scale");
}

int mt_md_max_disp(int N, const double* pos, const double* ref, double* out, void* stream) {
    if (N <= 0 || !pos || !ref || !out) { set_error("N must be positive, pointers not NULL"); return MT_EINVAL; }
    auto bits = reinterpret_cast<unsigned long long*>(out);
    hipLaunchKernelGGL(k_clear, dim3(1), dim3(1), 0, (hipStream_t)stream, bits);
    hipLaunchKernelGGL(k_max_disp, dim3(blocks_for(N)), dim3(256), 0, (hipStream_t)stream, N, pos, ref, bits);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? MT_OK : hip_fail(e, "k_max_disp");
}

int mt_md_kinetic(int N, const double* vel, const double* mass, double* out, void* stream) {
    if (N <= 0 || !vel || !mass || !out) { set_error("N must be positive, pointers not NULL"); return MT_EINVAL; }
    hipLaunchKernelGGL(k_kinetic, dim3(1), dim3(1024), 0, (hipStream_t)stream, N, vel, mass, out);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? MT_OK : hip_fail(e, "k_kinetic");
}

}  // extern "C"
