// obs.hip -- structural observables of every walker at a sample point (the axial
// density and the lateral radial distribution of a layer, Sec. III.A), as integer
// counts per sample for the reweighting of Eq. (11).  One workgroup per walker,
// histograms in LDS.  Compiled without FP contraction: the bin of every particle
// and pair is the one a plain FP64 evaluation gives (minimum image by comparison
// with half the box, r = sqrt(dx^2 + dy^2), bin = floor(r / dr)).
#include "regc_dev.h"

namespace regc {

constexpr int kObsMaxBins = 2048;

__device__ __forceinline__ double obs_min_image(double d, double box)
{
    return d > 0.5 * box ? d - box : (d < -0.5 * box ? d + box : d);
}

// The layer's members are put into LDS first and their pairs dealt evenly to the
// threads: member i with the next (M - 1) / 2 of the ring of M, and for even M the first
// half with their opposites.  (A wave per walker that went through the particles one by one,
// each against the later ones read from memory: 104 us for 1024 walkers with N <= 200; this
// 7 us, bound by the pairs' FP64 roots and quotients.)  More members than kObsMembers are
// read from memory as before.
constexpr int kObsMembers = 1024, kObsThreads = 256;

__global__ void __launch_bounds__(kObsThreads) obs_kernel(ObsArgs a)
{
    __shared__ uint32_t hist[kObsMaxBins];
    __shared__ double2 member[kObsMembers];
    __shared__ int count;
    const int w = blockIdx.x, tid = threadIdx.x;
    const ClassDev &C = a.cls[a.walker_class[w]];
    const int n = a.n[w];
    const double *x = a.xyz + (size_t)w * a.xyz_stride * 3;
    for (int k = tid; k < a.n_obs; k += kObsThreads) hist[k] = 0u;
    if (tid == 0) count = 0;
    __syncthreads();
    const int nz = (int)ceil((C.zhi - C.zlo) / a.dz);
    const double lx = C.lx, ly = C.ly;
    for (int i = tid; i < n; i += kObsThreads) {
        const double z = x[3 * i + 2];
        int kz = (int)floor((z - C.zlo) / a.dz);
        kz = kz < 0 ? 0 : (kz > nz - 1 ? nz - 1 : kz);
        atomicAdd(hist + kz, 1u);
        if (z >= a.layer_lo && z < a.layer_hi) {
            const int k = atomicAdd(&count, 1);
            if (k < kObsMembers) member[k] = make_double2(x[3 * i], x[3 * i + 1]);
        }
    }
    __syncthreads();
    const int M = count;
    auto pair = [&](double xi, double yi, double xj, double yj) {
        const double dx = obs_min_image(xi - xj, lx);
        const double dy = obs_min_image(yi - yj, ly);
        const double r = sqrt(dx * dx + dy * dy);
        const int kr = (int)floor(r / a.dr);
        if (kr < a.n_r) atomicAdd(hist + a.n_z + kr, 1u);
    };
    if (M <= kObsMembers) {
        const int pairs = M * ((M - 1) / 2) + (M % 2 == 0 ? M / 2 : 0);
        for (int p = tid; p < pairs; p += kObsThreads) {
            const int k = p / M, i = p - k * M;
            const int j = i + k + 1 < M ? i + k + 1 : i + k + 1 - M;
            const double2 u = member[i], v = member[j];
            pair(u.x, u.y, v.x, v.y);
        }
    } else {
        for (int i = 0; i < n; ++i) {
            const double zi = x[3 * i + 2];
            if (!(zi >= a.layer_lo && zi < a.layer_hi)) continue;       // uniform across the block
            const double xi = x[3 * i], yi = x[3 * i + 1];
            for (int j = i + 1 + tid; j < n; j += kObsThreads) {
                const double zj = x[3 * j + 2];
                if (zj >= a.layer_lo && zj < a.layer_hi) pair(xi, yi, x[3 * j], x[3 * j + 1]);
            }
        }
    }
    if (tid == 0) hist[a.n_z + a.n_r] = (uint32_t)M;
    __syncthreads();
    uint32_t *out = a.out + (size_t)w * a.n_obs;
    for (int k = tid; k < a.n_obs; k += kObsThreads) out[k] = hist[k];
}

// IEEE double -> unsigned key of the same order (zero of either sign as +0)
__device__ __forceinline__ unsigned long long energy_key(double e)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(e == 0.0 ? 0.0 : e);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__device__ __forceinline__ unsigned long long load_u64(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int load_i32(const int *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One workgroup: (0) remember the keys, (1) atomic minimum of every walker's energy
// key per (class, N), (2) among walkers at a new strict minimum the lowest index,
// (3) that walker stores its energy and configuration; the index slots are cleared.
// The result is the oracle's sequential rule (walkers in index order, replaced only
// by a strictly lower energy).
__global__ void __launch_bounds__(1024) minima_kernel(MinArgs a)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    const int slots = a.n_class * a.nN;
    for (int k = tid; k < slots; k += nt) a.old_key[k] = load_u64(a.key + k);
    __syncthreads();
    for (int w = tid; w < a.n_walkers; w += nt)
        atomicMin(a.key + a.walker_class[w] * a.nN + a.n[w], energy_key(a.e[w]));
    __syncthreads();
    for (int w = tid; w < a.n_walkers; w += nt) {
        const int k = a.walker_class[w] * a.nN + a.n[w];
        const unsigned long long ek = energy_key(a.e[w]);
        if (ek == load_u64(a.key + k) && ek < a.old_key[k]) atomicMin(a.widx + k, w);
    }
    __syncthreads();
    for (int w = tid; w < a.n_walkers; w += nt) {
        const int k = a.walker_class[w] * a.nN + a.n[w];
        if (load_i32(a.widx + k) != w) continue;
        a.e_min[k] = a.e[w];
        const double *src = a.xyz + (size_t)w * a.xyz_stride * 3;
        double *dst = a.xyz_min + (size_t)k * a.xyz_stride * 3;
        for (int q = 0; q < 3 * a.n[w]; ++q) dst[q] = src[q];
    }
    __syncthreads();
    for (int w = tid; w < a.n_walkers; w += nt) {
        const int k = a.walker_class[w] * a.nN + a.n[w];
        if (load_i32(a.widx + k) == w) a.widx[k] = 0x7fffffff;
    }
}

hipError_t launch_minima(const MinArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(minima_kernel, dim3(1), dim3(1024), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_observables(const ObsArgs &a, hipStream_t s)
{
    if (a.n_obs > kObsMaxBins) return hipErrorInvalidValue;
    hipLaunchKernelGGL(obs_kernel, dim3(a.n_walkers), dim3(kObsThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace regc
