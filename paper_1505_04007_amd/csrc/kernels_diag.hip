// Probe DFT (FP64 accumulators) and FP64 check-path diagnostics.
#include "pic_internal.hpp"

namespace pic {

constexpr int PROBE_BLOCK = 256;

// LARGE as in probe_dft.  Its code here and in the H update made one step of 32x32x32
// cells, alone, 0.25 us of 21.1 slower.
template <int LARGE>
__global__ __launch_bounds__(PROBE_BLOCK) void k_probe(ProbeArgs a, int advance)
{
    const gp<DevState> st = G(a.st);
    const long long n1 = st->step + advance;
    probe_dft<LARGE>(a, n1, threadIdx.x, PROBE_BLOCK);
    if (!advance) return;
    __syncthreads();  // every thread has read the clock before it moves
    if (threadIdx.x == 0) {
        st->parity ^= 1;
        st->since_sort += 1;
        st->step = n1;
    }
}

__global__ __launch_bounds__(PROBE_BLOCK) void k_probe_batch(const ProbeArgs *args)
{
    const ProbeArgs &a = args[blockIdx.x];
    probe_dft<1>(a, G(a.st)->step, threadIdx.x, PROBE_BLOCK);
}

void launch_probe(const ProbeArgs &a, bool advance, hipStream_t s)
{
    if (a.nprobe <= 0 && !advance) return;
    if (a.large) hipLaunchKernelGGL(k_probe<1>, dim3(1), dim3(PROBE_BLOCK), 0, s, a, advance ? 1 : 0);
    else hipLaunchKernelGGL(k_probe<0>, dim3(1), dim3(PROBE_BLOCK), 0, s, a, advance ? 1 : 0);
}

void launch_probe_batch(const ProbeArgs *args, int n, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_probe_batch, dim3(n), dim3(PROBE_BLOCK), 0, s, args);
}

// Node-centred cloud-in-cell charge density in FP64 (nodes (nx+1)(ny+1)(nz+1)).
__global__ void k_rho(DiagArgs a)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.np) return;
    if (!live_pos(a.x[p], a.y[p], a.z[p], a.nx, a.ny, a.nz)) return;
    const double X[3] = {(double)a.x[p], (double)a.y[p], (double)a.z[p]};
    int i0[3];
    double fr[3];
    const int n[3] = {a.nx, a.ny, a.nz};
    for (int d = 0; d < 3; ++d) {
        const double f = floor(X[d]);
        i0[d] = (int)f;
        fr[d] = X[d] - f;
    }
    for (int c = 0; c < 2; ++c)
        for (int b = 0; b < 2; ++b)
            for (int q = 0; q < 2; ++q) {
                int id[3] = {i0[0] + q, i0[1] + b, i0[2] + c};
                bool skip = false;
                for (int d = 0; d < 3; ++d) {
                    if (a.per[d]) id[d] = id[d] >= n[d] ? id[d] - n[d] : id[d];
                    if (id[d] < 0 || id[d] > n[d]) skip = true;
                }
                if (skip) continue;
                const double w = (q ? fr[0] : 1 - fr[0]) * (b ? fr[1] : 1 - fr[1]) * (c ? fr[2] : 1 - fr[2]);
                atomicAdd(&a.rho[id[0] + (a.nx + 1) * (id[1] + (a.ny + 1) * id[2])], a.qw_over_vol * w);
            }
}

void launch_rho(const DiagArgs &a, hipStream_t s)
{
    if (a.np <= 0) return;
    hipLaunchKernelGGL(k_rho, dim3((unsigned)(((long long)a.np + 255) / 256)), dim3(256), 0, s, a);
}

__device__ __forceinline__ double warp_sum(double v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ double warp_max(double v)
{
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ __forceinline__ void atomic_max_pos(double *addr, double v)
{
    // non-negative doubles order like their bit patterns
    atomicMax((unsigned long long *)addr, (unsigned long long)__double_as_longlong(v));
}

// acc layout: [0] sum (E^2 + Ht^2), [1] count, [2..4] sum x, [5..7] sum x^2,
// [8..10] sum u, [11] max |G|, [12] max |rho0|, [13] checked nodes
__global__ __launch_bounds__(256) void k_diag_fields(DiagArgs a)
{
    const long long n = (long long)a.nx * a.ny * a.nz;
    double s = 0.0;
    for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < n;
         q += (long long)gridDim.x * blockDim.x) {
        for (int c = 0; c < 3; ++c) {
            const double e = a.E[c][q], h = a.H[c][q];
            s += e * e + h * h;
        }
    }
    // (one atomic per workgroup: they follow each other at 13 ns, and one per
    // wavefront took 52 us on the smallest grid)
    __shared__ double part[4];
    s = warp_sum(s);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(&a.acc[0], part[0] + part[1] + part[2] + part[3]);
}

// Grid-stride sums over the live particles, reduced per wavefront, then per
// workgroup in LDS, then one FP64 atomic per workgroup and quantity (a fixed
// grid keeps the same-address atomics to a few thousand).
__global__ __launch_bounds__(256) void k_diag_particles(DiagArgs a)
{
    __shared__ double part[4][10];
    double v[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < a.np;
         p += (long long)gridDim.x * blockDim.x) {
        if (!live_pos(a.x[p], a.y[p], a.z[p], a.nx, a.ny, a.nz)) continue;
        const double X[3] = {a.x[p], a.y[p], a.z[p]};
        const double U[3] = {a.ux[p], a.uy[p], a.uz[p]};
        v[0] += 1.0;
        for (int d = 0; d < 3; ++d) {
            v[1 + d] += X[d];
            v[4 + d] += X[d] * X[d];
            v[7 + d] += U[d];
        }
    }
    const int w = threadIdx.x >> 6;
    for (int q = 0; q < 10; ++q) {
        const double t = warp_sum(v[q]);
        if ((threadIdx.x & 63) == 0) part[w][q] = t;
    }
    __syncthreads();
    if (threadIdx.x < 10) {
        const double t = part[0][threadIdx.x] + part[1][threadIdx.x] + part[2][threadIdx.x] +
                         part[3][threadIdx.x];
        if (t != 0.0) atomicAdd(&a.acc[1 + threadIdx.x], t);
    }
}

// G = eps0 div E - rho at interior nodes away from CPML layers and the metal
// box, compared with its initial value -rho0 (E^0 = 0).
__global__ void k_diag_gauss(DiagArgs a)
{
    const long long n = (long long)(a.nx + 1) * (a.ny + 1) * (a.nz + 1);
    double gm = 0.0, rm = 0.0, cnt = 0.0;
    for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < n;
         q += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(q % (a.nx + 1));
        const int j = (int)((q / (a.nx + 1)) % (a.ny + 1));
        const int k = (int)(q / ((long long)(a.nx + 1) * (a.ny + 1)));
        if (a.rho0) rm = fmax(rm, fabs(a.rho0[q]));
        const int id[3] = {i, j, k};
        const int nn[3] = {a.nx, a.ny, a.nz};
        bool ok = true;
        for (int d = 0; d < 3; ++d)
            if (id[d] < 1 + a.npml[d] || id[d] > nn[d] - 1 - a.npml[d]) ok = false;
        if (ok && i >= a.mlo[0] - 1 && i <= a.mhi[0] && j >= a.mlo[1] - 1 && j <= a.mhi[1] &&
            k >= a.mlo[2] - 1 && k <= a.mhi[2])
            ok = false;
        if (!ok) continue;
        const long long c0 = i + (long long)a.nx * (j + (long long)a.ny * k);
        const double dE = ((double)a.E[0][c0] - (double)a.E[0][c0 - 1]) +
                          ((double)a.E[1][c0] - (double)a.E[1][c0 - a.nx]) +
                          ((double)a.E[2][c0] - (double)a.E[2][c0 - (long long)a.nx * a.ny]);
        double g = a.eps0_over_dx * dE - a.rho[q];
        if (a.rho0) g += a.rho0[q];
        gm = fmax(gm, fabs(g));
        cnt += 1.0;
    }
    gm = warp_max(gm);
    rm = warp_max(rm);
    cnt = warp_sum(cnt);
    if ((threadIdx.x & 63) == 0) {
        atomic_max_pos(&a.acc[11], gm);
        atomic_max_pos(&a.acc[12], rm);
        atomicAdd(&a.acc[13], cnt);
    }
}

// Live particles and pushes, summed per workgroup into out[2 b], out[2 b + 1] (the
// host adds the pairs up: no word to clear first, no atomics on one address), and
// the particle box behind them.
__global__ __launch_bounds__(STATS_BLOCK) void k_stats(DiagArgs a, const unsigned long long *pushes, int nslots,
                                                       const int *box, unsigned long long *out)
{
    const int t = blockIdx.x * STATS_BLOCK + threadIdx.x, step = gridDim.x * STATS_BLOCK;
    int live = 0;
#pragma unroll 4
    for (long long p = t; p < a.np; p += step) live += live_pos(a.x[p], a.y[p], a.z[p], a.nx, a.ny, a.nz);
    unsigned long long n = 0;
    for (long long w = t; w < nslots; w += step) n += pushes[w];
    __shared__ unsigned long long part[STATS_BLOCK / 64][2];
    unsigned long long l = live;
    for (int off = 32; off > 0; off >>= 1) {
        l += __shfl_xor(l, off, 64);
        n += __shfl_xor(n, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        part[threadIdx.x >> 6][0] = l;
        part[threadIdx.x >> 6][1] = n;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned long long v = 0;
        for (int w = 0; w < STATS_BLOCK / 64; ++w) v += part[w][threadIdx.x];
        out[2 * blockIdx.x + threadIdx.x] = v;
    }
    if (blockIdx.x == 0 && threadIdx.x < 6) reinterpret_cast<int *>(out + 2 * STATS_BLOCKS)[threadIdx.x] = box[threadIdx.x];
}

int launch_stats(const DiagArgs &a, const unsigned long long *pushes, int nslots, const int *box,
                 unsigned long long *out, hipStream_t s)
{
    const int nb = (int)std::min<long long>(STATS_BLOCKS, ((long long)a.np + STATS_BLOCK - 1) / STATS_BLOCK);
    hipLaunchKernelGGL(k_stats, dim3(nb), dim3(STATS_BLOCK), 0, s, a, pushes, nslots, box, out);
    return nb;
}

void launch_diag_reduce(const DiagArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_diag_fields, dim3(1024), dim3(256), 0, s, a);
    if (a.np > 0) hipLaunchKernelGGL(k_diag_particles, dim3(1024), dim3(256), 0, s, a);
    if (a.rho) hipLaunchKernelGGL(k_diag_gauss, dim3(1024), dim3(256), 0, s, a);
}

}  // namespace pic
