// Kernels that consume the dFD outputs (robot independent, built into the library).
//
// Vector-Jacobian product of forward dynamics (Sec. IV-B: dqdd/du = -M^-1 dRNEA/du,
// dqdd/dtau = M^-1):
//   qbar = (dqdd/dq)^T g,  qdbar = (dqdd/dqd)^T g,  taubar = M^-1 g  (M^-1 symmetric).
// One thread per (knot, joint j); for a fixed row i the threads of a knot read the
// contiguous row i of each matrix.
//
// Jacobians of one semi-implicit Euler step, the discrete-time dynamics of trajectory
// optimisation: qd' = qd + dt qdd(q, qd, tau), q' = q + dt qd', x = (q, qd):
//   A = dx'/dx   = [[1 + dt^2 Dq, dt 1 + dt^2 Dqd], [dt Dq, 1 + dt Dqd]]   [2n][2n]
//   B = dx'/dtau = [[dt^2 M^-1], [dt M^-1]]                               [2n][n]
// with Dq = dqdd/dq, Dqd = dqdd/dqd.
#include <hip/hip_runtime.h>

extern "C" __global__ void __launch_bounds__(256)
grid_vjp_kernel(int nknots, int n, const float* __restrict__ dq, const float* __restrict__ dqd,
                const float* __restrict__ Minv, const float* __restrict__ g,
                float* __restrict__ qbar, float* __restrict__ qdbar, float* __restrict__ taubar)
{
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long)nknots * n)
        return;
    const long k = idx / n;
    const int j = (int)(idx % n);
    const long m0 = k * n * n;
    const float* gk = g + k * n;
    float sq = 0.0f, sqd = 0.0f, st = 0.0f;
    for (int i = 0; i < n; ++i) {
        const float gi = gk[i];
        const long o = m0 + (long)i * n + j;
        sq += dq[o] * gi;
        sqd += dqd[o] * gi;
        st += Minv[o] * gi;
    }
    qbar[idx] = sq;
    qdbar[idx] = sqd;
    taubar[idx] = st;
}

// x / n for the x < 2^16 met here; magic = floor(2^32 / n) + 1 (n > 1)
__device__ __forceinline__ unsigned div_small(unsigned x, unsigned n, unsigned magic)
{
    return n == 1 ? x : __umulhi(x, magic);
}

// A workgroup takes `kpb` whole knots. The upper half of a knot's A is the rows of Dq and Dqd side
// by side and the lower half the same with other factors, so a thread reads one entry and writes
// two, and consecutive threads read runs of n and write without gaps; B likewise from M^-1.
// Bound by memory (9 n^2 floats per knot). One entry per thread, its place found by four 64-bit
// divisions, took 89 us for 12 joints at 32768 knots (1.9 TB/s).
extern "C" __global__ void __launch_bounds__(256)
grid_dt_kernel(int nknots, int n, int kpb, unsigned magic_n, unsigned magic_2n, float dt,
               const float* __restrict__ dq, const float* __restrict__ dqd,
               const float* __restrict__ Minv, float* __restrict__ A, float* __restrict__ B)
{
    const long k0 = (long)blockIdx.x * kpb;
    const unsigned nn = n * n, n2 = 2 * n;
    const unsigned knots = (unsigned)min((long)kpb, nknots - k0);
    const float* q0 = dq + k0 * nn;
    const float* v0 = dqd + k0 * nn;
    const float* m0 = Minv + k0 * nn;
    float* A0 = A + k0 * 4 * nn;
    float* B0 = B + k0 * 2 * nn;
    const float dt2 = dt * dt;
    for (unsigned e = threadIdx.x; e < knots * 2 * nn; e += 256) {
        const unsigned row = div_small(e, n2, magic_2n);       // knot n + i
        const unsigned k = div_small(row, n, magic_n);
        const unsigned c = e - row * n2, i = row - k * n;
        const bool left = c < (unsigned)n;
        const unsigned j = left ? c : c - n;
        const float d = (left ? q0 : v0)[row * n + j];
        const float eye = i == j ? 1.0f : 0.0f;
        float* a = A0 + k * 2 * nn + e;                        // knot k's A starts at 4 k n^2
        a[0] = (left ? eye : dt * eye) + dt2 * d;
        a[2 * nn] = left ? dt * d : eye + dt * d;
    }
    for (unsigned e = threadIdx.x; e < knots * nn; e += 256) {
        const unsigned k = div_small(div_small(e, n, magic_n), n, magic_n);
        const float m = m0[e];
        float* b = B0 + k * nn + e;                            // knot k's B starts at 2 k n^2
        b[0] = dt2 * m;
        b[nn] = dt * m;
    }
}

namespace grid_impl {

hipError_t launch_dt(int nknots, int n, float dt, const float* dq, const float* dqd,
                     const float* Minv, float* A, float* B, hipStream_t stream)
{
    // about eight entries per thread of the two loops; at most 2048 entries of A's half a knot
    const int kpb = n * n >= 1024 ? 1 : 1024 / (n * n);
    const unsigned blocks = (unsigned)((nknots + kpb - 1L) / kpb);
    const auto magic = [](unsigned d) { return (unsigned)((1ull << 32) / d + 1); };
    hipLaunchKernelGGL(grid_dt_kernel, dim3(blocks), dim3(256), 0, stream, nknots, n, kpb,
                       magic(n), magic(2 * n), dt, dq, dqd, Minv, A, B);
    return hipGetLastError();
}

hipError_t launch_vjp(int nknots, int n, const float* dq, const float* dqd, const float* Minv,
                      const float* g, float* qbar, float* qdbar, float* taubar, hipStream_t stream)
{
    const long total = (long)nknots * n;
    const unsigned blocks = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(grid_vjp_kernel, dim3(blocks), dim3(256), 0, stream, nknots, n, dq, dqd,
                       Minv, g, qbar, qdbar, taubar);
    return hipGetLastError();
}

}  // namespace grid_impl
