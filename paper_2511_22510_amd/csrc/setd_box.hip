// setd_box.hip -- box-averaged widths of 1D lattices (SETD_OBS_BOXWIDTH).
#include "setd_kernels.hpp"
#include "setd_launch.hpp"

namespace setd {

// ---------------------------------------------------------------- box-averaged width of lines
// The class sums A_c of box size l have c modulo P = N/l.  Since
// D_2l(a) = D_l(a) (1 + e^{2 pi i a l/N})/2 and e^{2 pi i a l/N} = e^{2 pi i c/P}
// depends on the class only, the sums of box size 2l follow from those of l by
//   A'_c = (A_c + A_{c+P/2})/2 + e^{2 pi i c/P} (A_c - A_{c+P/2})/2,  c < P/2,
// starting from A_c = h_c (l = 1, a = 0 left out): N - 1 pair sums per line
// instead of one Dirichlet factor and atomic per mode and level.  One
// wavefront per line: lane t holds the modes t + 64 q, so the pairs of the
// first rounds share a lane and those of the last six are lane XOR P/2.
// Bound by reading the stored modes once; KPZ line N = 1024 x 4096
// realizations: 72 ms (three launches per realization, FP64 atomics) before.
template <typename T, int EPL>
__global__ void __launch_bounds__(256) k_boxline(BoxLineArgs a)
{
    constexpr int RL = ilog2(EPL);   // rounds within a lane
    const Geo& g = a.g;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int N = a.N;
    double s0 = 0.0, s[RL + 6];
#pragma unroll
    for (int i = 0; i < RL + 6; i++) s[i] = 0.0;
    // e^{2 pi i c / P}
    auto zof = [&](int c, int P) {
        const int k = c * (N / P);
        return make_double2(a.tw[2 * k], -a.tw[2 * k + 1]);
    };
    auto half_sum = [](double2 u, double2 w, double2 z) {
        const double dx = 0.5 * (u.x - w.x), dy = 0.5 * (u.y - w.y);
        return make_double2(0.5 * (u.x + w.x) + z.x * dx - z.y * dy, 0.5 * (u.y + w.y) + z.x * dy + z.y * dx);
    };
    for (int r = (int)blockIdx.x * 4 + wv; r < a.nitems; r += (int)gridDim.x * 4) {
        const cx<T>* phi = reinterpret_cast<const cx<T>*>(a.items[r].phi);
        double2 e[EPL];
#pragma unroll
        for (int q = 0; q < EPL; q++) {
            // lanes past a line of fewer than 64 sites repeat its modes
            const int k = (EPL == 1) ? (lane & (N - 1)) : lane + 64 * q;
            e[q] = make_double2(0.0, 0.0);
            const bool mirror = !g.cplx && 2 * k > N;
            const int i = g.cplx ? stored_idx(k, N, g.kept[0], g.kp[0]) : (mirror ? N - k : k);
            if (k != 0 && i >= 0 && i < g.kept[0]) {
                const cx<T> p = phi[i];
                e[q] = make_double2((double)p.x, mirror ? -(double)p.y : (double)p.y);
            }
            if (EPL > 1 || lane < N) s0 += e[q].x * e[q].x + e[q].y * e[q].y;
        }
#pragma unroll
        for (int i = 0; i < RL; i++) {
            constexpr int E2 = EPL / 2;
            const int hl = E2 >> i;   // lane elements of the new classes
#pragma unroll
            for (int q = 0; q < E2; q++) {
                if (q >= hl) continue;
                e[q] = half_sum(e[q], e[q + hl], zof(lane + 64 * q, 128 * hl));
                s[i] += e[q].x * e[q].x + e[q].y * e[q].y;
            }
        }
#pragma unroll
        for (int u = 0; u < 6; u++) {
            const int P = 64 >> u, h = P / 2;
            if (EPL == 1 && P > N) continue;
            const double2 o = make_double2(__shfl_xor(e[0].x, h), __shfl_xor(e[0].y, h));
            const bool up = (lane & h) != 0;
            e[0] = half_sum(up ? o : e[0], up ? e[0] : o, zof(lane & (h - 1), P));
            if (lane < h) s[RL + u] += e[0].x * e[0].x + e[0].y * e[0].y;
        }
    }
    __shared__ double red[4][RL + 7];
    auto wave_sum = [](double v) {
#pragma unroll
        for (int h = 32; h > 0; h >>= 1) v += __shfl_xor(v, h);
        return v;
    };
    s0 = wave_sum(s0);
    if (lane == 0) red[wv][0] = s0;
#pragma unroll
    for (int i = 0; i < RL + 6; i++) {
        const double v = wave_sum(s[i]);
        if (lane == 0) red[wv][i + 1] = v;
    }
    __syncthreads();
    // round i is level i + 1; a line of N < 64 sites starts at round 6 - J
    const int skip = RL + 6 - a.J;
    const int i = threadIdx.x;
    if (i <= RL + 6 && (i == 0 || i > skip))
        atomicAdd(&a.sums[i == 0 ? 0 : i - skip], red[0][i] + red[1][i] + red[2][i] + red[3][i]);
}

// one wavefront per line; at most 1024 blocks, so that the per-level atomics
// stay few (one per block and level)
template <typename T>
hipError_t launch_boxline(const BoxLineArgs& a, hipStream_t s)
{
    int blocks = (a.nitems + 3) / 4;
    if (blocks > 1024) blocks = 1024;
    switch (a.N) {
    case 128: hipLaunchKernelGGL((k_boxline<T, 2>), dim3(blocks), dim3(256), 0, s, a); break;
    case 256: hipLaunchKernelGGL((k_boxline<T, 4>), dim3(blocks), dim3(256), 0, s, a); break;
    case 512: hipLaunchKernelGGL((k_boxline<T, 8>), dim3(blocks), dim3(256), 0, s, a); break;
    case 1024: hipLaunchKernelGGL((k_boxline<T, 16>), dim3(blocks), dim3(256), 0, s, a); break;
    default:
        if (a.N > 64) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_boxline<T, 1>), dim3(blocks), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

template hipError_t launch_boxline<float>(const BoxLineArgs&, hipStream_t);
template hipError_t launch_boxline<double>(const BoxLineArgs&, hipStream_t);

}  // namespace setd
