// setd_small_impl.hpp -- whole time steps of small 2D lattices in one kernel.
//
// A 2D real field of 32 or 64 points per axis fits one workgroup: the stored
// columns of its axis-0 intermediate (64 x 22 modes: 11 KiB in FP32) stay in
// LDS and the state, history and coefficients in the registers of the threads
// that update them, for up to 256 steps per launch (as on 1D lines).  The
// passes of the general path need two dependent launches a step, of a few
// microseconds each whatever the size.
//
// A step is the row pass (row pairs as complex lines: inverse, nonlinearity,
// forward) and the axis-0 pass (forward, update, inverse) of the general path
// on LDS data.  Every line lies within one wavefront, so the transforms order
// their exchanges by wavefront only and a step takes two block barriers.
// The noise is drawn by wavefronts of its own, one step ahead into a second
// LDS buffer, beside the transforms.
//
// Bound by the latency of a step's two dependent transform pairs on one CU.
// 64^2, us per step (the two-pass path before): FP64 SETD1 4.6 (14.7), FP32
// SETD2 2.5 (11.0), KPZ FP32 3.5; 256 realizations 2.8 (14.6).
#pragma once

#include "setd_kernels.hpp"
#include "setd_launch.hpp"

namespace setd {

struct SmallArgs {
    Geo g;
    const Item* items;
    int sub;      // first sub-step of the scheduler tick
    int nsteps;   // steps of this launch (each item at most its own steps)
    Record rec;   // the time-series window, if one is open
};

template <typename T, int N0, int N1, bool KPZ>
struct SmallShape {
    static constexpr int TPL0 = N0 / 8, TPL1 = N1 / 8, PAD = 3;
    static constexpr int K0 = (N0 - 1) / 3, K1 = (N1 - 1) / 3;
    static constexpr int KEPT0 = 2 * K0 + 1, KC = K1 + 1;   // stored rows, stored columns
    static constexpr int PC = KC | 1;                       // LDS row pitch of the intermediate
    static constexpr int LINES = KPZ ? 2 : 1;
    static constexpr int RW = N0 / 2 * TPL1 / 64;           // row wavefronts
    static constexpr int CPW = 64 / TPL0;                   // columns of a wavefront
    static constexpr int CW = (KC + CPW - 1) / CPW;         // column wavefronts
    static constexpr int FW = RW > CW ? RW : CW;
    static constexpr int TASKS = 3 * TPL0 * KC;             // Philox blocks of a step
    // noise wavefronts: one round of tasks beside the row pass, the others
    // beside the axis-0 pass, which leaves FW - CW of the rest idle
    static constexpr int NW = (TASKS - 64 * (FW - CW) + 127) / 128;
    static constexpr int THREADS = 64 * (FW + NW);
    static constexpr int XR = N0 / 2 * LINES * lds_len<N1, PAD>();
    static constexpr int XC = CW * CPW * lds_len<N0, PAD>();
    static constexpr int X = XR > XC ? XR : XC;             // exchange slots
    // coefficient entries: registers in FP32; FP64 threads have none to spare
    // and read them from LDS, or where that is full from global memory
    static constexpr int NCOEF = (K0 + 1) * KC;
    static constexpr size_t BASE = ((size_t)LINES * N0 * PC + X + 2 * 6 * 64 * CW) * 2 * sizeof(T);
    static constexpr bool CREG = sizeof(T) == 4;
    static constexpr bool CLDS = !CREG && BASE + (size_t)NCOEF * 4 * sizeof(T) <= 160 * 1024;
};

template <typename T, int N0, int N1, bool KPZ, bool LEAN>
__global__ void __launch_bounds__((SmallShape<T, N0, N1, KPZ>::THREADS)) k_small2d(SmallArgs a)
{
    typedef SmallShape<T, N0, N1, KPZ> SH;
    constexpr int TPL0 = SH::TPL0, TPL1 = SH::TPL1, PAD = SH::PAD, K0 = SH::K0, K1 = SH::K1, PC = SH::PC,
                  KC = SH::KC, KEPT0 = SH::KEPT0, CPW = SH::CPW, FW = SH::FW;
    __shared__ cx<T> pre[SH::LINES][N0 * PC];
    __shared__ cx<T> X[SH::X];
    __shared__ cx<T> eta[2][6][64 * SH::CW];
    __shared__ T4<T> ctab[SH::CLDS ? SH::NCOEF : 1];
    const Item it = a.items[blockIdx.x];
    const int ns = min(a.nsteps, it.steps - a.sub);
    if (ns <= 0) return;
    const Geo& g = a.g;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t nstep = it.ctrl->step;
    const int hp0 = it.ctrl->have_prev;
    cx<T>* const gpre[2] = {reinterpret_cast<cx<T>*>(it.pre0), reinterpret_cast<cx<T>*>(it.pre1)};
    for (int i = tid; i < N0 * KC; i += SH::THREADS) {
#pragma unroll
        for (int u = 0; u < SH::LINES; u++) pre[u][i / KC * PC + i % KC] = gpre[u][i / KC * g.pitch + i % KC];
    }

    // column threads: column col, bins t + q N0/8; bins q = 3, 4 hold no stored mode
    const int cc = lane % CPW, t = lane / CPW, col = wave * CPW + cc;
    const bool cv = wave < SH::CW && col < KC;
    auto stored = [&](int q, int tt) {
        return q == 2 ? tt + 2 * TPL0 <= K0 : (q == 5 ? tt + 5 * TPL0 >= N0 - K0 : q != 3 && q != 4);
    };
    // stored entry u = 0..5 of bins 0, 1, 2, 5, 6, 7
    auto bin = [](int u) { return u < 3 ? u : u + 2; };
    auto sidx = [&](int u) { return (t + bin(u) * TPL0 - (u < 3 ? 0 : N0 - KEPT0)) * g.pitch + col; };
    cx<T>* const phi = reinterpret_cast<cx<T>*>(it.phi);
    cx<T>* const prev = reinterpret_cast<cx<T>*>(it.prev);
    cx<T> ph[6], pv[LEAN ? 1 : 6];   // LEAN: the carry in ph
    T4<T> cf[SH::CREG ? 6 : 1];
    const T4<T>* const gcoef = reinterpret_cast<const T4<T>*>(it.coef);   // rows |a0|
    if constexpr (SH::CLDS)
        for (int i = tid; i < SH::NCOEF; i += SH::THREADS) ctab[i] = gcoef[i / KC * g.pitch + i % KC];
    auto arow = [&](int u) { return u < 3 ? t + u * TPL0 : N0 - (t + (u + 2) * TPL0); };   // |a0|
#pragma unroll
    for (int u = 0; u < 6; u++) {
        const bool sv = cv && stored(bin(u), t);
        ph[u] = czero<T>();
        if constexpr (!LEAN) pv[u] = czero<T>();
        if constexpr (SH::CREG) cf[u] = {T(0), T(0), T(0), T(0)};
        if (sv) {
            ph[u] = LEAN ? prev[sidx(u)] : phi[sidx(u)];
            if constexpr (!LEAN) {
                if (it.order == 2) pv[u] = prev[sidx(u)];
            }
            if constexpr (SH::CREG) cf[u] = gcoef[arow(u) * g.pitch + col];
        }
    }
    const T dk0 = (T)it.dk[0], dk1 = (T)it.dk[1];
    const T P0 = nl_pref<T>(it, T(0)).x, P2 = nl_pref<T>(it, T(1)).x - P0;
    const T inv = (T)it.inv_vol;

    // noise of step index n, round h of the tasks, into buffer b: a task is one
    // Philox block for bins k and 7 - k of a column thread (a second one where
    // a Hermitian partner draws for one of them)
    auto draw = [&](uint32_t n, int b, int h) {
        constexpr int FIRST = SH::NW * 64 < SH::TASKS ? SH::NW * 64 : SH::TASKS;
        const int i = h ? FIRST + (wave - SH::CW) * 64 + lane : (wave - FW) * 64 + lane;
        if (i >= (h ? SH::TASKS : FIRST)) return;
        const int k = i / (TPL0 * KC), w = i % (TPL0 * KC), tt = w / KC, cl = w % KC;
        const NoiseSlot sa = noise_slot(g, tt + k * TPL0, 0, cl), sb = noise_slot(g, tt + (7 - k) * TPL0, 0, cl);
        uint32_t x[4];
        philox_block(it.seed, sa.P, n, it.r, 0u, x);
        cx<T> ea = eta_of<T>(x, sa);
        if (sb.P != sa.P) philox_block(it.seed, sb.P, n, it.r, 0u, x);
        cx<T> eb = eta_of<T>(x, sb);
        if (!stored(k, tt)) ea = czero<T>();
        if (!stored(7 - k, tt)) eb = czero<T>();
        const int id = cl / CPW * 64 + tt * CPW + cl % CPW;
        eta[b][k][id] = ea;
        eta[b][5 - k][id] = eb;
    };
    const uint32_t n0 = (uint32_t)(nstep + (LEAN ? 1 : 0));   // the carry holds the next step's noise
    if (wave >= FW) draw(n0, 0, 0);
    if (wave >= SH::CW) draw(n0, 0, 1);
    // row threads: rows 2 pr, 2 pr + 1, bins tr + q N1/8
    const int tr = lane % TPL1, pr = wave * (64 / TPL1) + lane / TPL1;
    LineTw<T, N0> tw0;
    LineTw<T, N1> tw1;
    line_tw_load(tw0, t, twid<T>(it.tw0));
    line_tw_load(tw1, tr, twid<T>(it.tw1));
    T nfacc = T(0);
    __syncthreads();

#pragma unroll 1
    for (int s = 0; s < ns; s++) {
        if (wave >= FW) {
            if (s + 1 < ns) draw(n0 + (uint32_t)(s + 1), (s + 1) & 1, 0);
        } else if (wave < SH::RW) {
            cx<T>* const ra[2] = {&pre[0][2 * pr * PC], &pre[SH::LINES - 1][2 * pr * PC]};
            cx<T>* const L = X + pr * SH::LINES * lds_len<N1, PAD>();
            cx<T> v[1][8];
            // stored column of bin q (its mirror above N1/2) and whether there is one
            auto column = [&](int q) { return q <= 2 ? tr + q * TPL1 : N1 - (tr + q * TPL1); };
            auto has = [&](int q) { return q != 3 && q != 4 && (q < 2 || q > 5 || column(q) <= K1); };
            if constexpr (KPZ) {
                // per row d0 h + i d1 h (pre1 holds the inverse of i k0 h)
                cx<T> w[2][8];
#pragma unroll
                for (int r = 0; r < 2; r++) {
#pragma unroll
                    for (int q = 0; q < 8; q++) {
                        w[r][q] = czero<T>();
                        if (!has(q)) continue;
                        const int k = column(q);
                        const cx<T> h = ra[0][r * PC + k], d = ra[1][r * PC + k];
                        const T kk = dk1 * (T)k;
                        cx<T> A = d, B = {-kk * h.y, kk * h.x};
                        if (q == 0 && tr == 0) A.y = B.y = T(0);
                        w[r][q] = q <= 2 ? cx<T>{A.x - B.y, A.y + B.x} : cx<T>{A.x + B.y, B.x - A.y};
                    }
                }
                fft_lines<T, N1, +1, PAD, 2, true>(w, tr, L, 2, 1, tw1);
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    const T x0 = w[0][q].x * inv, y0 = w[0][q].y * inv, x1 = w[1][q].x * inv, y1 = w[1][q].y * inv;
                    v[0][q] = {x0 * x0 + y0 * y0, x1 * x1 + y1 * y1};
                }
            } else {
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    v[0][q] = czero<T>();
                    if (!has(q)) continue;
                    cx<T> A = ra[0][column(q)], B = ra[0][PC + column(q)];
                    if (q == 0 && tr == 0) A.y = B.y = T(0);
                    v[0][q] = q <= 2 ? cx<T>{A.x - B.y, A.y + B.x} : cx<T>{A.x + B.y, B.x - A.y};
                }
                fft_lines<T, N1, +1, PAD, 1, true>(v, tr, L, 1, 0, tw1);
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    const T x = v[0][q].x * inv, y = v[0][q].y * inv;
                    v[0][q] = {x * x * x, y * y * y};
                }
            }
            fft_lines<T, N1, -1, PAD, 1, true>(v, tr, L, 1, 0, tw1);
            exchange_sync<true>();
#pragma unroll
            for (int q = 0; q < 8; q++)
                if (q != 3 && q != 4) L[lds_slot<PAD>(tr + q * TPL1)] = v[0][q];
            exchange_sync<true>();
#pragma unroll
            for (int q = 0; q < 3; q++) {
                const int k = tr + q * TPL1;
                if (k > K1) continue;
                const cx<T> Zk = L[lds_slot<PAD>(k)], Zm = L[lds_slot<PAD>((N1 - k) & (N1 - 1))];
                ra[0][k] = {T(0.5) * (Zk.x + Zm.x), T(0.5) * (Zk.y - Zm.y)};
                ra[0][PC + k] = {T(0.5) * (Zk.y + Zm.y), T(0.5) * (Zm.x - Zk.x)};
            }
        }
        __syncthreads();
        if (wave >= SH::CW) {
            if (s + 1 < ns) draw(n0 + (uint32_t)(s + 1), (s + 1) & 1, 1);
        } else {
            const int cl = col < KC ? col : KC - 1;   // lanes past the last column repeat it and write nothing
            cx<T>* const L = X + wave * CPW * lds_len<N0, PAD>() + cc;
            const bool hp = s > 0 || hp0;
            cx<T> v[1][8];
#pragma unroll
            for (int q = 0; q < 8; q++) v[0][q] = pre[0][(t + q * TPL0) * PC + cl];
            fft_lines<T, N0, -1, PAD, 1, true>(v, t, L, CPW, 0, tw0);
            v[0][3] = v[0][4] = czero<T>();
            const T k1 = dk1 * (T)col;
#pragma unroll
            for (int u = 0; u < 6; u++) {
                const int q = bin(u);
                const T k0 = dk0 * (T)sgn_idx(t + q * TPL0, N0);
                const cx<T> F = (P0 + ksq(k0, T(0), k1) * P2) * v[0][q];
                const cx<T> e = eta[s & 1][u][wave * 64 + lane];
                const bool sv = cv && stored(q, t);
                T4<T> c;   // E, w_a, w_b, G
                if constexpr (SH::CREG) c = cf[u];
                else if constexpr (SH::CLDS) c = ctab[sv ? arow(u) * KC + col : 0];
                else c = gcoef[sv ? arow(u) * g.pitch + col : 0];
                cx<T> nw;
                if constexpr (LEAN) {
                    // phi_{n+1} = Y_n + w F_n, Y_{n+1} = E phi_{n+1} + w_b F_n + G eta_{n+1}
                    nw = ph[u] + (hp ? c.b : c.b + c.c) * F;
                    ph[u] = c.a * nw + c.c * F + c.d * e;
                } else {
                    // (contracted as in k_axis0r)
                    nw = fma_cx(c.d, e, fma_cx(c.a, ph[u], c.b * F));
                    if (it.order == 2) nw = fma_cx(c.c, hp ? pv[u] : F, nw);
                    pv[u] = F;
                    ph[u] = nw;
                }
                v[0][q] = sv ? nw : czero<T>();
                nfacc += (v[0][q].x - v[0][q].x) + (v[0][q].y - v[0][q].y);
            }
            // column a_last = 0 Hermitian: rows j and N0 - j, the lower one
            // independent (column 1's exchange slots hold the carry)
            if (wave == 0) {
                exchange_sync<true>();
                if (cc == 0) {
#pragma unroll
                    for (int u = 0; u < 3; u++) {
                        if (!stored(u, t)) continue;
                        const int sl = lds_slot<PAD>(t + u * TPL0) * CPW;
                        L[sl] = v[0][u];
                        if constexpr (LEAN) L[sl + 1] = ph[u];
                    }
                }
                exchange_sync<true>();
                if (cc == 0) {
#pragma unroll
                    for (int u = 3; u < 6; u++) {
                        const int q = u + 2;
                        if (!stored(q, t)) continue;
                        const int sl = lds_slot<PAD>(N0 - (t + q * TPL0)) * CPW;
                        const cx<T> p = L[sl];
                        v[0][q] = {p.x, -p.y};
                        if constexpr (LEAN) {
                            const cx<T> y = L[sl + 1];
                            ph[u] = {y.x, -y.y};
                        } else {
                            ph[u] = v[0][q];
                        }
                    }
                    if (t == 0) {
                        v[0][0].y = T(0);
                        ph[0].y = T(0);
                    }
                }
            }
            if (a.rec.slot && cv) {
                cx<T>* const smp = reinterpret_cast<cx<T>*>((char*)it.phi + a.rec.first + s * a.rec.slot);
#pragma unroll
                for (int u = 0; u < 6; u++)
                    if (stored(bin(u), t)) smp[sidx(u)] = v[0][bin(u)];
            }
            cx<T> v2[1][8];
            if constexpr (KPZ) {
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    const T kk = dk0 * (T)sgn_idx(t + q * TPL0, N0);
                    v2[0][q] = {-kk * v[0][q].y, kk * v[0][q].x};
                }
            }
            fft_lines<T, N0, +1, PAD, 1, true>(v, t, L, CPW, 0, tw0);
            if (cv) {
#pragma unroll
                for (int q = 0; q < 8; q++) pre[0][(t + q * TPL0) * PC + col] = v[0][q];
            }
            if constexpr (KPZ) {
                fft_lines<T, N0, +1, PAD, 1, true>(v2, t, L, CPW, 0, tw0);
                if (cv) {
#pragma unroll
                    for (int q = 0; q < 8; q++) pre[1][(t + q * TPL0) * PC + col] = v2[0][q];
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 6; u++) {
        if (cv && stored(bin(u), t)) {
            if constexpr (LEAN) {
                prev[sidx(u)] = ph[u];
            } else {
                phi[sidx(u)] = ph[u];
                if (it.order == 2) prev[sidx(u)] = pv[u];
            }
        }
    }
    for (int i = tid; i < N0 * KC; i += SH::THREADS) {
#pragma unroll
        for (int u = 0; u < SH::LINES; u++) gpre[u][i / KC * g.pitch + i % KC] = pre[u][i / KC * PC + i % KC];
    }
    if (!(nfacc == nfacc)) atomicOr(&it.ctrl->nonfinite, 1);
    // every thread has read the counters before the barriers above
    if (tid == 0) {
        it.ctrl->step = nstep + ns;
        it.ctrl->have_prev = 1;
    }
}

template <typename T, int N0, int N1>
static hipError_t launch_small_n(const Geo& g, const Item* items, int nitems, int sub, int nsteps, bool kpz, bool lean,
                                 const Record& rec, hipStream_t s)
{
    const SmallArgs a = {g, items, sub, nsteps, rec};
    const dim3 grid(nitems);
    const dim3 bk(SmallShape<T, N0, N1, true>::THREADS), bp(SmallShape<T, N0, N1, false>::THREADS);
    if (kpz && lean) hipLaunchKernelGGL((k_small2d<T, N0, N1, true, true>), grid, bk, 0, s, a);
    else if (kpz) hipLaunchKernelGGL((k_small2d<T, N0, N1, true, false>), grid, bk, 0, s, a);
    else if (lean) hipLaunchKernelGGL((k_small2d<T, N0, N1, false, true>), grid, bp, 0, s, a);
    else hipLaunchKernelGGL((k_small2d<T, N0, N1, false, false>), grid, bp, 0, s, a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_small2d(const Geo& g, const Item* items, int nitems, int sub, int nsteps, int nl, bool lean,
                          const Record& rec, hipStream_t s)
{
    const bool kpz = nl == NL_KPZ;
    if (!small2d_ok(g, nl) || nitems <= 0) return hipErrorInvalidValue;
    if (g.n[0] == 64 && g.n[1] == 64) return launch_small_n<T, 64, 64>(g, items, nitems, sub, nsteps, kpz, lean, rec, s);
    if (g.n[0] == 64) return launch_small_n<T, 64, 32>(g, items, nitems, sub, nsteps, kpz, lean, rec, s);
    if (g.n[1] == 64) return launch_small_n<T, 32, 64>(g, items, nitems, sub, nsteps, kpz, lean, rec, s);
    return launch_small_n<T, 32, 32>(g, items, nitems, sub, nsteps, kpz, lean, rec, s);
}

}  // namespace setd
