// setd_part3.hip -- the 3D step of complex fields in two passes over memory.
//
// The general 3D step moves the line buffer through four passes (axis-1
// inverse, rows, axis-1 forward, axis 0).  Here the axis-1 transform is split
// as N1 = RA x 32 and its two factors join the neighbouring passes, so that
// one array Z in the place of the line buffer is read and written twice per
// step (CGL 256^3 at 4 realizations: 2.71 -> 1.76 GB and 621 -> 428 us a
// step; 128^3 at 16: 298 -> 205 us, at 1: 38.4 -> 36.4 us, where the two
// launches' own latency is what is left).  With
// a1 = 32 p + s and n1 = m + RA r (p, m < RA; s, r < 32)
//   Z[n0][m][s] = e^{2 pi i s m/N1} sum_p X[32 p + s] e^{2 pi i p m/RA}
//   x[n0][m + RA r] = sum_s Z[n0][m][s] e^{2 pi i s r/32}
// and the conjugate sums in the reverse order on the way back:
//   k_ax01:   a block owns one s and a tile of columns over all of axis 0.
//             Each thread's RA x 8 values of Z give the lines a1 = 32 p + s
//             by DFTs of RA points in registers; every kept line goes
//             through the axis-0 transform, the SETD2 update and the inverse
//             (as in k_axis0r), and the lines go back to Z.
//   k_rows32: a block owns the 32 rows of one (n0, m): 32-point DFTs down the
//             columns in registers, the rows through LDS to the nonlinearity
//             and back.
// Complex64 plans with the SETD2 carry, the
// 2/3 rule, Fourier-space noise and 32..256 points per axis (part3_ok):
// longer axes or FP64 would need more registers than two wavefronts per SIMD
// allow in k_ax01.
#include "setd_kernels.hpp"
#include "setd_launch.hpp"

namespace setd {

// cos(2 pi k / 32), sin(2 pi k / 32)
__device__ __forceinline__ constexpr float cos32(int k)
{
    constexpr float c[9] = {1.0f, 0.98078528040323044913f, 0.92387953251128675613f, 0.83146961230254523708f,
                            0.70710678118654752440f, 0.55557023301960222474f, 0.38268343236508977173f,
                            0.19509032201612826785f, 0.0f};
    k &= 31;
    if (k > 16) k = 32 - k;
    return k <= 8 ? c[k] : -c[16 - k];
}
__device__ __forceinline__ constexpr float sin32(int k) { return cos32(k - 8); }

// X_r = sum_s v_s e^{SIGN 2 pi i s r / 32} as 4 x 8; X_{c + 4d} ends in v[8c + d]
template <int SIGN>
__device__ __forceinline__ void dft32(cx<float> (&v)[32])
{
#pragma unroll
    for (int b = 0; b < 8; b++) dft4s<SIGN, 8>(v + b);
#pragma unroll
    for (int c = 1; c < 4; c++) {
#pragma unroll
        for (int b = 1; b < 8; b++) {
            const int k = b * c;
            const cx<float> u = v[8 * c + b];
            if (k % 8 == 0) {
                v[8 * c + b] = (k == 8) ? mul_si<SIGN>(u) : cx<float>{-u.x, -u.y};
            } else {
                const cx<float> w = {cos32(k), SIGN * sin32(k)};
                v[8 * c + b] = cmul(u, w);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 4; c++) dft8<SIGN>(v + 8 * c);
}

// Z is stored [n0/2][m][s][column/8][n0 mod 2][column mod 8]: a tile of eight
// columns in k_ax01 reads whole 128-byte lines (two neighbouring n0), the rows
// of k_rows32 64-byte halves of lines whose other half the next block reads.
// CGL 256^3 x 4, k_ax01 / k_rows32: 280 / 167 us; with four columns and four
// n0 to a line 292 / 178 us; with plain rows of columns 329 / 165 us at tiles
// of 8 columns and 482 us at 4.
constexpr int ZC = 8, ZN = 16 / ZC;   // columns and n0 values of a 128-byte line
__device__ __forceinline__ uint32_t z_col(int col) { return (uint32_t)(col / ZC) * 128u + (uint32_t)(col % ZC) * 8u; }

struct Part3Args {
    Geo g;
    const Item* items;
    int ntiles;     // k_ax01: column tiles of the padded last axis
    int per_item;   // blocks per realization
    int sub;
};

// ---------------------------------------------------------------- axis 0 with the outer factor of axis 1
// Bound by how much of its traffic two wavefronts per SIMD keep in flight (the
// RA x 8 values of a thread and its six lines take the registers): CGL 256^3
// x 4 moves 1.04 GB in 280 us with about 150 us of VALU issue.
// MODE_STEP:    Z -> lines -> update of the carry -> Z.
// MODE_SYNC:    phi -> Z (after phi was set).
// MODE_RECOVER: Z -> phi (the carry storage keeps no phi between steps).
template <int N0, int TILE, int RA, int MODE>
__global__ void __launch_bounds__(TILE * N0 / 8) __attribute__((amdgpu_waves_per_eu(2)))
k_ax01(Part3Args a)
{
    typedef float T;
    const unsigned lg = xcd_logical(blockIdx.x, gridDim.x);
    const int item = (int)(lg / (unsigned)a.per_item);
    const int blk = (int)(lg % (unsigned)a.per_item);
    const Item it = a.items[item];
    if (MODE == MODE_STEP && a.sub >= it.steps) return;
    constexpr int TPL = N0 / 8, PAD = 3, N1 = 32 * RA, NTHR = TILE * TPL;
    constexpr int K0 = (N0 - 1) / 3;
    constexpr uint32_t ES = sizeof(cx<T>);
    __shared__ cx<T> lds[TILE * lds_len<N0, PAD>()];
    // coefficient entries of |a0| <= K0 for the tile's columns, re-staged per line
    __shared__ T4<T> ctab[MODE == MODE_STEP ? (K0 + 1) * TILE * 2 : 1];
    const Geo& g = a.g;
    const int tid = threadIdx.x;
    const int c0 = tid % TILE, t = tid / TILE;
    const int tile = blk % a.ntiles, s = blk / a.ntiles;
    const int keptl = g.kept[2], kept1 = g.kept[1];
    constexpr int kept0 = 2 * K0 + 1;
    const int colm = tile * TILE + c0;
    const bool cv = colm < keptl;
    const uint32_t prow = (uint32_t)g.pitch * ES;   // one row of columns
    const rsrc_t rz = make_rsrc(it.big, (uint32_t)(N0 * N1) * prow);
    const uint32_t zrow = (uint32_t)(t / ZN) * (uint32_t)N1 * (ZN * prow) + z_col(colm) + (uint32_t)(t % ZN) * (ZC * ES);
    const uint32_t zcol = cv ? zrow : BUF_OOB;
    auto zoff = [&](int q, int m) { return (uint32_t)(q * TPL / ZN * N1 + m * 32 + s) * (ZN * prow); };
    // state arrays: row (i0, i1); bins q = 3, 4 hold no stored mode
    const uint32_t lstride = (uint32_t)kept1 * prow;
    const rsrc_t rst = make_rsrc(MODE == MODE_STEP ? it.prev : it.phi, (uint32_t)kept0 * lstride);
    auto live = [](int q) { return q != 3 && q != 4; };
    auto stored = [&](int q) {
        if (q == 3 || q == 4) return false;
        if (q == 2) return t + 2 * TPL <= K0;
        if (q == 5) return t + 5 * TPL >= N0 - K0;
        return true;
    };
    const uint32_t vcol = cv ? (uint32_t)t * lstride + (uint32_t)colm * ES : BUF_OOB;
    auto voff = [&](int q) { return (q == 2 || q == 5) ? (stored(q) ? vcol : BUF_OOB) : vcol; };
    auto soff = [&](int q, int i1) {
        return (uint32_t)(q * TPL + (q <= 2 ? 0 : kept0 - N0)) * lstride + (uint32_t)i1 * prow;
    };
    const int jl = fft_pos(colm, g.n[2], keptl, g.kp[2]);
    const int al = sgn_idx(jl, g.n[2]);
    LineTw<T, N0> tw;
    line_tw_load(tw, t, twid<T>(it.tw0));
    cx<T>* const L = lds + c0;
    // e^{-2 pi i s m / N1}, the same in every lane
    cx<T> wm[RA];
#pragma unroll
    for (int m = 1; m < RA; m++) {
        const cx<T> w = gload<T>(it.tw1, (uint32_t)((s * m) & (N1 - 1)) * ES);
        wm[m] = {__uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(w.x))),
                 __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(w.y)))};
    }
    // stored index of line p, -1 where the 2/3 rule removes it
    auto line_of = [&](int p) { return stored_idx(32 * p + s, N1, kept1, g.kp[1]); };

    cx<T> st[RA][8];
    if constexpr (MODE != MODE_SYNC) {
#pragma unroll
        for (int q = 0; q < 8; q++) {
#pragma unroll
            for (int m = 0; m < RA; m++) st[m][q] = bload<T>(rz, zrow, zoff(q, m));
        }
#pragma unroll
        for (int q = 0; q < 8; q++) {
            cx<T> u[RA];
#pragma unroll
            for (int m = 0; m < RA; m++) u[m] = m ? cmul(st[m][q], wm[m]) : st[m][q];
            if constexpr (RA > 1) dft<RA, -1>(u);
#pragma unroll
            for (int m = 0; m < RA; m++) st[m][q] = u[m];
        }
    }
    int64_t nstep = 0;
    int hp = 0;
    if constexpr (MODE == MODE_STEP) {
        // the row pass has begun the step
        nstep = *(const SETD_GLOBAL int64_t*)&it.ctrl->step - 1;
        hp = *(const SETD_GLOBAL int*)&it.ctrl->have_prev >= 2;
    }
    const uint32_t nn = (uint32_t)(nstep + 1);   // the carry holds the next step's noise
    const rsrc_t rcoef = make_rsrc(it.coef, it.coef_bytes);
    const uint32_t S = (uint32_t)g.n[1] * (uint32_t)g.nh_last;
    const cx<T> pref = {T(-1), -(T)it.par0};
    T nfacc = T(0);

#pragma unroll 1
    for (int pi = 0; pi < RA; pi++) {
        const int i1 = line_of(pi);
        if (i1 < 0) continue;
        const int j1 = 32 * pi + s, a1 = sgn_idx(j1, N1);
        cx<T> v[1][8];
        if constexpr (MODE == MODE_SYNC) {
#pragma unroll
            for (int q = 0; q < 8; q++) v[0][q] = live(q) ? bload<T>(rst, voff(q), soff(q, i1)) : czero<T>();
        } else {
#pragma unroll
            for (int p = 0; p < RA; p++) {
                if (RA == 8 && (p == 3 || p == 4)) continue;
                if (p == pi) {
#pragma unroll
                    for (int q = 0; q < 8; q++) v[0][q] = st[p][q];
                }
            }
        }
        if constexpr (MODE == MODE_STEP) {
            cx<T> y0[8], eta[8];
#pragma unroll
            for (int q = 0; q < 8; q++) y0[q] = live(q) ? bload<T>(rst, voff(q), soff(q, i1)) : czero<T>();
            // this line's coefficients, each gathered once (a0 and -a0 share one)
            constexpr int NG = ((K0 + 1) * TILE + NTHR - 1) / NTHR;
            T4<T> cg[NG][2];
#pragma unroll
            for (int u = 0; u < NG; u++) {
                const int e = tid + u * NTHR;
                const int col = tile * TILE + e % TILE;
                const int key = coef_key(it, e / TILE, a1, sgn_idx(fft_pos(col, g.n[2], keptl, g.kp[2]), g.n[2]));
                const uint32_t vo = (e < (K0 + 1) * TILE && col < keptl) ? (uint32_t)key * (uint32_t)(8 * sizeof(T)) : BUF_OOB;
                cg[u][0] = bload4<T>(rcoef, vo, 0u);
                cg[u][1] = bload4<T>(rcoef, vo, 16u);
            }
            // noise of bins k and 7 - k from one Philox block, while the loads are in flight
            const uint32_t rest = (uint32_t)j1 * (uint32_t)g.nh_last + (uint32_t)jl;
#pragma unroll
            for (int k = 0; k < 3; k++) {
                uint32_t x[4];
                philox_block(it.seed, (uint32_t)(t + k * TPL) * S + rest, nn, it.r, 0u, x);
                eta[k] = box_muller_cx(x[0], x[1], T(0));
                eta[7 - k] = box_muller_cx(x[2], x[3], T(0));
            }
            // (the previous line's entries were last read before the barriers
            // of its inverse transform)
#pragma unroll
            for (int u = 0; u < NG; u++) {
                const int e = tid + u * NTHR;
                if (e < (K0 + 1) * TILE) {
                    ctab[2 * e] = cg[u][0];
                    ctab[2 * e + 1] = cg[u][1];
                }
            }
            fft_lines<T, N0, -1, PAD, 1>(v, t, L, TILE, 0, tw);
#pragma unroll
            for (int q = 0; q < 8; q++) {
                if (!live(q)) {
                    v[0][q] = czero<T>();
                    continue;
                }
                const bool sv = cv && stored(q);
                const int a0 = sgn_idx(t + q * TPL, N0);
                const int m = sv ? (a0 < 0 ? -a0 : a0) : 0;
                const T4<T> u = ctab[(m * TILE + c0) * 2], w = ctab[(m * TILE + c0) * 2 + 1];
                const cx<T> E = {u.a, u.b}, wa = {u.c, u.d}, wb = {w.a, w.b};
                const cx<T> F = cmul(pref, v[0][q]);
                // phi_{n+1} = Y_n + w F_n, Y_{n+1} = E phi_{n+1} + w_b F_n + G eta_{n+1}
                const cx<T> nw = y0[q] + cmul(hp ? wa : wa + wb, F);
                const cx<T> y = cmul(E, nw) + cmul(wb, F) + w.c * eta[q];
                bstore<T>(rst, voff(q), soff(q, i1), y);
                v[0][q] = sv ? nw : czero<T>();
                nfacc += (v[0][q].x - v[0][q].x) + (v[0][q].y - v[0][q].y);
            }
        } else if constexpr (MODE == MODE_RECOVER) {
            fft_lines<T, N0, -1, PAD, 1>(v, t, L, TILE, 0, tw);
#pragma unroll
            for (int q = 0; q < 8; q++)
                if (live(q)) bstore<T>(rst, voff(q), soff(q, i1), (T(1) / T(N0 * RA)) * v[0][q]);
            continue;
        }
        fft_lines<T, N0, +1, PAD, 1>(v, t, L, TILE, 0, tw);
#pragma unroll
        for (int p = 0; p < RA; p++) {
            if (RA == 8 && (p == 3 || p == 4)) continue;
            if (p == pi) {
#pragma unroll
                for (int q = 0; q < 8; q++) st[p][q] = v[0][q];
            }
        }
    }
    if constexpr (MODE == MODE_RECOVER) return;
#pragma unroll
    for (int p = 0; p < RA; p++) {
        if ((RA == 8 && (p == 3 || p == 4)) || line_of(p) < 0) {
#pragma unroll
            for (int q = 0; q < 8; q++) st[p][q] = czero<T>();
        }
    }
#pragma unroll
    for (int q = 0; q < 8; q++) {
        cx<T> u[RA];
#pragma unroll
        for (int p = 0; p < RA; p++) u[p] = st[p][q];
        if constexpr (RA > 1) dft<RA, +1>(u);
#pragma unroll
        for (int m = 0; m < RA; m++) bstore<T>(rz, zcol, zoff(q, m), m ? cmulc(u[m], wm[m]) : u[m]);
    }
    if constexpr (MODE == MODE_STEP) {
        const bool bad = !(nfacc == nfacc);
        if (__syncthreads_or(bad) && tid == 0) atomicOr(&it.ctrl->nonfinite, 1);
    }
}

// ---------------------------------------------------------------- rows with the inner factor of axis 1
// Bound by VALU issue (2,540 instructions per wavefront, 135 of 167 us at CGL
// 256^3 x 4; 0.72 GB moved once).  A row's transform stays within a wavefront,
// so only the four turns between rows and columns take block barriers.
template <int N2>
constexpr int rows32_threads() { return N2 < 64 ? 64 : N2; }

template <int N2>
__global__ void __launch_bounds__(rows32_threads<N2>()) __attribute__((amdgpu_waves_per_eu(3)))
k_rows32(Part3Args a)
{
    typedef float T;
    const unsigned lg = xcd_logical(blockIdx.x, gridDim.x);
    const int item = (int)(lg / (unsigned)a.per_item);
    const int blk = (int)(lg % (unsigned)a.per_item);
    const Item it = a.items[item];
    if (a.sub >= it.steps) return;
    if (blk == 0 && threadIdx.x == 0) begin_step(it.ctrl);
    constexpr int NT = rows32_threads<N2>(), TPL = N2 / 8, PAD = 3;
    constexpr int K = (N2 - 1) / 3, KL = 2 * K + 1;      // stored columns
    constexpr int G = NT / TPL, NP = 32 / G;             // rows at a time, rounds
    constexpr int XL = G * 2 * lds_len<N2, PAD>();       // exchange slots: two rows per thread group
    constexpr uint32_t ES = sizeof(cx<T>);
    // the 32 rows (stored columns only); between the row loads and stores the
    // transforms use the same space for their exchanges
    __shared__ cx<T> lds[32 * KL > XL ? 32 * KL : XL];
    const Geo& g = a.g;
    const int tid = threadIdx.x;
    const uint32_t prow = (uint32_t)g.pitch * ES;
    // blk = ((n0/2) RA + m) 2 + n0 mod 2
    const rsrc_t rz = make_rsrc(reinterpret_cast<char*>(it.big) + (size_t)(blk / ZN) * (32 * ZN) * prow, 32u * ZN * prow);
    const uint32_t vc = tid < KL ? z_col(tid) + (uint32_t)(blk % ZN) * (ZC * ES) : BUF_OOB;
    const int l = tid / TPL, t = tid - l * TPL;
    LineTw<T, N2> tw;
    line_tw_load(tw, t, twid<T>(it.tw2));
    {
        cx<T> z[32];
#pragma unroll
        for (int s = 0; s < 32; s++) z[s] = bload<T>(rz, vc, (uint32_t)s * (ZN * prow));
        dft32<+1>(z);
        if (tid < KL) {
#pragma unroll
            for (int c = 0; c < 4; c++) {
#pragma unroll
                for (int d = 0; d < 8; d++) lds[(c + 4 * d) * KL + tid] = z[8 * c + d];
            }
        }
    }
    __syncthreads();
    const T inv = (T)it.inv_vol;
    // stored column of bin t + q N2/8 (q = 3, 4 none), -1 where removed
    auto col_of = [&](int q) {
        const int k = t + q * TPL;
        if (q <= 1) return k;
        if (q >= 6) return k - N2 + KL;
        if (q == 2) return k <= K ? k : -1;
        if (q == 5) return k >= N2 - K ? k - N2 + KL : -1;
        return -1;
    };
    cx<T> w[NP][8];
#pragma unroll
    for (int k = 0; k < NP; k++) {
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const int c = col_of(q);
            w[k][q] = czero<T>();
            if (q != 3 && q != 4 && c >= 0) w[k][q] = lds[(l + k * G) * KL + c];
        }
    }
    __syncthreads();
    cx<T>* const X = lds + l * 2 * lds_len<N2, PAD>();
#pragma unroll
    for (int k = 0; k < NP; k += 2) {
        cx<T>(&u)[2][8] = reinterpret_cast<cx<T>(&)[2][8]>(w[k]);
        fft_lines<T, N2, +1, PAD, 2, true>(u, t, X, 2, 1, tw);
        // |A|^2 A in real space (CGL)
#pragma unroll
        for (int i = 0; i < 2; i++) {
#pragma unroll
            for (int q = 0; q < 8; q++) {
                const T x = u[i][q].x * inv, y = u[i][q].y * inv;
                const T m = x * x + y * y;
                u[i][q] = {m * x, m * y};
            }
        }
        fft_lines<T, N2, -1, PAD, 2, true>(u, t, X, 2, 1, tw);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NP; k++) {
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const int c = col_of(q);
            if (q != 3 && q != 4 && c >= 0) lds[(l + k * G) * KL + c] = w[k][q];
        }
    }
    __syncthreads();
    {
        cx<T> z[32];
#pragma unroll
        for (int r = 0; r < 32; r++) z[r] = lds[r * KL + (tid < KL ? tid : 0)];
        dft32<-1>(z);
#pragma unroll
        for (int c = 0; c < 4; c++) {
#pragma unroll
            for (int d = 0; d < 8; d++) bstore<T>(rz, vc, (uint32_t)(c + 4 * d) * (ZN * prow), z[8 * c + d]);
        }
    }
}

// ---------------------------------------------------------------- launches
template <int N0, int RA>
static hipError_t launch_ax01(const Geo& g, const Item* items, int nitems, int mode, int sub, hipStream_t s)
{
    // more columns on short axes, to fill a wavefront
    constexpr int TILE = N0 >= 512 / ZC ? ZC : 512 / N0;
    Part3Args a;
    a.g = g;
    a.items = items;
    a.ntiles = g.pitch / TILE;
    a.per_item = a.ntiles * 32;
    a.sub = sub;
    const dim3 grid(a.per_item * nitems), block(TILE * N0 / 8);
    if (mode == MODE_STEP) hipLaunchKernelGGL((k_ax01<N0, TILE, RA, MODE_STEP>), grid, block, 0, s, a);
    else if (mode == MODE_SYNC) hipLaunchKernelGGL((k_ax01<N0, TILE, RA, MODE_SYNC>), grid, block, 0, s, a);
    else if (mode == MODE_RECOVER) hipLaunchKernelGGL((k_ax01<N0, TILE, RA, MODE_RECOVER>), grid, block, 0, s, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int N0>
static hipError_t launch_ax01_n(const Geo& g, const Item* items, int nitems, int mode, int sub, hipStream_t s)
{
    switch (g.n[1]) {
    case 32: return launch_ax01<N0, 1>(g, items, nitems, mode, sub, s);
    case 64: return launch_ax01<N0, 2>(g, items, nitems, mode, sub, s);
    case 128: return launch_ax01<N0, 4>(g, items, nitems, mode, sub, s);
    case 256: return launch_ax01<N0, 8>(g, items, nitems, mode, sub, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_part3_axis0(const Geo& g, const Item* items, int nitems, int mode, int sub, hipStream_t s)
{
    switch (g.n[0]) {
    case 32: return launch_ax01_n<32>(g, items, nitems, mode, sub, s);
    case 64: return launch_ax01_n<64>(g, items, nitems, mode, sub, s);
    case 128: return launch_ax01_n<128>(g, items, nitems, mode, sub, s);
    case 256: return launch_ax01_n<256>(g, items, nitems, mode, sub, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_part3_rows(const Geo& g, const Item* items, int nitems, int sub, hipStream_t s)
{
    Part3Args a;
    a.g = g;
    a.items = items;
    a.ntiles = 0;
    a.per_item = g.n[0] * (g.n[1] / 32);
    a.sub = sub;
    const dim3 grid(a.per_item * nitems);
    switch (g.n[2]) {
    case 32: hipLaunchKernelGGL((k_rows32<32>), grid, dim3(rows32_threads<32>()), 0, s, a); break;
    case 64: hipLaunchKernelGGL((k_rows32<64>), grid, dim3(rows32_threads<64>()), 0, s, a); break;
    case 128: hipLaunchKernelGGL((k_rows32<128>), grid, dim3(rows32_threads<128>()), 0, s, a); break;
    case 256: hipLaunchKernelGGL((k_rows32<256>), grid, dim3(rows32_threads<256>()), 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace setd
