// setd_part3.hip -- the 3D step of complex fields in two passes over memory.
//
// The general 3D step moves the line buffer through four passes (axis-1
// inverse, rows, axis-1 forward, axis 0).  Here the axis-1 transform is split
// as N1 = RA x 32 and its two factors join the neighbouring passes, so that
// one array Z in the place of the line buffer is read and written twice per
// step (CGL 256^3 at 4 realizations: 2.71 -> 1.76 GB and 621 -> 428 us a
// step; 128^3 at 16: 298 -> 205 us, at 1: 38.4 -> 31.6 us).  With
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

// The step of k_ax01 for launches that leave the chip idle (fewer wavefronts
// than SIMDs): the same arithmetic in the same order, so the same bits, with
// the lines of a block taken side by side instead of in turn.  The block's
// threads take (n0, column) points for the DFTs of RA points over m and leave
// the kept lines in LDS; each wavefront then takes one line of CPW columns (64
// = CPW x N0/8 threads) through the axis-0 transform, the update and the
// inverse without a block barrier; and the points go back by the conjugate
// DFTs.  us per step against k_ax01's: 128^3 x 1 31.6 / 36.4, 64^3 x 4 17.6 /
// 21.0; with the chip filled it loses by its 16 to 32-byte segments of the
// carry: 128^3 x 4 55.6 / 53.6, x 16 225 / 205, 256^3 x 4 458 / 428.
template <int N0, int RA>
struct Ax01LdsShape {
    static constexpr int TPL = N0 / 8, CPW = 64 / TPL, N1 = 32 * RA;
    static constexpr int TILE = CPW > ZC ? CPW : ZC;
    // kept lines p of a block: at most 6 of 8 (p = 3, 4 never), 3 of 4 (p = 1 for
    // s <= 10, p = 2 for s >= 22), both of 2
    static constexpr int NL = RA == 8 ? 6 : (RA == 4 ? 3 : RA);
    static constexpr int LSTR = lds_len<N0, 3>() + 4;   // line pitch: columns on different banks
    static constexpr int TASKS = NL * (TILE / CPW);
    static constexpr int NW = TASKS < 8 ? TASKS : 8;
    static constexpr int THREADS = 64 * NW;
};

template <int N0, int RA>
__global__ void __launch_bounds__((Ax01LdsShape<N0, RA>::THREADS)) __attribute__((amdgpu_waves_per_eu(4)))
k_ax01_lds(Part3Args a)
{
    typedef float T;
    typedef Ax01LdsShape<N0, RA> SH;
    const unsigned lg = xcd_logical(blockIdx.x, gridDim.x);
    const int item = (int)(lg / (unsigned)a.per_item);
    const int blk = (int)(lg % (unsigned)a.per_item);
    const Item it = a.items[item];
    if (a.sub >= it.steps) return;
    constexpr int TPL = SH::TPL, CPW = SH::CPW, TILE = SH::TILE, N1 = SH::N1, PAD = 3;
    constexpr int K0 = (N0 - 1) / 3, KEPT0 = 2 * K0 + 1;
    constexpr uint32_t ES = sizeof(cx<T>);
    __shared__ cx<T> lines[SH::NL * TILE * SH::LSTR];
    const Geo& g = a.g;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int tile = blk % a.ntiles, s = blk / a.ntiles;
    const int keptl = g.kept[2], kept1 = g.kept[1];
    const uint32_t prow = (uint32_t)g.pitch * ES;   // one row of columns
    const rsrc_t rz = make_rsrc(it.big, (uint32_t)(N0 * N1) * prow);
    // stored index of line p, -1 where the 2/3 rule removes it, and the LDS
    // line it takes
    auto line_of = [&](int p) { return stored_idx(32 * p + s, N1, kept1, g.kp[1]); };
    auto slot_of = [](int p) { return RA == 8 ? (p < 3 ? p : p - 2) : (RA == 4 ? (p + 1) / 2 : p); };
    // e^{-2 pi i s m / N1}, the same in every lane
    cx<T> wm[RA];
#pragma unroll
    for (int m = 1; m < RA; m++) {
        const cx<T> w = gload<T>(it.tw1, (uint32_t)((s * m) & (N1 - 1)) * ES);
        wm[m] = {__uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(w.x))),
                 __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(w.y)))};
    }
    // point i of the tile: ZC columns of ZN neighbouring n0 (a 128-byte line),
    // the next n0, the next ZC columns
    constexpr int POINTS = N0 * TILE;
    auto point = [&](int i, int& n0, int& c) {
        c = i % ZC + i / (ZC * N0) * ZC;
        n0 = i / ZC % N0;
    };
    auto zpt = [&](int n0, int c) {
        return (uint32_t)(n0 / ZN * N1) * (ZN * prow) + z_col(tile * TILE + c) + (uint32_t)(n0 % ZN) * (ZC * ES);
    };
    auto zoff = [&](int m) { return (uint32_t)(m * 32 + s) * (ZN * prow); };
#pragma unroll 2
    for (int i = tid; i < POINTS; i += SH::THREADS) {
        int n0, c;
        point(i, n0, c);
        const uint32_t z = zpt(n0, c);
        cx<T> u[RA];
#pragma unroll
        for (int m = 0; m < RA; m++) u[m] = bload<T>(rz, z, zoff(m));
#pragma unroll
        for (int m = 1; m < RA; m++) u[m] = cmul(u[m], wm[m]);
        dft<RA, -1>(u);
        cx<T>* const dst = lines + c * SH::LSTR + lds_slot<PAD>(n0);
#pragma unroll
        for (int p = 0; p < RA; p++) {
            if (RA == 8 && (p == 3 || p == 4)) continue;
            if (line_of(p) >= 0) dst[slot_of(p) * TILE * SH::LSTR] = u[p];
        }
    }
    __syncthreads();

    const int cw = lane % CPW, t = lane / CPW;   // column within the wavefront's, bins t + q N0/8
    auto live = [](int q) { return q != 3 && q != 4; };
    auto stored = [&](int q) {
        if (q == 3 || q == 4) return false;
        if (q == 2) return t + 2 * TPL <= K0;
        if (q == 5) return t + 5 * TPL >= N0 - K0;
        return true;
    };
    // state arrays: row (i0, i1); bins q = 3, 4 hold no stored mode
    const uint32_t lstride = (uint32_t)kept1 * prow;
    const rsrc_t rst = make_rsrc(it.prev, (uint32_t)KEPT0 * lstride);
    const rsrc_t rcoef = make_rsrc(it.coef, it.coef_bytes);
    LineTw<T, N0> tw;
    line_tw_load(tw, t, twid<T>(it.tw0));
    // the row pass has begun the step; the carry holds the next step's noise
    const uint32_t nn = (uint32_t)*(const SETD_GLOBAL int64_t*)&it.ctrl->step;
    const bool hp = *(const SETD_GLOBAL int*)&it.ctrl->have_prev >= 2;
    const cx<T> pref = {T(-1), -(T)it.par0};
    T nfacc = T(0);
    // tasks: the columns of line p in groups of CPW
    constexpr int CG = TILE / CPW;
#pragma unroll 1
    for (int k = wave; k < SH::TASKS; k += SH::NW) {
        const int sl = k / CG;   // LDS line; for RA = 4 line 1 is p = 1 or 2
        const int p = RA == 8 ? (sl < 3 ? sl : sl + 2) : (RA == 4 && sl == 2 ? 3 : (RA == 4 && sl == 1 && s >= 16 ? 2 : sl));
        const int i1 = line_of(p);
        if (i1 < 0) continue;
        const int c = k % CG * CPW + cw, colm = tile * TILE + c;
        const bool cv = colm < keptl;
        const int j1 = 32 * p + s, a1 = sgn_idx(j1, N1);
        const int jl = fft_pos(colm, g.n[2], keptl, g.kp[2]), al = sgn_idx(jl, g.n[2]);
        const uint32_t vcol = cv ? (uint32_t)t * lstride + (uint32_t)colm * ES : BUF_OOB;
        auto voff = [&](int q) { return (q == 2 || q == 5) ? (stored(q) ? vcol : BUF_OOB) : vcol; };
        auto soff = [&](int q) {
            return (uint32_t)(q * TPL + (q <= 2 ? 0 : KEPT0 - N0)) * lstride + (uint32_t)i1 * prow;
        };
        cx<T>* const L = lines + (sl * TILE + c) * SH::LSTR;
        cx<T> v[1][8];
        cx<T> y0[8], eta[8];
        T4<T> ce[3][2];   // entries of |a0| = t + u N0/8: E, w_a, w_b, G
#pragma unroll
        for (int q = 0; q < 8; q++) y0[q] = live(q) ? bload<T>(rst, voff(q), soff(q)) : czero<T>();
#pragma unroll
        for (int u = 0; u < 3; u++) {
            const int m = t + u * TPL;
            const uint32_t vo = (cv && m <= K0) ? (uint32_t)coef_key(it, m, a1, al) * (uint32_t)(8 * sizeof(T)) : BUF_OOB;
            ce[u][0] = bload4<T>(rcoef, vo, 0u);
            ce[u][1] = bload4<T>(rcoef, vo, 16u);
        }
        // noise of bins u and 7 - u from one Philox block, while the loads are in flight
        const uint32_t S = (uint32_t)g.n[1] * (uint32_t)g.nh_last;
        const uint32_t rest = (uint32_t)j1 * (uint32_t)g.nh_last + (uint32_t)jl;
#pragma unroll
        for (int u = 0; u < 3; u++) {
            uint32_t x[4];
            philox_block(it.seed, (uint32_t)(t + u * TPL) * S + rest, nn, it.r, 0u, x);
            eta[u] = box_muller_cx(x[0], x[1], T(0));
            eta[7 - u] = box_muller_cx(x[2], x[3], T(0));
        }
#pragma unroll
        for (int q = 0; q < 8; q++) v[0][q] = L[lds_slot<PAD>(t + q * TPL)];
        fft_lines<T, N0, -1, PAD, 1, true>(v, t, L, 1, 0, tw);
        // bin 7 - u of thread t has |a0| = (u + 1) N0/8 - t: entry u of
        // thread N0/8 - t, or for t = 0 entry u + 1 of its own
        const int src = (((TPL - t) & (TPL - 1)) * CPW + cw) * 4;
        auto from = [&](T x) {
            return __uint_as_float((unsigned)__builtin_amdgcn_ds_bpermute(src, (int)__float_as_uint(x)));
        };
        auto update = [&](int q, const T4<T>& e0, const T4<T>& e1) {
            const bool sv = cv && stored(q);
            const cx<T> E = {e0.a, e0.b}, wa = {e0.c, e0.d}, wb = {e1.a, e1.b};
            const cx<T> F = cmul(pref, v[0][q]);
            // phi_{n+1} = Y_n + w F_n, Y_{n+1} = E phi_{n+1} + w_b F_n + G eta_{n+1}
            const cx<T> nw = y0[q] + cmul(hp ? wa : wa + wb, F);
            const cx<T> y = cmul(E, nw) + cmul(wb, F) + e1.c * eta[q];
            bstore<T>(rst, voff(q), soff(q), y);
            v[0][q] = sv ? nw : czero<T>();
            nfacc += (v[0][q].x - v[0][q].x) + (v[0][q].y - v[0][q].y);
        };
        v[0][3] = v[0][4] = czero<T>();
#pragma unroll
        for (int u = 0; u < 3; u++) {
            update(u, ce[u][0], ce[u][1]);
            const T4<T>&e0 = (t == 0 && u < 2) ? ce[u < 2 ? u + 1 : u][0] : ce[u][0],
                 &e1 = (t == 0 && u < 2) ? ce[u < 2 ? u + 1 : u][1] : ce[u][1];
            const T4<T> m0 = {from(e0.a), from(e0.b), from(e0.c), from(e0.d)};
            const T4<T> m1 = {from(e1.a), from(e1.b), from(e1.c), T(0)};
            update(7 - u, m0, m1);
        }
        fft_lines<T, N0, +1, PAD, 1, true>(v, t, L, 1, 0, tw);
        exchange_sync<true>();
#pragma unroll
        for (int q = 0; q < 8; q++) L[lds_slot<PAD>(t + q * TPL)] = v[0][q];
    }
    __syncthreads();
#pragma unroll 2
    for (int i = tid; i < POINTS; i += SH::THREADS) {
        int n0, c;
        point(i, n0, c);
        const uint32_t z = tile * TILE + c < keptl ? zpt(n0, c) : BUF_OOB;
        const cx<T>* const src = lines + c * SH::LSTR + lds_slot<PAD>(n0);
        cx<T> u[RA];
#pragma unroll
        for (int p = 0; p < RA; p++) {
            u[p] = czero<T>();
            if (RA == 8 && (p == 3 || p == 4)) continue;
            if (line_of(p) >= 0) u[p] = src[slot_of(p) * TILE * SH::LSTR];
        }
        dft<RA, +1>(u);
#pragma unroll
        for (int m = 0; m < RA; m++) bstore<T>(rz, z, zoff(m), m ? cmulc(u[m], wm[m]) : u[m]);
    }
    if (!(nfacc == nfacc)) atomicOr(&it.ctrl->nonfinite, 1);
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
    if constexpr (RA > 1) {
        // fewer wavefronts than the chip has SIMDs: the lines side by side
        // (with RA = 1 there is one line a block)
        if (mode == MODE_STEP && (long)a.per_item * nitems * (TILE * N0 / 8) <= 64L * 1024) {
            typedef Ax01LdsShape<N0, RA> SH;
            a.ntiles = g.pitch / SH::TILE;
            a.per_item = a.ntiles * 32;
            hipLaunchKernelGGL((k_ax01_lds<N0, RA>), dim3(a.per_item * nitems), dim3(SH::THREADS), 0, s, a);
            return hipGetLastError();
        }
    }
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
