// henry_wave.hpp -- the V-cycle of the levels of at most 512 cells, run by
// one wavefront (included by henry_device.hpp, inside its namespace).
//
// What bounds it: a chain of about ninety dependent phases per pair of
// cycles (half-sweeps, line solves, transfers, on 32x16 and the levels below
// it) with at most eight cells per lane in each, so the chain's length is
// the instructions and LDS round trips of one phase.  Everything that does
// not depend on the state is therefore a compile-time constant: one
// instantiation per level width, the neighbours of a lane's cells at
// immediate offsets of one LDS address, halo cells that hold zero instead of
// clamped indices and selects, couplings and reciprocal diagonals formed once
// per cycle and kept in registers, cyclic reduction through DPP lane shifts
// (a line's lanes lie within one row of 16).  Lanes beyond a small level's
// cells repeat the cells of the lower lanes (same values to the same
// addresses), so no phase branches.
//
// The sweeps, line solves and transfers and the order of their arithmetic
// are those of the larger levels (rbgs, line_sweep_m with two rows per lane,
// restrict_residual -- whose products are rounded before they are added, as
// a select stands between them there --, prolong_add): bitwise the same results as when these
// levels ran through them.  FP32, per outer iteration of one solve (phase
// timers), with the generic loops before and here:
//   32x16 and below  pressure 22.5 -> 6.8 us, transport 26.1 -> 8.0 us
//   16x8 and below   pressure 11.4 -> 3.3 us, transport 16.3 -> 5.0 us
#pragma once

__device__ inline int wave_lane() { return (int)threadIdx.x & (kWave - 1); }

template <typename T, int kElems>
__device__ inline void wave_zero(LdsPtr<T> p) {
    const Vec4<T> z = {(T)0, (T)0, (T)0, (T)0};
#pragma unroll
    for (int k = 0; k < kElems / 4; k += kWave) {
        const int at = k + wave_lane();
        if (k + kWave <= kElems / 4 || at < kElems / 4) ((typename AsPtr<Vec4<T>, 3>::type)p)[at] = z;
    }
}

// ------------------------------------------------------------------ pressure
// V(2,2), red-black Gauss-Seidel.  A lane owns cell k = kr + H j' of each
// colour (j' = its row), NC of them 64 apart (rows of equal parity).
template <typename T, int NX>
struct WaveP {
    using D = WaveDim<NX>;
    static constexpr int NY = D::NY, H = D::H, CS = D::CS, RS = D::RS;
    static constexpr int M = D::N / 2;  // cells per colour
    static constexpr int NC = M > kWave ? M / kWave : 1;
    static constexpr int kRows = NC > 1 ? kWave / H : 0;  // rows between a lane's cells

    // te, tn in the colour-split layout; b and the result x in the lane's
    // cells, [colour][cell].  x also stays in the region for the finer level.
    __device__ static inline void run(LdsPtr<T> W, LdsPtr<T> te, LdsPtr<T> tn, const T (&b)[2][NC], T (&x)[2][NC]) {
        LdsPtr<T> X = W + D::base();
        if constexpr (NX == 2) {
            // 2 x 1 cells: direct solve
            const T e0 = te[0], e1 = te[1], n0 = tn[0], n1 = tn[1];
            const T d0 = e0 + (T)0 + n0 + (T)0, d1 = e1 + e0 + n1 + (T)0;
            const T det = fused(d0, d1, -rounded_mul(e0, e0));
            x[0][0] = fused(b[0][0], d1, rounded_mul(e0, b[1][0])) / det;
            x[1][0] = fused(d0, b[1][0], rounded_mul(e0, b[0][0])) / det;
            X[RS + 1] = x[0][0];
            X[RS + CS + 1] = x[1][0];
            WaveTeam::sync();
            return;
        } else {
            LdsPtr<T> R = X + D::kX;
            const int l = wave_lane() & (M < kWave ? M - 1 : kWave - 1);
            const int kr = l & (H - 1), jr = l >> ilog2(H);
            wave_zero<T, D::kXR>(X);
            // couplings of the lane's cells; o: column 2 kr + o
            T cw[2][NC], ce[2][NC], cs[2][NC], cn[2][NC], cd[2][NC], dred[NC];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int o = (jr + c) & 1;
                const bool hw = o + kr > 0, he = !(o == 1 && kr == H - 1);
#pragma unroll
                for (int u = 0; u < NC; ++u) {
                    const int j = jr + u * kRows;
                    const int row = j * NX;
                    const T tE = te[row + c * H + kr], tN = tn[row + c * H + kr];
                    const T tW = te[row + (1 - c) * H + (hw ? kr - 1 + o : kr)];
                    const bool hs = u > 0 || j > 0;
                    const T tS = tn[hs ? row - NX + (1 - c) * H + kr : row];
                    cw[c][u] = hw ? tW : (T)0;
                    ce[c][u] = he ? tE : (T)0;  // the seawater coefficient is diagonal only
                    cn[c][u] = tN;
                    cs[c][u] = hs ? tS : (T)0;
                    const T d = tE + cw[c][u] + cn[c][u] + cs[c][u];
                    if (c == 0) dred[u] = d;
                    cd[c][u] = diag_prep(d);
                }
            }
            auto own = [&](int c, int u) { return X + (jr + u * kRows + 1) * RS + c * CS + kr + 1; };
            // one half-sweep; the other colour's cells west and east of the
            // lane's lie side by side, those south and north one row away
            auto half = [&](int c) {
                const int o = (jr + c) & 1;
                T num[NC];
#pragma unroll
                for (int u = 0; u < NC; ++u) {
                    LdsPtr<T> q = X + (jr + u * kRows) * RS + (1 - c) * CS + kr;
                    const T xW = q[RS + o], xE = q[RS + o + 1], xS = q[1], xN = q[2 * RS + 1];
                    T a = b[c][u];
                    a += cw[c][u] * xW;
                    a += ce[c][u] * xE;
                    a += cs[c][u] * xS;
                    a += cn[c][u] * xN;
                    num[u] = a;
                }
#pragma unroll
                for (int u = 0; u < NC; ++u) {
                    x[c][u] = diag_div(num[u], cd[c][u]);
                    *own(c, u) = x[c][u];
                }
                WaveTeam::sync();
            };
            WaveTeam::sync();
            // from x = 0 the first half-sweep is the division alone
#pragma unroll
            for (int u = 0; u < NC; ++u) {
                x[0][u] = diag_div(b[0][u], cd[0][u]);
                *own(0, u) = x[0][u];
            }
            WaveTeam::sync();
            half(1);
            half(0);
            half(1);
            // residual of the red cells (the black ones' is zero to rounding)
            {
                const int o = jr & 1;
#pragma unroll
                for (int u = 0; u < NC; ++u) {
                    LdsPtr<T> q = X + (jr + u * kRows) * RS + CS + kr;
                    const T xW = q[RS + o], xE = q[RS + o + 1], xS = q[1], xN = q[2 * RS + 1];
                    T ax = fused(dred[u], x[0][u], -rounded_mul(cw[0][u], xW));
                    ax -= ce[0][u] * xE;
                    ax -= cs[0][u] * xS;
                    ax -= cn[0][u] * xN;
                    R[(jr + u * kRows + 1) * CS + kr + 1] = b[0][u] - ax;
                }
            }
            WaveTeam::sync();
            // coarser level: coefficients and restricted residual
            using P = WaveP<T, NX / 2>;
            using C = WaveDim<NX / 2>;
            LdsPtr<T> tec = W + C::base() + C::kXR, tnc = tec + C::N;
            T bc[2][P::NC], xc[2][P::NC];
            {
                const int lc = wave_lane() & (P::M < kWave ? P::M - 1 : kWave - 1);
                const int krc = lc & (C::H - 1), jrc = lc >> ilog2(C::H);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int I = 2 * krc + ((jrc + c) & 1);
                    const T w1 = I == 0 ? (T)1 : (T)0.75, w2 = I == C::H * 2 - 1 ? (T)1 : (T)0.75;
#pragma unroll
                    for (int u = 0; u < P::NC; ++u) {
                        const int J = jrc + u * P::kRows;
                        LdsPtr<T> f0 = te + 2 * J * NX + I, f1 = tn + (2 * J + 1) * NX + I;
                        tec[J * (NX / 2) + c * C::H + krc] = (T)0.5 * (f0[H] + f0[NX]);
                        tnc[J * (NX / 2) + c * C::H + krc] = (T)0.5 * (f1[H] + f1[0]);
                        LdsPtr<T> q = R + 2 * J * CS + I;
                        const T r0 = rounded_mul(q[0], (T)0.25) + rounded_mul(q[1], w2);
                        const T r1 = rounded_mul(q[CS + 1], w1) + rounded_mul(q[CS + 2], (T)0.25);
                        const T r2 = rounded_mul(q[2 * CS], (T)0.25) + rounded_mul(q[2 * CS + 1], w2);
                        const T r3 = rounded_mul(q[3 * CS + 1], w1) + rounded_mul(q[3 * CS + 2], (T)0.25);
                        const T v1 = J == 0 ? (T)1 : (T)0.75, v2 = J == C::NY - 1 ? (T)1 : (T)0.75;
                        T s = rounded_mul(r0, (T)0.25) + rounded_mul(r1, v1);
                        s += rounded_mul(r2, v2);
                        s += rounded_mul(r3, (T)0.25);
                        bc[c][u] = s;
                    }
                }
            }
            WaveTeam::sync();
            P::run(W, tec, tnc, bc, xc);
            // prolongation, then the post-smoothing
            LdsPtr<T> XC = W + C::base();
            auto cat = [&](int I, int J) { return XC[(J + 1) * C::RS + ((I + J) & 1) * C::CS + (I >> 1) + 1]; };
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int o = (jr + c) & 1;
                const int I = kr, In = o ? min(kr + 1, H - 1) : max(kr - 1, 0);
#pragma unroll
                for (int u = 0; u < NC; ++u) {
                    const int j = jr + u * kRows;
                    const int J = j >> 1, Jn = (j & 1) ? min(J + 1, C::NY - 1) : max(J - 1, 0);
                    x[c][u] = x[c][u] + prolonged(cat(I, J), cat(In, J), cat(I, Jn), cat(In, Jn));
                    *own(c, u) = x[c][u];
                }
            }
            WaveTeam::sync();
            for (int s = 0; s < 2; ++s) {
                half(0);
                half(1);
            }
        }
    }

    // The cycle of a hierarchy whose first wave level is v.
    __device__ static __attribute__((noinline)) void cycle(const Level<T>& v0, T* region) {
        const LV<T, 3> v(v0);
        const int l = wave_lane() & (M < kWave ? M - 1 : kWave - 1);
        const int kr = l & (H - 1), jr = l >> ilog2(H);
        T b[2][NC], x[2][NC];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int u = 0; u < NC; ++u) b[c][u] = v.b[(jr + u * kRows) * NX + c * H + kr];
        run(as_ptr<3>(region), v.te, v.tn, b, x);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int u = 0; u < NC; ++u) v.x[(jr + u * kRows) * NX + c * H + kr] = x[c][u];
    }
};

// ------------------------------------------------------------------ transport
// Zebra lines, two rows per lane: x-lines before the coarse correction,
// y-lines after it.
template <typename T>
struct WaveCoef {
    LdsPtr<T> acc, mx, my, dx, dy, b, dl, dr, mr, ml;
};

// Couplings and diagonal of a lane's two cells of a line.
template <typename T>
struct WavePair {
    T w[2], e[2], s[2], n[2], d[2];
};

// One step of parallel cyclic reduction of the lines' interface equations
// (line_sweep_m's): lanes whose partner lies outside the line have a zero
// coupling to it, so what the shift brings them (another line's finite
// coefficients, or 0 at the row's end) does not count.
template <int kS, int TL, typename T>
__device__ inline void wave_pcr(T& A, T& B, T& C, T& D, int t) {
    if constexpr (kS < TL) {
        T k1, k2;
        if constexpr (sizeof(T) == 4) {
            const T rB = __builtin_amdgcn_rcpf(B);
            k1 = A * lane_below<kS>(rB);
            k2 = C * lane_above<kS>(rB);
        } else {
            const T Bl = lane_below<kS>(B), Br = lane_above<kS>(B);
            k1 = t >= kS ? A / Bl : (T)0;
            k2 = t + kS < TL ? C / Br : (T)0;
        }
        const T nA = -lane_below<kS>(A) * k1, nC = -lane_above<kS>(C) * k2;
        T nB = B, nD = D;
        nB -= lane_below<kS>(C) * k1;
        nD -= lane_below<kS>(D) * k1;
        nB -= lane_above<kS>(A) * k2;
        nD -= lane_above<kS>(D) * k2;
        A = nA; B = nB; C = nC; D = nD;
        wave_pcr<2 * kS, TL>(A, B, C, D, t);
    }
}

// Solves the line that this lane holds two rows of: a0/a1, c0/c1 the
// couplings to the rows before and after (as positive off-diagonals), d the
// diagonals, r the right-hand sides.
template <int TL, typename T>
__device__ inline void wave_line(T a0, T c0, T d0, T r0, T a1, T c1, T d1, T r1, int t, T& x0, T& x1) {
    const T inv = qdiv((T)1, d0);
    const T y = r0 * inv, u = a0 * inv, w = c0 * inv;
    const T ar = -a1, cr = -c1;
    const T yN = TL > 1 ? lane_above<1>(y) : (T)0, uN = TL > 1 ? lane_above<1>(u) : (T)0,
            wN = TL > 1 ? lane_above<1>(w) : (T)0;
    T A = ar * u;
    T B = d1 + ar * w + cr * uN;
    T C = cr * wN;
    T D = r1 - ar * y - cr * yN;
    wave_pcr<1, TL>(A, B, C, D, t);
    const T iota = qdiv(D, B);
    const T left = TL > 1 ? lane_below<1>(iota) : (T)0;
    x0 = y + u * left + w * iota;
    x1 = iota;
}

template <typename T, int NX, bool kTrans>
struct WaveC {
    using D = WaveDim<NX>;
    static constexpr int NY = D::NY, RS = D::RS, N = D::N;
    static constexpr int kTX = NX / 2, kTY = NY > 1 ? NY / 2 : 1;  // lanes per x-line, y-line
    static constexpr int kSlots = NY > 1 ? N / 4 : 1;              // lanes' pairs per colour of lines
    static constexpr int NS = kSlots > kWave ? kSlots / kWave : 1;
    static constexpr int kMask = kSlots < kWave ? kSlots - 1 : kWave - 1;
    static constexpr int kXJump = 2 * (kWave / kTX), kYJump = 2 * (kWave / kTY);  // between a lane's lines

    // couplings across one face: from the cell on its low side to the one
    // on its high side (up: out of the high side's equation) and back
    __device__ static inline T in_high(T m, T d) { return pos(m) + d; }
    __device__ static inline T in_low(T m, T d) { return pos(-m) + d; }

    // Cells (2t, j) and (2t + 1, j).
    __device__ static inline WavePair<T> xpair(const WaveCoef<T>& a, int t, int j) {
        WavePair<T> p;
        const int k = j * NX + 2 * t;
        const bool hw = t > 0, he = t + 1 < kTX, hs = j > 0, hn = j + 1 < NY;
        const Vec2<T> ac = lds_load2<T>(a.acc + k), mE = lds_load2<T>(a.mx + k), dE = lds_load2<T>(a.dx + k),
                      mN = lds_load2<T>(a.my + k), dN = lds_load2<T>(a.dy + k);
        const int ks = hs ? k - NX : k, kw = hw ? k - 1 : k;
        const Vec2<T> mS = lds_load2<T>(a.my + ks), dS = lds_load2<T>(a.dy + ks);
        const T mW = a.mx[kw], dW = a.dx[kw];
        const T bE = pos(-a.mr[j]) + a.dr[j], bW = a.dl[j] + a.ml[j];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bool w_in = q > 0 || hw, e_in = q == 0 || he;
            const T mw = q == 0 ? mW : mE[0], dw = q == 0 ? dW : dE[0];
            const T e = in_low(mE[q], dE[q]), w = in_high(mw, dw), n = in_low(mN[q], dN[q]), s = in_high(mS[q], dS[q]);
            T d = ac[q];
            d += e_in ? e : bE;
            d += w_in ? w : bW;
            d += hn ? n : (T)0;
            d += hs ? s : (T)0;
            p.d[q] = d;
            p.e[q] = e_in ? (kTrans ? in_high(mE[q], dE[q]) : e) : (T)0;
            p.w[q] = w_in ? (kTrans ? in_low(mw, dw) : w) : (T)0;
            p.n[q] = hn ? (kTrans ? in_high(mN[q], dN[q]) : n) : (T)0;
            p.s[q] = hs ? (kTrans ? in_low(mS[q], dS[q]) : s) : (T)0;
        }
        return p;
    }

    // Cells (i, 2t) and (i, 2t + 1).
    __device__ static inline WavePair<T> ypair(const WaveCoef<T>& a, int t, int i) {
        WavePair<T> p;
        const int k = 2 * t * NX + i;
        const bool hw = i > 0, he = i + 1 < NX;
        const int kw = hw ? k - 1 : k;
        const int ks = t > 0 ? k - NX : k;
        const T mS0 = a.my[ks], dS0 = a.dy[ks];
        const Vec2<T> mr = lds_load2<T>(a.mr + 2 * t), dr = lds_load2<T>(a.dr + 2 * t), dl = lds_load2<T>(a.dl + 2 * t),
                      ml = lds_load2<T>(a.ml + 2 * t);
        T mN0 = (T)0, dN0 = (T)0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bool hs = q > 0 || t > 0, hn = q == 0 || t + 1 < kTY;
            const T mE = a.mx[k + q * NX], dE = a.dx[k + q * NX], mW = a.mx[kw + q * NX], dW = a.dx[kw + q * NX];
            const T mN = a.my[k + q * NX], dN = a.dy[k + q * NX];
            const T mS = q == 0 ? mS0 : mN0, dS = q == 0 ? dS0 : dN0;
            const T bE = pos(-mr[q]) + dr[q], bW = dl[q] + ml[q];
            const T e = in_low(mE, dE), w = in_high(mW, dW), n = in_low(mN, dN), s = in_high(mS, dS);
            T d = a.acc[k + q * NX];
            d += he ? e : bE;
            d += hw ? w : bW;
            d += hn ? n : (T)0;
            d += hs ? s : (T)0;
            p.d[q] = d;
            p.e[q] = he ? (kTrans ? in_high(mE, dE) : e) : (T)0;
            p.w[q] = hw ? (kTrans ? in_low(mW, dW) : w) : (T)0;
            p.n[q] = hn ? (kTrans ? in_high(mN, dN) : n) : (T)0;
            p.s[q] = hs ? (kTrans ? in_low(mS, dS) : s) : (T)0;
            mN0 = mN; dN0 = dN;
        }
        return p;
    }

    // One colour of x-lines; with kZero the rows beside them are still zero.
    // Leaves the pairs, right-hand sides and solutions with the caller.
    template <bool kZero>
    __device__ static inline void xlines(LdsPtr<T> X, const WaveCoef<T>& a, int col, WavePair<T> (&p)[NS], T (&b)[NS][2],
                                         T (&x)[NS][2]) {
        const int l = wave_lane() & kMask;
        const int t = l & (kTX - 1), j0 = col + 2 * (l >> ilog2(kTX));
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int j = j0 + u * kXJump;
            p[u] = xpair(a, t, j);
            const Vec2<T> bv = lds_load2<T>(a.b + j * NX + 2 * t);
            b[u][0] = bv[0];
            b[u][1] = bv[1];
        }
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int j = j0 + u * kXJump;
            T r[2] = {b[u][0], b[u][1]};
            if constexpr (!kZero) {
                const Vec2<T> xS = lds_load2<T>(X + j * RS + 2 * t + 2), xN = lds_load2<T>(X + (j + 2) * RS + 2 * t + 2);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    r[q] += p[u].s[q] * xS[q];
                    r[q] += p[u].n[q] * xN[q];
                }
            }
            wave_line<kTX>(p[u].w[0], p[u].e[0], p[u].d[0], r[0], p[u].w[1], p[u].e[1], p[u].d[1], r[1], t, x[u][0],
                           x[u][1]);
        }
#pragma unroll
        for (int u = 0; u < NS; ++u) lds_store2<T>(X + (j0 + u * kXJump + 1) * RS + 2 * t + 2, x[u][0], x[u][1]);
        WaveTeam::sync();
    }

    __device__ static inline void ylines(LdsPtr<T> X, const WaveCoef<T>& a, int col) {
        const int l = wave_lane() & kMask;
        const int t = l & (kTY - 1), i0 = col + 2 * (l >> ilog2(kTY));
        T x[NS][2];
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int i = i0 + u * kYJump;
            const WavePair<T> p = ypair(a, t, i);
            LdsPtr<T> q0 = X + (2 * t + 1) * RS + i + 1;  // west of the first cell
            T r[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                r[q] = a.b[(2 * t + q) * NX + i];
                r[q] += p.w[q] * q0[q * RS];
                r[q] += p.e[q] * q0[q * RS + 2];
            }
            wave_line<kTY>(p.s[0], p.n[0], p.d[0], r[0], p.s[1], p.n[1], p.d[1], r[1], t, x[u][0], x[u][1]);
        }
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            LdsPtr<T> q0 = X + (2 * t + 1) * RS + i0 + u * kYJump + 2;
            q0[0] = x[u][0];
            q0[RS] = x[u][1];
        }
        WaveTeam::sync();
    }

    __device__ static inline void run(LdsPtr<T> W, const WaveCoef<T>& a) {
        LdsPtr<T> X = W + D::base();
        WavePair<T> p[NS];
        T b[NS][2], x[NS][2];
        if constexpr (NX == 2) {
            xlines<true>(X, a, 0, p, b, x);  // one row: its line is the whole system
            return;
        } else {
            LdsPtr<T> R = X + D::kX;
            wave_zero<T, D::kXR>(X);
            WaveTeam::sync();
            {
                WavePair<T> p1[NS];
                T b1[NS][2], x1[NS][2];
                xlines<true>(X, a, 0, p, b, x);
                xlines<false>(X, a, 1, p1, b1, x1);
            }
            // residual of the even rows (the odd ones' is zero to rounding)
            {
                const int l = wave_lane() & kMask;
                const int t = l & (kTX - 1), j0 = 2 * (l >> ilog2(kTX));
#pragma unroll
                for (int u = 0; u < NS; ++u) {
                    const int j = j0 + u * kXJump;
                    LdsPtr<T> q0 = X + (j + 1) * RS + 2 * t + 2;
                    const Vec2<T> xS = lds_load2<T>(q0 - RS), xN = lds_load2<T>(q0 + RS);
                    const T xW = q0[-1], xE = q0[2];
                    T r[2];
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        T ax = fused(p[u].d[q], x[u][q], -rounded_mul(p[u].w[q], q == 0 ? xW : x[u][0]));
                        ax -= p[u].e[q] * (q == 0 ? x[u][1] : xE);
                        ax -= p[u].s[q] * xS[q];
                        ax -= p[u].n[q] * xN[q];
                        r[q] = b[u][q] - ax;
                    }
                    lds_store2<T>(R + (j >> 1) * RS + 2 * t + 2, r[0], r[1]);
                }
            }
            WaveTeam::sync();
            // coarser level: coefficients and restricted residual
            using C = WaveDim<NX / 2>;
            constexpr int kXC = NX / 2;
            LdsPtr<T> s0 = W + C::base() + C::kXR;
            WaveCoef<T> ac;
            ac.acc = s0; ac.mx = s0 + C::N; ac.my = s0 + 2 * C::N; ac.dx = s0 + 3 * C::N; ac.dy = s0 + 4 * C::N;
            ac.b = s0 + 5 * C::N;
            ac.dl = s0 + 6 * C::N; ac.dr = ac.dl + C::NY; ac.mr = ac.dr + C::NY; ac.ml = ac.mr + C::NY;
            constexpr int kPer = C::N > kWave ? C::N / kWave : 1;
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int k = (wave_lane() & (C::N < kWave ? C::N - 1 : kWave - 1)) + u * kWave;
                const int I = k & (kXC - 1), J = k >> ilog2(kXC);
                const int f = 2 * J * NX + 2 * I;
                const Vec2<T> a0 = lds_load2<T>(a.acc + f), a1 = lds_load2<T>(a.acc + f + NX);
                ac.acc[k] = (a0[0] + a0[1]) + (a1[0] + a1[1]);
                const T mx = a.mx[f + 1] + a.mx[f + NX + 1], dx = (T)0.5 * (a.dx[f + 1] + a.dx[f + NX + 1]);
                const Vec2<T> my = lds_load2<T>(a.my + f + NX), dy = lds_load2<T>(a.dy + f + NX);
                ac.mx[k] = I + 1 < kXC ? mx : (T)0;
                ac.dx[k] = I + 1 < kXC ? dx : (T)0;
                ac.my[k] = J + 1 < C::NY ? my[0] + my[1] : (T)0;
                ac.dy[k] = J + 1 < C::NY ? (T)0.5 * (dy[0] + dy[1]) : (T)0;
                LdsPtr<T> q = R + J * RS + 2 * I + 1;
                const T w1 = I == 0 ? (T)1 : (T)0.75, w2 = I == kXC - 1 ? (T)1 : (T)0.75;
                T r1 = rounded_mul(q[0], (T)0.25) + rounded_mul(q[1], w1);
                r1 += rounded_mul(q[2], w2);
                r1 += rounded_mul(q[3], (T)0.25);
                T r3 = rounded_mul(q[RS], (T)0.25) + rounded_mul(q[RS + 1], w1);
                r3 += rounded_mul(q[RS + 2], w2);
                r3 += rounded_mul(q[RS + 3], (T)0.25);
                ac.b[k] = rounded_mul(r1, J == 0 ? (T)1 : (T)0.75) + rounded_mul(r3, (T)0.25);
            }
            {
                const int J = wave_lane() & (C::NY - 1);
                ac.dl[J] = (T)0.5 * (a.dl[2 * J] + a.dl[2 * J + 1]);
                ac.dr[J] = (T)0.5 * (a.dr[2 * J] + a.dr[2 * J + 1]);
                ac.mr[J] = a.mr[2 * J] + a.mr[2 * J + 1];
                ac.ml[J] = a.ml[2 * J] + a.ml[2 * J + 1];
            }
            WaveTeam::sync();
            WaveC<T, NX / 2, kTrans>::run(W, ac);
            // prolongation, then the post-smoothing
            LdsPtr<T> XC = W + C::base();
            auto cat = [&](int I, int J) { return XC[(J + 1) * C::RS + I + 2]; };
            constexpr int kFine = N > kWave ? N / kWave : 1;
            const int l = wave_lane() & (N < kWave ? N - 1 : kWave - 1);
            const int i = l & (NX - 1), jr = l >> ilog2(NX);
            const int I = i >> 1, In = (i & 1) ? min(I + 1, kXC - 1) : max(I - 1, 0);
            T xf[kFine];
#pragma unroll
            for (int u = 0; u < kFine; ++u) {
                const int j = jr + u * (kWave / NX);
                const int J = j >> 1, Jn = (j & 1) ? min(J + 1, C::NY - 1) : max(J - 1, 0);
                xf[u] = X[(j + 1) * RS + i + 2] + prolonged(cat(I, J), cat(In, J), cat(I, Jn), cat(In, Jn));
            }
#pragma unroll
            for (int u = 0; u < kFine; ++u) X[(jr + u * (kWave / NX) + 1) * RS + i + 2] = xf[u];
            WaveTeam::sync();
            ylines(X, a, 0);
            ylines(X, a, 1);
        }
    }

    __device__ static __attribute__((noinline)) void cycle(const Level<T>& v0, T* region) {
        const LV<T, 3> v(v0);
        WaveCoef<T> a;
        a.acc = v.acc; a.mx = v.mx; a.my = v.my; a.dx = v.dx; a.dy = v.dy; a.b = v.b;
        a.dl = v.dl; a.dr = v.dr; a.mr = v.mr; a.ml = v.ml;
        LdsPtr<T> W = as_ptr<3>(region);
        run(W, a);
        constexpr int kPairs = N / 2;
        LdsPtr<T> X = W + D::base();
#pragma unroll
        for (int u = 0; u < (kPairs > kWave ? kPairs / kWave : 1); ++u) {
            const int k = 2 * ((wave_lane() & (kPairs < kWave ? kPairs - 1 : kWave - 1)) + u * kWave);
            const Vec2<T> x = lds_load2<T>(X + ((k >> ilog2(NX)) + 1) * RS + (k & (NX - 1)) + 2);
            lds_store2<T>(v.x + k, x[0], x[1]);
        }
        WaveTeam::sync();
    }
};

// The V-cycle from level v down (v.x from zero), by the calling wavefront.
template <typename T, bool kTransport, bool kTrans>
__device__ inline void wave_cycle(const Level<T>& v, T* region) {
    switch (v.nx) {
        case 2: if constexpr (kTransport) WaveC<T, 2, kTrans>::cycle(v, region); else WaveP<T, 2>::cycle(v, region); break;
        case 4: if constexpr (kTransport) WaveC<T, 4, kTrans>::cycle(v, region); else WaveP<T, 4>::cycle(v, region); break;
        case 8: if constexpr (kTransport) WaveC<T, 8, kTrans>::cycle(v, region); else WaveP<T, 8>::cycle(v, region); break;
        case 16: if constexpr (kTransport) WaveC<T, 16, kTrans>::cycle(v, region); else WaveP<T, 16>::cycle(v, region); break;
        default: if constexpr (kTransport) WaveC<T, 32, kTrans>::cycle(v, region); else WaveP<T, 32>::cycle(v, region); break;
    }
}
