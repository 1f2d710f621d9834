// Device helpers shared by the dense and the sparse kernels of the MBD stage.
#pragma once

#include "lmbd_internal.h"

namespace lmbd {

__host__ __device__ inline size_t al4(size_t x) { return (x + 3) / 4 * 4; }

// Per-site arrays (LDS, or the workspace) and the small per-atom arrays (LDS).  The
// pair sums g of the force stage take the place of sqrt(alpha~), whose last use (the
// operands of Tbar) precedes them.
struct MbdLds {
    double *px, *py, *pz, *sa, *sqa, *Rt, *fs, *dfs, *ab, *g, *rb, *fg, *mu, *cf, *lz;
};
// sa and ab hold every frequency of the energy: 0 and the nq nodes.  cf (fitted
// coefficients, [nq][kMaxNmax + 1] and [kMaxNmax + 1][nq]) and lz (Lanczos: alpha and beta [steps][nq], the steps
// taken and the two bounds per node) exist only when used.  The site arrays take
// mbd_site_doubles(nk, nq) from b, the small ones start at sm.
__device__ inline MbdLds mbd_lds(double* b, int nk, int nq, double* sm, int n_max, bool fit) {
    const int nw = nq + 1;
    MbdLds L;
    L.px = b;
    L.py = L.px + nk;
    L.pz = L.py + nk;
    L.sa = L.pz + nk;
    L.sqa = L.sa + (size_t)nk * nw;   // [nk][nq]
    L.g = L.sqa;                      // [4 parts][nk][3], nq >= 12 (force stage only)
    L.Rt = L.sqa + (size_t)nk * max(nq, 12);
    L.fs = L.Rt + nk;
    L.dfs = L.fs + nk;
    L.ab = L.dfs + nk;
    L.rb = L.ab + (size_t)nk * nw;    // [4 parts][nk]
    L.fg = L.rb + 4 * (size_t)nk;     // [nk][3]
    L.mu = sm;
    L.cf = L.mu + (size_t)(n_max + 1) * nq;
    L.lz = L.cf + (fit ? 2 * (size_t)(kMaxNmax + 1) * nq : 0);
    return L;
}

// The output function of SplitMix64 (Steele, Lea and Flood, OOPSLA 2014) on a 64-bit counter.
__device__ inline uint64_t splitmix64(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Coefficients c_0 .. c_n_max (c_0 = c_1 = 0 on return) of the least-squares polynomial
// of ln(1 - x) on [lo, hi] over the Gauss-Legendre points x_i of [-1, 1] mapped to it:
// the Legendre coefficients a_j = (2 j + 1) / 2 sum_i w_i ln(1 - lambda_i) P_j(x_i),
// then sum_j a_j P_j(t), t = (x - mid) / half, in powers of x by Clenshaw's recurrence
// b_j = a_j + (2j+1)/(j+1) t b_{j+1} - (j+1)/(j+2) b_{j+2} carried out on coefficient
// arrays (b_0 is the polynomial).  No width (hi - lo <= 1e-12): the Taylor
// coefficients -1/n.
__host__ __device__ inline void log_fit(double lo, double hi, int n_max, const double* gx, const double* gw,
                                        double (&c)[kMaxNmax + 1]) {
#pragma unroll
    for (int n = 0; n <= kMaxNmax; ++n) c[n] = n >= 2 ? -1.0 / n : 0.0;
    if (!(hi - lo > 1e-12)) return;
    const double h = 0.5 * (hi - lo), m = 0.5 * (hi + lo), ih = 1.0 / h;
    double cl[kMaxNmax + 1];
#pragma unroll
    for (int j = 0; j <= kMaxNmax; ++j) cl[j] = 0.0;
    for (int i = 0; i < kFitNodes; ++i) {
        const double x = gx[i];
        const double f = gw[i] * log1p(-(m + h * x));
        double p0 = 1.0, p1 = x;
        cl[0] += f;
        cl[1] += f * x;
#pragma unroll
        for (int j = 2; j <= kMaxNmax; ++j) {
            const double p2 = ((2 * j - 1) * x * p1 - (j - 1) * p0) / j;
            cl[j] += f * p2;
            p0 = p1;
            p1 = p2;
        }
    }
    // b1 = b_{j+1}, b2 = b_{j+2}; b_j overwrites b2, then the two swap roles
    double b1[kMaxNmax + 1], b2[kMaxNmax + 1];
#pragma unroll
    for (int t = 0; t <= kMaxNmax; ++t) b1[t] = b2[t] = 0.0;
#pragma unroll
    for (int j = kMaxNmax; j >= 0; --j) {
        if (j > n_max) continue;
        const double aj = 0.5 * (2 * j + 1) * cl[j];
        const double al = (2.0 * j + 1.0) / (j + 1.0) * ih, be = -(j + 1.0) / (j + 2.0);
#pragma unroll
        for (int t = kMaxNmax; t >= 0; --t)
            b2[t] = (t == 0 ? aj : 0.0) + al * ((t > 0 ? b1[t - 1] : 0.0) - m * b1[t]) + be * b2[t];
#pragma unroll
        for (int t = 0; t <= kMaxNmax; ++t) {
            const double x = b1[t];
            b1[t] = b2[t];
            b2[t] = x;
        }
    }
#pragma unroll
    for (int n = 0; n <= kMaxNmax; ++n) c[n] = n >= 2 ? b1[n] : 0.0;
}

// T_LR pair coefficients: T_LR = A rhat rhat^T + B I with radial derivatives,
// and dT_LR/dS~ = fLR (df/dS~) T.
template <typename P>
struct LrPair {
    P A, B, dA, dB, dfS, fLR;
};
template <typename P>
__device__ inline LrPair<P> lr_pair(P r, P S, P damp_d, P rcut, P rb) {
    P dfdr, dfdS, dcut;
    const P f = fermi<P>(r, S, damp_d, dfdr, dfdS);
    const P fc = cutoff_poly<P>(r, rcut, rb, dcut);
    const P w = fc * f;
    const P dw = dcut * f + fc * dfdr;
    const P ir = P(1) / r;
    const P ir3 = ir * ir * ir;
    LrPair<P> p;
    p.A = P(3) * w * ir3;
    p.B = -w * ir3;
    p.dA = P(3) * dw * ir3 - P(9) * w * ir3 * ir;
    p.dB = -dw * ir3 + P(3) * w * ir3 * ir;
    p.dfS = dfdS;
    p.fLR = fc;
    return p;
}

// Value of `x` in lane l (l uniform over the wavefront).
__device__ inline double read_lane(double x, int l) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Sums over the 64 lanes of nine per-lane values, returned to every lane.  A
// transposed butterfly: at the exchanges over lane bits 5, 4, 3 and 2 a lane keeps
// half of the (zero-padded to 16) values it carries and sends the other half, so
// lane l ends with value 8 b5 + 4 b4 + 2 b3 + b2 (b_n: bit n of l) summed over its
// 16 partners; two plain exchanges finish the sum and one lane per value gives it
// out: 17 exchanges instead of 54.
__device__ inline void wave_sum9(const double (&v)[9], double (&out)[9]) {
    const int lane = threadIdx.x & 63;
    double a[8], b[4], c[2];
    bool hi = lane & 32;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const double lo_v = v[t], hi_v = (t == 0) ? v[8] : 0.0;
        a[t] = (hi ? hi_v : lo_v) + __shfl_xor(hi ? lo_v : hi_v, 32);
    }
    hi = lane & 16;
#pragma unroll
    for (int t = 0; t < 4; ++t) b[t] = (hi ? a[4 + t] : a[t]) + __shfl_xor(hi ? a[t] : a[4 + t], 16);
    hi = lane & 8;
#pragma unroll
    for (int t = 0; t < 2; ++t) c[t] = (hi ? b[2 + t] : b[t]) + __shfl_xor(hi ? b[t] : b[2 + t], 8);
    hi = lane & 4;
    double d = (hi ? c[1] : c[0]) + __shfl_xor(hi ? c[0] : c[1], 4);
    d += __shfl_xor(d, 2);
    d += __shfl_xor(d, 1);
#pragma unroll
    for (int x = 0; x < 9; ++x)
        out[x] = read_lane(d, ((x >> 3) & 1) << 5 | ((x >> 2) & 1) << 4 | ((x >> 1) & 1) << 3 | (x & 1) << 2);
}

// Spectrum bounds of G~ at every node (Lanczos) and, with a.fit, the fitted c_n, by one
// workgroup.  vecs: three vectors per node, column-major ([nq][N3p]).  start(r): entry r
// of the unnormalised start vector; put(q, r, v): called for every entry of a new v_j
// (the dense products keep D v as their operand); product(v, w): w = G~ v at every node,
// ending with a barrier (a node that has stopped has v = 0).
template <typename W, class Start, class Put, class Product>
__device__ __forceinline__ void lanczos_fit(const MbdArgs& a, int k, int N3, int N3p, const MbdLds& L, W* vecs,
                                            Start start, Put put, Product product) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwave = blockDim.x >> 6;
    const int nq = a.nq, n_max = a.n_max;
    const bool fit = a.fit != 0;
    double* const cfn = L.cf + (size_t)(kMaxNmax + 1) * nq;
    const int m = a.lz_steps;
    W* vb[3] = {vecs, vecs + (size_t)nq * N3p, vecs + 2 * (size_t)nq * N3p};
    double* la = L.lz;                            // alpha_j of node q at [j nq + q]
    double* lb = la + (size_t)m * nq;             // beta_{j+1} at [j nq + q]
    double* lm = lb + (size_t)m * nq;             // steps taken per node
    double* bnd = lm + nq;                        // [nq][2] bounds
    auto wave_total = [&](double x) -> double {   // same order, same value in every lane
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
        return x;
    };
    for (int q = wave; q < nq; q += nwave) {
        double s2 = 0.0;
        for (int r = lane; r < N3; r += 64) {
            const double x = start(r);
            s2 += x * x;
        }
        const double inv = 1.0 / sqrt(wave_total(s2));
        W* v1 = vb[1] + (size_t)q * N3p;
        W* v0 = vb[0] + (size_t)q * N3p;
        for (int r = lane; r < N3; r += 64) {
            const W v = W(start(r) * inv);
            v1[r] = v;
            v0[r] = W(0);
            put(q, r, v);
        }
        if (lane == 0) lm[q] = m;
    }
    __syncthreads();
    int ip = 0, ic = 1, iw = 2;
    for (int j = 0; j < m; ++j) {
        // w = G~ v_j at every node (a node that has stopped has v_j = 0)
        product(vb[ic], vb[iw]);   // ends with a barrier
        // w -= beta_j v_{j-1}; alpha_j = <v_j, w>; w -= alpha_j v_j; beta_{j+1} = |w|;
        // v_{j+1} = w / beta_{j+1} (zero once the node stops)
        for (int q = wave; q < nq; q += nwave) {
            if (lm[q] <= j) continue;
            const W* vp = vb[ip] + (size_t)q * N3p;
            const W* vc = vb[ic] + (size_t)q * N3p;
            W* w = vb[iw] + (size_t)q * N3p;
            const double bj = j > 0 ? lb[(size_t)(j - 1) * nq + q] : 0.0;
            double s = 0.0;
            for (int r = lane; r < N3; r += 64) {
                const double t = double(w[r]) - bj * double(vp[r]);
                w[r] = W(t);
                s += double(vc[r]) * t;
            }
            const double al = wave_total(s);
            double s2 = 0.0;
            for (int r = lane; r < N3; r += 64) {
                const double t = double(w[r]) - al * double(vc[r]);
                w[r] = W(t);
                s2 += t * t;
            }
            const double bn = sqrt(wave_total(s2));
            const bool stop = j == m - 1 || !(bn > 1e-10 * (fabs(al) + bj));
            const double inv = stop ? 0.0 : 1.0 / bn;
            for (int r = lane; r < N3; r += 64) {
                const W v = W(double(w[r]) * inv);
                w[r] = v;
                put(q, r, v);
            }
            if (lane == 0) {
                la[(size_t)j * nq + q] = al;
                lb[(size_t)j * nq + q] = bn;
                if (stop) lm[q] = j + 1;
            }
        }
        __syncthreads();
        const int t = ip;
        ip = ic;
        ic = iw;
        iw = t;
    }
    // extreme eigenvalues of each node's tridiagonal matrix: bisection on the number
    // of eigenvalues below x (the negative pivots of T - x I = L D L^T), one lane per end
    if (tid < 2 * nq) {
        const int q = tid >> 1, top = tid & 1;
        const int me = (int)lm[q];
        double glo = 0.0, ghi = 0.0;
        for (int j = 0; j < me; ++j) {
            const double b0 = j > 0 ? fabs(lb[(size_t)(j - 1) * nq + q]) : 0.0;
            const double b1 = j + 1 < me ? fabs(lb[(size_t)j * nq + q]) : 0.0;
            const double aj = la[(size_t)j * nq + q];
            glo = j == 0 ? aj - b0 - b1 : fmin(glo, aj - b0 - b1);
            ghi = j == 0 ? aj + b0 + b1 : fmax(ghi, aj + b0 + b1);
        }
        const double pad = 1e-14 * (fabs(glo) + fabs(ghi)) + 1e-300;
        double lo = glo - pad, hi = ghi + pad;
        const int target = top ? me : 1;   // count(lo) < target <= count(hi)
        for (int it = 0; it < 256; ++it) {
            const double mid = 0.5 * (lo + hi);
            if (!(mid > lo && mid < hi)) break;
            int cnt = 0;
            double d = 1.0;
            for (int j = 0; j < me; ++j) {
                const double bb = j > 0 ? lb[(size_t)(j - 1) * nq + q] : 0.0;
                d = la[(size_t)j * nq + q] - mid - (j > 0 ? bb * bb / d : 0.0);
                if (fabs(d) < 1e-300) d = -1e-300;
                cnt += d < 0.0 ? 1 : 0;
            }
            if (cnt >= target)
                hi = mid;
            else
                lo = mid;
        }
        bnd[tid] = hi;
        if (a.spectrum) a.spectrum[((size_t)k * nq + q) * 2 + top] = hi;
    }
    __syncthreads();
    if (fit && tid < nq) {
        const int q = tid;
        const double lo = bnd[2 * q], hi = bnd[2 * q + 1];
        double c[kMaxNmax + 1];
        if (!(hi < 1.0)) {   // polarisation catastrophe: ln(1 - x) has no fit
            atomicOr(a.err, 16);
            atomicMin(a.err_atom, k);
#pragma unroll
            for (int n = 0; n <= kMaxNmax; ++n) c[n] = 0.0;
        } else {
            log_fit(lo, hi, n_max, a.gl_x, a.gl_w, c);
        }
#pragma unroll
        for (int n = 0; n <= kMaxNmax; ++n) {
            L.cf[q * (kMaxNmax + 1) + n] = c[n];
            cfn[n * nq + q] = c[n];
        }
    }
    __syncthreads();
}

// Entry r of the Lanczos start vector of frame k, keyed on (k, base atom, lattice shift,
// component) in the structure's numbering.
__device__ inline double lanczos_start(const StructInfo& SI, int k, const Site& st, int r) {
    const uint64_t h = splitmix64(((uint64_t)(k - SI.atom_offset) << 32) + (uint64_t)(st.base - SI.atom_offset));
    const uint64_t z = splitmix64(h + 4ull * (uint64_t)(uint32_t)st.shift + (uint64_t)(r % 3));
    return (double)(z >> 11) * 0x1.0p-53 - 0.5;
}

}  // namespace lmbd
