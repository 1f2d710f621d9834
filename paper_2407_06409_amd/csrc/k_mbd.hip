// Local MBD energy of every atom and its adjoint (Sec. III.A and III.B).
//
// For central atom k with neighbourhood K (central atom first):
//   alpha~_i(w) = (1 - f_SCS(r_ik)) alpha~_K,i(w) + f_SCS(r_ik) alpha~_I,i(w)  (r_ik < r_scs)
//               = alpha~_I,i(w)                                              (otherwise)
//   R~_i = R0_i (alpha~_i(0) / alpha0_i)^(1/3),  S~_ij = beta (R~_i + R~_j)
//   T_LR,ij = f_LR(r_ij; p) f(r_ij, S~_ij) T_ij      (frequency independent)
//   G~(w) = D T_LR D,  D = diag(sqrt(alpha~_i(w)))
//   E_k = (1/2pi) sum_q w_q sum_{n=2}^{n_max} c_n Tr[G~(w_q)^n]_kk.
// With u_m = G~^m e_k (e_k = the three columns of the central atom),
// Tr[G~^n]_kk = <u_a, u_b> for any a + b = n, so only ceil(n_max/2) products
// with G~ are needed for the energy; all quadrature nodes are stacked as
// columns (3 per node) so each product is one (3n x 3n) x (3n x 3 n_q) GEMM.
//
// Adjoint (seed w_k on E_k):
//   dE/d alpha~_i(w_q) = (W_q / alpha~_i) sum_n c_n sum_{a=0}^{n-1} <u_a, u_{n-a}>_i
//   Tbar = sum_q W_q D Gbar_q D,  Gbar_q = sum_n c_n sum_{a=0}^{n-1} u_a u_{n-1-a}^T
// then contracted pair by pair with dT_LR/dr and dT_LR/dS~, and pushed
// through the blend (local part to this atom's SCS, central part scattered to
// the neighbours' own SCS through a per-site contribution buffer).
//
// Approximate forces of Sec. III.D (a.paper): the seed is the functional of the
// frame whose r_k-gradient is the paper's force, int dw/2pi [c_2 Tr(G~^2) + sum_{n>=3}
// c_n n Tr(g~_k B_n g~_k^T)] (B_n = G~^(n-2) fixed), so that
//   Gbar_q = 2 c_2 G~ + sum_{n>=3} c_n n (u_{n-1} e_k^T + e_k u_{n-1}^T):
// the low-rank part keeps the Tbar product with Z_0 = sum_{n>=3} c_n n u_{n-1} and
// Z_{n-1} = c_n n e_k, the full n = 2 part is added to Tbar element by element, and
//   dE/d alpha~_i(w_q) = W_q [2 c_2 sum_j alpha~_j |T_ij|^2 + sum_{n>=3} c_n n
//                             (<u_{n-1}, u_1>_i + delta_ik mu_n) / alpha~_i];
// the central polarisabilities are held fixed (nothing is scattered to the
// neighbours), and the host keeps only the gradient of the frame's own atom.
//
// Two-body radii (Sec. III.A; SI.two_body): the n = 2 term takes a T_LR of its own, cut
// at r_2b1 on the pairs touching k and r_2b2 on the others.  Its moment is formed
// directly, mu_2 = sum_j alpha~_k alpha~_j |T2_kj|^2 (the central block row), its
// polarisability adjoint likewise, it leaves the Krylov coefficients of Tbar, and its
// pair derivative C2_kj = 2 w_k sum_q W_q c_2 alpha~_k alpha~_j T2_kj is contracted with
// dT2/dr where the pair visits of the contraction meet it (the sparse lists hold the
// central pairs out to max(r_mbd1, r_2b1)).  The approximate forces take the n = 2
// trace of the whole frame with T2: |T2_ij|^2 in the polarisability adjoint and
// C2_ij = 4 w_k sum_q W_q c_2 alpha~_i alpha~_j T2_ij on every pair within the two-body radii.
//
// Eigenvalue-bounded coefficients (Sec. III.A, Eqs. diagonal_appr, eigendecomp and
// polynomial-fit; a.fit): per atom and node, a.lz_steps Lanczos steps on G~ (all nodes
// side by side as columns: each step one (3n x 3n) x (3n x nq) product) give the
// tridiagonal matrix whose extreme eigenvalues (bisection on its Sturm counts) bound
// the spectrum; c_0 .. c_n_max are the least-squares polynomial of ln(1 - x) on that
// interval over the 32 Gauss-Legendre points, formed as the Legendre projection (the
// rule makes the discrete inner product exact for the Legendre polynomials up to
// degree 2 n_max) and converted to powers of x.  The adjoint holds them fixed.
//
// Two-point frequency model (Sec. III.C, Eqs. alpha_SCS_freq and char-freq):
// the SCS is solved at 0 and w_ref only; the blend gives a0 = alpha~_i(0) and
// ar = alpha~_i(w_ref), and alpha~_i(w) = a0 / (1 + (w / w~_i)^2) with
// w~_i = w_ref / sqrt(a0 / ar - 1), evaluated as a0 ar / (rho a0 + (1 - rho) ar),
// rho = (w / w_ref)^2.  Its adjoint: d alpha/d a0 = (1 - rho) (alpha / a0)^2 and
// d alpha/d ar = rho (alpha / ar)^2.
#include <algorithm>
#include <type_traits>

#include "mbd_common.h"

namespace lmbd {


// Doubles of the site arrays before the polarisability adjoints (see mbd_lds)
__host__ __device__ inline size_t mbd_adjoint_offset(int nk, int nq) {
    return (size_t)nk * (3 + (nq + 1) + (nq > 12 ? nq : 12) + 3);
}

size_t mbd_lds_bytes(int nkmax, int nq, int n_max, int lz_steps, bool fit) {
    return sizeof(double) * (mbd_site_doubles((size_t)nkmax, nq) + mbd_small_doubles(nq, n_max, lz_steps, fit));
}

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

// MFMA 16x16x4 in the workspace type (lane layouts as measured on gfx950: A[i][k]
// <- lane i + 16k, B[k][j] <- lane j + 16k; D[i][j] in lane j + 16 (i % 4), register
// i / 4 for f64 and lane j + 16 (i / 4), register i % 4 for f32).
template <typename W> struct MfmaW;
template <> struct MfmaW<double> {
    typedef d4_t acc;
    static __device__ inline acc mma(double a, double b, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline int acc_row(int g, int q) { return g + 4 * q; }
};
template <> struct MfmaW<float> {
    typedef f4_t acc;
    static __device__ inline acc mma(float a, float b, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int acc_row(int g, int q) { return 4 * g + q; }
};

// Symmetric workgroup product on the matrix cores: out(m, n) = sum_k A[m][k] B[n][k] for the
// items holding entries on or below the diagonal of the M x M result (the rest of the output
// is left as it was), both operands k-contiguous (row-major, ld a multiple of 4, K a multiple
// of 4; K = 0: zeros, and nothing is read).  Lane (i, g) of an MFMA operand reads the 4-vector
// k = 16 c + 4 g .. + 3 and feeds element e to k-step e, the same permutation of k for both operands.  Items of MR 16-row
// strips times up to MR 16-column tiles; the next chunk of 16 k is in flight in a second set
// of registers, every load with clamped indices and no condition (rows past M repeat the last
// one, nothing stores them; k past K is zeroed in A).  Tbar per atom of 64 C open: 39.7k ->
// 29.9k cycles against conditional loads, which were waited for at once (1,728 C at 6 A,
// where more wavefronts hide them: 293k -> 289k).
template <int MR, typename W, typename ST>
__device__ __forceinline__ void mfma_syrk_nt(int M, int K, const W* __restrict__ A, const W* __restrict__ B, int ld,
                                             ST st) {
    typedef MfmaW<W> Mf;
    typedef W V4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, nwave = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int mt = (M + 16 * MR - 1) / (16 * MR);   // items of MR 16-row strips
    const int nt = (M + 15) / 16;
    const int nch = (K + 15) / 16;
    // MR 16-row strips times NV column tiles (NV = the tiles of the group inside M)
    auto item = [&](int m0, int tc0, auto nvc) {
        constexpr int NV = decltype(nvc)::value;
        typename Mf::acc acc[MR][NV];
#pragma unroll
        for (int x = 0; x < MR; ++x)
#pragma unroll
            for (int c = 0; c < NV; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[x][c][q] = W(0);
        unsigned oa[MR], ob[NV];
#pragma unroll
        for (int x = 0; x < MR; ++x) oa[x] = (unsigned)min(m0 + 16 * x + li, M - 1) * (unsigned)ld;
#pragma unroll
        for (int c = 0; c < NV; ++c) ob[c] = (unsigned)min((tc0 + c) * 16 + li, M - 1) * (unsigned)ld;
        struct Set {
            V4 a[MR], b[NV];
        };
        auto fetch = [&](Set& s, int ch) {
            const unsigned k0 = (unsigned)min(16 * min(ch, nch - 1) + 4 * lk, K - 4);
#pragma unroll
            for (int x = 0; x < MR; ++x) s.a[x] = *reinterpret_cast<const V4*>(A + (oa[x] + k0));
#pragma unroll
            for (int c = 0; c < NV; ++c) s.b[c] = *reinterpret_cast<const V4*>(B + (ob[c] + k0));
            __builtin_amdgcn_sched_barrier(0);
        };
        auto mma = [&](Set& s, int ch) {
#pragma unroll
            for (int x = 0; x < MR; ++x) arrive(s.a[x]);
#pragma unroll
            for (int c = 0; c < NV; ++c) arrive(s.b[c]);
            if (16 * ch + 16 > K) {   // uniform: the last chunk of a K that is no multiple of 16
                const bool in = 16 * ch + 4 * lk < K;
#pragma unroll
                for (int x = 0; x < MR; ++x)
#pragma unroll
                    for (int e = 0; e < 4; ++e) s.a[x][e] = in ? s.a[x][e] : W(0);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int x = 0; x < MR; ++x)
#pragma unroll
                    for (int c = 0; c < NV; ++c) acc[x][c] = Mf::mma(s.a[x][e], s.b[c][e], acc[x][c]);
        };
        if (nch > 0) {   // uniform: with no column there is nothing to clamp the loads to
            Set s0, s1;
            fetch(s0, 0);
            for (int ch = 0; ch < nch; ch += 2) {
                fetch(s1, ch + 1);
                mma(s0, ch);
                fetch(s0, ch + 2);
                if (ch + 1 < nch) mma(s1, ch + 1);   // uniform
            }
        }
#pragma unroll
        for (int x = 0; x < MR; ++x)
#pragma unroll
            for (int c = 0; c < NV; ++c) {
                const int n = (tc0 + c) * 16 + li;
                if (n < M) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int m = m0 + 16 * x + Mf::acc_row(lk, q);
                        if (m < M) st(m, n, acc[x][c][q]);
                    }
                }
            }
    };
    for (int t = wave; t < mt * mt; t += nwave) {
        const int m0 = (t / mt) * 16 * MR;
        const int tc0 = (t % mt) * MR;
        if (16 * tc0 > m0 + 16 * MR - 1) continue;   // wholly above the diagonal
        const int nv = min(MR, nt - tc0);   // uniform over the wavefront
        if (nv >= 3) item(m0, tc0, std::integral_constant<int, MR >= 3 ? 3 : 1>());
        else if (nv == 2) item(m0, tc0, std::integral_constant<int, MR >= 2 ? 2 : 1>());
        else item(m0, tc0, std::integral_constant<int, 1>());
    }
    __syncthreads();
}

// Products with T_LR.  T_LR is stored as one 4-vector per unordered pair of sites, s =
// sqrt(A) rhat and B (block = s s^T + B I, A >= 0), and expanded on the way into the matrix
// cores: a product reads T_LR once and nothing else of size, and with stored elements it
// ran at the rate of those reads (600 KB per product at 91 sites: 112k cycles, 5 TB/s over
// the chip in the Lanczos iteration).  The 4-vectors are 134 KB, about an XCD's L2 over its
// compute units.  They are FP64 on the mixed path too, whose elements are thus formed in FP64
// and rounded once: from FP32 4-vectors the energies of frames with one atom per local SCS
// were 5 % further from FP64 (rms; a dimer's block over its directions 8.9e-8 against 3.2e-8
// with rounded elements and 1.2e-8 now), for 15.71 instead of 15.83 ms on 1,728 C at 6 A.
// out(m, n) = sum_k T[m][k] X[n][k] over k = (site j, component y): a k-step of the MFMA
// takes one component of four sites (lane group lk: site j0 + lk), a chunk three steps.
// X: in LDS where it fits, rows by column and planes by component, X[n ldx + y ldp + j]
// (planes padded with zeros to ldp, a multiple of four chunks); else in global memory by row
// of the block, X[(3 j + y) ldp + n], so that sixteen lanes read one line (by column, 306
// sites per neighbourhood took 41.0 ms for the stage, by row 29.8).  Items of one 16-row strip times NV column tiles; a wavefront takes its
// strips in groups of kDeep chunks, the loads of the next group (clamped indices, no
// conditions: a load in a conditional block is waited for at once) on their way during
// the matrix work of this one.  Strips of 16 rows also spread evenly over the SIMDs (18
// strips at 91 sites: 5, 5, 4, 4), where six 48-row items kept two of eight wavefronts
// idle.  1,728 C at 6 A, per atom: four products 551k -> 396k cycles (FP32, then with FP32
// 4-vectors, 325k -> 257k), the Lanczos iteration's eleven 2,427k -> 1,596k.
constexpr int kDeep = 4;
typedef double LrRec __attribute__((ext_vector_type(4), aligned(16)));   // (as the workspace is)
__device__ inline int tri(int i, int j) {
    const int hi = max(i, j), lo = min(i, j);
    return ((hi * (hi + 1)) >> 1) + lo;
}
template <int NV, bool LDSX, typename W, typename ST>
__device__ __forceinline__ void mfma_strips(int nK, int N, const LrRec* __restrict__ rec, const W* X, int ldx, int ldp,
                                            int tc0, ST st) {
    typedef MfmaW<W> Mf;
    const int lane = threadIdx.x & 63, nwave = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int M = 3 * nK;
    const int mt = (M + 15) / 16, ng = (nK + 4 * kDeep - 1) / (4 * kDeep);
    const int total = (wave < mt ? (mt - wave + nwave - 1) / nwave : 0) * ng;   // groups of this wavefront
    if (total == 0) return;
    auto row_of = [&](int strip) { return min((16 * strip + li) / 3, nK - 1); };
    int ls = wave, lg = 0;   // strip and group of the next loads
    int row = row_of(ls);
    auto fetch = [&](LrRec(&v)[kDeep]) {
#pragma unroll
        for (int j = 0; j < kDeep; ++j) v[j] = rec[(unsigned)tri(row, min(4 * (kDeep * lg + j) + lk, nK - 1))];
        lg = lg + 1 == ng ? 0 : lg + 1;
        ls = lg == 0 ? ls + nwave : ls;
        row = row_of(ls);
    };
    const W* px[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) px[c] = X + (size_t)min(16 * (tc0 + c) + li, N - 1) * ldx;
    typename Mf::acc acc[NV];
    double unit[3];          // the row's component as a unit vector
    auto begin = [&](int strip) {
        const int comp = (16 * strip + li) % 3;
#pragma unroll
        for (int y = 0; y < 3; ++y) unit[y] = comp == y ? 1.0 : 0.0;
#pragma unroll
        for (int c = 0; c < NV; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[c][q] = W(0);
    };
    int cs = wave, cg = 0;   // strip and group in work
    begin(cs);
    LrRec cur[kDeep], nxt[kDeep];
    fetch(cur);
    for (int x = 0; x < total; ++x) {
        fetch(nxt);
#pragma unroll
        for (int j = 0; j < kDeep; ++j) {
            const int site = 4 * (kDeep * cg + j) + lk;
            W b[3][NV];
#pragma unroll
            for (int y = 0; y < 3; ++y)
#pragma unroll
                for (int c = 0; c < NV; ++c) {
                    if constexpr (LDSX) {
                        b[y][c] = px[c][y * ldp + site];
                    } else {
                        const W v = px[c][(3 * min(site, nK - 1) + y) * ldp];
                        b[y][c] = site < nK ? v : W(0);
                    }
                }
            const LrRec r = cur[j];
            const double sx = unit[0] * r[0] + unit[1] * r[1] + unit[2] * r[2];
#pragma unroll
            for (int y = 0; y < 3; ++y) {
                const W t = W(sx * r[y] + unit[y] * r[3]);
#pragma unroll
                for (int c = 0; c < NV; ++c) acc[c] = Mf::mma(t, b[y][c], acc[c]);
            }
        }
        if (++cg == ng) {   // uniform
#pragma unroll
            for (int c = 0; c < NV; ++c) {
                const int n = 16 * (tc0 + c) + li;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int m = 16 * cs + Mf::acc_row(lk, q);
                    if (n < N && m < M) st(m, n, acc[c][q]);
                }
            }
            cg = 0;
            cs += nwave;
            begin(cs);
        }
#pragma unroll
        for (int j = 0; j < kDeep; ++j) cur[j] = nxt[j];
    }
}
// all column tiles, three at a time; ends with a barrier
template <bool LDSX, typename W, typename ST>
__device__ __forceinline__ void product_tlr(int nK, int N, const LrRec* rec, const W* X, int ldx, int ldp, ST st) {
    const int nt = (N + 15) / 16;
    for (int tc0 = 0; tc0 < nt; tc0 += 3) {
        if (nt - tc0 >= 3) mfma_strips<3, LDSX, W>(nK, N, rec, X, ldx, ldp, tc0, st);
        else if (nt - tc0 == 2) mfma_strips<2, LDSX, W>(nK, N, rec, X, ldx, ldp, tc0, st);
        else mfma_strips<1, LDSX, W>(nK, N, rec, X, ldx, ldp, tc0, st);
    }
    __syncthreads();
}
// The operand in LDS: planes of whole groups of chunks, and an odd row stride, so that the
// sixteen columns of a tile start on different banks
__host__ __device__ inline int operand_plane(int nK) { return (nK + 4 * kDeep - 1) / (4 * kDeep) * (4 * kDeep); }
__host__ __device__ inline int operand_ld(int nK) { return (3 * operand_plane(nK)) | 1; }

// 512 threads: the eight wavefronts share the strips of a product (18 at 91 sites) and the 21
// lower-triangle items of Tbar; four, six, twelve and sixteen wavefronts were slower with
// 48-row items in both places (4.42 ms FP64 and 2.62 ms FP32 with eight on 1,728 C atoms).
constexpr int kMbdThreads = 512;

// The dense form: T_LR is stored and every product runs on the matrix cores (the sparse
// forms are in k_mbd_rows.hip).
// TB: the atoms' structures have two-body radii of their own (a separate instantiation,
// so that the other kernel carries none of its registers)
template <typename W, bool TB>
__global__ void __launch_bounds__(kMbdThreads, 1) k_mbd(MbdArgs a, int nkmax, int vlds) {
    extern __shared__ double lds[];
    const int k = a.order[blockIdx.x];
    const int tid = threadIdx.x;
    const Counts cnt = a.counts[k];
    const int nK = cnt.nK, n1 = cnt.n1, nall = cnt.n_all;
    const int N3 = 3 * nK;
    const int nw = a.nw, nq = a.nq, ncol = a.ncol, n_max = a.n_max;
    const int nwe = nq + 1;   // row stride of L.sa and L.ab (nw is that of the SCS arrays)
    const StructInfo& SI = a.sinfo[a.atom_struct[k]];
    const double rs = SI.r_scs;
    const bool fit = a.fit != 0;
    constexpr bool has2b = TB;
    W* const wbase = static_cast<W*>(a.work) + a.work_off[k];
    // vlds: doubles of LDS from the polarisability adjoints on (a multiple of two), which the
    // products' operand takes until those are formed; 0: the operand stays in global memory
    const size_t adj = mbd_adjoint_offset(nkmax, nq);
    MbdLds L = mbd_lds(lds, nkmax, nq, lds + (vlds ? adj + vlds : mbd_site_doubles((size_t)nkmax, nq)), n_max, fit);
    W* const Vl = reinterpret_cast<W*>(lds + ((adj + 1) & ~(size_t)1));
    // c_n at node q: fitted per atom and node, or the common series
    // (fitted: two copies in LDS, [kMaxNmax + 1][nq] here and [nq][kMaxNmax + 1] for the adjoint operands,
    // whose per-element loop keeps one node's coefficients at fixed offsets)
    double* const cfn = L.cf + (size_t)(kMaxNmax + 1) * nq;
    auto cfq = [&](int n, int q) -> double { return fit ? cfn[n * nq + q] : a.coef[n]; };
    const int lane = tid & 63, wave = tid >> 6, nwave = blockDim.x >> 6;
    const Site* S = a.sites + a.site_off[k];
    const double* aloc = a.alpha_loc + a.aloc_off[k];
    // sub-arrays start on multiples of 4 elements (aligned 4-vector loads)
    // Tbar's product runs over u_1 .. u_{n_max-2}: u_0 = e_k only reaches the central block
    // row and column, which are added apart (0 columns for the approximate forces, which
    // have no other part)
    const int na = a.paper ? 0 : max(n_max - 2, 0);
    const int KK = na * ncol, KKp = (KK + 3) / 4 * 4;
    const int N3p = (int)al4(N3);                            // row stride of T and of V^T (zero padded)
    W* T = wbase;                                            // T_LR's 4-vectors, then Tbar
    W* U = T + al4((size_t)N3 * N3p);                        // u_1 .. u_mmax
    W* V = U + al4((size_t)a.mmax * N3 * ncol);              // Lanczos vectors, central terms of Tbar
    W* V2 = V + al4((size_t)ncol * N3p);                     // the products' operand where LDS has no room for it
    W* Pm = V2 + al4((size_t)ncol * N3p);                    // D u_a side by side, a = 1 .. na
    W* Qm = Pm + (size_t)N3 * KKp;                           // W D Z_a side by side
    auto Uat = [&](int m) { return U + (size_t)(m - 1) * N3 * ncol; };

    // --- blend (Sec. III.B, central/local combination) and SCS radii
    for (int s = tid; s < nK; s += blockDim.x) {
        const Site st = S[s];
        L.px[s] = st.x;
        L.py[s] = st.y;
        L.pz[s] = st.z;
        const double r = sqrt(st.x * st.x + st.y * st.y + st.z * st.z);
        const double* cen = a.alpha_loc + a.aloc_off[st.base];  // row 0 = central value
        double fsv = 1.0, dfsv = 0.0;
        if (s == 0) {
            fsv = 0.0;
        } else if (s < n1) {
            const double x = r / rs;
            fsv = 3.0 * x * x - 2.0 * x * x * x;
            dfsv = (6.0 * x - 6.0 * x * x) / rs;
        }
        L.fs[s] = fsv;
        L.dfs[s] = dfsv;
        if (a.lorentz) {
            const double a0 = (s == 0) ? aloc[0] : (s < n1) ? (1.0 - fsv) * aloc[(size_t)s * nw] + fsv * cen[0] : cen[0];
            const double ar = (s == 0) ? aloc[1] : (s < n1) ? (1.0 - fsv) * aloc[(size_t)s * nw + 1] + fsv * cen[1] : cen[1];
            if (!(ar > 0.0 && a0 >= ar)) {   // no real characteristic frequency
                atomicOr(a.err, 8);
                atomicMin(a.err_atom, k);
            }
            L.sa[(size_t)s * nwe] = a0;
            for (int q = 0; q < nq; ++q) {
                const double v = a0 * ar / (a.rho[q] * a0 + (1.0 - a.rho[q]) * ar);
                L.sa[(size_t)s * nwe + 1 + q] = v;
                L.sqa[(size_t)s * nq + q] = sqrt(v);
            }
        } else {
            for (int w = 0; w < nw; ++w) {
                const double al = (s < n1) ? aloc[(size_t)s * nw + w] : 0.0;
                const double v = (s == 0) ? al : (1.0 - fsv) * al + fsv * cen[w];
                L.sa[(size_t)s * nwe + w] = v;
                if (w > 0) L.sqa[(size_t)s * nq + (w - 1)] = sqrt(v);
            }
        }
        L.Rt[s] = a.r0v[st.base] * cbrt(L.sa[(size_t)s * nwe] / a.a0v[st.base]);
    }
    __syncthreads();

    // --- T_LR, one 4-vector per unordered pair (see the products), zero on the diagonal and
    // for uncoupled pairs
    LrRec* const rec = reinterpret_cast<LrRec*>(T);
    for (int p = tid; p < nK * (nK + 1) / 2; p += blockDim.x) {
        int i = (int)((sqrtf(8.0f * (float)p + 1.0f) - 1.0f) * 0.5f);   // an estimate, corrected in integers
        while ((i + 1) * (i + 2) / 2 <= p) ++i;
        while (i * (i + 1) / 2 > p) --i;
        const int j = p - i * (i + 1) / 2;
        LrRec e = {0.0, 0.0, 0.0, 0.0};
        if (i != j) {
            const double v[3] = {L.px[i] - L.px[j], L.py[i] - L.py[j], L.pz[i] - L.pz[j]};
            const double r = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
            const double rcut = j == 0 ? SI.r_mbd1 : SI.r_mbd2;
            if (r < rcut) {
                const LrPair<W> t = lr_pair<W>(W(r), W(a.beta * (L.Rt[i] + L.Rt[j])), W(a.damp_d), W(rcut),
                                               W(a.r_buf));
                const double sA = sqrt(fmax(double(t.A), 0.0)) / r;
                e = LrRec{sA * v[0], sA * v[1], sA * v[2], double(t.B)};
            }
        }
        rec[p] = e;
    }
    __syncthreads();

    // the products' operand: column `col`, site and component of row r
    W* const X = vlds ? Vl : V2;
    const int ldx = vlds ? operand_ld(nK) : 1, ldp = vlds ? operand_plane(nK) : ncol, ldj = vlds ? 1 : 3 * ncol;
    auto operand_at = [&](int r, int col) -> size_t { return (size_t)col * ldx + (r % 3) * ldp + (size_t)(r / 3) * ldj; };
    for (int e = tid; e < (vlds ? ncol * 3 * (ldp - nK) : 0); e += blockDim.x) {   // the planes' padding
        const int row = e / (ldp - nK);
        Vl[(size_t)(row / 3) * ldx + (row % 3) * ldp + nK + e % (ldp - nK)] = W(0);
    }
    // --- u_1 = D T D e_k, V = D u_1
    W* U1 = Uat(1);
    for (int e = tid; e < N3 * ncol; e += blockDim.x) {
        const int row = e / ncol, col = e % ncol;
        const int q = col / 3, c = col % 3, x = row % 3;
        const double sq = L.sqa[(size_t)(row / 3) * nq + q];
        const LrRec t = rec[tri(row / 3, 0)];
        const double tx = x == 0 ? t[0] : x == 1 ? t[1] : t[2], tc = c == 0 ? t[0] : c == 1 ? t[1] : t[2];
        const double u = sq * (tx * tc + (x == c ? t[3] : 0.0)) * L.sqa[q];
        U1[e] = W(u);
        X[operand_at(row, col)] = W(sq * u);
    }
    __syncthreads();
    // --- u_{m+1} = D (T X), then the next operand X = D u_{m+1}
    for (int m = 1; m < a.mmax; ++m) {
        W* Un = Uat(m + 1);
        auto st = [&](int r, int col, W v) {
            Un[(size_t)r * ncol + col] = W(L.sqa[(size_t)(r / 3) * nq + col / 3]) * v;
        };
        // (two calls, so that the compiler knows which memory the operand is in)
        if (vlds) product_tlr<true, W>(nK, ncol, rec, Vl, ldx, ldp, st);
        else product_tlr<false, W>(nK, ncol, rec, V2, ldx, ldp, st);
        if (m + 1 < a.mmax) {
            for (int e = tid; e < nK * ncol; e += blockDim.x) {
                const int i = e / ncol, col = e - i * ncol;
                const W sq = W(L.sqa[(size_t)i * nq + col / 3]);
                const W* u = Un + (size_t)(3 * i) * ncol + col;
                W* x = X + (size_t)col * ldx + (size_t)i * ldj;
                const W u0 = u[0], u1 = u[ncol], u2 = u[2 * ncol];
                x[0] = sq * u0;
                x[ldp] = sq * u1;
                x[2 * ldp] = sq * u2;
            }
            __syncthreads();
        }
    }

    // --- spectrum bounds of G~ at every node (Lanczos) and, with a.fit, the fitted c_n: the
    // vectors in the space of V, the products' operand D v as above
    if (a.lz_steps > 0)
        lanczos_fit<W>(
            a, k, N3, N3p, L, V, [&](int r) { return lanczos_start(SI, k, S[r / 3], r); },
            [&](int q, int r, W v) { X[operand_at(r, q)] = W(L.sqa[(size_t)(r / 3) * nq + q]) * v; },
            [&](const W*, W* wv) {
                auto st = [&](int r, int q, W v) {
                    wv[(size_t)q * N3p + r] = W(L.sqa[(size_t)(r / 3) * nq + q]) * v;
                };
                if (vlds) product_tlr<true, W>(nK, nq, rec, Vl, ldx, ldp, st);   // ends with a barrier
                else product_tlr<false, W>(nK, nq, rec, V2, ldx, ldp, st);
            });

    // --- moments mu_n(q) = <u_a, u_b>, a + b = n: eight moments (consecutive in the
    // node, so that a row's reads are contiguous) per wavefront, eight lanes per moment
    // over rows r = part (mod 8), combined by lane exchanges in a fixed order
    const int nmom = (n_max - 1) * nq;
    for (int g0 = 8 * wave; g0 < nmom; g0 += 8 * nwave) {
        const int t = g0 + (lane & 7), part = lane >> 3;
        double s = 0.0;
        if (t < nmom) {
            const int n = 2 + t / nq, q = t % nq;
            const int ia = n / 2, ib = n - ia;
            const W* ua = Uat(ia);
            const W* ub = Uat(ib);
            for (int row = part; row < N3; row += 8)
                for (int c = 0; c < 3; ++c)
                    s += double(ua[(size_t)row * ncol + 3 * q + c]) * double(ub[(size_t)row * ncol + 3 * q + c]);
        }
        s += __shfl_xor(s, 8);
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (t < nmom && part == 0) L.mu[(2 + t / nq) * nq + t % nq] = s;
    }
    __syncthreads();
    // two-body radii: t2_j = |T2_kj|^2 (into the space of the blend gradients, unused until
    // the force stage), then mu_2 = alpha~_k sum_j alpha~_j t2_j per node, in site order
    // over the lanes of one wavefront per node
    auto t2pair = [&](int i, int j, double& r, double rh[3], LrPair<double>& t) -> bool {
        const double v[3] = {L.px[i] - L.px[j], L.py[i] - L.py[j], L.pz[i] - L.pz[j]};
        r = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
        const double rc = (i == 0 || j == 0) ? SI.r_2b1 : SI.r_2b2;
        if (i == j || !(r < rc)) return false;
        t = lr_pair<double>(r, a.beta * (L.Rt[i] + L.Rt[j]), a.damp_d, rc, a.r_buf);
        rh[0] = v[0] / r;
        rh[1] = v[1] / r;
        rh[2] = v[2] / r;
        return true;
    };
    if (has2b) {
        for (int j = tid; j < nK; j += blockDim.x) {
            double r, rh[3];
            LrPair<double> t;
            L.fg[j] = t2pair(0, j, r, rh, t) ? (t.A + t.B) * (t.A + t.B) + 2.0 * t.B * t.B : 0.0;
        }
        __syncthreads();
        for (int q = wave; q < nq; q += nwave) {
            double x = 0.0;
            for (int j = lane; j < nK; j += 64) x += L.sa[(size_t)j * nwe + 1 + q] * L.fg[j];
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
            if (lane == 0) L.mu[2 * nq + q] = L.sa[1 + q] * x;
        }
        __syncthreads();
    }
    const double wk = a.e_weight ? a.e_weight[k] : 1.0;
    if (tid == 0) {
        double e = 0.0;
        for (int q = 0; q < nq; ++q) {
            double eq = 0.0;
            for (int n = 2; n <= n_max; ++n) eq += cfq(n, q) * L.mu[n * nq + q];
            e += a.wq[q] * eq;
        }
        a.e_atom[k] = e;
    }
    if (!a.forces) return;

    // --- dE/d alpha~_i(w_q) from the moments (row-local Krylov products)
    if (a.paper) {
        // the full n = 2 trace: 2 c_2 sum_j alpha~_j |T_ij|^2, one site per thread over
        // its block row; the central terms of n >= 3 from u_{n-1} and u_1 (this form
        // only: the host never runs the approximate forces with the sparse products)
        for (int i = tid; i < nK; i += blockDim.x) {
            L.ab[(size_t)i * nwe] = 0.0;
            for (int q0 = 0; q0 < nq; q0 += 4) {   // four nodes at a time, |T_ij|^2 formed again for each group
                double acc2[4] = {0.0, 0.0, 0.0, 0.0};
                for (int j = 0; j < nK; ++j) {
                    if (j == i) continue;
                    double nrm = 0.0;
                    if (has2b) {   // |T2_ij|^2 = (A + B)^2 + 2 B^2 of the two-body tensor
                        double r, rh[3];
                        LrPair<double> t;
                        if (t2pair(i, j, r, rh, t)) nrm = (t.A + t.B) * (t.A + t.B) + 2.0 * t.B * t.B;
                    } else {
                        // |T_ij|^2 = (A + B)^2 + 2 B^2, A = |s|^2
                        const LrRec t = rec[tri(i, j)];
                        const double A = t[0] * t[0] + t[1] * t[1] + t[2] * t[2];
                        const double B = t[3];
                        nrm = (A + B) * (A + B) + 2.0 * B * B;
                    }
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        if (q0 + x < nq) acc2[x] += L.sa[(size_t)j * nwe + 1 + q0 + x] * nrm;
                }
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int q = q0 + x;
                    if (q >= nq) continue;
                    double s = 2.0 * cfq(2, q) * acc2[x];
                    double sn = 0.0;
                    for (int n = 3; n <= n_max; ++n) {
                        const W* ua = Uat(n - 1);
                        const W* u1 = Uat(1);
                        double d = (i == 0) ? L.mu[n * nq + q] : 0.0;
                        for (int r = 3 * i; r < 3 * i + 3; ++r)
                            for (int c = 0; c < 3; ++c)
                                d += double(ua[(size_t)r * ncol + 3 * q + c]) * double(u1[(size_t)r * ncol + 3 * q + c]);
                        sn += cfq(n, q) * n * d;
                    }
                    s += sn / L.sa[(size_t)i * nwe + 1 + q];
                    L.ab[(size_t)i * nwe + 1 + q] = wk * a.wq[q] * s;
                }
            }
        }
    } else
    for (int t = tid; t < nK * nwe; t += blockDim.x) {
        const int i = t / nwe, w = t % nwe;
        double v = 0.0;
        if (w > 0) {
            const int q = w - 1;
            double s = 0.0;
            for (int n = 2; n <= n_max; ++n) {
                double sn = (i == 0) ? L.mu[n * nq + q] : 0.0;
                if (n == 2 && has2b) {   // alpha~_k alpha~_i t2_i (the central term is mu_2 itself)
                    if (i > 0) sn = L.sa[1 + q] * L.sa[(size_t)i * nwe + 1 + q] * L.fg[i];
                    s += cfq(n, q) * sn;
                    continue;
                }
                // sum over a = 1 .. n-1 of the row block of u_a u_{n-a}^T: the terms a and
                // n - a are equal, so each unordered pair is formed once
                double pr = 0.0;
                for (int aa = 1; 2 * aa <= n; ++aa) {
                    const W* ua = Uat(aa);
                    const W* ub = Uat(n - aa);
                    double d = 0.0;
                    for (int r = 3 * i; r < 3 * i + 3; ++r)
                        for (int c = 0; c < 3; ++c)
                            d += double(ua[(size_t)r * ncol + 3 * q + c]) * double(ub[(size_t)r * ncol + 3 * q + c]);
                    pr += (2 * aa == n) ? d : 2.0 * d;
                }
                s += cfq(n, q) * (sn + pr);
            }
            v = wk * a.wq[q] * s / L.sa[(size_t)i * nwe + w];
        }
        L.ab[t] = v;
    }
    // --- operands of Tbar = sum_a (D u_a)(W D Z_a)^T, Z_a = sum_b c_{a+b+1} u_b (u_0 = e_k).
    // Away from the central block row and column u_0 vanishes, so the product runs over
    // a, b = 1 .. n_max - 2 only (144 instead of 216 columns at n_max = 6 and 12 nodes),
    // k-contiguous: P[r][(a-1) ncol + col] = sqrt(alpha~_r) u_a[r][col] and
    // Q[s][(a-1) ncol + col] = w_k W_q sqrt(alpha~_s) sum_{b>=1} c_{a+b+1} u_b[s][col].
    // One (row, column) of the Krylov blocks per thread: u_1 .. u_{n_max-1} read once, all
    // na column blocks of P and Q written.  The u_0 terms of Tbar's central block column,
    // entry (row r >= 3, x): w_k sum_q W_q sqrt(alpha~_r alpha~_k) sum_{b>=1} c_{b+1}
    // u_b[r][3q + x] (the approximate forces: b >= 2 with c_{b+1} (b + 1); with two-body
    // radii the n = 2 term is apart), get their summand over q from the same values, into
    // the space of V.  Leaving u_0 out of the product: Tbar 395k -> 293k cycles per atom
    // of 1,728 C at 6 A.
    // (two instantiations: the common series coefficients are kernel arguments at
    // fixed offsets, the fitted ones LDS entries of the column's node)
    auto build_pq = [&](auto coef) {
        for (int e = tid; e < N3 * ncol; e += blockDim.x) {
            const int r = e / ncol, col = e % ncol, q = col / 3;
            const double sq = L.sqa[(size_t)(r / 3) * nq + q];
            const double scale = wk * a.wq[q] * sq;
            double u[kMaxNmax];
#pragma unroll
            for (int b = 1; b < kMaxNmax; ++b) u[b] = (b < n_max) ? double(Uat(b)[(size_t)r * ncol + col]) : 0.0;
            W* pr = Pm + (size_t)r * KKp + col;
            W* qr = Qm + (size_t)r * KKp + col;
            double z0 = 0.0;
#pragma unroll
            for (int b = 1; b < kMaxNmax; ++b) {
                if (a.paper) {
                    if (b > 1) z0 += coef(b + 1, q) * (b + 1) * u[b];
                } else if (!(has2b && b == 1)) {
                    z0 += coef(b + 1, q) * u[b];
                }
            }
            V[e] = W(scale * L.sqa[q] * z0);
#pragma unroll
            for (int aa = 1; aa < kMaxNmax - 1; ++aa) {
                if (aa > na) break;
                double z = 0.0;
#pragma unroll
                for (int b = 1; b < kMaxNmax - 1; ++b)
                    if (b <= n_max - 1 - aa) z += coef(min(aa + b + 1, kMaxNmax), q) * u[b];
                pr[(size_t)(aa - 1) * ncol] = W(sq * u[aa]);
                qr[(size_t)(aa - 1) * ncol] = W(scale * z);
            }
        }
    };
    if (fit) build_pq([&](int n, int q) { return L.cf[q * (kMaxNmax + 1) + n]; });
    else build_pq([&](int n, int) { return a.coef[n]; });
    for (int e = tid; e < N3 * (KKp - KK); e += blockDim.x) {   // padding columns
        const int r = e / (KKp - KK), kk = KK + e % (KKp - KK);
        Pm[(size_t)r * KKp + kk] = W(0);
        Qm[(size_t)r * KKp + kk] = W(0);
    }
    __syncthreads();
    // --- Tbar (overwrites T).  Tbar is symmetric (the terms a, b and b, a of
    // Gbar are transposes of each other), so only blocks on or below the
    // diagonal are formed and read.
    if (a.paper) {   // 2 w_k sum_q c_2(q) W_q D_q^2 T D_q^2 (with two-body radii: apart), the central column below
        // (evaluated again: Tbar takes the space of the 4-vectors)
        const double c2 = 2.0 * wk;
        for (int p = tid; p < nK * nK; p += blockDim.x) {
            const int i = p / nK, j = p % nK;
            if (j > i) continue;
            double blk[9] = {};
            if (j < i && !has2b) {
                const double v[3] = {L.px[i] - L.px[j], L.py[i] - L.py[j], L.pz[i] - L.pz[j]};
                const double r = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
                const double rcut = j == 0 ? SI.r_mbd1 : SI.r_mbd2;
                if (r < rcut) {
                    const LrPair<W> t = lr_pair<W>(W(r), W(a.beta * (L.Rt[i] + L.Rt[j])), W(a.damp_d), W(rcut),
                                                   W(a.r_buf));
                    double f = 0.0;
                    for (int q = 0; q < nq; ++q)
                        f += a.wq[q] * cfq(2, q) * L.sa[(size_t)i * nwe + 1 + q] * L.sa[(size_t)j * nwe + 1 + q];
                    for (int x = 0; x < 3; ++x)
                        for (int y = 0; y < 3; ++y)
                            blk[3 * x + y] =
                                c2 * f * (double(t.A) * (v[x] / r) * (v[y] / r) + (x == y ? double(t.B) : 0.0));
                }
            }
            for (int x = 0; x < 3; ++x)
                for (int y = 0; y < 3; ++y) T[(size_t)(3 * i + x) * N3p + 3 * j + y] = W(blk[3 * x + y]);
        }
        __syncthreads();
    } else {
        mfma_syrk_nt<3, W>(N3, KKp, Pm, Qm, KKp, [&](int r, int s, W v) { T[(size_t)r * N3p + s] = v; });
    }
    for (int e = 9 + tid; e < 3 * N3; e += blockDim.x) {
        W* const t = T + (size_t)(e / 3) * N3p + e % 3;
        double c = 0.0;
        for (int q = 0; q < nq; ++q) c += double(V[(size_t)(e / 3) * ncol + 3 * q + e % 3]);
        *t = W(double(*t) + c);
    }
    __syncthreads();

    // --- pair contraction: dE/dp_i and dE/dR~_i (each unordered pair from both ends)
    const int parts = max(1, min(4, (int)blockDim.x / max(nK, 1)));
    // the two-body term's pair derivative C2 = kappa T2_ij, kappa = 2 w_k sum_q W_q c_2
    // alpha~_i alpha~_j (central pairs; 4 and every pair for the approximate forces),
    // contracted with dT2/dp_i and, through S~, with dT2/dR~
    auto add2b = [&](int i, int j, double g[3], double& Rb) {
        if (!has2b || (!a.paper && i != 0 && j != 0)) return;
        double r, rh[3];
        LrPair<double> t;
        if (!t2pair(i, j, r, rh, t)) return;
        double kap = 0.0;
        for (int q = 0; q < nq; ++q)
            kap += a.wq[q] * cfq(2, q) * L.sa[(size_t)i * nwe + 1 + q] * L.sa[(size_t)j * nwe + 1 + q];
        kap *= (a.paper ? 4.0 : 2.0) * wk;
        double C[9];
        for (int x = 0; x < 3; ++x)
            for (int c = 0; c < 3; ++c) C[3 * x + c] = kap * (t.A * rh[x] * rh[c] + (x == c ? t.B : 0.0));
        double gp[3];
        radial_tensor_grad(rh, r, t.A, t.dA, t.dB, C, gp);
        g[0] += gp[0];
        g[1] += gp[1];
        g[2] += gp[2];
        Rb += a.beta * t.fLR * t.dfS * 2.0 * kap * t.A / (r * r * r);   // <C2, T_dip> = 2 kappa A / r^3
    };
    for (int t = tid; t < nK * parts; t += blockDim.x) {
        const int i = t % nK, part = t / nK;
        double g[3] = {0.0, 0.0, 0.0};
        double Rb = 0.0;
        for (int j = part; j < nK; j += parts) {
            if (j == i) continue;
            const double v[3] = {L.px[i] - L.px[j], L.py[i] - L.py[j], L.pz[i] - L.pz[j]};
            const double r = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
            const double rcut = (i == 0 || j == 0) ? SI.r_mbd1 : SI.r_mbd2;
            if (!(r < rcut)) continue;
            const double rh[3] = {v[0] / r, v[1] / r, v[2] / r};
            const LrPair<W> lp = lr_pair<W>(W(r), W(a.beta * (L.Rt[i] + L.Rt[j])), W(a.damp_d), W(rcut),
                                            W(a.r_buf));
            // C = Tbar_ij + Tbar_ji = Tbar_IJ + Tbar_IJ^T with I > J
            const int I = max(i, j), J = min(i, j);
            double C[9];
            for (int q = 0; q < 3; ++q)
                for (int c = 0; c < 3; ++c)
                    C[3 * q + c] = double(T[(size_t)(3 * I + q) * N3p + 3 * J + c]) +
                                   double(T[(size_t)(3 * I + c) * N3p + 3 * J + q]);
            double gp[3];
            radial_tensor_grad(rh, r, double(lp.A), double(lp.dA), double(lp.dB), C, gp);
            g[0] += gp[0];
            g[1] += gp[1];
            g[2] += gp[2];
            // <C, T_ij> with T = (3 rhat rhat^T - I)/r^3, times fLR df/dS~
            double rCr = 0.0;
            for (int q = 0; q < 3; ++q)
                for (int c = 0; c < 3; ++c) rCr += rh[q] * C[3 * q + c] * rh[c];
            const double ct = (3.0 * rCr - (C[0] + C[4] + C[8])) / (r * r * r);
            Rb += a.beta * double(lp.fLR) * double(lp.dfS) * ct;
        }
        L.g[(size_t)(part * nK + i) * 3 + 0] = g[0];
        L.g[(size_t)(part * nK + i) * 3 + 1] = g[1];
        L.g[(size_t)(part * nK + i) * 3 + 2] = g[2];
        L.rb[(size_t)part * nK + i] = Rb;
    }
    __syncthreads();
    if (has2b) {   // the two-body term's pairs, each from both ends, one site per thread
        for (int i = tid; i < nK; i += blockDim.x) {
            double g[3] = {0.0, 0.0, 0.0}, Rb = 0.0;
            if (a.paper || i == 0)
                for (int j = 0; j < nK; ++j) add2b(i, j, g, Rb);
            else
                add2b(i, 0, g, Rb);
            L.g[(size_t)i * 3 + 0] += g[0];
            L.g[(size_t)i * 3 + 1] += g[1];
            L.g[(size_t)i * 3 + 2] += g[2];
            L.rb[i] += Rb;
        }
        __syncthreads();
    }
    // reduce the parts in a fixed order; R~ adjoint into alpha~(0); blend adjoint
    double* abl = a.abar_loc + a.aloc_off[k];
    double* cap = a.ca + a.site_off[k] * nw;
    for (int i = tid; i < nK; i += blockDim.x) {
        double g0 = 0.0, g1 = 0.0, g2 = 0.0, Rb = 0.0;
        for (int part = 0; part < parts; ++part) {
            g0 += L.g[(size_t)(part * nK + i) * 3 + 0];
            g1 += L.g[(size_t)(part * nK + i) * 3 + 1];
            g2 += L.g[(size_t)(part * nK + i) * 3 + 2];
            Rb += L.rb[(size_t)part * nK + i];
        }
        // R~_i = R0 (alpha~_i(0)/alpha0)^(1/3): dR~/d alpha~(0) = R~ / (3 alpha~(0))
        L.ab[(size_t)i * nwe] += Rb * L.Rt[i] / (3.0 * L.sa[(size_t)i * nwe]);
        const Site st = S[i];
        const double* cen = a.alpha_loc + a.aloc_off[st.base];
        if (a.lorentz) {
            // back through the two-point model onto alpha~_i(0) and alpha~_i(w_ref)
            const double fsv = L.fs[i];
            const double a0 = L.sa[(size_t)i * nwe];
            const double ar = (i == 0) ? aloc[1] : (i < n1) ? (1.0 - fsv) * aloc[(size_t)i * nw + 1] + fsv * cen[1] : cen[1];
            double b0 = L.ab[(size_t)i * nwe], br = 0.0;
            for (int q = 0; q < nq; ++q) {
                const double v = L.sa[(size_t)i * nwe + 1 + q], g = L.ab[(size_t)i * nwe + 1 + q];
                b0 += g * (1.0 - a.rho[q]) * (v / a0) * (v / a0);
                br += g * a.rho[q] * (v / ar) * (v / ar);
            }
            L.ab[(size_t)i * nwe] = b0;
            L.ab[(size_t)i * nwe + 1] = br;
        }
        double gf = 0.0;  // sum_w abar_i(w) (alpha~_I,i(w) - alpha~_K,i(w))
        for (int w = 0; w < nw; ++w) {
            const double ai = L.ab[(size_t)i * nwe + w];
            // (the approximate forces hold the central polarisabilities fixed: nothing is scattered)
            if (i == 0) {
                abl[w] = ai;
                cap[w] = 0.0;
            } else if (i < n1) {
                abl[(size_t)i * nw + w] = (1.0 - L.fs[i]) * ai;
                cap[(size_t)i * nw + w] = a.paper ? 0.0 : L.fs[i] * ai;
                gf += ai * (cen[w] - aloc[(size_t)i * nw + w]);
            } else {
                cap[(size_t)i * nw + w] = a.paper ? 0.0 : ai;
            }
        }
        // f_SCS(r_ik), r_ik = |p_i| (the central atom sits at the origin)
        double fg[3] = {0.0, 0.0, 0.0};
        if (i > 0 && i < n1) {
            const double r = sqrt(L.px[i] * L.px[i] + L.py[i] * L.py[i] + L.pz[i] * L.pz[i]);
            const double c = L.dfs[i] * gf / r;
            fg[0] = c * L.px[i];
            fg[1] = c * L.py[i];
            fg[2] = c * L.pz[i];
        }
        L.fg[(size_t)i * 3 + 0] = fg[0];
        L.fg[(size_t)i * 3 + 1] = fg[1];
        L.fg[(size_t)i * 3 + 2] = fg[2];
        L.g[(size_t)i * 3 + 0] = g0 + fg[0];
        L.g[(size_t)i * 3 + 1] = g1 + fg[1];
        L.g[(size_t)i * 3 + 2] = g2 + fg[2];
    }
    // local polarisabilities of K1 sites outside K carry no energy adjoint
    for (int e = tid; e < (n1 > nK ? (n1 - nK) * nw : 0); e += blockDim.x) abl[(size_t)nK * nw + e] = 0.0;
    __syncthreads();
    double* out = a.cf0 + a.site_off[k] * 3;
    const double fconv = -1.0 / kBohr;  // force = -dE/dx per Angstrom
    if (wave == 0) {
        // moving the central atom changes every r_ik of the blend
        double c[3] = {0.0, 0.0, 0.0};
        for (int i = 1 + lane; i < nK; i += 64)
            for (int d = 0; d < 3; ++d) c[d] += L.fg[(size_t)i * 3 + d];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1)
            for (int d = 0; d < 3; ++d) c[d] += __shfl_xor(c[d], o);
        if (lane < 3) out[lane] = fconv * (L.g[lane] - (lane == 0 ? c[0] : lane == 1 ? c[1] : c[2]));
    }
    for (int s = 1 + tid; s < nall; s += blockDim.x) {
        const bool in = s < nK;
        double* const o = out + 3 * (size_t)s;
        o[0] = in ? fconv * L.g[(size_t)s * 3 + 0] : 0.0;
        o[1] = in ? fconv * L.g[(size_t)s * 3 + 1] : 0.0;
        o[2] = in ? fconv * L.g[(size_t)s * 3 + 2] : 0.0;
    }
    for (int e = tid; e < (nall - nK) * nw; e += blockDim.x) cap[(size_t)nK * nw + e] = 0.0;
}

hipError_t launch_mbd_dense(hipStream_t st, const MbdArgs& a, int nkmax, bool mixed, bool two_body) {
    size_t lds = mbd_lds_bytes(nkmax, a.nq, a.n_max, a.lz_steps, a.fit != 0);
    const dim3 grid(a.n), blk(kMbdThreads);
    // the products' operand in LDS where it fits: in all of it (FP64, one workgroup per compute
    // unit by its registers: up to 147 sites at 12 nodes) or in half (FP32, two workgroups: up
    // to 118 sites; one workgroup with the operand in LDS ran slower than two without)
    const size_t wsz = mixed ? sizeof(float) : sizeof(double);
    const int ldv = operand_ld(nkmax);
    const size_t adj = mbd_adjoint_offset(nkmax, a.nq);
    const size_t own = mbd_site_doubles((size_t)nkmax, a.nq) - adj;                // adjoints, reduction parts, gradients
    const size_t op = (wsz * (size_t)a.ncol * ldv + sizeof(double) - 1) / sizeof(double) + 1;   // (+ 1: 16-byte start)
    int vlds = (int)((std::max(own, op) + 1) & ~(size_t)1);
    const size_t with = sizeof(double) * (adj + vlds + mbd_small_doubles(a.nq, a.n_max, a.lz_steps, a.fit != 0));
    if (with <= (mixed ? kLdsBytes / 2 : kLdsBytes)) lds = with;
    else vlds = 0;
    if (mixed) {
        if (two_body) hipLaunchKernelGGL((k_mbd<float, true>), grid, blk, lds, st, a, nkmax, vlds);
        else hipLaunchKernelGGL((k_mbd<float, false>), grid, blk, lds, st, a, nkmax, vlds);
    } else {
        if (two_body) hipLaunchKernelGGL((k_mbd<double, true>), grid, blk, lds, st, a, nkmax, vlds);
        else hipLaunchKernelGGL((k_mbd<double, false>), grid, blk, lds, st, a, nkmax, vlds);
    }
    return hipGetLastError();
}

}  // namespace lmbd
