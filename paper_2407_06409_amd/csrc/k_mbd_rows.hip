// Local MBD energy and its adjoint in the two-radius regime (Sec. III.A: a site couples to
// the central atom up to r_MBD,1 but to the others only up to r_MBD,2, so the block rows
// of T_LR other than the central one are sparse).  The quantities are those of the dense
// form (k_mbd.hip); here T_LR is kept as lists of coupled sites and one atom is spread
// over many workgroups, one launch per step:
//   k_rows_setup     site order, blend, SCS radii                     one workgroup per atom
//   k_rows_lists     coupled-site lists, u_1                          three rows per wavefront
//   k_rows_product   u_{m+1} = D T D u_m                              three rows per wavefront
//   k_rows_energy    spectrum bounds, moments, energy                 one workgroup per atom
//   k_rows_operands  polarisability adjoints, operands of Tbar        a (site, node) per lane
//   k_rows_pairs     Tbar and gradient of every coupled pair          three rows per wavefront
//   k_rows_sums      pair terms summed per site                       three rows per wavefront
//   k_rows_final     blend adjoint, outputs                           one workgroup per atom
// All of it is bound by gathers of the partners' rows.  What makes them cheap is where they
// hit: the sites are ordered along a space-filling curve, so that the rows at work share
// most of their partners, and the workgroups of one atom are dealt to one XCD one atom
// after the other, so that this atom's Krylov block (2.1 MB of FP64 for 2,450 sites) and
// not those of 32 atoms is what the XCD's L2 has to hold.  What is left is then the rate
// at which the L1 returns data, so rows go through the products and the pair sums three at
// a time: neighbours on the curve share two thirds of their partners, and a partner's row
// is loaded once for the three.
//
// Storage per atom (RowsLayout): the Krylov blocks scaled, P_m = D u_m, which are the
// products' operands and Tbar's left operand at once; moments and adjoints divide by
// alpha~ where they need u itself.
#include <algorithm>
#include <type_traits>

#include "mbd_common.h"

namespace lmbd {

constexpr int kRowsThreads = 256;    // row kernels: four wavefronts
constexpr int kRowsWaves = kRowsThreads / 64;
constexpr int kAtomThreads = 1024;   // one-workgroup-per-atom kernels
constexpr int kBox = 16;             // slots per bounding box
constexpr int kTriple = 3;           // rows taken together: group 0 is the central row, group t >= 1
                                     // rows 1 + 3 (t - 1) .. (nK + 1) / 3 groups in all
constexpr int kSlotBits = 15;        // a union entry is slot | (bit per row of the group) << kSlotBits
static_assert(kMaxSites <= (1 << kSlotBits), "slots fit their field");

// What every kernel of this file derives from its atom.
template <typename W>
struct RowsAtom {
    typedef W W4 __attribute__((ext_vector_type(4), aligned(16)));   // (as the workspace is)
    typedef double T4 __attribute__((ext_vector_type(4), aligned(16)));
    static constexpr bool kPacked = sizeof(W) < sizeof(double);   // pair terms side by side, see term0
    int k, nK, n1, nall, N3, N3p, nq, nwe, nw, ncol, na, ldq, stride, nbox;
    const StructInfo* SI;
    const Site* S;
    MbdLds L;             // site arrays, in the workspace
    int32_t* slot_site;   // site of each slot
    uint32_t* keys;       // curve keys per site (setup only)
    int32_t* low;         // kPacked, in the place of the keys: places of the rows' first pair terms
    double* boxes;        // bounding boxes of kBox slots
    W4* rec;              // list entries: s = sqrt(A) rhat and B (T_LR = s s^T + B I; A >= 0)
    T4* term;             // pair terms, in the place of rec after the products
    size_t cap;           // entries that the lists have space for
    int32_t* pj;          // list entries: slot, ascending in each row
    int32_t* uni;         // per group, from its first row's place: the union of its rows' entries, ascending
    int32_t* len;         // entries per row
    int32_t* ulen;        // union entries per group
    W *P, *V, *Q;         // P: block m - 1 holds D u_m
    __device__ W* block(int m) const { return P + (size_t)(m - 1) * N3 * ncol; }
    __device__ size_t row0(int i) const { return i == 0 ? 0 : (size_t)nK + (size_t)(i - 1) * stride; }
    // Place of row i's first pair term (a pair's term belongs to the higher of its slots, whose
    // row has it among its first entries).  Terms are FP64 on both paths and take the space of
    // the 4-vectors: entry by entry where those are FP64 too, side by side where those have
    // half the size, as every pair has two entries and one term.  (Terms rounded to FP32 are
    // what the sums' FP64 would be lost on: forces of frames with one atom per local SCS at
    // 6 + 3 A were 0.7 % further from FP64 in rms.  FP64 terms cost the mixed path 0 .. 1 %:
    // 256 C at 10 + 8 A 27.7 -> 28.0 ms.)
    __device__ size_t term0(int i) const { return kPacked ? (size_t)low[i] : row0(i); }
    __device__ size_t terms() const { return kPacked ? cap / 2 : cap; }
};

// The atom and part of workgroup b when every atom has `parts` workgroups: an atom's
// workgroups all on one XCD (workgroups go to the eight XCDs in turn), one after the other.
__device__ inline void rows_place(int b, int parts, int& slot, int& part) {
    const int xcd = b & 7, loc = b >> 3;
    slot = (loc / parts) * 8 + xcd;
    part = loc % parts;
}

template <typename W>
__device__ inline RowsAtom<W> rows_atom(const MbdArgs& a, int k, double* small) {
    RowsAtom<W> R;
    const Counts cnt = a.counts[k];
    R.k = k;
    R.nK = cnt.nK;
    R.n1 = cnt.n1;
    R.nall = cnt.n_all;
    R.N3 = 3 * R.nK;
    R.N3p = (R.N3 + 3) / 4 * 4;
    R.nq = a.nq;
    R.nwe = a.nq + 1;
    R.nw = a.nw;
    R.ncol = a.ncol;
    R.na = a.forces ? max(a.n_max - 2, 0) : 0;
    R.ldq = R.na * a.ncol;
    R.SI = &a.sinfo[a.atom_struct[k]];
    R.S = a.sites + a.site_off[k];
    R.stride = rows_stride(R.nK, R.SI->m2max);
    const RowsLayout G = rows_layout(R.nK, R.SI->m2max, R.nq, a.n_max, a.mmax, (int64_t)sizeof(W), a.forces != 0);
    W* const w = static_cast<W*>(a.work) + a.work_off[k];
    R.L = mbd_lds(reinterpret_cast<double*>(w + G.sites), R.nK, R.nq, small, a.n_max, a.fit != 0);
    // slots, keys and boxes take the parts of L.rb beyond the first
    R.slot_site = reinterpret_cast<int32_t*>(R.L.rb + R.nK);
    R.keys = reinterpret_cast<uint32_t*>(R.slot_site + R.nK);
    R.low = R.slot_site + R.nK;
    R.boxes = R.L.rb + 2 * (size_t)R.nK;
    R.nbox = (R.nK + kBox - 1) / kBox;
    R.cap = (size_t)rows_cap(R.nK, R.SI->m2max);
    R.rec = reinterpret_cast<typename RowsAtom<W>::W4*>(w + G.lists);
    R.term = reinterpret_cast<typename RowsAtom<W>::T4*>(w + G.lists);
    R.pj = reinterpret_cast<int32_t*>(R.rec + R.cap);
    R.uni = R.pj + R.cap;
    R.len = R.uni + R.cap;
    R.ulen = R.len + R.nK;
    R.P = w + G.P;
    R.V = w + G.V;
    R.Q = w + G.Q;
    return R;
}

// whether the pair (i, j) couples (central pairs out to the two-body radius too: their MBD
// coefficients are 0 there)
template <typename W, bool TB>
__device__ inline bool rows_coupled(const RowsAtom<W>& R, int i, int j, double v[3], double& r) {
    if (j >= R.nK || j == i) return false;
    v[0] = R.L.px[i] - R.L.px[j];
    v[1] = R.L.py[i] - R.L.py[j];
    v[2] = R.L.pz[i] - R.L.pz[j];
    r = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    const StructInfo& SI = *R.SI;
    return r < ((i == 0 || j == 0) ? (TB ? fmax(SI.r_mbd1, SI.r_2b1) : SI.r_mbd1) : SI.r_mbd2);
}

// ---------------------------------------------------------------------------
// Slots along the curve, blended polarisabilities, SCS radii, bounding boxes.
// ---------------------------------------------------------------------------
template <typename W>
__global__ void __launch_bounds__(kAtomThreads) k_rows_setup(MbdArgs a) {
    const int k = a.order[blockIdx.x], tid = threadIdx.x;
    const RowsAtom<W> R = rows_atom<W>(a, k, nullptr);
    const MbdLds& L = R.L;
    const StructInfo& SI = *R.SI;
    const int nK = R.nK, n1 = R.n1, nw = a.nw, nq = a.nq, nwe = R.nwe;
    const double rs = SI.r_scs;
    const double* aloc = a.alpha_loc + a.aloc_off[k];
    // Morton keys of a grid over the ball; the central atom takes slot 0, the others follow
    // by (key, site): a fixed order, found by counting (the neighbourhoods are small)
    auto spread = [](uint32_t x) -> uint32_t {   // bits of x (10) to every third bit
        x &= 0x3ffu;
        x = (x | (x << 16)) & 0x030000ffu;
        x = (x | (x << 8)) & 0x0300f00fu;
        x = (x | (x << 4)) & 0x030c30c3u;
        return (x | (x << 2)) & 0x09249249u;
    };
    const double h = fmax(2.0, SI.r_nbr / 511.0);   // bohr per step of the grid
    auto step = [&](double x) -> uint32_t { return (uint32_t)min(max((int)((x + SI.r_nbr) / h), 0), 1023); };
    for (int s = tid; s < nK; s += blockDim.x)
        R.keys[s] = spread(step(R.S[s].x)) | (spread(step(R.S[s].y)) << 1) | (spread(step(R.S[s].z)) << 2);
    if (tid == 0) R.slot_site[0] = 0;
    __syncthreads();
    for (int s = 1 + tid; s < nK; s += blockDim.x) {
        const uint32_t ks = R.keys[s];
        int rank = 1;
        for (int t = 1; t < nK; ++t) {
            const uint32_t kt = R.keys[t];
            rank += (kt < ks || (kt == ks && t < s)) ? 1 : 0;
        }
        R.slot_site[rank] = s;
    }
    __syncthreads();
    for (int s = tid; s < nK; s += blockDim.x) {
        const int si = R.slot_site[s];
        const Site st = R.S[si];
        L.px[s] = st.x;
        L.py[s] = st.y;
        L.pz[s] = st.z;
        const double r = sqrt(st.x * st.x + st.y * st.y + st.z * st.z);
        const double* cen = a.alpha_loc + a.aloc_off[st.base];  // row 0 = central value
        double fsv = 1.0, dfsv = 0.0;
        if (s == 0) {
            fsv = 0.0;
        } else if (si < n1) {
            const double x = r / rs;
            fsv = 3.0 * x * x - 2.0 * x * x * x;
            dfsv = (6.0 * x - 6.0 * x * x) / rs;
        }
        L.fs[s] = fsv;
        L.dfs[s] = dfsv;
        const double* al = aloc + (size_t)si * nw;
        if (a.lorentz) {
            const double a0 = (s == 0) ? aloc[0] : (si < n1) ? (1.0 - fsv) * al[0] + fsv * cen[0] : cen[0];
            const double ar = (s == 0) ? aloc[1] : (si < n1) ? (1.0 - fsv) * al[1] + fsv * cen[1] : cen[1];
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
                const double lo = (si < n1) ? al[w] : 0.0;
                const double v = (s == 0) ? lo : (1.0 - fsv) * lo + fsv * cen[w];
                L.sa[(size_t)s * nwe + w] = v;
                if (w > 0) L.sqa[(size_t)s * nq + (w - 1)] = sqrt(v);
            }
        }
        L.Rt[s] = a.r0v[st.base] * cbrt(L.sa[(size_t)s * nwe] / a.a0v[st.base]);
    }
    if (nK <= 64) return;   // the lists test every pair: no boxes
    __syncthreads();
    for (int b = tid; b < R.nbox; b += blockDim.x) {
        double lo[3], hi[3];
        for (int s = kBox * b; s < min(kBox * (b + 1), nK); ++s) {
            const double x[3] = {L.px[s], L.py[s], L.pz[s]};
            for (int d = 0; d < 3; ++d) {
                lo[d] = s == kBox * b ? x[d] : fmin(lo[d], x[d]);
                hi[d] = s == kBox * b ? x[d] : fmax(hi[d], x[d]);
            }
        }
        for (int d = 0; d < 3; ++d) {
            R.boxes[6 * b + d] = lo[d];
            R.boxes[6 * b + 3 + d] = hi[d];
        }
    }
}

// ---------------------------------------------------------------------------
// Coupled sites of every block row and their coefficients, ascending in the slot, the
// union of the entries of three rows, and the rows of D u_1 (u_1 = D T D e_k needs the
// central block column only).  A wavefront per group of rows, its lanes testing four boxes
// of 16 slots at a time: the first box (the central atom) and those that reach within
// r_mbd2 of a row (all of them for the central row).  Row i has space for every site
// within r_mbd2 of the structure's fullest atom, so the rows need no counting pass.  The
// coupled pairs wait in a ring in LDS until 64 are there, so that their coefficients are
// evaluated with a pair on every lane (a tenth of the lanes where the pairs were found:
// 988 -> 637 us for 1,728 C at 6 + 3 A, 7.9 -> 5.8 ms for 512 C at 10 + 8 A).
// ---------------------------------------------------------------------------
constexpr int kListRing = 256;   // at most 63 pairs wait when three rows add up to 64 each
template <typename W, bool TB>
__global__ void __launch_bounds__(kRowsThreads, 4) k_rows_lists(MbdArgs a, int parts) {
    int at, part;
    rows_place(blockIdx.x, parts, at, part);
    if (at >= a.n) return;
    typedef typename RowsAtom<W>::W4 W4;
    const RowsAtom<W> R = rows_atom<W>(a, a.order[at], nullptr);
    const MbdLds& L = R.L;
    const StructInfo& SI = *R.SI;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nK = R.nK, nq = a.nq, ncol = a.ncol;
    const double rcull = SI.r_mbd2 * SI.r_mbd2 * (1.0 + 1e-9);
    const int grp = part * kRowsWaves + wave;
    const int i0 = grp == 0 ? 0 : 1 + kTriple * (grp - 1);
    if (i0 >= nK) return;
    const int nr = grp == 0 ? 1 : min(kTriple, nK - i0);
    const int cap = grp == 0 ? nK : R.stride;
    const unsigned long long below = (1ull << lane) - 1ull;
    __shared__ int ring_all[kRowsWaves][2][kListRing];   // slot and row of the group; place in the lists
    __shared__ double first_all[kRowsWaves][kTriple][4];
    int(*const ring)[kListRing] = ring_all[wave];
    double(*const first)[4] = first_all[wave];           // the entry of the central atom, per row
    int n[kTriple] = {0, 0, 0}, nu = 0, head = 0, tail = 0;
    for (int e = lane; e < 4 * kTriple; e += 64) first[e / 4][e % 4] = 0.0;
    // the coefficients of up to 64 waiting pairs
    auto evaluate = [&](int cnt) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        if (lane < cnt) {
            const int p = (head + lane) % kListRing;
            const int ent = ring[0][p], e = ring[1][p];
            const int j = ent & ((1 << kSlotBits) - 1), x = ent >> kSlotBits, i = i0 + x;
            double v[3], r;
            (void)rows_coupled<W, TB>(R, i, j, v, r);
            const double rcut = (i == 0 || j == 0) ? SI.r_mbd1 : SI.r_mbd2;
            const LrPair<W> t = lr_pair<W>(W(r), W(a.beta * (L.Rt[i] + L.Rt[j])), W(a.damp_d), W(rcut), W(a.r_buf));
            const double sA = sqrt(fmax(double(t.A), 0.0)) / r;
            const double u[4] = {sA * v[0], sA * v[1], sA * v[2], double(t.B)};
            const W4 rec = {W(u[0]), W(u[1]), W(u[2]), W(u[3])};
            if (e >= 0) {
                R.rec[R.row0(i) + e] = rec;
                R.pj[R.row0(i) + e] = j;
            }
            if (j == 0)
#pragma unroll
                for (int c = 0; c < 4; ++c) first[x][c] = u[c];   // (u_1 is rounded once, at its end)
        }
        head += cnt;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    };
    for (int b0 = 0; b0 < R.nbox; b0 += 64) {
        const int b = b0 + lane;
        bool near = b < R.nbox;
        if (near && grp != 0 && b != 0 && nK > 64) {
            const double* bx = R.boxes + 6 * b;
            near = false;
            for (int x = 0; x < nr; ++x) {
                const int i = i0 + x;
                const double dx = fmax(0.0, fmax(bx[0] - L.px[i], L.px[i] - bx[3]));
                const double dy = fmax(0.0, fmax(bx[1] - L.py[i], L.py[i] - bx[4]));
                const double dz = fmax(0.0, fmax(bx[2] - L.pz[i], L.pz[i] - bx[5]));
                near = near || dx * dx + dy * dy + dz * dz < rcull;
            }
        }
        unsigned long long m = __ballot(near);
        while (m) {
            int box = 0;
            bool have = false;
#pragma unroll
            for (int u = 0; u < 64 / kBox; ++u) {   // the next four near boxes
                const int bit = m ? __ffsll((long long)m) - 1 : -1;
                m &= m - 1;
                if (lane / kBox == u) {
                    have = bit >= 0;
                    box = b0 + max(bit, 0);
                }
            }
            const int j = have ? kBox * box + lane % kBox : nK;
            int bits = 0;
#pragma unroll
            for (int x = 0; x < kTriple; ++x) {
                if (x >= nr) continue;   // uniform
                double v[3], r;
                const bool in = rows_coupled<W, TB>(R, i0 + x, j, v, r);
                const unsigned long long mask = __ballot(in);
                const int off = __popcll(mask & below);
                if (in) {
                    bits |= 1 << x;
                    ring[0][(tail + off) % kListRing] = j | (x << kSlotBits);
                    ring[1][(tail + off) % kListRing] = n[x] + off < cap ? n[x] + off : -1;
                }
                n[x] += __popcll(mask);
                tail += __popcll(mask);
            }
            const unsigned long long any = __ballot(bits != 0);
            const int at_u = nu + __popcll(any & below);
            if (bits != 0 && at_u < nr * cap) R.uni[R.row0(i0) + at_u] = j | (bits << kSlotBits);
            nu += __popcll(any);
            while (tail - head >= 64) evaluate(64);
        }
    }
    if (tail > head) evaluate(tail - head);
#pragma unroll
    for (int x = 0; x < kTriple; ++x) {
        if (x >= nr) continue;
        const int i = i0 + x;
        if (n[x] > cap && lane == 0) {   // the row outgrew its bound: refuse the call
            atomicOr(a.err, 32);
            atomicMin(a.err_atom, R.k);
        }
        if (lane == 0) R.len[i] = min(n[x], cap);
        const double r0 = first[x][0], r1 = first[x][1], r2 = first[x][2], r3 = first[x][3];   // zero if not coupled
        for (int col = lane; col < ncol; col += 64) {
            const int q = col / 3, c = col % 3;
            const double si = L.sqa[(size_t)i * nq + q];
            const double s = si * si * L.sqa[q], rc = c == 0 ? r0 : c == 1 ? r1 : r2;
            for (int y = 0; y < 3; ++y)
                R.P[(size_t)(3 * i + y) * ncol + col] =
                    W(s * ((y == 0 ? r0 : y == 1 ? r1 : r2) * rc + (y == c ? r3 : 0.0)));
        }
    }
    // (an entry beyond a row's capacity is in no list: the products would read past it)
    if (lane == 0) R.ulen[grp] = (n[0] > cap || n[1] > cap || n[2] > cap) ? 0 : nu;
}

// ---------------------------------------------------------------------------
// D u_{m+1} = D^2 T (D u_m), three block rows per wavefront.  A wavefront holds ng groups
// of nl lanes, a lane VW consecutive columns (16-byte loads: 18 lanes and three groups for
// 36 FP64 columns, nine and seven for FP32).  The union of the rows' entries is taken 64
// at a time: every lane brings one entry's coefficients for the three rows to LDS (zero for
// a row that it is not in), then each group walks every ng-th entry, loading the partner's
// rows once for its three accumulators.  The groups' parts are summed through LDS in order.
// One row per group, with its entries read by every lane of it, was bound by the L1's
// return rate (84 cycles for three entries, 32 of them for the coefficients): 512 C at
// 10 + 8 A 15.6 -> 8.0 ms per product.
// ---------------------------------------------------------------------------
template <typename W>
static size_t rows_product_lds(int ncol) {   // per wavefront: the window, or the groups' parts
    const int vw = 16 / (int)sizeof(W), nlt = ncol / (ncol % vw ? 1 : vw), nl = std::min(nlt, 64), ng = 64 / nl;
    return std::max<size_t>(64 * (kTriple * 4 * sizeof(W) + 4), (size_t)ng * 9 * nl * (ncol % vw ? 1 : vw) * sizeof(W));
}

template <typename W, int VW>
__global__ void __launch_bounds__(kRowsThreads) k_rows_product(MbdArgs a, int parts, int m, int lds_wave) {
    extern __shared__ double lds[];
    int at, part;
    rows_place(blockIdx.x, parts, at, part);
    if (at >= a.n) return;
    typedef typename RowsAtom<W>::W4 W4;
    typedef W VV __attribute__((ext_vector_type(VW)));
    const RowsAtom<W> R = rows_atom<W>(a, a.order[at], nullptr);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nK = R.nK, ncol = a.ncol;
    const int nlt = ncol / VW;                           // lanes of all columns
    const int nl = min(nlt, 64), ng = 64 / nl;
    const int ngrp = (nK + 1) / kTriple + 1;             // the central row, then three rows each
    const int it = part * kRowsWaves + wave;
    const int grp = it % ngrp, chunk = it / ngrp;
    const int i0 = grp == 0 ? 0 : 1 + kTriple * (grp - 1);
    if (chunk * 64 >= nlt || i0 >= nK) return;
    const int nr = grp == 0 ? 1 : min(kTriple, nK - i0);
    const int g = lane / nl;
    const int cl = chunk * 64 + lane - g * nl;
    const bool act = g < ng && cl < nlt;
    const int col = act ? VW * cl : 0;
    char* const mine = reinterpret_cast<char*>(lds) + (size_t)wave * lds_wave;
    W4* const wrec = reinterpret_cast<W4*>(mine);                    // [64][kTriple]
    int* const wj = reinterpret_cast<int*>(wrec + 64 * kTriple);     // [64]
    const W* const vc = R.block(m) + col;
    const int nu = R.ulen[grp];
    size_t e0[kTriple];                                  // next entry of each row
#pragma unroll
    for (int x = 0; x < kTriple; ++x) e0[x] = R.row0(min(i0 + x, nK - 1));
    const size_t u0 = R.row0(i0);
    VV acc[kTriple][3];
#pragma unroll
    for (int x = 0; x < kTriple; ++x)
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[x][c] = VV(W(0));
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int t0 = 0; t0 < nu; t0 += 64) {
        const int cnt = min(64, nu - t0);
        const int ent = lane < cnt ? R.uni[u0 + t0 + lane] : 0;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // the last window has been read
        wj[lane] = ent & ((1 << kSlotBits) - 1);
#pragma unroll
        for (int x = 0; x < kTriple; ++x) {
            const bool in = (ent >> (kSlotBits + x)) & 1;
            const unsigned long long mask = __ballot(in);
            W4 r = {W(0), W(0), W(0), W(0)};
            if (in) r = R.rec[e0[x] + __popcll(mask & below)];
            wrec[lane * kTriple + x] = r;
            e0[x] += __popcll(mask);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        for (int s = g; s < cnt; s += ng) {
            const W* v = vc + (size_t)(3 * wj[s]) * ncol;
            const VV x0 = *reinterpret_cast<const VV*>(v), x1 = *reinterpret_cast<const VV*>(v + ncol),
                     x2 = *reinterpret_cast<const VV*>(v + 2 * ncol);
#pragma unroll
            for (int x = 0; x < kTriple; ++x) {
                const W4 r = wrec[s * kTriple + x];
                const VV d = r[0] * x0 + r[1] * x1 + r[2] * x2;
                acc[x][0] += r[0] * d + r[3] * x0;
                acc[x][1] += r[1] * d + r[3] * x1;
                acc[x][2] += r[2] * d + r[3] * x2;
            }
        }
    }
    // the groups' parts, in order: part g, row x, component c at ((g * 9 + 3x + c) nl + lane) VV
    VV* const red = reinterpret_cast<VV*>(mine);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    if (g < ng)
#pragma unroll
        for (int y = 0; y < 9; ++y) red[(g * 9 + y) * nl + lane - g * nl] = acc[y / 3][y % 3];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    // lanes over (row, component, columns)
    for (int e = lane; e < 3 * nr * nl; e += 64) {
        const int y = e / nl, c = chunk * 64 + e % nl;
        if (c >= nlt) continue;
        VV t = red[e];
        for (int gg = 1; gg < ng; ++gg) t += red[gg * 9 * nl + e];
        const int i = i0 + y / 3;
        VV al;
#pragma unroll
        for (int v = 0; v < VW; ++v) al[v] = W(R.L.sa[(size_t)i * R.nwe + 1 + (VW * c + v) / 3]);
        *reinterpret_cast<VV*>(R.block(m + 1) + (size_t)(3 * i0 + y) * ncol + VW * c) = al * t;
    }
}

// T2 of the pair (i, j) at the two-body radii
template <typename W>
__device__ inline bool rows_t2(const MbdArgs& a, const RowsAtom<W>& R, int i, int j, double& r, double rh[3],
                               LrPair<double>& t) {
    const MbdLds& L = R.L;
    const double v[3] = {L.px[i] - L.px[j], L.py[i] - L.py[j], L.pz[i] - L.pz[j]};
    r = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    const double rc = (i == 0 || j == 0) ? R.SI->r_2b1 : R.SI->r_2b2;
    if (i == j || !(r < rc)) return false;
    t = lr_pair<double>(r, a.beta * (L.Rt[i] + L.Rt[j]), a.damp_d, rc, a.r_buf);
    rh[0] = v[0] / r;
    rh[1] = v[1] / r;
    rh[2] = v[2] / r;
    return true;
}

// <u_a, u_b> of site i at node q, times alpha~_i(q)
template <typename W>
__device__ inline double rows_dot(const RowsAtom<W>& R, int i, int q, int x, int y) {
    const size_t o = (size_t)(3 * i) * R.ncol + 3 * q;
    const W *px = R.block(x) + o, *py = R.block(y) + o;
    double d = 0.0;
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) d += double(px[r * R.ncol + c]) * double(py[r * R.ncol + c]);
    return d;
}

// dE/d alpha~_i(w_q) from the moments (row-local Krylov products); mu: the moments (the
// central site only)
template <typename W, bool TB, class CF>
__device__ inline double rows_alpha_adjoint(const MbdArgs& a, const RowsAtom<W>& R, double wk, int i, int q,
                                            const double* mu, CF cfq) {
    const double al = R.L.sa[(size_t)i * R.nwe + 1 + q];
    double s = 0.0;
    for (int n = 2; n <= a.n_max; ++n) {
        const double sn = (i == 0) ? mu[n * R.nq + q] : 0.0;
        if (n == 2 && TB) {   // alpha~_k alpha~_i t2_i (the central term is mu_2 itself)
            s += cfq(n, q) * (i > 0 ? R.L.sa[1 + q] * al * R.L.fg[i] : sn);
            continue;
        }
        // sum over x = 1 .. n-1 of the row block of u_x u_{n-x}^T: the terms x and n - x
        // are equal, so each unordered pair is formed once
        double pr = 0.0;
        for (int x = 1; 2 * x <= n; ++x) {
            const double d = rows_dot(R, i, q, x, n - x);
            pr += (2 * x == n) ? d : 2.0 * d;
        }
        s += cfq(n, q) * (sn + pr / al);
    }
    return wk * a.wq[q] * s / al;
}

// Adjoints of the polarisabilities (sites other than the central one), Q = W D Z and the
// u_0 terms of Tbar's central block column (into V: nine values per site, see k_mbd.hip).
// One (site, node) per lane, 64 / nq sites per wavefront (wavefronts first, first + step,
// ..): its nine values of each Krylov block are read once for all three.  part: nine
// doubles per lane of the wavefront's in LDS, for the sum of the central terms over the
// nodes.  NM: body orders up to NM (register arrays).
template <typename W, bool TB, int NM, class CF>
__device__ inline void rows_operands(const MbdArgs& a, const RowsAtom<W>& R, double wk, int first, int step,
                                        double* part, CF cfq) {
    const MbdLds& L = R.L;
    const int nq = R.nq, ncol = R.ncol, n_max = a.n_max, lane = threadIdx.x & 63;
    const int spw = 64 / nq;                       // nq <= 32
    const int s = lane / nq, q = lane - s * nq;
    for (int i0 = spw * first; i0 < R.nK; i0 += spw * step) {
        const int i = i0 + s;
        if (s < spw && i < R.nK) {
            const double al = L.sa[(size_t)i * R.nwe + 1 + q];
            const double scale = wk * a.wq[q], sc = scale * L.sqa[q];
            double pr[NM + 1];                     // <u_x, u_{n-x}>_i summed over x, times alpha~_i
#pragma unroll
            for (int n = 2; n <= NM; ++n) pr[n] = 0.0;
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                const size_t o = (size_t)(3 * i + r) * ncol + 3 * q;
                double u[NM][3];
#pragma unroll
                for (int b = 1; b < NM; ++b)
#pragma unroll
                    for (int c = 0; c < 3; ++c) u[b][c] = b < n_max ? double(R.block(b)[o + c]) : 0.0;
#pragma unroll
                for (int n = 2; n <= NM; ++n)
#pragma unroll
                    for (int x = 1; 2 * x <= n; ++x)
#pragma unroll
                        for (int c = 0; c < 3; ++c) pr[n] += (2 * x == n ? 1.0 : 2.0) * u[x][c] * u[n - x][c];
                W* qr = R.Q + (size_t)(3 * i + r) * R.ldq + 3 * q;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double z0 = 0.0;
#pragma unroll
                    for (int b = 1; b < NM; ++b)
                        if (b < n_max) z0 += ((TB && b == 1) ? 0.0 : cfq(b + 1, q)) * u[b][c];
                    part[9 * lane + 3 * r + c] = sc * z0;
#pragma unroll
                    for (int x = 1; x < NM - 1; ++x) {
                        double z = 0.0;
#pragma unroll
                        for (int b = 1; x + b < NM; ++b)
                            if (x + b < n_max) z += cfq(x + b + 1, q) * u[b][c];
                        if (x <= R.na) qr[(size_t)(x - 1) * ncol + c] = W(scale * z);
                    }
                }
            }
            if (i > 0) {   // (the central site's with the moments, in k_rows_energy)
                double t = 0.0;
#pragma unroll
                for (int n = 2; n <= NM; ++n) {
                    if (n > n_max) continue;
                    if (TB && n == 2) t += cfq(2, q) * L.sa[1 + q] * al * L.fg[i];   // alpha~_k alpha~_i t2_i
                    else t += cfq(n, q) * (pr[n] / al);
                }
                L.ab[(size_t)i * R.nwe + 1 + q] = scale * t / al;
            }
            if (q == 0) L.ab[(size_t)i * R.nwe] = 0.0;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        for (int e = lane; e < 9 * spw; e += 64) {
            const int se = e / 9;
            if (i0 + se >= R.nK) continue;
            double t = 0.0;
            for (int y = 0; y < nq; ++y) t += part[9 * (se * nq + y) + e % 9];
            R.V[(size_t)9 * (i0 + se) + e % 9] = W(t);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
}
// ---------------------------------------------------------------------------
// Spectrum bounds and fitted coefficients, moments, energy, and the central site's
// adjoints; with fitted coefficients or two-body radii (whose state stays in this
// workgroup) also the operands.
// ---------------------------------------------------------------------------
template <typename W, bool TB, int NM>
__global__ void __launch_bounds__(kAtomThreads) k_rows_energy(MbdArgs a) {
    extern __shared__ double lds[];
    const int k = a.order[blockIdx.x], tid = threadIdx.x;
    const RowsAtom<W> R = rows_atom<W>(a, k, lds);
    const MbdLds& L = R.L;
    const int nK = R.nK, nq = a.nq, n_max = a.n_max, nwe = R.nwe;
    const int lane = tid & 63, wave = tid >> 6, nwave = blockDim.x >> 6;
    const bool fit = a.fit != 0;
    double* const cfn = L.cf + (size_t)(kMaxNmax + 1) * nq;
    auto cfq = [&](int n, int q) -> double { return fit ? cfn[n * nq + q] : a.coef[n]; };
    if (R.kPacked && a.forces) {
        // places of the rows' pair terms: partners below each row (none for a group that outgrew
        // its lists), then their sum over the rows before, by one wavefront
        for (int i = tid; i < nK; i += blockDim.x) {
            const size_t e0 = R.row0(i);
            int lo = 0, hi = R.ulen[(i + kTriple - 1) / kTriple] > 0 ? R.len[i] : 0;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (R.pj[e0 + mid] < i) lo = mid + 1;
                else hi = mid;
            }
            R.low[i] = lo;
        }
        __syncthreads();
    }
    if (R.kPacked && a.forces && wave == nwave - 1) {
        int carry = 0;
        for (int i0 = 0; i0 < nK; i0 += 64) {
            const int v = i0 + lane < nK ? R.low[i0 + lane] : 0;
            int x = v;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_up(x, o);
                if (lane >= o) x += t;
            }
            if (i0 + lane < nK) R.low[i0 + lane] = carry + x - v;
            carry += __shfl(x, 63);
        }
    }
    if (a.lz_steps > 0)
        lanczos_fit<W>(
            a, k, R.N3, R.N3p, L, R.V,
            [&](int r) { return lanczos_start(*R.SI, k, R.S[R.slot_site[r / 3]], r); }, [](int, int, W) {},
            [&](const W* Vin, W* Vout) {
                // one block row per wavefront, lanes over the nodes, the row's sites in order
                const int q = lane < nq ? lane : 0;
                for (int i = wave; i < nK; i += nwave) {
                    const int n = R.len[i];
                    const size_t e0 = R.row0(i);
                    W acc0 = W(0), acc1 = W(0), acc2 = W(0);
                    for (int t = 0; t < n; ++t) {
                        const int j = R.pj[e0 + t];
                        const typename RowsAtom<W>::W4 rc = R.rec[e0 + t];
                        const W sj = W(L.sqa[(size_t)j * nq + q]);
                        const W* x = Vin + (size_t)q * R.N3p + 3 * j;
                        const W x0 = sj * x[0], x1 = sj * x[1], x2 = sj * x[2];
                        const W ax = rc[0] * x0 + rc[1] * x1 + rc[2] * x2;
                        acc0 += ax * rc[0] + rc[3] * x0;
                        acc1 += ax * rc[1] + rc[3] * x1;
                        acc2 += ax * rc[2] + rc[3] * x2;
                    }
                    if (lane < nq) {
                        const W si = W(L.sqa[(size_t)i * nq + q]);
                        W* y = Vout + (size_t)q * R.N3p + 3 * i;
                        y[0] = si * acc0;
                        y[1] = si * acc1;
                        y[2] = si * acc2;
                    }
                }
                __syncthreads();
            });
    // moments mu_n(q) = <u_x, u_y>, x + y = n: eight moments (consecutive in the node) per
    // wavefront, eight lanes per moment over the sites, the wavefronts in `rs` ranges of
    // sites; combined by lane exchanges and over the ranges in a fixed order
    const int nmom = (n_max - 1) * nq;
    const int sets = (nmom + 7) / 8, rs = max(1, nwave / sets);
    double* const parts = lds + mbd_small_doubles(nq, n_max, a.lz_steps, fit);   // [rs][(n_max + 1) nq]
    for (int w0 = wave; w0 < sets * rs; w0 += nwave) {
        const int range = w0 / sets;
        const int t = 8 * (w0 % sets) + (lane & 7), part = lane >> 3;
        double s = 0.0;
        if (t < nmom) {
            const int n = 2 + t / nq, q = t % nq;
            const int ia = n / 2, ib = n - ia;
            for (int i = part + 8 * range; i < nK; i += 8 * rs)
                s += rows_dot(R, i, q, ia, ib) / L.sa[(size_t)i * nwe + 1 + q];
        }
        s += __shfl_xor(s, 8);
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (t < nmom && part == 0) parts[(size_t)range * (n_max + 1) * nq + 2 * nq + t] = s;
    }
    __syncthreads();
    for (int t = 2 * nq + tid; t < (n_max + 1) * nq; t += blockDim.x) {
        double s = 0.0;
        for (int range = 0; range < rs; ++range) s += parts[(size_t)range * (n_max + 1) * nq + t];
        L.mu[t] = s;
    }
    __syncthreads();
    if constexpr (TB) {
        // two-body radii: t2_j = |T2_kj|^2 (into the space of the blend gradients), then
        // mu_2 = alpha~_k sum_j alpha~_j t2_j per node, in site order over the lanes of one
        // wavefront per node
        for (int j = tid; j < nK; j += blockDim.x) {
            double r, rh[3];
            LrPair<double> t;
            L.fg[j] = rows_t2(a, R, 0, j, r, rh, t) ? (t.A + t.B) * (t.A + t.B) + 2.0 * t.B * t.B : 0.0;
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
    if (tid < nq) L.ab[1 + tid] = rows_alpha_adjoint<W, TB>(a, R, wk, 0, tid, L.mu, cfq);
    if (!(fit || TB)) return;   // k_rows_operands follows
    double* const op = parts + (size_t)rs * (n_max + 1) * nq + (size_t)wave * 64 * 9;
    if (fit) rows_operands<W, TB, NM>(a, R, wk, wave, nwave, op, [&](int n, int q) { return L.cf[q * (kMaxNmax + 1) + n]; });
    else rows_operands<W, TB, NM>(a, R, wk, wave, nwave, op, [&](int n, int) { return a.coef[n]; });
    if constexpr (TB) {
        // the two-body term's pair derivative C2 = kappa T2_kj, kappa = 2 w_k sum_q W_q c_2
        // alpha~_k alpha~_j, contracted with dT2/dp and, through S~, with dT2/dR~: the central
        // pairs from both ends; the gradient waits in the space of the blend gradients, the
        // radius term goes straight into the adjoint of alpha~(0)
        __syncthreads();
        for (int i = tid; i < nK; i += blockDim.x) {
            double g[3] = {0.0, 0.0, 0.0}, Rb = 0.0;
            auto add = [&](int j) {
                double r, rh[3];
                LrPair<double> t;
                if (!rows_t2(a, R, i, j, r, rh, t)) return;
                double kap = 0.0;
                for (int q = 0; q < nq; ++q)
                    kap += a.wq[q] * cfq(2, q) * L.sa[(size_t)i * nwe + 1 + q] * L.sa[(size_t)j * nwe + 1 + q];
                kap *= 2.0 * wk;
                double C[9];
                for (int x = 0; x < 3; ++x)
                    for (int c = 0; c < 3; ++c) C[3 * x + c] = kap * (t.A * rh[x] * rh[c] + (x == c ? t.B : 0.0));
                double gp[3];
                radial_tensor_grad(rh, r, t.A, t.dA, t.dB, C, gp);
                for (int d = 0; d < 3; ++d) g[d] += gp[d];
                Rb += a.beta * t.fLR * t.dfS * 2.0 * kap * t.A / (r * r * r);   // <C2, T_dip> = 2 kappa A / r^3
            };
            if (i == 0)
                for (int j = 1; j < nK; ++j) add(j);
            else
                add(0);
            for (int d = 0; d < 3; ++d) L.fg[(size_t)i * 3 + d] = g[d];
            L.ab[(size_t)i * nwe] = Rb * L.Rt[i] / (3.0 * L.sa[(size_t)i * nwe]);
        }
    }
}

template <typename W, int NM>
__global__ void __launch_bounds__(kRowsThreads) k_rows_operands(MbdArgs a, int parts) {
    int at, part;
    rows_place(blockIdx.x, parts, at, part);
    if (at >= a.n) return;
    const int k = a.order[at];
    const RowsAtom<W> R = rows_atom<W>(a, k, nullptr);
    const double wk = a.e_weight ? a.e_weight[k] : 1.0;
    __shared__ double terms[kRowsWaves * 64 * 9];
    const int wave = threadIdx.x >> 6;
    rows_operands<W, false, NM>(a, R, wk, part * kRowsWaves + wave, parts * kRowsWaves, terms + wave * 64 * 9,
                            [&](int n, int) { return a.coef[n]; });
}

// ---------------------------------------------------------------------------
// Each unordered coupled pair once: from row i over its partners j < i, Tbar_ij = P_i Q_j^T
// (and the u_0 terms for j = 0), C = Tbar_ij + Tbar_ij^T, and the pair's terms (its
// gradient with respect to r_i and its R~ term) in FP64 into a buffer in the place of the
// lists' T_LR coefficients (used for the last time by the products; term0).  Three rows per
// wavefront, over the union of their entries: eight entries at a time, eight lanes per
// entry (16 bytes of a row each), the partner's Q loaded once for the three rows' P in LDS;
// the pairs' C wait in LDS so that the evaluation of the radial parts, longer than a
// pair's sums, runs with a pair on every lane.
// ---------------------------------------------------------------------------
constexpr int kPairWindow = 64 / kTriple;   // union entries per window: a lane per pair

template <typename W, int VW>
__global__ void __launch_bounds__(kRowsThreads) k_rows_pairs(MbdArgs a, int parts) {
    extern __shared__ double lds[];
    int at, part;
    rows_place(blockIdx.x, parts, at, part);
    if (at >= a.n) return;
    typedef W VV __attribute__((ext_vector_type(VW)));
    const RowsAtom<W> R = rows_atom<W>(a, a.order[at], nullptr);
    const MbdLds& L = R.L;
    const StructInfo& SI = *R.SI;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
    const int nK = R.nK, KK = R.ldq, ncol = a.ncol;
    double* const cb = lds + (size_t)wave * 64 * 7;      // six values of C per pair, padded to seven
    W* const pi = reinterpret_cast<W*>(lds + nwave * 64 * 7) + (size_t)wave * ((9 * KK + 3) / 4 * 4);
    const int pu = lane >> 3, pt = lane & 7;
    const int grp = 1 + part * nwave + wave;             // (the central row has no partner below)
    const int i0 = 1 + kTriple * (grp - 1);
    if (i0 >= nK) return;
    const int nr = min(kTriple, nK - i0);
    const int nu = R.ulen[grp];
    const size_t u0 = R.row0(i0);
    size_t e0[kTriple];                                  // place of the next entry's term of each row
#pragma unroll
    for (int x = 0; x < kTriple; ++x) e0[x] = R.term0(min(i0 + x, nK - 1));
    for (int e = VW * lane; e < 3 * nr * KK; e += VW * 64) {   // P of the rows: [row][b ncol + col]
        const int row = e / KK, kk = e - row * KK, b = kk / ncol;
        *reinterpret_cast<VV*>(pi + e) =
            *reinterpret_cast<const VV*>(R.block(b + 1) + (size_t)(3 * i0 + row) * ncol + (kk - b * ncol));
    }
    for (int e = 3 * nr * KK + lane; e < 9 * KK; e += 64) pi[e] = W(0);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int t0 = 0; t0 < nu; t0 += kPairWindow) {
        const int cnt = min(kPairWindow, nu - t0);
        const int ent = lane < cnt ? R.uni[u0 + t0 + lane] : 0;
        const int jw = ent & ((1 << kSlotBits) - 1);
        if (__ballot(lane < cnt && jw < i0 + nr - 1) == 0) break;   // ascending: no partner below is left
        // rank of this lane's entry in each row's list
        int rank[kTriple];
#pragma unroll
        for (int x = 0; x < kTriple; ++x) rank[x] = __popcll(__ballot((ent >> (kSlotBits + x)) & 1) & below);
        for (int s0 = 0; s0 < cnt; s0 += 8) {
            const int j = __shfl(jw, min(s0 + pu, cnt - 1));
            const W* qj = R.Q + (size_t)(3 * j) * R.ldq;
            double c[kTriple][6];   // C's 00, 01, 02, 11, 12, 22 (the diagonal halved)
#pragma unroll
            for (int x = 0; x < kTriple; ++x)
#pragma unroll
                for (int y = 0; y < 6; ++y) c[x][y] = 0.0;
            // the next columns of Q are on their way while these are used
            VV qn[3];
            auto fetch = [&](int kk) {
                const int ks = kk < KK ? kk : 0;
#pragma unroll
                for (int d = 0; d < 3; ++d) qn[d] = *reinterpret_cast<const VV*>(qj + (size_t)d * R.ldq + ks);
            };
            if (KK > 0) fetch(VW * pt);
            for (int kk = VW * pt; kk < KK; kk += 8 * VW) {
                const VV qv[3] = {qn[0], qn[1], qn[2]};
                fetch(kk + 8 * VW);
#pragma unroll
                for (int x = 0; x < kTriple; ++x) {
                    VV pv[3];
#pragma unroll
                    for (int y = 0; y < 3; ++y) pv[y] = *reinterpret_cast<const VV*>(pi + (3 * x + y) * KK + kk);
#pragma unroll
                    for (int v = 0; v < VW; ++v) {
                        const double p0 = pv[0][v], p1 = pv[1][v], p2 = pv[2][v];
                        const double q0 = qv[0][v], q1 = qv[1][v], q2 = qv[2][v];
                        c[x][0] += p0 * q0;
                        c[x][1] += p0 * q1;
                        c[x][1] += p1 * q0;
                        c[x][2] += p0 * q2;
                        c[x][2] += p2 * q0;
                        c[x][3] += p1 * q1;
                        c[x][4] += p1 * q2;
                        c[x][4] += p2 * q1;
                        c[x][5] += p2 * q2;
                    }
                }
            }
#pragma unroll
            for (int x = 0; x < kTriple; ++x) {
#pragma unroll
                for (int y = 0; y < 6; ++y) {
                    c[x][y] += __shfl_xor(c[x][y], 1);
                    c[x][y] += __shfl_xor(c[x][y], 2);
                    c[x][y] += __shfl_xor(c[x][y], 4);
                }
                if (pt == 0 && s0 + pu < cnt)
#pragma unroll
                    for (int y = 0; y < 6; ++y) cb[7 * (x * kPairWindow + s0 + pu) + y] = c[x][y];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        // lane x kPairWindow + s: row x, entry s
        const int x = lane / kPairWindow, s = lane - x * kPairWindow;
        const int es = __shfl(ent, s), j = es & ((1 << kSlotBits) - 1);
        const int k0 = __shfl(rank[0], s), k1 = __shfl(rank[1], s), k2 = __shfl(rank[2], s);
        const int i = i0 + x;
        if (x < nr && s < cnt && ((es >> (kSlotBits + x)) & 1) && j < i) {
            const double* c = cb + 7 * lane;
            double C[9] = {2.0 * c[0], c[1], c[2], c[1], 2.0 * c[3], c[4], c[2], c[4], 2.0 * c[5]};
            if (j == 0) {   // the central column's u_0 terms
                const W* t = R.V + (size_t)9 * i;
#pragma unroll
                for (int y = 0; y < 3; ++y)
#pragma unroll
                    for (int z = 0; z < 3; ++z) C[3 * y + z] += double(t[3 * y + z]) + double(t[3 * z + y]);
            }
            const double v[3] = {L.px[i] - L.px[j], L.py[i] - L.py[j], L.pz[i] - L.pz[j]};
            const double r = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
            const double rcut = (i == 0 || j == 0) ? SI.r_mbd1 : SI.r_mbd2;
            const double rh[3] = {v[0] / r, v[1] / r, v[2] / r};
            const LrPair<W> lp = lr_pair<W>(W(r), W(a.beta * (L.Rt[i] + L.Rt[j])), W(a.damp_d), W(rcut), W(a.r_buf));
            double gp[3];
            radial_tensor_grad(rh, r, double(lp.A), double(lp.dA), double(lp.dB), C, gp);
            double rCr = 0.0;
            for (int y = 0; y < 3; ++y)
                for (int z = 0; z < 3; ++z) rCr += rh[y] * C[3 * y + z] * rh[z];
            const double ct = (3.0 * rCr - (C[0] + C[4] + C[8])) / (r * r * r);
            const size_t e = (x == 0 ? e0[0] + k0 : x == 1 ? e0[1] + k1 : e0[2] + k2);
            if (e < R.terms())   // (always, but in a call that is refused for an outgrown list)
                R.term[e] = typename RowsAtom<W>::T4{gp[0], gp[1], gp[2], a.beta * double(lp.fLR) * double(lp.dfS) * ct};
        }
#pragma unroll
        for (int y = 0; y < kTriple; ++y) e0[y] += __popcll(__ballot((ent >> (kSlotBits + y)) & 1));
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
}

// ---------------------------------------------------------------------------
// Every row's pair terms summed over its partners: partner j < i from the row's own slots,
// j > i from the slot in j's row with the gradient's sign turned: it is odd in rhat, the
// R~ term even.  Three rows per wavefront over the union of their entries: lane l takes the
// entries l, l + 64, ..; one binary search in j's sorted row finds the slots of all three
// rows, which follow one another there.  The lanes are combined in a fixed order.
// ---------------------------------------------------------------------------
template <typename W>
__global__ void __launch_bounds__(kRowsThreads) k_rows_sums(MbdArgs a, int parts) {
    int at, part;
    rows_place(blockIdx.x, parts, at, part);
    if (at >= a.n) return;
    const RowsAtom<W> R = rows_atom<W>(a, a.order[at], nullptr);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = part * kRowsWaves + wave;
    const int i0 = grp == 0 ? 0 : 1 + kTriple * (grp - 1);
    if (i0 >= R.nK) return;
    const int nr = grp == 0 ? 1 : min(kTriple, R.nK - i0);
    const int nu = R.ulen[grp];
    const size_t u0 = R.row0(i0);
    const unsigned long long below = (1ull << lane) - 1ull;
    size_t e0[kTriple];
    double g[kTriple][9];
#pragma unroll
    for (int x = 0; x < kTriple; ++x) {
        e0[x] = R.term0(min(i0 + x, R.nK - 1));
#pragma unroll
        for (int y = 0; y < 9; ++y) g[x][y] = 0.0;
    }
    for (int t0 = 0; t0 < nu; t0 += 64) {
        const int ent = t0 + lane < nu ? R.uni[u0 + t0 + lane] : 0;
        const int j = ent & ((1 << kSlotBits) - 1), bits = ent >> kSlotBits;
        size_t up = 0, ut = 0;   // the entry of the first of the rows in j's row, and its term
        int end = 0;
        if (bits != 0 && j > i0) {
            const size_t b = R.row0(j);
            const int n = R.len[j];
            int lo = 0, hi = n;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (R.pj[b + mid] < i0) lo = mid + 1;
                else hi = mid;
            }
            up = b + lo;
            ut = R.term0(j) + lo;
            end = n - lo;
        }
#pragma unroll
        for (int x = 0; x < kTriple; ++x) {
            const bool in = (bits >> x) & 1;
            const unsigned long long mask = __ballot(in);
            const int i = i0 + x;
            if (in) {
                size_t src = e0[x] + __popcll(mask & below);
                double sg = 1.0;
                bool ok = true;
                if (j > i) {
                    ok = end > 0 && R.pj[up] == i;
                    src = ut;
                    sg = -1.0;
                    ++up;
                    ++ut;
                    --end;
                }
                if (ok && src < R.terms()) {
                    const typename RowsAtom<W>::T4 t = R.term[src];
                    g[x][0] += sg * t[0];
                    g[x][1] += sg * t[1];
                    g[x][2] += sg * t[2];
                    g[x][3] += t[3];
                } else {   // the coupling relation is symmetric: never taken
                    atomicOr(a.err, 32);
                    atomicMin(a.err_atom, R.k);
                }
            }
            e0[x] += __popcll(mask);
        }
    }
#pragma unroll
    for (int x = 0; x < kTriple; ++x) {
        if (x >= nr) continue;
        double tot[9];
        wave_sum9(g[x], tot);
        if (lane == 0) {
            const int i = i0 + x;
            R.L.g[(size_t)i * 3 + 0] = tot[0];
            R.L.g[(size_t)i * 3 + 1] = tot[1];
            R.L.g[(size_t)i * 3 + 2] = tot[2];
            R.L.rb[i] = tot[3];
        }
    }
}

// ---------------------------------------------------------------------------
// R~ adjoint into alpha~(0), two-point model, blend adjoint, f_SCS gradients; outputs per site.
// ---------------------------------------------------------------------------
template <typename W, bool TB>
__global__ void __launch_bounds__(kAtomThreads) k_rows_final(MbdArgs a) {
    const int k = a.order[blockIdx.x], tid = threadIdx.x, lane = tid & 63;
    const RowsAtom<W> R = rows_atom<W>(a, k, nullptr);
    const MbdLds& L = R.L;
    const int nK = R.nK, n1 = R.n1, nall = R.nall, nw = a.nw, nq = a.nq, nwe = R.nwe;
    const double* aloc = a.alpha_loc + a.aloc_off[k];
    double* abl = a.abar_loc + a.aloc_off[k];
    double* cap = a.ca + a.site_off[k] * nw;
    double* out = a.cf0 + a.site_off[k] * 3;
    const double fconv = -1.0 / kBohr;  // force = -dE/dx per Angstrom
    for (int i = tid; i < nK; i += blockDim.x) {
        double g[3];
        for (int d = 0; d < 3; ++d) g[d] = L.g[(size_t)i * 3 + d] + (TB ? L.fg[(size_t)i * 3 + d] : 0.0);
        const double a0 = L.sa[(size_t)i * nwe];
        // R~_i = R0 (alpha~_i(0)/alpha0)^(1/3): dR~/d alpha~(0) = R~ / (3 alpha~(0))
        double b0 = L.ab[(size_t)i * nwe] + L.rb[i] * L.Rt[i] / (3.0 * a0), br = 0.0;
        const int si = R.slot_site[i];
        const Site st = R.S[si];
        const double* cen = a.alpha_loc + a.aloc_off[st.base];
        const double* al = aloc + (size_t)si * nw;
        const double fsv = L.fs[i];
        if (a.lorentz) {
            // back through the two-point model onto alpha~_i(0) and alpha~_i(w_ref)
            const double ar = (i == 0) ? aloc[1] : (si < n1) ? (1.0 - fsv) * al[1] + fsv * cen[1] : cen[1];
            for (int q = 0; q < nq; ++q) {
                const double v = L.sa[(size_t)i * nwe + 1 + q], x = L.ab[(size_t)i * nwe + 1 + q];
                b0 += x * (1.0 - a.rho[q]) * (v / a0) * (v / a0);
                br += x * a.rho[q] * (v / ar) * (v / ar);
            }
        }
        double gf = 0.0;  // sum_w abar_i(w) (alpha~_I,i(w) - alpha~_K,i(w))
        for (int w = 0; w < nw; ++w) {
            const double ai = w == 0 ? b0 : a.lorentz ? br : L.ab[(size_t)i * nwe + w];
            if (i == 0) {
                abl[w] = ai;
                cap[w] = 0.0;
            } else if (si < n1) {
                abl[(size_t)si * nw + w] = (1.0 - fsv) * ai;
                cap[(size_t)si * nw + w] = fsv * ai;
                gf += ai * (cen[w] - al[w]);
            } else {
                cap[(size_t)si * nw + w] = ai;
            }
        }
        // f_SCS(r_ik), r_ik = |p_i| (the central atom sits at the origin)
        double fg[3] = {0.0, 0.0, 0.0};
        if (i > 0 && si < n1) {
            const double p[3] = {L.px[i], L.py[i], L.pz[i]};
            const double c = L.dfs[i] * gf / sqrt(p[0] * p[0] + p[1] * p[1] + p[2] * p[2]);
            for (int d = 0; d < 3; ++d) fg[d] = c * p[d];
        }
        for (int d = 0; d < 3; ++d) {
            L.fg[(size_t)i * 3 + d] = fg[d];
            if (i > 0) out[3 * (size_t)si + d] = fconv * (g[d] + fg[d]);
            else L.g[d] = g[d];
        }
    }
    // local polarisabilities of K1 sites outside K carry no energy adjoint
    for (int e = tid; e < (n1 > nK ? (n1 - nK) * nw : 0); e += blockDim.x) abl[(size_t)nK * nw + e] = 0.0;
    __syncthreads();
    if (tid < 64) {
        // moving the central atom changes every r_ik of the blend
        double c[3] = {0.0, 0.0, 0.0};
        for (int i = 1 + lane; i < nK; i += 64)
            for (int d = 0; d < 3; ++d) c[d] += L.fg[(size_t)i * 3 + d];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1)
            for (int d = 0; d < 3; ++d) c[d] += __shfl_xor(c[d], o);
        if (lane < 3) out[lane] = fconv * (L.g[lane] - (lane == 0 ? c[0] : lane == 1 ? c[1] : c[2]));
    }
    for (int e = 3 * nK + tid; e < 3 * nall; e += blockDim.x) out[e] = 0.0;
    for (int e = tid; e < (nall - nK) * nw; e += blockDim.x) cap[(size_t)nK * nw + e] = 0.0;
}

// dynamic LDS (operands: k_rows_energy forms them too)
static size_t rows_energy_lds(const MbdArgs& a, bool operands) {
    const size_t sets = ((size_t)(a.n_max - 1) * a.nq + 7) / 8;
    const size_t rs = std::max<size_t>(1, kAtomThreads / 64 / sets);
    return sizeof(double) * (mbd_small_doubles(a.nq, a.n_max, a.lz_steps, a.fit != 0) + rs * (a.n_max + 1) * a.nq +
                             (operands ? (size_t)kAtomThreads * 9 : 0));
}
static size_t rows_pairs_lds(const MbdArgs& a, size_t wsz) {   // per wavefront
    const size_t KK = (size_t)std::max(a.n_max - 2, 0) * a.ncol;
    return sizeof(double) * 64 * 7 + wsz * ((9 * KK + 3) / 4 * 4);
}

// Atoms of one set of launches of at most `threads` work-items per atom: a launch's work-items
// are counted in 32 bits.  Every atom has the workgroups of the call's largest neighbourhood,
// so one of 31,000 sites (a one-atom cell at 42 A) leaves room for 6,400 atoms.
static int rows_atoms_per_launch(int n, long long threads) {
    return (int)std::min<long long>(n, std::max<long long>(8, 0xffffffffll / threads / 8 * 8));
}

template <typename W, bool TB, int NM>
static hipError_t launch_rows_t(hipStream_t st, const MbdArgs& all, int nkmax) {
    constexpr int VW = 16 / sizeof(W);
    const bool vec = all.ncol % VW == 0;
    auto parts_of = [](int items, int waves) { return (items + waves - 1) / waves; };
    const int groups = (nkmax + 1) / kTriple + 1;                  // three rows per wavefront
    const int rows = parts_of(groups, kRowsWaves);                 // workgroups per atom
    const int nlt = all.ncol / (vec ? VW : 1);
    const int prod = parts_of(groups * ((nlt + 63) / 64), kRowsWaves);
    const int wl = (int)((rows_product_lds<W>(all.ncol) + 15) / 16 * 16);
    const bool operands = all.forces && (all.fit || TB);   // in k_rows_energy
    const int per = 2 * kRowsWaves * (64 / all.nq);        // sites of an operands workgroup: two rounds per wavefront
    const int ops = parts_of(nkmax, per);
    // P of three rows in LDS per wavefront (10 KB at 12 nodes and n_max = 6): small workgroups
    const size_t lw = rows_pairs_lds(all, sizeof(W));
    const int pw = 2 * lw <= 64 * 1024 ? 2 : 1, pr = parts_of(groups, pw);
    const int most = rows_atoms_per_launch(
        all.n, std::max(std::max((long long)kAtomThreads, 64ll * pw * pr), (long long)kRowsThreads * std::max(std::max(rows, prod), ops)));
    for (int first = 0; first < all.n; first += most) {
        MbdArgs a = all;
        a.n = std::min(most, all.n - first);
        a.order = all.order + first;
        const unsigned atoms8 = 8u * (unsigned)((a.n + 7) / 8);
        const dim3 per_atom(a.n);
        hipLaunchKernelGGL((k_rows_setup<W>), per_atom, dim3(kAtomThreads), 0, st, a);
        hipLaunchKernelGGL((k_rows_lists<W, TB>), dim3(atoms8 * rows), dim3(kRowsThreads), 0, st, a, rows);
        for (int m = 1; m < a.mmax; ++m) {
            const dim3 grid(atoms8 * prod);
            const size_t lds = (size_t)kRowsWaves * wl;
            if (vec) hipLaunchKernelGGL((k_rows_product<W, VW>), grid, dim3(kRowsThreads), lds, st, a, prod, m, wl);
            else hipLaunchKernelGGL((k_rows_product<W, 1>), grid, dim3(kRowsThreads), lds, st, a, prod, m, wl);
        }
        hipLaunchKernelGGL((k_rows_energy<W, TB, NM>), per_atom, dim3(kAtomThreads), rows_energy_lds(a, operands), st, a);
        if (!a.forces) continue;
        if (!operands)
            hipLaunchKernelGGL((k_rows_operands<W, NM>), dim3(atoms8 * ops), dim3(kRowsThreads), 0, st, a, ops);
        if (vec) hipLaunchKernelGGL((k_rows_pairs<W, VW>), dim3(atoms8 * pr), dim3(64 * pw), pw * lw, st, a, pr);
        else hipLaunchKernelGGL((k_rows_pairs<W, 1>), dim3(atoms8 * pr), dim3(64 * pw), pw * lw, st, a, pr);
        hipLaunchKernelGGL((k_rows_sums<W>), dim3(atoms8 * rows), dim3(kRowsThreads), 0, st, a, rows);
        hipLaunchKernelGGL((k_rows_final<W, TB>), per_atom, dim3(kAtomThreads), 0, st, a);
    }
    return hipGetLastError();
}

template <typename W, bool TB>
static hipError_t launch_rows_nm(hipStream_t st, const MbdArgs& a, int nkmax) {   // register arrays by the body order
    return a.n_max <= 6 ? launch_rows_t<W, TB, 6>(st, a, nkmax) : launch_rows_t<W, TB, kMaxNmax>(st, a, nkmax);
}

hipError_t launch_mbd_rows(hipStream_t st, const MbdArgs& a, int nkmax, bool mixed, bool two_body) {
    if (mixed) return two_body ? launch_rows_nm<float, true>(st, a, nkmax) : launch_rows_nm<float, false>(st, a, nkmax);
    return two_body ? launch_rows_nm<double, true>(st, a, nkmax) : launch_rows_nm<double, false>(st, a, nkmax);
}

}  // namespace lmbd
