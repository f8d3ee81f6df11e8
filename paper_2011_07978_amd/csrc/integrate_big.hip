// Per-cell stiff chemistry integration for large mechanisms (64 < n <= ~138
// unknowns), FP64, gfx950.
//
// A workgroup of eight wavefronts owns one cell; threads 2i and 2i + 1 hold
// unknown i of y = (T, Y_1..Y_N).  The iteration matrix M = I/(gamma h) - J
// (n x n) lives in LDS (up to ~150 KB, so one cell per CU for the largest
// mechanisms).
//   - right-hand side and analytic Jacobian: the formulas of the wavefront
//     kernel, reaction pass over all threads.  Production rates are summed
//     with LDS float atomics into one array per wavefront (as many as the LDS
//     holds) added in a fixed order; the Jacobian's scatter is issued one
//     wavefront at a time; block reductions combine in a fixed order, so the
//     result does not depend on scheduling.  The Jacobian is assembled in the
//     matrix's place and turned into M there; after a rejected step it is
//     assembled again (the same y gives the same bits), which happens for
//     about 1 % of the steps and costs less than keeping a copy for all;
//   - block Gauss-Jordan elimination with partial pivoting, 16 columns at a
//     time: one wavefront inverts the panel's pivot block in registers while
//     the others update the columns behind the next panel on the FP64 matrix
//     cores (v_mfma_f64_16x16x4f64);
//   - a stage's solve is one pass over the panels (nine steps for 131
//     unknowns) and a product with the inverted pivot blocks.
// 8192 cells of a 130-species flame: 58.3 ms (LU by columns, triangular solves
// and four wavefronts: 154 ms).  Bound by the panels' chain, 1240 cycles a
// column, 47 % of an attempted step.
#include <hip/hip_runtime.h>
#include <math.h>
#include "mech_dev.hpp"
#include "wave.hpp"

namespace chem {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Eight wavefronts, two per SIMD: the reaction pass and the trailing updates
// have twice the wavefronts of a four-wavefront group to hide their latencies
// with.
constexpr int BT = 512;
constexpr int NW = BT / 64;
constexpr int NB = 16;    // panel width: four K = 4 matrix-core steps
constexpr size_t kBigLds = 160 * 1024;   // LDS of a CU

__constant__ double kBigA[6][6] = {
    {0, 0, 0, 0, 0, 0},
    {1.544, 0, 0, 0, 0, 0},
    {0.9466785280815826, 0.2557011698983284, 0, 0, 0, 0},
    {3.314825187068521, 2.896124015972201, 0.9986419139977817, 0, 0, 0},
    {1.221224509226641, 6.019134481288629, 12.53708332932087, -0.6878860361058950, 0, 0},
    {1.221224509226641, 6.019134481288629, 12.53708332932087, -0.6878860361058950, 1.0, 0}};
__constant__ double kBigC[6][6] = {
    {0, 0, 0, 0, 0, 0},
    {-5.6688, 0, 0, 0, 0, 0},
    {-2.430093356833875, -0.2063599157091915, 0, 0, 0, 0},
    {-0.1073529058151375, -9.594562251023355, -20.47028614809616, 0, 0, 0},
    {7.496443313967647, -10.24680431464352, -33.99990352819905, 11.70890893206160, 0, 0},
    {8.083246795921522, -7.981132988064893, -31.52159432874371, 16.31930543123136,
     -6.058818238834054, 0}};
constexpr double kBigGamma = 0.25;

__device__ __forceinline__ void lds_add_b(double *p, double v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// LDS layout of one cell (in doubles); lda is odd so that thread-per-row
// accesses fall into distinct banks.
struct BigLds {
    int n, N, lda, nw;   // nw: copies of the production-rate array
    double *A, *C, *g, *col, *hh, *e, *cp, *tb, *w, *red;   // col: partial column sums
    int *step, *prow;    // row -> elimination step, step -> pivot row
};

constexpr int kRedDoubles = 48;
__host__ __device__ inline int big_lda(int n) { return n | 1; }
// everything but the copies of the production rates past the first
__host__ __device__ inline size_t big_base_doubles(int n) {
    const int N = n - 1;
    return (size_t)n * big_lda(n) + 5 * (N + 1) + 2 * N + n + kRedDoubles + n;  // step, prow share n doubles
}
// One production-rate array per wavefront where the LDS holds them (up to 135
// unknowns); fewer are shared by wavefronts taking turns.
__host__ __device__ inline int big_rate_copies(int n) {
    int c = NW;
    while (c > 1 && (big_base_doubles(n) + (size_t)(c - 1) * n) * sizeof(double) > kBigLds) c /= 2;
    return c;
}
__host__ __device__ inline size_t big_lds_doubles(int n) {
    return big_base_doubles(n) + (size_t)(big_rate_copies(n) - 1) * n;
}

__device__ __forceinline__ BigLds big_layout(int n, double *lds) {
    BigLds L;
    L.n = n;
    L.N = n - 1;
    L.lda = big_lda(n);
    L.nw = big_rate_copies(n);
    double *q = lds;
    L.A = q; q += (size_t)n * L.lda;
    L.C = q; q += L.N + 1;
    L.g = q; q += L.N + 1;
    L.col = q; q += L.N + 1;
    L.hh = q; q += L.N + 1;
    L.e = q; q += L.N;
    L.cp = q; q += L.N;
    L.tb = q; q += n;
    L.red = q; q += kRedDoubles;
    L.step = (int *)q;          // n ints
    L.prow = L.step + n;        // n ints (2n ints fit in n doubles)
    q += n;
    L.w = q;                    // nw x (N + 1)
    return L;
}

__device__ __forceinline__ int opaque_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Max over the workgroup; every thread returns the same bits.
__device__ __forceinline__ double block_max(double v, double *red) {
    const double s = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[36 + (threadIdx.x >> 6)] = s;
    __syncthreads();
    double m = red[36];
#pragma unroll
    for (int i = 1; i < NW; ++i) m = max2(m, red[36 + i]);
    return m;
}
__device__ __forceinline__ bool block_any(bool p, double *red) {
    return block_max(p ? 1.0 : 0.0, red) > 0.0;
}
// Wavefront partial sums of quantity i into red[8 i ..]; after a barrier
// block_total adds them in order.
__device__ __forceinline__ void block_part(double v, int i, double *red) {
    const double s = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[NW * i + (threadIdx.x >> 6)] = s;
}
template <int WAVES>
__device__ __forceinline__ double block_total(int i, const double *red) {
    const double *r = red + NW * i;
    const double s = (r[0] + r[1]) + (r[2] + r[3]);
    return WAVES == 4 ? s : s + ((r[4] + r[5]) + (r[6] + r[7]));
}

// NASA-7 coefficients and molar mass of a species
struct Species {
    double a1, a2, a3, a4, a5, a6, a7, h2, h3, h4, h5, s3, s4, s5, W, iW;
};
__device__ __forceinline__ Species load_species(const MechDev &M, int k) {
    const auto *a = gbl(M.spc) + k * SPC_STRIDE;
    return {a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13], a[14], a[15]};
}

__device__ __forceinline__ RxnRec load_rxn(const RxnRec *__restrict__ rxn, int j) {
    const auto *r = gbl(rxn) + j;
    RxnRec o;
    o.lnA = r->lnA; o.b = r->b; o.EaR = r->EaR;
#pragma unroll
    for (int i = 0; i < 3; ++i) o.eff[i] = r->eff[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) o.idx[i] = r->idx[i];
    return o;
}

// -----------------------------------------------------------------------------
// f(y) and, with JAC, the analytic Jacobian into L.A (row-major, stride lda),
// or with MAT the iteration matrix diag I - J.  Threads 2i, 2i + 1 return f_i.
// Without MAT, rows 1.. of the Jacobian go straight to Jg (n x n, nullable), row
// 0 last.  NT threads; 3 n of them map the columns.  Same formulas as the
// wavefront kernel.
// -----------------------------------------------------------------------------
template <bool JAC, bool MAT, int NT>
__device__ __forceinline__ double rhs_big(const MechDev *__restrict__ Mp, const double p, const double y,
                                          const double diag, const BigLds &L, double *__restrict__ Jg) {
    constexpr int WAVES = NT / 64;
    // The opaque thread index and sizes keep the addresses and trip counts
    // derived from them local to this call instead of held (spilled) across
    // the step loop; so below.
    asm volatile("" ::: "memory");
    const MechDev &M = *Mp;
    const int tid = opaque_tid(), own = tid >> 1, half = tid & 1, wv = uniform_i(tid >> 6);
    int N = M.N, R = M.R, n = M.n;
    asm volatile("" : "+s"(N), "+s"(R), "+s"(n));
    const int lda = big_lda(n);
    const bool sp = own >= 1 && own <= N;
    const int k = sp ? own - 1 : 0;
    // the species record and the first reaction record are on their way while
    // the first sums run
    const Species S = load_species(M, k);
    RxnRec next = load_rxn(M.rxn, tid < R ? tid : R - 1);

    const double yw = sp ? y * S.iW : 0.0;
    block_part(half == 0 ? yw : 0.0, 0, L.red);
    if (tid == 0) L.red[32] = y;
    __syncthreads();
    const double T = L.red[32];
    const double sumYW = block_total<WAVES>(0, L.red);
    const double lnT = log(T);
    const double ln_patm_RT = kLnPatmRu - lnT;
    const double invT = recip_nr(T);
    const double pv = RU_ERG * T * sumYW;
    const double irho = pv * recip_nr(p);
    const double rho = p * recip_nr(pv);
    const double Ctot = rho * sumYW;
    double cpR = 0.0, hRT = 0.0, dcpR = 0.0;
    if (sp) {
        cpR = S.a1 + T * (S.a2 + T * (S.a3 + T * (S.a4 + T * S.a5)));
        hRT = S.a1 + T * (S.h2 + T * (S.h3 + T * (S.h4 + T * S.h5))) + S.a6 * invT;
        const double sR = S.a1 * lnT + T * (S.a2 + T * (S.s3 + T * (S.s4 + T * S.s5))) + S.a7;
        if (JAC) dcpR = S.a2 + T * (2.0 * S.a3 + T * (3.0 * S.a4 + T * (4.0 * S.a5)));
        if (half) {
            if (JAC) {
                L.e[k] = hRT * S.iW;
                L.cp[k] = cpR * S.iW;
            }
        } else {
            L.g[k] = hRT - sR - ln_patm_RT;
            L.C[k] = rho * yw;
            if (JAC) L.hh[k] = hRT;
        }
    }
    if (tid == 0) {   // the sentinel of missing slots
        L.C[N] = 1.0;
        L.g[N] = 0.0;
        if (JAC) L.hh[N] = 0.0;
    }
    for (int i = tid; i < L.nw * (N + 1); i += NT) L.w[i] = 0.0;
    if (JAC) {
        for (int i = tid; i < n * lda; i += NT) L.A[i] = 0.0;
        if (tid < n) L.tb[tid] = 0.0;
    }
    __syncthreads();

    const double lnp = M.has_fo ? log(p) : 0.0;
    double *Cl = L.C, *gl = L.g, *hl = L.hh, *Jl = L.A, *tbl = L.tb;
    // Every wavefront adds to production-rate copy wv % nw; where copies are
    // shared, and for the Jacobian, the wavefronts take turns, so the order of
    // every sum is fixed.
    double *wl = L.w + (size_t)(wv & (L.nw - 1)) * (N + 1);
    const int turns = JAC ? WAVES : WAVES / L.nw;
    const int my_turn = JAC ? wv : wv / L.nw;
#pragma unroll 1
    for (int j0 = 0; j0 < R; j0 += NT) {
        const bool valid = j0 + tid < R;
        const RxnRec rec = next;
        if (j0 + NT < R) next = load_rxn(M.rxn, j0 + NT + tid < R ? j0 + NT + tid : R - 1);
        const int ix0 = rec.idx[0], ix1 = rec.idx[1], ix2 = rec.idx[2], ix3 = rec.idx[3];
        const int r0 = ix0 & 0xffff, r1 = (int)((unsigned)ix0 >> 16);
        const int p0 = ix1 & 0xffff, p1 = (int)((unsigned)ix1 >> 16);
        const int p2 = ix2 & 0xffff, tbw = (int)((unsigned)ix2 >> 16);
        const int tb = tbw & TB_CODE;
        const double snu = (double)((ix3 & 0xff) - 8);
        const int es0 = (ix3 >> 8) & 0xff, es1 = (ix3 >> 16) & 0xff;
        const int es2 = (int)((unsigned)ix3 >> 24);
        const double Cr0 = Cl[r0], Cr1 = Cl[r1], Cp0 = Cl[p0], Cp1 = Cl[p1], Cp2 = Cl[p2];
        double lnAj = rec.lnA, bj = rec.b, EaRj = rec.EaR;
        if (tbw & TB_PLOG)
            plog_arrhenius(M.plog + (size_t)(valid ? j0 + tid : R - 1) * PLOG_STRIDE, lnp, lnAj, bj, EaRj);
        const double ln_kf = lnAj + bj * lnT - EaRj * invT;
        const double kf = exp(ln_kf);
        // k_r = k_f / K_c from the differences of g_k = G_k / RT - ln(p_atm / RT):
        // exp(+-g_k) by itself leaves the range of doubles for large species at
        // low temperatures (|g| of 700 is 1.7 MJ/mol at 300 K), and products of
        // two of them at half of that
        const double kr = exp(ln_kf + (((gl[p0] - gl[r0]) + (gl[p1] - gl[r1])) + gl[p2]));
        const double Pf = Cr0 * Cr1;
        const double Pr = Cp0 * Cp1 * Cp2;
        const double e0v = rec.eff[0], e1v = rec.eff[1], e2v = rec.eff[2];
        double m = 1.0;
        if (tb != TB_NONE) m = Ctot + e0v * Cl[es0] + e1v * Cl[es1] + e2v * Cl[es2];
        if (tb >= TB_LIST0) {
            const int e1 = M.tb_ptr[tb - TB_LIST0 + 1];
            for (int e = M.tb_ptr[tb - TB_LIST0]; e < e1; ++e) m += M.eff_am1[e] * Cl[M.eff_sp[e]];
        }
        // fall-off: the rate constant is k_inf G([M], T) in place of k [M]
        double dGdM = 1.0, dlnGdT = 0.0;
        if (tbw & TB_FALLOFF) {
            double G;
            falloff_eval(M.fo + (size_t)(valid ? j0 + tid : R - 1) * FO_STRIDE, T, invT, lnT, kf,
                         bj * invT + EaRj * invT * invT, m, G, dGdM, dlnGdT);
            m = G;
        }
        const double Delta = kf * Pf - kr * Pr;
        const double q = m * Delta;
        double dqdT = 0.0, ds[5] = {0, 0, 0, 0, 0};
        if (JAC) {
            const double dlnkf = bj * invT + EaRj * invT * invT + dlnGdT;
            const double dH = -hl[r0] - hl[r1] + hl[p0] + hl[p1] + hl[p2];
            const double dlnkr = dlnkf - (dH - snu) * invT;
            const double mkf = m * kf, mkr = m * kr;
            dqdT = mkf * dlnkf * Pf - mkr * dlnkr * Pr;
            ds[0] = mkf * Cr1;
            ds[1] = mkf * Cr0;
            ds[2] = -mkr * Cp1 * Cp2;
            ds[3] = -mkr * Cp0 * Cp2;
            ds[4] = -mkr * Cp0 * Cp1;
        }
        for (int turn = 0; turn < turns; ++turn) {
            if (my_turn == turn && valid) {
                lds_add_b(wl + r0, -q);
                lds_add_b(wl + r1, -q);
                lds_add_b(wl + p0, q);
                lds_add_b(wl + p1, q);
                lds_add_b(wl + p2, q);
                if (JAC) {
                    const int sl[5] = {r0, r1, p0, p1, p2};
#pragma unroll
                    for (int a = 0; a < 5; ++a) {
                        const int sa = sl[a];
                        if (sa >= N) continue;
                        const double nu = a < 2 ? -1.0 : 1.0;
                        double *row = Jl + (sa + 1) * lda;
                        lds_add_b(row, nu * dqdT);
#pragma unroll
                        for (int b = 0; b < 5; ++b)
                            if (sl[b] < N) lds_add_b(row + 1 + sl[b], nu * ds[b]);
                        if (tb != TB_NONE) {
                            const double nd = nu * Delta * dGdM;
                            lds_add_b(tbl + sa + 1, nd);
                            if (es0 < N) lds_add_b(row + 1 + es0, nd * e0v);
                            if (es1 < N) lds_add_b(row + 1 + es1, nd * e1v);
                            if (es2 < N) lds_add_b(row + 1 + es2, nd * e2v);
                            if (tb >= TB_LIST0) {
                                const int e1 = M.tb_ptr[tb - TB_LIST0 + 1];
                                for (int e = M.tb_ptr[tb - TB_LIST0]; e < e1; ++e)
                                    lds_add_b(row + 1 + M.eff_sp[e], nd * M.eff_am1[e]);
                            }
                        }
                    }
                }
            }
            if (turns > 1) __syncthreads();
        }
    }
    __syncthreads();

    double om = 0.0;
    if (sp) {
        const double *w = L.w + k;
        if (L.nw == NW) {   // all copies loaded before the first is added
            double x[NW];
#pragma unroll
            for (int c = 0; c < NW; ++c) x[c] = w[c * (N + 1)];
#pragma unroll
            for (int c = 0; c < NW; ++c) om += x[c];
        } else {
            for (int c = 0; c < L.nw; ++c) om += w[c * (N + 1)];
        }
    }
    const double fk = sp ? S.W * om * irho : 0.0;
    const bool one = sp && half == 0;
    block_part(one ? hRT * S.iW * fk : 0.0, 0, L.red);
    block_part(one ? y * cpR * S.iW : 0.0, 1, L.red);
    if (JAC) {
        block_part(one ? cpR * S.iW * fk : 0.0, 2, L.red);
        block_part(one ? y * dcpR * S.iW : 0.0, 3, L.red);
        if (one) L.hh[k] = fk;
    }
    __syncthreads();
    const double hs = block_total<WAVES>(0, L.red);
    const double icps = recip_nr(block_total<WAVES>(1, L.red));
    const double fT = -T * hs * icps;
    if (JAC) {
        const double cpf = block_total<WAVES>(2, L.red);
        const double dcps = block_total<WAVES>(3, L.red);
        const double Wbar = recip_nr(sumYW);
        // species rows, chain rule from concentrations to (T, Y): four threads
        // a row form its sum over the concentrations and its T column; the
        // rest of the row is an affine map per entry, x -> (W_k x + g_k) / W_c
        for (int r = tid >> 2; r < N; r += NT / 4) {
            double *row = Jl + (r + 1) * lda;
            const double tbk = tbl[r + 1];
            double s = 0.0;
#pragma unroll 4
            for (int l = tid & 3; l < N; l += 4) s += (row[1 + l] + tbk) * Cl[l];
            s += dpp_d<0xB1>(s);
            s += dpp_d<0x4E>(s);
            if ((tid & 3) == 0) {
                const double f = hl[r], Wk = gbl(M.W)[r];
                gl[r] = Wk * tbk + (f * Wbar - Wk * Wbar * s * irho);
                row[0] = Wk * irho * (row[0] - s * invT) + f * invT;
                hl[r] = Wk;
            }
        }
        __syncthreads();
        // one thread per column and third of the rows: the map, the column's
        // part of the temperature row sum_k e_k J_kc, and the sign
        const int seg = (tid >= n) + (tid >= 2 * n);
        const int c = tid - seg * n;
        double *part = seg == 0 ? L.col : seg == 1 ? L.w : tbl;   // free by now
        if (c < n) {
            const int ch = (N + 2) / 3;
            const int k1 = (seg + 1) * ch < N ? (seg + 1) * ch : N;
            const double iw = c > 0 ? gbl(M.invW)[c - 1] : 0.0;
            double acc = 0.0;
            // eight rows at a time, loaded before any is written back
            auto rows = [&](const int k0, const int cnt) {
                double x[8], wk[8], gk[8], ek[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (i >= cnt) break;
                    x[i] = Jl[(k0 + i + 1) * lda + c];
                    wk[i] = hl[k0 + i];
                    gk[i] = gl[k0 + i];
                    ek[i] = L.e[k0 + i];
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (i >= cnt) break;
                    if (c > 0) x[i] = iw * (wk[i] * x[i] + gk[i]);
                    acc += ek[i] * x[i];
                    if (MAT) Jl[(k0 + i + 1) * lda + c] = (k0 + i + 1 == c ? diag : 0.0) - x[i];
                    else if (Jg) Jg[(k0 + i + 1) * n + c] = x[i];
                }
            };
            int k0 = seg * ch;
            for (; k0 + 8 <= k1; k0 += 8) rows(k0, 8);
            for (; k0 < k1; ++k0) rows(k0, 1);
            part[c] = acc;
        }
        __syncthreads();
        // temperature row: J_T,c = -(sum_k e_k J_kc) T / cp - f_T dcp/dy_c / cp
        if (tid < n) {
            const double acc = ((L.col[tid] + L.w[tid]) + tbl[tid]) * T;
            const double v = tid == 0 ? -(cpf + acc) * icps - fT * dcps * icps
                                      : -acc * icps - fT * L.cp[tid - 1] * icps;
            if (MAT) Jl[tid] = (tid == 0 ? diag : 0.0) - v;
            else if (Jg) Jg[tid] = v;
        }
        __syncthreads();
    }
    return own == 0 ? fT : fk;
}

// -----------------------------------------------------------------------------
// Block Gauss-Jordan elimination of L.A (n x n) with partial pivoting.  Rows
// never move.  Panel b (columns 16 b ..) picks its pivot rows p_s among the
// rows not yet pivot and turns its columns into
//   E[r][s] = -(A[r][.] D)[s] for every other row r, and D = A_pivot^-1 in the
// rows p_q (L.step[p_q] = L.prow^-1 = 16 b + q), after which the columns behind
// it are updated as A[r][j] += sum_s E[r][s] A[p_s][j], rows above and below
// alike; the pivot rows keep their values.  With b the right-hand side, the
// same updates panel by panel and x = D b of each pivot block solve the system.
// The sizes of n and of the LDS leave one cell per CU, so nothing hides a
// panel's dependent chain but the rest of the same elimination: wavefront 0
// runs the panels, one ahead of the others, which do the trailing updates.
// Solve errors against 80-bit arithmetic at accepted steps of the 130-species
// mechanism: median 1.6e-16 (LU: 3.0e-16), largest 4.0e-16 (LU: 6.8e-16).
// -----------------------------------------------------------------------------

// One panel in the registers of a wavefront, NR rows per lane.  In-place
// inversion step by step: with pivot row p of column q, every other row
// subtracts m = a_q / pivot times the pivot row, keeping -m in column q.  The
// pivot row itself is left unscaled with 1 in column q and scaled once at the
// end.  The search compares the upper 32 bits of |a|, ties to the lowest row;
// a zero or non-finite pivot gives a NaN reciprocal (false is returned).  The
// next column is updated first, so that its search runs beside the other
// columns' updates.
template <int NR>
__device__ __forceinline__ bool panel_big(const BigLds &L, int kb, int jb, bool (&fr)[NR]) {
    const int lane = opaque_tid() & 63, n = L.n, lda = L.lda;
    double a[NR][NB], rs[NR];
    int st[NR];
#pragma unroll
    for (int s = 0; s < NR; ++s) {
        const int row = lane + 64 * s;
        const double *ar = L.A + (row < n ? row : 0) * lda + kb;
        rs[s] = 1.0;
        st[s] = -1;
#pragma unroll
        for (int q = 0; q < NB; ++q) a[s][q] = row < n && q < jb ? ar[q] : 0.0;
    }
    bool ok = true;
    // The search is cut into stages that the column updates are interleaved
    // with: a lane's best of its rows, the wavefront's maximum, the lane that
    // holds it, its slot and value, the reciprocal.
    unsigned key = 0u, v = 0u;
    int bs = 0, pl = 0, ps = 0;
    double bx = 0.0, piv = 0.0, rinv = 0.0, e = 0.0;
    auto stage = [&](const int i, const int q) {
        switch (i) {
            case 0: {
                key = fr[0] ? (unsigned)__double2hiint(a[0][q]) & 0x7fffffffu : 0u;
                bx = a[0][q];
                bs = 0;
#pragma unroll
                for (int s = 1; s < NR; ++s) {
                    const unsigned ks = fr[s] ? (unsigned)__double2hiint(a[s][q]) & 0x7fffffffu : 0u;
                    const bool up = ks > key;
                    key = up ? ks : key;
                    bx = up ? a[s][q] : bx;
                    bs = up ? s : bs;
                }
                v = max(key, (unsigned)__builtin_amdgcn_update_dpp(0, (int)key, 0xB1, 0xf, 0xf, false));
                break;
            }
            case 1: v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false)); break;
            case 2: v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false)); break;
            case 3: v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, false)); break;
            case 4: v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false)); break;
            case 5: v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false)); break;
            case 6: v = (unsigned)__builtin_amdgcn_readlane((int)v, 63); break;
            case 7: pl = (int)__builtin_ctzll(ballot(key == v)); break;
            case 8:
                ps = __builtin_amdgcn_readlane(bs, pl);
                piv = readlane_d(bx, pl);
                break;
            case 9: rinv = __builtin_amdgcn_rcp(piv); e = fma(-piv, rinv, 1.0); break;
            case 10: rinv = fma(rinv, e, rinv); e = fma(-piv, rinv, 1.0); break;
            default: rinv = fma(rinv, e, rinv); break;
        }
    };
    constexpr int kStages = 12;
    static_assert(kStages <= NB - 2, "one stage per column update");
#pragma unroll
    for (int i = 0; i < kStages; ++i) stage(i, 0);
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        if (q < jb) {
            double pj[NB];
#pragma unroll
            for (int s = 0; s < NR; ++s)
                if (ps == s) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) pj[j] = readlane_d(a[s][j], pl);
                }
            const double r = rinv;
            ok = ok && v != 0u && fabs(r) < INFINITY;   // v = 0: no free row with a nonzero entry
            double m[NR];   // minus the multiplier
#pragma unroll
            for (int s = 0; s < NR; ++s) {
                const bool mine = ps == s && lane == pl;
                m[s] = a[s][q] * -r;
                a[s][q] = mine ? 1.0 : m[s];
                m[s] = mine ? 0.0 : m[s];
                rs[s] = mine ? r : rs[s];
                st[s] = mine ? kb + q : st[s];
                fr[s] = fr[s] && !mine;
            }
            if (q + 1 < NB) {
#pragma unroll
                for (int s = 0; s < NR; ++s) a[s][q + 1] = fma(m[s], pj[q + 1], a[s][q + 1]);
            }
            int i = 0;
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if (j != q && j != q + 1) {
                    if (q + 1 < NB && i < kStages) stage(i, q + 1);
                    ++i;
#pragma unroll
                    for (int s = 0; s < NR; ++s) a[s][j] = fma(m[s], pj[j], a[s][j]);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
    }
#pragma unroll
    for (int s = 0; s < NR; ++s) {
        const int row = lane + 64 * s;
        if (row < n) {
            double *ar = L.A + row * lda + kb;
#pragma unroll
            for (int q = 0; q < NB; ++q)
                if (q < jb) ar[q] = a[s][q] * rs[s];
            if (st[s] >= 0) {
                L.step[row] = st[s];
                L.prow[st[s]] = row;
            }
        }
    }
    return ok;
}

// 16 x 16 tiles i0 <= i < i1 of the update behind panel kb (tile i: row tile
// i / nc, column tile c0 + i % nc) on the matrix cores.  v_mfma_f64_16x16x4f64:
// lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and D[l / 16 + 4 i][l % 16],
// i = 0..3 (checked on gfx950).  The panel's own pivot rows take no update.
__device__ __forceinline__ void update_tiles(const BigLds &L, int kb, int i0, int i1, int c0, int nc) {
    const int lane = opaque_tid() & 63, lr = lane & 15, lk = lane >> 4;
    const int n = L.n, lda = L.lda;
    double *A = L.A;
    const double *bp[NB / 4];
#pragma unroll
    for (int ks = 0; ks < NB / 4; ++ks) bp[ks] = A + L.prow[kb + 4 * ks + lk] * lda;
    double a[NB / 4];
    bool ok[4];
    int rt = -1;
    for (int i = i0; i < i1; ++i) {
        const int t = i / nc;
        if (t != rt) {
            rt = t;
            const int ar = 16 * rt + lr;
            const int as = ar < n ? L.step[ar] : kb;
            const bool live = (unsigned)(as - kb) >= (unsigned)NB;
            const double *ap = A + (ar < n ? ar : 0) * lda + kb + lk;
#pragma unroll
            for (int ks = 0; ks < NB / 4; ++ks) a[ks] = live ? ap[4 * ks] : 0.0;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int dr = 16 * rt + lk + 4 * d;
                ok[d] = dr < n && (unsigned)(L.step[dr < n ? dr : 0] - kb) >= (unsigned)NB;
            }
        }
        const int col = 16 * (c0 + i - rt * nc) + lr;
        const bool cok = col < n;
        const int cc = cok ? col : 0;
        double *dp = A + (16 * rt + lk) * lda + cc;
        f64x4 acc;
#pragma unroll
        for (int d = 0; d < 4; ++d) acc[d] = ok[d] && cok ? dp[4 * d * lda] : 0.0;
        double b[NB / 4];
#pragma unroll
        for (int ks = 0; ks < NB / 4; ++ks) b[ks] = bp[ks][cc];
#pragma unroll
        for (int ks = 0; ks < NB / 4; ++ks)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks], b[ks], acc, 0, 0, 0);
#pragma unroll
        for (int d = 0; d < 4; ++d)
            if (ok[d] && cok) dp[4 * d * lda] = acc[d];
    }
}

// Returns false if a pivot is zero or not finite.
template <int NR>
__device__ __forceinline__ bool gj_big(const BigLds &L) {
    const int tid = opaque_tid(), wv = uniform_i(tid >> 6);
    const int n = L.n, nt = (n + NB - 1) / NB;
    bool fr[NR];
#pragma unroll
    for (int s = 0; s < NR; ++s) fr[s] = (tid & 63) + 64 * s < n;
    if (tid < n) L.step[tid] = 0x7fffffff;
    __syncthreads();
    bool ok = true;
#pragma unroll 1
    for (int b = -1; b + 1 < nt; ++b) {
        const int kb = NB * b, ke = kb + NB;
        if (b >= 0) {
            // the next panel's columns first, by all wavefronts
            for (int rt = wv; rt < nt; rt += NW) update_tiles(L, kb, rt, rt + 1, b + 1, 1);
            __syncthreads();
        }
        if (wv == 0) {
            __builtin_amdgcn_s_setprio(2);
            ok = panel_big<NR>(L, ke, n - ke < NB ? n - ke : NB, fr) && ok;
            __builtin_amdgcn_s_setprio(0);
        } else if (b >= 0) {
            const int nc = nt - b - 2, items = nt * nc;
            if (nc > 0)
                update_tiles(L, kb, items * (wv - 1) / (NW - 1), items * wv / (NW - 1), b + 2, nc);
        }
        __syncthreads();
    }
    if (tid == 0) L.red[33] = ok ? 1.0 : 0.0;
    __syncthreads();
    return L.red[33] != 0.0;
}

// Solve with the panels of gj_big; threads 2i, 2i + 1 pass b_i and receive
// x_i.  Each pair owns row i and half of every dot product: panel by panel the
// pivot rows' values (L.hh, by step) times the row's E, then the rows of D
// times the final values (L.g).  One barrier per panel; the next panel's E is
// loaded ahead of it.
__device__ __forceinline__ double solve_big(const BigLds &L, double b) {
    const int tid = opaque_tid(), own = tid >> 1, half = tid & 1;
    const int n = L.n, lda = L.lda;
    double *v = L.hh, *vf = L.g;
    const bool act = own < n;
    const int st = act ? L.step[own] : -1;
    const double *row = L.A + (act ? own : 0) * lda + 8 * half;
    double x = act ? b : 0.0;
    if (act && half == 0 && st < NB) v[st] = x;
    double r[8];
    const bool busy = uniform_i(tid & ~63) < 2 * n;   // wavefronts past the rows only wait
    if (busy) {
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = row[i];
    }
    __syncthreads();
    int kb = 0;
    for (; kb + NB < n; kb += NB) {
        if (busy) {
            const double *vk = v + kb + 8 * half;
            double w[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = vk[i];
            double s0 = r[0] * w[0], s1 = r[1] * w[1];
#pragma unroll
            for (int i = 2; i < 8; i += 2) {
                s0 = fma(r[i], w[i], s0);
                s1 = fma(r[i + 1], w[i + 1], s1);
            }
            double s = s0 + s1;
            s += dpp_d<0xB1>(s);
            if ((unsigned)(st - kb) >= (unsigned)NB) x += s;
            const int kn = kb + NB;
            if (act && half == 0 && (unsigned)(st - kn) < (unsigned)NB) v[st] = x;
            if (kn + NB <= n) {
#pragma unroll
                for (int i = 0; i < 8; ++i) r[i] = row[kn + i];
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) r[i] = kn + 8 * half + i < n ? row[kn + i] : 0.0;
            }
        }
        __syncthreads();
    }
    if (busy) {
        // the last panel, up to 16 columns
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = kb + 8 * half + i;
            s = fma(r[i], c < n ? v[c] : 0.0, s);
        }
        s += dpp_d<0xB1>(s);
        if ((unsigned)(st - kb) >= (unsigned)NB) x += s;
        if (act && half == 0) vf[st] = x;
    }
    __syncthreads();
    // unknown own = kb + q: row prow[own] of D in the panel's columns
    double s = 0.0;
    if (act) {
        const int kb = own & ~(NB - 1);
        const double *d = L.A + L.prow[own] * lda + kb + 8 * half;
        const int jb = n - kb - 8 * half;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < jb) s = fma(d[i], vf[kb + 8 * half + i], s);
    }
    s += dpp_d<0xB1>(s);
    return act ? s : 0.0;
}

// One Rodas4 attempt of size h from y with f0 = f(y) and M in L.A; false when
// M is singular.
template <int NR>
__device__ __forceinline__ bool rodas_attempt_big(const MechDev *__restrict__ M, const BigLds &L, double p,
                                                  double y, double f0, double h, double &ynew, double &err) {
    if (!gj_big<NR>(L)) return false;
    const double hinv = 1.0 / h;
    double u[6] = {0, 0, 0, 0, 0, 0};
    double ys = y;
#pragma unroll 1
    for (int s = 0; s < 6; ++s) {
        double rv = f0;
        if (s > 0) {
            ys = y;
#pragma unroll
            for (int j = 0; j < 5; ++j) ys += kBigA[s][j] * u[j];
            rv = rhs_big<false, false, BT>(M, p, ys, 0.0, L, nullptr);
#pragma unroll
            for (int j = 0; j < 5; ++j) rv += (kBigC[s][j] * hinv) * u[j];
        }
        const double us = solve_big(L, rv);
#pragma unroll
        for (int j = 0; j < 6; ++j) u[j] = j == s ? us : u[j];
    }
    ynew = ys + u[5];
    err = u[5];
    return true;
}

__device__ __forceinline__ double load_unknown(const IntParams &P, int64_t cell, int N) {
    const int own = threadIdx.x >> 1;
    return own == 0 ? P.T[cell] : own <= N ? P.Y[(int64_t)(own - 1) * P.ncells + cell] : 0.0;
}

// Adaptive integration of one cell; control logic of the wavefront kernel.
template <int NR>
__device__ void integrate_cell_big(const MechDev *__restrict__ M, const IntParams &P, int64_t cell,
                                   const BigLds &L) {
    const int tid = threadIdx.x, own = tid >> 1;
    const int n = M->n, N = M->N;
    const double dt = P.dt;
    const double p = P.p[cell];
    double y = load_unknown(P, cell, N);
    const bool bad_in = block_any((own < n && !isfinite(y)) || (own == 0 && !(y > 0.0)), L.red) ||
                        !(p > 0.0) || !isfinite(p);
    if (bad_in) {
        if (tid == 0) {
            if (P.status) P.status[cell] = 4;
            if (P.ref_status && P.flags && P.flags[cell] == 1) *P.ref_status = 4;
            if (P.steps) { P.steps[2 * cell] = 0; P.steps[2 * cell + 1] = 0; }
            if (P.cost) P.cost[cell] = 0;
            atomicAdd(&P.stats[0], 1ull);
            atomicAdd(&P.stats[3], 1ull);
        }
        __syncthreads();
        return;
    }
    double h = P.h ? P.h[cell] : 0.0;
    if (!(h > 0.0)) h = dt;
    double hnext = h, t = 0.0;
    int nacc = 0, nrej = 0, status = 0;
    bool rej_last = false;
    while (t < dt) {
        if (nacc + nrej >= P.max_steps) { status = 1; break; }
        bool last = false;
        if (h >= dt - t) { h = dt - t; last = true; }
        if (h < P.hmin_frac * dt) { status = 2; break; }
        // f and the Jacobian of y, assembled as the matrix of this step size
        const double f0 = rhs_big<true, true, BT>(M, p, y, 1.0 / (kBigGamma * h), L, nullptr);
        double ynew = 0.0, ev = 0.0;
        const bool ok = rodas_attempt_big<NR>(M, L, p, y, f0, h, ynew, ev);
        // largest scaled error; a NaN counts as infinite (both shrink by 0.2)
        double e = INFINITY;
        if (ok) {
            const double sc = P.atol + P.rtol * fmax(fabs(y), fabs(ynew));
            const double r = own < n ? fabs(ev) / sc : 0.0;
            e = block_max(r != r ? (double)INFINITY : r, L.red);
        }
        if (e <= 1.0) {
            double fac = (e == 0.0) ? 5.0 : fmin(5.0, fmax(0.2, 0.9 * pow(e, -0.25)));
            if (rej_last) fac = fmin(fac, 1.0);
            y = ynew;
            t = last ? dt : t + h;
            ++nacc;
            hnext = h * fac;
            h = hnext;
            rej_last = false;
        } else {
            const double fac = ok ? fmax(0.2, 0.9 * pow(e, -0.25)) : 0.2;
            h = h * fac;
            ++nrej;
            rej_last = true;
        }
    }
    if (status == 0 && block_any(own < n && !isfinite(y), L.red)) status = 3;
    if ((tid & 1) == 0) {
        if (own == 0) P.T[cell] = y;
        else if (own <= N) P.Y[(int64_t)(own - 1) * P.ncells + cell] = y;
    }
    if (tid == 0) {
        if (P.h) P.h[cell] = hnext;
        if (P.cost) P.cost[cell] = (uint32_t)(nacc + nrej);
        if (P.status) P.status[cell] = (uint8_t)status;
        if (P.ref_status && P.flags && P.flags[cell] == 1) *P.ref_status = status;
        if (P.steps) { P.steps[2 * cell] = nacc; P.steps[2 * cell + 1] = nrej; }
        atomicAdd(&P.stats[0], 1ull);
        atomicAdd(&P.stats[1], (unsigned long long)nacc);
        atomicAdd(&P.stats[2], (unsigned long long)nrej);
        if (status) atomicAdd(&P.stats[3], 1ull);
        atomicMax(&P.stats[4], (unsigned long long)(nacc + nrej));
    }
    __syncthreads();
}

// Static schedule: workgroup b takes cells b, b + grid, b + 2 grid, ...
template <int NR>
__global__ __launch_bounds__(BT) void k_big_plain(const MechDev *__restrict__ M, IntParams P) {
    extern __shared__ double lds[];
    const BigLds L = big_layout(M->n, lds);
    // round robin over the slots, or (block_static) one contiguous block each
    const int64_t B = (P.ncells + gridDim.x - 1) / gridDim.x;
    const int64_t c0 = P.block_static ? blockIdx.x * B : blockIdx.x;
    const int64_t c1 = P.block_static ? (c0 + B < P.ncells ? c0 + B : P.ncells) : P.ncells;
    const int64_t stride = P.block_static ? 1 : gridDim.x;
    for (int64_t cell = c0; cell < c1; cell += stride) {
        if (P.flags && P.flags[cell] >= 2) continue;
        integrate_cell_big<NR>(M, P, cell, L);
    }
}

// Work queue with XCD segments and stealing, as in the wavefront kernel.
template <int NR>
__global__ __launch_bounds__(BT) void k_big_queue(const MechDev *__restrict__ M, IntParams P) {
    extern __shared__ double lds[];
    const BigLds L = big_layout(M->n, lds);
    const int nact = *P.n_active;
    const int chunk = P.chunk;
    int seg = blockIdx.x % NSEG;
    int probes = 0;
    while (probes < NSEG) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const int c = atomicAdd(&P.seg_ctr[seg], chunk);
            L.red[34] = (double)c;
        }
        __syncthreads();
        const int c = (int)L.red[34];
        const int first = seg + NSEG * c;
        if (first >= nact) {
            seg = seg + 1 == NSEG ? 0 : seg + 1;
            ++probes;
            continue;
        }
        probes = 0;
        for (int q = 0; q < chunk; ++q) {
            const int pos = first + NSEG * q;
            if (pos >= nact) break;
            integrate_cell_big<NR>(M, P, P.queue[pos], L);
        }
    }
}

// Kernel-level checks: f and J per cell; one fixed Rodas4 step per cell.  f and J
// need no elimination, so where three threads a column fit in 256, three
// four-wavefront workgroups share a CU and hide one another's barriers (65
// unknowns, 1001 cells, one eight-wavefront workgroup per CU: 70 us).
template <int NT>
__global__ __launch_bounds__(NT, NT == 256 ? 3 : 2) void k_big_rhs_jac(const MechDev *__restrict__ M, IntParams P,
                                                                       double *fout, double *Jout) {
    extern __shared__ double lds[];
    const BigLds L = big_layout(M->n, lds);
    const int64_t cell = P.first + blockIdx.x;
    const int tid = threadIdx.x, own = tid >> 1, n = M->n;
    const double y = load_unknown(P, cell, M->N);
    const double f = rhs_big<true, false, NT>(M, P.p[cell], y, 0.0, L, Jout ? Jout + cell * n * n : nullptr);
    if (fout && own < n && (tid & 1) == 0) fout[cell * n + own] = f;
}

template <int NR>
__global__ __launch_bounds__(BT) void k_big_rodas_step(const MechDev *__restrict__ M, IntParams P,
                                                       double h, double *ynew_out, double *err_out) {
    extern __shared__ double lds[];
    const BigLds L = big_layout(M->n, lds);
    const int64_t cell = P.first + blockIdx.x;
    const int tid = threadIdx.x, own = tid >> 1, n = M->n;
    const double y = load_unknown(P, cell, M->N);
    const double p = P.p[cell];
    const double f0 = rhs_big<true, true, BT>(M, p, y, 1.0 / (kBigGamma * h), L, nullptr);
    double ynew = 0.0, err = 0.0;
    const bool ok = rodas_attempt_big<NR>(M, L, p, y, f0, h, ynew, err);
    if (!ok) { ynew = NAN; err = NAN; }
    if (own < n && (tid & 1) == 0) {
        ynew_out[cell * n + own] = ynew;
        err_out[cell * n + own] = err;
    }
}

// ---------------------------------------------------------------- host ------
size_t big_lds_bytes(int n) { return sizeof(double) * big_lds_doubles(n); }

// Rows per lane of a panel: two up to 128 unknowns, three beyond (the LDS ends
// at 138).
static int big_rows(int n) { return n <= 128 ? 2 : 3; }

// Three threads a column in four wavefronts.
static bool small_group(int n) { return 3 * n <= 256; }

static hipError_t set_lds(const void *k, size_t sh) {
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
}

hipError_t big_prepare(int n) {
    const size_t sh = big_lds_bytes(n);
    const bool two = big_rows(n) == 2;
    hipError_t e;
    if ((e = set_lds(two ? (const void *)k_big_plain<2> : (const void *)k_big_plain<3>, sh))) return e;
    if ((e = set_lds(two ? (const void *)k_big_queue<2> : (const void *)k_big_queue<3>, sh))) return e;
    if ((e = set_lds(small_group(n) ? (const void *)k_big_rhs_jac<256> : (const void *)k_big_rhs_jac<BT>, sh))) return e;
    return set_lds(two ? (const void *)k_big_rodas_step<2> : (const void *)k_big_rodas_step<3>, sh);
}

template <int NR>
static void launch_big(const MechDev &M, const MechDev *Md, const IntParams &P, int schedule, int grid,
                       hipStream_t s) {
    const size_t sh = big_lds_bytes(M.n);
    if (schedule != 1)   // plain round robin, or static blocks (P.block_static)
        hipLaunchKernelGGL(k_big_plain<NR>, dim3((unsigned)grid), dim3(BT), sh, s, Md, P);
    else
        hipLaunchKernelGGL(k_big_queue<NR>, dim3((unsigned)grid), dim3(BT), sh, s, Md, P);
}

hipError_t launch_integrate_big(const MechDev &M, const MechDev *Md, const IntParams &P,
                                int schedule, int grid, hipStream_t s) {
    if (big_rows(M.n) == 2) launch_big<2>(M, Md, P, schedule, grid, s);
    else launch_big<3>(M, Md, P, schedule, grid, s);
    return hipGetLastError();
}

hipError_t launch_big_rhs_jac(const MechDev &M, const MechDev *Md, const IntParams &P, double *f,
                              double *J, hipStream_t s) {
    const size_t sh = big_lds_bytes(M.n);
    each_launch(P, [&](const IntParams &Q, unsigned cells) {
        if (small_group(M.n))
            hipLaunchKernelGGL(k_big_rhs_jac<256>, dim3(cells), dim3(256), sh, s, Md, Q, f, J);
        else
            hipLaunchKernelGGL(k_big_rhs_jac<BT>, dim3(cells), dim3(BT), sh, s, Md, Q, f, J);
    });
    return hipGetLastError();
}

hipError_t launch_big_rodas_step(const MechDev &M, const MechDev *Md, const IntParams &P, double h,
                                 double *ynew, double *err, hipStream_t s) {
    const size_t sh = big_lds_bytes(M.n);
    each_launch(P, [&](const IntParams &Q, unsigned cells) {
        if (big_rows(M.n) == 2)
            hipLaunchKernelGGL(k_big_rodas_step<2>, dim3(cells), dim3(BT), sh, s, Md, Q, h, ynew, err);
        else
            hipLaunchKernelGGL(k_big_rodas_step<3>, dim3(cells), dim3(BT), sh, s, Md, Q, h, ynew, err);
    });
    return hipGetLastError();
}

int big_occupancy(int n) {
    int blocks = 0;
    const size_t sh = big_lds_bytes(n);
    const hipError_t e = big_rows(n) == 2
        ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_big_queue<2>, BT, sh)
        : hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_big_queue<3>, BT, sh);
    return e == hipSuccess ? blocks : 0;
}

}  // namespace chem
