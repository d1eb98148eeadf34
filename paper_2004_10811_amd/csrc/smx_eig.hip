// Batched symmetric eigensolver of the submatrices (Sec. IV-F: the paper's
// production path diagonalises every submatrix, A_g = Q Lambda Q^T, and takes
// D_g = Q f(Lambda) Q^T with f the Fermi function at finite temperature, or
// the signum of Eq. signev at T = 0; Algorithm 1 of Sec. IV-G then finds mu
// from the stored decompositions without solving again).
//
// Four stages, each one launch over all groups of a wave:
//   1. Householder reduction A_g = Q T Q^T to symmetric tridiagonal form, one
//      512-lane workgroup per group (the reflectors stay in the slab, below
//      the subdiagonal, as in LAPACK's sytrd), then splitting of T where an
//      off-diagonal entry is negligible;
//   2. eigenvalues of T by bisection on Sturm counts, one lane per eigenvalue
//      (each unreduced block on its own);
//   3. eigenvectors of T by twisted factorisations, one lane per eigenvalue;
//      clusters of nearly equal eigenvalues by inverse iteration with
//      orthogonalisation;
//   4. the group's own columns only (that is all D needs): Y = Q^T E (E the
//      own-column selector; reflectors applied to a thin block), C = S^T Y
//      (S the eigenvectors of T; C's rows give Algorithm 1's weights
//      w_l = sum_c C_lc^2 = sum_{c in own} Q_cl^2), Z = S diag(g) C and
//      G = Q Z = Q diag(g) Q^T E with g = 1 - 2 f = tanh(lambda / 2kT) (signum
//      at T = 0, 0 for |lambda| <= 1e-14 ||A_g||_inf).  D's own columns are
//      (E - G) / 2, which the scatter of the sign path forms.
#include "smx_internal.h"

#include <algorithm>

namespace smx {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// lanes of the reduction workgroups: two waves per SIMD, so that the
// compiler may hold 256 registers and keep eight loads per lane in flight in
// the row dots of A_s v (at 1024 lanes and 128 registers it issued them one
// at a time)
constexpr int kEigBlock = 512;
constexpr int kReflBlock = 512;     // lanes of the reflector workgroups

// Sum over a kEigBlock-lane workgroup in a fixed order (lanes by a xor tree, lane
// 0's value per wave, then the waves in order); every lane gets the same bits.
__device__ inline double block_sum(double v, double *red)
{
    const int tid = threadIdx.x;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((tid & 63) == 0) red[tid >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < kEigBlock / 64; w++) s += red[w];
    __syncthreads();
    return s;
}

__device__ inline double wave_sum0(double v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return __shfl(v, 0, 64);
}

// ---- 1. Householder tridiagonalisation --------------------------------------
// Step k (0 <= k < n - 2): x = A[k+1:, k]; the reflector H_k = I - tau v v^T
// (v_0 = 1) maps x to beta e_1 (beta = -sign(x_0) ||x||, tau = (beta - x_0) /
// beta); with p = tau A22 v and w = p - (tau / 2)(p^T v) v the trailing block
// becomes A22 - v w^T - w v^T.  d_k = A_kk, e_k = beta; v is stored in
// A[k+1:, k].  A is column-major with leading dimension n_pad (full storage).
//
// Blocked as in LAPACK's sytrd: the steps of a panel of kPanel columns leave
// the trailing block as it was at the panel's start (A_s) and keep their
// vectors V (in A's columns) and W (n_pad x kPanel, in the second slab); a
// step first brings its own column up to date, A[:, k] -= V W[k, :]^T + W
// V[k, :]^T, and forms p = tau (A_s v - V (W^T v) - W (V^T v)); after the
// panel one pass applies A22 -= V W^T + W V^T to the trailing block.  Each
// step then reads the trailing block once instead of reading it twice and
// writing it once.
// sum over columns jj in [jb, je) of row[jj * ld] * v[jj], with eight partial
// sums in flight (eight independent loads per lane) added in a fixed order
__device__ inline double row_dot(const double *__restrict__ row, int ld, const double *v, int jb, int je)
{
    double a[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int jj = jb;
    for (; jj + 7 < je; jj += 8) {
#pragma unroll
        for (int u = 0; u < 8; u++) a[u] += row[(int64_t)(jj + u) * ld] * v[jj + u];
    }
    for (; jj < je; jj++) a[0] += row[(int64_t)jj * ld] * v[jj];
    return ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
}

constexpr int kPanel = 16;
constexpr int kTrailCols = 64;      // columns of V and W rows staged per trailing-update pass

// Sum over the 64 lanes of each of 16 values: lane l returns the sum of
// val[l % 16].  Each of the first four exchanges halves the values a lane
// carries, so the whole takes 17 exchanges instead of 6 for every value.
__device__ inline double lane_sums16(const double (&val)[16], int lane)
{
    double a[8], b[4], c[2], d;
#pragma unroll
    for (int u = 0; u < 8; u++) {
        const bool hi = lane & 8;
        a[u] = (hi ? val[u + 8] : val[u]) + __shfl_xor(hi ? val[u] : val[u + 8], 8, 64);
    }
#pragma unroll
    for (int u = 0; u < 4; u++) {
        const bool hi = lane & 4;
        b[u] = (hi ? a[u + 4] : a[u]) + __shfl_xor(hi ? a[u] : a[u + 4], 4, 64);
    }
#pragma unroll
    for (int u = 0; u < 2; u++) {
        const bool hi = lane & 2;
        c[u] = (hi ? b[u + 2] : b[u]) + __shfl_xor(hi ? b[u] : b[u + 2], 2, 64);
    }
    {
        const bool hi = lane & 1;
        d = (hi ? c[1] : c[0]) + __shfl_xor(hi ? c[0] : c[1], 1, 64);
    }
    d += __shfl_xor(d, 16, 64);
    d += __shfl_xor(d, 32, 64);
    return d;
}

// A_s v from the lower triangle alone, rows and columns k0 .. n - 1 (vs is
// zero outside [k0, n)): an element a_ij (i > j) adds a v_j to row i and a v_i
// to row j.  A wave takes strips of 16 columns and runs down each in pieces of
// 64 rows; the column sums stay in registers until the strip's end, the row
// sums go to the wave's own acc[wave][.], which starts at zero (the caller adds
// the waves' sums in order).  Strips go to the waves back and forth, so that
// each wave gets about the same number of pieces.  A piece's 16 loads are in
// flight while the previous piece is worked on (two register sets in turn,
// loads unconditional: rows and columns beyond n read the last one).
template <int NR>
__device__ inline void sym_mv(const double *__restrict__ A, int ld, int n, int k0, const double *vs,
                              double (*acc)[NR], int lane, int wave)
{
    constexpr int NWV = kEigBlock / 64;
    const int nch = (n + 63) / 64, nst = (n + 15) / 16;
    int round = 0, s = k0 / 16 + wave, c = s >> 2;
    if (s >= nst) return;
    auto load = [&](int ss, int cc, double (&r)[16]) {
        const unsigned row = (unsigned)min(64 * cc + lane, n - 1);
#pragma unroll
        for (int u = 0; u < 16; u++) r[u] = (A + (int64_t)min(16 * ss + u, n - 1) * ld)[row];
    };
    double vj[16], col[16];
    auto begin = [&](int ss) {
#pragma unroll
        for (int u = 0; u < 16; u++) {
            vj[u] = vs[16 * ss + u];
            col[u] = 0.0;
        }
    };
    // one piece; `last`: no piece follows.  Returns false after the last one.
    auto step = [&](const double (&cur)[16], double (&nxt)[16]) -> bool {
        int s2 = s, c2 = c + 1, round2 = round;
        if (c2 >= nch) {                               // next strip of this wave
            round2++;
            s2 = k0 / 16 + round2 * NWV + ((round2 & 1) ? NWV - 1 - wave : wave);
            c2 = s2 >> 2;
        }
        const bool last = s2 >= nst;
        load(last ? s : s2, last ? c : c2, nxt);
        const int i = 64 * c + lane;
        const double vi = vs[i];
        double y0 = 0.0, y1 = 0.0;
        if (c > (s >> 2)) {
#pragma unroll
            for (int u = 0; u < 16; u += 2) {
                y0 += cur[u] * vj[u];
                y1 += cur[u + 1] * vj[u + 1];
                col[u] += cur[u] * vi;
                col[u + 1] += cur[u + 1] * vi;
            }
        } else {                                       // the piece meets the diagonal
#pragma unroll
            for (int u = 0; u < 16; u++) {
                const int j = 16 * s + u;
                y0 += i >= j ? cur[u] * vj[u] : 0.0;
                col[u] += i > j ? cur[u] * vi : 0.0;
            }
        }
        acc[wave][i] += y0 + y1;
        if (s2 != s || last) {
            const double sum = lane_sums16(col, lane);
            if (lane < 16) acc[wave][16 * s + lane] += sum;
            if (!last) begin(s2);
        }
        s = s2;
        c = c2;
        round = round2;
        return !last;
    };
    double ra[16], rb[16];
    load(s, c, ra);
    begin(s);
    for (;;) {
        if (!step(ra, rb)) break;
        if (!step(rb, ra)) break;
    }
}

// Trailing update of a panel, lower triangle from row and column k1 on:
// A_ij -= sum_q V_iq W_jq + W_iq V_jq, a product of n x 32 blocks [V W] [W V]^T
// on v_mfma_f64_16x16x4_f64.  The matrix core's row index is the matrix column
// and its column index the matrix row, so that 16 lanes hold 16 consecutive
// rows of a column.  Pieces of 64 rows x 16 columns, chunk of rows by chunk; the
// waves take a chunk's column strips in turn.  nb < 16 (the last panel): the
// missing columns of V and W count as zero.
__device__ inline void sym_rank32(double *__restrict__ A, const double *__restrict__ V, const double *__restrict__ W,
                                  int ld, int n, int k1, int nb, int lane, int wave)
{
    constexpr int NWV = kEigBlock / 64;
    const int li = lane & 15, lq = lane >> 4;
    const int nch = (n - k1 + 63) / 64;
    // lane (li, lq), t: column 4 t + lq of [V W] (vw) or [W V] at row r
    auto frag = [&](const double *__restrict__ F, const double *__restrict__ S, int r, double (&f)[8]) {
        const int rr = min(r, n - 1);
#pragma unroll
        for (int t = 0; t < 8; t++) {
            const int q = (4 * t + lq) & 15;
            const double v = (t < 4 ? F : S)[rr + (int64_t)min(q, nb - 1) * ld];
            f[t] = q < nb ? v : 0.0;
        }
    };
    for (int c = 0; c < nch; c++) {
        const int r0 = k1 + 64 * c;
        const int ns = min(4 * c + 4, (n - k1 + 15) / 16);     // strips up to the diagonal
        if (wave >= ns) continue;
        double q[4][8];
#pragma unroll
        for (int b = 0; b < 4; b++) frag(V, W, r0 + 16 * b + li, q[b]);
        for (int s = wave; s < ns; s += NWV) {
            double p[8], x[4][4];
            const int j0 = k1 + 16 * s;
#pragma unroll
            for (int b = 0; b < 4; b++)
#pragma unroll
                for (int v = 0; v < 4; v++)
                    x[b][v] = A[min(r0 + 16 * b + li, n - 1) + (int64_t)min(j0 + lq + 4 * v, n - 1) * ld];
            frag(W, V, j0 + li, p);
            f64x4 d[4];
#pragma unroll
            for (int b = 0; b < 4; b++) d[b] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int t = 0; t < 8; t++)
#pragma unroll
                for (int b = 0; b < 4; b++)
                    d[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[t], q[b][t], d[b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < 4; b++)
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const int i = r0 + 16 * b + li, j = j0 + lq + 4 * v;
                    if (i < n && j <= i) A[i + (int64_t)j * ld] = x[b][v] - d[b][v];
                }
        }
    }
}

// sum_q V_iq a_q + W_iq b_q over q < j in order, eight columns of both loaded
// at a time (columns beyond j read column 0 and count as zero: j >= 1).
__device__ inline double panel_row(const double *__restrict__ V, const double *__restrict__ W, int ld, int i, int j,
                                   const double *a, const double *b, double s)
{
    for (int q0 = 0; q0 < j; q0 += 8) {
        double v[8], w[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int64_t o = (int64_t)(q0 + u < j ? q0 + u : 0) * ld;
            v[u] = V[i + o];
            w[u] = W[i + o];
        }
#pragma unroll
        for (int u = 0; u < 8; u++)
            if (q0 + u < j) s -= v[u] * a[q0 + u] + w[u] * b[q0 + u];
    }
    return s;
}

constexpr int kHalfMaxN = kEigHalfMaxN;

// HALF: the trailing block is read and kept up to date in its lower triangle
// only, n <= kHalfMaxN; otherwise in full, larger n.  A launch covers all groups
// and returns at once from those of the other kind; where a wave has both kinds, the
// two launches run side by side (launch_eig_tridiag).
//
// What bounds it: HBM.  With one group per CU the trailing blocks (5.8 MB each
// at n = 850) stay in no cache, and A_s v reads them once per step.  water256 at
// kT = 0.01 (n 700-1053), whole reduction: 130 ms reading the full block, 87 ms
// from the triangle with the column sums reduced over the lanes for every
// piece, 72 ms with the column sums kept down a strip, the trailing update on
// the matrix cores (on the vector units it was bound by its LDS reads of V and
// W) and the panel's rows and dot products loaded eight at a time.  Of a group
// of n = 799, A_s v then takes 30 of 47 ms at 23 GB/s per CU, 5.8 TB/s over the
// chip.  32 groups of n ~ 330 (latency): 10.3, 11.9, 8.7 ms.
template <bool HALF>
__global__ __launch_bounds__(kEigBlock)
void tridiag_kernel(const GroupDesc *__restrict__ groups, int g0, double *__restrict__ abase,
                    double *__restrict__ wbase, EigVecs ev)
{
    constexpr int NR = HALF ? kHalfMaxN : kEigMaxN;
    __shared__ double vs[NR + 64];                    // v; zero outside it
    __shared__ double ws[NR];
    __shared__ double red[kEigBlock / 64];
    __shared__ double rowk[2 * kPanel];               // V[k, t], W[k, t] of the panel's earlier steps
    __shared__ double dots[2 * kPanel];               // W[:, t]^T v, V[:, t]^T v
    __shared__ double vwc[HALF ? 1 : kTrailCols][2 * kPanel];    // V[c, t], W[c, t] of a run of trailing columns
    __shared__ double psum[HALF ? 1 : kEigBlock];     // column-part sums of A_s v
    __shared__ double acc[HALF ? kEigBlock / 64 : 1][HALF ? NR : 1];   // the waves' sums of A_s v
    const int g = g0 + blockIdx.x;
    const GroupDesc gd = groups[g];
    const int n = gd.n, ld = gd.npad, tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double *A = abase + gd.off;
    double *W = wbase + gd.off;                       // W[:, t] at W + t * ld (kPanel <= 32 <= n_pad)
    double *d = ev.d + gd.rinfo_off, *e = ev.e + gd.rinfo_off, *tau = ev.tau + gd.rinfo_off;
    if ((n <= kHalfMaxN) != HALF) return;
    for (int i = tid; i < NR + 64; i += kEigBlock) vs[i] = 0.0;
    __syncthreads();
    for (int kp = 0; kp + 2 < n; kp += kPanel) {
        const int nb = min(kPanel, n - 2 - kp);
        const double *V = A + (int64_t)kp * ld;       // V[:, t] = A[:, kp + t] below its subdiagonal
        bool any = false;                             // a reflector of the panel is not the identity
        for (int j = 0; j < nb; j++) {
            const int k = kp + j;
            double *col = A + (int64_t)k * ld;
            // column k (rows k ..) up to date with the panel's steps 0 .. j - 1
            if (tid < j) {
                rowk[tid] = V[k + (int64_t)tid * ld];
                rowk[kPanel + tid] = W[k + (int64_t)tid * ld];
            }
            __syncthreads();
            if (j > 0)
                for (int i = k + tid; i < n; i += kEigBlock) col[i] = panel_row(V, W, ld, i, j, rowk + kPanel, rowk, col[i]);
            __syncthreads();
            const double x0 = col[k + 1];             // read by every lane before the barrier in
            double part = 0.0;                        // block_sum; lane 0 overwrites it with v_0 below
            for (int i = k + 2 + tid; i < n; i += kEigBlock) part += col[i] * col[i];
            const double sigma = block_sum(part, red);
            double beta = x0, tk = 0.0, sc = 0.0;
            if (sigma > 0.0) {
                const double nrm = sqrt(x0 * x0 + sigma);
                beta = x0 >= 0.0 ? -nrm : nrm;
                tk = (beta - x0) / beta;
                sc = 1.0 / (x0 - beta);
            }
            for (int i = k + 1 + tid; i < n; i += kEigBlock) {
                const double vi = (i == k + 1) ? 1.0 : col[i] * sc;
                vs[i] = vi;
                col[i] = vi;
            }
            if (tid == 0) {
                d[k] = col[k];
                e[k] = beta;
                tau[k] = tk;
                vs[k] = 0.0;                          // sym_mv reads whole 64-row chunks
            }
            if constexpr (HALF) {
                for (int i = ((k + 1) & ~63) + tid; i < ((n + 63) & ~63); i += kEigBlock)
#pragma unroll
                    for (int w = 0; w < kEigBlock / 64; w++) acc[w][i] = 0.0;
            }
            __syncthreads();
            double *wj = W + (int64_t)j * ld;
            any = any || tk != 0.0;                   // the same in every lane
            if (tk != 0.0) {
                // W[:, q]^T v and V[:, q]^T v over rows k + 1 .., one wave per product,
                // eight loads in flight (rows beyond n read row n - 1, where v is zero)
                for (int q = wave; q < 2 * j; q += kEigBlock / 64) {
                    const double *src = q < j ? W + (int64_t)q * ld : V + (int64_t)(q - j) * ld;
                    double s = 0.0;
                    for (int i0 = k + 1 + lane; i0 < n; i0 += 512) {
                        double r[8];
#pragma unroll
                        for (int u = 0; u < 8; u++) r[u] = src[min(i0 + 64 * u, n - 1)];
#pragma unroll
                        for (int u = 0; u < 8; u++)
                            if (i0 + 64 * u < n) s += r[u] * vs[i0 + 64 * u];
                    }
                    s = wave_sum0(s);
                    if (lane == 0) dots[q] = s;
                }
                __syncthreads();
                // p = tau (A_s v - V (W^T v) - W (V^T v)).  A_s v: the lanes of a
                // row slot read consecutive rows of a column (coalesced); while the
                // trailing block has at most kEigBlock rows, the columns are split into
                // kEigBlock / (rows rounded up to 64) parts so every lane streams,
                // and the parts' sums are added in order
                const int R = n - k - 1;
                if constexpr (HALF) {
                    sym_mv<NR>(A, ld, n, k + 1, vs, acc, lane, wave);
                    __syncthreads();
                    for (int i = k + 1 + tid; i < n; i += kEigBlock) {
                        double s = 0.0;
#pragma unroll
                        for (int w = 0; w < kEigBlock / 64; w++) s += acc[w][i];
                        ws[i] = tk * panel_row(V, W, ld, i, j, dots, dots + j, s);
                    }
                } else if (R <= kEigBlock) {
                    const int RS = (R + 63) & ~63, P = kEigBlock / RS;
                    const int sl = tid % RS, part = tid / RS;
                    if (part < P) {
                        double acc = 0.0;
                        if (sl < R) {
                            const int i = k + 1 + sl, cl = (R + P - 1) / P;
                            const int jb = k + 1 + part * cl, je = min(n, jb + cl);
                            acc = row_dot(A + i, ld, vs, jb, je);
                        }
                        psum[part * RS + sl] = acc;
                    }
                    __syncthreads();
                    for (int sl2 = tid; sl2 < R; sl2 += kEigBlock) {
                        double s = 0.0;
                        for (int pp = 0; pp < P; pp++) s += psum[pp * RS + sl2];
                        const int i = k + 1 + sl2;
                        ws[i] = tk * panel_row(V, W, ld, i, j, dots, dots + j, s);
                    }
                } else {
                    for (int i = k + 1 + tid; i < n; i += kEigBlock) {
                        double s = row_dot(A + i, ld, vs, k + 1, n);
                        ws[i] = tk * panel_row(V, W, ld, i, j, dots, dots + j, s);
                    }
                }
                __syncthreads();
                double pv = 0.0;
                for (int i = k + 1 + tid; i < n; i += kEigBlock) pv += ws[i] * vs[i];
                const double kk = -0.5 * tk * block_sum(pv, red);
                for (int i = k + 1 + tid; i < n; i += kEigBlock) wj[i] = ws[i] + kk * vs[i];
            } else {
                for (int i = k + 1 + tid; i < n; i += kEigBlock) wj[i] = 0.0;
            }
            __syncthreads();
        }
        // trailing block (rows and columns from k1 on): A -= V W^T + W V^T over the panel
        const int k1 = kp + nb;
        if (HALF && any) sym_rank32(A, V, W, ld, n, k1, nb, lane, wave);
        for (int c0 = k1; !HALF && any && c0 < n; c0 += kTrailCols) {
            const int ncol = min(kTrailCols, n - c0);
            __syncthreads();
            for (int u = tid; u < kTrailCols * 2 * kPanel; u += kEigBlock) {
                const int cl = u / (2 * kPanel), q = u % (2 * kPanel);
                const int qq = q % kPanel;
                double v = 0.0;
                if (cl < ncol && qq < nb) v = (q < kPanel ? V : W)[c0 + cl + (int64_t)qq * ld];
                vwc[cl][q] = v;
            }
            __syncthreads();
            for (int r = k1 + tid; r < n; r += kEigBlock) {
                double vr[kPanel], wr[kPanel];
#pragma unroll
                for (int q = 0; q < kPanel; q++) {
                    vr[q] = q < nb ? V[r + (int64_t)q * ld] : 0.0;
                    wr[q] = q < nb ? W[r + (int64_t)q * ld] : 0.0;
                }
                // Eight columns' entries of the row at a time (the row is this
                // lane's alone, and V's columns lie left of k1); the next eight
                // are loaded, unconditionally (columns past the chunk read its last
                // one), before this batch is updated and stored, into two
                // register sets in turn, so no load waits behind the stores.
                auto load8 = [&](int cb, double (&dst)[8]) {
#pragma unroll
                    for (int u = 0; u < 8; u++) dst[u] = A[r + (int64_t)(c0 + min(cb + u, ncol - 1)) * ld];
                };
                auto update8 = [&](int cb, const double (&src)[8]) {
#pragma unroll
                    for (int u = 0; u < 8; u++) {
                        if (cb + u >= ncol) break;
                        const int cl = cb + u;
                        double s = src[u];
#pragma unroll
                        for (int q = 0; q < kPanel; q++) s -= vr[q] * vwc[cl][kPanel + q] + wr[q] * vwc[cl][q];
                        A[r + (int64_t)(c0 + cl) * ld] = s;
                    }
                };
                double ba[8], bb[8];
                load8(0, ba);
                for (int cb = 0; cb < ncol; cb += 16) {
                    load8(cb + 8, bb);
                    update8(cb, ba);
                    if (cb + 8 >= ncol) break;
                    load8(cb + 16, ba);
                    update8(cb + 8, bb);
                }
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        if (n >= 2) {
            d[n - 2] = A[(n - 2) + (int64_t)(n - 2) * ld];
            e[n - 2] = A[(n - 1) + (int64_t)(n - 2) * ld];
            tau[n - 2] = 0.0;
            d[n - 1] = A[(n - 1) + (int64_t)(n - 1) * ld];
        } else {
            d[0] = A[0];
        }
        e[n - 1] = 0.0;
        if (n >= 1) tau[n - 1] = 0.0;
    }
}

// Split T into unreduced blocks: e_i is set to 0 where |e_i| <= 2u ||T||_inf
// (u the FP64 unit roundoff; a change of T of the size of the reduction's own
// rounding) or |e_i| <= u (|d_i| + |d_{i+1}|); bs[i] / be[i] are the first row
// and one past the last row of the block holding row i.  One workgroup per
// group, a run of consecutive rows per lane; the lanes' last (first) block ends
// are scanned forwards (backwards).  One lane per group walked the rows at one
// memory round trip each: 1.9 ms on water256, under 0.05 ms this way.
__global__ __launch_bounds__(256)
void split_kernel(const GroupDesc *__restrict__ groups, int g0, EigVecs ev)
{
    constexpr int RPL = kEigMaxN / 256;               // rows per lane
    __shared__ double red[4];
    __shared__ int fwd[256], bwd[256];
    const GroupDesc gd = groups[g0 + blockIdx.x];
    const int n = gd.n, tid = threadIdx.x;
    double *d = ev.d + gd.rinfo_off, *e = ev.e + gd.rinfo_off;
    int32_t *bs = ev.bs + gd.rinfo_off, *be = ev.be + gd.rinfo_off;
    double tn = 0.0;
    for (int i = tid; i < n; i += 256)
        tn = fmax(tn, fabs(d[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0));
    for (int o = 32; o > 0; o >>= 1) tn = fmax(tn, __shfl_xor(tn, o, 64));
    if ((tid & 63) == 0) red[tid >> 6] = tn;
    __syncthreads();
    tn = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    // bit u of `ends`: row i0 + u ends a block
    const int i0 = tid * RPL;
    unsigned ends = 0;
#pragma unroll
    for (int u = 0; u < RPL; u++) {
        const int i = i0 + u;
        if (i >= n) break;
        if (i == n - 1) {
            ends |= 1u << u;
        } else if (fabs(e[i]) <= 2.220446049250313e-16 * tn ||
                   fabs(e[i]) <= 1.1102230246251565e-16 * (fabs(d[i]) + fabs(d[i + 1]))) {
            e[i] = 0.0;
            ends |= 1u << u;
        }
    }
    fwd[tid] = ends ? i0 + 32 - __builtin_clz(ends) : 0;        // row after the lane's last end
    bwd[tid] = ends ? i0 + __builtin_ctz(ends) + 1 : n;         // row after its first end
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {               // inclusive max from below, min from above
        const int f = tid >= o ? fwd[tid - o] : 0, w = tid + o < 256 ? bwd[tid + o] : n;
        __syncthreads();
        fwd[tid] = max(fwd[tid], f);
        bwd[tid] = min(bwd[tid], w);
        __syncthreads();
    }
    int first = tid > 0 ? fwd[tid - 1] : 0;
    const int after = tid < 255 ? bwd[tid + 1] : n;
#pragma unroll
    for (int u = 0; u < RPL; u++) {
        const int i = i0 + u;
        if (i >= n) break;
        const unsigned rest = ends >> u;
        bs[i] = first;
        be[i] = rest ? i + __builtin_ctz(rest) + 1 : after;
        if (ends & (1u << u)) first = i + 1;
    }
}

// Number of eigenvalues of the block T[s:t, s:t] below x: the sign changes of
// the leading principal minors of T - x I, p_i = (d_i - x) p_{i-1} - e_{i-1}^2
// p_{i-2}.  T is scaled so that ||T|| <= 1 and |e| >= 2^-55 inside a block, so
// eight steps change a pair of minors by less than 2^-450 or 2^24; they are then
// scaled by a power of two.  A minor of either zero counts one change with its
// neighbours.  (d_i, e_{i-1}^2) staged in LDS by the caller.
__device__ inline int sturm_count(const double2 *de, int s, int t, double x)
{
    double p0 = 1.0, p1 = de[s].x - x;
    unsigned cnt = (unsigned)__double2hiint(p1) >> 31;
    auto step = [&](const double2 q) {
        const double p2 = fma(q.x - x, p1, -(q.y * p0));
        cnt += (unsigned)(__double2hiint(p2) ^ __double2hiint(p1)) >> 31;
        p0 = p1;
        p1 = p2;
    };
    int i = s + 1;
    for (; i + 8 <= t; i += 8) {
        double2 q[8];
#pragma unroll
        for (int u = 0; u < 8; u++) q[u] = de[i + u];
#pragma unroll
        for (int u = 0; u < 8; u++) step(q[u]);
        const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
        p0 = __builtin_amdgcn_ldexp(p0, -e);
        p1 = __builtin_amdgcn_ldexp(p1, -e);
    }
    for (; i < t; i++) step(de[i]);
    return (int)cnt;
}

// ---- 2. eigenvalues by bisection --------------------------------------------
// Lane l of group g finds the (l - s)-th smallest eigenvalue of its block
// [s, t) (ascending within each block), inside the block's Gershgorin
// interval, to the width of a few units in the last place.  The workgroup
// first stages d and e^2 of its group in LDS, scaled by the power of two that
// brings ||T|| below 1 (exact; the eigenvalue is scaled back): every Sturm
// count then reads them there (the lanes of a wave mostly at the same index:
// broadcasts) instead of waiting on a global load per recurrence step.
// Bound by instruction issue: the counts' steps.  The recurrence of the minors
// takes no division (the ratio q_i = d_i - x - e^2 / q_{i-1} does): water256
// 3.5 against 13.1 ms.
__global__ __launch_bounds__(256)
void bisect_kernel(const GroupDesc *__restrict__ groups, int g0, EigVecs ev)
{
    __shared__ double2 de[kEigMaxN];
    __shared__ double red[4];
    const int g = g0 + blockIdx.y;
    const GroupDesc gd = groups[g];
    const int l = blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x * 256 >= gd.n) return;             // whole workgroup beyond this group
    const double *d = ev.d + gd.rinfo_off, *e = ev.e + gd.rinfo_off;
    double tg = 0.0;                                  // ||T||_inf, up to a factor of 3
    for (int i = threadIdx.x; i < gd.n; i += 256) tg = fmax(tg, fmax(fabs(d[i]), fabs(e[i])));
    for (int o = 32; o > 0; o >>= 1) tg = fmax(tg, __shfl_xor(tg, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = tg;
    __syncthreads();
    tg = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    const int sc = tg > 0.0 ? __builtin_amdgcn_frexp_exp(tg) + 2 : 0;
    for (int i = threadIdx.x; i < gd.n; i += 256) {
        const double ep = i > 0 ? __builtin_amdgcn_ldexp(e[i - 1], -sc) : 0.0;
        de[i] = double2{__builtin_amdgcn_ldexp(d[i], -sc), ep * ep};
    }
    __syncthreads();
    if (l >= gd.n) return;
    const int s = ev.bs[gd.rinfo_off + l], t = ev.be[gd.rinfo_off + l], m = l - s;
    double lo = 1.0, hi = -1.0, tn = 0.0;
    for (int i = s; i < t; i++) {
        const double r = (i > s ? sqrt(de[i].y) : 0.0) + (i + 1 < t ? sqrt(de[i + 1].y) : 0.0);
        lo = fmin(lo, de[i].x - r);
        hi = fmax(hi, de[i].x + r);
        tn = fmax(tn, fabs(de[i].x) + r);
    }
    const double pad = 8.881784197001252e-16 * tn + 1e-300;
    lo -= pad;
    hi += pad;
    // count(lo) <= m < count(hi)
    for (int it = 0; it < 400; it++) {
        const double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi) break;
        if (hi - lo <= 4.440892098500626e-16 * fmax(fabs(lo), fabs(hi)) + 2.220446049250313e-16 * tn + 1e-300) break;
        if (sturm_count(de, s, t, mid) > m) hi = mid;
        else lo = mid;
    }
    ev.lam[gd.rinfo_off + l] = __builtin_amdgcn_ldexp(0.5 * (lo + hi), sc);
}

// ---- 3. eigenvectors by twisted factorisations ------------------------------
// For lambda of block [s, t): the stationary factorisation T - lambda I =
// L+ D+ L+^T from the top (D+_s = d_s - lambda, L+_i = e_i / D+_i,
// D+_{i+1} = d_{i+1} - lambda - L+_i e_i) and the progressive one from the
// bottom (D-_{t-1} = d_{t-1} - lambda, U-_i = e_i / D-_{i+1},
// D-_i = d_i - lambda - U-_i e_i) meet at the twist r minimising |gamma_r|,
// gamma_r = D+_r + D-_r - (d_r - lambda); the eigenvector then follows from
// z_r = 1, z_i = -L+_i z_{i+1} (i < r), z_{i+1} = -U-_i z_i (i >= r).
// S[i * n_pad + l] holds component i of eigenvector l (U-_i is parked there
// at row i + 1 until z overwrites it); lbuf holds D- and then L+.
template <int NR>
__global__ __launch_bounds__(256)
void tvec_kernel(const GroupDesc *__restrict__ groups, int g0, EigVecs ev, double *__restrict__ sbase,
                 double *__restrict__ lbase)
{
    const int g = g0 + blockIdx.y;
    const GroupDesc gd = groups[g];
    const int l = blockIdx.x * 256 + threadIdx.x;
    const int ld = gd.npad;
    __shared__ double d[NR], e[NR];
    if ((int)blockIdx.x * 256 >= ld) return;          // whole workgroup beyond this group
    for (int i = threadIdx.x; i < gd.n; i += 256) {
        d[i] = ev.d[gd.rinfo_off + i];
        e[i] = ev.e[gd.rinfo_off + i];
    }
    __syncthreads();
    if (l >= ld) return;
    double *S = sbase + gd.off;
    double *Lb = lbase + gd.off;
    if (l >= gd.n) {                       // padding: the identity's columns
        for (int i = 0; i < ld; i++) S[(int64_t)i * ld + l] = (i == l) ? 1.0 : 0.0;
        return;
    }
    const int s = ev.bs[gd.rinfo_off + l], t = ev.be[gd.rinfo_off + l];
    const double lam = ev.lam[gd.rinfo_off + l];
    double emax = 0.0;
    for (int i = s; i + 1 < t; i++) emax = fmax(emax, fabs(e[i]));
    const double pivmin = 2.2250738585072014e-308 * fmax(1.0, emax * emax) * 1e10;
    auto guard = [&](double q) { return fabs(q) < pivmin ? (q < 0.0 ? -pivmin : pivmin) : q; };
    for (int i = 0; i < s; i++) S[(int64_t)i * ld + l] = 0.0;
    for (int i = t; i < ld; i++) S[(int64_t)i * ld + l] = 0.0;
    if (t - s == 1) {
        S[(int64_t)s * ld + l] = 1.0;
        return;
    }
    // progressive (bottom-up): D- into lbuf, U- into S one row down
    double dm = guard(d[t - 1] - lam);
    Lb[(int64_t)(t - 1) * ld + l] = dm;
    for (int i = t - 2; i >= s; i--) {
        const double u = e[i] / dm;
        S[(int64_t)(i + 1) * ld + l] = u;
        dm = guard(d[i] - lam - u * e[i]);
        Lb[(int64_t)i * ld + l] = dm;
    }
    // stationary (top-down): gamma at every row, L+ replaces D- in lbuf.  Here
    // and below eight rows are loaded at a time, all in flight before their use
    // (rows beyond the block read its last one and are not used; a break out of the
    // unrolled rows kept the compiler from that).  d and e are in LDS: a load from
    // memory waits for the stores issued before it.  256 groups of n ~ 855: 10.3 ms one
    // row at a time, 8.7 with eight, 7.9 with d and e in LDS and no breaks; 32 of ~ 390
    // 0.75, 0.66, 0.43 ms.
    double dp = guard(d[s] - lam);
    int r = s;
    double gbest = 1.7976931348623157e308;
    for (int i0 = s; i0 < t; i0 += 8) {
        double dmi[8];
#pragma unroll
        for (int u = 0; u < 8; u++) dmi[u] = Lb[(int64_t)min(i0 + u, t - 1) * ld + l];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int i = i0 + u;
            const double gam = dp + dmi[u] - (d[min(i, t - 1)] - lam);
            if (i < t && fabs(gam) < gbest) {
                gbest = fabs(gam);
                r = i;
            }
            if (i + 1 < t) {
                const double lp = e[i] / dp;
                Lb[(int64_t)i * ld + l] = lp;
                dp = guard(d[i + 1] - lam - lp * e[i]);
            }
        }
    }
    double nrm = 1.0;
    double z = 1.0;
    S[(int64_t)r * ld + l] = 1.0;
    for (int i0 = r - 1; i0 >= s; i0 -= 8) {
        double lp[8];
#pragma unroll
        for (int u = 0; u < 8; u++) lp[u] = Lb[(int64_t)max(i0 - u, s) * ld + l];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            if (i0 - u >= s) {
                z = -lp[u] * z;
                S[(int64_t)(i0 - u) * ld + l] = z;
                nrm += z * z;
            }
        }
    }
    z = 1.0;
    for (int i0 = r; i0 + 1 < t; i0 += 8) {
        double un[8];
#pragma unroll
        for (int u = 0; u < 8; u++) un[u] = S[(int64_t)min(i0 + u + 1, t - 1) * ld + l];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            if (i0 + u + 1 < t) {
                z = -un[u] * z;
                S[(int64_t)(i0 + u + 1) * ld + l] = z;
                nrm += z * z;
            }
        }
    }
    const double inv = 1.0 / sqrt(nrm);
    for (int i0 = s; i0 < t; i0 += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = S[(int64_t)min(i0 + u, t - 1) * ld + l];
#pragma unroll
        for (int u = 0; u < 8; u++)
            if (i0 + u < t) S[(int64_t)(i0 + u) * ld + l] = v[u] * inv;
    }
}

// Clusters: consecutive eigenvalues of one block closer than 1e-8 ||T|| (for
// instance the pairs of a degenerate spectrum when the reduction leaves them
// in one block) need not get independent vectors from twisted
// factorisations.  The lane of a cluster's first member recomputes all its
// vectors by inverse iteration with orthogonalisation against the members
// already done (as LAPACK's stein does): three steps of
// (T - lambda I) y = x by the LDL^T factorisation (pivots smaller than
// 1e-14 ||T|| raised to that size), each followed by modified Gram-Schmidt and
// normalisation, from deterministic start vectors that differ per member.
// Clusters are rare and small; everything else keeps its twisted vector.
__global__ __launch_bounds__(256)
void cluster_kernel(const GroupDesc *__restrict__ groups, int g0, EigVecs ev, double *__restrict__ sbase,
                    double *__restrict__ lbase)
{
    const int g = g0 + blockIdx.y;
    const GroupDesc gd = groups[g];
    const int l = blockIdx.x * 256 + threadIdx.x;
    if (l >= gd.n) return;
    const int ro = gd.rinfo_off, ld = gd.npad;
    const int s = ev.bs[ro + l], t = ev.be[ro + l];
    const double *lam = ev.lam + ro, *d = ev.d + ro, *e = ev.e + ro;
    double tn = 0.0;
    for (int i = s; i < t; i++)
        tn = fmax(tn, fabs(d[i]) + (i > s ? fabs(e[i - 1]) : 0.0) + (i + 1 < t ? fabs(e[i]) : 0.0));
    const double delta = 1e-8 * fmax(tn, 1e-300);
    auto close = [&](int a, int b) { return lam[b] - lam[a] <= delta; };
    if (l > s && close(l - 1, l)) return;            // not the first member
    if (l + 1 >= t || !close(l, l + 1)) return;      // a single eigenvalue
    int last = l + 1;
    while (last + 1 < t && close(last, last + 1)) last++;
    double *S = sbase + gd.off;
    double *Lb = lbase + gd.off;
    const double piv = 1e-14 * fmax(tn, 1e-300);
    for (int m = l; m <= last; m++) {
        double *x = S + m;                       // column m: x[i * ld]
        double *lm = Lb + m;
        for (int i = s; i < t; i++) x[(int64_t)i * ld] = 1.0 + 0.5 * sin(0.7 * (i - s + 1) * (m - l + 1) + m - l);
        for (int iter = 0; iter < 3; iter++) {
            // forward: LDL^T of T - lambda I with the solve of L z = x, w = D^-1 z
            double dd = d[s] - lam[m];
            if (fabs(dd) < piv) dd = dd < 0.0 ? -piv : piv;
            double z = x[(int64_t)s * ld];
            x[(int64_t)s * ld] = z / dd;
            for (int i = s; i + 1 < t; i++) {
                const double li = e[i] / dd;
                lm[(int64_t)i * ld] = li;
                dd = d[i + 1] - lam[m] - li * e[i];
                if (fabs(dd) < piv) dd = dd < 0.0 ? -piv : piv;
                z = x[(int64_t)(i + 1) * ld] - li * z;
                x[(int64_t)(i + 1) * ld] = z / dd;
            }
            // backward: L^T y = w
            for (int i = t - 2; i >= s; i--) x[(int64_t)i * ld] -= lm[(int64_t)i * ld] * x[(int64_t)(i + 1) * ld];
            // against the members already done, then normalise
            for (int p = l; p < m; p++) {
                double dot = 0.0;
                for (int i = s; i < t; i++) dot += S[(int64_t)i * ld + p] * x[(int64_t)i * ld];
                for (int i = s; i < t; i++) x[(int64_t)i * ld] -= dot * S[(int64_t)i * ld + p];
            }
            double nrm = 0.0;
            for (int i = s; i < t; i++) nrm += x[(int64_t)i * ld] * x[(int64_t)i * ld];
            const double inv = nrm > 0.0 ? 1.0 / sqrt(nrm) : 0.0;
            for (int i = s; i < t; i++) x[(int64_t)i * ld] *= inv;
        }
    }
}

// ---- 4. own columns ---------------------------------------------------------
// y (n_pad x m_own, column-major at thin_off) = the own-column selector E.
__global__ __launch_bounds__(256)
void own_select_kernel(const GroupDesc *__restrict__ groups, const int32_t *__restrict__ own_list, int g0,
                       double *__restrict__ y)
{
    const GroupDesc gd = groups[g0 + blockIdx.y];
    const int64_t tot = (int64_t)gd.npad * gd.m_own;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < tot; q += (int64_t)gridDim.x * 256) {
        const int r = (int)(q % gd.npad), c = (int)(q / gd.npad);
        y[gd.thin_off + q] = (r == own_list[gd.own_off + c]) ? 1.0 : 0.0;
    }
}

// The reflectors applied to a thin block, 16 at a time in compact WY form:
// H_a ... H_{a+15} = I - V T V^T with T upper triangular, T_ii = tau_i and
// T_ri = -tau_i sum_{r <= p < i} T_rp (V^T V)_pi.  Y <- Q^T Y takes the blocks in
// order, Y <- Y - V T^T (V^T Y); Y <- Q Y in reverse, Y <- Y - V T (V^T Y).
//
// One reflector at a time is a serial chain of n steps, each a reduction over
// the workgroup (water256: 10 ms a pass); a block of 16 is three products on the
// matrix cores and one reduction (1.07 ms a pass, and 0.26 ms for all T).
constexpr int kWy = 16;

// Column k0 + q of the reflectors at `row` (V is zero above row k0 + q + 1).
__device__ inline double v_mask(double x, int row, int q, int k0, int n)
{
    return (row > k0 + q && row < n && k0 + q < n - 2) ? x : 0.0;
}

// T of the block of reflectors k0 .. k0 + 15 of every group, one workgroup each,
// to twy (at the group's slab, block b at 256 b, T_rc at 16 r + c).
__global__ __launch_bounds__(256)
void wy_t_kernel(const GroupDesc *__restrict__ groups, int g0, const double *__restrict__ abase, EigVecs ev,
                 double *__restrict__ twy)
{
    __shared__ double gs[4][16][17];
    const GroupDesc gd = groups[g0 + blockIdx.y];
    const int n = gd.n, ld = gd.npad, k0 = blockIdx.x * kWy;
    if (k0 + 2 >= n) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int li = lane & 15, lq = lane >> 4;
    const double *vc = abase + gd.off + (int64_t)min(k0 + li, n - 1) * ld;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int r0 = (k0 & ~15) + 16 * wave; r0 < n; r0 += 64) {
        double v[4];
#pragma unroll
        for (int t = 0; t < 4; t++) v[t] = v_mask(vc[r0 + 4 * lq + t], r0 + 4 * lq + t, li, k0, n);
#pragma unroll
        for (int t = 0; t < 4; t++) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v[t], v[t], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; v++) gs[wave][lq + 4 * v][li] = acc[v];
    __syncthreads();
    {
        const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
        gs[0][r][c] = ((gs[0][r][c] + gs[1][r][c]) + gs[2][r][c]) + gs[3][r][c];
    }
    __syncthreads();
    if (threadIdx.x < 16) {
        const int r = threadIdx.x;
        const double *tau = ev.tau + gd.rinfo_off;
        double tr[16];
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const double ti = k0 + i < n - 2 ? tau[k0 + i] : 0.0;
            double s = 0.0;
#pragma unroll
            for (int p = 0; p < i; p++) s += (p >= r ? tr[p] : 0.0) * gs[0][p][i];
            tr[i] = i < r ? 0.0 : (i == r ? ti : -ti * s);
        }
        double *to = twy + gd.off + (int64_t)blockIdx.x * (kWy * kWy) + 16 * r;
#pragma unroll
        for (int i = 0; i < 16; i++) to[i] = tr[i];
    }
}

// One 512-lane workgroup per group and block of 16 columns keeps the columns in
// registers: wave w holds the 16-row tiles w, w + 8, ... (NT of them), lane
// (li, lq) = (l % 16, l / 16) rows 4 lq + t, t < 4, of column li.  That is the
// layout of a right operand of V^T Y (with the sum index permuted, k = 4 lq + t
// in both operands), and of the output of V (T V^T Y) when its row m stands for
// row 4 (m % 4) + m / 4 of the tile, so the block never changes its layout.
// NT = 0: any n, the columns stay in memory, where each lane reads and writes
// its own elements.
template <bool FORWARD, int NT>
__global__ __launch_bounds__(kReflBlock)
void reflect_kernel(const GroupDesc *__restrict__ groups, int g0, const double *__restrict__ abase,
                    const double *__restrict__ twy, double *__restrict__ y)
{
    constexpr int NWV = kReflBlock / 64;
    __shared__ double us[NWV][16][17];
    __shared__ double ts[16][17];
    const GroupDesc gd = groups[g0 + blockIdx.y];
    const int c0 = blockIdx.x * 16;
    if (c0 >= gd.m_own) return;
    const int n = gd.n, ld = gd.npad, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lq = lane >> 4;
    const int nt = (n + 15) / 16;                      // row tiles (n_pad is a multiple of 32)
    const double *A = abase + gd.off;
    const double *T = twy + gd.off;
    double *yc = y + gd.thin_off + (int64_t)min(c0 + li, gd.m_own - 1) * ld;
    const bool mine = c0 + li < gd.m_own;
    const int nq = NT > 0 ? NT : (nt + NWV - 1) / NWV;
    auto tile_in = [&](int q) {
        f64x4 f;
        const int r = 16 * (wave + NWV * q) + 4 * lq;
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const double v = yc[min(r + t, n - 1)];
            f[t] = (mine && r + t < n) ? v : 0.0;
        }
        return f;
    };
    auto tile_out = [&](int q, const f64x4 &f) {
        const int r = 16 * (wave + NWV * q) + 4 * lq;
#pragma unroll
        for (int t = 0; t < 4; t++)
            if (mine && r + t < ld) yc[r + t] = r + t < n ? f[t] : 0.0;
    };
    f64x4 yr[NT > 0 ? NT : 1];
    if constexpr (NT > 0) {
#pragma unroll
        for (int q = 0; q < NT; q++) yr[q] = tile_in(q);
    }
    const int nb = (n - 2 + kWy - 1) / kWy;
    for (int s = 0; s < nb; s++) {
        const int b = FORWARD ? s : nb - 1 - s, k0 = b * kWy;
        const int tb = k0 >> 4;                        // first tile with rows of the block
        if (tid < 256) ts[tid >> 4][tid & 15] = T[(int64_t)b * (kWy * kWy) + tid];
        // U = V^T Y over this wave's tiles
        f64x4 u = {0.0, 0.0, 0.0, 0.0};
        const double *vc = A + (int64_t)min(k0 + li, n - 1) * ld;
        auto dot_tile = [&](int q, const f64x4 &f) {
            const int tile = wave + NWV * q, r = 16 * tile + 4 * lq;
            if (tile >= nt || tile < tb) return;
            double v[4];
#pragma unroll
            for (int t = 0; t < 4; t++) v[t] = v_mask(vc[r + t], r + t, li, k0, n);
#pragma unroll
            for (int t = 0; t < 4; t++) u = __builtin_amdgcn_mfma_f64_16x16x4f64(v[t], f[t], u, 0, 0, 0);
        };
        if constexpr (NT > 0) {
#pragma unroll
            for (int q = 0; q < NT; q++) dot_tile(q, yr[q]);
        } else {
            for (int q = 0; q < nq; q++) dot_tile(q, tile_in(q));
        }
#pragma unroll
        for (int v = 0; v < 4; v++) us[wave][lq + 4 * v][li] = u[v];
        __syncthreads();
        // U summed over the waves in order, as the right operand of T U (T^T U)
        double ub[4], ta[4];
#pragma unroll
        for (int t = 0; t < 4; t++) {
            double a = 0.0;
#pragma unroll
            for (int w = 0; w < NWV; w++) a += us[w][4 * t + lq][li];
            ub[t] = a;
            ta[t] = FORWARD ? ts[4 * t + lq][li] : ts[li][4 * t + lq];
        }
        f64x4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < 4; t++) x = __builtin_amdgcn_mfma_f64_16x16x4f64(ta[t], ub[t], x, 0, 0, 0);
        // lane (li, lq) holds rows lq + 4 v of X: the right operand of V X with
        // the sum index k = lq + 4 t in sub-step t
        auto update_tile = [&](int q, f64x4 &f) {
            const int tile = wave + NWV * q, r = 16 * tile + 4 * (li & 3) + (li >> 2);
            if (tile >= nt || tile < tb) return;
            double v[4];
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const int qc = 4 * t + lq;
                v[t] = -v_mask(A[r + (int64_t)min(k0 + qc, n - 1) * ld], r, qc, k0, n);
            }
#pragma unroll
            for (int t = 0; t < 4; t++) f = __builtin_amdgcn_mfma_f64_16x16x4f64(v[t], x[t], f, 0, 0, 0);
        };
        if constexpr (NT > 0) {
#pragma unroll
            for (int q = 0; q < NT; q++) update_tile(q, yr[q]);
        } else {
            for (int q = 0; q < nq; q++) {
                f64x4 f = tile_in(q);
                update_tile(q, f);
                tile_out(q, f);
            }
        }
        __syncthreads();                               // us and ts are free again
    }
    // rows from n on as zero: in the last tiles here, in those beyond them below
    if constexpr (NT > 0) {
#pragma unroll
        for (int q = 0; q < NT; q++) tile_out(q, yr[q]);
    } else {
        for (int q = 0; q < nq; q++) tile_out(q, tile_in(q));
    }
    for (int r = 16 * nt + 4 * (tid >> 4); r < ld; r += 128)
        if (c0 + li < gd.m_own) {
#pragma unroll
            for (int t = 0; t < 4; t++) yc[r + t] = 0.0;
        }
}

// g(lambda) = 1 - 2 f(lambda): tanh(lambda / 2kT) for kT > 0; at T = 0 the
// signum, 0 for |lambda| <= tau0 (Eq. signevext).
__device__ inline double occ_sign(double x, double kT, double tau0)
{
    if (kT > 0.0) return tanh(x / (2.0 * kT));
    if (fabs(x) <= tau0) return 0.0;
    return x < 0.0 ? -1.0 : 1.0;
}

// Thin products with S on v_mfma_f64_16x16x4_f64:
//   MODE 0: C = S^T Y (rows l);
//   MODE 1: Z = S diag(g) C (rows i), g at lambda_l - dmu.
// Bound by HBM: S (n_g^2 values) is read once, and only m_own columns are
// formed.  A workgroup has 64 output rows (16 per wave) and up to 16 CB columns
// per pass; the thin operand is staged through LDS 64 rows at a time, S goes
// straight to registers, the next 64 in flight during the products.  S is read
// as it lies: 16 consecutive l of four rows k (MODE 0, k = 4 t + lane / 16 in
// sub-step t), or four consecutive l of 16 rows i (MODE 1, k = 4 (lane / 16) +
// t); the thin operand's rows follow the same order.  The grid is a multiple of
// 8 workgroups, which go round-robin over the XCDs: each XCD takes a contiguous
// run of (group, row block) items, so a group's row blocks share its L2 for the
// thin operand.  water256: 0.40 and 0.48 ms, against 7.6 and 8.1 ms on the
// vector units from LDS tiles of S.
template <int MODE, int CB>
__global__ __launch_bounds__(256)
void eig_thin_kernel(const GroupDesc *__restrict__ groups, int g0, EigVecs ev, const double *__restrict__ sbase,
                     const double *__restrict__ in, double *__restrict__ out, double dmu, double kT,
                     const unsigned long long *__restrict__ scale_bits, int gx, int nwork)
{
    constexpr int KC = 64;
    constexpr int ZU = KC * 16 * CB / 256;             // staged values per lane
    __shared__ double zs[KC][16 * CB + 1];
    const int item = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    if (item >= nwork) return;                         // padding of the grid to a multiple of 8
    const int g = g0 + item / gx;
    const GroupDesc gd = groups[g];
    const int ld = gd.npad, n = gd.n, r0 = (item % gx) * 64;
    if (r0 >= ld) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lq = lane >> 4;
    const double *S = sbase + gd.off;
    const double *lam = ev.lam + gd.rinfo_off;
    const double tau0 = 1e-14 * __longlong_as_double((long long)scale_bits[g]);
    const int row = min(r0 + 16 * wave + li, ld - 1);  // this lane's row of the left operand
    // rows k beyond n meet zeros of the thin operand (S is defined up to n_pad)
    auto load_s = [&](int k0, double (&s)[KC / 4]) {
#pragma unroll
        for (int h = 0; h < KC / 16; h++) {
            if (MODE == 0) {
#pragma unroll
                for (int t = 0; t < 4; t++)
                    s[4 * h + t] = S[(int64_t)min(k0 + 16 * h + 4 * t + lq, ld - 1) * ld + row];
            } else {
                const f64x4 v = *reinterpret_cast<const f64x4 *>(S + (int64_t)row * ld +
                                                                 min(k0 + 16 * h, ld - 16) + 4 * lq);
#pragma unroll
                for (int t = 0; t < 4; t++) s[4 * h + t] = v[t];
            }
        }
    };
    const int kk = tid & (KC - 1);
    const int nst = (n + KC - 1) / KC;
    for (int c0 = 0; c0 < gd.m_own; c0 += 16 * CB) {
        auto load_z = [&](int k0, double (&z)[ZU]) {
            const int k = min(k0 + kk, n - 1);
#pragma unroll
            for (int m = 0; m < ZU; m++)
                z[m] = in[gd.thin_off + k + (int64_t)min(c0 + tid / KC + 4 * m, gd.m_own - 1) * ld];
        };
        f64x4 acc[CB];
#pragma unroll
        for (int cb = 0; cb < CB; cb++) acc[cb] = f64x4{0.0, 0.0, 0.0, 0.0};
        double sa[KC / 4], sb[KC / 4], z[ZU];
        load_s(0, sa);
        load_z(0, z);
        auto stage = [&](int st, double (&cur)[KC / 4], double (&nxt)[KC / 4]) {
            const int k0 = st * KC;
            double gk = 1.0;
            if (MODE == 1) gk = occ_sign(lam[min(k0 + kk, n - 1)] - dmu, kT, tau0);
            __syncthreads();                           // every wave is done with the previous stage
#pragma unroll
            for (int m = 0; m < ZU; m++) {
                const int c = tid / KC + 4 * m;
                zs[kk][c] = (k0 + kk < n && c0 + c < gd.m_own) ? (MODE == 1 ? gk * z[m] : z[m]) : 0.0;
            }
            __syncthreads();
            const int kn = min(st + 1, nst - 1) * KC;
            load_s(kn, nxt);
            load_z(kn, z);
#pragma unroll
            for (int h = 0; h < KC / 16; h++)
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    const double *zr = zs[16 * h + (MODE == 0 ? 4 * t + lq : 4 * lq + t)];
#pragma unroll
                    for (int cb = 0; cb < CB; cb++)
                        acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[4 * h + t], zr[16 * cb + li], acc[cb], 0, 0, 0);
                }
        };
        for (int st = 0; st < nst; st += 2) {
            stage(st, sa, sb);
            if (st + 1 < nst) stage(st + 1, sb, sa);
        }
#pragma unroll
        for (int cb = 0; cb < CB; cb++) {
            const int c = c0 + 16 * cb + li;
            if (c >= gd.m_own) continue;
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int r = r0 + 16 * wave + lq + 4 * v;
                if (r < ld) out[gd.thin_off + r + (int64_t)c * ld] = r < n ? acc[cb][v] : 0.0;
            }
        }
        __syncthreads();                               // before the next columns' first stage
    }
}

// Algorithm 1's weights w_l = sum over the own columns of C_lc^2 (= sum_{c in
// own} Q_cl^2), in column order, and the unshifted eigenvalues lambda_l + mu0.
__global__ __launch_bounds__(256)
void weights_kernel(const GroupDesc *__restrict__ groups, int g0, EigVecs ev, const double *__restrict__ cbuf,
                    double mu0)
{
    const GroupDesc gd = groups[g0 + blockIdx.y];
    const int l = blockIdx.x * 256 + threadIdx.x;
    if (l >= gd.n) return;
    double w = 0.0;
    for (int c = 0; c < gd.m_own; c++) {
        const double v = cbuf[gd.thin_off + l + (int64_t)c * gd.npad];
        w += v * v;
    }
    ev.w[gd.rinfo_off + l] = w;
    ev.lam_abs[gd.rinfo_off + l] = ev.lam[gd.rinfo_off + l] + mu0;
}

// N(mu_m) = sum_g sum_l w_gl (1 - g(lambda_gl - mu_m)) / 2 for nmu trial values
// (Algorithm 1): part[q * nmu + m] over the eigenvalues of group g0 + q, one
// wave per (group, trial): lane l takes eigenvalues l, l + 64, ... in order, then
// a fixed tree.  One lane per (group, trial) is a chain of n tanh: 209 us for 32
// groups of n ~ 330 and 128 trials, 15 us this way.
__global__ __launch_bounds__(256)
void n_of_mu_kernel(const GroupDesc *__restrict__ groups, int g0, EigVecs ev, const double *__restrict__ mus, int nmu,
                    double kT, const unsigned long long *__restrict__ scale_bits, double *__restrict__ part)
{
    const int q = blockIdx.y, m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (m >= nmu) return;
    const GroupDesc gd = groups[g0 + q];
    const double mu = mus[m];
    const double tau0 = 1e-14 * __longlong_as_double((long long)scale_bits[g0 + q]);
    double s = 0.0;
    for (int l = lane; l < gd.n; l += 64)
        s += ev.w[gd.rinfo_off + l] * 0.5 * (1.0 - occ_sign(ev.lam_abs[gd.rinfo_off + l] - mu, kT, tau0));
    s = wave_sum0(s);
    if (lane == 0) part[(int64_t)q * nmu + m] = s;
}

// out[m] = sum over the groups of part[q * nmu + m], one wave per trial.
__global__ __launch_bounds__(64)
void n_reduce_kernel(int ng, int nmu, const double *__restrict__ part, double *__restrict__ out)
{
    const int m = blockIdx.x;
    double s = 0.0;
    for (int q = threadIdx.x; q < ng; q += 64) s += part[(int64_t)q * nmu + m];
    s = wave_sum0(s);
    if (threadIdx.x == 0) out[m] = s;
}

}  // namespace

hipError_t launch_eig_tridiag(hipStream_t st, const SideStream &side, int g0, int ngroups, int min_npad, int max_npad,
                              const GroupDesc *groups, double *a, double *wpanel, const EigVecs &ev)
{
    if (ngroups <= 0) return hipSuccess;
    const auto go = [&](auto kernel, hipStream_t on) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)ngroups), dim3(kEigBlock), 0, on, groups, g0, a, wpanel, ev);
        return hipGetLastError();
    };
    hipError_t e = hipSuccess;
    // A workgroup holds its CU to itself for its group's whole reduction.  Groups of
    // both kinds reduced one kind after the other leave the CUs of the second kind
    // idle during the first: 256 groups of n 583-1395 348 ms, in full and all at once
    // 316 ms, side by side on two streams 304 ms.  (Both bodies in one kernel lost
    // their loads in flight: 926 ms.)
    if (max_npad <= kEigHalfMaxN) {
        e = go(tridiag_kernel<true>, st);
    } else if (min_npad > kEigHalfMaxN) {
        e = go(tridiag_kernel<false>, st);
    } else {
        e = hipEventRecord(side.fork, st);
        if (e == hipSuccess) e = hipStreamWaitEvent(side.stream, side.fork, 0);
        if (e == hipSuccess) e = go(tridiag_kernel<false>, side.stream);
        if (e == hipSuccess) e = hipEventRecord(side.join, side.stream);
        if (e == hipSuccess) e = go(tridiag_kernel<true>, st);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, side.join, 0);
        if (e != hipSuccess) (void)hipStreamSynchronize(side.stream);   // nothing stays behind unjoined
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(split_kernel, dim3((unsigned)ngroups), dim3(256), 0, st, groups, g0, ev);
    return hipGetLastError();
}

hipError_t launch_eig_values_vectors(hipStream_t st, int g0, int ngroups, int max_npad, const GroupDesc *groups,
                                     const EigVecs &ev, double *s, double *scratch)
{
    if (ngroups <= 0) return hipSuccess;
    const dim3 grid((unsigned)((max_npad + 255) / 256), (unsigned)ngroups);
    hipLaunchKernelGGL(bisect_kernel, grid, dim3(256), 0, st, groups, g0, ev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (max_npad <= kHalfMaxN)
        hipLaunchKernelGGL(tvec_kernel<kHalfMaxN>, grid, dim3(256), 0, st, groups, g0, ev, s, scratch);
    else
        hipLaunchKernelGGL(tvec_kernel<kEigMaxN>, grid, dim3(256), 0, st, groups, g0, ev, s, scratch);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(cluster_kernel, grid, dim3(256), 0, st, groups, g0, ev, s, scratch);
    return hipGetLastError();
}

hipError_t launch_eig_own_select(hipStream_t st, int g0, int ngroups, int max_npad, int max_own,
                                 const GroupDesc *groups, const int32_t *own_list, double *y)
{
    if (ngroups <= 0) return hipSuccess;
    const int64_t tot = (int64_t)max_npad * max_own;
    const dim3 grid((unsigned)std::min<int64_t>((tot + 255) / 256, 1024), (unsigned)ngroups);
    hipLaunchKernelGGL(own_select_kernel, grid, dim3(256), 0, st, groups, own_list, g0, y);
    return hipGetLastError();
}

hipError_t launch_eig_wy(hipStream_t st, int g0, int ngroups, int max_npad, const GroupDesc *groups, const double *a,
                         const EigVecs &ev, double *twy)
{
    if (ngroups <= 0 || max_npad <= 2) return hipSuccess;
    const dim3 grid((unsigned)((max_npad + kWy - 1) / kWy), (unsigned)ngroups);
    hipLaunchKernelGGL(wy_t_kernel, grid, dim3(256), 0, st, groups, g0, a, ev, twy);
    return hipGetLastError();
}

hipError_t launch_eig_reflect(hipStream_t st, int forward, int g0, int ngroups, int max_npad, int max_own,
                              const GroupDesc *groups, const double *a, const double *twy, double *y)
{
    if (ngroups <= 0 || max_own <= 0) return hipSuccess;
    const dim3 grid((unsigned)((max_own + 15) / 16), (unsigned)ngroups);
    // tiles per wave held in registers: 8 are 1024 rows, 12 are 1536 (24 for all
    // kEigMaxN rows would spill most of them)
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(kReflBlock), 0, st, groups, g0, a, twy, y);
    };
    if (max_npad <= 1024) {
        if (forward) go(reflect_kernel<true, 8>);
        else go(reflect_kernel<false, 8>);
    } else if (max_npad <= 1536) {
        if (forward) go(reflect_kernel<true, 12>);
        else go(reflect_kernel<false, 12>);
    } else {
        if (forward) go(reflect_kernel<true, 0>);
        else go(reflect_kernel<false, 0>);
    }
    return hipGetLastError();
}

hipError_t launch_eig_thin(hipStream_t st, int mode, int g0, int ngroups, int max_npad, int max_own,
                           const GroupDesc *groups, const EigVecs &ev, const double *s, const double *in, double *out,
                           double mu0, double dmu, double kT, const unsigned long long *scale_bits)
{
    if (ngroups <= 0 || max_own <= 0) return hipSuccess;
    const int gx = (max_npad + 63) / 64, nwork = gx * ngroups;
    const dim3 grid((unsigned)((nwork + 7) / 8 * 8));
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, groups, g0, ev, s, in, out, dmu, kT, scale_bits, gx, nwork);
    };
    // one 16-column block per pass when every group owns at most 16 columns
    if (mode == 0 && max_own <= 16) go(eig_thin_kernel<0, 1>);
    else if (mode == 0) go(eig_thin_kernel<0, 2>);
    else if (max_own <= 16) go(eig_thin_kernel<1, 1>);
    else go(eig_thin_kernel<1, 2>);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || mode != 0) return e;
    hipLaunchKernelGGL(weights_kernel, dim3((unsigned)((max_npad + 255) / 256), (unsigned)ngroups), dim3(256), 0, st,
                       groups, g0, ev, out, mu0);
    return hipGetLastError();
}

hipError_t launch_n_of_mu(hipStream_t st, int ngroups, const GroupDesc *groups, const EigVecs &ev, const double *mus,
                          int nmu, double kT, const unsigned long long *scale_bits, double *part, double *out)
{
    if (ngroups <= 0 || nmu <= 0) return hipSuccess;
    // groups along the grid's second dimension, at most 65535 a launch
    for (int q0 = 0; q0 < ngroups; q0 += 65535) {
        hipLaunchKernelGGL(n_of_mu_kernel, dim3((unsigned)((nmu + 3) / 4), (unsigned)std::min(ngroups - q0, 65535)),
                           dim3(256), 0, st, groups, q0, ev, mus, nmu, kT, scale_bits, part + (int64_t)q0 * nmu);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(n_reduce_kernel, dim3((unsigned)nmu), dim3(64), 0, st, ngroups, nmu, part, out);
    return hipGetLastError();
}

}  // namespace smx
