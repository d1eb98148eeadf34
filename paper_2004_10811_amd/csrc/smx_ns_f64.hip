// FP64 Newton-Schulz products on the gfx950 matrix cores.
//
// One step of the second-order Newton-Schulz sign iteration (Sec. II-B),
// X_{k+1} = X_k (3I - X_k^2) / 2, is split into two batched products over
// all submatrices:
//   mode 0 ("square"): T = a^2 X_k X_k; the step-k residual max|T - I| over the
//                      true n_g x n_g part; W = 1.5 I - 0.5 T.
//   mode 1 ("update"): X_{k+1} = a X_k W, unless the step-k residual already
//                      meets the stopping rule (then X_k is the result).
// a = 1/s_g at k = 0 (Gershgorin prescaling folded into the first step), 1 after.
// The third-order Pade iteration X_{k+1} = X_k (15I - 10X_k^2 + 3X_k^4) / 8
// (Sec. VI-A) takes three products per step:
//   mode 5 ("Pade square"):  T = a^2 X_k X_k and its residual, as mode 0, T stored;
//   mode 6 ("Pade combine"): W = (15 I - 10 T + 3 T T) / 8 (T read at the output position);
//   mode 1 ("update") as above.
// The derivative of a Newton-Schulz step in a symmetric direction Xd takes two
// products of two operand pairs each, one pair's K range after the other's:
//   mode 3 ("square tangent"): Wd = -0.5 (X Xd + Xd X);
//   mode 4 ("update tangent"): Xd_{k+1} = Xd W + X Wd.
//
// Every iterate is a polynomial in the symmetric A_g, so X, T and W are
// symmetric and X W = W X.  Each workgroup therefore computes one
// lower-triangle tile and writes it twice (tile and mirror); both operands are
// read as columns (A(i, k) = X(k, i)), which keeps every global load
// contiguous along k.
//
// Workgroup: 256 threads = 4 waves in a 2 x 2 arrangement, each wave owns
// WB x WB blocks of v_mfma_f64_16x16x4_f64, so a tile has an edge of 32 WB.
// K is staged through LDS in steps of 16 with double buffering; the loads run
// two steps ahead in two register sets.  Inside a 16-step the k index handed to
// the matrix core is permuted (lane group q, sub-step t -> k = 4q + t) so each
// lane's four operand values are contiguous in LDS; the same permutation is
// applied to both operands, so the sum is unchanged.  The order of the sum does
// not depend on the tile edge: results are bitwise the same.
//
// What bounds it: the FP64 matrix pipe (one product occupies it for 64 cycles).
// Edge 64 puts four workgroups on a CU, whose waves fill each other's barrier
// and epilogue times, and its waves skip the padding and the upper half of the
// diagonal in 32 x 32 pieces.  water1024 (n_g 602-1055), square / update per
// launch: edge 128, two workgroups per CU and loads under a column condition
// (the compiler waited for them before the products) 11.7 / 10.9 ms; edge 96
// 10.9 / 10.4; edge 64 10.1 / 9.6 with loads one step ahead, 9.9 / 9.4 two
// steps ahead, the matrix pipe busy for 0.75 of them by the counters; edge 32 11.8 / 11.3
// (one block per wave: each operand value read from LDS feeds one product);
// edge 64 with K steps of 32 12.2 / 11.0 (two workgroups per CU).
#include "smx_internal.h"

namespace smx {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

constexpr int BK = 16;
constexpr int SK = BK + 2;     // LDS row stride in doubles (breaks bank aliasing)

__device__ inline double wave_max(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// QUARTERS (WB = 2): the list holds nlist 128 x 128 tiles, see TileList.
template <int MODE, int WB, bool QUARTERS>
__global__ __launch_bounds__(256, 4)
void ns_f64_kernel(const TileDesc *__restrict__ tiles, const GroupDesc *__restrict__ groups,
                   const double *__restrict__ xin, const double *__restrict__ bin,
                   double *__restrict__ out, IterState it, int k, double tol, int max_iter, int polish,
                   const double *__restrict__ x2, const double *__restrict__ b2, int nlist)
{
    static_assert(WB == 2 || !QUARTERS, "a quarter of a 128 x 128 tile has edge 64");
    constexpr int BM = 32 * WB;        // tile edge: 2 x 2 waves of WB x WB blocks of 16 x 16
    constexpr int WE = 16 * WB;        // edge of a wave's part of the tile
    __shared__ double As[2][BM][SK];
    __shared__ double Bs[2][BM][SK];

    if (MODE == 0 || MODE == 5) publish_step(it, k);
    if (WB == 1) {
        loaded(groups, it.done);
        loaded(it.resid_bits, it.scale_bits);
        loaded(xin, bin);
    }
    const TileDesc td = QUARTERS ? quarter_tile(tiles, nlist) : tiles[blockIdx.x];
    const int g = td.x;
    if (g < 0) return;                            // idle slot of the launch order
    // The group's state and extent in one wait, and the first operand loads before
    // the stopping test: each of these is a trip to memory that no cache holds
    // right after the previous launch, and small batches are short of other work.
    // An evaluation of 12 groups of n ~ 90 324 -> 317 us, 100 of ~ 503 unchanged (8.95 ms);
    // the larger tiles leave the order of the loads to the compiler (1024 groups of ~ 847
    // 364.3 ms with it forced, 362.5 without).
    const GroupDesc gd = groups[g];
    constexpr bool reads_x0 = MODE < 2 || MODE == 5;
    const int dn = MODE <= 2 || MODE >= 5 ? it.done[g] : 0;
    const unsigned long long sb = reads_x0 ? it.scale_bits[g] : 0;
    const unsigned long long rb = MODE == 1 ? it.resid_bits[(int64_t)g * it.resid_stride + k] : 0;
    if (WB == 1) {
        loaded(gd.off, gd.npad);
        loaded(gd.n, dn);
        loaded(sb, rb);
    }
    if (it.kact >= 0 && it.kfix && it.kact >= it.kfix[g]) return;   // group not in this adjoint step
    if (!polish && (MODE <= 2 || MODE >= 5) && dn) return;  // finished at an earlier step
    const int ti = td.y >> 16, tj = td.y & 0xffff;
    const int ld = gd.npad;
    if (QUARTERS && ti * BM >= ld) return;        // beyond the matrix

    // the prescaling enters the products that read X_0: squares and the update
    double a = 1.0;
    if (k == 0 && !polish && reads_x0) {
        const double s = __longlong_as_double((long long)sb);
        a = s > 0.0 ? 1.0 / s : 0.0;
    }
    if (MODE == 2 && dn) return;                  // tangent only while the group iterates

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wr = wave >> 1, wc = wave & 1;

    // global -> LDS staging: a K step is 16 k = 128 B per tile column, i.e. eight
    // 16-B chunks.  Chunk q*256 + tid (q < WB) is column 32 q + tid/8, part
    // tid%8: eight consecutive lanes read one full cache line.  Every lane
    // loads (columns beyond ld read column ld - 1, whose products reach only
    // outputs that are not stored): under a branch the compiler waits for the
    // loads where the paths join, before the products they should overlap.
    const int part = tid & 7;
    const int col8 = tid >> 3;
    const double *pa[WB], *pb[WB];
#pragma unroll
    for (int q = 0; q < WB; q++) {
        pa[q] = xin + gd.off + (int64_t)min(ti * BM + 32 * q + col8, ld - 1) * ld + part * 2;
        pb[q] = bin + gd.off + (int64_t)min(tj * BM + 32 * q + col8, ld - 1) * ld + part * 2;
    }

    // waves whose part of the tile lies wholly in the padding, or strictly
    // above the diagonal of a diagonal tile (never stored), skip the math
    const int row_w = ti * BM + wr * WE, col_w = tj * BM + wc * WE;
    const bool wave_live = (row_w < ld) && (col_w < ld) && !(ti == tj && wr < wc);

    d4 acc[WB][WB];
#pragma unroll
    for (int i = 0; i < WB; i++)
#pragma unroll
        for (int j = 0; j < WB; j++) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

    d2 r0[2 * WB], r1[2 * WB];         // two K steps in flight
    constexpr bool dual = MODE == 3 || MODE == 4;    // a second operand pair follows the first
    const int nk1 = ld / BK, nk = dual ? 2 * nk1 : nk1;
    auto gload = [&](int kt, d2 (&r)[2 * WB]) {
        kt = min(kt, nk - 1);
        int64_t ka = (int64_t)kt * BK, kb = ka;
        if (dual && kt >= nk1) {
            ka += (x2 - xin) - ld;
            kb += (b2 - bin) - ld;
        }
#pragma unroll
        for (int q = 0; q < WB; q++) {
            r[q] = *reinterpret_cast<const d2 *>(pa[q] + ka);
            r[WB + q] = *reinterpret_cast<const d2 *>(pb[q] + kb);
        }
    };
    auto sstore = [&](int buf, const d2 (&r)[2 * WB]) {
#pragma unroll
        for (int q = 0; q < WB; q++) {
            *reinterpret_cast<d2 *>(&As[buf][32 * q + col8][part * 2]) = r[q];
            *reinterpret_cast<d2 *>(&Bs[buf][32 * q + col8][part * 2]) = r[WB + q];
        }
    };
    const int li = lane & 15;
    const int lq = (lane >> 4) * 4;
    auto products = [&](int buf) {
        if (!wave_live) return;
        d4 av[WB], bv[WB];
#pragma unroll
        for (int i = 0; i < WB; i++) {
            const double *sa = &As[buf][wr * WE + i * 16 + li][lq];
            const double *sb = &Bs[buf][wc * WE + i * 16 + li][lq];
            const d2 a0 = *reinterpret_cast<const d2 *>(sa);
            const d2 a1 = *reinterpret_cast<const d2 *>(sa + 2);
            const d2 b0 = *reinterpret_cast<const d2 *>(sb);
            const d2 b1 = *reinterpret_cast<const d2 *>(sb + 2);
            av[i] = d4{a0.x, a0.y, a1.x, a1.y};
            bv[i] = d4{b0.x, b0.y, b1.x, b1.y};
        }
#pragma unroll
        for (int t = 0; t < 4; t++)
#pragma unroll
            for (int i = 0; i < WB; i++)
#pragma unroll
                for (int j = 0; j < WB; j++)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i][t], bv[j][t], acc[i][j], 0, 0, 0);
    };
    // step kt: the loads of step kt + 2 go out, the products of step kt run from
    // LDS, and step kt + 1 (loaded one step earlier) is stored for the next
    gload(0, r0);
    gload(1, r1);
    if (MODE == 1 && !polish) {
        const double rk = __longlong_as_double((long long)rb);
        const bool finite = rk <= 1.7976931348623157e308;
        const bool stop = it.kfix ? (k >= it.kfix[g]) : (rk <= tol || k >= max_iter);
        if (stop || !finite) {
            if (ti == 0 && tj == 0 && threadIdx.x == 0) {
                it.done[g] = 1;
                it.kfinal[g] = k;
                int fl = 0;
                if (!it.kfix && !(rk <= tol)) fl |= 1;
                if (!finite) fl |= 2;
                it.flags[g] = fl;
                atomicAdd(it.ndone, 1);
            }
            return;
        }
    }
    sstore(0, r0);
    __syncthreads();
    for (int kt = 0; kt < nk; kt += 2) {
        gload(kt + 2, r0);
        products(0);
        sstore(1, r1);
        __syncthreads();
        if (kt + 1 >= nk) break;
        gload(kt + 3, r1);
        products(1);
        sstore(0, r0);
        __syncthreads();
    }

    if (!wave_live) return;

    // Epilogue.  Block (i, j) of this wave, lane l, register v holds element
    // (row l/16 + 4 v, column l%16) of the 16 x 16 block (the f64 16x16x4
    // output layout; operands: lane l gives A[l%16][l/16] and B[l/16][l%16]).
    double *og = out + gd.off;
    const int n = gd.n;
    // The prescaling a = 1/s_g belongs to the true n_g x n_g block only: the
    // padded identity is a fixed point of the iteration and must stay exactly
    // I (a scaled padding entry 1/s_g would leave [-1, 1] when s_g < 1 and
    // grow without bound).  The padding never mixes with the true block, so
    // setting it after the product is exact.
    const bool pad_fix = (k == 0 && !polish && reads_x0);
    double rmax = 0.0;
#pragma unroll
    for (int i = 0; i < WB; i++) {
#pragma unroll
        for (int j = 0; j < WB; j++) {
            const int c = col_w + j * 16 + li;
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int r = row_w + i * 16 + (lane >> 4) + 4 * v;
                double val;
                if (MODE == 0 || MODE == 5) {
                    const double t = a * a * acc[i][j][v];
                    if (r < n && c < n) {
                        double d = fabs(t - (r == c ? 1.0 : 0.0));
                        if (!(d <= 1.7976931348623157e308)) d = __builtin_huge_val();
                        rmax = fmax(rmax, d);
                    }
                    val = MODE == 0 ? -0.5 * t + (r == c ? 1.5 : 0.0) : t;
                } else if (MODE == 6) {
                    // W = (15 I - 10 T + 3 T^2) / 8, T = x at this position
                    val = (r < ld && c < ld)
                              ? 0.125 * ((r == c ? 15.0 : 0.0) - 10.0 * xin[gd.off + r + (int64_t)c * ld] + 3.0 * acc[i][j][v])
                              : 0.0;
                } else if (MODE == 1) {
                    val = a * acc[i][j][v];
                } else if (MODE == 2) {
                    // tangent: 3 Xd W - 3 Xd (Xd and W commute, so the product is symmetric)
                    val = (r < ld && c < ld) ? 3.0 * acc[i][j][v] - 3.0 * xin[gd.off + r + (int64_t)c * ld] : 0.0;
                } else if (MODE == 3) {
                    val = -0.5 * acc[i][j][v];
                } else {
                    val = acc[i][j][v];
                }
                if (pad_fix && (r >= n || c >= n)) val = (r == c) ? 1.0 : 0.0;
                if (r < ld && c < ld && r >= c) {
                    og[r + (int64_t)c * ld] = val;
                    if (r > c) og[c + (int64_t)r * ld] = val;
                }
            }
        }
    }
    if (MODE == 0 || MODE == 5) {
        rmax = wave_max(rmax);
        if (lane == 0) {
            unsigned long long *slot = it.resid_bits + (int64_t)g * it.resid_stride + k;
            atomicMax(slot, (unsigned long long)__double_as_longlong(rmax));
        }
    }
}

}  // namespace

namespace {

template <int WB, bool QUARTERS>
hipError_t launch_wb(hipStream_t st, int mode, const TileList &tiles, const GroupDesc *groups,
                     const double *x, const double *b, double *out, const IterState &it, int k, double tol,
                     int max_iter, int polish, const double *x2, const double *b2)
{
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(tile_grid(tiles)), dim3(256), 0, st, tiles.tiles, groups, x, b, out, it, k, tol,
                           max_iter, polish, x2, b2, tiles.n);
        return hipGetLastError();
    };
    switch (mode) {
    case 0: return go(ns_f64_kernel<0, WB, QUARTERS>);
    case 1: return go(ns_f64_kernel<1, WB, QUARTERS>);
    case 5: return go(ns_f64_kernel<5, WB, QUARTERS>);
    case 6: return go(ns_f64_kernel<6, WB, QUARTERS>);
    }
    if constexpr (!QUARTERS) {          // tangents and the adjoint are never evaluated from the fixed array
        switch (mode) {
        case 2: return go(ns_f64_kernel<2, WB, false>);
        case 3: return go(ns_f64_kernel<3, WB, false>);
        case 4: return go(ns_f64_kernel<4, WB, false>);
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_ns_f64(hipStream_t st, int mode, int edge, const TileList &tiles, const GroupDesc *groups,
                         const double *x, const double *b, double *out, const IterState &it, int k, double tol,
                         int max_iter, int polish, const double *x2, const double *b2)
{
    if (tiles.n <= 0) return hipSuccess;
    if (edge == 64 && tiles.quarters)
        return launch_wb<2, true>(st, mode, tiles, groups, x, b, out, it, k, tol, max_iter, polish, x2, b2);
    if (edge == 64)
        return launch_wb<2, false>(st, mode, tiles, groups, x, b, out, it, k, tol, max_iter, polish, x2, b2);
    if (edge == 32 && !tiles.quarters)
        return launch_wb<1, false>(st, mode, tiles, groups, x, b, out, it, k, tol, max_iter, polish, x2, b2);
    return hipErrorInvalidValue;
}

}  // namespace smx
