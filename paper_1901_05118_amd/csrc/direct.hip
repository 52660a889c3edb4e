// DSOLVE of Algorithm 1 (the two coarsest levels) on gfx950: Cholesky A_h = L L^T of the
// banded operator, then L y = b and L^T x = y.
//
// In lexicographic order (x fastest) the farthest coupling of the scheme is two lines (2D)
// or two planes (3D) away, and the folded fictitious points stay inside that reach, so A_h
// and L have lower bandwidth w = 2 (N-1)^(dim-1).  Only band entries are stored and
// visited: every entry of L outside the band is an exact zero of the dense elimination, and
// dropping its products (signed zeros) leaves every stored value unchanged.  Each
// accumulation keeps the textbook order of the dense algorithm: entry (i, j) of the
// factor subtracts L(i,k) L(j,k) for k ascending, y_i subtracts L(i,k) y_k for k
// ascending, and x_i subtracts L(k,i) x_k for k ascending from i+1.
//
// Band storage (column-major band of the lower triangle): column c of the matrix occupies
// C[c (w+1) + d], d = 0..w, holding entry (c+d, c); slots past the last row stay zero.
#include "common.hpp"
#include "internal.hpp"

namespace excmg {

namespace {

// Scatter row r of A_h into the band: a term on a fictitious point folds onto the mirrored
// unknown with factor +1 (first kind) or -1 (second kind), a term on a boundary node is
// data.  Row r writes the entries (r, c) with c <= r, which nobody else writes.  Entries
// are small integers, exact in any order.  A coupling outside the band sets bad[0].
template <int DIM>
__global__ void __launch_bounds__(256) k_band_assemble(int N, int bc, int w, double *C, int *bad) {
    const int n = N - 1;
    const int nu = DIM == 3 ? n * n * n : n * n;
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nu) return;
    constexpr int NT = DIM == 3 ? 25 : 13;
    const int off3[25][3] = {{0, 0, 0},   {-1, 0, 0},  {1, 0, 0},   {0, -1, 0},  {0, 1, 0},
                             {0, 0, -1},  {0, 0, 1},   {-2, 0, 0},  {2, 0, 0},   {0, -2, 0},
                             {0, 2, 0},   {0, 0, -2},  {0, 0, 2},   {-1, -1, 0}, {-1, 1, 0},
                             {1, -1, 0},  {1, 1, 0},   {-1, 0, -1}, {1, 0, -1},  {0, -1, -1},
                             {0, 1, -1},  {-1, 0, 1},  {1, 0, 1},   {0, -1, 1},  {0, 1, 1}};
    const int off2[13][2] = {{0, 0},  {-1, 0}, {1, 0},   {0, -1},  {0, 1},  {-2, 0}, {2, 0},
                             {0, -2}, {0, 2},  {-1, -1}, {-1, 1}, {1, -1}, {1, 1}};
    int q[3] = {r % n + 1, (r / n) % n + 1, DIM == 3 ? r / (n * n) + 1 : 1};
    const double sgn = (bc == 1) ? 1.0 : -1.0;
    const i64 ld = (i64)w + 1;
    for (int t = 0; t < NT; t++) {
        double coef;
        int p[3];
        if (DIM == 3) {
            coef = (t == 0) ? 42.0 : (t <= 6) ? -12.0 : (t <= 12) ? 1.0 : 2.0;
            for (int a = 0; a < 3; a++) p[a] = q[a] + off3[t][a];
        } else {
            coef = (t == 0) ? 20.0 : (t <= 4) ? -8.0 : (t <= 8) ? 1.0 : 2.0;
            p[0] = q[0] + off2[t][0];
            p[1] = q[1] + off2[t][1];
            p[2] = 1;
        }
        bool bnd = false, ghost = false;
        for (int a = 0; a < DIM; a++) {
            if (p[a] == 0 || p[a] == N) bnd = true;
            if (p[a] == -1) { p[a] = 1; ghost = true; }
            if (p[a] == N + 1) { p[a] = N - 1; ghost = true; }
        }
        if (bnd) continue;
        const int c = ((p[2] - 1) * n + (p[1] - 1)) * n + (p[0] - 1);
        if (c > r) continue;
        if (r - c > w) {
            bad[0] = 1;
            continue;
        }
        C[(i64)c * ld + (r - c)] += ghost ? sgn * coef : coef;
    }
}

// Right-looking Cholesky of the band in one workgroup.  Step k takes the pivot (already
// reduced by steps 0..k-1), scales column k, and subtracts L(i,k) L(j,k) from every band
// entry (i, j) of the trailing window; each entry thus receives its subtractions in the
// order k = 0, 1, ... of the dense left-looking form.  info = k+1 for a pivot that is not
// positive.
__global__ void __launch_bounds__(1024) k_band_cholesky(int n, int w, double *C, int *info) {
    __shared__ double piv;
    __shared__ int fail;
    const int tid = threadIdx.x;
    const i64 ld = (i64)w + 1;
    if (tid == 0) fail = 0;
    for (int k = 0; k < n; k++) {
        double *col = C + (i64)k * ld;
        const int m = min(w, n - 1 - k);
        if (tid == 0) {
            const double s = col[0];
            if (!(s > 0.0)) fail = k + 1;
            const double d = sqrt(s);
            col[0] = d;
            piv = d;
        }
        __syncthreads();
        if (fail) break;
        const double d = piv;
        for (int e = 1 + tid; e <= m; e += blockDim.x) col[e] = col[e] / d;
        __syncthreads();
        for (int e = tid; e < m * m; e += blockDim.x) {
            const int a = e / m, b = e - a * m;  // column k+1+a, row k+1+b
            if (b < a) continue;
            C[(i64)(k + 1 + a) * ld + (b - a)] -= col[1 + b] * col[1 + a];
        }
        __syncthreads();
    }
    if (tid == 0) *info = fail;
}

constexpr int kBandMaxN = 4096;

// a / d from y = 1/d (correctly rounded; 0: not usable) by two corrections of a y: the second
// starts from a quotient within one unit of the last place, with an exact remainder, so it
// gives the correctly rounded one (P. Markstein, IBM J. Res. Dev. 34, 1990).  Five dependent
// operations instead of the dozen of a general division.  Quotients that come near the ends
// of the exponent range, zeros, infinities and NaN take the general one.  a is the same in
// all lanes.
__device__ __forceinline__ double quotient(double a, double d, double y) {
    double q = a * y;
    q = fma(fma(-q, d, a), y, q);
    q = fma(fma(-q, d, a), y, q);
    const int e = (__builtin_amdgcn_readfirstlane(__double2hiint(a)) >> 20) & 2047;
    const int outside = (int)((unsigned)(e - 256) >= 1536u) |
                        (int)(__builtin_amdgcn_readfirstlane(__double2hiint(y)) == 0);
    if (__builtin_expect(outside, 0)) q = a / d;
    return q;
}
__device__ __forceinline__ double reciprocal(double d) {
    return d >= 0x1p-100 && d <= 0x1p100 ? 1.0 / d : 0.0;
}
__device__ __forceinline__ double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// Orders LDS accesses of one wavefront (which the LDS takes in program order).
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// L y = b, then L^T x = y, in one wavefront (b and x may alias).
//
// What bounds it: a serial chain.  Forward, y_k = t_k / L(k,k) must be there before y_k+1 can
// be formed; backward, row i subtracts its w products in ascending k starting with the one
// that needs x_{i+1}, so the whole solve is n w dependent subtractions.
//
// Forward: the rows of a block of 64 and those its columns reach are in registers, row
// 64 (block + q) + lane in slot q; a step broadcasts its pivot row's value by a lane read.
// Backward: the chain runs in every lane alike on products read from LDS, 16 ahead.  The
// products of the next row (all but the first, which needs x_i) are formed by the lanes
// meanwhile; what lies past a column's last row is +0, which changes no difference.  The
// diagonal's reciprocals are formed for 64 rows at once.  The columns come in chunks of DP:
// while the steps of one run, the next one's loads are in flight.
// Per row at w = 126 (64^2): forward 460 cycles (readlane, quotient, update), backward 1550, 9
// a subtraction: reading a product pair costs the wave about as much as its two additions
// (5.3 each).  Against a step with LDS round trips forward, and products formed and waited
// for before each row's chain by one lane: 64^2 6.8 -> 3.3 ms, 32^2 1.02 -> 0.55, 16^3
// 15.7 -> 8.4, 8^3 0.45 -> 0.30.
template <int PER, int NG, int DP>
__global__ void __launch_bounds__(64) k_band_solve(int n, int w, const double *C, const double *b,
                                                   double *x) {
    constexpr int S = PER + 1;          // slots of 64 rows that a block's columns reach
    constexpr int PROD = 64 * PER + 32;  // >= 16 NG
    static_assert(NG % 2 == 0 && PER == (NG + 3) / 4);
    __shared__ double t[kBandMaxN];
    __shared__ __align__(16) double prod[2][PROD];
    const int lane = threadIdx.x;
    const i64 ld = (i64)w + 1;
    for (int i = lane; i < 2 * PROD; i += 64) prod[0][i] = 0.0;

    // forward
    {
        double v[S], cur[DP][S], nxt[DP][S];
        auto load_rows = [&](int row) { return row < n ? b[row] : 0.0; };
        auto load_col = [&](int k, double (&c)[S]) {
            const double *col = C + (i64)min(k, n - 1) * ld;
#pragma unroll
            for (int q = 0; q < S; q++) c[q] = col[(unsigned)min(max(64 * q + lane - (k & 63), 0), w)];
        };
#pragma unroll
        for (int q = 0; q < S; q++) v[q] = load_rows(64 * q + lane);
        double diag = C[(i64)min(lane, n - 1) * ld];
#pragma unroll
        for (int s = 0; s < DP; s++) load_col(s, cur[s]);
        for (int k0 = 0; k0 < n; k0 += 64) {
            const double inv = reciprocal(diag);
            const double next_diag = C[(i64)min(k0 + 64 + lane, n - 1) * ld];
            const double next_rows = load_rows(k0 + 64 * S + lane);
#pragma unroll 1
            for (int s0 = 0; s0 < min(64, n - k0); s0 += DP) {
                // unconditional (clamped) requests, so the loads in flight are counted exactly
#pragma unroll
                for (int s = 0; s < DP; s++) load_col(k0 + s0 + DP + s, nxt[s]);
#pragma unroll
                for (int s = 0; s < DP; s++) {
                    const int l = s0 + s;
                    __builtin_amdgcn_sched_barrier(0);
                    const double yk = quotient(lane_value(v[0], l), lane_value(diag, l),
                                               lane_value(inv, l));
#pragma unroll
                    for (int q = 0; q < S; q++) {
                        const int e = 64 * q + lane - l;
                        const double u = v[q] - cur[s][q] * yk;
                        if (q == 0) v[q] = e >= 1 && e <= w ? u : (e == 0 ? yk : v[q]);
                        else v[q] = e <= w ? u : v[q];
                    }
                }
#pragma unroll
                for (int s = 0; s < DP; s++)
#pragma unroll
                    for (int q = 0; q < S; q++) cur[s][q] = nxt[s][q];
            }
            t[k0 + lane] = k0 + lane < n ? v[0] : 0.0;
#pragma unroll
            for (int q = 0; q + 1 < S; q++) v[q] = v[q + 1];
            v[S - 1] = next_rows;
            diag = next_diag;
        }
        wave_order();
    }

    // backward
    {
        double cur[DP][PER], nxt[DP][PER];
        const int k1 = (n - 1) & ~63;
        auto load_col = [&](int k, double (&c)[PER]) {
            const double *col = C + (i64)min(max(k, 0), n - 1) * ld;
#pragma unroll
            for (int q = 0; q < PER; q++) c[q] = col[(unsigned)min(lane + 64 * q, w)];
        };
        // the rows past the last one of its chunk are zeros (t holds zeros there)
        int s0 = (63 - (n - 1 - k1)) / DP * DP;
        double xi = 0.0, ti = t[k1 + 63 - s0];
        double first[16], second[16];     // products: of the row at hand, 16 ahead of the chain
#pragma unroll
        for (int e = 0; e < 16; e++) first[e] = 0.0;
        double diag = C[(i64)min(k1 + lane, n - 1) * ld];
#pragma unroll
        for (int s = 0; s < DP; s++) load_col(k1 + 63 - s0 - s, cur[s]);
        for (int k0 = k1; k0 >= 0; k0 -= 64) {
            const double inv = reciprocal(diag);
            const double next_diag = C[(i64)max(k0 - 64 + lane, 0) * ld];
#pragma unroll 1
            for (; s0 < 64; s0 += DP) {
#pragma unroll
                for (int s = 0; s < DP; s++) load_col(k0 + 63 - (s0 + DP + s), nxt[s]);
#pragma unroll
                for (int s = 0; s < DP; s++) {
                    const int l = 63 - (s0 + s), i = k0 + l;
                    __builtin_amdgcn_sched_barrier(0);
                    const double *P = prod[i & 1];
                    double *Q = prod[(i & 1) ^ 1];
                    double tv[PER];
#pragma unroll
                    for (int q = 0; q < PER; q++) tv[q] = t[min(max(i - 1 + lane + 64 * q, 0), n - 1)];
                    const double t_next = t[max(i - 1, 0)];
#pragma unroll
                    for (int e = 0; e < 16; e++) second[e] = P[16 + e];
                    __builtin_amdgcn_sched_barrier(0);
                    double acc = ti - lane_value(cur[s][0], 1) * xi;
#pragma unroll
                    for (int e = 0; e < 16; e++) acc -= first[e];
                    // the next row's products from its third entry on
                    const int m = min(w, n - i);
#pragma unroll
                    for (int q = 0; q < PER; q++) {
                        const int e = lane + 64 * q;
                        const double c = s + 1 < DP ? cur[s + 1 < DP ? s + 1 : 0][q] : nxt[0][q];
                        if (e >= 2) Q[e - 2] = e <= m ? c * tv[q] : 0.0;
                    }
                    wave_order();
#pragma unroll
                    for (int g = 1; g < NG; g++) {
                        double (&now)[16] = (g & 1) ? second : first;
                        double (&then)[16] = (g & 1) ? first : second;
                        const double *F = g + 1 < NG ? P + 16 * (g + 1) : Q;
#pragma unroll
                        for (int e = 0; e < 16; e++) then[e] = F[e];
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int e = 0; e < 16; e++) acc -= now[e];
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    xi = quotient(acc, lane_value(diag, l), lane_value(inv, l));
                    t[i] = xi;
                    ti = t_next;
                    wave_order();
                }
#pragma unroll
                for (int s = 0; s < DP; s++)
#pragma unroll
                    for (int q = 0; q < PER; q++) cur[s][q] = nxt[s][q];
            }
            s0 = 0;
            diag = next_diag;
        }
    }
    for (int i = lane; i < n; i += 64) x[i] = t[i];
}

}  // namespace

int band_width(int N, int dim) { return dim == 2 ? 2 * (N - 1) : 2 * (N - 1) * (N - 1); }

hipError_t band_assemble(int N, int bc, int dim, int w, double *C, int *bad, hipStream_t st) {
    const int n = N - 1;
    const int nu = dim == 3 ? n * n * n : n * n;
    hipError_t e = hipMemsetAsync(C, 0, (size_t)nu * (w + 1) * sizeof(double), st);
    if (e != hipSuccess) return e;
    if (dim == 3)
        hipLaunchKernelGGL(k_band_assemble<3>, dim3((nu + 255) / 256), dim3(256), 0, st, N, bc, w,
                           C, bad);
    else
        hipLaunchKernelGGL(k_band_assemble<2>, dim3((nu + 255) / 256), dim3(256), 0, st, N, bc, w,
                           C, bad);
    return hipGetLastError();
}

hipError_t band_cholesky(int n, int w, double *C, int *info, hipStream_t st) {
    hipLaunchKernelGGL(k_band_cholesky, dim3(1), dim3(1024), 0, st, n, w, C, info);
    return hipGetLastError();
}

hipError_t band_solve(int n, int w, const double *C, const double *b, double *x, hipStream_t st) {
    if (n < 1 || n > kBandMaxN || w < 0 || w + 1 > 64 * 8) return hipErrorInvalidValue;
    // 16 NG >= w-1 products of a row and 64 PER >= w+1 entries of a column, PER = ceil(NG / 4)
#define EXCMG_SOLVE(NG, DP)                                                                     \
    if (w - 1 <= 16 * NG && w + 1 <= (NG + 3) / 4 * 64) {                                       \
        hipLaunchKernelGGL((k_band_solve<(NG + 3) / 4, NG, DP>), dim3(1), dim3(64), 0, st, n, w, C, b, x); \
        return hipGetLastError();                                                               \
    }
    // up to 32 unknowns most of a solve is fetching its code, which chunks of one column keep
    // short (whole calls, chunks of 8 / of 1: 1 unknown 17.9 / 14.0 us, 9 21.3 / 18.0, 25
    // 28.6 / 26.2; from 36 on no different)
    if (n <= 32) {
        EXCMG_SOLVE(2, 1)
    }
    EXCMG_SOLVE(2, 8)
    EXCMG_SOLVE(4, 8)
    EXCMG_SOLVE(6, 8)
    EXCMG_SOLVE(8, 8)
    EXCMG_SOLVE(12, 4)
    EXCMG_SOLVE(16, 4)
    EXCMG_SOLVE(20, 4)
    EXCMG_SOLVE(24, 4)
    EXCMG_SOLVE(28, 4)
    EXCMG_SOLVE(32, 4)
#undef EXCMG_SOLVE
    return hipErrorInvalidValue;
}

}  // namespace excmg
