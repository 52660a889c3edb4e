// The 3D grid transfers of the cascade on gfx950: EXP_finite (Sec. 4.2.3) and EXP_true
// (Sec. 4.2.1).
//
// Both are bound by HBM: EXP_true reads the fine solution and the coarse one (1/8 of its
// size) and writes a fine array; EXP_finite writes its fine array from inputs of 1/8 and 1/64
// of its size.  A workgroup owns a tile of fine nodes (128 x 4 for the midpoints, 64 x 16 for the
// interpolation) and marches in z, so a node's
// place is found once, a plane's coarse values are staged once in LDS (with the coarse nodes
// on the tile's far sides), and every fine value is read and written once, in rows.  One
// barrier per step: the staged planes are a ring long enough that a step's writes miss what
// the step before still reads, and the next step's loads are in flight meanwhile.  Measured,
// whole calls, against one thread per node with its neighbours from global memory: EXP_true
// at 512^3 1361 -> 512 us (4.5 TB/s of the bytes it must move), at 256^3 189 -> 92 us;
// EXP_finite at 256^3 381 -> 64 us on one set of arrays, 82 on new ones (of the 381, its two
// kernels took 300, an allocation and a free of the intermediate grid the rest), at 128^3 100 ->
// 27 us, at 512^3 2862 -> 890.
//
// Every formula is evaluated in the order it is written in (contraction off).
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"

namespace excmg {

namespace {

// A tile of fine nodes and the coarse (every second) nodes in it and on its far sides.
template <int TX, int TY>
struct Tile {
    static constexpr int kX = TX, kY = TY, kThreads = TX * TY;
    static constexpr int kCoarseX = TX / 2 + 1, kCoarse = kCoarseX * (TY / 2 + 1);
};
// EXP_true at 512^3: 64 x 8 605 us, 128 x 4 512 us (long rows: fewer lines split between
// tiles), 256 x 2 568 us.  The interpolation (EXP_finite at 256^3 as a whole): one node per
// thread, 64 x 8, 89 us: lanes on Z1 planes of x waited for those between, and 184 registers
// left one workgroup per CU; two nodes per thread, one plane of Z1 at a time, 71 us with 166
// registers, 66 with 128.
using MidTile = Tile<128, 4>;
using CellTile = Tile<64, 16>;
constexpr int kCellThreads = CellTile::kThreads / 2;    // two nodes each
constexpr int kCellWaves = 4;                           // per SIMD: 128 registers

// Midpoint extrapolation of the grid of N cells (even) from the fine solution H on it and the
// coarse one C on every second node.  Nodes of the coarse grid: eq. (t1) (TRUE: (4 H - C) / 3)
// or eq. (secfff) (else: (5 H - C) / 4); midpoints of coarse edges: the fine value plus 1/6
// (eq. chenlin) or 1/8 (eq. bfsec) of the sum of H - C over the edge's two ends; centres of
// coarse faces and cells: the mean of that formula over the two face diagonals or the four
// space diagonals.
template <bool TRUE>
__global__ void __launch_bounds__(MidTile::kThreads)
    k_midpoints(int N, int planes, const double *H, const double *C, double *out) {
    constexpr int kTileX = MidTile::kX, kTileY = MidTile::kY, kCoarseX = MidTile::kCoarseX,
                  kCoarse = MidTile::kCoarse;
    __shared__ double sh[3][kCoarse], sc[3][kCoarse];
    const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * kTileX + tx;
    const int i = blockIdx.x * kTileX + tx, j = blockIdx.y * kTileY + ty;
    const int NC = N / 2, K0 = blockIdx.z * planes, K1 = min(K0 + planes, NC + 1);
    const i64 M = (i64)N + 1, MC = (i64)NC + 1;
    const bool valid = i <= N && j <= N;
    // lanes beyond the grid request its last nodes
    const double *mid = H + (i64)min(j, N) * M + min(i, N);
    const i64 plane = M * M;
    const int I = min((int)blockIdx.x * (kTileX / 2) + tid % kCoarseX, NC),
              J = min((int)blockIdx.y * (kTileY / 2) + tid / kCoarseX, NC);
    const bool stages = tid < kCoarse;
    const double *hc = H + (i64)(2 * J) * M + 2 * I, *cc = C + (i64)J * MC + I;
    // ends of this node's edge or diagonals: A = (-, -), B = (+, -), E = (-, +), F = (+, +)
    const int oi = tx & 1, oj = ty & 1;
    const int a = (ty >> 1) * kCoarseX + (tx >> 1);
    const int b = a + oi, e = a + oj * kCoarseX, f = e + oi;
    constexpr double s = TRUE ? 1.0 / 6.0 : 1.0 / 8.0;

    double h0 = 0.0, c0 = 0.0;
    if (stages) {
        sh[K0 % 3][tid] = hc[2 * K0 * plane];
        sc[K0 % 3][tid] = cc[K0 * MC * MC];
        h0 = hc[2 * min(K0 + 1, NC) * plane];
        c0 = cc[min(K0 + 1, NC) * MC * MC];
    }
    double m0 = mid[2 * K0 * plane], m1 = mid[min(2 * K0 + 1, N) * plane];
    for (int K = K0; K < K1; K++) {
        const int p = K % 3, q = (K + 1) % 3;
        if (stages) {
            sh[q][tid] = h0;
            sc[q][tid] = c0;
        }
        __syncthreads();
        const double v0 = m0, v1 = m1;
        if (stages) {
            h0 = hc[2 * min(K + 2, NC) * plane];
            c0 = cc[min(K + 2, NC) * MC * MC];
        }
        m0 = mid[min(2 * K + 2, N) * plane];
        m1 = mid[min(2 * K + 3, N) * plane];
        // from the end `u` of plane K to the end `w` of plane K + up
        auto along = [&](double v, int u, int w, int up) {
            const int t = up ? q : p;
            return v + s * (sh[p][u] - sc[p][u] + sh[t][w] - sc[t][w]);
        };
        double even, odd;
        if (oj == 0) {
            if (oi == 0) {
                even = TRUE ? (4.0 * v0 - sc[p][a]) / 3.0 : (5.0 * v0 - sc[p][a]) / 4.0;
                odd = along(v1, a, a, 1);
            } else {
                even = along(v0, a, b, 0);
                odd = (along(v1, a, b, 1) + along(v1, b, a, 1)) / 2.0;
            }
        } else {
            if (oi == 0) {
                even = along(v0, a, e, 0);
                odd = (along(v1, a, e, 1) + along(v1, e, a, 1)) / 2.0;
            } else {
                even = (along(v0, a, f, 0) + along(v0, b, e, 0)) / 2.0;
                odd = (along(v1, a, f, 1) + along(v1, b, e, 1) + along(v1, e, b, 1) +
                       along(v1, f, a, 1)) / 4.0;
            }
        }
        if (valid) {
            double *o = out + (i64)(2 * K) * plane + (i64)j * M + i;
            o[0] = even;
            if (2 * K + 1 <= N) o[plane] = odd;
        }
    }
}

// Quadratic Lagrange weights at the positions xi = 1/4 and 3/4 of an interpolation cell,
// eqs. (inter)-(iinter); positions 0, 2/4 and 1 are nodes.
__device__ __forceinline__ double lagrange(int pos, int node) {
    const double w = node == 1 ? 0.75 : ((pos == 1) == (node == 0) ? 0.375 : -0.125);
    return w;
}

// Step 5: the grid of N cells from Z1 (N/2 cells): tri-quadratic interpolation in cells of four
// fine cells.  A node at an odd position of an axis takes the cell's three Z1 planes of that
// axis, at an even one the plane it lies on; terms are summed in the node order of the cell
// (z slowest, x fastest).  (The weights are multiples of 1/512, so their products are exact.)
// A thread takes the nodes 2t (on a Z1 plane of x) and 2t+1 (between) of a row, whose Z1 nodes
// it reads once, for the four fine planes of a cell.
template <int NY>
__device__ __forceinline__ void interpolate(const double *const (&P)[3], int at, int second, int py,
                                            double (&even)[4], double (&odd)[4]) {
    const int px = second ? 3 : 1;
    double wxy[NY][3], wy[NY];
#pragma unroll
    for (int y = 0; y < NY; y++) {
        wy[y] = NY == 1 ? 1.0 : lagrange(py, y);
#pragma unroll
        for (int x = 0; x < 3; x++) wxy[y][x] = lagrange(px, x) * wy[y];
    }
#pragma unroll
    for (int c = 0; c < 4; c++) even[c] = odd[c] = 0.0;
#pragma unroll
    for (int z = 0; z < 3; z++) {
        double v[NY][3], ve[NY];
#pragma unroll
        for (int y = 0; y < NY; y++) {
#pragma unroll
            for (int x = 0; x < 3; x++) v[y][x] = P[z][at + y * CellTile::kCoarseX + x];
            ve[y] = second ? v[y][1] : v[y][0];
        }
#pragma unroll
        for (int c = 0; c < 4; c++) {
            if ((c & 1) == 0 && z != c / 2) continue;
            const double wz = (c & 1) == 0 ? 1.0 : lagrange(c, z);
#pragma unroll
            for (int y = 0; y < NY; y++) {
                even[c] = NY == 1 && (c & 1) == 0 ? ve[y] : even[c] + (wy[y] * wz) * ve[y];
#pragma unroll
                for (int x = 0; x < 3; x++) odd[c] = odd[c] + (wxy[y][x] * wz) * v[y][x];
            }
        }
    }
}

__global__ void __launch_bounds__(kCellThreads, kCellWaves)
    k_interpolate(int N, int cells, const double *V, double *out) {
    constexpr int kTileX = CellTile::kX, kTileY = CellTile::kY, kCoarseX = CellTile::kCoarseX,
                  kCoarse = CellTile::kCoarse;
    __shared__ double sv[5][kCoarse];
    // a wave takes two rows of 32 pairs whose positions in y are both on or both between Z1's
    const int tid = threadIdx.x, wave = tid >> 6, t = tid & 31;
    const int ty = 4 * (wave >> 1) + (wave & 1) + 2 * ((tid >> 5) & 1);
    const int i = blockIdx.x * kTileX + 2 * t, j = blockIdx.y * kTileY + ty;
    const int N1 = N / 2, N0 = N / 4;
    const int c0 = blockIdx.z * cells, c1 = min(c0 + cells, N0);
    const i64 M = (i64)N + 1, M1 = (i64)N1 + 1, plane1 = M1 * M1;
    const bool valid = i <= N && j <= N, pair = valid && i < N;
    // staging: two planes of Z1 a step, in turns
    constexpr int kLoads = (2 * kCoarse + kCellThreads - 1) / kCellThreads;
    auto source = [&](int k, int plane) {
        const int e = tid + k * kCellThreads, half = e >= kCoarse ? 1 : 0, node = e - half * kCoarse;
        const int I = min((int)blockIdx.x * (kTileX / 2) + node % kCoarseX, N1),
                  J = min((int)blockIdx.y * (kTileY / 2) + node / kCoarseX, N1);
        return e < 2 * kCoarse ? V[min(plane + half, N1) * plane1 + (i64)J * M1 + I] : 0.0;
    };
    // the cell's first Z1 node in the tile, and the row's position in it
    const int second = t & 1, py = ty & 3;
    const int at = 2 * (t >> 1) + ((py & 1) ? 2 * (ty >> 2) : ty >> 1) * kCoarseX;

    for (int e = tid; e < kCoarse; e += kCellThreads) {
        const int I = min((int)blockIdx.x * (kTileX / 2) + e % kCoarseX, N1),
                  J = min((int)blockIdx.y * (kTileY / 2) + e / kCoarseX, N1);
        sv[(2 * c0) % 5][e] = V[2 * c0 * plane1 + (i64)J * M1 + I];
    }
    double next[kLoads];
#pragma unroll
    for (int k = 0; k < kLoads; k++) next[k] = source(k, 2 * c0 + 1);
    for (int c = c0; c < c1; c++) {
#pragma unroll
        for (int k = 0; k < kLoads; k++) {
            const int e = tid + k * kCellThreads, half = e >= kCoarse ? 1 : 0;
            if (e < 2 * kCoarse) sv[(2 * c + 1 + half) % 5][e - half * kCoarse] = next[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kLoads; k++) next[k] = source(k, 2 * c + 3);
        const double *const P[3] = {sv[(2 * c) % 5], sv[(2 * c + 1) % 5], sv[(2 * c + 2) % 5]};
        double even[4], odd[4];
        if (py & 1) interpolate<3>(P, at, second, py, even, odd);
        else interpolate<1>(P, at, second, py, even, odd);
        double *w = out + ((i64)(4 * c) * M + j) * M + i;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            if (valid) w[k * M * M] = even[k];
            if (pair) w[k * M * M + 1] = odd[k];
        }
    }
    if (c1 == N0) {       // the last plane of nodes
        const double *const P[3] = {sv[(2 * N0) % 5], sv[(2 * N0) % 5], sv[(2 * N0) % 5]};
        double even[4], odd[4];
        if (py & 1) interpolate<3>(P, at, second, py, even, odd);
        else interpolate<1>(P, at, second, py, even, odd);
        double *w = out + ((i64)N * M + j) * M + i;
        if (valid) w[0] = even[0];
        if (pair) w[1] = odd[0];
    }
}

// Steps per workgroup: long marches stage fewer shared planes, `groups` workgroups or more
// hide the loads (EXP_true at 512^3: 2048 groups 573 us, 4096 550, 16384 512; EXP_finite at
// 256^3 / 384^3: 512 groups 64 / 280 us, 1024 66 / 252, 2048 69 / 238).
int march_steps(int tiles, int steps, int groups) {
    const int want = std::max(1, groups / tiles);
    return std::max(std::min(steps, 2), (steps + want - 1) / want);
}

template <bool TRUE>
hipError_t midpoints(int N, const double *H, const double *C, double *out, hipStream_t st) {
    const int tx = N / MidTile::kX + 1, ty = N / MidTile::kY + 1, K = N / 2 + 1;
    const int planes = march_steps(tx * ty, K, 16384);
    hipLaunchKernelGGL(k_midpoints<TRUE>, dim3(tx, ty, (K + planes - 1) / planes),
                       dim3(MidTile::kX, MidTile::kY), 0, st, N, planes, H, C, out);
    return hipGetLastError();
}

}  // namespace

hipError_t exp_finite(int N, const double *u1, const double *u0, double *v_scratch, double *w,
                      hipStream_t st) {
    // Steps 1-4: Z1, then Step 5
    hipError_t e = midpoints<false>(N / 2, u1, u0, v_scratch, st);
    if (e != hipSuccess) return e;
    const int tx = N / CellTile::kX + 1, ty = N / CellTile::kY + 1, N0 = N / 4;
    const int cells = march_steps(tx * ty, N0, 1024);
    hipLaunchKernelGGL(k_interpolate, dim3(tx, ty, (N0 + cells - 1) / cells),
                       dim3(kCellThreads), 0, st, N, cells, v_scratch, w);
    return hipGetLastError();
}

hipError_t exp_true(int N, const double *uh, const double *u2h, double *ut, hipStream_t st) {
    return midpoints<true>(N, uh, u2h, ut, st);
}

}  // namespace excmg
