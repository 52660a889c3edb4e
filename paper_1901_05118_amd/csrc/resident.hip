// Resident Bi-CG (gfx950): a whole run of Algorithm 2 in one launch, for grids whose vectors
// fit on the chip.
//
// What bounds the launch-per-sweep form there: two launches per iteration, each with its
// drain, its dispatch and a merge of the other sweep's partials (9 us a launch on 16^3 and
// 32^3), and from 64^3 on the vectors' way through the caches.  Here every workgroup owns a
// brick of the grid (of the plane in 2D, the rows of which are z here) for the whole run: the iterate and r, r*, p, p*, q, q* of its cells stay
// in registers, the marched array (p, then p*) in LDS with a 2-wide halo.  An iteration
// exchanges, all past the L2 (which the XCDs do not share),
//  * the partials of sigma, and of rho' and r.r (all to all: every workgroup merges all of
//    them in one order, so all take the same scalars and the same decisions), and
//  * r and r* of the cells that other bricks read (within two of a brick's face, within one of
//    its edges); p and p* of the halo are then formed by the reader, r + beta p as the owner
//    forms them, so there are two exchanges per iteration (with sigma's and with rho's
//    partials), not three.
// A word of a partial carries 4 bytes of data and the number of the exchange, so it proves
// itself new: no flag, no clearing.  The exchanged cells are plain: a workgroup sends its
// partials of rho' only when its sent cells have arrived (agent-scope stores, waited for), so
// who has all partials may read all cells.  Either is overwritten one iteration later, after
// a reduction that needed all its readers.
//
// What bounds an iteration now (cycles at 2.35 GHz, 64^3 on 128 workgroups, of 21000): the two
// exchanges (a load past the L2 takes 1800), the two stencils (4600: LDS reads, 16 per
// output), the directions, the update with its dot products.
//
// Measured choices: exchanged cells in mailboxes, contiguous per reader, against cells in
// grid order, each word proving itself: 64^3 10.6 -> 8.5 us, 96^3 22.3 -> 17.5 us (half the
// bytes and whole lines: what the CUs can load past the L2 bounds the exchange); q* formed
// while sigma's partials travel; partials first looked for kFirstLook after they are sent
// (at once: 32^3 6.1 -> 5.3 us, a look that comes too early costs another); the iterate in
// registers, not in memory (96^3 32 -> 26 us).
//
// Arithmetic: element for element that of the sweeps (zmarch.hpp, k_bicg_update), so the
// iterates are the same; only the partition of the compensated sums differs, as it does
// between launch shapes.
//
// The workgroups wait for each other, so they are launched cooperatively (one per CU, all
// resident) and every wait is bounded: past kWaitTicks the launch gives up (err set, the
// caller's vectors untouched) and the host runs the launch-per-sweep form instead.
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"
#include "step.hpp"

namespace excmg {

typedef unsigned long long u64;

namespace {

constexpr int kFirstLook = 24;              // s_sleep units (64 cycles)
constexpr u64 kWaitTicks = 200000000ull;    // 2 s of the 100 MHz constant clock

// Exchanged memory is accessed 16 bytes at a time, at agent scope (sc1: past the L2 that the
// XCDs do not share): two 8-byte words of {4 bytes of data, exchange number}, each proving
// itself, so nothing is assumed of the two together.  A place out of range reads as zeros,
// without a memory access, and takes no store.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
constexpr int kAgent = 0x10;     // sc1
constexpr unsigned kNoPlace = 0xfffffff0u;
constexpr unsigned kNoCell = 0x0fffffffu;     // (its place is out of range in 8 and 16 bytes)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t exchange_rsrc(void *p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(p, (short)0, (int)bytes, 0x00027000);
}
__device__ __forceinline__ u32x4 get(__amdgpu_buffer_rsrc_t r, unsigned place, unsigned plane) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, (int)place, (int)plane, kAgent);
}
__device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, unsigned place, unsigned plane,
                                    unsigned a, unsigned b, unsigned ep) {
    const u32x4 w = {a, ep, b, ep};
    __builtin_amdgcn_raw_buffer_store_b128(w, r, (int)place, (int)plane, kAgent);
}
__device__ __forceinline__ bool is_new(u32x4 w, unsigned ep) { return w[1] == ep && w[3] == ep; }
__device__ __forceinline__ unsigned low(double v) { return (unsigned)(u64)__double_as_longlong(v); }
__device__ __forceinline__ unsigned high(double v) {
    return (unsigned)((u64)__double_as_longlong(v) >> 32);
}
__device__ __forceinline__ double as_double(u32x4 w) {
    return __longlong_as_double((long long)(((u64)w[2] << 32) | w[0]));
}

// r and r* of one cell in a mailbox: 8 or 16 bytes, at agent scope.
__device__ __forceinline__ void put_cell(__amdgpu_buffer_rsrc_t x, unsigned cell, float r, float s) {
    const u32x2 w = {__float_as_uint(r), __float_as_uint(s)};
    __builtin_amdgcn_raw_buffer_store_b64(w, x, (int)(8 * cell), 0, kAgent);
}
__device__ __forceinline__ void put_cell(__amdgpu_buffer_rsrc_t x, unsigned cell, double r, double s) {
    const u32x4 w = {low(r), high(r), low(s), high(s)};
    __builtin_amdgcn_raw_buffer_store_b128(w, x, (int)(16 * cell), 0, kAgent);
}
__device__ __forceinline__ void get_cell(__amdgpu_buffer_rsrc_t x, unsigned cell, float &r, float &s) {
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(x, (int)(8 * cell), 0, kAgent);
    r = __uint_as_float(w[0]);
    s = __uint_as_float(w[1]);
}
__device__ __forceinline__ void get_cell(__amdgpu_buffer_rsrc_t x, unsigned cell, double &r, double &s) {
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(x, (int)(16 * cell), 0, kAgent);
    r = __longlong_as_double((long long)(((u64)w[1] << 32) | w[0]));
    s = __longlong_as_double((long long)(((u64)w[3] << 32) | w[2]));
}

// v of the lane that a DPP control pairs with this one.
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
    const u64 b = (u64)__double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((u64)hi << 32) | lo));
}
template <int NV, int CTRL>
__device__ __forceinline__ void merge_dpp(Pair (&v)[NV]) {
#pragma unroll
    for (int q = 0; q < NV; q++)
        v[q] = pair_merge(v[q], Pair{dpp_double<CTRL>(v[q].s), dpp_double<CTRL>(v[q].c)});
}
// v of both rows (ROWS16) or both halves of the wave that this lane's row or half is paired
// with: x from the even one, y from the odd one, on all lanes.
template <bool ROWS16>
__device__ __forceinline__ void swap_double(double v, double &x, double &y) {
    const u64 b = (u64)__double_as_longlong(v);
    const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
    u64 xb, yb;
    if constexpr (ROWS16) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        xb = ((u64)h[0] << 32) | l[0];
        yb = ((u64)h[1] << 32) | l[1];
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        xb = ((u64)h[0] << 32) | l[0];
        yb = ((u64)h[1] << 32) | l[1];
    }
    x = __longlong_as_double((long long)xb);
    y = __longlong_as_double((long long)yb);
}
template <int NV, bool ROWS16>
__device__ __forceinline__ void merge_swap(Pair (&v)[NV]) {
#pragma unroll
    for (int q = 0; q < NV; q++) {
        Pair x, y;
        swap_double<ROWS16>(v[q].s, x.s, y.s);
        swap_double<ROWS16>(v[q].c, x.c, y.c);
        v[q] = pair_merge(x, y);
    }
}
// Merge over the first 16 lanes (the others hold zeros or are not looked at), over the wave:
// lane pairs by DPP (neighbours, quads' halves, mirrored quads, mirrored eights), then rows
// and halves swapped; the merge is commutative bit for bit, so all lanes hold the same pair.
template <int NV>
__device__ __forceinline__ void row_merge_n(Pair (&v)[NV]) {
    merge_dpp<NV, 0xB1>(v);
    merge_dpp<NV, 0x4E>(v);
    merge_dpp<NV, 0x141>(v);
    merge_dpp<NV, 0x140>(v);
}
template <int NV>
__device__ __forceinline__ void wave_merge_n(Pair (&v)[NV]) {
    row_merge_n<NV>(v);
    merge_swap<NV, true>(v);
    merge_swap<NV, false>(v);
}

// The pairs of one value of up to 64 workgroups (`place`: this lane's in the exchange memory,
// kNoPlace: none; its sum and its compensation in two planes), merged over the wave.  Sets
// *bad when the wait runs out.
constexpr int kMaxGroups = 256;
constexpr unsigned kSlotPlane = kMaxGroups * 16;
__device__ __forceinline__ Pair gather_pairs(__amdgpu_buffer_rsrc_t slots, unsigned place,
                                             unsigned plane, unsigned ep, int *bad) {
    u32x4 s, c;
    const u64 t0 = wall_clock64();
    bool late = false;
    for (;;) {
        asm volatile("" ::: "memory");     // (every trip loads again)
        s = get(slots, place, plane);
        c = get(slots, place, plane + kSlotPlane);
        if (__all((is_new(s, ep) && is_new(c, ep)) || place == kNoPlace)) break;
        late = wall_clock64() - t0 > kWaitTicks;
        if (late) break;
    }
    if (late) *bad = 1;
    Pair v[1] = {Pair{as_double(s), as_double(c)}};     // (no place reads as zeros)
    wave_merge_n<1>(v);
    return v[0];
}

// The 25-point sums of C consecutive outputs of one column.  B points two rows, two cells and
// two planes below output 0 in LDS (row stride RS, plane stride ps), so that every read of a
// plane is one address and a constant offset.  Terms in the order of eq. (method1), as
// column_step.
template <int C, int RS, typename T, class Emit>
__device__ __forceinline__ void column_outputs(const T *B, int ps, Emit emit) {
    constexpr int O = 2 * RS + 2;     // the column itself
    auto around = [&](const T *P) {
        const double n0 = P[O - 1], n1 = P[O + 1], n2 = P[O - RS], n3 = P[O + RS];
        return n0 + n1 + n2 + n3;
    };
    const T *P = B + 2 * ps;          // plane of output k
    double cm2 = B[O], cm1 = B[ps + O], c0 = P[O], c1 = P[ps + O];
    double am1 = around(B + ps), a0 = around(P);
#pragma unroll
    for (int k = 0; k < C; k++, P += ps) {
        const double c2 = P[2 * ps + O];
        const double a1 = around(P + ps);
        const double f0 = P[O - 2], f1 = P[O + 2], f2 = P[O - 2 * RS], f3 = P[O + 2 * RS];
        const double d0 = P[O - 1 - RS], d1 = P[O - 1 + RS], d2 = P[O + 1 - RS], d3 = P[O + 1 + RS];
        const double s1 = (a0 + cm1) + c1;
        const double s2 = ((f0 + f1 + f2 + f3) + cm2) + c2;
        const double s3 = ((d0 + d1 + d2 + d3) + am1) + a1;
        emit(k, 42.0 * c0 - 12.0 * s1 + s2 + 2.0 * s3);
        if (C >= 8) __builtin_amdgcn_sched_barrier(0);
        cm2 = cm1;
        cm1 = c0;
        c0 = c1;
        c1 = c2;
        am1 = a0;
        a0 = a1;
    }
}

// The 13-point sums of the plane (2D): C consecutive rows of one column, B two cells and two
// rows below output 0 (rows ps apart).  Terms in the order of plane2d.hpp.
template <int C, typename T, class Emit>
__device__ __forceinline__ void column_outputs_2d(const T *B, int ps, Emit emit) {
    const T *P = B + 2 * ps;
    double cm2 = B[2], cm1 = B[ps + 2], c0 = P[2], c1 = P[ps + 2];
    double lm1 = B[ps + 1], rm1 = B[ps + 3], l0 = P[1], r0 = P[3];   // x-, x+ of rows k-1, k
#pragma unroll
    for (int k = 0; k < C; k++, P += ps) {
        const double c2 = P[2 * ps + 2], l1 = P[ps + 1], r1 = P[ps + 3];
        const double f0 = P[0], f1 = P[4];
        const double s1 = l0 + r0 + cm1 + c1;
        const double s2 = f0 + f1 + cm2 + c2;
        const double s3 = lm1 + l1 + rm1 + r1;
        emit(k, 20.0 * c0 - 8.0 * s1 + s2 + 2.0 * s3);
        cm2 = cm1;
        cm1 = c0;
        c0 = c1;
        c1 = c2;
        lm1 = l0;
        rm1 = r0;
        l0 = l1;
        r0 = r1;
    }
}

// Halo cell h of a brick of bx x by x bz cells: its coordinates relative to the brick
// (-2..b+1).  The scheme reaches two cells along an axis and one along two axes.  In 2D the
// plane's rows are z, and y is 0 (by = 1).
template <int DIM>
__device__ __forceinline__ bool halo_cell(int h, int bx, int by, int bz, int &x, int &y, int &z) {
    auto side = [](int s, int b) { return s < 2 ? s - 2 : b + s - 2; };   // -2, -1, b, b+1
    auto near = [](int s, int b) { return s == 0 ? -1 : b; };
    if constexpr (DIM == 2) {
        y = 0;
        if (h < 4 * bx) {
            x = h % bx; z = side(h / bx, bz);
            return true;
        }
        h -= 4 * bx;
        if (h < 4 * bz) {
            x = side(h & 3, bx); z = h >> 2;
            return true;
        }
        h -= 4 * bz;
        x = near(h & 1, bx); z = near(h >> 1, bz);
        return h < 4;
    }
    if (h < 4 * bx * by) {
        x = h % bx; y = (h / bx) % by; z = side(h / (bx * by), bz);
        return true;
    }
    h -= 4 * bx * by;
    if (h < 4 * bx * bz) {
        x = h % bx; z = (h / bx) % bz; y = side(h / (bx * bz), by);
        return true;
    }
    h -= 4 * bx * bz;
    if (h < 4 * by * bz) {
        const int s = h & 3;
        h >>= 2;
        x = side(s, bx); y = h % by; z = h / by;
        return true;
    }
    h -= 4 * by * bz;
    if (h < 4 * bx) {
        x = h % bx; h /= bx; y = near(h & 1, by); z = near(h >> 1, bz);
        return true;
    }
    h -= 4 * bx;
    if (h < 4 * by) {
        y = h % by; h /= by; x = near(h & 1, bx); z = near(h >> 1, bz);
        return true;
    }
    h -= 4 * by;
    if (h < 4 * bz) {
        z = h % bz; h /= bz; x = near(h & 1, bx); y = near(h >> 1, by);
        return true;
    }
    return false;
}

// One run.  C: consecutive z-cells per thread; NH: halo cells per thread; MT: the largest
// workgroup (threads); MULTI: more than one brick.
template <int DIM, typename T, int C, int RS, int NH, int MT, bool MULTI>
__global__ void __launch_bounds__(MT) k_resident(ResidentRun<T> a) {
    extern __shared__ char lds_raw[];
    __shared__ Pair red[2 * (MT / kWave)];
    __shared__ Pair all_a[4], all_b[8];
    __shared__ int bad;
    T *M = (T *)lds_raw;
    int tid = threadIdx.x;
    const int nt = blockDim.x, nw = nt >> 6;
    const int W = MULTI ? gridDim.x : 1, blk = MULTI ? blockIdx.x : 0;
    const int n = a.n, bx = a.bx, by = a.by, bz = a.bz;
    const int x0 = (blk % a.nbx) * bx, y0 = ((blk / a.nbx) % a.nby) * by,
              z0 = (blk / (a.nbx * a.nby)) * bz;
    const int groups = (bz + C - 1) / C;
    constexpr int BX = RS;
    constexpr int HY = DIM == 3 ? 2 : 0;       // halo rows in y
    const int ny = DIM == 3 ? n : 1;
    const int PS = DIM == 3 ? BX * (by + 4) : BX, LE = PS * (groups * C + 4);
    BicgState *S = a.state;
    int status = S->status, iter = S->iter;
    if (status != kRunning) return;            // uniform

    // the box of the marched array; one more element takes what has no place in it
    for (int e = tid; e <= LE; e += nt) M[e] = (T)0;
    if (tid == 0) bad = 0;
    if (tid < 4) all_a[tid] = all_b[2 * tid] = all_b[2 * tid + 1] = Pair{0.0, 0.0};

    // this thread's column of C cells (those from `cells` on are none)
    const int lx = tid % bx, ly = (tid / bx) % by, lg = tid / (bx * by);
    const int gx = x0 + lx, gy = y0 + ly, gz = z0 + lg * C;
    int cells = (lg < groups && gx < n && gy < ny) ? max(0, min(C, min(n, z0 + bz) - gz)) : 0;
    int ob = ((min(lg, groups - 1) * C + 2) * (by + 2 * HY) + ly + HY) * BX + lx + 2;
    int gi = cells > 0 ? (gz * ny + gy) * n + gx : 0;
    const int gplane = cells > 0 ? ny * n : 0;
    // fictitious points that mirror this column
    const int ghx = cells == 0 ? 0 : gx == 0 ? -2 : (gx == n - 1 ? 2 : 0);
    const int ghy = cells == 0 || DIM == 2 ? 0 : gy == 0 ? -2 * BX : (gy == n - 1 ? 2 * BX : 0);
    const int ghz0 = cells > 0 && gz == 0, ghz1 = cells > 0 && gz + cells == n;
    // Mailboxes: the halo cells of a brick, in the order of halo_cell, in one piece of memory.
    // This thread reads cells tid, tid + nt, ... of its own box, and sends the same cells of
    // its neighbours' boxes, as far as this brick owns them (bricks but the last of an axis
    // are whole, so cell h of a neighbour's box is owned by the brick on the other side).
    const int hn = DIM == 3 ? 4 * (bx * by + bx * bz + by * bz + bx + by + bz) : 4 * (bx + bz + 1);
    const __amdgpu_buffer_rsrc_t xc = exchange_rsrc(a.cells, 2u * sizeof(T) * (unsigned)(W * hn)),
                                 xs = exchange_rsrc(a.slots, 6 * kSlotPlane);
    const int own = bx * by * groups * C;     // staged r and r* of the brick: R, R + own
    T *R = M + LE + 1;
    const int os = cells > 0 ? (lg * C * by + ly) * bx + lx : 0, oplane = bx * by;
    int hplace[MULTI ? NH : 1];               // place in LDS (LE: none) | staged source << 16
    unsigned hdest[MULTI ? NH : 1];           // cell of a neighbour's box (kNoCell: none)
    T hr[MULTI ? NH : 1], hs[MULTI ? NH : 1], hv[MULTI ? NH : 1];  // r, r*, the direction not in LDS
    if (MULTI) {
#pragma nounroll
        for (int q = 0; q < NH; q++) {
            // (a scratch-free loop: every trip decodes slot q and keeps it by selects)
            int x, y, z, place = LE;
            unsigned dest = kNoCell;
            const int h = tid + q * nt;
            if (halo_cell<DIM>(h, bx, by, bz, x, y, z)) {
                const int X = x0 + x, Y = y0 + y, Z = z0 + z;
                if (X >= 0 && X < n && Y >= 0 && Y < ny && Z >= 0 && Z < n)
                    place = ((z + 2) * (by + 2 * HY) + y + HY) * BX + x + 2;
                // the brick that has cell h of its box here, and the cell's place in this one
                const int dx = x < 0 ? 1 : (x >= bx ? -1 : 0), dy = y < 0 ? 1 : (y >= by ? -1 : 0),
                          dz = z < 0 ? 1 : (z >= bz ? -1 : 0);
                const int X0 = x0 + dx * bx, Y0 = y0 + dy * by, Z0 = z0 + dz * bz;
                const int sx = x + dx * bx, sy = y + dy * by, sz = z + dz * bz;
                if (X0 >= 0 && X0 < n && Y0 >= 0 && Y0 < ny && Z0 >= 0 && Z0 < n && x0 + sx < n &&
                    y0 + sy < ny && z0 + sz < n) {
                    dest = (unsigned)((blk + dx + a.nbx * (dy + a.nby * dz)) * hn + h);
                    place |= ((sz * by + sy) * bx + sx) << 16;
                }
            }
#pragma unroll
            for (int u = 0; u < NH; u++) {
                hplace[u] = u == q ? place : (q == 0 ? LE : hplace[u]);
                hdest[u] = u == q ? dest : (q == 0 ? kNoCell : hdest[u]);
            }
        }
    }
    auto hoff = [&](int q) { return hplace[q] & 0xffff; };

    // own values into LDS, and into the fictitious points that mirror them
    const bool edge = ghx || ghy || ghz0 || ghz1;
    auto place = [&](const T (&v)[C]) {
#pragma unroll
        for (int c = 0; c < C; c++) M[c < cells ? ob + c * PS : LE] = v[c];
        if (edge) {
            const bool neg = a.sgn < 0;
#pragma unroll
            for (int c = 0; c < C; c++) {
                if (c < cells) {
                    T *P = M + ob + c * PS;
                    const T g = neg ? -v[c] : v[c];
                    if (ghx) P[ghx] = g;
                    if (ghy) P[ghy] = g;
                    if (c == 0 && ghz0) P[-2 * PS] = g;
                    if (c == cells - 1 && ghz1) P[2 * PS] = g;
                }
            }
        }
    };

    // ---- start or resume: scalars, then r, r*, p, p* of the brick and its halo
    const int maxit = S->maxit;
    const double thr = S->thr;
    double rho = S->rho, rr = S->rr, beta = 0.0, alpha = S->alpha, sigma = S->sigma;
    double rho_old = rho;
    const bool first = (iter == 0);
    __syncthreads();
    if (!first) {
        // rho of the replaced residual and the checks of the loop (see link_step)
        rho_old = S->rho_slot[(iter & 1) ^ 1];
        Pair v[2];
        merge_fixed<2>(a.part, a.part_count, v, red);
        rho = pair_value(v[0]);
        rr = pair_value(v[1]);
        if (rr <= thr) status = kConverged;
        else if (iter >= maxit) status = kNoConv;
        else if (rho == 0.0 || !isfinite(rho)) status = kBreakdown;
        beta = rho / rho_old;
    }

    // In the first iteration of a run p = r and p* = r*: the old directions are zeros and
    // beta is 0.
    T r[C], s[C], o[C];      // r, r*, and p while LDS holds p* (p* while it holds p)
    double xv[C];            // the iterate
    {
        const T *p = a.p[iter & 1], *ps = a.ps[iter & 1];
#pragma unroll
        for (int c = 0; c < C; c++) {
            r[c] = s[c] = o[c] = (T)0;
            xv[c] = 0.0;
            if (c < cells) {
                const unsigned i = gi + c * gplane;
                r[c] = a.r[i];
                s[c] = a.rs[i];
                xv[c] = a.x[i];
                if (!first) {
                    o[c] = p[i];
                    M[ob + c * PS] = ps[i];
                }
            }
        }
        if (MULTI) {
#pragma unroll
            for (int q = 0; q < NH; q++) {
                hr[q] = hs[q] = hv[q] = (T)0;
                int x, y, z;
                if (hoff(q) != LE && halo_cell<DIM>(tid + q * nt, bx, by, bz, x, y, z)) {
                    const unsigned i = (unsigned)(((z0 + z) * ny + y0 + y) * n + x0 + x);
                    hr[q] = a.r[i];
                    hs[q] = a.rs[i];
                    if (!first) {
                        hv[q] = p[i];
                        M[hoff(q)] = ps[i];
                    }
                }
            }
        }
    }
    unsigned ep = a.epoch;
    // Phases of an iteration are kept apart in the registers: addresses and FP64 forms of FP32
    // values that one phase derives are not carried into the next.
    auto keep = [&]() {
        asm volatile("" : "+v"(ob), "+v"(cells));
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int c = 0; c < C; c++) asm volatile("" : "+v"(r[c]), "+v"(s[c]), "+v"(o[c]));
        }
        if (MULTI) {
#pragma unroll
            for (int q = 0; q < NH; q++) asm volatile("" : "+v"(hplace[q]), "+v"(hdest[q]));
        }
    };

    auto stencil = [&](auto emit) {
        const T *B = M + (ob - 2 * PS - HY * RS - 2);
        if constexpr (DIM == 3) column_outputs<C, RS, T>(B, PS, emit);
        else column_outputs_2d<C, T>(B, PS, emit);
    };

    while (status == kRunning) {
        ep++;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63, wave = tid >> 6;
        keep();
        // ---- directions: p into LDS, p* into o and hv
        T ho[MULTI ? NH : 1];
        {
            T pn[C], so[C];
#pragma unroll
            for (int c = 0; c < C; c++) so[c] = M[ob + c * PS];
            if (MULTI) {
#pragma unroll
                for (int q = 0; q < NH; q++) ho[q] = M[hoff(q)];
            }
#pragma unroll
            for (int c = 0; c < C; c++) {
                pn[c] = (T)((double)r[c] + beta * (double)o[c]);
                o[c] = (T)((double)s[c] + beta * (c < cells ? (double)so[c] : 0.0));
            }
            place(pn);
        }
        if (MULTI) {
#pragma unroll
            for (int q = 0; q < NH; q++)
                M[hoff(q)] = (T)((double)hr[q] + beta * (double)hv[q]);
#pragma unroll
            for (int q = 0; q < NH; q++) hv[q] = (T)((double)hs[q] + beta * (double)ho[q]);
        }
        __syncthreads();
        keep();

        // ---- q = A p, sigma = p*.q
        T qv[C], qs[C];
        Pair sg[1] = {{0.0, 0.0}};
        stencil([&](int c, double y) {
            qv[c] = c < cells ? (T)y : (T)0;
            dot2_acc(sg[0], (double)o[c], (double)qv[c]);
            // (one output after the other)
            if (C >= 8) asm volatile("" : "+v"(sg[0].s), "+v"(sg[0].c), "+v"(qv[c]));
        });
        wave_merge_n<1>(sg);
        if (lane == 0) red[wave] = sg[0];
        __syncthreads();     // also: every thread has read p
        if (wave == 0) {
            Pair v[1] = {lane < nw ? red[lane] : Pair{0.0, 0.0}};
            row_merge_n<1>(v);
            if (MULTI) {
                if (lane < 2) {
                    const double b = lane == 0 ? v[0].s : v[0].c;
                    put(xs, 16u * (unsigned)blk + lane * kSlotPlane, 0, low(b), high(b), ep);
                }
            } else if (lane == 0) {
                all_a[0] = v[0];
            }
        }
        // ---- p* into LDS, p into o and hv; q* = A^T p*
        keep();
        {
            T pv[C];
#pragma unroll
            for (int c = 0; c < C; c++) pv[c] = M[ob + c * PS];
            if (MULTI) {
#pragma unroll
                for (int q = 0; q < NH; q++) ho[q] = M[hoff(q)];
            }
            place(o);
#pragma unroll
            for (int c = 0; c < C; c++) o[c] = c < cells ? pv[c] : (T)0;
        }
        if (MULTI) {
#pragma unroll
            for (int q = 0; q < NH; q++) {
                M[hoff(q)] = hv[q];
                hv[q] = ho[q];
            }
        }
        __syncthreads();
        keep();
        stencil([&](int c, double y) {
            qs[c] = c < cells ? (T)y : (T)0;
            if (C >= 8) asm volatile("" : "+v"(qs[c]));
        });
        // (q* is formed here, before the wait, not carried over it as its 21 C terms)
#pragma unroll
        for (int c = 0; c < C; c++) asm volatile("" : "+v"(qs[c]));

        // ---- sigma and alpha
        if (MULTI) {
            if (64 * wave < W) {
                const Pair v = gather_pairs(xs, tid < W ? 16u * (unsigned)tid : kNoPlace, 0, ep, &bad);
                if (lane == 0) all_a[wave] = v;
            }
            __syncthreads();
            if (bad) break;
        }
        {
            Pair v = all_a[0];
            if (W > 64) v = pair_merge(pair_merge(v, all_a[1]), pair_merge(all_a[2], all_a[3]));
            sigma = wave_uniform(pair_value(v));
        }
        if (sigma == 0.0 || !isfinite(sigma)) {
            status = kBreakdown;
            break;
        }
        alpha = wave_uniform(rho / sigma);
        iter++;

        keep();
        // ---- r -= alpha q, r* -= alpha q*; rho' = r*.r and r.r; x += alpha p
        Pair dt[2] = {{0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
        for (int c = 0; c < C; c++) {
            r[c] = (T)((double)r[c] - alpha * (double)qv[c]);
            s[c] = (T)((double)s[c] - alpha * (double)qs[c]);
            if (MULTI && c < cells) {
                R[os + c * oplane] = r[c];
                R[own + os + c * oplane] = s[c];
            }
        }
        if (MULTI) {
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NH; q++) {
                const int src = (unsigned)hplace[q] >> 16;
                put_cell(xc, hdest[q], R[src], R[own + src]);
            }
        }
        keep();
#pragma unroll
        for (int c = 0; c < C; c++) {
            dot2_acc(dt[0], (double)s[c], (double)r[c]);
            dot2_acc(dt[1], (double)r[c], (double)r[c]);
            xv[c] = xv[c] + alpha * (double)o[c];
        }
        wave_merge_n<2>(dt);
        if (lane == 0) {
            red[2 * wave] = dt[0];
            red[2 * wave + 1] = dt[1];
        }
        // the sent cells have arrived (stores past the L2) before the partials announce them
        if (MULTI) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (wave == 0) {
            Pair v[2] = {{0.0, 0.0}, {0.0, 0.0}};
            if (lane < nw) {
                v[0] = red[2 * lane];
                v[1] = red[2 * lane + 1];
            }
            row_merge_n<2>(v);
            if (MULTI) {
                if (lane < 4) {
                    const Pair pv = lane < 2 ? v[0] : v[1];
                    const double b = (lane & 1) ? pv.c : pv.s;
                    put(xs, 16u * (unsigned)blk + (2 + lane) * kSlotPlane, 0, low(b), high(b), ep);
                }
            } else if (lane == 0) {
                all_b[0] = v[0];
                all_b[1] = v[1];
            }
        }
        if (MULTI) {
            // A load takes about 1800 cycles (past the L2); asked too early it is asked twice.
            __builtin_amdgcn_s_sleep(kFirstLook);
            if (64 * (wave >> 1) < W) {     // even waves: rho', odd waves: r.r
                const int w = (wave >> 1) * 64 + lane;
                const Pair v = gather_pairs(xs, w < W ? 16u * (unsigned)w : kNoPlace,
                                            (2 + 2 * (wave & 1)) * kSlotPlane, ep, &bad);
                if (lane == 0) all_b[wave] = v;
            }
            __syncthreads();
            // all partials are here, so all cells are: r and r* of the halo (a cell of the box
            // that the grid does not have reads as anything and goes nowhere)
            unsigned cell = (unsigned)(blk * hn + tid);
#pragma unroll
            for (int q = 0; q < NH; q++, cell += nt) get_cell(xc, cell, hr[q], hs[q]);
        } else {
            __syncthreads();
        }
        if (MULTI && bad) break;
        // ---- end of the iteration: the stopping checks in the order of the loop, then beta
        rho_old = rho;
        {
            Pair v[2] = {all_b[0], all_b[1]};
            if (W > 64) {
#pragma unroll
                for (int q = 0; q < 2; q++)
                    v[q] = pair_merge(pair_merge(v[q], all_b[2 + q]),
                                      pair_merge(all_b[4 + q], all_b[6 + q]));
            }
            rho = wave_uniform(pair_value(v[0]));
            rr = wave_uniform(pair_value(v[1]));
        }
        if (rr <= thr) status = kConverged;
        else if (iter >= maxit) status = kNoConv;
        else if (rho == 0.0 || !isfinite(rho)) status = kBreakdown;
        beta = wave_uniform(rho / rho_old);
    }
    if (MULTI && bad) {
        if (tid == 0) atomicExch(&S->err, 1);
        return;
    }
    // the iterate, and the directions for a run that goes on after its residuals are replaced
    {
        T *p = a.p[iter & 1], *ps = a.ps[iter & 1];
#pragma unroll
        for (int c = 0; c < C; c++) {
            if (c < cells) {
                const unsigned i = gi + c * gplane;
                a.x_work[i] = xv[c];
                p[i] = o[c];
                ps[i] = M[ob + c * PS];
            }
        }
    }
    if (blk == 0 && tid == 0) {
        S->rr = rr;
        S->rho = rho;
        S->rho_slot[iter & 1] = rho;
        S->rho_slot[(iter & 1) ^ 1] = rho_old;
        S->alpha = alpha;
        S->beta = beta;
        S->sigma = sigma;
        S->iter = iter;
        S->status = status;
        S->poll_status = status;
    }
}

template <int DIM, typename T, int C, int RS, int NH, int MT>
hipError_t launch_resident(const ResidentPlan &pl, ResidentRun<T> run, hipStream_t st) {
    const void *fn = pl.blocks > 1 ? (const void *)k_resident<DIM, T, C, RS, NH, MT, true>
                                   : (const void *)k_resident<DIM, T, C, RS, NH, MT, false>;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds);
    if (e != hipSuccess) return e;
    void *args[] = {&run};
    return hipLaunchCooperativeKernel(fn, dim3(pl.blocks), dim3(pl.threads), args,
                                      (unsigned)pl.lds, st);
}

// Halo cells per thread and largest workgroup of the kernel with C cells per thread (what
// its registers hold without spilling; 16 cells: FP32 in 3D only).
constexpr int halo_slots(int C, int dim) { return dim == 2 ? 2 : C <= 2 ? 4 : C == 4 ? 6 : C == 8 ? 8 : 11; }
constexpr int max_threads(int C, bool fp64, int dim) {
    return C == 16 && (fp64 || dim == 2) ? 0 : C <= 2 && !fp64 ? 1024 : 512;
}
constexpr size_t kMaxLds = 158 * 1024;     // of 160 KB per workgroup; the rest is static

// Partition of the grid into nbx x nby x nbz bricks (2D: rows are z, nby = 1) with C cells
// per thread; false if the kernels cannot take it.
bool try_plan(int n, int dim, bool fp64, int nbx, int nby, int nbz, int C, ResidentPlan &p) {
    const int ny = dim == 2 ? 1 : n;
    p.bx = (n + nbx - 1) / nbx;
    p.by = (ny + nby - 1) / nby;
    p.bz = (n + nbz - 1) / nbz;
    p.nbx = (n + p.bx - 1) / p.bx;
    p.nby = (ny + p.by - 1) / p.by;
    p.nbz = (n + p.bz - 1) / p.bz;
    p.C = C;
    p.dim = dim;
    p.blocks = p.nbx * p.nby * p.nbz;
    const bool one = p.blocks == 1;
    // rows of the LDS box hold up to 32 cells; a brick is at least as wide as the scheme reaches
    if (p.blocks > kMaxGroups || p.bx > 32) return false;
    if (!one && (std::min(p.bx, p.bz) < 2 || (dim == 3 && p.by < 2))) return false;
    const int groups = (p.bz + C - 1) / C;
    const long long columns = (long long)p.bx * p.by * groups;
    // at least the four waves of merge_fixed, and two waves per 64 workgroups to gather the
    // partials of rho' and r.r
    const long long waves = std::max({4LL, (columns + 63) / 64, (p.blocks + 63) / 64 * 2LL});
    if (64 * waves > max_threads(C, fp64, dim)) return false;
    p.threads = (int)(64 * waves);
    const long long halo = dim == 2 ? 4LL * (p.bx + p.bz + 1)
                                    : 4LL * (p.bx * p.by + p.bx * p.bz + p.by * p.bz + p.bx + p.by + p.bz);
    if (!one && halo > (long long)halo_slots(C, dim) * p.threads) return false;
    const size_t es = fp64 ? 8 : 4;
    p.rs = p.bx <= 16 && dim == 3 ? 20 : 36;
    p.lds = ((size_t)p.rs * (dim == 2 ? 1 : p.by + 4) * (groups * C + 4) + 1) * es;
    if (!one) p.lds += 2 * (size_t)columns * C * es;
    p.exchange = one ? 0 : (size_t)p.blocks * halo * 2 * es;
    return p.lds <= kMaxLds;
}

}  // namespace

// The partition of an n^3 grid or n^2 plane: the cheapest by a model of an iteration's time
// (us), fitted to some 5000 partitions of 3D grids of 12 to 96 cells (FP64; what it picks takes
// 0-12% longer than the best of each grid): work per wave and per thread, exchanges that grow
// with the number of workgroups, cells exchanged.  Measured per iteration against the
// launch-per-sweep form: 16^3 5.3 / 17.9, 32^3 5.4 / 18.3, 48^3 7.7 / 21.3, 64^3 10.0 / 26.1,
// 96^3 16.5 / 45.0 us.  FP32 vectors: 96^3 13.4 / 37.3, 112^3 20.1 / 48.9, 128^3 (8192 cells
// per workgroup, 16 per thread) 22 / 45.  Planes, FP64: 128^2 4.7 / 12.1, 256^2 5.0 / 13.3,
// 512^2 7.3 / 24.2, 1024^2 (whole run of 15) 24 / 64.
// FP64 grids above about 100^3 do not fit (16 cells of six FP64 vectors and the halo take more
// than the 256 registers of 512 threads), nor do planes above about 1000^2; smaller grids are
// levels solved directly.
bool resident_plan(int n, int dim, bool fp64, ResidentPlan &plan) {
    if (n < 7 || n > (dim == 2 ? 1024 : 128)) return false;
    double best = 1e30;
    const int most = dim == 2 ? kMaxGroups : 16;
    for (int C : {1, 2, 4, 8, 16})
        for (int bz = 1; bz <= most; bz++)
            for (int by = 1; by <= (dim == 2 ? 1 : most); by++)
                for (int bx = 1; bx <= (dim == 2 ? 32 : 8) && bx * by * bz <= kMaxGroups; bx++) {
                    ResidentPlan p;
                    if (!try_plan(n, dim, fp64, bx, by, bz, C, p)) continue;
                    const double waves = p.threads / 64, W = p.blocks;
                    double t = 0.056 * waves * C + 0.086 * waves + 0.36 * C;
                    if (p.blocks > 1)
                        t += 0.83 + 0.094 * W / 64 + 0.32 * ((p.blocks + 63) / 64) +
                             0.048 * waves * halo_slots(C, dim) +
                             2.1e-7 * (double)p.exchange * (fp64 ? 1 : 2);
                    if (t < best) {
                        best = t;
                        plan = p;
                    }
                }
    return best < 1e30;
}

template <int DIM, typename T, int C>
hipError_t run_cells(const ResidentPlan &p, const ResidentRun<T> &run, hipStream_t st) {
    constexpr int MT = max_threads(C, sizeof(T) == 8, DIM), NH = halo_slots(C, DIM);
    if constexpr (MT == 0) {
        return hipErrorInvalidValue;
    } else {
        if constexpr (DIM == 3) {
            if (p.rs == 20) return launch_resident<DIM, T, C, 20, NH, MT>(p, run, st);
        }
        return launch_resident<DIM, T, C, 36, NH, MT>(p, run, st);
    }
}

template <typename T>
hipError_t resident_run(const ResidentPlan &p, const ResidentRun<T> &run, hipStream_t st) {
#define EXCMG_RESIDENT(CV) \
    case CV: return p.dim == 2 ? run_cells<2, T, CV>(p, run, st) : run_cells<3, T, CV>(p, run, st);
    switch (p.C) {
        EXCMG_RESIDENT(1)
        EXCMG_RESIDENT(2)
        EXCMG_RESIDENT(4)
        EXCMG_RESIDENT(8)
        EXCMG_RESIDENT(16)
        default: return hipErrorInvalidValue;
    }
#undef EXCMG_RESIDENT
}
template hipError_t resident_run<float>(const ResidentPlan &, const ResidentRun<float> &, hipStream_t);
template hipError_t resident_run<double>(const ResidentPlan &, const ResidentRun<double> &, hipStream_t);

}  // namespace excmg
