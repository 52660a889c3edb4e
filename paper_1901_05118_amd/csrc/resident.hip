// Resident Bi-CG (gfx950): a whole run of Algorithm 2 in one launch, for grids whose vectors
// fit on the chip.
//
// What bounds the launch-per-sweep form there: two launches per iteration, each with its
// drain, its dispatch and a merge of the other sweep's partials (9 us a launch on 16^3 and
// 32^3), and from 64^3 on the vectors' way through the caches.  Here every workgroup owns a
// brick of the grid (of the plane in 2D, the rows of which are z here) for the whole run: the
// iterate and r, r*, p, p*, q, q* of its cells stay in registers, the marched array (p, then p*)
// in LDS with a 2-wide halo.  (FP64 with 16 cells per thread, 112^3 and 128^3: the iterate in
// memory, q* not kept; see resident_body.hpp.)  An iteration
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
// What bounds an iteration (64^3, 9.2 us): the two exchanges with the wait for the slowest
// workgroup (2.9; a load past the L2 takes 1800 cycles), the two stencils (2.4: LDS reads, 16 per
// output), the directions, the update with its dot products.
//
// Measured choices (each when it was made, on the partition taken then): exchanged cells in mailboxes, contiguous per reader, against cells in
// grid order, each word proving itself: 64^3 10.6 -> 8.5 us, 96^3 22.3 -> 17.5 us (half the
// bytes and whole lines: what the CUs can load past the L2 bounds the exchange); q* formed
// while sigma's partials travel; partials first looked for some time after they are sent
// (at once: 32^3 6.1 -> 5.3 us, a look that comes too early costs another); the iterate in
// registers, not in memory (96^3 32 -> 26 us).
//
// Small grids run on one XCD (at most 32 workgroups; where they are is found out by the
// workgroups themselves): their stores end in the L2 that they share, and an all-to-all
// exchange takes 1100 cycles instead of 3100.  16^3 5.9 -> 4.9 us, 128^2 4.7 -> 4.0; 32^3 as
// fast either way (5.4 / 5.3: twice the cells per workgroup).  Every wave merging all partials
// itself (no barrier, no way through LDS) was no faster: 4.9 -> 4.8 us on one XCD, 4.7 -> 5.0
// past the L2s.
//
// Arithmetic: element for element that of the sweeps (zmarch.hpp, k_bicg_update), so the
// iterates are the same; only the partition of the compensated sums differs, as it does
// between launch shapes.
//
// The workgroups wait for each other, so they are launched cooperatively (one per CU, all
// resident) and every wait is bounded: past the run's `wait` the launch gives up (err set, a
// single run's vectors untouched) and the host goes on with the launch-per-sweep form.
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"
#include "step.hpp"

namespace excmg {

typedef unsigned long long u64;

namespace {

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
// AUX: kAgent, or 0 between workgroups of one XCD (the store ends in the L2 they share, where
// the reader's load, past its own L1, finds it).
template <int AUX>
__device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, unsigned place, unsigned plane,
                                    unsigned a, unsigned b, unsigned ep) {
    const u32x4 w = {a, ep, b, ep};
    __builtin_amdgcn_raw_buffer_store_b128(w, r, (int)place, (int)plane, AUX);
}
__device__ __forceinline__ bool is_new(u32x4 w, unsigned ep) { return w[1] == ep && w[3] == ep; }
__device__ __forceinline__ unsigned low(double v) { return (unsigned)(u64)__double_as_longlong(v); }
__device__ __forceinline__ unsigned high(double v) {
    return (unsigned)((u64)__double_as_longlong(v) >> 32);
}
__device__ __forceinline__ double as_double(u32x4 w) {
    return __longlong_as_double((long long)(((u64)w[2] << 32) | w[0]));
}

// r and r* of one cell in a mailbox: 8 or 16 bytes.
template <int AUX>
__device__ __forceinline__ void put_cell(__amdgpu_buffer_rsrc_t x, unsigned cell, float r, float s) {
    const u32x2 w = {__float_as_uint(r), __float_as_uint(s)};
    __builtin_amdgcn_raw_buffer_store_b64(w, x, (int)(8 * cell), 0, AUX);
}
template <int AUX>
__device__ __forceinline__ void put_cell(__amdgpu_buffer_rsrc_t x, unsigned cell, double r, double s) {
    const u32x4 w = {low(r), high(r), low(s), high(s)};
    __builtin_amdgcn_raw_buffer_store_b128(w, x, (int)(16 * cell), 0, AUX);
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

// One FP64 value of a mailbox.
__device__ __forceinline__ void put_value(__amdgpu_buffer_rsrc_t x, unsigned cell, double v) {
    const u32x2 w = {low(v), high(v)};
    __builtin_amdgcn_raw_buffer_store_b64(w, x, (int)(8 * cell), 0, kAgent);
}
__device__ __forceinline__ double get_value(__amdgpu_buffer_rsrc_t x, unsigned cell) {
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(x, (int)(8 * cell), 0, kAgent);
    return __longlong_as_double((long long)(((u64)w[1] << 32) | w[0]));
}

// One FP64 value of this workgroup's own (no value past the end).
__device__ __forceinline__ double load_f64(__amdgpu_buffer_rsrc_t x, unsigned i) {
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(x, (int)(8 * i), 0, 0);
    return __longlong_as_double((long long)(((u64)w[1] << 32) | w[0]));
}
__device__ __forceinline__ void store_f64(__amdgpu_buffer_rsrc_t x, unsigned i, double v) {
    const u32x2 w = {low(v), high(v)};
    __builtin_amdgcn_raw_buffer_store_b64(w, x, (int)(8 * i), 0, 0);
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
// *bad when it has waited for `wait` ticks of the constant clock (0: for one look).
constexpr int kMaxGroups = 256;
constexpr unsigned kSlotPlane = kMaxGroups * 16;
__device__ __forceinline__ Pair gather_pairs(__amdgpu_buffer_rsrc_t slots, unsigned place,
                                             unsigned plane, unsigned ep, u64 wait, int *bad) {
    u32x4 s, c;
    const u64 t0 = wall_clock64();
    bool late = false;
    for (;;) {
        asm volatile("" ::: "memory");     // (every trip loads again)
        s = get(slots, place, plane);
        c = get(slots, place, plane + kSlotPlane);
        if (__all((is_new(s, ep) && is_new(c, ep)) || place == kNoPlace)) break;
        late = wall_clock64() - t0 >= wait;
        if (late) break;
    }
    if (late) *bad = 1;
    Pair v[1] = {Pair{as_double(s), as_double(c)}};     // (no place reads as zeros)
    wave_merge_n<1>(v);
    return v[0];
}

// Whether all of up to 64 workgroups sent this value.
__device__ __forceinline__ bool gather_same(__amdgpu_buffer_rsrc_t slots, unsigned place,
                                            unsigned plane, unsigned ep, unsigned value, u64 wait,
                                            int *bad) {
    const u64 t0 = wall_clock64();
    for (;;) {
        asm volatile("" ::: "memory");
        const u32x4 s = get(slots, place, plane);
        if (__all(is_new(s, ep) || place == kNoPlace)) return __all(s[0] == value || place == kNoPlace);
        if (wall_clock64() - t0 >= wait) {
            *bad = 1;
            return false;
        }
    }
}

// The XCD that this workgroup runs on (hardware register XCC_ID, 4 bits).
__device__ __forceinline__ unsigned xcd_id() { return __builtin_amdgcn_s_getreg((3 << 11) | 20); }

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

// A run of its own.  MT: the largest workgroup (threads).
template <int DIM, typename T, int C, int RS, int NH, int MT, bool MULTI>
__global__ void __launch_bounds__(MT) k_resident(ResidentRun<T> a) {
    extern __shared__ char lds_raw[];
    __shared__ Pair red[2 * (MT / kWave)];
    __shared__ Pair all_a[4], all_b[8];
    __shared__ int bad;
    T *M = (T *)lds_raw;
    constexpr bool BATCH = false;
    // one XCD: the launch has 8 times the workgroups, which the XCDs take in turn
    const bool one_xcd = MULTI && C <= 8 && a.one_xcd;
    if (one_xcd && (blockIdx.x & 7)) return;
    const int blk = !MULTI ? 0 : one_xcd ? blockIdx.x >> 3 : blockIdx.x;
    const int W = !MULTI ? 1 : one_xcd ? gridDim.x >> 3 : gridDim.x, nt = blockDim.x;
#include "resident_body.hpp"
}

template <int DIM, typename T, int C, int RS, int NH, int MT>
hipError_t launch_resident(const ResidentPlan &pl, ResidentRun<T> run, hipStream_t st) {
    const void *fn = (const void *)k_resident<DIM, T, C, RS, NH, MT, true>;
    if constexpr (sizeof(T) == 4 || C < 16) {      // (the lean kernel is of several bricks only)
        if (pl.blocks == 1) fn = (const void *)k_resident<DIM, T, C, RS, NH, MT, false>;
    }
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds);
    if (e != hipSuccess) return e;
    void *args[] = {&run};
    return hipLaunchCooperativeKernel(fn, dim3(run.one_xcd ? 8 * pl.blocks : pl.blocks),
                                      dim3(pl.threads), args, (unsigned)pl.lds, st);
}

// Halo cells per thread and largest workgroup of the kernel with C cells per thread (what
// its registers hold; 16 cells: in 3D only).
constexpr int halo_slots(int C, int dim) { return dim == 2 ? 2 : C <= 2 ? 4 : C == 4 ? 6 : C == 8 ? 8 : 11; }
constexpr int max_threads(int C, bool fp64, int dim) {
    return C == 16 && dim == 2 ? 0 : C <= 2 && !fp64 ? 1024 : 512;
}
// (a run of a batch: FP32 with at least 4 cells per thread)
constexpr int max_batch_threads(int C, bool fp64) {
    return C <= 2 && !fp64 ? 0 : 512;
}
constexpr int kXcdGroups = 32;              // CUs of an XCD
constexpr size_t kMaxLds = 158 * 1024;     // of 160 KB per workgroup; the rest is static

// Partition of the grid into nbx x nby x nbz bricks (2D: rows are z, nby = 1) with C cells
// per thread; false if the kernels cannot take it.
bool try_plan(int n, int dim, bool fp64, bool batch, int nbx, int nby, int nbz, int C,
              ResidentPlan &p) {
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
    // at least a wave per SIMD (the model is fitted to no fewer), and two waves per 64 workgroups
    // to gather the partials of rho' and r.r
    const long long waves = std::max({4LL, (columns + 63) / 64, (p.blocks + 63) / 64 * 2LL});
    if (64 * waves > (batch ? max_batch_threads(C, fp64) : max_threads(C, fp64, dim))) return false;
    if (batch && one) return false;
    p.threads = (int)(64 * waves);
    const long long halo = dim == 2 ? 4LL * (p.bx + p.bz + 1)
                                    : 4LL * (p.bx * p.by + p.bx * p.bz + p.by * p.bz + p.bx + p.by + p.bz);
    if (!one && halo > (long long)halo_slots(C, dim) * p.threads) return false;
    const size_t es = fp64 ? 8 : 4;
    p.rs = p.bx <= 16 && dim == 3 ? 20 : 36;
    p.lds = ((size_t)p.rs * (dim == 2 ? 1 : p.by + 4) * (groups * C + 4) + 1) * es;
    const bool lean = fp64 && C == 16;
    if (lean && one) return false;
    if (!one) p.lds += (lean ? (size_t)p.bx * p.by : 2 * (size_t)columns) * C * es;
    p.exchange = one ? 0 : (size_t)p.blocks * halo * 2 * es;
    return p.lds <= kMaxLds;
}

// Every partition that the kernels can take, with its modelled time of an iteration.
template <class Use>
void for_plans(int n, int dim, bool fp64, bool batch, Use use) {
    if (n < 7 || n > (dim == 2 ? 1024 : 128)) return;
    const int most = dim == 2 ? kMaxGroups : 16;
    auto whole = [&](int k) { return (n + (n + k - 1) / k - 1) / ((n + k - 1) / k) == k; };
    for (int C : {1, 2, 4, 8, 16})
        for (int bz = 1; bz <= most; bz++)
            for (int by = 1; by <= (dim == 2 ? 1 : most); by++)
                for (int bx = 1; bx <= (dim == 2 ? 32 : 8) && bx * by * bz <= kMaxGroups; bx++) {
                    ResidentPlan p;
                    // (a number of bricks per axis that rounds to a smaller one comes up there)
                    if (!whole(bz) || !whole(bx) || (dim == 3 && !whole(by))) continue;
                    if (!try_plan(n, dim, fp64, batch, bx, by, bz, C, p)) continue;
                    const double waves = p.threads / 64, W = p.blocks;
                    p.us = fp64 && C == 16 ? 8.0 : 0.0;     // (the iterate in memory)
                    // (rows of other lengths leave LDS banks idle; a cell of the plane has half
                    // the terms)
                    const double cell = 0.0214 + (p.bx % 4 ? 0.0256 : 0.0) + (p.bx % 16 ? 0.0134 : 0.0);
                    p.us += (dim == 2 ? 0.5 : 1.0) * (cell * waves * C + 0.559 * C) + 0.277 * waves;
                    if (p.blocks > 1)
                        p.us += 2.53 + 0.1225 * W / 64 + 0.0853 * ((p.blocks + 63) / 64) +
                                0.005 * waves * halo_slots(C, dim) +
                                6.5e-6 * (double)p.exchange / (fp64 ? 16 : 8);
                    // fewer workgroups, on one XCD (the kernels with 16 cells have no
                    // register for the choice)
                    if (!batch && C <= 8 && p.blocks > 1 && p.blocks <= kXcdGroups) {
                        p.one_xcd = true;
                        p.us -= 0.514;
                    }
                    // The partials of rho' come when the slowest workgroup has sent its own, the
                    // later the longer an iteration is; looks before that delay what they wait
                    // for.  (256 cycles: 28^3 best 5, 48^3 8, 64^3 10-12, 96^3 16; looking at
                    // once 1 us slower throughout, at 6 everywhere 8% at 48^3, 4% at 64^3.)
                    p.look = p.one_xcd ? 1 : (int)std::min(16.0, std::max(5.0, 1.2 * p.us));
                    use(p);
                }
}

}  // namespace

// The partition of an n^3 grid or n^2 plane: the cheapest by a model of an iteration's time
// (us), fitted to 800 partitions of 3D grids of 12 to 96 cells in FP64: work per wave and per
// thread, exchanges that grow with the number of workgroups, cells exchanged.  FP32, planes (half
// the terms a cell) and 16 cells per thread (8 us more) take it with those constants; against the
// best of the 28 cheapest partitions, all timed, what it picks takes longer by: FP64 32^3 9%, 64^3
// 6%, 96^3 0, 112^3 1%, 128^3 0; FP32 32^3 2%, 64^3 4%, 96^3 1%, 112^3 0, 128^3 4%; planes 128^2
// 0, 256^2 2%, 512^2 and 1024^2 0.
// Measured per iteration against the launch-per-sweep form: 16^3 4.1 / 17.9, 32^3 5.2 / 18.3,
// 48^3 6.5 / 21.3, 64^3 9.2 / 26.1, 96^3 15.7 / 45.0 us.  FP32 vectors: 96^3 13.4 / 37.3, 112^3
// 20.1 / 48.9, 128^3 (8192 cells per workgroup, 16 per thread) 22 / 45.  Planes, FP64: 128^2 3.8 /
// 12.1, 256^2 4.9 / 13.3, 512^2 6.4 / 24.2, 1024^2 9.1 / 64.
// FP64 with 16 cells per thread (112^3, 128^3): 31.3 / 46.9, 35.6 / 51.4; half of it is what
// goes past the L2 (the iterate, 33 MB an iteration, and the halo, 44 MB, at about 4.5 TB/s),
// and 26 registers are in scratch memory.  Planes above 1024^2 are not tried; smaller grids are
// levels solved directly.
bool resident_plan(int n, int dim, bool fp64, ResidentPlan &plan) {
    plan.us = 1e30;
    for_plans(n, dim, fp64, false, [&](const ResidentPlan &p) {
        if (p.us < plan.us) plan = p;
    });
    return plan.blocks > 0;
}

void resident_batch_plans(int n, bool fp64, ResidentPlan (&plans)[kBatchShares]) {
    for (ResidentPlan &p : plans) p = ResidentPlan{};
    for_plans(n, 3, fp64, true, [&](const ResidentPlan &p) {
        for (int k = 0; k < kBatchShares; k++)
            if (p.blocks <= batch_share(k) && (plans[k].blocks == 0 || p.us < plans[k].us)) plans[k] = p;
    });
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

// ------------------------------------------------------------------ several runs

namespace {

// The table of runs is read through the scalar cache, where it is needed: a run's parameters
// held in registers for the whole run would cost the large partitions spills.
#define EXCMG_CONSTANT __attribute__((address_space(4)))
struct ResidentShared {
    Pair red[2 * (512 / kWave)];
    Pair all_a[4], all_b[8];
    int bad;
};
template <typename T, int C, int RS>
__device__ __forceinline__ void batch_run(const EXCMG_CONSTANT ResidentRun<T> &a, const int blk, const int W,
                                          const int nt, ResidentShared &sh, T *M) {
    constexpr int DIM = 3, NH = halo_slots(C, 3);
    constexpr bool MULTI = true, BATCH = true;
    Pair *red = sh.red, *all_a = sh.all_a, *all_b = sh.all_b;
    int &bad = sh.bad;
#include "resident_body.hpp"
}

// Several runs at once, each on its own workgroups, FP64 and FP32 ones together.  A run that
// stops says so in a.stop; the others then leave between two iterations (not before min_steps),
// with their state in memory, so that the host can start what comes next on the free CUs.
// The waves that a run's partition has no work for end here (a barrier waits for the
// workgroup's remaining waves only).  24 problems of 32^3 to 128^3 in mixed precision: 775 ms
// by steps of four launches (20 us a step at the least), 312 ms resident, of which 223 in 91
// launches; one after the other with launches of their own they take 376 ms.  In FP64 830 by
// steps, 358 resident (480 with the 128^3 systems by steps).  All kinds in one kernel, which has
// 42 registers in scratch memory (168 bytes a lane; the FP64 kernel with 16 cells alone 26).
__global__ void __launch_bounds__(512) k_resident_batch(const ResidentBatchRun *table, int count) {
    extern __shared__ char lds_raw[];
    __shared__ ResidentShared sh;
    const auto *runs = (const EXCMG_CONSTANT ResidentBatchRun *)table;
    int j = 0;
    while (j + 1 < count && (int)blockIdx.x >= runs[j + 1].first) j++;
    const EXCMG_CONSTANT ResidentBatchRun &b = runs[j];
    const int blk = (int)blockIdx.x - b.first, W = b.blocks, nt = b.threads;
    const int kind = b.kind;
    if ((int)threadIdx.x >= nt) return;
#define EXCMG_BATCH_RUN(T, C, RS)                                                              \
    case batch_kind(sizeof(T) == 8, C, RS):                                                    \
        batch_run<T, C, RS>((const EXCMG_CONSTANT ResidentRun<T> &)b.run, blk, W, nt, sh,     \
                            (T *)lds_raw);                                                     \
        break;
    switch (kind) {
        EXCMG_BATCH_RUN(double, 1, 20)
        EXCMG_BATCH_RUN(double, 1, 36)
        EXCMG_BATCH_RUN(double, 2, 20)
        EXCMG_BATCH_RUN(double, 2, 36)
        EXCMG_BATCH_RUN(double, 4, 20)
        EXCMG_BATCH_RUN(double, 4, 36)
        EXCMG_BATCH_RUN(double, 8, 20)
        EXCMG_BATCH_RUN(double, 8, 36)
        EXCMG_BATCH_RUN(double, 16, 20)
        EXCMG_BATCH_RUN(double, 16, 36)
        EXCMG_BATCH_RUN(float, 4, 20)
        EXCMG_BATCH_RUN(float, 4, 36)
        EXCMG_BATCH_RUN(float, 8, 20)
        EXCMG_BATCH_RUN(float, 8, 36)
        EXCMG_BATCH_RUN(float, 16, 20)
        EXCMG_BATCH_RUN(float, 16, 36)
    }
#undef EXCMG_BATCH_RUN
}

}  // namespace

hipError_t resident_batch(const ResidentBatchRun *runs, int count, int blocks, size_t lds, hipStream_t st) {
    const void *fn = (const void *)k_resident_batch;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    void *args[] = {&runs, &count};
    return hipLaunchCooperativeKernel(fn, dim3(blocks), dim3(512), args, (unsigned)lds, st);
}

}  // namespace excmg
