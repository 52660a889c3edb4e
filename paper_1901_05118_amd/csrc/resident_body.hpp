// The body of a resident run (resident.hip): brick `blk` of W, on nt threads, LDS box M.
// DIM, T; C: consecutive z-cells per thread; RS: row stride of the box; NH: halo cells per
// thread; MULTI: more than one brick; BATCH: one of several runs of a launch, which may be
// halted between two iterations.  Included where it is compiled: called as a function, the
// kernel with 16 cells per thread needs 11 more registers than there are.
    // FP64 with 16 cells per thread: what does not fit is left out of the registers.  The
    // iterate is in memory; q* is not kept (alpha is waited for before it is formed, and r* takes
    // it term by term); phases go through the cells G at a time; r and r* are sent in parts.
    constexpr bool kLean = sizeof(T) == 8 && C == 16;
    constexpr int G = kLean ? 4 : C;
    int tid = threadIdx.x;
    const int nw = nt >> 6;
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
    // Uniform: a run that starts makes at least one exchange, so the state is written (by the
    // first workgroup, at the end) only when every wave of the run has read it.
    if (status != kRunning) {
        if (BATCH && blk == 0 && tid == 0)
            __hip_atomic_store(a.stop, a.epoch + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }

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
    const int gplane = kLean || cells > 0 ? ny * n : 0;
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
    [[maybe_unused]] const __amdgpu_buffer_rsrc_t xw =
        exchange_rsrc(a.x_work, kLean ? 8u * (unsigned)(n * n * n) : 0u);
    const int own = bx * by * groups * C;     // staged r and r* of the brick: R, R + own
    T *R = M + LE + 1;
    int os = cells > 0 ? (lg * C * by + ly) * bx + lx : 0, oplane = bx * by;
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

    // own values c0 .. c0 + G - 1 into LDS, and into the fictitious points that mirror them
    const bool edge = ghx || ghy || ghz0 || ghz1;
    auto place = [&](const int c0, const T (&v)[G]) {
#pragma unroll
        for (int k = 0; k < G; k++) M[c0 + k < cells ? ob + (c0 + k) * PS : LE] = v[k];
        if (edge) {
            const bool neg = a.sgn < 0;
#pragma unroll
            for (int k = 0; k < G; k++) {
                const int c = c0 + k;
                if (c < cells) {
                    T *P = M + ob + c * PS;
                    const T g = neg ? -v[k] : v[k];
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
    if (!first) beta = S->beta;
    __syncthreads();

    // In the first iteration of a run p = r and p* = r*: the old directions are zeros and
    // beta is 0.
    T r[C], s[C], o[C];      // r, r*, and p while LDS holds p* (p* while it holds p)
    double xv[kLean ? 1 : C];   // the iterate
    {
        const T *p = a.p[iter & 1], *ps = a.ps[iter & 1];
#pragma unroll
        for (int c = 0; c < C; c++) {
            r[c] = s[c] = o[c] = (T)0;
            if (!kLean) xv[kLean ? 0 : c] = 0.0;
            if (c < cells) {
                const unsigned i = gi + c * gplane;
                r[c] = a.r[i];
                s[c] = a.rs[i];
                if (kLean) a.x_work[i] = a.x[i];
                else xv[kLean ? 0 : c] = a.x[i];
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
    unsigned ep = a.epoch, halted = 0;
    // Workgroups launched for one XCD tell each other where they are (past the L2s, in the
    // plane of rho', which is next written after an exchange that needs them all).
    bool l2 = false;
    if constexpr (MULTI && !BATCH && C <= 8) {
        if (a.one_xcd) {
            ep++;
            const unsigned xcd = xcd_id();
            if (tid < 64) {
                if (tid == 0) put<kAgent>(xs, 16u * (unsigned)blk, 2 * kSlotPlane, xcd, 0, ep);
                const bool same = gather_same(xs, tid < W ? 16u * (unsigned)tid : kNoPlace,
                                              2 * kSlotPlane, ep, xcd, a.wait, &bad);
                if (tid == 0) all_a[0].s = same ? 1.0 : 0.0;
            }
            __syncthreads();
            l2 = __builtin_amdgcn_readfirstlane(all_a[0].s != 0.0);
            __syncthreads();
            if (bad) status = kStopping;    // (no iteration; the host sees err)
        }
    }
    // Phases of an iteration are kept apart in the registers: addresses and FP64 forms of FP32
    // values that one phase derives are not carried into the next.
    auto keep = [&]() {
        asm volatile("" : "+v"(ob), "+v"(cells));
        if constexpr (kLean) asm volatile("" : "+v"(gi), "+v"(os), "+v"(tid));
        if constexpr (sizeof(T) == 4 || kLean) {
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

    // (lean) One of r and r* of the cells that others read, the threads of one z-group at a time.
    [[maybe_unused]] auto send = [&](const T (&v)[C], const unsigned box) {
        const int part = own / groups;
        for (int g = 0; g < groups; g++) {
            keep();
            if (lg == g && cells > 0) {    // (cells past the grid have their place, too)
                T *to = R + (os - g * part);
#pragma unroll
                for (int c = 0; c < C; c++) to[c * oplane] = v[c];
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NH; q++) {
                const int src = (int)((unsigned)hplace[q] >> 16) - g * part;
                const bool here = hdest[q] != kNoCell && src >= 0 && src < part;
                put_value(xc, here ? box + hdest[q] : kNoCell, R[here ? src : 0]);
            }
            __syncthreads();
        }
    };

    while (status == kRunning) {
        ep++;
        asm volatile("" : "+v"(tid));
        // (batch) the first workgroup of a run looks whether the launch is to end
        unsigned ended = 0;
        if (BATCH && blk == 0)
            ended = __hip_atomic_load(a.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int lane = tid & 63, wave = tid >> 6;
        keep();
        // ---- directions: p into LDS, p* into o and hv
        T ho[MULTI ? NH : 1];
        if constexpr (kLean) {
#pragma unroll
            for (int q = 0; q < NH; q++) {
                const T h = M[hoff(q)];
                M[hoff(q)] = (T)((double)hr[q] + beta * (double)hv[q]);
                hv[q] = (T)((double)hs[q] + beta * (double)h);
            }
            keep();
        }
#pragma unroll
        for (int c0 = 0; c0 < C; c0 += G) {
            T pn[G], so[G];
#pragma unroll
            for (int k = 0; k < G; k++) so[k] = M[ob + (c0 + k) * PS];
            if (MULTI && !kLean) {
#pragma unroll
                for (int q = 0; q < NH; q++) ho[q] = M[hoff(q)];
            }
#pragma unroll
            for (int k = 0; k < G; k++) {
                const int c = c0 + k;
                pn[k] = (T)((double)r[c] + beta * (double)o[c]);
                o[c] = (T)((double)s[c] + beta * (c < cells ? (double)so[k] : 0.0));
            }
            place(c0, pn);
            if (kLean) keep();
        }
        if (MULTI && !kLean) {
#pragma unroll
            for (int q = 0; q < NH; q++)
                M[hoff(q)] = (T)((double)hr[q] + beta * (double)hv[q]);
#pragma unroll
            for (int q = 0; q < NH; q++) hv[q] = (T)((double)hs[q] + beta * (double)ho[q]);
        }
        __syncthreads();
        keep();

        // ---- q = A p, sigma = p*.q
        T qv[C], qs[kLean ? 1 : C];
        Pair sg[1] = {{0.0, 0.0}};
        stencil([&](int c, double y) {
            qv[c] = c < cells ? (T)y : (T)0;
            dot2_acc(sg[0], (double)o[c], (double)qv[c]);
            // (one output after the other)
            if (C >= 8) asm volatile("" : "+v"(sg[0].s), "+v"(sg[0].c), "+v"(qv[c]));
            if (kLean) asm volatile("" ::: "memory");
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
                    const unsigned at = 16u * (unsigned)blk + lane * kSlotPlane;
                    if (l2) put<0>(xs, at, 0, low(b), high(b), ep);
                    else put<kAgent>(xs, at, 0, low(b), high(b), ep);
                }
            } else if (lane == 0) {
                all_a[0] = v[0];
            }
        }
        // ---- p* into LDS, p into o and hv; q* = A^T p*
        keep();
#pragma unroll
        for (int c0 = 0; c0 < C; c0 += G) {
            T pv[G], po[G];
#pragma unroll
            for (int k = 0; k < G; k++) pv[k] = M[ob + (c0 + k) * PS];
            if (MULTI && c0 == 0) {
#pragma unroll
                for (int q = 0; q < NH; q++) ho[q] = M[hoff(q)];
            }
#pragma unroll
            for (int k = 0; k < G; k++) po[k] = o[c0 + k];
            place(c0, po);
#pragma unroll
            for (int k = 0; k < G; k++) o[c0 + k] = c0 + k < cells ? pv[k] : (T)0;
            if (MULTI && c0 == 0) {
#pragma unroll
                for (int q = 0; q < NH; q++) {
                    M[hoff(q)] = hv[q];
                    hv[q] = ho[q];
                }
            }
            if (kLean) keep();
        }
        __syncthreads();
        keep();
        if constexpr (!kLean) {
            stencil([&](int c, double y) {
                qs[c] = c < cells ? (T)y : (T)0;
                if (C >= 8) asm volatile("" : "+v"(qs[c]));
            });
            // (q* is formed here, before the wait, not carried over it as its 21 C terms)
#pragma unroll
            for (int c = 0; c < C; c++) asm volatile("" : "+v"(qs[c]));
        }

        // ---- sigma and alpha
        if (MULTI) {
            if (64 * wave < W) {
                const Pair v = gather_pairs(xs, tid < W ? 16u * (unsigned)tid : kNoPlace, 0, ep, a.wait,
                                            &bad);
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
        if constexpr (kLean) {
#pragma unroll
            for (int c = 0; c < C; c++) {
                r[c] = (T)((double)r[c] - alpha * (double)qv[c]);
                asm volatile("" : "+v"(r[c]));
            }
            send(r, 0u);
            stencil([&](int c, double y) {
                s[c] = (T)((double)s[c] - alpha * (c < cells ? y : 0.0));
                asm volatile("" : "+v"(s[c]) :: "memory");
            });
            send(s, (unsigned)(W * hn));
        } else {
#pragma unroll
            for (int c = 0; c < C; c++) {
                r[c] = (T)((double)r[c] - alpha * (double)qv[c]);
                s[c] = (T)((double)s[c] - alpha * (double)qs[kLean ? 0 : c]);
                if (MULTI && c < cells) {
                    R[os + c * oplane] = r[c];
                    R[own + os + c * oplane] = s[c];
                }
            }
        }
        if (MULTI && !kLean) {
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NH; q++) {
                const int src = (unsigned)hplace[q] >> 16;
                if (l2) put_cell<0>(xc, hdest[q], R[src], R[own + src]);
                else put_cell<kAgent>(xc, hdest[q], R[src], R[own + src]);
            }
        }
        keep();
#pragma unroll
        for (int c = 0; c < C; c++) {
            dot2_acc(dt[0], (double)s[c], (double)r[c]);
            dot2_acc(dt[1], (double)r[c], (double)r[c]);
            if (!kLean) xv[kLean ? 0 : c] = xv[kLean ? 0 : c] + alpha * (double)o[c];
        }
        wave_merge_n<2>(dt);
        if (lane == 0) {
            red[2 * wave] = dt[0];
            red[2 * wave + 1] = dt[1];
        }
        if (BATCH && blk == 0 && tid == 0 &&
            ((ended == a.epoch + 1 && ep - a.epoch >= a.min_steps) || ep - a.epoch >= a.max_steps))
            __hip_atomic_store(a.halt, ep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
                    const unsigned at = 16u * (unsigned)blk + (2 + lane) * kSlotPlane;
                    if (l2) put<0>(xs, at, 0, low(b), high(b), ep);
                    else put<kAgent>(xs, at, 0, low(b), high(b), ep);
                }
            } else if (lane == 0) {
                all_b[0] = v[0];
                all_b[1] = v[1];
            }
        }
        // (while the partials travel)
        if constexpr (kLean) {
            constexpr int GX = 8;
#pragma unroll
            for (int c0 = 0; c0 < C; c0 += GX) {
                double xv[GX];
                unsigned at[GX];
#pragma unroll
                for (int k = 0; k < GX; k++) {
                    at[k] = c0 + k < cells ? (unsigned)(gi + (c0 + k) * gplane) : kNoCell;
                    xv[k] = load_f64(xw, at[k]);
                }
#pragma unroll
                for (int k = 0; k < GX; k++) store_f64(xw, at[k], xv[k] + alpha * (double)o[c0 + k]);
                asm volatile("" ::: "memory");
            }
        }
        if (MULTI) {
            // A load takes about 1800 cycles (past the L2); asked too early it is asked twice.
            for (int k = a.look; k > 0; k--) __builtin_amdgcn_s_sleep(4);
            if (64 * (wave >> 1) < W) {     // even waves: rho', odd waves: r.r
                const int w = (wave >> 1) * 64 + lane;
                const Pair v = gather_pairs(xs, w < W ? 16u * (unsigned)w : kNoPlace,
                                            (2 + 2 * (wave & 1)) * kSlotPlane, ep, a.wait, &bad);
                if (lane == 0) all_b[wave] = v;
            }
            __syncthreads();
            // all partials are here, so all cells are: r and r* of the halo (a cell of the box
            // that the grid does not have reads as anything and goes nowhere)
            unsigned cell = (unsigned)(blk * hn + tid);
#pragma unroll
            for (int q = 0; q < NH; q++, cell += nt) {
                if constexpr (kLean) {
                    hr[q] = get_value(xc, cell);
                    hs[q] = get_value(xc, (unsigned)(W * hn) + cell);
                } else {
                    get_cell(xc, cell, hr[q], hs[q]);
                }
            }
            if (BATCH) halted = __hip_atomic_load(a.halt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
        // (halt: written before the partials of this iteration were sent, so every workgroup of
        // the run reads the same, and not overwritten before all have sent their next sigma)
        if (BATCH ? halted == ep : ep - a.epoch >= a.max_steps) break;
    }
    if (MULTI && bad) {
        if (tid == 0) atomicExch(&S->err, 1);
        return;
    }
    // the iterate, the directions for a run that goes on after its residuals are replaced, and
    // all of the state of a run that is halted
    {
        T *p = BATCH ? a.p[iter & 1] : a.p_out, *ps = BATCH ? a.ps[iter & 1] : a.ps_out;
        T *r_out = BATCH ? a.r : a.r_out, *rs_out = BATCH ? a.rs : a.rs_out;
#pragma unroll
        for (int c = 0; c < C; c++) {
            if (c < cells) {
                const unsigned i = gi + c * gplane;
                if (!kLean) a.x_work[i] = xv[kLean ? 0 : c];
                p[i] = o[c];
                ps[i] = M[ob + c * PS];
                if (status == kRunning) {
                    r_out[i] = r[c];
                    rs_out[i] = s[c];
                }
            }
        }
    }
    if (blk == 0 && tid == 0) {
        if (BATCH && status != kRunning)
            __hip_atomic_store(a.stop, a.epoch + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        S->rr = rr;
        S->rho = rho;
        S->rho_slot[iter & 1] = rho;
        S->rho_slot[(iter & 1) ^ 1] = rho_old;
        if (BATCH) S->rho_slot[1] = rho_old;    // (where batch_resume looks)
        S->alpha = alpha;
        S->beta = beta;
        S->sigma = sigma;
        S->iter = iter;
        S->status = status;
        S->poll_status = status;
    }
