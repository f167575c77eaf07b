// Resident lanes: the solves of a lane whose grid fits the registers and the
// LDS of its group. Included by pt_engine.hip; it uses the engine's flags,
// step descriptions and barrier.
//
// A solve is a conjugate gradient in the single-reduction form of Chronopoulos
// and Gear with a polynomial preconditioner: u = q(D^{-1}A) D^{-1} r, the result
// of d + 1 Richardson sweeps z += omega_i D^{-1} (r - A z) from z = 0 whose
// omega_i are the inverse roots of the Chebyshev polynomial of degree d + 1 on
// an interval inside the spectrum's bounds (res_omegas). A round of a group is
// bound by latency, not by arithmetic: the barrier, the partial sums and the
// halo each cost a trip through the memory side of the chip, about 4 us
// together, while one application of the operator to a tile costs about half a
// microsecond. d further applications per round cut the rounds of a solve by
// nearly d + 1.
//
// The applications need no exchange: each workgroup owns a rectangle of
// tw x th nodes and carries r and s on a window of d + 1 rings of nodes around
// it, updated with the same arithmetic as their owner's; every application
// leaves one ring less of the window valid and the last one exactly the owned
// nodes. Only w = A u crosses workgroups, d + 1 rings deep, once per round.
// Rectangles keep those rings short: with full grid rows as tiles a 64-workgroup
// sweep at 257 x 257 nodes would apply the operator to 28 rows per 4 owned ones,
// on 33 x 33 squares it is 4.8 times the owned nodes.
//
// On chip: a thread holds NR consecutive rows of one window column. The
// operator's coefficients at its nodes (east, west, north, the diagonals), r, s
// and D^{-1} are registers for the whole lane; p and x, used once a round, are
// LDS slots of their own thread; the operand z is the only LDS array that
// threads share, in two buffers, so an application costs one synchronisation
// and 3 + 6/NR LDS reads per node instead of 17 (nine operands, eight element
// values) when the coefficients are formed anew. Six rows are the most that
// leave the rounds without spills: with eight, reloads behind the published
// stores in flight made a round 17.6 us instead of 11.0.
//
// Two rounds less per step: the round that checks the true residual of a
// finished solve also sets up the next one (right-hand side, initial residual,
// first preconditioned direction), with all sums in one reduction. And a fine
// step starts from the extrapolation of the slice's states, whose residual is a
// higher difference of them in time; the plain start's residual, formed beside
// it, lowers the order where the states are not smooth.
//
// Measured at 256^2, 512 steps in 32 slices, cg_rtol 1e-12, one warm cycle,
// against Jacobi CG on full-row tiles with one halo row: 94 -> 31.5 ms; CG
// rounds per fine step 42 -> 8 (degree 3, extrapolated), per coarse step 169 ->
// 36 (degree 4); sequential 100^2 with 480 steps: 741 -> 131 ms.

namespace pt {

namespace {

constexpr int kResMaxDeg = 6;       // degree of the preconditioner's polynomial
constexpr int kResRows = 6;         // most rows of a window column per thread
constexpr int kResSums = 8;         // sums per reduction, at most
constexpr int kResGroup = kMaxGroup / 2;  // workgroups per resident group, at most

// Sum over the 64 lanes of a wave, in every lane, in a fixed order: within rows
// of 16 lanes by data-parallel moves, then the four row sums.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
    const long long v = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double read_lane(double x, int l) {
    const long long v = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)v, l);
    const int hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wave_sum(double x) {
    x += dpp_move<0xB1>(x);   // quad_perm: neighbours
    x += dpp_move<0x4E>(x);   // quad_perm: pairs
    x += dpp_move<0x141>(x);  // row_half_mirror: quads
    x += dpp_move<0x140>(x);  // row_mirror: halves of a row
    return (read_lane(x, 0) + read_lane(x, 16)) + (read_lane(x, 32) + read_lane(x, 48));
}

// Bounds of the eigenvalues of D^{-1}A, D the diagonal of A = C/delta + K, from
// those of the element matrices: A and D are sums over elements, so every
// quotient x^T A x / x^T D x lies between the smallest and the largest element
// quotient, and dropping the fixed nodes can only narrow the range. An element
// matrix of mass m = c hx hy/(36 delta) and stiffness k/6 has the eigenvectors
// (constant, x, y, xy) with 9m, 3m + k ex', 3m + k ey', m + k exy' over the
// diagonal 4m + k e_self; each quotient is monotone in k/m.
__device__ __forceinline__ void res_bounds(const Consts &C, double kmin_m, double kmax_m,
                                           double &lo, double &hi) {
    lo = 1e300;
    hi = 0.0;
    const double ms[4] = {9.0, 3.0, 3.0, 1.0};
    const double ks[4] = {0.0, C.e_self - C.e_x + C.e_y - C.e_d,
                          C.e_self + C.e_x - C.e_y - C.e_d, C.e_self - C.e_x - C.e_y + C.e_d};
    for (int e = 0; e < 2; ++e) {
        const double q = e ? kmax_m : kmin_m;
        for (int k = 0; k < 4; ++k) {
            const double v = (ms[k] + q * ks[k]) / (4.0 + q * C.e_self);
            lo = fmin(lo, v);
            hi = fmax(hi, v);
        }
    }
}

// The inverse roots of the Chebyshev polynomial of degree deg + 1 on [a, hi].
// The preconditioned operator's eigenvalues are 1 - T(l)/T(0): positive for
// every l in (0, hi], so CG stays CG whatever a is. The element bound lo lies
// a factor 2 to 6 below the smallest eigenvalue of the fields measured; a
// polynomial of low degree does better with an interval that leaves the lowest
// modes to CG (256^2, degree 3: 13 rounds per fine step at a = hi/16 against 18
// on [lo, hi]; 52 per coarse step at hi/60 against 74).
__device__ __forceinline__ double res_omega(double lo, double hi, int deg, int i) {
    if (deg == 0) return 1.0;
    const double n = deg + 1;
    const double a = fmax(2.0 * lo, hi / (4.0 * n * n));
    // largest and smallest roots in turn, so that no partial product grows
    const int k = (i & 1) ? deg - (i >> 1) : (i >> 1);
    return 1.0 / (0.5 * (hi + a) + 0.5 * (hi - a) * cospi((2 * k + 1) / (2.0 * n)));
}

// Node n of a row of values, as a global-memory access: a resident grid has far
// fewer than 2^29 nodes, so the byte offset fits 32 bits and the access needs one
// offset register beside a scalar base. (64-bit addresses per node were hoisted
// out of the rounds and filled the scratch; pointers read from a descriptor in
// memory would be generic ones.)
typedef __attribute__((address_space(1))) double gdouble;
typedef __attribute__((address_space(1))) char gchar;
__device__ __forceinline__ gdouble *nd(const double *p, unsigned n) {
    return (gdouble *)((gchar *)p + n * 8u);
}
__device__ __forceinline__ double ldg(const double *p, unsigned n) {
    return __hip_atomic_load(nd(p, n), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stg(const double *p, unsigned n, double v) {
    __hip_atomic_store(nd(p, n), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A value the compiler forms again at each use instead of keeping it, and all
// that follows from it, in registers from outside the loops.
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
// A part of the descriptor, read anew where it is needed by scalar loads (the
// descriptor does not change during a launch): what a rare phase reads of it is
// not held in scalar registers, and spilled, throughout the rounds. The copy's
// unused members are never loaded.
typedef __attribute__((address_space(4))) const unsigned long long cword;
template <typename T>
__device__ __forceinline__ T fetch(const T *p) {
    static_assert(sizeof(T) % 8 == 0, "whole words");
    asm volatile("" : "+s"(p));
    unsigned long long raw[sizeof(T) / 8];
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 8); ++k) raw[k] = ((cword *)p)[k];
    T out;
    __builtin_memcpy(&out, raw, sizeof(T));
    return out;
}

template <int NR>
struct ResCoef {
    double er[NR], el[NR];                        // east, west neighbour
    double nn[NR + 1], dl[NR + 1], dr[NR + 1];    // per gap below row k: straight, left, right
};

// r - (A - D) z at the thread's NR nodes, z an LDS window with rows of sz
// values, `cell` the LDS index of the row below the first node (an index, not a
// pointer chosen between buffers: that would make every access a generic one).
template <int NR>
__device__ __forceinline__ void res_apply(const ResCoef<NR> &A, int cell, int sz,
                                          const double (&r)[NR], double (&zc)[NR],
                                          double (&t)[NR]) {
    extern __shared__ double lds[];
    const double *q = lds + cell;
    double l0 = q[-1], c0 = q[0], r0 = q[1];
    q += sz;
    double l1 = q[-1], c1 = q[0], r1 = q[1];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        q += sz;
        const double l2 = q[-1], c2 = q[0], r2 = q[1];
        double v = r[k];
        v = fma(-A.dl[k], l0, v);
        v = fma(-A.nn[k], c0, v);
        v = fma(-A.dr[k], r0, v);
        v = fma(-A.el[k], l1, v);
        v = fma(-A.er[k], r1, v);
        v = fma(-A.dl[k + 1], l2, v);
        v = fma(-A.nn[k + 1], c2, v);
        v = fma(-A.dr[k + 1], r2, v);
        t[k] = v;
        zc[k] = c1;
        l0 = l1;
        c0 = c1;
        r0 = r1;
        l1 = l2;
        c1 = c2;
        r1 = r2;
    }
}

struct ResTimers {
    unsigned long long work = 0, bar = 0, red = 0, flag = 0;
    long long mark = 0;
};

// Runs lane L of design *Dp on this workgroup's group (rank of g workgroups);
// returns false when a wait timed out or another workgroup aborted, alike in
// every workgroup.
template <int NR, bool TIMED, bool SPLIT>
__device__ __forceinline__ bool res_lane(const EngineDesc *Dp, const Lane L, const Launch &S,
                                         const Group &G, unsigned *bar, double *part,
                                         unsigned &nbar, unsigned long long *trec, double *red) {
    extern __shared__ double lds[];
    __shared__ double om_s[kResMaxDeg + 1];
    __shared__ double tot_s[kResSums];
    const int rank = blockIdx.x - G.wg0, g = G.nwg;
    const int tid = threadIdx.x;
    const bool leader = rank == 0 && tid == 0;
    const bool is_adj = is_adjoint_kind(L.kind);
    const bool sweep = L.kind == SWEEP_PRI || L.kind == SWEEP_ADJ;
    const bool fine = L.kind == F_PRI || L.kind == F_ADJ;
    const Consts C0 = fetch(&Dp->C);
    const Bufs B0 = fetch(&Dp->B);
    Control *ctl = B0.ctl;
    const long long tmo = C0.timeout_ticks;
    const int W = C0.W, HN = C0.ny + 1;
    const double rtol = C0.rtol;
    const int max_iter = C0.max_iter;
    const int coarse_iters = fine ? 0 : C0.coarse_iters;
    const bool trunc = coarse_iters > 0;
    const int deg = trunc ? 0 : L.deg;
    // group vectors by consecutive pool slots, so that a choice between them is
    // arithmetic on one base: w by round parity; right-hand sides of the solve
    // being finished and of the next one (each value read by its writer only);
    // the last four solutions
    const double *gv0 = group_vec(B0, G.vec, V_R0);
    const size_t gvs = B0.pool_stride;
    auto wv = [&](unsigned par) { return gv0 + (size_t)(V_W0 - V_R0 + (par & 1)) * gvs; };
    auto bvec = [&](int j) { return gv0 + (size_t)(j & 1) * gvs; };
    auto xh = [&](int j) { return gv0 + (size_t)(V_S0 - V_R0 + (j & 3)) * gvs; };

    // geometry: owned rectangle, window, this thread's column and rows
    const int TX = (W + L.tw - 1) / L.tw, TY = (HN + L.th - 1) / L.th;
    const int hx = TX > 1 ? deg + 1 : 0, hy = TY > 1 ? deg + 1 : 0;
    const int wc = L.tw + 2 * hx, wr = L.th + 2 * hy;
    const int nq = min(kThreads / wc, (wr + NR - 1) / NR);
    const int sz = wc + 2, rows = nq * NR;
    const int zlen = sz * (rows + 2);   // doubles per operand window
    double *LP = lds + 2 * zlen + tid;  // thread's p, then x
    double *LX = LP + NR * kThreads;
    const int q = tid / wc;
    const bool act = q < nq;
    const int col = act ? tid - q * wc : 0, row0 = act ? q * NR : 0;
    const int cell0 = row0 * sz + col + 1;  // cell of the row below the first node
    int gx, gy0;                            // the first node
    // node sets as bits per row: live (in the grid, the window and not fixed),
    // fill (the same with one row more above the window), own, nodes that a
    // neighbour's window (edge) or set-up window (edge1: one ring more) holds
    unsigned live = 0, fill = 0, own = 0, edge = 0, edge1 = 0;
    // cells around the window that no thread's rows cover: node (-1: none), cell
    constexpr int kRim = 2;
    int rim_id[kRim], rim_cell[kRim];
    ResCoef<NR> A;
    double dinv[NR], cc[NR], r[NR], s[NR], w[NR];
    {
        const Consts C = fetch(&Dp->C);
        const Bufs B = fetch(&Dp->B);
        const int tx = rank % TX, ty = rank / TX;  // ty >= TY: nothing owned
        const int ox0 = tx * L.tw, oy0 = ty * L.th;
        const int ox1 = min(ox0 + L.tw, W), oy1 = min(oy0 + L.th, HN);
        gx = ox0 - hx + col;
        gy0 = oy0 - hy + row0;
        const bool inx = act && gx >= 0 && gx < W && ty < TY;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int y = gy0 + k, row = row0 + k;
            if (!inx || y < 0 || y >= HN || row > wr) continue;
            const bool free_ = B.mask[(size_t)y * W + gx] == 0;
            if (free_) fill |= 1u << k;
            if (row >= wr) continue;
            if (free_) live |= 1u << k;
            if (gx >= ox0 && gx < ox1 && y >= oy0 && y < oy1) {
                own |= 1u << k;
                auto near = [&](int h) {
                    return (tx > 0 && gx - ox0 < h) || (tx < TX - 1 && ox1 - gx <= h) ||
                           (ty > 0 && y - oy0 < h) || (ty < TY - 1 && oy1 - y <= h);
                };
                if (near(deg + 1)) edge |= 1u << k;
                if (near(deg + 2)) edge1 |= 1u << k;
            }
        }
#pragma unroll
        for (int i = 0; i < kRim; ++i) {
            const int e = tid + i * kThreads;
            int cx, cy;
            if (e < 2 * sz) {
                cx = e < sz ? e : e - sz;
                cy = e < sz ? 0 : rows + 1;
            } else {
                cx = (e & 1) ? sz - 1 : 0;
                cy = 1 + ((e - 2 * sz) >> 1);
            }
            const int x = ox0 - hx - 1 + cx, y = oy0 - hy - 1 + cy;
            const bool in = e < 2 * sz + 2 * rows && x >= 0 && x < W && y >= 0 && y < HN &&
                            cy <= wr + 1 && ty < TY;
            const int id = in ? y * W + x : -1;
            rim_id[i] = in && B.mask[id] == 0 ? id : -1;
            rim_cell[i] = cy * sz + cx;
        }
        // coefficients: gap k lies below row k, its elements left and right of the
        // column are (gx - 1, gy0 + k - 1) and (gx, gy0 + k - 1)
        const double ms = fine ? C.inv_dt : C.inv_dtau;
        double sl = 0.0, sr = 0.0, xl = 0.0, xr = 0.0;
#pragma unroll
        for (int k = 0; k <= NR; ++k) {
            const int ey = gy0 + k;  // padded element row
            const bool in = inx && ey >= 0 && ey <= C.ny + 1;
            const unsigned e = in ? (unsigned)(ey * C.EW + gx) : 0u;
            const double ml = in ? *nd(B.cm, e) * ms : 0.0, mr = in ? *nd(B.cm, e + 1) * ms : 0.0;
            const double kl = in ? *nd(B.kq, e) : 0.0, kr = in ? *nd(B.kq, e + 1) : 0.0;
            A.dl[k] = ml + C.e_d * kl;
            A.dr[k] = mr + C.e_d * kr;
            A.nn[k] = 2.0 * (ml + mr) + C.e_y * (kl + kr);
            const double nsl = 4.0 * ml + C.e_self * kl, nsr = 4.0 * mr + C.e_self * kr;
            const double nxl = 2.0 * ml + C.e_x * kl, nxr = 2.0 * mr + C.e_x * kr;
            if (k > 0) {
                A.el[k - 1] = xl + nxl;
                A.er[k - 1] = xr + nxr;
                cc[k - 1] = (sl + sr) + (nsl + nsr);
            }
            sl = nsl;
            sr = nsr;
            xl = nxl;
            xr = nxr;
        }
        const double *dinv_g = fine ? B.dinv_f : B.dinv_c;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const unsigned id = (live >> k) & 1u ? (unsigned)((gy0 + k) * W + gx) : 0u;
            const double v = *nd(dinv_g, id);
            dinv[k] = (live >> k) & 1u ? v : 0.0;
            r[k] = s[k] = w[k] = 0.0;
        }
        double lo, hi;
        res_bounds(C, __longlong_as_double((long long)ctl->kmin_bits) / ms,
                   __longlong_as_double((long long)ctl->kmax_bits) / ms, lo, hi);
        lds_sync();
        if (tid <= deg) om_s[tid] = res_omega(lo, hi, deg, tid);
        // both operand windows: every cell outside the grid stays 0
        for (int c = tid; c < 2 * zlen; c += kThreads) lds[c] = 0.0;
#pragma unroll
        for (int k = 0; k < 2 * NR; ++k) LP[k * kThreads] = 0.0;
        lds_sync();
    }
    const int n0 = gy0 * W + gx;
    auto id_of = [&](int k) { return (unsigned)(fresh(n0) + k * W); };
    auto is = [](unsigned m, int k) { return (((unsigned)fresh((int)m) >> k) & 1u) != 0; };

    ResTimers tm;
    if constexpr (TIMED) tm.mark = now_ticks();
    auto barrier = [&](bool release) -> bool {
        ++nbar;
        long long t0 = 0;
        if constexpr (TIMED) t0 = now_ticks();
        const bool ok = group_barrier<SPLIT>(bar, (unsigned)g, nbar * (unsigned)g, ctl, tmo,
                                             release);
        if constexpr (TIMED) {
            const long long t1 = now_ticks();
            tm.work += t0 - tm.mark;
            tm.bar += t1 - t0;
            tm.mark = t1;
        }
        return ok;
    };
    auto waitf = [&](int idx) -> bool {
        long long t0 = 0;
        if constexpr (TIMED) t0 = now_ticks();
        const Bufs B = fetch(&Dp->B);
        const LaunchInfo I = fetch(&Dp->I);
        const bool ok = wait_flag(B.flags, idx, I.epoch, ctl, tmo);
        if constexpr (TIMED) {
            const long long t1 = now_ticks();
            tm.work += t0 - tm.mark;
            tm.flag += t1 - t0;
            tm.mark = t1;
        }
        return ok;
    };
    // this workgroup's Q sums to its partial slots of the coming barrier
    auto put_sums = [&](auto &v) {
        constexpr int Q = sizeof(v) / sizeof(double);
        const int t = fresh(tid), wave = t >> 6;
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const double x = wave_sum(v[k]);
            if ((t & 63) == 0) red[k * kWaves + wave] = x;
        }
        lds_sync();
        if (t < Q) {
            double x = 0.0;
#pragma unroll
            for (int k = 0; k < kWaves; ++k) x += red[t * kWaves + k];
            stc(part + ((size_t)(nbar & 1) * kResSums + t) * kResGroup + rank, x);
        }
    };
    // the group's sums after the barrier: wave k adds component k
    auto get_sums = [&](auto &v) {
        constexpr int Q = sizeof(v) / sizeof(double);
        const int t = fresh(tid), wave = t >> 6, ln = t & 63;
        if (wave < Q) {
            const double *p = part + ((size_t)((nbar - 1) & 1) * kResSums + wave) * kResGroup;
            double x = 0.0;
            for (int k = ln; k < g; k += 64) x += ldc(p + k);
            x = wave_sum(x);
            if (ln == 0) tot_s[wave] = x;
        }
        lds_sync();
#pragma unroll
        for (int k = 0; k < Q; ++k) v[k] = read_lane(tot_s[k], 0);
        if constexpr (TIMED) {
            const long long t1 = now_ticks();
            tm.red += t1 - tm.mark;
            tm.mark = t1;
        }
    };
    // A row of global values at the thread's nodes in m, all loads in flight at
    // once: no load is conditional (the other nodes read node 0), since a masked
    // load whose value is used in its own branch waits for it there, node by node.
    auto load = [&](const double *row, unsigned m, double (&v)[NR]) {
#pragma unroll
        for (int k = 0; k < NR; ++k) v[k] = ldg(row, is(m, k) ? id_of(k) : 0u);
    };
    auto load_rim = [&](const double *row, double (&v)[kRim]) {
#pragma unroll
        for (int i = 0; i < kRim; ++i) v[i] = ldg(row, rim_id[i] >= 0 ? (unsigned)rim_id[i] : 0u);
    };
    // the operand window at LDS index zb
    auto put_win = [&](int zb, const double (&v)[NR], const double (&vr)[kRim]) {
        if (act) {
#pragma unroll
            for (int k = 0; k < NR; ++k) lds[zb + cell0 + (k + 1) * sz] = is(fill, k) ? v[k] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < kRim; ++i)
            if (rim_id[i] >= 0) lds[zb + rim_cell[i]] = vr[i];
    };
    auto store = [&](const double *row, unsigned m, const double (&v)[NR]) {
#pragma unroll
        for (int k = 0; k < NR; ++k)
            if (is(m, k)) *nd(row, id_of(k)) = v[k];
    };
    // x of the finished solve on the window (and its rim): own values from the
    // thread's slots, the others as their owners published them
    auto load_x = [&](const double *xp, double (&v)[NR], double (&vr)[kRim]) {
        load(xp, fill & ~own, v);
        load_rim(xp, vr);
#pragma unroll
        for (int k = 0; k < NR; ++k) v[k] = is(own, k) ? LX[k * kThreads] : v[k];
    };
    // u = q(D^{-1}A) D^{-1} r; leaves u in operand window zc_buf, w = A u in w
    // and adds (r, u) and (u, w) of the owned nodes
    int zc_buf = 0;
    auto precond = [&](double &gam, double &del) {
        double zc[NR], t[NR];
        const double om0 = om_s[0];
        int b = zc_buf ^ 1;
        if (act) {
#pragma unroll
            for (int k = 0; k < NR; ++k)
                lds[b * zlen + cell0 + (k + 1) * sz] = om0 * dinv[k] * r[k];
        }
        lds_sync();
        for (int i = 1; i <= deg; ++i) {
            const double om = om_s[i];
            res_apply<NR>(A, b * zlen + cell0, sz, r, zc, t);
            b ^= 1;
            if (act) {
#pragma unroll
                for (int k = 0; k < NR; ++k)
                    lds[b * zlen + cell0 + (k + 1) * sz] = zc[k] + om * (dinv[k] * t[k] - zc[k]);
            }
            lds_sync();
        }
        double zero[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) zero[k] = 0.0;
        res_apply<NR>(A, b * zlen + cell0, sz, zero, zc, t);
        zc_buf = b;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            w[k] = dinv[k] != 0.0 ? cc[k] * zc[k] - t[k] : 0.0;
            const double u = is(own, k) ? zc[k] : 0.0;
            gam += r[k] * u;
            del += u * w[k];
        }
    };
    // w of the window's other nodes, published in the round of the last barrier
    auto halo_w = [&]() {
        const double *P = wv(nbar - 1);
        double h[NR];
        load(P, live & ~own, h);
#pragma unroll
        for (int k = 0; k < NR; ++k) w[k] = is(live & ~own, k) ? h[k] : w[k];
    };
    auto publish_x = [&](int j) {
        const double *row = xh(j);
#pragma unroll
        for (int k = 0; k < NR; ++k)
            if (is(edge1, k)) stg(row, id_of(k), LX[k * kThreads]);
    };

    double theta = 0.0, src_scale = 0.0;
    int nsteps;
    {
        const Consts C = fetch(&Dp->C);
        const Bufs B = fetch(&Dp->B);
        const LaunchInfo I = fetch(&Dp->I);
        nsteps = lane_steps(C, L.kind);
        if (is_adj) {
            const double Th = *B.Theta;
            src_scale = C.plt ? (double)C.p / (double)C.Ne
                              : pow_call(Th, 1.0 - C.p) / (double)C.Ne;
            if (!(Th > 0.0) || !isfinite(Th)) set_status(ctl, -5);
        }
        if (L.kind == F_PRI) {
            if (L.slice > 0 && !I.cold && !C.plt) theta = B.in_th[L.slice];
        } else if (L.kind == GK_PRI) {
            theta = B.in_th[L.slice];
        }
    }
    const unsigned nbar0 = nbar;
    unsigned long long iters_all = 0;
    if (leader) {
        trec[TR_KIND] = L.kind;
        trec[TR_SLICE] = L.slice;
        trec[TR_NWG] = g;
        trec[TR_TILE] = L.tw * L.th;
        trec[TR_START] = (unsigned long long)now_ticks();
    }

    // the solve last set up (number `step`, 1..nsteps) and its progress
    enum { SETUP, RESTART, ITER };
    int mode = SETUP, step = 0;
    int sp_n = 0, sp_j = 0, sp_jprev = 0, st_n = 0, st_j = 0, st_jprev = 0;
    double bnorm = 0.0, relres = 0.0, rnorm = 0.0, alpha = 0.0, beta = 0.0, gamma = 0.0;
    int iter = 0, restarts = 0, ext_cap = 1, order = 0;
    bool capped = false, first = true, shown = false;
    for (;;) {
        const bool prev = step > 0, next = step < nsteps, last = prev && !next;
        // x of solve `step` is kept in history slot `step` once it is finished
        const double *xp = xh(step);
        // sums: SETUP residual, ||x||_p^p, b, r0, (r, u), (u, w), plain start's r0;
        // otherwise (r, u), (u, w), (r, r)
        double sum[7] = {0, 0, 0, 0, 0, 0, 0};
        if (mode == ITER) {
            // s = w + beta s, p = u + beta p, x += alpha p, r -= alpha s (p and x
            // of nodes that are not owned are formed too, and never read)
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                const double u = lds[zc_buf * zlen + cell0 + (k + 1) * sz];
                const double p0 = LP[k * kThreads], x0 = LX[k * kThreads];
                s[k] = first ? w[k] : w[k] + beta * s[k];
                const double pn = first ? u : u + beta * p0;
                LP[k * kThreads] = pn;
                LX[k * kThreads] = x0 + alpha * pn;
                r[k] -= alpha * s[k];
                const double ro = is(own, k) ? r[k] : 0.0;
                sum[2] += ro * ro;
            }
        } else if (mode == RESTART) {
            // CG anew from the true residual of x: the owned values cross to the
            // neighbours' windows first
            double zc[NR], t[NR], v[NR], vr[kRim];
            load(xp, fill | own, v);
            load_rim(xp, vr);
#pragma unroll
            for (int k = 0; k < NR; ++k) LX[k * kThreads] = v[k];
            put_win(0, v, vr);
            load(bvec(step), own & live, v);
            lds_sync();
            res_apply<NR>(A, cell0, sz, v, zc, t);
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                w[k] = is(live & own, k) ? t[k] - cc[k] * zc[k] : 0.0;
                sum[2] += w[k] * w[k];
                if (is(edge, k)) stg(wv(nbar), id_of(k), w[k]);
            }
            if (!barrier(false)) return false;
            halo_w();
#pragma unroll
            for (int k = 0; k < NR; ++k) r[k] = w[k];
            zc_buf = 0;
        } else {
            const Consts C = fetch(&Dp->C);
            const Bufs B = fetch(&Dp->B);
            const LaunchInfo I = fetch(&Dp->I);
            const size_t Nn = C.Nn;
            StepInfo st{};
            if (next) {
                st = step_info(C, B, I, L, step, xp);
                st_n = st.n;
                st_j = st.j;
                st_jprev = st.jprev;
            }
            // waits: the guess of a cold-started slice; what a sweep's step reads
            if (next && st.wait) {
                if (!waitf(st.wait_idx)) return false;
                if (L.kind == F_PRI && I.cold && L.slice > 0) theta = ldc(B.Gk_th + L.slice - 1);
            }
            if (sweep) {
                if (step == 0) {
                    if (!waitf(flag_index(FL_F, L.kind == SWEEP_PRI ? 0 : C.Ntau))) return false;
                    if (L.kind == SWEEP_PRI) theta = ldc(B.F_th);
                } else if (!waitf(flag_index(FL_F, sp_n))) {
                    return false;
                }
                if (next && (I.cold || I.gk_lanes))
                    if (!waitf(flag_index(I.cold ? FL_COLD : FL_GK, st.n))) return false;
            }
            // window 0: x of the finished solve, window 1: the operand tp of the
            // next right-hand side where it is another vector (a sweep's next input
            // u = x + F_n - G(u^k_n), a lane's first input)
            double zc[NR], t[NR], v[NR], bv[NR], vr[kRim], br[kRim];
            zc_buf = 0;
            if (prev) {
                load_x(xp, v, vr);
                load(bvec(step), own & live, bv);
                if (sweep) {
                    const double *Fp = L.kind == SWEEP_PRI
                                           ? B.S + (size_t)(C.M * (sp_n + 1) - 1) * Nn
                                           : B.FL + (size_t)sp_n * Nn;
                    const double *Gp = B.Gk + (size_t)sp_n * Nn;
                    double fr[kRim], gr[kRim];
                    load(Fp, fill, zc);
                    load(Gp, fill, t);
                    load_rim(Fp, fr);
                    load_rim(Gp, gr);
#pragma unroll
                    for (int k = 0; k < NR; ++k) zc[k] = v[k] + (zc[k] - t[k]);
#pragma unroll
                    for (int i = 0; i < kRim; ++i) br[i] = vr[i] + (fr[i] - gr[i]);
                    put_win(zlen, zc, br);
                }
                put_win(0, v, vr);
            } else {
                load(st.tp_src, fill, v);
                load_rim(st.tp_src, vr);
                put_win(zlen, v, vr);
#pragma unroll
                for (int i = 0; i < kRim; ++i) br[i] = vr[i];
            }
            lds_sync();
            if (prev) {
                // ---- the finished solve: true residual and outputs --------------
                res_apply<NR>(A, cell0, sz, bv, zc, t);
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    const double rv = is(live & own, k) ? t[k] - cc[k] * zc[k] : 0.0;
                    sum[0] += rv * rv;
                }
                // zc: x at the thread's nodes
#pragma unroll
                for (int k = 0; k < NR; ++k)
                    if (is(own, k)) stg(xp, id_of(k), zc[k]);
                if (!is_adj) {
#pragma unroll
                    for (int k = 0; k < NR; ++k)
                        sum[1] += ipow(is(own, k) ? zc[k] : 0.0, C.p);
                }
                if (L.kind == F_PRI) {
                    store(B.S + (size_t)(sp_j - 1) * Nn, own, zc);
                    if (C.plt && last) store(B.out_T + (size_t)(L.slice + 1) * Nn, own, zc);
                } else if (L.kind == F_ADJ) {
                    if (last) store(B.FL + (size_t)L.slice * Nn, own, zc);
                    if (C.plt && last) store(B.out_L + (size_t)(L.slice - 1) * Nn, own, zc);
                } else {
                    store((sweep ? B.Gn : B.Gk) + (size_t)sp_n * Nn, own, zc);
                }
                if (sweep) {
                    // (the slice-end slot of S, still read as F_n by the neighbours
                    // in this round, follows after the barrier)
                    const double *row = L.kind == SWEEP_PRI ? B.out_T + (size_t)(sp_n + 1) * Nn
                                                            : B.out_L + (size_t)(sp_n - 1) * Nn;
#pragma unroll
                    for (int k = 0; k < NR; ++k) v[k] = lds[zlen + cell0 + (k + 1) * sz];
                    store(row, own, v);
                }
                if (L.kind == F_ADJ || L.kind == SWEEP_ADJ) {
                    // sensitivity terms of the elements right above the owned nodes;
                    // they wait in p's slots until the residual has been accepted
                    const double *Tr = B.S + (size_t)(sp_j - 1) * Nn;
                    const double *Tp = sp_jprev > 0 ? B.S + (size_t)(sp_jprev - 1) * Nn : nullptr;
                    const double *Gp = B.Gk + (size_t)sp_n * Nn;
                    const int gxf = fresh(gx), gyf = fresh(gy0);
                    const double idl = fine ? C.inv_dt : C.inv_dtau;
                    auto corner = [&](const double *row, int k, int dx) {
                        const int y = gyf + k;
                        const bool in = act && gxf >= 0 && gxf + dx < W && y >= 0 && y < HN;
                        return *nd(row, in ? (unsigned)(y * W + gxf + dx) : 0u);
                    };
                    // lower corners of the element row, left and right
                    double ta = corner(Tr, 0, 0), tb = corner(Tr, 0, 1), pa = 0.0, pb = 0.0;
                    if (I.has_dc && Tp) {
                        pa = corner(Tp, 0, 0);
                        pb = corner(Tp, 0, 1);
                    }
#pragma unroll
                    for (int k = 0; k < NR; ++k) {
                        const double tc = corner(Tr, k + 1, 0), td = corner(Tr, k + 1, 1);
                        const int y = gyf + k;
                        const bool el = is(own, k) && gxf < C.nx && y < C.ny;
                        const unsigned e = el ? (unsigned)(y * C.nx + gxf) : 0u;
                        const int z = cell0 + (k + 1) * sz;
                        double l0 = lds[z], l1 = lds[z + 1], l2 = lds[z + sz + 1], l3 = lds[z + sz];
                        if (sweep) {
                            const unsigned id = el ? id_of(k) : 0u;
                            const unsigned up = el ? id + W : 0u;
                            l0 -= ldg(Gp, id);
                            l1 -= ldg(Gp, id + 1);
                            l2 -= ldg(Gp, up + 1);
                            l3 -= ldg(Gp, up);
                        }
                        double term = *nd(B.dk, e) * elem_k(C, l0, l1, l2, l3, ta, tb, td, tc);
                        if (I.has_dc) {
                            double pc = 0.0, pd = 0.0;
                            if (Tp) {
                                pc = corner(Tp, k + 1, 0);
                                pd = corner(Tp, k + 1, 1);
                            }
                            term += *nd(B.dc, e) * idl *
                                    elem_c(C, l0, l1, l2, l3, ta - pa, tb - pb, td - pd, tc - pc);
                            pa = pc;
                            pb = pd;
                        }
                        LP[k * kThreads] = term;
                        ta = tc;
                        tb = td;
                    }
                }
            }
            if (next) {
                // ---- the next solve: b, x0, r0 ----------------------------------
                // states of the slice before this one extrapolate; differences that
                // reach back to the slice's given first state, which may be off in
                // its rough modes, are not used
                order = 0;
                if (fine && C.extrap) order = step >= 2 ? 1 : 0;
                else if (fine && prev) order = max(0, min(min(step - 2, 3), ext_cap));
                const int gxf = fresh(gx), gyf = fresh(gy0);
                const bool inx = act && gxf >= 0 && gxf < W;
                // source
                if (st.adjoint) {
                    load(B.S + (size_t)(st.j - 1) * Nn, live, bv);
#pragma unroll
                    for (int k = 0; k < NR; ++k) bv[k] = src_scale * ipow(bv[k], C.p - 1);
                } else {
                    const double f = B.qt[st.j] * C.quarter_area * (double)((gxf > 0) + (gxf < C.nx));
#pragma unroll
                    for (int k = 0; k < NR; ++k)
                        bv[k] = f * (double)((gyf + k > 0) + (gyf + k < C.ny));
                }
                {
                    // + (C/delta) tp on the window
                    const double ms = fine ? C.inv_dt : C.inv_dtau;
                    int z = (prev && !sweep ? 0 : zlen) + cell0;
                    auto elem = [&](int k, int dx) {
                        const int ey = gyf + k;
                        const bool in = inx && ey >= 0 && ey <= C.ny + 1;
                        const double m = *nd(B.cm, in ? (unsigned)(ey * C.EW + gxf + dx) : 0u);
                        return in ? m * ms : 0.0;
                    };
                    double ml0 = elem(0, 0), mr0 = elem(0, 1);
                    double l0 = lds[z - 1], c0 = lds[z], r0 = lds[z + 1];
                    z += sz;
                    double l1 = lds[z - 1], c1 = lds[z], r1 = lds[z + 1];
#pragma unroll
                    for (int k = 0; k < NR; ++k) {
                        z += sz;
                        const double l2 = lds[z - 1], c2 = lds[z], r2 = lds[z + 1];
                        const double ml1 = elem(k + 1, 0), mr1 = elem(k + 1, 1);
                        double m = 4.0 * ((ml0 + mr0) + (ml1 + mr1)) * c1;
                        m += 2.0 * ((mr0 + mr1) * r1 + (ml0 + ml1) * l1 + (ml1 + mr1) * c2 +
                                    (ml0 + mr0) * c0);
                        m += mr1 * r2 + ml1 * l2 + mr0 * r0 + ml0 * l0;
                        bv[k] = is(live, k) ? m + bv[k] : 0.0;
                        l0 = l1;
                        c0 = c1;
                        r0 = r1;
                        l1 = l2;
                        c1 = c2;
                        r1 = r2;
                        ml0 = ml1;
                        mr0 = mr1;
                    }
                }
                if (order > 0) {
                    // residual of the plain start x0 = x: it judges the extrapolation
                    res_apply<NR>(A, cell0, sz, bv, zc, t);
#pragma unroll
                    for (int k = 0; k < NR; ++k) {
                        const double rv = is(live & own, k) ? t[k] - cc[k] * zc[k] : 0.0;
                        sum[6] += rv * rv;
                    }
                    // x0 from x and the states before it
                    double a[NR], ar[kRim];
#pragma unroll
                    for (int k = 0; k < NR; ++k) v[k] = lds[cell0 + (k + 1) * sz];
                    load(xh(step - 1), fill, a);
                    load_rim(xh(step - 1), ar);
                    const double ca = order == 1 ? 2.0 : order == 2 ? 3.0 : 4.0;
                    const double cb = order == 1 ? -1.0 : order == 2 ? -3.0 : -6.0;
#pragma unroll
                    for (int k = 0; k < NR; ++k) v[k] = ca * v[k] + cb * a[k];
#pragma unroll
                    for (int i = 0; i < kRim; ++i) vr[i] = ca * vr[i] + cb * ar[i];
                    if (order > 1) {
                        load(xh(step - 2), fill, a);
                        load_rim(xh(step - 2), ar);
                        const double cd = order == 2 ? 1.0 : 4.0;
#pragma unroll
                        for (int k = 0; k < NR; ++k) v[k] += cd * a[k];
#pragma unroll
                        for (int i = 0; i < kRim; ++i) vr[i] += cd * ar[i];
                    }
                    if (order > 2) {
                        load(xh(step - 3), fill, a);
                        load_rim(xh(step - 3), ar);
#pragma unroll
                        for (int k = 0; k < NR; ++k) v[k] -= a[k];
#pragma unroll
                        for (int i = 0; i < kRim; ++i) vr[i] -= ar[i];
                    }
                } else if (!prev || sweep) {
                    // x0 from the step's description; uc, br: its operand tp
                    double uc[NR];
#pragma unroll
                    for (int k = 0; k < NR; ++k) uc[k] = lds[zlen + cell0 + (k + 1) * sz];
                    if (trunc) {
#pragma unroll
                        for (int k = 0; k < NR; ++k) v[k] = uc[k];
#pragma unroll
                        for (int i = 0; i < kRim; ++i) vr[i] = br[i];
                    } else {
                        load(st.x0_src, fill, v);
                        load_rim(st.x0_src, vr);
                        if (st.d1) {
                            double a[NR], ar[kRim];
                            load(st.d0, fill, a);
                            load_rim(st.d0, ar);
#pragma unroll
                            for (int k = 0; k < NR; ++k) v[k] += uc[k] - a[k];
#pragma unroll
                            for (int i = 0; i < kRim; ++i) vr[i] += br[i] - ar[i];
                        }
                    }
                    if (!prev && sweep) {
                        // what the sweep publishes of its input
                        store(L.kind == SWEEP_PRI ? B.out_T + Nn
                                                  : B.out_L + (size_t)(C.Ntau - 1) * Nn,
                              own, uc);
                        if (is_adj) {
#pragma unroll
                            for (int k = 0; k < NR; ++k) uc[k] = 0.0;
                            store(B.out_L + (size_t)C.Ntau * Nn, own, uc);
                        }
                    }
                }
                if (!prev || sweep || order > 0) {
                    lds_sync();
                    put_win(0, v, vr);
                    lds_sync();
                }
                res_apply<NR>(A, cell0, sz, bv, zc, t);
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    r[k] = is(live, k) ? t[k] - cc[k] * zc[k] : 0.0;
                    // x of the new solve (the finished x is in the history)
                    LX[k * kThreads] = zc[k];
                    const double bo = is(own, k) ? bv[k] : 0.0, ro = is(own, k) ? r[k] : 0.0;
                    sum[2] += bo * bo;
                    sum[3] += ro * ro;
                }
                store(bvec(step + 1), own, bv);
                lds_sync();  // both operand windows have been read
            }
        }
        // ---- every round: u, w, the sums, w's and x's edges, the barrier -----------
        const bool setup = mode == SETUP;
        if (!last || !setup) {
            precond(sum[setup ? 4 : 0], sum[setup ? 5 : 1]);
            const double *P = wv(nbar);
#pragma unroll
            for (int k = 0; k < NR; ++k)
                if (is(edge, k)) stg(P, id_of(k), w[k]);
        }
        double tot[7];
        if (setup) {
            put_sums(sum);
            // release: rows that other lanes read once this round's flags are set
            if (!barrier(prev && (last || L.kind == COLD_PRI || L.kind == COLD_ADJ))) return false;
            if (!last) halo_w();
            get_sums(tot);
        } else {
            // near the end x's edge goes out too, so that the round that closes the
            // solve can start at once (a round gains about a decimal digit)
            const int nit = iter + 1;
            shown = mode == ITER && (trunc ? nit >= coarse_iters
                                           : rnorm <= 200.0 * rtol * bnorm || nit >= max_iter);
            if (shown) publish_x(step);
            double s3[3] = {sum[0], sum[1], sum[2]};
            put_sums(s3);
            if (!barrier(false)) return false;
            halo_w();
            get_sums(s3);
            tot[0] = s3[0];
            tot[1] = s3[1];
            tot[2] = s3[2];
        }
        // ---- decisions ---------------------------------------------------------------
        bool closed = false;  // x of the current solve is final
        if (setup) {
            const Consts C = fetch(&Dp->C);
            const Bufs B = fetch(&Dp->B);
            bool again = false;
            if (prev && !trunc && !capped && bnorm > 0.0 && (C.verify || C.fp32)) {
                // the true residual decides
                const double rn = sqrt(tot[0]);
                relres = rn / bnorm;
                if (!(rn <= rtol * bnorm)) {
                    if (restarts >= (C.fp32 ? C.max_restarts : 2) || iter >= max_iter) {
                        if (leader) set_status(ctl, -4);
                    } else {
                        again = true;
                    }
                }
            }
            if (again) {
                ++restarts;
                mode = RESTART;
                continue;
            }
            if (prev) {
                // ---- the finished solve's sums and flags -------------------------
                if (L.kind == F_ADJ || L.kind == SWEEP_ADJ) {
                    const double *ac = fine ? B.acc + (size_t)(L.slice - 1) * C.Ne : B.accG;
                    const int gxf = fresh(gx), gyf = fresh(gy0);
                    double a[NR];
                    auto el = [&](int k) { return is(own, k) && gxf < C.nx && gyf + k < C.ny; };
                    auto eid = [&](int k) { return (unsigned)((gyf + k) * C.nx + gxf); };
                    if (step > 1) {
#pragma unroll
                        for (int k = 0; k < NR; ++k) a[k] = *nd(ac, el(k) ? eid(k) : 0u);
                    } else {
#pragma unroll
                        for (int k = 0; k < NR; ++k) a[k] = 0.0;
                    }
#pragma unroll
                    for (int k = 0; k < NR; ++k)
                        if (el(k)) *nd(ac, eid(k)) = a[k] + LP[k * kThreads];
                }
                if (L.kind == SWEEP_PRI) {
                    double u[NR];
                    const double *row = B.out_T + (size_t)(sp_n + 1) * C.Nn;
#pragma unroll
                    for (int k = 0; k < NR; ++k) u[k] = *nd(row, is(own, k) ? id_of(k) : 0u);
                    store(B.S + (size_t)(C.M * (sp_n + 1) - 1) * C.Nn, own, u);
                }
                if (!is_adj) {
                    const double inv = fine ? C.inv_NtNe : C.inv_NtauNe;
                    // with G = 0 a fine lane keeps its slice's part of Theta~ instead
                    const double thG = C.plt ? theta + tot[1] * inv
                                             : pow_call(ipow(theta, C.p) + tot[1] * inv, C.inv_p);
                    if (L.kind == SWEEP_PRI) {
                        const double thu = thG + ldc(B.F_th + sp_n) - ldc(B.Gk_th + sp_n);
                        if (leader) {
                            B.out_th[sp_n + 1] = thu;
                            B.Gn_th[sp_n] = thG;
                        }
                        theta = thu;
                    } else {
                        theta = thG;
                        if (leader && !fine) B.Gk_th[sp_n] = thG;
                        if (leader && fine && last) B.F_th[L.slice] = thG;
                    }
                }
                if (leader) {
                    const unsigned epoch = fetch(&Dp->I).epoch;
                    atomicAdd(fine ? &ctl->iters_fine : &ctl->iters_coarse,
                              (unsigned long long)iter);
                    atomicAdd(fine ? &ctl->solves_fine : &ctl->solves_coarse, 1ull);
                    atomicMax(&ctl->max_iters, iter);
                    atomicMax(&ctl->max_relres_bits,
                              (unsigned long long)__double_as_longlong(relres));
                    if (L.kind == GK_PRI || L.kind == GK_ADJ)
                        set_flag(B.flags, flag_index(FL_GK, sp_n), epoch);
                    if (L.kind == COLD_PRI || L.kind == COLD_ADJ)
                        set_flag(B.flags, flag_index(FL_COLD, sp_n), epoch);
                    if (fine && last) set_flag(B.flags, flag_index(FL_F, L.slice), epoch);
                    if (step - 1 < S.trace_stride - TR_HDR)
                        trec[TR_HDR + step - 1] = (unsigned long long)now_ticks();
                }
                iters_all += iter;
            } else if (leader && L.kind == SWEEP_PRI) {
                B.out_th[1] = theta;
            }
            if (last) break;
            // ---- the next solve becomes the current one --------------------------
            ext_cap = order == 0 ? 1 : tot[3] > tot[6] ? order - 1 : order + 1;
            sp_n = st_n;
            sp_j = st_j;
            sp_jprev = st_jprev;
            ++step;
            iter = restarts = 0;
            capped = shown = false;
            bnorm = sqrt(tot[2]);
            rnorm = sqrt(tot[3]);
            relres = bnorm > 0.0 ? rnorm / bnorm : 0.0;
            gamma = tot[4];
            alpha = tot[4] / tot[5];
            if (trunc) {
                closed = rnorm == 0.0;
            } else if (bnorm == 0.0) {
                closed = true;
#pragma unroll
                for (int k = 0; k < NR; ++k) LX[k * kThreads] = 0.0;
            } else {
                closed = rnorm <= rtol * bnorm;
            }
            mode = ITER;
            first = true;
        } else if (mode == RESTART) {
            gamma = tot[0];
            alpha = tot[0] / tot[1];
            rnorm = sqrt(tot[2]);
            mode = ITER;
            first = true;
        } else {
            iter += 1;
            rnorm = sqrt(tot[2]);
            const double target = rtol * bnorm;
            if (trunc ? (iter >= coarse_iters || rnorm == 0.0)
                      : (rnorm <= target || iter >= max_iter)) {
                relres = bnorm > 0.0 ? rnorm / bnorm : 0.0;
                capped = !trunc && !(rnorm <= target);
                if (capped && rnorm > target && leader) set_status(ctl, -4);
                closed = true;
            } else {
                beta = tot[0] / gamma;
                alpha = tot[0] / (tot[1] - beta * tot[0] / alpha);
                gamma = tot[0];
                first = false;
            }
        }
        if (closed) {
            if (!shown) {
                publish_x(step);
                if (!barrier(false)) return false;
            }
            mode = SETUP;
        }
    }
    if (leader) {
        trec[TR_ROUNDS] = nbar - nbar0;
        trec[TR_ITERS] = iters_all;
        if constexpr (TIMED) {
            trec[TR_T_WORK] = tm.work;
            trec[TR_T_BAR] = tm.bar;
            trec[TR_T_RED] = tm.red;
            trec[TR_T_FLAG] = tm.flag;
        }
    }
    return true;
}

}  // namespace

// One persistent cooperative launch whose fine and coarse lanes are all
// resident. MULTI: lanes of several designs (descriptors in D); CMESH: the
// launch also holds coarse-mesh lanes; TIMED: phase times go to the trace.
template <bool MULTI, bool CMESH, bool TIMED>
__global__ void __launch_bounds__(kThreads) k_resident(const EngineDesc *__restrict__ D, Launch S,
                                                       EngineDesc E1) {
    __shared__ double red[kWaves * kResSums];
    const int gid = S.wg_group[blockIdx.x];
    if (gid < 0) return;
    if constexpr (!MULTI) {
        if (E1.B.ctl->status == kStatusOrder) return;
    }
    const Group G = S.groups[gid];
    const int rank = blockIdx.x - G.wg0;
    unsigned *bar = S.bar + (size_t)gid * kBarStride;
    double *part = S.partials + (size_t)gid * 2 * kMaxGroup * 4;
    unsigned nbar = 0;
    Control *ctl = S.ctl0;
    bool ok = true;
    for (int li = 0; ok; ++li) {
        int lane_id;
        if (G.queue < 0) {
            if (li >= G.nlanes) break;
            lane_id = G.lane0 + li;
        } else {
            // shared queue: the group leader takes the next position and the
            // barrier hands it to the group's other workgroups
            if (rank == 0 && threadIdx.x == 0)
                stc(S.qslot + gid, (int)__hip_atomic_fetch_add(S.qhead + G.queue, 1u,
                                                               __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT));
            ++nbar;
            ok = group_barrier<!CMESH>(bar, (unsigned)G.nwg, nbar * (unsigned)G.nwg, ctl,
                                       S.timeout_ticks, false);
            if (!ok) break;
            const int pos = __builtin_amdgcn_readfirstlane(ldc(S.qslot + gid));
            if (pos >= G.nlanes) break;
            lane_id = G.lane0 + pos;
        }
        const Lane L = S.lanes[lane_id];
        unsigned long long *trec = S.trace + (size_t)lane_id * S.trace_stride;
        if constexpr (CMESH) {
            if (is_cm_kind(L.kind)) {
                ctl = E1.B.ctl;
                const long long r = cm_lane(D, L.kind, L.slice, rank, G.nwg, G.vec, bar, part,
                                            nbar, trec, S.trace_stride - TR_HDR);
                ok = r >= 0;
                nbar = (unsigned)r;
                continue;
            }
        }
        const EngineDesc *E = D + (MULTI ? L.design : 0);
        ctl = E->B.ctl;
        if (L.nr <= 2)
            ok = res_lane<2, TIMED, !CMESH>(E, L, S, G, bar, part, nbar, trec, red);
        else if (L.nr <= 4)
            ok = res_lane<4, TIMED, !CMESH>(E, L, S, G, bar, part, nbar, trec, red);
        else
            ok = res_lane<6, TIMED, !CMESH>(E, L, S, G, bar, part, nbar, trec, red);
    }
    if (!ok && threadIdx.x == 0) {
        atomicExch(&ctl->abort, 1);
        set_status(ctl, -3);
    }
}

}  // namespace pt
