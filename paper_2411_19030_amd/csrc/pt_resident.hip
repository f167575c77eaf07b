// Resident lanes: the solves of a lane whose grid fits the registers and the
// LDS of its group. Included by pt_engine.hip; it uses the engine's flags,
// step descriptions and barrier.
//
// A solve is a conjugate gradient in the single-reduction form of Chronopoulos
// and Gear with a polynomial preconditioner: u = q(D^{-1}A) D^{-1} r, the result
// of d + 1 Richardson sweeps z += omega_i D^{-1} (r - A z) from z = 0 whose
// omega_i are the inverse roots of the Chebyshev polynomial of degree d + 1 on
// an interval inside the spectrum's bounds (res_omega). A round of a group is
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
// Measured at 256^2, 512 steps in 32 slices, cg_rtol 1e-12, one warm cycle, against
// Jacobi CG on full-row tiles with one halo row: 106 -> 31.7 ms; CG rounds per fine
// step 42 -> 8 (degree 4, extrapolated), per coarse step 169 -> 38. Sequential 100^2 with
// 240 steps, forward and adjoint: 584 -> 78 ms.

namespace pt {

namespace {

constexpr int kResSums = 8;         // sums per reduction, at most

// A solve ends its rounds at this share of cg_rtol ||b||. What few rounds of the
// polynomial leave of a residual are its lowest modes, with more error to a residual
// than what a Jacobi CG leaves, which is spread over the spectrum; and what an
// extrapolated start leaves has the same sign at every step and adds up over a slice.
// Errors at shares of 1, against Jacobi CG on streaming lanes at the same cg_rtol
// (warm cycles of 14 problems of 32^2 to 512^2): Theta up to 144 times and states up
// to 9 times; with these shares states, multipliers and gradients are 0.02 to 0.1 of
// them at 1e-4 to 1e-12 (geometric means). A start within cg_rtol itself ends a
// solve as before. 256^2, 32 slices, warm, cg_rtol 1e-12: 29.0 -> 30.1 ms; sequential
// 100^2, 240 steps: 28.8 -> 34.1 ms.
constexpr double kStopFine = 0.1, kStopCoarse = 0.3;
// Solves again from the true residual, at most. Near what FP64 can certify each try
// rounds anew: 384^2, Gaussian design, cg_rtol 1e-12 was reported as PT_ENOCONV at
// shares of 1 and 2 tries.
constexpr int kResRestarts = 4;

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
typedef __attribute__((address_space(1))) unsigned char gbyte;
__device__ __forceinline__ gdouble *nd(const double *p, unsigned n) {
    return (gdouble *)((gchar *)p + n * 8u);
}
__device__ __forceinline__ const gbyte *ndb(const unsigned char *p, unsigned n) {
    return reinterpret_cast<const gbyte *>(reinterpret_cast<uintptr_t>(p)) + n;
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

// What one thread holds of its workgroup's window: its column gx, rows gy0 ..
// gy0 + NR - 1, and the node sets as bits per row: live (in the grid, the window
// and not fixed), fill (the same with one row more above the window), own, nodes
// that a neighbour's window (edge) or set-up window (edge1: one ring more) holds.
// The rim are the cells around the window that no thread's rows cover (id -1: no
// node there).
struct ResGeo {
    int W, gx, gy0;
    int cell0;     // LDS cell of the row below the first node
    int sz, zlen;  // row length and length of an operand window
    unsigned live, fill, own, edge, edge1;
    int rim_id[kRim], rim_cell[kRim];
    bool act;

    __device__ __forceinline__ unsigned id(int k) const {
        return (unsigned)(fresh(gy0 * W + gx) + k * W);
    }
    static __device__ __forceinline__ bool is(unsigned m, int k) {
        return (((unsigned)fresh((int)m) >> k) & 1u) != 0;
    }
    // this thread's slots of p, then of x
    template <int NR>
    __device__ __forceinline__ int slot_p() const { return 2 * zlen + (int)threadIdx.x; }
    template <int NR>
    __device__ __forceinline__ int slot_x() const {
        return 2 * zlen + NR * kThreads + (int)threadIdx.x;
    }
    // A row of global values at the thread's nodes in m, all loads in flight at
    // once: no load is conditional (the other nodes read node 0), since a masked
    // load whose value is used in its own branch waits for it there, node by node.
    template <int NR>
    __device__ __forceinline__ void load(const double *row, unsigned m, double (&v)[NR]) const {
#pragma unroll
        for (int k = 0; k < NR; ++k) v[k] = ldg(row, is(m, k) ? id(k) : 0u);
    }
    __device__ __forceinline__ void load_rim(const double *row, double (&v)[kRim]) const {
#pragma unroll
        for (int i = 0; i < kRim; ++i) v[i] = ldg(row, rim_id[i] >= 0 ? (unsigned)rim_id[i] : 0u);
    }
    template <int NR>
    __device__ __forceinline__ void store(const double *row, unsigned m,
                                          const double (&v)[NR]) const {
#pragma unroll
        for (int k = 0; k < NR; ++k)
            if (is(m, k)) *nd(row, id(k)) = v[k];
    }
    // the operand window at LDS index zb
    template <int NR>
    __device__ __forceinline__ void put(int zb, const double (&v)[NR],
                                        const double (&vr)[kRim]) const {
        extern __shared__ double lds[];
        if (act) {
#pragma unroll
            for (int k = 0; k < NR; ++k) lds[zb + cell0 + (k + 1) * sz] = is(fill, k) ? v[k] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < kRim; ++i)
            if (rim_id[i] >= 0) lds[zb + rim_cell[i]] = vr[i];
    }
    // The operator at the thread's nodes from the element values: gap k lies below
    // row k, its elements left and right of the column have mass ml, mr (c hx hy/36
    // over the step) and stiffness kl, kr (k/6); cc is the diagonal.
    template <int NR>
    static __device__ __forceinline__ void assemble(const Consts &C, const double (&ml)[NR + 1],
                                                    const double (&mr)[NR + 1],
                                                    const double (&kl)[NR + 1],
                                                    const double (&kr)[NR + 1], ResCoef<NR> &Q,
                                                    double (&cc)[NR]) {
        double sl = 0.0, sr = 0.0, xl = 0.0, xr = 0.0;
#pragma unroll
        for (int k = 0; k <= NR; ++k) {
            const double a = ml[k], b = mr[k];
            Q.dl[k] = a + C.e_d * kl[k];
            Q.dr[k] = b + C.e_d * kr[k];
            Q.nn[k] = 2.0 * (a + b) + C.e_y * (kl[k] + kr[k]);
            const double nsl = 4.0 * a + C.e_self * kl[k], nsr = 4.0 * b + C.e_self * kr[k];
            const double nxl = 2.0 * a + C.e_x * kl[k], nxr = 2.0 * b + C.e_x * kr[k];
            if (k > 0) {
                Q.el[k - 1] = xl + nxl;
                Q.er[k - 1] = xr + nxr;
                cc[k - 1] = (sl + sr) + (nsl + nsr);
            }
            sl = nsl;
            sr = nsr;
            xl = nxl;
            xr = nxr;
        }
    }
    // from the padded element values: elements (gx - 1, gy0 + k - 1), (gx, gy0 + k - 1)
    template <int NR>
    __device__ __forceinline__ void coefs(const Consts &C, const Bufs &B, bool fine,
                                          ResCoef<NR> &Q, double (&cc)[NR]) const {
        const double ms = fine ? C.inv_dt : C.inv_dtau;
        const bool inx = act && gx >= 0 && gx < W;
        double ml[NR + 1], mr[NR + 1], kl[NR + 1], kr[NR + 1];
#pragma unroll
        for (int k = 0; k <= NR; ++k) {
            const int ey = gy0 + k;  // padded element row
            const bool in = inx && ey >= 0 && ey <= C.ny + 1;
            // (element 0 is padding: its values are 0)
            const unsigned e = in ? (unsigned)(ey * C.EW + gx) : 0u, d = in ? 1u : 0u;
            ml[k] = *nd(B.cm, e) * ms;
            mr[k] = *nd(B.cm, e + d) * ms;
            kl[k] = *nd(B.kq, e);
            kr[k] = *nd(B.kq, e + d);
        }
        assemble<NR>(C, ml, mr, kl, kr, Q, cc);
    }

    // ---- the coarse mesh (W nodes per row as the window's grid) --------------------
    // masses over dtau of the elements around the thread's nodes
    template <int NR>
    __device__ __forceinline__ void cm_mass(const Consts &C, const CoarseMesh &M,
                                            double (&ml)[NR + 1], double (&mr)[NR + 1]) const {
        const double ms = 4.0 * C.cm_unit * C.inv_dtau;
        cm_elements<NR>(M, M.cE, ms, ml, mr);
    }
    template <int NR>
    __device__ __forceinline__ void cm_elements(const CoarseMesh &M, const double *v, double f,
                                                double (&l)[NR + 1], double (&r)[NR + 1]) const {
        const bool inl = act && gx >= 1 && gx <= M.nxc, inr = act && gx >= 0 && gx < M.nxc;
#pragma unroll
        for (int k = 0; k <= NR; ++k) {
            const int ey = gy0 + k - 1;
            const bool in = ey >= 0 && ey < M.nyc;
            const double a = *nd(v, in && inl ? (unsigned)(ey * M.nxc + gx - 1) : 0u);
            const double b = *nd(v, in && inr ? (unsigned)(ey * M.nxc + gx) : 0u);
            l[k] = in && inl ? a * f : 0.0;
            r[k] = in && inr ? b * f : 0.0;
        }
    }
    template <int NR>
    __device__ __forceinline__ void cm_coefs(const Consts &C, const CoarseMesh &M, ResCoef<NR> &Q,
                                             double (&cc)[NR]) const {
        double ml[NR + 1], mr[NR + 1], kl[NR + 1], kr[NR + 1];
        cm_mass<NR>(C, M, ml, mr);
        cm_elements<NR>(M, M.kE, 1.0 / 6.0, kl, kr);
        assemble<NR>(C, ml, mr, kl, kr, Q, cc);
    }
    // a fine row of values at the fine nodes of the thread's nodes in m, of the rim
    template <int NR>
    __device__ __forceinline__ void load_fine(const double *row, int Wf, unsigned m,
                                              double (&v)[NR]) const {
#pragma unroll
        for (int k = 0; k < NR; ++k)
            v[k] = ldg(row, is(m, k) ? (unsigned)(2 * ((gy0 + k) * Wf + gx)) : 0u);
    }
    __device__ __forceinline__ void load_rim_fine(const double *row, int Wf,
                                                  double (&v)[kRim]) const {
#pragma unroll
        for (int i = 0; i < kRim; ++i) {
            const int j = rim_id[i] >= 0 ? rim_id[i] / W : 0, c = rim_id[i] - j * W;
            v[i] = ldg(row, rim_id[i] >= 0 ? (unsigned)(2 * (j * Wf + c)) : 0u);
        }
    }
};

// A lane as its set-up, restart and commit phases see it. The rounds of CG are a loop
// of their own behind these phases: as one loop over phases the allocator put parts of
// the operator, which the rounds read, into scratch for the set-up's sake. Solve of 8
// rounds, set-up included, 257x257 nodes on 63 workgroups (NR 6): 13.6 -> 11.4 us a
// round; 101x101 on 40 (NR 2, no spill left): 7.1 -> 5.8 us.
struct ResLaneCtx {
    const EngineDesc *D;
    const double *gv0;  // group vectors from R0 on, gvs apart
    size_t gvs;
    unsigned long long *trec;
    int kind, slice, trace_steps;
    bool trunc, leader;
    int step, nsteps;  // the solve last set up (1..nsteps), solves of the lane
    int sp_n, sp_j, sp_jprev, st_n, st_j, st_jprev;  // of that solve, of the next one
    int order, ext_cap;  // extrapolation of the next solve's start; its cap
    // theta carried by the lane; on fine lanes its p-th power, whose root is taken
    // once at the end (with G = 0: the slice's part of Theta~)
    double theta, src_scale;
    // residual of the finished solve, ||x||_p^p, ||b||^2, ||r0||^2, two sums of the
    // round, and the plain start's ||r0||^2 (this thread's parts)
    double sum[7];
};

// group vectors by consecutive pool slots, so that a choice between them is
// arithmetic on one base: w by round parity; right-hand sides of the solve being
// finished and of the next one (each value read by its writer only); the last
// four solutions
__device__ __forceinline__ const double *res_w(const double *gv0, size_t gvs, unsigned par) {
    return gv0 + (size_t)(V_W0 - V_R0 + (par & 1)) * gvs;
}
__device__ __forceinline__ const double *res_b(const double *gv0, size_t gvs, int j) {
    return gv0 + (size_t)(j & 1) * gvs;
}
__device__ __forceinline__ const double *res_x(const double *gv0, size_t gvs, int j) {
    return gv0 + (size_t)(V_S0 - V_R0 + (j & 3)) * gvs;
}

// bv = (M v) + bv at the thread's live nodes, 0 elsewhere: M the masses ml, mr of the
// elements around them, v the operand window whose cell below the first node is z.
template <int NR>
__device__ __forceinline__ void res_mass(const ResGeo &g, int z, const double (&ml)[NR + 1],
                                         const double (&mr)[NR + 1], double (&bv)[NR]) {
    extern __shared__ double lds[];
    const int sz = g.sz;
    double l0 = lds[z - 1], c0 = lds[z], r0 = lds[z + 1];
    z += sz;
    double l1 = lds[z - 1], c1 = lds[z], r1 = lds[z + 1];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        z += sz;
        const double l2 = lds[z - 1], c2 = lds[z], r2 = lds[z + 1];
        const double ml0 = ml[k], mr0 = mr[k], ml1 = ml[k + 1], mr1 = mr[k + 1];
        double m = 4.0 * ((ml0 + mr0) + (ml1 + mr1)) * c1;
        m += 2.0 * ((mr0 + mr1) * r1 + (ml0 + ml1) * l1 + (ml1 + mr1) * c2 + (ml0 + mr0) * c0);
        m += mr1 * r2 + ml1 * l2 + mr0 * r0 + ml0 * l0;
        bv[k] = ResGeo::is(g.live, k) ? m + bv[k] : 0.0;
        l0 = l1;
        c0 = c1;
        r0 = r1;
        l1 = l2;
        c1 = c2;
        r1 = r2;
    }
}

// The set-up: true residual and outputs of the finished solve
// (ctx.step > 0), then right-hand side, start and residual of the next one. The
// residual r0 of the thread's nodes is left in their cells of window 1. Returns
// false when a wait timed out or another workgroup aborted.
template <int NR, bool TIMED>
__device__ __forceinline__ bool res_setup(const ResGeo &geo, ResLaneCtx &x, const ResCoef<NR> &A,
                                          const double (&cc)[NR], ResTimers &tm) {
    extern __shared__ double lds[];
    const ResGeo g = geo;
    auto is = [](unsigned m, int k) { return ResGeo::is(m, k); };
    const EngineDesc *Dp = x.D;
    const Consts C = fetch(&Dp->C);
    const Bufs B = fetch(&Dp->B);
    const LaunchInfo I = fetch(&Dp->I);
    Control *ctl = B.ctl;
    const long long tmo = C.timeout_ticks;
    Lane L;
    L.kind = x.kind;
    L.slice = x.slice;
    const int step = x.step, nsteps = x.nsteps;
    const bool trunc = x.trunc;
    const bool is_adj = is_adjoint_kind(L.kind);
    const bool sweep = L.kind == SWEEP_PRI || L.kind == SWEEP_ADJ;
    const bool fine = L.kind == F_PRI || L.kind == F_ADJ;
    const bool prev = step > 0, next = step < nsteps, last = prev && !next;
    const int sp_n = x.sp_n, sp_j = x.sp_j, sp_jprev = x.sp_jprev;
    const double *gv0 = x.gv0;
    const size_t gvs = x.gvs;
    auto xh = [&](int j) { return res_x(gv0, gvs, j); };
    // x of solve `step` is kept in history slot `step` once it is finished
    const double *xp = xh(step);
    const size_t Nn = C.Nn;
    const int sz = g.sz, zlen = g.zlen, cell0 = g.cell0, W = g.W, HN = C.ny + 1;
    const int LP = g.slot_p<NR>(), LX = g.slot_x<NR>();
    double sum[7] = {0, 0, 0, 0, 0, 0, 0};

    StepInfo st{};
    if (next) {
        st = step_info(C, B, I, L, step, xp);
        x.st_n = st.n;
        x.st_j = st.j;
        x.st_jprev = st.jprev;
    }
    // waits: the guess of a cold-started slice; what a sweep's step reads
    auto waitf = [&](int idx) -> bool {
        if constexpr (TIMED) {
            const long long t0 = now_ticks();
            const bool ok = wait_flag(B.flags, idx, I.epoch, ctl, tmo);
            const long long t1 = now_ticks();
            tm.work += t0 - tm.mark;
            tm.flag += t1 - t0;
            tm.mark = t1;
            return ok;
        }
        return wait_flag(B.flags, idx, I.epoch, ctl, tmo);
    };
    if (next && st.wait) {
        if (!waitf(st.wait_idx)) return false;
        if (L.kind == F_PRI && I.cold && L.slice > 0)
            x.theta = ipow(ldc(B.Gk_th + L.slice - 1), C.p);
    }
    if (sweep) {
        if (step == 0) {
            if (!waitf(flag_index(FL_F, L.kind == SWEEP_PRI ? 0 : C.Ntau))) return false;
            if (L.kind == SWEEP_PRI) x.theta = ldc(B.F_th);
        } else if (!waitf(flag_index(FL_F, sp_n))) {
            return false;
        }
        if (next && (I.cold || I.gk_lanes))
            if (!waitf(flag_index(I.cold ? FL_COLD : FL_GK, st.n))) return false;
    }
    const bool terms = L.kind == F_ADJ || L.kind == SWEEP_ADJ;
    // window 0: x of the finished solve, window 1: the operand tp of the next
    // right-hand side where it is another vector (a sweep's next input
    // u = x + F_n - G(u^k_n), a lane's first input)
    double zc[NR], t[NR], v[NR], bv[NR], vr[kRim], br[kRim];
    // states of the slice before this one extrapolate; differences that reach back
    // to the slice's given first state, which may be off in its rough modes, are
    // not used
    int order = 0;
    if (fine && next && C.extrap) order = step >= 2 ? 1 : 0;
    else if (fine && next && prev) order = max(0, min(min(step - 2, 3), x.ext_cap));
    x.order = order;
    // x0 = ca x + h, h the older states' part: loaded here with the others, so that
    // the round pays for one memory latency instead of one a state
    const double ca = (double)(order + 1);
    double h[NR], hr[kRim];
    if (order > 0) {
        g.load<NR>(xh(step - 1), g.fill, h);
        g.load_rim(xh(step - 1), hr);
        const double cb = order == 1 ? -1.0 : order == 2 ? -3.0 : -6.0;
        if (order > 1) {
            double a[NR], ar[kRim], a3[NR], a3r[kRim];
            // (a third state that the order does not use is read all the same)
            g.load<NR>(xh(step - 2), g.fill, a);
            g.load_rim(xh(step - 2), ar);
            g.load<NR>(xh(step - 3), g.fill, a3);
            g.load_rim(xh(step - 3), a3r);
            const double cd = order == 2 ? 1.0 : 4.0;
#pragma unroll
            for (int k = 0; k < NR; ++k) h[k] = cb * h[k] + cd * a[k] - (order > 2 ? a3[k] : 0.0);
#pragma unroll
            for (int i = 0; i < kRim; ++i)
                hr[i] = cb * hr[i] + cd * ar[i] - (order > 2 ? a3r[i] : 0.0);
        } else {
#pragma unroll
            for (int k = 0; k < NR; ++k) h[k] = cb * h[k];
#pragma unroll
            for (int i = 0; i < kRim; ++i) hr[i] = cb * hr[i];
        }
    }
    if (prev) {
        // own values of x from the thread's slots, the others as published
        g.load<NR>(xp, g.fill & ~g.own, v);
        g.load_rim(xp, vr);
        if (!terms) g.load<NR>(res_b(gv0, gvs, step), g.own & g.live, bv);
#pragma unroll
        for (int k = 0; k < NR; ++k) v[k] = is(g.own, k) ? lds[LX + k * kThreads] : v[k];
        if (sweep) {
            const double *Fp = L.kind == SWEEP_PRI ? B.S + (size_t)(C.M * (sp_n + 1) - 1) * Nn
                                                   : B.FL + (size_t)sp_n * Nn;
            const double *Gp = B.Gk + (size_t)sp_n * Nn;
            double fr[kRim], gr[kRim];
            g.load<NR>(Fp, g.fill, zc);
            g.load<NR>(Gp, g.fill, t);
            g.load_rim(Fp, fr);
            g.load_rim(Gp, gr);
#pragma unroll
            for (int k = 0; k < NR; ++k) zc[k] = v[k] + (zc[k] - t[k]);
#pragma unroll
            for (int i = 0; i < kRim; ++i) br[i] = vr[i] + (fr[i] - gr[i]);
            g.put<NR>(zlen, zc, br);
        }
        g.put<NR>(0, v, vr);
    } else {
        g.load<NR>(st.tp_src, g.fill, v);
        g.load_rim(st.tp_src, vr);
        g.put<NR>(zlen, v, vr);
#pragma unroll
        for (int i = 0; i < kRim; ++i) br[i] = vr[i];
    }
    lds_sync();
    if (prev && terms) {
        // terms of the elements right above the owned nodes; they wait in p's
        // slots until the residual has been accepted
        const double *Tr = B.S + (size_t)(sp_j - 1) * Nn;
        const double *Tp = sp_jprev > 0 ? B.S + (size_t)(sp_jprev - 1) * Nn : nullptr;
        const double *Gp = B.Gk + (size_t)sp_n * Nn;
        const double idl = fine ? C.inv_dt : C.inv_dtau;
        auto corner = [&](const double *row, int k, int dx) {
            const int y = g.gy0 + k;
            const bool in = g.act && g.gx >= 0 && g.gx + dx < W && y >= 0 && y < HN;
            return *nd(row, in ? (unsigned)(y * W + g.gx + dx) : 0u);
        };
        double ta[NR + 1], tb[NR + 1], pa[NR + 1], pb[NR + 1], dk[NR], dc[NR];
        unsigned e[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int y = g.gy0 + k;
            const bool el = is(g.own, k) && g.gx < C.nx && y < C.ny;
            e[k] = el ? (unsigned)(y * C.nx + g.gx) : 0u;
            dk[k] = *nd(B.dk, e[k]);
        }
#pragma unroll
        for (int k = 0; k <= NR; ++k) {
            ta[k] = corner(Tr, k, 0);
            tb[k] = corner(Tr, k, 1);
        }
        if (I.has_dc) {
#pragma unroll
            for (int k = 0; k < NR; ++k) dc[k] = *nd(B.dc, e[k]);
#pragma unroll
            for (int k = 0; k <= NR; ++k) {
                pa[k] = Tp ? corner(Tp, k, 0) : 0.0;
                pb[k] = Tp ? corner(Tp, k, 1) : 0.0;
            }
        }
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int z = cell0 + (k + 1) * sz;
            double l0 = lds[z], l1 = lds[z + 1], l2 = lds[z + sz + 1], l3 = lds[z + sz];
            if (sweep) {
                const int y = g.gy0 + k;
                const bool el = is(g.own, k) && g.gx < C.nx && y < C.ny;
                const unsigned id = el ? (unsigned)(y * W + g.gx) : 0u;
                const unsigned up = el ? id + W : 0u, dx = el ? 1u : 0u;
                l0 -= ldg(Gp, id);
                l1 -= ldg(Gp, id + dx);
                l2 -= ldg(Gp, up + dx);
                l3 -= ldg(Gp, up);
            }
            double term = dk[k] * elem_k(C, l0, l1, l2, l3, ta[k], tb[k], tb[k + 1], ta[k + 1]);
            if (I.has_dc)
                term += dc[k] * idl *
                        elem_c(C, l0, l1, l2, l3, ta[k] - pa[k], tb[k] - pb[k],
                               tb[k + 1] - pb[k + 1], ta[k + 1] - pa[k + 1]);
            lds[LP + k * kThreads] = term;
        }
    }
    if (prev) {
        // ---- the finished solve: true residual, norm -----------------------------
        if (terms) g.load<NR>(res_b(gv0, gvs, step), g.own & g.live, bv);
#pragma unroll
        for (int k = 0; k < NR; ++k) bv[k] = is(g.own & g.live, k) ? bv[k] : 0.0;
        res_apply<NR>(A, cell0, sz, bv, zc, t);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const double rv = is(g.live & g.own, k) ? t[k] - cc[k] * zc[k] : 0.0;
            sum[0] += rv * rv;
        }
        if (!is_adj) {
#pragma unroll
            for (int k = 0; k < NR; ++k) sum[1] += ipow(is(g.own, k) ? zc[k] : 0.0, C.p);
        }
    }
    if (next) {
        // ---- the next solve: b, x0, r0 --------------------------------------------
        // source
        if (st.adjoint) {
            const double ss = x.src_scale;
            g.load<NR>(B.S + (size_t)(st.j - 1) * Nn, g.live, bv);
#pragma unroll
            for (int k = 0; k < NR; ++k) bv[k] = ss * ipow(bv[k], C.p - 1);
        } else {
            const double f = B.qt[st.j] * C.quarter_area * (double)((g.gx > 0) + (g.gx < C.nx));
#pragma unroll
            for (int k = 0; k < NR; ++k)
                bv[k] = f * (double)((g.gy0 + k > 0) + (g.gy0 + k < C.ny));
        }
        {
            // + (C/delta) tp on the window
            const double ms = fine ? C.inv_dt : C.inv_dtau;
            const int z = (prev && !sweep ? 0 : zlen) + cell0;
            double ml[NR + 1], mr[NR + 1];
            if (I.has_dc) {
                const bool inx = g.act && g.gx >= 0 && g.gx < W;
#pragma unroll
                for (int k = 0; k <= NR; ++k) {
                    const int ey = g.gy0 + k;
                    const bool in = inx && ey >= 0 && ey <= C.ny + 1;
                    const unsigned e = in ? (unsigned)(ey * C.EW + g.gx) : 0u;
                    ml[k] = *nd(B.cm, e) * ms;
                    mr[k] = *nd(B.cm, e + (in ? 1u : 0u)) * ms;
                }
            } else {
                // c is the same everywhere: no loads
                const double m = *nd(B.cm, (unsigned)C.EW + 1u) * ms;
#pragma unroll
                for (int k = 0; k <= NR; ++k) {
                    const bool in = g.gy0 + k >= 1 && g.gy0 + k <= C.ny;
                    ml[k] = in && g.gx >= 1 ? m : 0.0;
                    mr[k] = in && g.gx < C.nx ? m : 0.0;
                }
            }
            res_mass<NR>(g, z, ml, mr, bv);
        }
        if (order > 0) {
            // residual of the plain start x0 = x: it judges the extrapolation
            res_apply<NR>(A, cell0, sz, bv, zc, t);
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                const double rv = is(g.live & g.own, k) ? t[k] - cc[k] * zc[k] : 0.0;
                sum[6] += rv * rv;
                v[k] = ca * zc[k] + h[k];
            }
            // (a row that only the set-up window holds has no node in zc's rows)
#pragma unroll
            for (int i = 0; i < kRim; ++i) vr[i] = ca * vr[i] + hr[i];
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
                g.load<NR>(st.x0_src, g.fill, v);
                g.load_rim(st.x0_src, vr);
                if (st.d1) {
                    double a[NR], ar[kRim];
                    g.load<NR>(st.d0, g.fill, a);
                    g.load_rim(st.d0, ar);
#pragma unroll
                    for (int k = 0; k < NR; ++k) v[k] += uc[k] - a[k];
#pragma unroll
                    for (int i = 0; i < kRim; ++i) vr[i] += br[i] - ar[i];
                }
            }
            if (!prev && sweep) {
                // what the sweep publishes of its input
                g.store<NR>(L.kind == SWEEP_PRI ? B.out_T + Nn
                                                : B.out_L + (size_t)(C.Ntau - 1) * Nn,
                            g.own, uc);
                if (is_adj) {
#pragma unroll
                    for (int k = 0; k < NR; ++k) uc[k] = 0.0;
                    g.store<NR>(B.out_L + (size_t)C.Ntau * Nn, g.own, uc);
                }
            }
        }
        if (!prev || sweep || order > 0) {
            lds_sync();
            g.put<NR>(0, v, vr);
            lds_sync();
        }
        res_apply<NR>(A, cell0, sz, bv, zc, t);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            t[k] = is(g.live, k) ? t[k] - cc[k] * zc[k] : 0.0;
            const double bo = is(g.own, k) ? bv[k] : 0.0, ro = is(g.own, k) ? t[k] : 0.0;
            sum[2] += bo * bo;
            sum[3] += ro * ro;
        }
    }
    if (prev) {
        // the finished x to its outputs and the history, behind the round's loads: a
        // load or a register reload issued after these stores would wait for them
#pragma unroll
        for (int k = 0; k < NR; ++k) v[k] = lds[LX + k * kThreads];
#pragma unroll
        for (int k = 0; k < NR; ++k)
            if (is(g.own, k)) stg(xp, g.id(k), v[k]);
        if (L.kind == F_PRI) {
            g.store<NR>(B.S + (size_t)(sp_j - 1) * Nn, g.own, v);
            if (C.plt && last) g.store<NR>(B.out_T + (size_t)(L.slice + 1) * Nn, g.own, v);
        } else if (L.kind == F_ADJ) {
            if (last) g.store<NR>(B.FL + (size_t)L.slice * Nn, g.own, v);
            if (C.plt && last) g.store<NR>(B.out_L + (size_t)(L.slice - 1) * Nn, g.own, v);
        } else {
            g.store<NR>((sweep ? B.Gn : B.Gk) + (size_t)sp_n * Nn, g.own, v);
        }
        if (sweep) {
            // (the slice-end slot of S, still read as F_n by the neighbours in this
            // round, follows after the barrier)
            const double *row = L.kind == SWEEP_PRI ? B.out_T + (size_t)(sp_n + 1) * Nn
                                                    : B.out_L + (size_t)(sp_n - 1) * Nn;
#pragma unroll
            for (int k = 0; k < NR; ++k) v[k] = lds[zlen + cell0 + (k + 1) * sz];
            g.store<NR>(row, g.own, v);
        }
    }
    if (next) {
        g.store<NR>(res_b(gv0, gvs, step + 1), g.own, bv);
        // x of the new solve (the finished x is in the history)
#pragma unroll
        for (int k = 0; k < NR; ++k) lds[LX + k * kThreads] = zc[k];
        lds_sync();  // both operand windows have been read
        if (g.act) {
#pragma unroll
            for (int k = 0; k < NR; ++k) lds[zlen + cell0 + (k + 1) * sz] = t[k];
        }
    }
#pragma unroll
    for (int k = 0; k < 7; ++k) x.sum[k] = sum[k];
    return true;
}

// ---- coarse-mesh lanes ---------------------------------------------------------
// The lanes of pt_cm_lane.hip with the solver of this file on the coarse mesh: the
// operator's registers are formed from the coarse element values, everything around
// the solves reads and writes the same rows. Bound by the rounds' latency as the
// others; 256^2, 32 slices, coarse steps on 129 x 129 nodes, cg_rtol 1e-12: 100 Jacobi
// rounds of 10.0 us per step -> 23 of 7.4 (degree 4), one warm cycle 74.2 -> 24.5 ms.

// The set-up of a coarse-mesh lane: as res_setup, with the step's input u restricted
// from fine states and the norm taken of the prolonged solution. A correction sweep's
// step needs F_n only for the next input u = x + R F_n - G(R u^k_n).
__device__ __forceinline__ int cm_step_slice(const Consts &C, const LaunchInfo &I, int kind,
                                             int slice, int s) {
    const bool adj = kind == CM_GK_ADJ || kind == CM_SWEEP_ADJ;
    if (kind == CM_GK_PRI || kind == CM_GK_ADJ) return slice;
    if (I.cold) return adj ? C.Ntau - s : s;
    return adj ? C.Ntau - 1 - s : s + 1;
}

template <int NR>
__device__ __forceinline__ bool res_setup_cm(const ResGeo &g, ResLaneCtx &x,
                                             const ResCoef<NR> &A, const double (&cc)[NR]) {
    extern __shared__ double lds[];
    auto is = [](unsigned m, int k) { return ResGeo::is(m, k); };
    const EngineDesc *Dp = x.D;
    const Consts C = fetch(&Dp->C);
    const Bufs B = fetch(&Dp->B);
    const LaunchInfo I = fetch(&Dp->I);
    const CoarseMesh M = fetch(&Dp->cm);
    const int kind = x.kind, step = x.step;
    const bool adj = kind == CM_GK_ADJ || kind == CM_SWEEP_ADJ;
    const bool gk = kind == CM_GK_PRI || kind == CM_GK_ADJ;
    const bool cold = !gk && I.cold, sweep = !gk && !cold;
    const bool prev = step > 0, next = step < x.nsteps;
    const int np = prev ? cm_step_slice(C, I, kind, x.slice, step - 1) : 0;
    const int n = cm_step_slice(C, I, kind, x.slice, next ? step : step - 1);
    const double *xp = res_x(x.gv0, x.gvs, step);
    const size_t Nn = C.Nn, Nc = M.Nc;
    const int sz = g.sz, zlen = g.zlen, cell0 = g.cell0, Wf = C.W, LX = g.slot_x<NR>();
    double sum[7] = {0, 0, 0, 0, 0, 0, 0};

    auto waitf = [&](int fk, int k) {
        return wait_flag(B.flags, flag_index(fk, k), I.epoch, B.ctl, C.timeout_ticks);
    };
    if (sweep) {
        if (!waitf(FL_F, prev ? np : adj ? C.Ntau : 0)) return false;
        if (!prev && !adj) x.theta = ldc(B.F_th);
        if (next && I.gk_lanes && !waitf(FL_GK, n)) return false;
    }
    // the fine state of an input, the guess u^k_n and the batched output of a slice
    auto state = [&](int k) {
        return adj ? B.FL + (size_t)k * Nn : B.S + (size_t)(C.M * (k + 1) - 1) * Nn;
    };
    auto guess = [&](int k) { return (adj ? B.in_L : B.in_T) + (size_t)k * Nn; };
    auto row = [&](int k) { return M.Gk + (size_t)k * Nc; };
    double zc[NR], t[NR], v[NR], u[NR], bv[NR], vr[kRim], ur[kRim];
    if (prev) {
        g.load<NR>(xp, g.fill & ~g.own, v);
        g.load_rim(xp, vr);
        g.load<NR>(res_b(x.gv0, x.gvs, step), g.own & g.live, bv);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            v[k] = is(g.own, k) ? lds[LX + k * kThreads] : v[k];
            bv[k] = is(g.own & g.live, k) ? bv[k] : 0.0;
        }
        g.put<NR>(0, v, vr);
    } else {
#pragma unroll
        for (int k = 0; k < NR; ++k) v[k] = 0.0;
#pragma unroll
        for (int i = 0; i < kRim; ++i) vr[i] = 0.0;
    }
    // u in window 1
    if (cold) {
#pragma unroll
        for (int k = 0; k < NR; ++k) u[k] = v[k];
#pragma unroll
        for (int i = 0; i < kRim; ++i) ur[i] = vr[i];
    } else {
        const double *in = sweep ? state(prev ? np : adj ? C.Ntau : 0) : guess(n);
        g.load_fine<NR>(in, Wf, g.fill, u);
        g.load_rim_fine(in, Wf, ur);
        if (sweep && prev) {
            double a[NR], ar[kRim];
            g.load<NR>(row(np), g.fill, a);
            g.load_rim(row(np), ar);
#pragma unroll
            for (int k = 0; k < NR; ++k) u[k] = v[k] + (u[k] - a[k]);
#pragma unroll
            for (int i = 0; i < kRim; ++i) ur[i] = vr[i] + (ur[i] - ar[i]);
        }
    }
    if (next) g.put<NR>(zlen, u, ur);
    lds_sync();
    if (prev) {
        res_apply<NR>(A, cell0, sz, bv, zc, t);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const double rv = is(g.live & g.own, k) ? t[k] - cc[k] * zc[k] : 0.0;
            sum[0] += rv * rv;
        }
        if (!adj) {
            // the fine nodes of an owned node and of the edges and the cell right
            // and above it
            unsigned char mk[NR][4];
#pragma unroll
            for (int k = 0; k < NR; ++k)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int fx = 2 * g.gx + (q & 1), fy = 2 * (g.gy0 + k) + (q >> 1);
                    const bool in = is(g.own, k) && fx <= C.nx && fy <= C.ny;
                    const unsigned char m = *ndb(B.mask, in ? (unsigned)(fy * Wf + fx) : 0u);
                    mk[k][q] = in ? m : 1;
                }
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                const int z = cell0 + (k + 1) * sz;
                const double a = lds[z], b = lds[z + 1], c = lds[z + sz], d = lds[z + sz + 1];
                const double pv[4] = {a, 0.5 * a + 0.5 * b, 0.5 * a + 0.5 * c,
                                      0.25 * a + 0.25 * b + 0.25 * c + 0.25 * d};
#pragma unroll
                for (int q = 0; q < 4; ++q) sum[1] += mk[k][q] ? 0.0 : ipow(pv[q], C.p);
            }
        }
    }
    if (next) {
        // ---- b, x0, r0 -------------------------------------------------------------
        if (!adj) {
            const double qn = B.qt[C.M * (n + 1)];
            g.load<NR>(M.fc, g.live, bv);
#pragma unroll
            for (int k = 0; k < NR; ++k) bv[k] *= qn;
        } else {
            // P^T of the fine source: weights 1, 1/2, 1/4 of the fine nodes around
            const double *Tm = B.S + (size_t)(C.M * (n - 1)) * Nn;
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                double tv[9];
                unsigned char mk[9];
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    const int fx = 2 * g.gx + q % 3 - 1, fy = 2 * (g.gy0 + k) + q / 3 - 1;
                    const bool in = is(g.live, k) && fx >= 0 && fx <= C.nx && fy >= 0 &&
                                    fy <= C.ny;
                    const unsigned id = in ? (unsigned)(fy * Wf + fx) : 0u;
                    tv[q] = ldg(Tm, id);
                    const unsigned char m = *ndb(B.mask, id);
                    mk[q] = in ? m : 1;
                }
                double sv = 0.0;
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    const double w = (q % 3 == 1 ? 1.0 : 0.5) * (q / 3 == 1 ? 1.0 : 0.5);
                    sv += mk[q] ? 0.0 : w * (x.src_scale * ipow(tv[q], C.p - 1));
                }
                bv[k] = sv;
            }
        }
        {
            double ml[NR + 1], mr[NR + 1];
            g.cm_mass<NR>(C, M, ml, mr);
            res_mass<NR>(g, zlen + cell0, ml, mr, bv);
        }
        // x0: the input, in a correction sweep G(R u^k_n) + (u - R u^k_n)
        if (sweep) {
            double a[NR], ar[kRim];
            g.load<NR>(row(n), g.fill, v);
            g.load_rim(row(n), vr);
            g.load_fine<NR>(guess(n), Wf, g.fill, a);
            g.load_rim_fine(guess(n), Wf, ar);
#pragma unroll
            for (int k = 0; k < NR; ++k) v[k] += u[k] - a[k];
#pragma unroll
            for (int i = 0; i < kRim; ++i) vr[i] += ur[i] - ar[i];
        } else {
#pragma unroll
            for (int k = 0; k < NR; ++k) v[k] = u[k];
#pragma unroll
            for (int i = 0; i < kRim; ++i) vr[i] = ur[i];
        }
        lds_sync();
        g.put<NR>(0, v, vr);
        lds_sync();
        res_apply<NR>(A, cell0, sz, bv, zc, t);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            t[k] = is(g.live, k) ? t[k] - cc[k] * zc[k] : 0.0;
            const double bo = is(g.own, k) ? bv[k] : 0.0, ro = is(g.own, k) ? t[k] : 0.0;
            sum[2] += bo * bo;
            sum[3] += ro * ro;
        }
    }
    if (prev) {
#pragma unroll
        for (int k = 0; k < NR; ++k) v[k] = lds[LX + k * kThreads];
        double *out = (sweep ? M.Gn : M.Gk) + (size_t)np * Nc;
#pragma unroll
        for (int k = 0; k < NR; ++k)
            if (is(g.own, k)) {
                stg(xp, g.id(k), v[k]);
                stg(out, g.id(k), v[k]);
            }
    }
    if (next) {
        g.store<NR>(res_b(x.gv0, x.gvs, step + 1), g.own, bv);
#pragma unroll
        for (int k = 0; k < NR; ++k) lds[LX + k * kThreads] = zc[k];
        lds_sync();
        if (g.act) {
#pragma unroll
            for (int k = 0; k < NR; ++k) lds[zlen + cell0 + (k + 1) * sz] = t[k];
        }
    }
#pragma unroll
    for (int k = 0; k < 7; ++k) x.sum[k] = sum[k];
    return true;
}

// theta, outputs and flags of a finished coarse-mesh solve (Alg. 1 with dtau and N_tau)
__device__ __forceinline__ void res_commit_cm(ResLaneCtx &x, double pn, double relres) {
    const EngineDesc *Dp = x.D;
    const Consts C = fetch(&Dp->C);
    const Bufs B = fetch(&Dp->B);
    const LaunchInfo I = fetch(&Dp->I);
    const int kind = x.kind, n = cm_step_slice(C, I, kind, x.slice, x.step - 1);
    const bool gk = kind == CM_GK_PRI || kind == CM_GK_ADJ;
    if (kind == CM_GK_PRI || kind == CM_SWEEP_PRI) {
        const double thG = pow_call(ipow(x.theta, C.p) + pn * C.inv_NtauNe, C.inv_p);
        x.theta = thG;
        if (gk || I.cold) {
            if (x.leader) B.Gk_th[n] = thG;
        } else {
            x.theta = thG + ldc(B.F_th + n) - ldc(B.Gk_th + n);
            if (x.leader) {
                B.Gn_th[n] = thG;
                B.out_th[n + 1] = x.theta;
            }
        }
    }
    if (x.leader) {
        if (!isfinite(relres)) set_status(B.ctl, -5);
        if (gk) set_flag(B.flags, flag_index(FL_GK, n), I.epoch);
        if (x.step - 1 < x.trace_steps)
            x.trec[TR_HDR + x.step - 1] = (unsigned long long)now_ticks();
    }
}

// The true residual of the finished solve again, x taken back from the history:
// left at the owned nodes' cells of window 1.
template <int NR>
__device__ __forceinline__ void res_residual(const ResGeo &geo, ResLaneCtx &x, const ResCoef<NR> &A,
                                             const double (&cc)[NR]) {
    extern __shared__ double lds[];
    const ResGeo g = geo;
    const EngineDesc *Dp = x.D;
    const Consts C = fetch(&Dp->C);
    const Bufs B = fetch(&Dp->B);
    const int step = x.step, kind = x.kind;
    const double *gv0 = x.gv0;
    const size_t gvs = x.gvs;
    const double *xp = res_x(gv0, gvs, step);
    double zc[NR], t[NR], v[NR], vr[kRim];
    g.load<NR>(xp, g.fill | g.own, v);
    g.load_rim(xp, vr);
    const int LX = g.slot_x<NR>();
#pragma unroll
    for (int k = 0; k < NR; ++k) lds[LX + k * kThreads] = v[k];
    g.put<NR>(0, v, vr);
    g.load<NR>(res_b(gv0, gvs, step), g.own & g.live, v);
    lds_sync();
    res_apply<NR>(A, g.cell0, g.sz, v, zc, t);
    if (g.act) {
#pragma unroll
        for (int k = 0; k < NR; ++k)
            lds[g.zlen + g.cell0 + (k + 1) * g.sz] =
                ResGeo::is(g.live & g.own, k) ? t[k] - cc[k] * zc[k] : 0.0;
    }
}

// Books the finished solve after its residual has been accepted: sensitivity
// sums, the corrected slice end, theta (pn: the group's ||x||_p^p), flags.
template <int NR>
__device__ __forceinline__ void res_commit(const ResGeo &geo, ResLaneCtx &x, double pn) {
    extern __shared__ double lds[];
    const ResGeo g = geo;
    auto is = [](unsigned m, int k) { return ResGeo::is(m, k); };
    const EngineDesc *Dp = x.D;
    const Consts C = fetch(&Dp->C);
    const Bufs B = fetch(&Dp->B);
    const int kind = x.kind, slice = x.slice, step = x.step;
    const int n = x.sp_n;
    const bool fine = kind == F_PRI || kind == F_ADJ, last = step == x.nsteps;
    const bool leader = x.leader;
    if (kind == F_ADJ || kind == SWEEP_ADJ) {
        const double *ac = fine ? B.acc + (size_t)(slice - 1) * C.Ne : B.accG;
        const int LP = g.slot_p<NR>();
        auto el = [&](int k) { return is(g.own, k) && g.gx < C.nx && g.gy0 + k < C.ny; };
        auto eid = [&](int k) { return (unsigned)((g.gy0 + k) * C.nx + g.gx); };
        double a[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) a[k] = step > 1 ? *nd(ac, el(k) ? eid(k) : 0u) : 0.0;
#pragma unroll
        for (int k = 0; k < NR; ++k)
            if (el(k)) *nd(ac, eid(k)) = a[k] + lds[LP + k * kThreads];
    }
    if (kind == SWEEP_PRI) {
        double u[NR];
        const double *row = B.out_T + (size_t)(n + 1) * C.Nn;
#pragma unroll
        for (int k = 0; k < NR; ++k) u[k] = *nd(row, is(g.own, k) ? g.id(k) : 0u);
        g.store<NR>(B.S + (size_t)(C.M * (n + 1) - 1) * C.Nn, g.own, u);
    }
    if (!is_adjoint_kind(kind)) {
        double theta = x.theta;
        if (fine) {
            theta += pn * C.inv_NtNe;
            if (leader && last) B.F_th[slice] = C.plt ? theta : pow_call(theta, C.inv_p);
        } else {
            const double thG = pow_call(ipow(theta, C.p) + pn * C.inv_NtauNe, C.inv_p);
            theta = thG;
            if (kind == SWEEP_PRI) {
                theta = thG + ldc(B.F_th + n) - ldc(B.Gk_th + n);
                if (leader) {
                    B.out_th[n + 1] = theta;
                    B.Gn_th[n] = thG;
                }
            } else if (leader) {
                B.Gk_th[n] = thG;
            }
        }
        x.theta = theta;
    }
    if (leader) {
        const unsigned epoch = fetch(&Dp->I).epoch;
        if (kind == GK_PRI || kind == GK_ADJ) set_flag(B.flags, flag_index(FL_GK, n), epoch);
        if (kind == COLD_PRI || kind == COLD_ADJ) set_flag(B.flags, flag_index(FL_COLD, n), epoch);
        if (fine && last) set_flag(B.flags, flag_index(FL_F, slice), epoch);
        if (step - 1 < x.trace_steps) x.trec[TR_HDR + step - 1] = (unsigned long long)now_ticks();
    }
}

// Runs lane L of design *Dp on this workgroup's group (rank of g workgroups);
// returns false when a wait timed out or another workgroup aborted, alike in
// every workgroup.
// CM: L is a coarse-mesh lane, the grid the coarse mesh's.
template <int NR, bool TIMED, bool SPLIT, bool CM = false>
__device__ __forceinline__ bool res_lane(const EngineDesc *Dp, const Lane L, const Launch &S,
                                         const Group &G, unsigned *bar, double *part,
                                         unsigned &nbar, unsigned long long *trec, double *red) {
    extern __shared__ double lds[];
    __shared__ double om_s[kResMaxDeg + 1];
    __shared__ double tot_s[kResSums];
    const int rank = blockIdx.x - G.wg0, g = G.nwg;
    const int tid = threadIdx.x;
    const bool leader = rank == 0 && tid == 0;
    const bool is_adj =
        CM ? L.kind == CM_GK_ADJ || L.kind == CM_SWEEP_ADJ : is_adjoint_kind(L.kind);
    const bool fine = L.kind == F_PRI || L.kind == F_ADJ;
    ResGeo q;
    ResLaneCtx x;
    Control *ctl;
    long long tmo;
    double rtol, stop;
    int max_iter, coarse_iters, max_restarts;
    bool verify;
    int rows;
    {
        const Consts C = fetch(&Dp->C);
        const Bufs B = fetch(&Dp->B);
        const LaunchInfo I = fetch(&Dp->I);
        ctl = B.ctl;
        tmo = C.timeout_ticks;
        rtol = C.rtol;
        max_iter = C.max_iter;
        coarse_iters = fine || CM ? 0 : C.coarse_iters;
        verify = CM || C.verify || C.fp32;
        stop = rtol * (fine ? kStopFine : kStopCoarse);
        max_restarts = !CM && C.fp32 ? C.max_restarts : kResRestarts;
        x.D = Dp;
        x.gv0 = group_vec(B, G.vec, V_R0);
        x.gvs = B.pool_stride;
        x.trec = trec;
        x.kind = L.kind;
        x.slice = L.slice;
        x.trace_steps = S.trace_stride - TR_HDR;
        x.trunc = coarse_iters > 0;
        x.leader = leader;
        x.step = 0;
        if constexpr (CM)
            x.nsteps = L.kind == CM_GK_PRI || L.kind == CM_GK_ADJ ? 1
                                                                   : C.Ntau - (I.cold ? 0 : 1);
        else
            x.nsteps = lane_steps(C, L.kind);
        x.sp_n = x.sp_j = x.sp_jprev = x.st_n = x.st_j = x.st_jprev = 0;
        x.order = 0;
        x.ext_cap = 1;
        x.theta = x.src_scale = 0.0;
        if (is_adj) {
            const double Th = *B.Theta;
            x.src_scale = C.plt ? (double)C.p / (double)C.Ne
                                : pow_call(Th, 1.0 - C.p) / (double)C.Ne;
            if (!(Th > 0.0) || !isfinite(Th)) set_status(ctl, -5);
        }
        if (L.kind == F_PRI) {
            if (L.slice > 0 && !I.cold && !C.plt) x.theta = ipow(B.in_th[L.slice], C.p);
        } else if (L.kind == GK_PRI || L.kind == CM_GK_PRI) {
            x.theta = B.in_th[L.slice];
        }
        // geometry: owned rectangle, window, this thread's column and rows
        int W = C.W, HN = C.ny + 1;
        if constexpr (CM) {
            const CoarseMesh M = fetch(&Dp->cm);
            W = M.Wc;
            HN = M.nyc + 1;
        }
        // a coarse node is fixed iff its fine node is
        auto fixed = [&](int y, int gx) {
            return B.mask[CM ? (size_t)(2 * y) * C.W + 2 * gx : (size_t)y * W + gx] != 0;
        };
        const int deg = coarse_iters > 0 ? 0 : L.deg;
        const int TX = (W + L.tw - 1) / L.tw, TY = (HN + L.th - 1) / L.th;
        const int hx = TX > 1 ? deg + 1 : 0, hy = TY > 1 ? deg + 1 : 0;
        const int wc = L.tw + 2 * hx, wr = L.th + 2 * hy;
        const int nq = min(kThreads / wc, (wr + NR - 1) / NR);
        rows = nq * NR;
        const int tq = tid / wc;
        const int tx = rank % TX, ty = rank / TX;  // ty >= TY: nothing owned
        const int ox0 = tx * L.tw, oy0 = ty * L.th;
        const int ox1 = min(ox0 + L.tw, W), oy1 = min(oy0 + L.th, HN);
        q.act = tq < nq;
        const int col = q.act ? tid - tq * wc : 0, row0 = q.act ? tq * NR : 0;
        q.W = W;
        q.sz = wc + 2;
        q.zlen = q.sz * (rows + 2);
        q.cell0 = row0 * q.sz + col + 1;
        q.gx = ox0 - hx + col;
        q.gy0 = oy0 - hy + row0;
        q.live = q.fill = q.own = q.edge = q.edge1 = 0;
        const bool inx = q.act && q.gx >= 0 && q.gx < W && ty < TY;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int y = q.gy0 + k, row = row0 + k;
            if (!inx || y < 0 || y >= HN || row > wr) continue;
            const bool free_ = !fixed(y, q.gx);
            if (free_) q.fill |= 1u << k;
            if (row >= wr) continue;
            if (free_) q.live |= 1u << k;
            if (q.gx >= ox0 && q.gx < ox1 && y >= oy0 && y < oy1) {
                q.own |= 1u << k;
                auto near = [&](int h) {
                    return (tx > 0 && q.gx - ox0 < h) || (tx < TX - 1 && ox1 - q.gx <= h) ||
                           (ty > 0 && y - oy0 < h) || (ty < TY - 1 && oy1 - y <= h);
                };
                if (near(deg + 1)) q.edge |= 1u << k;
                if (near(deg + 2)) q.edge1 |= 1u << k;
            }
        }
#pragma unroll
        for (int i = 0; i < kRim; ++i) {
            const int e = tid + i * kThreads;
            int cx, cy;
            if (e < 2 * q.sz) {
                cx = e < q.sz ? e : e - q.sz;
                cy = e < q.sz ? 0 : rows + 1;
            } else {
                cx = (e & 1) ? q.sz - 1 : 0;
                cy = 1 + ((e - 2 * q.sz) >> 1);
            }
            const int gx = ox0 - hx - 1 + cx, gy = oy0 - hy - 1 + cy;
            const bool in = e < 2 * q.sz + 2 * rows && gx >= 0 && gx < W && gy >= 0 && gy < HN &&
                            cy <= wr + 1 && ty < TY;
            q.rim_id[i] = in && !fixed(gy, gx) ? gy * W + gx : -1;
            q.rim_cell[i] = cy * q.sz + cx;
        }
        // (a coarse element's quotient k/m lies between a quarter of the least and of
        // the largest fine one: its k and c are means, its area four times theirs)
        const double ms = (fine ? C.inv_dt : C.inv_dtau) * (CM ? 4.0 : 1.0);
        double lo, hi;
        res_bounds(C, __longlong_as_double((long long)ctl->kmin_bits) / ms,
                   __longlong_as_double((long long)ctl->kmax_bits) / ms, lo, hi);
        lds_sync();
        if (tid <= deg) om_s[tid] = res_omega(lo, hi, deg, tid);
        // operand windows: every cell outside the grid stays 0; p and x slots
        for (int c = tid; c < 2 * q.zlen + 2 * NR * kThreads; c += kThreads) lds[c] = 0.0;
        lds_sync();
    }
    const bool trunc = coarse_iters > 0;
    const int deg = trunc ? 0 : L.deg;
    const int cell0 = q.cell0, sz = q.sz, zlen = q.zlen, W = q.W;
    const int LP = q.slot_p<NR>(), LX = q.slot_x<NR>();
    const unsigned live = q.live, own = q.own, edge = q.edge, edge1 = q.edge1;
    const bool act = q.act;
    const int n0 = q.gy0 * W + q.gx;
    const double *gv0 = x.gv0;
    const size_t gvs = x.gvs;
    const int nsteps = x.nsteps;
    auto id_of = [&](int k) { return (unsigned)(fresh(n0) + k * W); };
    auto is = [](unsigned m, int k) { return ResGeo::is(m, k); };
    ResCoef<NR> A;
    double dinv[NR], cc[NR], r[NR], s[NR], w[NR];

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
    // this workgroup's Q sums to its partial slots of the coming barrier
    auto put_sums = [&](auto &v) {
        constexpr int Q = sizeof(v) / sizeof(double);
        const int t = fresh(tid), wave = t >> 6;
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const double y = wave_sum(v[k]);
            if ((t & 63) == 0) red[k * kWaves + wave] = y;
        }
        lds_sync();
        if (t < Q) {
            double y = 0.0;
#pragma unroll
            for (int k = 0; k < kWaves; ++k) y += red[t * kWaves + k];
            stc(part + ((size_t)(nbar & 1) * kResSums + t) * kResGroup + rank, y);
        }
    };
    // the group's sums after the barrier: wave k adds component k
    auto get_sums = [&](auto &v) {
        constexpr int Q = sizeof(v) / sizeof(double);
        const int t = fresh(tid), wave = t >> 6, ln = t & 63;
        if (wave < Q) {
            const double *p = part + ((size_t)((nbar - 1) & 1) * kResSums + wave) * kResGroup;
            double y = 0.0;
            for (int k = ln; k < g; k += 64) y += ldc(p + k);
            y = wave_sum(y);
            if (ln == 0) tot_s[wave] = y;
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
            const double u = is(own, k) ? zc[k] : 0.0;
            w[k] = is(live, k) ? cc[k] * zc[k] - t[k] : 0.0;
            gam += r[k] * u;
            del += u * w[k];
        }
    };
    auto publish_w = [&]() {
        const double *P = res_w(gv0, gvs, nbar);
#pragma unroll
        for (int k = 0; k < NR; ++k)
            if (is(edge, k)) stg(P, id_of(k), w[k]);
    };
    // w of the window's other nodes, published in the round of the last barrier
    auto halo_w = [&]() {
        const double *P = res_w(gv0, gvs, nbar - 1);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const bool in = is(live & ~own, k);
            const double v = ldg(P, in ? id_of(k) : 0u);
            w[k] = in ? v : w[k];
        }
    };
    auto publish_x = [&](int j) {
        const double *row = res_x(gv0, gvs, j);
#pragma unroll
        for (int k = 0; k < NR; ++k)
            if (is(edge1, k)) stg(row, id_of(k), lds[LX + k * kThreads]);
    };

    const unsigned nbar0 = nbar;
    unsigned long long iters_all = 0;
    int iters_max = 0;
    long long relres_max = 0;  // as double bits, so that a NaN counts as the largest
    if (leader) {
        trec[TR_KIND] = L.kind;
        trec[TR_SLICE] = L.slice;
        trec[TR_NWG] = g;
        trec[TR_TILE] = L.tw * L.th;
        trec[TR_SHAPE] = (unsigned long long)(NR + 256 * deg);
        trec[TR_START] = (unsigned long long)now_ticks();
    }

    {
        const Consts C = fetch(&Dp->C);
        const Bufs B = fetch(&Dp->B);
        const double *dg = fine ? B.dinv_f : B.dinv_c;
        if constexpr (CM) {
            const CoarseMesh M = fetch(&Dp->cm);
            q.cm_coefs<NR>(C, M, A, cc);
            dg = M.dinv;
        } else {
            q.coefs<NR>(C, B, fine, A, cc);
        }
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const double d = *nd(dg, is(live, k) ? id_of(k) : 0u);
            dinv[k] = is(live, k) ? d : 0.0;
        }
    }
    int step = 0;
    double bnorm = 0.0, relres = 0.0, rnorm = 0.0, alpha = 0.0, beta = 0.0, gamma = 0.0;
    int iter = 0, restarts = 0;
    bool capped = false, restart = false;
    for (;;) {
        // ---- set-up or restart, then the first u, w and sums ------------------------
        const bool prev = step > 0, last = prev && step == nsteps;
        double sum[3] = {0.0, 0.0, 0.0};  // (r, u), (u, w), (r, r)
        x.step = step;
        if (!restart) {
            if constexpr (CM) {
                if (!res_setup_cm<NR>(q, x, A, cc)) return false;
            } else {
                if (!res_setup<NR, TIMED>(q, x, A, cc, tm)) return false;
            }
        } else {
            res_residual<NR>(q, x, A, cc);
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                const double v = lds[zlen + cell0 + (k + 1) * sz];
                w[k] = act ? v : 0.0;
                sum[2] += w[k] * w[k];
            }
            // the residual's owned values cross to the neighbours' windows
            publish_w();
            if (!barrier(false)) return false;
            halo_w();
            if (act) {
#pragma unroll
                for (int k = 0; k < NR; ++k) lds[zlen + cell0 + (k + 1) * sz] = w[k];
            }
        }
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const double v = lds[zlen + cell0 + (k + 1) * sz];
            r[k] = is(live, k) ? v : 0.0;
            s[k] = w[k] = 0.0;
        }
        zc_buf = 0;
        if (!last || restart) {
            precond(sum[0], sum[1]);
            publish_w();
        }
        bool closed = false;  // x of the current solve is final
        if (!restart) {
            double tot[7];
#pragma unroll
            for (int k = 0; k < 7; ++k) tot[k] = x.sum[k];
            tot[4] = sum[0];
            tot[5] = sum[1];
            put_sums(tot);
            // release: rows that other lanes read once this round's flags are set
            if (!barrier(prev && (last || L.kind == COLD_PRI || L.kind == COLD_ADJ))) return false;
            if (!last) halo_w();
            get_sums(tot);
            if (prev && !trunc && !capped && bnorm > 0.0 && verify) {
                // the true residual decides
                const double rn = sqrt(tot[0]);
                relres = rn / bnorm;
                if (!(rn <= rtol * bnorm)) {
                    if (restarts < max_restarts && iter < max_iter) {
                        ++restarts;
                        restart = true;
                        continue;
                    }
                    if (leader) set_status(ctl, -4);
                }
            }
            if (prev) {
                if constexpr (CM) res_commit_cm(x, tot[1], relres);
                else res_commit<NR>(q, x, tot[1]);
                iters_all += iter;
                iters_max = max(iters_max, iter);
                relres_max = max(relres_max, __double_as_longlong(relres));
            } else if (leader && (CM ? L.kind == CM_SWEEP_PRI && !fetch(&Dp->I).cold
                                     : L.kind == SWEEP_PRI)) {
                fetch(&Dp->B).out_th[1] = x.theta;
            }
            if (last) break;
            // ---- the next solve becomes the current one --------------------------
            x.ext_cap = x.order == 0 ? 1 : tot[3] > tot[6] ? x.order - 1 : x.order + 1;
            x.sp_n = x.st_n;
            x.sp_j = x.st_j;
            x.sp_jprev = x.st_jprev;
            ++step;
            iter = restarts = 0;
            capped = false;
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
                for (int k = 0; k < NR; ++k) lds[LX + k * kThreads] = 0.0;
            } else {
                // (an extrapolated start is never the solution: its error has the same
                // sign at every step)
                closed = x.order > 0 ? rnorm == 0.0 : rnorm <= rtol * bnorm;
            }
        } else {
            put_sums(sum);
            if (!barrier(false)) return false;
            halo_w();
            get_sums(sum);
            rnorm = sqrt(sum[2]);
            gamma = sum[0];
            alpha = sum[0] / sum[1];
            restart = false;
        }
        // ---- the rounds of CG, a loop of its own: what only the set-up needs is kept
        // out of its registers --------------------------------------------------------
        beta = 0.0;
#pragma unroll
        for (int k = 0; k < NR; ++k) lds[LP + k * kThreads] = 0.0;
        bool shown = false;
        while (!closed) {
            // s = w + beta s, p = u + beta p, x += alpha p, r -= alpha s (p and x
            // of nodes that are not owned are formed too, and never read)
            sum[0] = sum[1] = sum[2] = 0.0;
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                const double u = lds[zc_buf * zlen + cell0 + (k + 1) * sz];
                const double p0 = lds[LP + k * kThreads], x0 = lds[LX + k * kThreads];
                s[k] = w[k] + beta * s[k];
                const double pn = u + beta * p0;
                lds[LP + k * kThreads] = pn;
                lds[LX + k * kThreads] = x0 + alpha * pn;
                r[k] -= alpha * s[k];
                const double ro = is(own, k) ? r[k] : 0.0;
                sum[2] += ro * ro;
            }
            precond(sum[0], sum[1]);
            publish_w();
            // near the end x's edge goes out too, so that the round that closes the
            // solve can start at once (a round gains about a decimal digit)
            ++iter;
            shown = trunc ? iter >= coarse_iters
                          : rnorm <= 200.0 * stop * bnorm || iter >= max_iter;
            if (shown) publish_x(step);
            put_sums(sum);
            if (!barrier(false)) return false;
            halo_w();
            get_sums(sum);
            rnorm = sqrt(sum[2]);
            if (trunc ? (iter >= coarse_iters || rnorm == 0.0)
                      : (rnorm <= stop * bnorm || iter >= max_iter)) {
                relres = bnorm > 0.0 ? rnorm / bnorm : 0.0;
                capped = !trunc && !(rnorm <= rtol * bnorm);
                if (capped && rnorm > rtol * bnorm && leader) set_status(ctl, -4);
                closed = true;
            } else {
                beta = sum[0] / gamma;
                alpha = sum[0] / (sum[1] - beta * sum[0] / alpha);
                gamma = sum[0];
            }
        }
        if (!shown) {
            publish_x(step);
            if (!barrier(false)) return false;
        }
    }
    if (leader) {
        atomicAdd(fine ? &ctl->iters_fine : &ctl->iters_coarse, iters_all);
        atomicAdd(fine ? &ctl->solves_fine : &ctl->solves_coarse, (unsigned long long)nsteps);
        atomicMax(&ctl->max_iters, iters_max);
        atomicMax(&ctl->max_relres_bits, (unsigned long long)relres_max);
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
        const EngineDesc *E = D + (MULTI ? L.design : 0);
        ctl = E->B.ctl;
        if constexpr (CMESH) {
            if (is_cm_kind(L.kind)) {
                if (L.nr <= 2)
                    ok = res_lane<2, false, false, true>(E, L, S, G, bar, part, nbar, trec, red);
                else if (L.nr <= 4)
                    ok = res_lane<4, false, false, true>(E, L, S, G, bar, part, nbar, trec, red);
                else
                    ok = res_lane<6, false, false, true>(E, L, S, G, bar, part, nbar, trec, red);
                continue;
            }
        }
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
