// The finite-difference form of Sec. III, one read and one write of every
// population per step.
//
// The fused kernel (k_fd_step in kernels.hip) reads each population's upwind
// neighbours from cache.  The rows around the cells in flight on one XCD,
// over all 2Q planes, exceed its L2, so neighbour rows are fetched from HBM
// again and again.  Here a step works from a per-cell record instead (the
// macroscopic state of the time-n populations, and kappa rho of the
// energy-conserving collision), with which populations can be updated plane
// by plane.  Two kernels do that:
//
//   k_fd_tile    FP64, grids of some size (fd_tiles): a workgroup walks a
//                tile of cells through all planes, each plane's tile and its
//                stencil's halo in LDS; the new populations' moment sums stay
//                in registers and become the next record.  One launch a step.
//   k_fd_update  FP32, and FP64 on small grids and those of one plane: one lane
//                per cell, a chunk of populations per launch, neighbours read
//                through L1/L2, the moment sums passed on from chunk to chunk
//                in memory.  It has more waves, each with a shorter chain of
//                planes.  With rows of whole 256-cell tiles in FP32, and in 3D
//                FP64 with more than a workgroup a CU, k_fd_update_lds instead,
//                which stages each population's stencil rows in LDS.
//
// (FP32 keeps the chunks' order of sums.  k_fd_tile sums pairs, from the last
// population to the first; FP32 in such tiles took 6.4 ms against 10.2 a step at
// 256^3, but moved the deviations' last bits: the velocity's error against FP64
// after six steps 2.6e-7, 2.3e-7 in chunks.  Tiles that walk the populations in
// the chunks' order and keep their partial sums are not built.)
//
// The first record is made with the initial state (k_fd_init), and from the
// populations (k_fd_moments) only after a fused step.
//
// The scheme is that of the fused kernel: the same equilibrium, the same
// exact-moment correction of the targets in deviation storage, the same
// relaxation and convection terms; the kernels agree to rounding.
#include <type_traits>

#include "lbm_internal.h"
#include "step_core.h"

namespace lbm {
namespace {

using namespace core;

// Record of k_fd_update.  Its fields, each a plane (stride P, the population planes' stride) of
// values in the arithmetic type:
//   0 drho (deviation storage) or rho; 1..D u; D+1 t = T - 1; D+2 kappa rho;
//   deviation storage only: D+3 dm_g, D+4 .. 2D+3 dj_g, 2D+4 de_g, 2D+5 dm_h.
template <int D, bool DEV>
constexpr int kRecFields = DEV ? 2 * D + 6 : D + 3;
// After the record: the running moment sums of the new state, s0, sj (D),
// se and sh (sum of h), accumulated chunk by chunk.
template <int D>
constexpr int kAccFields = D + 3;

// Population chunks of the update passes: the rest and axis populations
// (which take the correction) with the first pairs, then 21 at a time in 3D
// (6 launches) and the other 24 in 2D (2 launches).
template <int D>
constexpr int kChunk0 = D == 2 ? 13 : 15;
template <int D>
constexpr int kChunkW = D == 2 ? 24 : 21;
template <int D>
constexpr int chunk_count() {
    constexpr int Q = VelSet<D>::Q;
    return 1 + (Q - kChunk0<D> + kChunkW<D> - 1) / kChunkW<D>;
}
template <int D>
constexpr int chunk_begin(int c) { return c == 0 ? 0 : kChunk0<D> + (c - 1) * kChunkW<D>; }
template <int D>
constexpr int chunk_end(int c) {
    constexpr int Q = VelSet<D>::Q;
    const int e = kChunk0<D> + c * kChunkW<D>;
    return c == 0 ? kChunk0<D> : (e < Q ? e : Q);
}

// Uncorrected targets' moment sums and the residuals of the exact-moment
// correction (as relax<…, DEV> forms them: per +- pair, group by group,
// then the rest population).
template <int D, typename T>
__device__ __forceinline__ void target_residuals(const Equilibrium<D, T, true>& eq,
                                                 const Physics& a, T arho, T beta, T want_m,
                                                 const T* want_j, T want_e, T je_on, T& dm,
                                                 T* dj, T& de) {
#pragma clang fp contract(off)
    constexpr VelSet<D> V = kVelSet<D>;
    constexpr int G = VelSet<D>::G;
    T sm = 0, sjx = 0, sjy = 0, sjz = 0, se = 0;
    static_for<1, G>([&](auto Gi) {
        constexpr int g = decltype(Gi)::value;
        T A0, A1, A2;
        eq.template coef<V.qn[g]>(A0, A1, A2);
        const T w = weight<T>(a, g);
        constexpr int first = group_start<D>(g);
        static_for<0, V.count[g] / 2>([&](auto Pi) {
            constexpr int i = first + 2 * decltype(Pi)::value;
            constexpr Vel v = V.v[i];
            const T c = eq.template dot<v.x, v.y, v.z>();
            T tp, tm;
            pair_targets(A0, A1, A2, c, w, arho, beta, tp, tm);
            const T sum = tp + tm;
            const T dif = tp - tm;
            sm += sum;
            if constexpr (v.x != 0) sjx = fmadd(T(v.x), dif, sjx);
            if constexpr (v.y != 0) sjy = fmadd(T(v.y), dif, sjy);
            if constexpr (D == 3 && v.z != 0) sjz = fmadd(T(v.z), dif, sjz);
            se = fmadd(T(V.qn[g]), sum, se);
        });
    });
    T A0, A1, A2;
    eq.template coef<0>(A0, A1, A2);
    sm += rest_target(A0, weight<T>(a, 0), arho, beta);
    dm = want_m - sm;
    de = je_on * (want_e - se);
    dj[0] = je_on * (want_j[0] - sjx);
    dj[1] = je_on * (want_j[1] - sjy);
    if constexpr (D == 3) dj[2] = je_on * (want_j[2] - sjz);
}

// The record of one cell from its moment sums (g: s0, sj, se; h: sh).
template <int D, class P>
__device__ __forceinline__ void write_record(typename P::T s0, typename P::T sx,
                                             typename P::T sy, typename P::T sz,
                                             typename P::T se, typename P::T sh,
                                             typename P::T* __restrict__ rec, int64_t N,
                                             int64_t cell, const Physics& ph) {
    using T = typename P::T;
    constexpr bool DEV = P::kDev;
    T sj[3] = {sx, sy, sz};
    T rho, drho, u[3] = {0, 0, 0}, t;
    macro<D, T, DEV>(s0, sj, se, sh, T(ph.r), ph.inv_dof, ph.half_delta, rho, drho, u, t);
    Equilibrium<D, T, DEV> eq;
    eq.setup(u, t, T(ph.r));
    const T want_e = (rho * eq.U + T(D) * (drho + rho * t)) / eq.r2;
    const T kr = energy_fix_kr<D, T, DEV>(ph, rho, eq, want_e, se);
    rec[cell] = DEV ? drho : rho;
#pragma unroll
    for (int k = 0; k < D; ++k) rec[(size_t)(1 + k) * N + cell] = u[k];
    rec[(size_t)(D + 1) * N + cell] = t;
    rec[(size_t)(D + 2) * N + cell] = kr;
    if constexpr (DEV) {
        const T hd = T(ph.half_delta);
        const T hdT = hd * (T(1) + t);
        T dm, dj[3] = {0, 0, 0}, de;
        target_residuals<D, T>(eq, ph, rho, drho, drho, sj, want_e, T(1), dm, dj, de);
        rec[(size_t)(D + 3) * N + cell] = dm;
#pragma unroll
        for (int k = 0; k < D; ++k) rec[(size_t)(D + 4 + k) * N + cell] = dj[k];
        rec[(size_t)(2 * D + 4) * N + cell] = de;
        T dmh, djh[3] = {0, 0, 0}, deh;
        target_residuals<D, T>(eq, ph, hdT * rho + kr, hdT * drho + hd * t + kr,
                               hd * (drho + rho * t) + kr, sj, T(0), T(0), dmh, djh, deh);
        rec[(size_t)(2 * D + 5) * N + cell] = dmh;
    }
}

// The +- pairs of a velocity set, for loops over pairs at run time: the first
// member's vector, the group and |e|^2, packed in a word (scalar loads).
template <int D>
struct PairWords {
    uint32_t w[VelSet<D>::Q / 2];
};
template <int D>
constexpr PairWords<D> make_pair_words() {
    PairWords<D> p{};
    for (int n = 0; n < VelSet<D>::Q / 2; ++n) {
        const Vel v = kVelSet<D>.v[1 + 2 * n];
        p.w[n] = (uint32_t)(v.x + 3) | (uint32_t)(v.y + 3) << 3 | (uint32_t)(v.z + 3) << 6 |
                 (uint32_t)v.group << 9 | (uint32_t)kVelSet<D>.qn[v.group] << 13;
    }
    return p;
}
__constant__ const PairWords<2> kPairs2 = make_pair_words<2>();
__constant__ const PairWords<3> kPairs3 = make_pair_words<3>();

struct PairVel {
    int x, y, z, g, q;
};
template <int D>
__device__ __forceinline__ PairVel pair_vel(int n) {
    uint32_t w;
    if constexpr (D == 2) w = kPairs2.w[n];
    else w = kPairs3.w[n];
    return PairVel{(int)(w & 7) - 3, (int)(w >> 3 & 7) - 3, (int)(w >> 6 & 7) - 3,
                   (int)(w >> 9 & 15), (int)(w >> 13)};
}

// The equilibrium of a cell (Equilibrium in step_core.h) with the shell
// |e|^2 = qn as a run-time value.
template <int D>
struct Shell {
    double qd, b, c, q2, q4;
    __device__ __forceinline__ Shell(double r2, int qn) {
        const double q = r2 * qn;
        qd = q - D;
        b = 6.0 * (D + 2 - q);
        c = 3.0 * (q * (q - 2 * (D + 2)) + D * (D + 2));
        q2 = 0.5 * (q - (D + 2));
        q4 = 0.25 * (q - (D + 4));
    }
    __device__ __forceinline__ void coef(double U, double t, double& A0, double& A1,
                                         double& A2) const {
        const double hi = fmadd(3.0 * U, U, t * fmadd(c, t, b * U));
        A0 = 1.0 + fmadd(1.0 / 24.0, hi, 0.5 * fmadd(t, qd, -U));
        A1 = fmadd(q2, t, fmadd(-0.5, U, 1.0));
        A2 = fmadd(q4, t, fmadd(-0.25, U, 0.5));
    }
};

// The macroscopic state of a cell as the targets take it.
template <int D>
struct FdState {
    double rho, t, U;  // t = T - 1, U = |u|^2
    double ru[3];      // r u
    double rho_h;      // (delta/2) T rho + kappa rho

    // from a record
    __device__ __forceinline__ void set(double rho_, const double* u, double t_, double kr,
                                        const Physics& ph) {
        rho = rho_;
        t = t_;
        U = u[0] * u[0] + u[1] * u[1];
        if constexpr (D == 3) U += u[2] * u[2];
#pragma unroll
        for (int k = 0; k < D; ++k) ru[k] = ph.r * u[k];
        rho_h = ph.half_delta * (1.0 + t) * rho + kr;
    }
};

template <int D, class P>
__global__ __launch_bounds__(256) void k_fd_moments(const void* __restrict__ src_v,
                                                    typename P::T* __restrict__ rec,
                                                    int64_t cells, int64_t N,
                                                    const Physics ph) {
    using T = typename P::T;
    using S = typename P::S;
    constexpr VelSet<D> V = kVelSet<D>;
    constexpr int Q = VelSet<D>::Q;
    const int64_t cell = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (cell >= cells) return;  // lanes are independent here (N: the plane stride)
    const S* src = static_cast<const S*>(src_v);
    // running sums over the centre values (moment_sums, streamed)
    T s0 = 0, sx = 0, sy = 0, sz = 0, se = 0, sh = 0;
    static_for<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr Vel v = V.v[i];
        const T x = from_store<P>(src[(size_t)(2 * i) * N + cell], ph, v.group);
        const T y = from_store<P>(src[(size_t)(2 * i + 1) * N + cell], ph, v.group);
        s0 += x;
        if constexpr (v.x != 0) sx += T(v.x) * x;
        if constexpr (v.y != 0) sy += T(v.y) * x;
        if constexpr (D == 3 && v.z != 0) sz += T(v.z) * x;
        if constexpr (V.qn[v.group] != 0) se += T(V.qn[v.group]) * x;
        sh += y;
    });
    write_record<D, P>(s0, sx, sy, sz, se, sh, rec, N, cell, ph);
}

// S_0, and from the values as stored its record (as k_fd_moments makes it; null:
// none).  What bounds it is the side written.  Made apart, the record read all of
// S_0 again: D3Q107 FP32 256^3 2.93 + 2.94 ms, together 3.78.
template <int D, class P>
__global__ __launch_bounds__(256) void k_fd_init(char* dst, typename P::T* __restrict__ rec,
                                                 const InitFields f, const WGroups wg,
                                                 const Physics ph) {
    using T = typename P::T;
    using S = typename P::S;
    constexpr VelSet<D> V = kVelSet<D>;
    const int64_t cell = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (cell >= f.N) return;
    InitCell<D> ic;
    ic.load(f, cell);
    const size_t plane = (size_t)f.P * sizeof(S);
    T s0 = 0, sx = 0, sy = 0, sz = 0, se = 0, sh = 0;
    static_for<0, VelSet<D>::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr Vel v = V.v[i];
        S g, h;
        ic.template values<P, i>(wg, g, h);
        // the sums take the values as stored, not the products they were
        // rounded from
        asm("" : "+v"(g), "+v"(h));
        char* at = dst + (size_t)(2 * i) * plane + (size_t)cell * sizeof(S);
        *reinterpret_cast<S*>(at) = g;
        *reinterpret_cast<S*>(at + plane) = h;
        const T x = g;
        s0 += x;
        if constexpr (v.x != 0) sx += T(v.x) * x;
        if constexpr (v.y != 0) sy += T(v.y) * x;
        if constexpr (D == 3 && v.z != 0) sz += T(v.z) * x;
        if constexpr (V.qn[v.group] != 0) se += T(V.qn[v.group]) * x;
        sh += T(h);
    });
    if (rec) write_record<D, P>(s0, sx, sy, sz, se, sh, rec, f.P, cell, ph);
}

// Sweep order of the update passes (2.5D blocking).  A tile is 256 cells of
// one x-row.  The rows are cut into y sub-bands of fd_yb rows, dealt to the
// XCDs round-robin (sub-band s to XCD s % 8, which is workgroup b % 8); an
// XCD sweeps each of its sub-bands x-chunk (fd_w tiles) by x-chunk, and
// within a chunk z-slab by z-slab, row by row.  The planes a stencil reads
// at y +- 1, 2 and z +- 1, 2 were then fetched by the same XCD within the
// last few sub-band slabs, which the host sizes to stay in its L2.  Returns
// false for the padding workgroups of the last round.
__device__ __forceinline__ bool sweep_tile(const StepArgs& a, int b, int& xt, int& cy, int& cz) {
    const int W = a.fd_w, YB = a.fd_yb;
    const int chunks = (a.tiles_per_row + W - 1) / W;
    const int per_chunk = W * YB * a.nz;
    const int per_sub = chunks * per_chunk;
    const int j = b >> 3;
    const int round = j / per_sub;
    const int in_sub = j - round * per_sub;
    const int chunk = in_sub / per_chunk;
    const int in_chunk = in_sub - chunk * per_chunk;
    cz = in_chunk / (YB * W);
    const int in_slab = in_chunk - cz * (YB * W);
    cy = (round * 8 + (b & 7)) * YB + in_slab / W;
    xt = chunk * W + in_slab % W;
    return xt < a.tiles_per_row && cy < a.ny;
}

// One cell of an update pass over populations [C0, C1): the record's
// macroscopic state and equilibrium, the correction residuals (first chunk
// only: it holds the rest and axis populations that take them), and the
// running moment sums of the new populations.
template <int D, class P, int C0, int C1>
struct FdCell {
    using T = typename P::T;
    using S = typename P::S;
    static constexpr bool DEV = P::kDev;
    Equilibrium<D, T, DEV> eq;
    T rho, arho_h, beta_g, beta_h, omf, omg, cs;
    T dm = 0, de = 0, dmh = 0, dj[3] = {0, 0, 0};
    T a0 = 0, ax = 0, ay = 0, az = 0, ae = 0, ah = 0;

    template <bool NT>
    __device__ __forceinline__ static void store(S* plane, uint32_t off, S v) {
        if constexpr (NT) store_at(reinterpret_cast<char*>(plane), off, v);
        else store_cached(reinterpret_cast<char*>(plane), off, v);
    }

    __device__ __forceinline__ void load(const T* __restrict__ rec, int64_t N, int64_t cell,
                                         const Physics& ph) {
        const T m0 = rec[cell];
        T u[3] = {0, 0, 0};
#pragma unroll
        for (int k = 0; k < D; ++k) u[k] = rec[(size_t)(1 + k) * N + cell];
        const T t = rec[(size_t)(D + 1) * N + cell];
        // kappa rho is zero unless the energy-conserving collision is on
        const T kr = ph.ec != 0 ? rec[(size_t)(D + 2) * N + cell] : T(0);
        rho = DEV ? T(1) + m0 : m0;
        const T drho = DEV ? m0 : m0 - T(1);
        eq.setup(u, t, T(ph.r));
        const T hd = T(ph.half_delta);
        const T hdT = hd * (T(1) + t);
        arho_h = hdT * rho + kr;
        beta_g = DEV ? drho : T(0);
        beta_h = DEV ? hdT * drho + hd * t + kr : T(0);
        if constexpr (DEV && C0 == 0) {
            dm = rec[(size_t)(D + 3) * N + cell];
#pragma unroll
            for (int k = 0; k < D; ++k) dj[k] = rec[(size_t)(D + 4 + k) * N + cell];
            de = rec[(size_t)(2 * D + 4) * N + cell];
            dmh = rec[(size_t)(2 * D + 5) * N + cell];
        }
        omf = T(ph.omega_f);
        omg = T(ph.omega_g);
        cs = fd_scale<T>(ph);
    }

    // Population i: target (uncorrected w (arho P~(c) + beta), +- pair
    // arithmetic, plus the correction on the rest and axis populations),
    // relaxation with the convection centre term (relax<..., FD>), neighbour
    // terms (fd_neighbours), store.  at(dist, axis, d) is the stored value
    // of distribution dist (0: g, 1: h) at the neighbour x + d along axis
    // (d = 0: the cell itself).
    // NT: streamed stores (otherwise cached).
    template <int i, bool NT, class At>
    __device__ __forceinline__ void update(const Physics& ph, At&& at, S* __restrict__ dst,
                                           int64_t N, int64_t cell) {
        constexpr VelSet<D> V = kVelSet<D>;
        constexpr Vel v = V.v[i];
        constexpr int g = v.group;
        T A0, A1, A2;
        eq.template coef<V.qn[g]>(A0, A1, A2);
        const T w = weight<T>(ph, g);
        // the targets exactly as relax<...> and target_residuals form them
        T tg, th;
        if constexpr (i == 0) {
            tg = rest_target(A0, w, rho, beta_g);
            th = rest_target(A0, w, arho_h, beta_h);
        } else {
            constexpr int first = (i - group_start<D>(g)) % 2 == 0 ? i : i - 1;
            constexpr Vel vf = V.v[first];
            const T c = eq.template dot<vf.x, vf.y, vf.z>();
            T gp, gm, hp, hm;
            pair_targets(A0, A1, A2, c, w, rho, beta_g, gp, gm);
            pair_targets(A0, A1, A2, c, w, arho_h, beta_h, hp, hm);
            tg = i == first ? gp : gm;
            th = i == first ? hp : hm;
        }
        if constexpr (DEV && i == 0) {
            tg += dm - de;
            th += dmh;
        }
        if constexpr (DEV && i >= 1 && i <= 2 * D) {
            constexpr int axis = v.x != 0 ? 0 : (v.y != 0 ? 1 : 2);
            constexpr int s = (v.x + v.y + v.z) > 0 ? 1 : -1;
            const T half = T(0.5) * dj[axis];
            tg += s > 0 ? de * T(1.0 / (2 * D)) + half : de * T(1.0 / (2 * D)) - half;
        }
        using Z = std::integral_constant<int, 0>;
        using G = std::integral_constant<int, 0>;
        using H = std::integral_constant<int, 1>;
        T xg = from_store<P>(at(G{}, Z{}, Z{}), ph, g);
        T xh = from_store<P>(at(H{}, Z{}, Z{}), ph, g);
        if constexpr (l1_of(v) != 0) {
            const T kc = T(3 * l1_of(v)) * cs;
            xg = relax_value(xg, tg, omf, kc);
            xh = relax_value(xh, th, omg, kc);
        } else {
            xg = relax_value(xg, tg, omf);
            xh = relax_value(xh, th, omg);
        }
        T nbg = T(0), nbh = T(0);
        static_for<0, D>([&](auto A) {
            constexpr int ax_ = decltype(A)::value;
            constexpr int e = ax_ == 0 ? v.x : (ax_ == 1 ? v.y : v.z);
            if constexpr (e != 0) {
                constexpr int s = e > 0 ? 1 : -1;
                constexpr int m = e > 0 ? e : -e;
                using M2 = std::integral_constant<int, -2 * s>;
                using M1 = std::integral_constant<int, -s>;
                using P1 = std::integral_constant<int, s>;
                nbg += T(m) * ((from_store<P>(at(G{}, A, M2{}), ph, g) -
                                T(6) * from_store<P>(at(G{}, A, M1{}), ph, g)) +
                               T(2) * from_store<P>(at(G{}, A, P1{}), ph, g));
                nbh += T(m) * ((from_store<P>(at(H{}, A, M2{}), ph, g) -
                                T(6) * from_store<P>(at(H{}, A, M1{}), ph, g)) +
                               T(2) * from_store<P>(at(H{}, A, P1{}), ph, g));
            }
        });
        const T ng = xg - cs * nbg;
        const T nh = xh - cs * nbh;
        const size_t pg_off = (size_t)(2 * i) * N, ph_off = pg_off + N;
        store<NT>(dst + pg_off, (uint32_t)(cell * sizeof(S)), to_store<P>(ng, ph, g));
        store<NT>(dst + ph_off, (uint32_t)(cell * sizeof(S)), to_store<P>(nh, ph, g));
        {
            a0 += ng;
            if constexpr (v.x != 0) ax += T(v.x) * ng;
            if constexpr (v.y != 0) ay += T(v.y) * ng;
            if constexpr (D == 3 && v.z != 0) az += T(v.z) * ng;
            if constexpr (V.qn[g] != 0) ae += T(V.qn[g]) * ng;
            ah += nh;
        }
    }

    // Running sums: the first chunk starts them, the last turns the totals
    // into the next step's record (this lane has read its cell's record).
    __device__ __forceinline__ void finish(T* __restrict__ rec, int64_t N, int64_t cell,
                                           const Physics& ph) {
        {
            T* acc = rec + (size_t)kRecFields<D, DEV> * N;
            T sums[6] = {a0, ax, ay, az, ae, ah};
            constexpr int kSlots[6] = {0, 1, 2, D == 3 ? 3 : -1, D + 1, D + 2};
            if constexpr (C0 != 0) {
#pragma unroll
                for (int k = 0; k < 6; ++k)
                    if (kSlots[k] >= 0) sums[k] += acc[(size_t)kSlots[k] * N + cell];
            }
            if constexpr (C1 == VelSet<D>::Q) {
                write_record<D, P>(sums[0], sums[1], sums[2], sums[3], sums[4], sums[5], rec, N,
                                   cell, ph);
            } else {
#pragma unroll
                for (int k = 0; k < 6; ++k)
                    if (kSlots[k] >= 0) acc[(size_t)kSlots[k] * N + cell] = sums[k];
            }
        }
    }
};

// Update of populations [C0, C1) of every cell, one lane per cell, the
// stencil values read straight from global memory (through L1/L2).  What
// bounds it at the sizes it serves is a launch's latency and the number of
// waves: D3Q107 FP32 on 32^3 takes 64 us a step in six launches, where a
// tile's walk through 214 planes alone takes 130.
template <int D, class P, int C0, int C1, bool NT>
__global__ __launch_bounds__(256) void k_fd_update(const void* __restrict__ src_v,
                                                   void* __restrict__ dst_v,
                                                   typename P::T* __restrict__ rec,
                                                   const StepArgs a) {
    using S = typename P::S;
    const int64_t N = a.P;  // plane stride (record and populations)
    int xt, cy, cz;
    if (!sweep_tile(a, (int)blockIdx.x, xt, cy, cz)) return;
    const int cx = xt * 256 + (int)threadIdx.x;
    if (cx >= a.nx) return;
    const int64_t cell = (int64_t)cx + (int64_t)a.nx * cy + (int64_t)a.nxy * cz;
    const Physics& ph = a.ph;
    PullTable<D> pt;  // entry e + 3: the coordinate x - e (wrapped or clamped)
    pt.fill(cx, cy, cz, a.nx, a.ny, a.nz, a.nxy, a.open_end);
    const S* src = static_cast<const S*>(src_v);
    S* dst = static_cast<S*>(dst_v);
    FdCell<D, P, C0, C1> c;
    c.load(rec, N, cell, ph);
    static_for<C0, C1>([&](auto I) {
        constexpr int i = decltype(I)::value;
        // offset of the neighbour x + d along axis ax of this cell
        auto at = [&](auto Dist, auto Ax, auto Dd) {
            constexpr int ax = decltype(Ax)::value;
            constexpr int d = decltype(Dd)::value;
            constexpr int dist = decltype(Dist)::value;
            int o = ax == 0 ? pt.x[3 - d] : pt.x[3];
            o += ax == 1 ? pt.y[3 - d] : pt.y[3];
            if constexpr (D == 3) o += ax == 2 ? pt.z[3 - d] : pt.z[3];
            return src[(size_t)(2 * i + dist) * N + o];
        };
        c.template update<i, NT>(ph, at, dst, N, cell);
    });
    c.finish(rec, N, cell, ph);
}

// LDS-staged update, for rows of whole tiles (nx a multiple of 256).  The
// one-lane-per-cell kernel issues a 4-byte load per stencil point, about
// eight per population and cell; its counters show the vector memory
// address unit busy 80-98% of the time while HBM is not saturated.  Here a
// workgroup serves one 256-cell tile and, per phase of kFdPhase
// populations, loads the rows their stencils read -- the tile's own row
// with two cells of halo either side, and the three upwind-biased rows
// along y and along z where a population moves along them -- four cells a
// lane (one 16-byte load per row and wave in FP32), stages them in LDS, and
// each lane takes its cell's stencil values from there.  The arithmetic is
// FdCell's, as in k_fd_update.
//
// LDS per population: the centre rows of g and h (264 slots each: two
// unused, two halo, 256 cells, two halo, two unused, so the cells start at a
// 16-byte boundary), then up to 12 neighbour rows of 256 (3 per moving axis
// y, z and per distribution).
template <int D>
constexpr int kLdsCentre = 264;
template <int D>
constexpr int kLdsSlots = 2 * kLdsCentre<D> + (D == 3 ? 12 : 6) * 256;
// Populations staged per barrier phase: two for D3Q107 in FP32 (2% faster at
// 256^3), one otherwise (FP64 needs twice the LDS, and D2Q37 rows are fewer).
template <int D, class P>
constexpr int kFdPhase = (D == 3 && P::kDev) ? 2 : 1;

// Stencil rows of population i staged per phase: the g and h centre rows,
// then per moving axis (y first) and distribution the rows at -2s, -s, +s.
template <int D>
constexpr int fd_rows(int i) {
    const Vel v = kVelSet<D>.v[i];
    return 2 + 6 * ((v.y != 0 ? 1 : 0) + (D == 3 && v.z != 0 ? 1 : 0));
}

template <int D, class P, int C0, int C1, int PB, bool NT>
__global__ __launch_bounds__(256) void k_fd_update_lds(const void* __restrict__ src_v,
                                                       void* __restrict__ dst_v,
                                                       typename P::T* __restrict__ rec,
                                                       const StepArgs a) {
    using S = typename P::S;
    typedef S S4 __attribute__((ext_vector_type(4)));
    constexpr VelSet<D> V = kVelSet<D>;
    constexpr int CW = kLdsCentre<D>;
    constexpr int SL = kLdsSlots<D>;  // LDS slots of one population
    static_assert(PB == 1 || PB == 2, "one or two populations per phase");
    __shared__ __attribute__((aligned(16))) S lds[PB * SL];
    const int64_t N = a.P;  // plane stride (record and populations)
    int xt, cy, cz;
    // the whole workgroup leaves together (it meets at barriers below)
    if (!sweep_tile(a, (int)blockIdx.x, xt, cy, cz)) return;
    const int tid = (int)threadIdx.x;
    // wave-uniform, in a scalar register: the row loads below branch on it
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int x0 = xt * 256;
    const int64_t cell = (int64_t)(x0 + tid) + (int64_t)a.nx * cy + (int64_t)a.nxy * cz;
    const Physics& ph = a.ph;
    const bool open_x = a.open_end & 1u, open_y = a.open_end & 2u, open_z = a.open_end & 4u;
    // starts (cells) of the tile's part of its own row and of rows y + d and
    // z + d, d = -2, -1, 1, 2: wave-uniform, computed once
    const int64_t own = (int64_t)a.nx * cy + (int64_t)a.nxy * cz + x0;
    int64_t ys[4], zs[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int d = k < 2 ? k - 2 : k - 1;
        ys[k] = own + (int64_t)(pull_coord(cy, -d, a.ny, open_y) - cy) * a.nx;
        zs[k] = D == 3 ? own + (int64_t)(pull_coord(cz, -d, a.nz, open_z) - cz) * a.nxy : own;
    }
    // halo cells x0 - 2, x0 - 1, x0 + 256, x0 + 257 of the tile's row (lanes 0..3)
    const int hsh = lane < 2 ? 2 - lane : -254 - lane;  // pull shift e: source x0 - e
    const int64_t halo_src = (int64_t)pull_coord(x0, hsh, a.nx, open_x) - x0;
    const int halo_slot = lane < 2 ? 2 + lane : 258 + lane;  // slots 2, 3, 260, 261
    const S* src = static_cast<const S*>(src_v);
    S* dst = static_cast<S*>(dst_v);
    // A phase stages PB populations.  Its rows, population by population, are
    // numbered R = 0, 1, ...; wave w loads rows w, w + 4, ..., picked branch-
    // free.  The next phase's loads are issued before this one is computed
    // and land in LDS after the barrier that ends this phase's reads.  The
    // halo of population j's distribution d is loaded by wave 2 j + d.
    constexpr int kMaxSets = (14 * PB + 3) / 4;
    S4 q[kMaxSets];
    int slot[kMaxSets];
    bool has[kMaxSets];
    S hv = S(0);
    bool halo = false;
    int halo_at = 0;
    auto issue = [&](auto Ph) {
        constexpr int i0 = C0 + PB * decltype(Ph)::value;
        constexpr int np = (C1 - i0) < PB ? (C1 - i0) : PB;
        constexpr int nr0 = fd_rows<D>(i0);
        constexpr int nrows = nr0 + (np > 1 ? fd_rows<D>(i0 + 1) : 0);
        // phase row R: its start in global memory and its LDS slot
        auto row_of = [&](auto RR, const S*& ptr, int& sl) {
            constexpr int R = decltype(RR)::value;
            constexpr int j = R < nr0 ? 0 : 1;
            constexpr int i = i0 + j;
            constexpr int r = R - (j ? nr0 : 0);
            constexpr Vel v = V.v[i];
            constexpr bool my = v.y != 0;
            constexpr int sy = v.y > 0 ? 1 : -1, sz = v.z > 0 ? 1 : -1;
            if constexpr (r < 2) {
                ptr = src + (size_t)(2 * i + r) * N + own;
                sl = j * SL + r * CW + 4;
            } else {
                constexpr int k = (r - 2) % 3;         // -2s, -s, +s
                constexpr int dist = ((r - 2) / 3) % 2;
                constexpr bool along_y = my && (r - 2) < 6;
                constexpr int sg = along_y ? sy : sz;
                constexpr int d = k == 0 ? -2 * sg : (k == 1 ? -sg : sg);
                constexpr int kk = d < 0 ? d + 2 : d + 1;  // index in ys / zs
                ptr = src + (size_t)(2 * i + dist) * N + (along_y ? ys[kk] : zs[kk]);
                sl = j * SL + 2 * CW + (r - 2) * 256;
            }
        };
        static_for<0, kMaxSets>([&](auto M) {
            constexpr int m = decltype(M)::value;
            const S* ptr = nullptr;
            int sl = 0;
            static_for<0, 4>([&](auto W) {
                constexpr int R = 4 * m + decltype(W)::value;
                if constexpr (R < nrows) {
                    const S* pr;
                    int sr;
                    row_of(std::integral_constant<int, R>{}, pr, sr);
                    ptr = wave == decltype(W)::value ? pr : ptr;
                    sl = wave == decltype(W)::value ? sr : sl;
                }
            });
            has[m] = 4 * m + 3 < nrows || ptr != nullptr;
            slot[m] = sl;
            if (has[m]) q[m] = *reinterpret_cast<const S4*>(ptr + 4 * lane);
        });
        // halo: population j = wave / 2, distribution wave % 2
        const int j = wave >> 1, dist = wave & 1;
        constexpr bool hx0 = V.v[i0].x != 0;
        constexpr bool hx1 = np > 1 && V.v[np > 1 ? i0 + 1 : i0].x != 0;
        const bool need = j == 0 ? hx0 : (j == 1 ? hx1 : false);
        halo = need && lane < 4;
        halo_at = j * SL + dist * CW + halo_slot;
        if (halo) hv = src[(size_t)(2 * (i0 + j) + dist) * N + own + halo_src];
    };
    FdCell<D, P, C0, C1> c;
    c.load(rec, N, cell, ph);
    constexpr int kPhases = (C1 - C0 + PB - 1) / PB;
    issue(std::integral_constant<int, 0>{});
    static_for<0, kPhases>([&](auto Ph) {
        constexpr int phz = decltype(Ph)::value;
        constexpr int i0 = C0 + PB * phz;
        constexpr int np = (C1 - i0) < PB ? (C1 - i0) : PB;
        if constexpr (phz != 0) __syncthreads();  // the previous phase's reads are done
#pragma unroll
        for (int m = 0; m < kMaxSets; ++m)
            if (has[m]) *reinterpret_cast<S4*>(lds + slot[m] + 4 * lane) = q[m];
        if (halo) lds[halo_at] = hv;
        __syncthreads();
        if constexpr (phz + 1 < kPhases) issue(std::integral_constant<int, phz + 1>{});
        static_for<0, np>([&](auto J) {
            constexpr int j = decltype(J)::value;
            constexpr int i = i0 + j;
            constexpr Vel v = V.v[i];
            constexpr bool my = v.y != 0;
            constexpr int sy = v.y > 0 ? 1 : -1, sz = v.z > 0 ? 1 : -1;
            const S* base = lds + j * SL;
            auto at = [&](auto Dist, auto Ax, auto Dd) {
                constexpr int dist = decltype(Dist)::value;
                constexpr int ax = decltype(Ax)::value;
                constexpr int d = decltype(Dd)::value;
                if constexpr (d == 0 || ax == 0) {
                    return base[dist * CW + 4 + tid + d];
                } else {
                    constexpr int s = ax == 1 ? sy : sz;
                    constexpr int k = d == -2 * s ? 0 : (d == -s ? 1 : 2);
                    constexpr int blk = (ax == 2 && my) ? 2 : 0;  // y's rows come first
                    return base[2 * CW + (3 * (blk + dist) + k) * 256 + tid];
                }
            };
            c.template update<i, NT>(ph, at, dst, N, cell);
        });
    });
    c.finish(rec, N, cell, ph);
}

// The update.  A workgroup serves a tile and walks through all populations
// plane by plane (g, then h, of each), so that a cell's record is read once
// and its new moment sums stay in registers until they become the next
// record.  A lane owns TZ cells in a column along the last axis (z in 3D, y
// in 2D), a wave 64 cells along x, and the TY waves of a workgroup TY rows
// along y (3D) or TY columns end to end (2D).  Each plane's tile and the
// cells its stencils reach beyond it go from memory straight into LDS, three
// planes ahead of the one being computed (four buffers).
//
// Why this split.  In chunks a step reads the record and the moment sums again
// for each (D3Q107: 540 B a cell and step on top of 3424), refetches stencil
// rows, and waits on the loads of one population at a time: D3Q107
// 256x256x128 9.9 ms a step, 100^3 1.96, D2Q37 4096^2 5.7, 1500x1100 0.72 (fused).
// In tiles 6.1, 1.12, 3.6 and 0.48 ms.  Staged through registers, one plane
// ahead, they took 7.5, 1.50, 4.1 and 0.53: direct loads into LDS free those
// registers and carry the loads three planes ahead.  A tile of 64 x 8 x 4 cells
// asks the L2 for 1.9 cells per cell (64 x 4 x 4: 2.2, 5% slower), part of the
// halo is found there, and HBM reads come to 1.44 times the populations in 3D
// (256^3), 1.21 in 2D (4096^2).  That traffic bounds it: with the writes 5.6 TB/s
// and 6.2.  Two cells a lane (64 x 8 x 2) took 6.6 ms and 3.7 in 2D, eight
// spilled.
constexpr int kTileZ = 4;

template <int D, int TY>
struct FdTile {
    static constexpr int TZ = kTileZ;
    static constexpr int kOwnI = TZ / 2;  // 16-byte loads (two rows of 64 cells) of a wave's own rows
    static constexpr int kEndI = 2;       // and of its column ends (three rows)
    static constexpr int kSideI = D == 3 ? (3 * TZ / 2 + TY - 1) / TY : 0;  // y halo
    // LDS of one plane, in values; every region's march positions are 64 apart
    static constexpr int kOwn = 0;                        // [TY][TZ][64]
    static constexpr int kEnd = TY * TZ * 64;             // [TY][3][64] far, near upwind; downwind
    static constexpr int kSide = kEnd + TY * 3 * 64;      // [3][TZ][64] likewise, 3D
    static constexpr int kLine = kSide + (D == 3 ? 3 * TZ * 64 : 0);  // [TZ][TY][4], rows of 64
    static constexpr int kBuf = kLine + TZ * 64;
    static_assert(TY >= TZ && TY <= 8, "the x halo: a wave per march position, 64 lanes for all rows");
};

// Access through a buffer resource of one plane: a 32-bit lane offset plus a
// scalar row offset, with the plane's base in scalar registers.  (As plain
// pointers the compiler keeps base + row + lane as one 64-bit vector address
// for each of a plane's rows across the loop over planes, 60 registers more.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000);
}
__device__ __forceinline__ double buf_load(__amdgpu_buffer_rsrc_t r, uint32_t lane_off,
                                           uint32_t row_off) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off,
                                                                          (int)row_off, 0));
}
// NT: non-temporal (cache policy bit 1)
template <bool NT>
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, uint32_t lane_off,
                                          uint32_t row_off, double v) {
    typedef uint32_t U2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, v), r, (int)lane_off,
                                          (int)row_off, NT ? 2 : 0);
}

// Tile of this workgroup; false if it has none.  Tiles are dealt in bricks
// (fd_bw x fd_bh x fd_bd tiles) to the XCDs in turn, so that the tiles that
// run at one time on an XCD are neighbours and find each other's halo rows
// in its L2 (bricks of 16 to 128 tiles time the same; of 512, in which the
// tiles running together no longer touch, up to 20% longer).
__device__ __forceinline__ bool fd_tile_of(const StepArgs& a, int& tx, int& ty, int& tz) {
    const int b = (int)blockIdx.x, j = b >> 3;
    const int vol = a.fd_bw * a.fd_bh * a.fd_bd;
    const int turn = j / vol, in = j - turn * vol;
    const int brick = turn * 8 + (b & 7);
    const int bx = (a.fd_tx + a.fd_bw - 1) / a.fd_bw, by = (a.fd_ty + a.fd_bh - 1) / a.fd_bh;
    const int row = brick / bx;
    tx = (brick - row * bx) * a.fd_bw + in % a.fd_bw;
    ty = (row % by) * a.fd_bh + in / a.fd_bw % a.fd_bh;
    tz = (row / by) * a.fd_bd + in / (a.fd_bw * a.fd_bh);
    return tx < a.fd_tx && ty < a.fd_ty && tz < a.fd_tz;
}

// LDS for a direct load: one address per wave, lanes follow each other.
typedef __attribute__((address_space(3))) void LdsVoid;
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t r, double* lds,
                                           uint32_t lane_off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (LdsVoid*)lds, 16, (int)lane_off, 0, 0, 0);
}
__device__ __forceinline__ void load_lds4(__amdgpu_buffer_rsrc_t r, double* lds,
                                          uint32_t lane_off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (LdsVoid*)lds, 4, (int)lane_off, 0, 0, 0);
}
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N < 64);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

template <int D, int TY, bool NT, int WAVES>
__global__ __launch_bounds__(64 * TY) __attribute__((amdgpu_waves_per_eu(WAVES, 8)))
void k_fd_tile(const double* __restrict__ src, double* __restrict__ dst,
               double* __restrict__ rec, const StepArgs a) {
    constexpr uint32_t S = sizeof(double);
    using K = FdTile<D, TY>;
    constexpr int TZ = K::TZ;
    __shared__ __attribute__((aligned(16))) double b0[K::kBuf], b1[K::kBuf], b2[K::kBuf],
        b3[K::kBuf];
    const Physics& ph = a.ph;
    int tx, ty, tz;
    if (!fd_tile_of(a, tx, ty, tz)) return;  // the whole workgroup
    // scalar, and with them every row offset below
    tx = __builtin_amdgcn_readfirstlane(tx);
    ty = __builtin_amdgcn_readfirstlane(ty);
    tz = __builtin_amdgcn_readfirstlane(tz);
    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool open_x = a.open_end & 1u, open_y = a.open_end & 2u;
    const bool open_m = D == 3 ? (a.open_end & 4u) != 0 : open_y;
    // march axis: z in 3D, y in 2D
    const int nm = D == 3 ? a.nz : a.ny;
    const uint32_t mstride = (uint32_t)(D == 3 ? a.nxy : a.nx) * S;
    const int x0 = tx * 64;
    const int xe = x0 + 64 < a.nx ? x0 + 64 : a.nx;  // end of the tile's cells along x
    const int y0 = ty * TY;                          // 3D
    // A position past the end is taken up to two cells out (a stencil's
    // reach) and then wrapped or clamped like the pull.
    auto at = [](int p, int n, bool open) { return pull_coord(p < n + 1 ? p : n + 1, 0, n, open); };
    auto first_m = [&](int w) { return D == 3 ? tz * TZ : (ty * TY + w) * TZ; };
    // byte offset of row (y0 + y, m) in a plane (2D: m alone)
    auto row_at = [&](int y, int m) {
        uint32_t o = (uint32_t)at(m, nm, open_m) * mstride;
        if constexpr (D == 3) o += (uint32_t)(at(y0 + y, a.ny, open_y) * a.nx) * S;
        return o;
    };
    const int m0 = first_m(wave);
    constexpr uint32_t kNone = 0x80000000u;  // past every plane: stores nothing

    // lane offsets of the direct loads (a load moves two rows, 16 bytes a
    // lane; bytes past a row's end are the next row's, unused)
    const int lrow = lane >> 5;
    const uint32_t lcol = (uint32_t)x0 * S + (uint32_t)(lane & 31) * 16;
    uint32_t v_own[K::kOwnI], v_end[2][K::kEndI];
    uint32_t v_side[2][K::kSideI > 0 ? K::kSideI : 1];
#pragma unroll
    for (int n = 0; n < K::kOwnI; ++n) v_own[n] = row_at(wave, m0 + n * 2 + lrow) + lcol;
#pragma unroll
    for (int n = 0; n < K::kEndI; ++n) {  // [0]: moving up, [1]: moving down the axis
        const int e = n * 2 + lrow;
        v_end[0][n] = row_at(wave, m0 + (e == 2 ? TZ : e - 2)) + lcol;
        v_end[1][n] = row_at(wave, m0 + (e == 2 ? -1 : TZ + 1 - e)) + lcol;
    }
    if constexpr (D == 3) {
#pragma unroll
        for (int n = 0; n < K::kSideI; ++n) {
            const int r = (wave + TY * n) * 2 + lrow, e = r / TZ;
            v_side[0][n] = row_at(e == 2 ? TY : e - 2, m0 + r % TZ) + lcol;
            v_side[1][n] = row_at(e == 2 ? -1 : TY + 1 - e, m0 + r % TZ) + lcol;
        }
    }
    // x halo, wave k that of march position k for all waves' rows at once:
    // cells x0 - 2, x0 - 1, xe, xe + 1 of each, in halves of 4 bytes
    const int hk = lane >> 1 & 3, hw = lane >> 3;
    const uint32_t v_line =
        row_at(hw, first_m(hw) + wave) + 4u * (lane & 1) +
        (uint32_t)at(hk < 2 ? x0 - 2 + hk : xe + hk - 2, a.nx, open_x) * S;
    // The waits below count on every lane count of a wave issuing the same
    // loads, so masks are by lane or by wave, never around the whole load.
    auto issue = [&](double* buf, int plane, bool valid, int ex, int ey, int em) {
        const uint32_t bytes = (uint32_t)a.P * S;
        const double* pl = src + (size_t)plane * a.P;
        const auto r = plane_rsrc(pl, valid ? bytes : 0u);
#pragma unroll
        for (int n = 0; n < K::kOwnI; ++n)
            load_lds16(r, buf + K::kOwn + (wave * TZ + n * 2) * 64, v_own[n]);
        // always issued, from an empty plane where nothing moves along the axis
        const auto re = plane_rsrc(pl, valid && em != 0 ? bytes : 0u);
#pragma unroll
        for (int n = 0; n < K::kEndI; ++n)
            if (n * 2 + lrow < 3)
                load_lds16(re, buf + K::kEnd + (wave * 3 + n * 2) * 64,
                             em > 0 ? v_end[0][n] : v_end[1][n]);
        if constexpr (D == 3) {
            if (ey != 0 && valid) {
#pragma unroll
                for (int n = 0; n < K::kSideI; ++n)
                    if ((wave + TY * n) * 2 < 3 * TZ)
                        load_lds16(r, buf + K::kSide + (wave + TY * n) * 2 * 64,
                                     ey > 0 ? v_side[0][n] : v_side[1][n]);
            }
        }
        if (ex != 0 && valid && wave < TZ && hw < TY)
            load_lds4(r, buf + K::kLine + wave * 64, v_line);
    };
    constexpr int kLoads = K::kOwnI + K::kEndI;  // of a plane, at the least

    // where a lane finds its stencil in a plane's LDS: byte offsets (march
    // positions: + 64 cells)
    const int own_i = K::kOwn + wave * TZ * 64 + lane;
    const int hline = K::kLine + wave * 4;
    auto left = [&](int d) { return (uint32_t)(lane >= d ? own_i - d : hline + 2 + lane - d) * S; };
    auto right = [&](int d) {
        const int x = x0 + lane + d;
        return (uint32_t)(x < xe ? own_i + d : hline + 2 + (x - xe < 1 ? x - xe : 1)) * S;
    };
    uint32_t own = (uint32_t)own_i * S, end = (uint32_t)(K::kEnd + wave * 3 * 64 + lane) * S;
    uint32_t xl1 = left(1), xl2 = left(2), xr1 = right(1), xr2 = right(2), cell = (uint32_t)lane * S;
    // row of wave w + d, or the halo row e beyond the tile
    auto side = [&](int d, int e) {
        const int w = wave + d;
        return (uint32_t)(w >= 0 && w < TY ? K::kOwn + w * TZ * 64 : K::kSide + e * TZ * 64) * S;
    };
    uint32_t up_far = 0, up_near = 0, up_ahead = 0, dn_far = 0, dn_near = 0, dn_ahead = 0;
    if constexpr (D == 3) {
        up_far = side(-2, wave == 0 ? 0 : 1);
        up_near = side(-1, 1);
        up_ahead = side(1, 2);
        dn_far = side(2, wave == TY - 1 ? 0 : 1);
        dn_near = side(1, 1);
        dn_ahead = side(-1, 2);
    }

    // the column's cells in memory
    const bool active = x0 + lane < a.nx && (D == 2 || y0 + wave < a.ny);
    const uint32_t xo = (uint32_t)(x0 + lane) * S;
    // (unsigned: a column past the end of a few long rows may wrap; it stores nothing)
    const uint32_t first = D == 3 ? (uint32_t)(y0 + wave) * (uint32_t)a.nx +
                                        (uint32_t)m0 * (uint32_t)a.nxy
                                  : (uint32_t)m0 * (uint32_t)a.nx;
    const uint32_t v_cell = active ? first * S + xo : kNone;
    // row k of the column in a plane; rows past the grid: an empty one
    auto row_rsrc = [&](const double* plane, int k) {
        return plane_rsrc(plane, m0 + k < nm ? (uint32_t)a.P * S : 0u);
    };
    auto load_field = [&](int f, int k) {
        return buf_load(row_rsrc(rec + (size_t)f * a.P, k), v_cell, k * mstride);
    };

    FdState<D> st[TZ];
#pragma unroll
    for (int k = 0; k < TZ; ++k) {
        double u[3] = {0, 0, 0};
#pragma unroll
        for (int d = 0; d < D; ++d) u[d] = load_field(1 + d, k);
        // kappa rho is zero unless the energy-conserving collision is on
        const double kr = ph.ec != 0 ? load_field(D + 2, k) : 0.0;
        st[k].set(load_field(0, k), u, load_field(D + 1, k), kr, ph);
    }
    double sums[TZ][6];  // of the new state: s0, sj, se of g, the sum of h
#pragma unroll
    for (int k = 0; k < TZ; ++k)
#pragma unroll
        for (int f = 0; f < 6; ++f) sums[k][f] = 0.0;

    // The column's new values: relaxation and the neighbour terms of each
    // axis.  SX: the sign of e_x where it is not zero; mx, my, mm: |e| along
    // x, y (3D) and the march axis.
    const double cs = ph.fd_cs;
    auto compute = [&](auto Sx, const double* buf, double mx, int ey, double my, int em, double mm, double omega,
                       const double* target, double* out) {
        constexpr int SX = decltype(Sx)::value;
        // opaque, or every buffer's addresses get registers of their own
        asm volatile("" : "+v"(own), "+v"(end), "+v"(cell));
        asm volatile("" : "+v"(xl1), "+v"(xl2), "+v"(xr1), "+v"(xr2));
        auto lds = [&](uint32_t off) {
            return reinterpret_cast<const double*>(reinterpret_cast<const char*>(buf) + off);
        };
        double c[TZ], nb[TZ];
#pragma unroll
        for (int k = 0; k < TZ; ++k) {
            c[k] = lds(own)[k * 64];
            nb[k] = 0.0;
        }
        if (mx != 0.0) {
            const double *f = lds(SX > 0 ? xl2 : xr2), *n1 = lds(SX > 0 ? xl1 : xr1),
                    *ah = lds(SX > 0 ? xr1 : xl1);
#pragma unroll
            for (int k = 0; k < TZ; ++k)
                nb[k] = mx * ((f[k * 64] - 6.0 * n1[k * 64]) + 2.0 * ah[k * 64]);
        }
        if constexpr (D == 3) {
            if (ey != 0) {
                const double *f = lds((ey > 0 ? up_far : dn_far) + cell),
                        *n1 = lds((ey > 0 ? up_near : dn_near) + cell),
                        *ah = lds((ey > 0 ? up_ahead : dn_ahead) + cell);
#pragma unroll
                for (int k = 0; k < TZ; ++k)
                    nb[k] += my * ((f[k * 64] - 6.0 * n1[k * 64]) + 2.0 * ah[k * 64]);
            }
        }
        if (em != 0) {
            const double e0 = lds(end)[0], e1 = lds(end)[64], e2 = lds(end)[128];
            if (em > 0) {
#pragma unroll
                for (int k = 0; k < TZ; ++k) {
                    const double far = k >= 2 ? c[k >= 2 ? k - 2 : 0] : (k == 0 ? e0 : e1);
                    const double near = k >= 1 ? c[k >= 1 ? k - 1 : 0] : e1;
                    const double ahead = k + 1 < TZ ? c[k + 1 < TZ ? k + 1 : 0] : e2;
                    nb[k] += mm * ((far - 6.0 * near) + 2.0 * ahead);
                }
            } else {
#pragma unroll
                for (int k = 0; k < TZ; ++k) {
                    const double far = k + 2 < TZ ? c[k + 2 < TZ ? k + 2 : 0] : (k == TZ - 1 ? e0 : e1);
                    const double near = k + 1 < TZ ? c[k + 1 < TZ ? k + 1 : 0] : e1;
                    const double ahead = k >= 1 ? c[k >= 1 ? k - 1 : 0] : e2;
                    nb[k] += mm * ((far - 6.0 * near) + 2.0 * ahead);
                }
            }
        }
        const double kc = 3.0 * cs * (mx + my + (D == 3 ? mm : 0.0));
#pragma unroll
        for (int k = 0; k < TZ; ++k) out[k] = relax_value(c[k], target[k], omega, kc) - cs * nb[k];
    };
    auto store = [&](int plane, const double* v) {
#pragma unroll
        for (int k = 0; k < TZ; ++k)
            buf_store<NT>(row_rsrc(dst + (size_t)plane * a.P, k), v_cell, k * mstride, v[k]);
    };
    // The wave's loads of the present plane have landed (N: how many of its
    // later loads and stores may still be under way), then everyone's; and
    // everyone has read the buffer of the plane before, which the next loads
    // overwrite.
    auto meet = [&](auto Nc) {
        wait_vm<decltype(Nc)::value>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    using W = std::integral_constant<int, 2 * kLoads + 3 * TZ>;  // two planes' loads, three's stores
    using W1 = std::integral_constant<int, kLoads + 3 * TZ>;
    using Up = std::integral_constant<int, 1>;
    using Down = std::integral_constant<int, -1>;
    const double omf = ph.omega_f, omg = ph.omega_g, r2 = ph.r * ph.r;
    constexpr int kPairsN = VelSet<D>::Q / 2;
    // The pairs from the last, then the rest population (as pair -1): the
    // outer groups' small values first keeps the sums' rounding small.
    auto velocity = [&](int n) {
        return n >= 0 ? pair_vel<D>(n) : PairVel{0, 0, 0, 0, 0};
    };
    auto march = [](const PairVel& p) { return D == 3 ? p.z : p.y; };
    // plane j of a pair: g, h of its first member, g, h of the second
    auto fetch = [&](double* buf, int n, const PairVel& p, auto Jc) {
        constexpr int j = decltype(Jc)::value;
        constexpr int s = j < 2 ? 1 : -1;
        const bool rest = n < 0;
        issue(buf, rest ? j : 2 + 4 * n + j, !rest || j < 2, s * p.x, s * p.y, s * march(p));
    };
    using J0 = std::integral_constant<int, 0>;
    using J1 = std::integral_constant<int, 1>;
    using J2 = std::integral_constant<int, 2>;
    using J3 = std::integral_constant<int, 3>;
    PairVel v = velocity(kPairsN - 1);
    fetch(b0, kPairsN - 1, v, J0{});
    fetch(b1, kPairsN - 1, v, J1{});
    fetch(b2, kPairsN - 1, v, J2{});
    // the waits below count the loads and stores from here on (a wait that
    // the compiler sees, so that it adds none of its own)
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    asm volatile("" ::: "memory");
#pragma unroll 1
    for (int n = kPairsN - 1; n >= 0; --n) {
        const PairVel nv = velocity(n - 1);
        const Shell<D> shell(r2, v.q);
        const double w = ph.w[v.g];
        const double ex = v.x, ey = v.y, ez = v.z, qn = v.q;
        const int em = march(v), next = n - 1;
        const double my = abs(v.y), mm = abs(em);
        double gp[TZ], gm[TZ], hp[TZ], hm[TZ];
#pragma unroll
        for (int k = 0; k < TZ; ++k) {
            double A0, A1, A2, even, odd;
            shell.coef(st[k].U, st[k].t, A0, A1, A2);
            double c = fmadd(ey, st[k].ru[1], ex * st[k].ru[0]);
            if constexpr (D == 3) c = fmadd(ez, st[k].ru[2], c);
            pair_parts(A0, A1, A2, c, even, odd);
            pair_finish(even, odd, w, st[k].rho, 0.0, gp[k], gm[k]);
            pair_finish(even, odd, w, st[k].rho_h, 0.0, hp[k], hm[k]);
        }
        const int p0 = 2 + 4 * n;  // planes g, h of the first member, g, h of the second
        double x[TZ], y[TZ], xh[TZ];
        meet(W{});
        fetch(b3, n, v, J3{});
        compute(Up{}, b0, ex, v.y, my, em, mm, omf, gp, x);
        store(p0, x);
        meet(W{});
        fetch(b0, next, nv, J0{});
        compute(Up{}, b1, ex, v.y, my, em, mm, omg, hp, xh);
        store(p0 + 1, xh);
        meet(W{});
        fetch(b1, next, nv, J1{});
        compute(Down{}, b2, ex, -v.y, my, -em, mm, omf, gm, y);
        store(p0 + 2, y);
        // a pair's sum and difference first: half as many roundings at the
        // size of the totals
#pragma unroll
        for (int k = 0; k < TZ; ++k) {
            const double sum = x[k] + y[k], dif = x[k] - y[k];
            sums[k][0] += sum;
            sums[k][1] = fmadd(ex, dif, sums[k][1]);
            sums[k][2] = fmadd(ey, dif, sums[k][2]);
            if constexpr (D == 3) sums[k][3] = fmadd(ez, dif, sums[k][3]);
            sums[k][4] = fmadd(qn, sum, sums[k][4]);
        }
        meet(W{});
        fetch(b2, next, nv, J2{});
        compute(Down{}, b3, ex, -v.y, my, -em, mm, omg, hm, y);
        store(p0 + 3, y);
#pragma unroll
        for (int k = 0; k < TZ; ++k) sums[k][5] += xh[k] + y[k];
        v = nv;
    }
    {
        const Shell<D> shell(r2, 0);
        double g[TZ], h[TZ], x[TZ];
#pragma unroll
        for (int k = 0; k < TZ; ++k) {
            double A0, A1, A2;
            shell.coef(st[k].U, st[k].t, A0, A1, A2);
            g[k] = rest_target(A0, ph.w[0], st[k].rho, 0.0);
            h[k] = rest_target(A0, ph.w[0], st[k].rho_h, 0.0);
        }
        meet(W{});
        compute(Up{}, b0, 0.0, 0, 0.0, 0, 0.0, omf, g, x);
        store(0, x);
#pragma unroll
        for (int k = 0; k < TZ; ++k) sums[k][0] += x[k];
        meet(W1{});
        compute(Up{}, b1, 0.0, 0, 0.0, 0, 0.0, omg, h, x);
        store(1, x);
#pragma unroll
        for (int k = 0; k < TZ; ++k) sums[k][5] += x[k];
    }
    wait_vm<0>();  // no load into LDS outlives the workgroup
    // the next record
#pragma unroll
    for (int k = 0; k < TZ; ++k) {
        auto put = [&](int f, double x) {
            buf_store<false>(row_rsrc(rec + (size_t)f * a.P, k), v_cell, k * mstride, x);
        };
        double rho, drho, u[3] = {0, 0, 0}, t;
        macro<D, double, false>(sums[k][0], sums[k] + 1, sums[k][4], sums[k][5], ph.r, ph.inv_dof,
                                ph.half_delta, rho, drho, u, t);
        put(0, rho);
#pragma unroll
        for (int d = 0; d < D; ++d) put(1 + d, u[d]);
        put(D + 1, t);
        if (ph.ec != 0) {
            Equilibrium<D, double, false> eq;
            eq.setup(u, t, ph.r);
            put(D + 2, energy_fix_kr<D, double, false>(ph, rho, eq, 0.0, sums[k][4]));
        }
    }
}

// Streamed stores where rows are whole cache lines; otherwise cached ones, so
// that the two halves of a line meet in the L2.
template <int D, int TY>
hipError_t launch_tiles(const StepArgs& a0, double* rec, hipStream_t s) {
    constexpr int TZ = kTileZ;
    // waves per SIMD the LDS of four planes leaves room for
    constexpr int WAVES = D == 3 && TY == 4 ? 1 : 2;
    StepArgs a = a0;
    a.fd_tx = (a.nx + 63) / 64;
    a.fd_ty = D == 3 ? (a.ny + TY - 1) / TY : (a.ny + TY * TZ - 1) / (TY * TZ);
    a.fd_tz = D == 3 ? (a.nz + TZ - 1) / TZ : 1;
    // bricks of up to 64 tiles (about what an XCD runs at one time), smaller
    // while that leaves fewer than four for each XCD
    const int64_t tiles = (int64_t)a.fd_tx * a.fd_ty * a.fd_tz;
    int64_t vol = tiles / 32 < 64 ? tiles / 32 : 64;
    if (vol < 1) vol = 1;
    a.fd_bw = a.fd_tx < 4 ? a.fd_tx : 4;
    if (a.fd_bw > vol) a.fd_bw = (int)vol;
    a.fd_bh = a.fd_bd = 1;
    while (2LL * a.fd_bw * a.fd_bh * a.fd_bd <= vol) {
        if (D == 3 && a.fd_bd * TZ < a.fd_bh * TY && a.fd_bd < a.fd_tz) a.fd_bd *= 2;
        else if (a.fd_bh < a.fd_ty) a.fd_bh *= 2;
        else if (D == 3 && a.fd_bd < a.fd_tz) a.fd_bd *= 2;
        else break;
    }
    const int64_t bricks = (int64_t)((a.fd_tx + a.fd_bw - 1) / a.fd_bw) *
                           ((a.fd_ty + a.fd_bh - 1) / a.fd_bh) * ((a.fd_tz + a.fd_bd - 1) / a.fd_bd);
    const int64_t grid = 8 * ((bricks + 7) / 8) * (int64_t)(a.fd_bw * a.fd_bh * a.fd_bd);
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    const double* src = static_cast<const double*>(a.src);
    double* dst = static_cast<double*>(a.dst);
    if (a.nx % 16 == 0)
        return launch_kernel(&k_fd_tile<D, TY, true, WAVES>, dim3((unsigned)grid), dim3(64 * TY),
                             s, src, dst, rec, a);
    return launch_kernel(&k_fd_tile<D, TY, false, WAVES>, dim3((unsigned)grid), dim3(64 * TY), s,
                         src, dst, rec, a);
}

// LDS: the staged kernel (its 16-byte row loads need every row to start on a
// tile boundary).
template <int D, class P, bool LDS, bool NT, int C = 0>
hipError_t launch_chunks(const StepArgs& a, typename P::T* rec, int grid, hipStream_t s) {
    if constexpr (C == chunk_count<D>()) {
        return hipSuccess;
    } else {
        constexpr int c0 = chunk_begin<D>(C), c1 = chunk_end<D>(C);
        hipError_t e;
        if constexpr (LDS)
            e = launch_kernel(&k_fd_update_lds<D, P, c0, c1, kFdPhase<D, P>, NT>, dim3(grid),
                              dim3(256), s, a.src, a.dst, rec, a);
        else
            e = launch_kernel(&k_fd_update<D, P, c0, c1, NT>, dim3(grid), dim3(256), s, a.src,
                              a.dst, rec, a);
        if (e != hipSuccess) return e;
        return launch_chunks<D, P, LDS, NT, C + 1>(a, rec, grid, s);
    }
}

// Bytes of the planes that one update chunk's stencils keep live: the
// reuse window (the slabs z-2 .. z+2 of a sub-band's x-chunk in 3D, the rows
// y-2 .. y+2 of an x-chunk in 2D) is held within this much of an XCD's L2.
constexpr int64_t kFdWindowBytes = 2 << 20;

// The sweep of an update chunk's launch over the grid (sweep_tile): sets the
// sweep fields of `a`, returns the number of workgroups.
template <int D, typename S>
int64_t chunk_sweep(StepArgs& a) {
    // one x-row tile of one chunk's planes (at most 14 populations, g and h)
    const int64_t tile_bytes = 256LL * 2 * kChunkW<D> * (int64_t)sizeof(S);
    a.tiles_per_row = (a.nx + 255) / 256;
    // tiles in a reuse window; D3Q107 FP64 gets twice the bytes (40^3 133 us a
    // step, 147 without; 1100x1100x1 2050 and 2430)
    const int64_t window = (D == 3 && sizeof(S) == 8) ? 2 * kFdWindowBytes : kFdWindowBytes;
    int64_t budget = window / (5 * tile_bytes);
    if (budget < 1) budget = 1;
    // x-chunks of whole rows when they fit
    a.fd_w = (int)(a.tiles_per_row < budget ? a.tiles_per_row : budget);
    if (D == 3) {
        // the window is 5 slabs of YB x W tiles: the tallest sub-band within
        // it that splits y into k rounds of eight (every XCD takes the same
        // number of sub-bands)
        const int64_t max_yb = budget / a.fd_w;
        int k = 1;
        while ((a.ny + 8 * k - 1) / (8 * k) > max_yb && 8 * k < a.ny) ++k;
        a.fd_yb = (a.ny + 8 * k - 1) / (8 * k);
    } else {
        // one sub-band per XCD; the window is 5 rows of a W-tile chunk
        a.fd_yb = (a.ny + 7) / 8;
    }
    const int chunks = (a.tiles_per_row + a.fd_w - 1) / a.fd_w;
    const int subs = (a.ny + a.fd_yb - 1) / a.fd_yb;
    const int rounds = (subs + 7) / 8;
    return 8LL * rounds * chunks * a.fd_w * a.fd_yb * a.nz;
}

// How long such a launch is, in waves one after the other on a SIMD, times
// four: the workgroups of a CU (32 CUs take an XCD's) times the waves of one
// that have cells.  D2Q37 FP64 takes 8 us + 3.7 us times this a step of two
// launches: 23 us at 4, 30 at 6, 37 at 8, 44 at 9, 52 at 12.
int64_t chunk_load(int nx, int64_t grid) {
    const int waves = (nx + 63) / 64;
    return ((grid / 8 + 31) / 32) * (waves < 4 ? waves : 4);
}

// Whether a grid (FP64) goes to k_fd_tile.  A tile's walk through the planes
// takes 160 us (3D) or 44 us (2D) however few tiles there are; on smaller grids
// k_fd_update is done sooner.  Both at the line (update, tiles): D3Q107 40^3 (64k
// cells) 131 and 162 us, 48^3 (111k) 213 and 161; D2Q37 2000x50 (load 8) 38
// and 45, 65x1231 (10) 46 and 44, 1500x67 (12) 52 and 44.  In 3D with one plane in z
// a tile is a quarter full at best: 300x300x1 257 and 473, 1100x1100x1 2060 and
// 2650, but 300x300x3 650 and 485, 600x600x2 1220 and 900.
template <int D>
bool fd_tiles(StepArgs a) {
    if constexpr (D == 3) return a.N >= 78000 && a.nz > 1;
    else return chunk_load(a.nx, chunk_sweep<2, double>(a)) >= 10;
}

template <int D, class P>
hipError_t fd_two_pass_impl(const StepArgs& a0, void* rec_v, bool record_valid, hipStream_t s) {
    using T = typename P::T;
    StepArgs a = a0;
    T* rec = static_cast<T*>(rec_v);
    const int tiles = (int)((a.N + 255) / 256);
    if (!record_valid) {
        hipError_t e = launch_kernel(&k_fd_moments<D, P>, dim3(tiles), dim3(256), s, a.src, rec,
                                     a.N, a.P, a.ph);
        if (e != hipSuccess) return e;
    }
    if constexpr (!P::kDev) {
        if (fd_tiles<D>(a)) {
            if constexpr (D == 3) {
                // 64 x 8 x 4 cells, or 64 x 4 x 4 where no CU gets two of those
                // (1000x16x16: 279 us a step with 128 of the larger, 185 with
                // 256 of the smaller; 300x300x2 450 with 190, 480 with 375) and
                // where the larger have no more rows to serve (20000x2x2 440, 316)
                const int64_t tiles4 = (int64_t)((a.nx + 63) / 64) * ((a.ny + 3) / 4) *
                                       ((a.nz + kTileZ - 1) / kTileZ);
                if (tiles4 <= 256 || a.ny <= 4) return launch_tiles<D, 4>(a, rec, s);
                return launch_tiles<D, 8>(a, rec, s);
            } else {
                return launch_tiles<D, 4>(a, rec, s);
            }
        }
    }
    const int64_t grid = chunk_sweep<D, typename P::S>(a);
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    // Stores: streamed where rows are whole cache lines (elsewhere the two
    // halves of a line meet in the L2: FP32 191x173x187 5740 us a step
    // streamed, 5570 cached, 2000x30 31 and 25) and the state does not stay in
    // the caches (D2Q37 FP32 256^2, 39 MB: 23.3 and 24.0; 1024x100, 61 MB: 35.5
    // and 27.2; D3Q107 FP32 48^3, 189 MB: 125 and 98; 64^3, 449 MB: 221 and 239;
    // D2Q37 FP64 512x48, 29 MB: 21.9 and 22.2; 1600x16, 30 MB: 26.3 and 22.4;
    // 400x100, 47 MB: 27.5 and 22.9; D3Q107 FP64 128x8x8, 28 MB: 88 and 75)
    constexpr int64_t least = int64_t(P::kDev ? 48 : 24) << 20;
    const int64_t state = state_bytes(D, sizeof(typename P::S), a.P);
    const bool stays = state > least && state <= (int64_t(256) << 20);
    const bool nt = !stays && a.nx * sizeof(typename P::S) % 128 == 0;
    if (a.nx % 256 == 0) {
        if constexpr (P::kDev) {
            return nt ? launch_chunks<D, P, true, true>(a, rec, (int)grid, s)
                      : launch_chunks<D, P, true, false>(a, rec, (int)grid, s);
        } else if constexpr (D == 3) {
            // one plane in z, and grids just short of the tiles (256x16x17: 133 us
            // staged, 143 not; 256x16x16, a workgroup a CU: 121 and 100;
            // 256x400x1 146 and 187, 1024x1024x1 1147 and 1540)
            if (chunk_load(a.nx, grid) > 4)
                return launch_chunks<D, P, true, true>(a, rec, (int)grid, s);
        }
    }
    return nt ? launch_chunks<D, P, false, true>(a, rec, (int)grid, s)
              : launch_chunks<D, P, false, false>(a, rec, (int)grid, s);
}

}  // namespace

// D2Q37 in FP64 only (D3Q107 FP64 48x13x11: 80 us from the record; 64^3 and up two
// to four times as long fused).  us a step, fused / chunks / tiles:
//   small grids, where one launch is done before two: 1000x16 21 / 23 / 44, 2000x12
//   21 / 22, 300x80 23 / 22;
//   up to four rows: three of a tile's four waves have no cells, and the chunks,
//   dealt to the XCDs by rows, leave half of them idle: 40000x3 47 / 84 / 94,
//   100000x1 41 / 196 / 198, 1000000x3 1350 / 2550 / 1680 (40000x6: 104 / 124 / 96);
//   up to one wave a SIMD (1024 of 64 cells of a row), with more than one of
//   the chunks': 300x133 25 / 37 / 44, 150x267 24 / 30 / 44 (500x128, one of the
//   chunks': 33 / 24);
//   and up to two, where the tiles are more than the CUs: 16400x5 42 fused, 57 in
//   tiles, 24000x5 54 and 59.
bool fd_fused_by_default(int dim, int precision, int64_t nx, int64_t ny) {
    if (dim != 2 || precision != LBM_FP64) return false;
    if (nx * ny < 25000 || ny <= 4) return true;
    StepArgs a{};
    a.nx = (int32_t)nx;
    a.ny = (int32_t)ny;
    a.nz = 1;
    const int64_t load = chunk_load(a.nx, chunk_sweep<2, double>(a));
    const int64_t cols = (nx + 63) / 64, waves = cols * ny, tiles = cols * ((ny + 15) / 16);
    if (load >= 10) return waves <= 2048 && tiles > 256;
    return waves <= 1024 && load > 4;
}

size_t fd_record_bytes(int dim, int precision, int64_t P) {
    const bool dev = precision != LBM_FP64;  // record (deviation storage: residuals too)
    const int fields = dim == 2 ? (dev ? kRecFields<2, true> : kRecFields<2, false>) + kAccFields<2>
                                : (dev ? kRecFields<3, true> : kRecFields<3, false>) + kAccFields<3>;
    return (size_t)fields * (size_t)P * (precision == LBM_FP64 ? 8 : 4);
}

hipError_t launch_fd_init(int dim, int precision, void* dst, void* record, const InitFields& f,
                          const Physics& ph, const double* w_group, hipStream_t s) {
    const WGroups wg = groups_of(w_group);
    const dim3 grid((unsigned)((f.N + 255) / 256)), block(256);
    char* d = static_cast<char*>(dst);
    if (precision == LBM_FP64) {
        double* rec = static_cast<double*>(record);
        return launch_kernel(dim == 2 ? &k_fd_init<2, F64> : &k_fd_init<3, F64>, grid, block, s, d,
                             rec, f, wg, ph);
    }
    if (precision != LBM_FP32_DEV) return hipErrorInvalidValue;  // no half storage in this form
    float* rec = static_cast<float*>(record);
    return launch_kernel(dim == 2 ? &k_fd_init<2, F32Dev> : &k_fd_init<3, F32Dev>, grid, block, s,
                         d, rec, f, wg, ph);
}

hipError_t launch_fd_two_pass(int dim, int precision, const StepArgs& a, void* record,
                              bool record_valid, hipStream_t s) {
    if (precision == LBM_FP64)
        return dim == 2 ? fd_two_pass_impl<2, F64>(a, record, record_valid, s)
                        : fd_two_pass_impl<3, F64>(a, record, record_valid, s);
    if (precision == LBM_FP32_DEV)
        return dim == 2 ? fd_two_pass_impl<2, F32Dev>(a, record, record_valid, s)
                        : fd_two_pass_impl<3, F32Dev>(a, record, record_valid, s);
    return hipErrorInvalidValue;
}

}  // namespace lbm
