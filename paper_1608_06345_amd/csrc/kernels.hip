// HIP kernels for gfx950: initialisation, the fused collide-and-stream step,
// the fused finite-difference step (Sec. III; the one that works from a record
// is in fd.hip), and the FP64 readout / conservation reductions.
//
// Data layout in HBM (one ping-pong side): population i owns a slab of 2 P
// values (P >= N, x fastest).  FP64 and FP32: the g plane, then the h plane
// ([Q][2][P]); half storage: the g and h halves of a cell side by side in
// one 32-bit word ([Q][P][2]; cell_bytes, h_offset).  Every value is read
// once and written once per step: one HBM read and one HBM write per
// population per cell.
//
// The step (Sec. II reduced BGK equations, Sec. IV equilibrium, lattice time
// step of Sec. V) at cell x:
//   1. pull   g_i(x) <- g_i'(x - e_i), h_i likewise (periodic wrap, or clamp
//             at a zero-gradient end), straight from the other ping-pong side;
//   2. moments rho = sum g_i, rho u = r sum e_i g_i,
//             rho E = r^2/2 sum |e_i|^2 g_i + sum h_i, T from
//             E = u^2/2 + (D + delta) T / 2;
//   3. equilibrium F_i = w_i rho P(c_i), c_i = xi_i . u, P the 4th-order
//             Hermite polynomial, evaluated as even/odd parts per +/- pair;
//   4. relax  g_i' = g_i + (F_i - g_i)/tau_f,
//             h_i' = h_i + ((delta/2) T F_i - h_i)/tau_g;
//   5. store  g_i', h_i' at x (coalesced).
// The D3Q107 step also comes with its pulled rows staged in LDS
// (k_step_split_lds, variant SPLIT_LDS): same results, measured slower.
#include <tuple>
#include <type_traits>
#include <utility>

#include "lbm_internal.h"
#include "step_core.h"

namespace lbm {
namespace {

using namespace core;

// First cell of the L cells this wave serves; false if there are none.  Waves
// take consecutive cells whatever the row length: every store is then whole
// 128-byte lines.  (With waves that stopped at row ends, a row that was no
// multiple of a line made each wave write two half lines: D2Q37 FP16 on
// 2047x1531 ran at 3.4 TB/s, D3Q107 FP16 on 191x173x187 at 2.7, and 5.3 and
// 5.2 where rows were whole lines.  Now 273 -> 167 us and 1816 -> 987 us a
// step there, and the same or 1-5% less on whole-line rows, where only the
// y and z offsets have moved from scalar to vector registers.)  The
// hardware deals workgroups to the eight XCDs round-robin by id: workgroup b
// is turn j = b / 8 of XCD b % 8.  The turns of one XCD walk runs of a.run
// consecutive tiles (a.waves waves each; about one row), so that the cache lines
// that x-shifted pulls share between neighbouring waves are fetched into one
// L2 once, while the eight XCDs together still sweep one compact band of
// rows.
template <int L>
__device__ __forceinline__ bool wave_cells(const StepArgs& a, int& first) {
    const int b = (int)blockIdx.x, j = b >> 3;
    const int tile = ((j / a.run) * 8 + (b & 7)) * a.run + j % a.run;
    const int wave = tile * a.waves + (int)(threadIdx.x >> 6);
    first = __builtin_amdgcn_readfirstlane(wave * L);
    return first < (int)a.N;
}

// Fused step, one lane per cell: the lane holds all 2Q populations.  A wave
// serves 64 consecutive cells.  P is the storage precision (F64, F32Dev,
// F16Dev).
template <int D, class P, int WAVES, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES, 8)))
void k_step(const StepArgs a) {
    using S = typename P::S;
    int first;
    if (!wave_cells<64>(a, first)) return;
    // Lanes past the last cell hold that cell (clamped), loaded and updated
    // exactly like the lane that owns it, so they store the same bits to the
    // same place.  No branch: a branch here lets the compiler sink the whole
    // relaxation into the store block and keep every target and population
    // live at once.
    const int cell = min(first + ((int)threadIdx.x & 63), (int)a.N - 1);
    CellOffsets<D, S> o;
    o.fill(cell, a.nx, a.ny, a.nz, a.nxy, a.pull, 0u);
    const uint32_t plane = (uint32_t)a.P * (uint32_t)sizeof(S);
    step_lane_cell<D, P, NT>(static_cast<const char*>(a.src), static_cast<char*>(a.dst), plane, o,
                         a.ph);
}

// Fused step, split layout (see collide_split): a wave serves 32
// consecutive cells.  This halves the registers a lane needs (Q instead of 2Q values).
template <int D, class P, int WAVES, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES, 8)))
void k_step_split(const StepArgs a) {
    using T = typename P::T;
    using S = typename P::S;
    constexpr int Q = VelSet<D>::Q;
    const int lane = (int)threadIdx.x & 63;
    const int role = lane >> 5;  // 0: g, 1: h
    const uint32_t plane = (uint32_t)a.P * (uint32_t)sizeof(S);
    int first;
    if (!wave_cells<32>(a, first)) return;
    // lanes past the last cell repeat it (see k_step)
    const int cell = min(first + (lane & 31), (int)a.N - 1);
    CellOffsets<D, S> o;
    o.fill(cell, a.nx, a.ny, a.nz, a.nxy, a.pull, role ? h_offset(sizeof(S), plane) : 0u);
    T p[Q];
    load_split<D, P>(static_cast<const char*>(a.src), plane, o, p, a.ph);
    collide_split<D, P>(p, role, a.ph);
    store_split<D, P, NT>(static_cast<char*>(a.dst), plane, o.own, p, a.ph);
}

// Fused step, split layout, with the pulled rows staged in LDS (D3Q107;
// rows of whole 128-cell tiles).  A workgroup serves one 128-cell tile of a
// row, its four waves 32 cells each as in k_step_split.  The pull of
// population i reads the tile's row shifted by e_i: row (y - e_y, z - e_z),
// cells x0 - e_x .. x0 - e_x + 127.  Instead of one 4-byte (or 2-byte) load
// per lane and population, the workgroup loads that row once with 4-cell
// loads per lane -- lanes 0..31 the g row, lanes 32..63 the h row, one
// instruction per population -- plus up to three halo cells either side,
// stages it in LDS, and each lane takes its cell's pulled value from there.
// Populations go through LDS in batches of kLdsBatch; the next batch's loads
// are issued before the current one is read back.  Collision and store are
// k_step_split's.
constexpr int kLdsBatch = 16;
constexpr int kLdsRow = 136;  // slots per staged row: 4 (3 halo), 128 cells, 4 (3 halo)

template <class P, int WAVES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES, 8)))
void k_step_split_lds(const StepArgs a) {
    constexpr int D = 3;
    using T = typename P::T;
    using S = typename P::S;
    typedef S S4 __attribute__((ext_vector_type(4)));
    typedef S S8 __attribute__((ext_vector_type(8)));
    // half storage: g/h words, two elements per cell (see cell_bytes)
    constexpr bool kPaired = sizeof(S) == 2;
    constexpr int64_t kCellElems = kPaired ? 2 : 1;
    constexpr VelSet<D> V = kVelSet<D>;
    constexpr int Q = VelSet<D>::Q;
    __shared__ __attribute__((aligned(16))) S lds[kLdsBatch * 2 * kLdsRow];
    // workgroup b: turn j = b / 8 on XCD b % 8 walks whole rows
    const int b = (int)blockIdx.x;
    const int j = b >> 3;
    const int row = (j / a.tiles_per_row) * 8 + (b & 7);
    if (row >= a.rows) return;  // the whole workgroup
    const int tile = j % a.tiles_per_row;
    const int y = row % a.ny, z = row / a.ny;
    const int x0 = tile * 128;
    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int role = lane >> 5;  // 0: g, 1: h
    const int c = wave * 32 + (lane & 31);  // the lane's cell in the tile
    const bool open_x = a.open_end & 1u, open_y = a.open_end & 2u, open_z = a.open_end & 4u;
    const int64_t N = a.P;  // plane stride
    const S* src = static_cast<const S*>(a.src);
    // halo lanes (k = lane & 31 < 6): cells x0 - 3 .. x0 - 1, x0 + 128 .. x0 + 130
    const int hk = lane & 31;
    const int hshift = hk < 3 ? 3 - hk : -125 - hk;  // pull shift e: source x0 - e
    const int hx = pull_coord(x0, hshift, a.nx, open_x);
    const int hslot = hk < 3 ? 1 + hk : 129 + hk;  // slots 1..3, 132..134
    // Batch loads: wave w takes the batch's populations w, w + 4, ...
    S4 q[kLdsBatch / 4];
    S hv[kLdsBatch / 4];
    auto issue = [&](auto Bt) {
        constexpr int b0 = decltype(Bt)::value * kLdsBatch;
        static_for<0, kLdsBatch / 4>([&](auto M) {
            constexpr int m = decltype(M)::value;
            // population of this slot for each wave, picked branch-free
            int64_t start = 0;
            bool has = false, hx_need = false;
            static_for<0, 4>([&](auto W) {
                constexpr int i = b0 + 4 * m + decltype(W)::value;
                if constexpr (i < Q) {
                    constexpr Vel v = V.v[i];
                    const int64_t st =
                        (int64_t)(2 * i) * N +
                        kCellElems * ((int64_t)pull_coord(y, v.y, a.ny, open_y) * a.nx +
                                      (int64_t)pull_coord(z, v.z, a.nz, open_z) * a.nxy);
                    const bool w = wave == decltype(W)::value;
                    start = w ? st : start;
                    has = w ? true : has;
                    hx_need = w ? (v.x != 0) : hx_need;
                }
            });
            hv[m] = S(0);
            if (has) {
                if constexpr (kPaired) {
                    // four cells' g/h words (16 bytes); keep this lane's halves
                    const S* rowp = src + start;
                    const S8 pw = *reinterpret_cast<const S8*>(rowp + 2 * (x0 + 4 * (lane & 31)));
                    q[m] = role ? __builtin_shufflevector(pw, pw, 1, 3, 5, 7)
                                : __builtin_shufflevector(pw, pw, 0, 2, 4, 6);
                    if (hx_need && hk < 6) hv[m] = rowp[2 * hx + role];
                } else {
                    const S* rowp = src + start + (role ? N : 0);
                    q[m] = *reinterpret_cast<const S4*>(rowp + x0 + 4 * (lane & 31));
                    if (hx_need && hk < 6) hv[m] = rowp[hx];
                }
            }
        });
    };
    T p[Q];
    constexpr int kBatches = (Q + kLdsBatch - 1) / kLdsBatch;
    issue(std::integral_constant<int, 0>{});
    static_for<0, kBatches>([&](auto Bt) {
        constexpr int bt = decltype(Bt)::value;
        constexpr int b0 = bt * kLdsBatch;
        if constexpr (bt != 0) __syncthreads();  // the previous batch's reads are done
        static_for<0, kLdsBatch / 4>([&](auto M) {
            constexpr int m = decltype(M)::value;
            // slot of population b0 + 4 m + wave
            const int pi = 4 * m + wave;
            if (b0 + pi < Q) {
                S* slot = lds + (pi * 2 + role) * kLdsRow;
                *reinterpret_cast<S4*>(slot + 4 + 4 * (lane & 31)) = q[m];
                if (hk < 6) slot[hslot] = hv[m];
            }
        });
        __syncthreads();
        if constexpr (bt + 1 < kBatches) issue(std::integral_constant<int, bt + 1>{});
        static_for<0, kLdsBatch>([&](auto K) {
            constexpr int i = b0 + decltype(K)::value;
            if constexpr (i < Q) {
                constexpr Vel v = V.v[i];
                const S x = lds[(decltype(K)::value * 2 + role) * kLdsRow + 4 + c - v.x];
                p[i] = from_store<P>(x, a.ph, v.group);
            }
        });
    });
    collide_split<D, P>(p, role, a.ph);
    const uint32_t plane = (uint32_t)N * (uint32_t)sizeof(S);
    const uint32_t own = (uint32_t)(y * a.nx + z * a.nxy + x0 + c) * cell_bytes(sizeof(S)) +
                         (role ? h_offset(sizeof(S), plane) : 0u);
    store_split<D, P, true>(static_cast<char*>(a.dst), plane, own, p, a.ph);
}

// ---------------------------------------------------------------------------
// S_0 and, from the values as stored, P_0 = Collide(S_0), in the register
// layouts of the step.  What bounds it is the two sides written: D3Q107 FP32
// 256^3 5.9 ms (S_0 alone, then a collision that read it again: 2.9 + 5.4), D2Q37
// FP64 4096^2 3.8 (1.95 + 3.75); in half storage also the double arithmetic, FP16
// 191x173x187 1.49 ms (2.0 + 1.0; 2.30 with the compiler's conversion to half).
template <int D, class P, bool SPLIT, int WAVES, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES, 8)))
void k_init_collide(char* s0, char* p0, const InitFields f, const WGroups wg, const Physics ph) {
    using T = typename P::T;
    using S = typename P::S;
    constexpr int Q = VelSet<D>::Q;
    constexpr VelSet<D> V = kVelSet<D>;
    constexpr int L = SPLIT ? 32 : 64;
    const int lane = (int)threadIdx.x & 63;
    const int role = SPLIT ? lane >> 5 : 0;
    const int first = ((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6)) * L;
    if (first >= (int)f.N) return;
    // lanes past the last cell repeat it (see k_step)
    const int cell = min(first + (SPLIT ? (lane & 31) : lane), (int)f.N - 1);
    const uint32_t plane = (uint32_t)f.P * (uint32_t)sizeof(S);
    const uint32_t ho = h_offset(sizeof(S), plane);
    const uint32_t own = (uint32_t)cell * cell_bytes(sizeof(S)) + (role ? ho : 0u);
    InitCell<D> ic;
    ic.load(f, cell);
    if constexpr (SPLIT) {
        T p[Q];
        static_for<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            S g, h;
            ic.template values<P, i>(wg, g, h);
            const S x = role ? h : g;
            store_at(s0 + (size_t)(2 * i) * plane, own, x);
            p[i] = from_store<P>(x, ph, V.v[i].group);
        });
        collide_split<D, P>(p, role, ph);
        store_split<D, P, NT>(p0, plane, own, p, ph);
    } else if constexpr (P::kScaled) {
        uint32_t w[Q];
        static_for<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            S g, h;
            ic.template values<P, i>(wg, g, h);
            w[i] = (uint32_t)__builtin_bit_cast(uint16_t, g) |
                   (uint32_t)__builtin_bit_cast(uint16_t, h) << 16;
            store_at(s0 + (size_t)(2 * i) * plane, own, w[i]);
        });
        collide_words<D, P, NT>(w, p0, plane, own, ph);
    } else {
        T g[Q], h[Q];
        static_for<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            ic.template values<P, i>(wg, g[i], h[i]);
            // the collision takes the values as stored, not the products
            // they were rounded from
            asm("" : "+v"(g[i]), "+v"(h[i]));
            store_at(s0 + (size_t)(2 * i) * plane, own, g[i]);
            store_at(s0 + (size_t)(2 * i) * plane + ho, own, h[i]);
        });
        collide_lane<D, P>(g, h, ph);
        store_lane<D, P, NT>(p0, plane, own, g, h, ph);
    }
}

// ---------------------------------------------------------------------------
// The finite-difference form (Sec. III): explicit Euler in time, third-order
// upwind-biased convection per axis, BGK with rates dt / tau.  A wave loads
// the centre values of its cells, collides them in registers (taking the
// convection centre term with them), then reads each population's upwind
// neighbours from the time-n state and stores the new value.  The
// neighbour reads come from cache.  Waves go out in launch order (row by
// row).  Ordering them in per-XCD y bands, whole or in x-chunks, was
// measured: at most 5% faster in 3D, 9% slower in 2D.  The rows around the
// cells in flight on one XCD, over all 2Q planes, exceed its L2 either way.
template <int D, typename S, int L>
__device__ __forceinline__ bool fd_item(const StepArgs& a, int lane_cell, uint32_t role_off,
                                        RowOffsets<S>& o) {
    const int item = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (item >= a.items) return false;
    int seg = item % a.segs;
    const int row = item / a.segs;
    int y = row % a.ny;
    int z = row / a.ny;
    seg = __builtin_amdgcn_readfirstlane(seg);
    y = __builtin_amdgcn_readfirstlane(y);
    z = __builtin_amdgcn_readfirstlane(z);
    const int xr = seg * L + lane_cell;
    const int x = xr < a.nx ? xr : a.nx - 1;  // tail lanes repeat the last cell
    fill_row_offsets<D, S>(o, x, y, z, a.nx, a.ny, a.nz, a.nxy, a.open_end, role_off);
    return true;
}

template <int D, class P, bool SPLIT, int WAVES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES, 8)))
void k_fd_step(const StepArgs a) {
    using T = typename P::T;
    using S = typename P::S;
    constexpr int Q = VelSet<D>::Q;
    const int lane = (int)threadIdx.x & 63;
    const uint32_t plane = (uint32_t)a.P * (uint32_t)sizeof(S);
    const char* src = static_cast<const char*>(a.src);
    char* dst = static_cast<char*>(a.dst);
    RowOffsets<S> o;
    if constexpr (SPLIT) {
        const int role = lane >> 5;  // 0: g, 1: h (see collide_split)
        if (!fd_item<D, S, 32>(a, lane & 31, role ? h_offset(sizeof(S), plane) : 0u, o)) return;
        T p[Q];
        load_centre_split<D, P>(src, plane, o, p, a.ph);
        collide_split<D, P, true>(p, role, a.ph);
        convect_store_split<D, P>(src, dst, plane, o, p, a.ph);
    } else {
        if (!fd_item<D, S, 64>(a, lane, 0u, o)) return;
        T g[Q], h[Q];
        load_centre_lane<D, P>(src, plane, o, g, h, a.ph);
        collide_lane<D, P, true>(g, h, a.ph);
        convect_store_lane<D, P>(src, dst, plane, o, g, h, a.ph);
    }
}

// ---------------------------------------------------------------------------
// Readout of S_n in double (Sec. II moments): per-cell rho, u, E, T and/or
// per-workgroup partial totals (rho, rho u, rho E), reduced across the wave
// and the workgroup in a fixed order.
template <int D, class P>
__global__ __launch_bounds__(kReadBlock) void k_readout(const ReadArgs a) {
    constexpr VelSet<D> V = kVelSet<D>;
    constexpr int Q = VelSet<D>::Q;
    constexpr int NT = D + 2;
    // tiles of kReadBlock cells, dealt to the XCDs in runs like the step's
    // (wave_cells): the cache lines that shifted pulls share are fetched once
    const int b = (int)blockIdx.x, j = b >> 3;
    const int tile = ((j / a.run) * 8 + (b & 7)) * a.run + j % a.run;
    if (tile >= a.blocks) return;  // the whole workgroup
    const int64_t cell = (int64_t)tile * kReadBlock + threadIdx.x;
    double tot[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) tot[k] = 0.0;
    if (cell < a.N) {
        using S = typename P::S;
        CellOffsets<D, S> o;
        o.fill((int)cell, a.nx, a.ny, a.nz, a.nxy, a.pull, 0u);
        constexpr bool DEV = P::kDev;
        const uint32_t plane = (uint32_t)a.P * (uint32_t)sizeof(S);
        const char* src = static_cast<const char*>(a.src);
        double s0 = 0, sj[3] = {0, 0, 0}, se = 0, sh = 0;
        static_for<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            constexpr Vel v = V.v[i];
            const uint32_t off = o.template src<v.x, v.y, v.z>();
            const char* base = src + (size_t)(2 * i) * plane;
            const double scale = P::kScaled ? a.w[v.group] : 1.0;
            const double gv = (double)load_at<S>(base, off) * scale;
            const double hv = (double)load_at<S>(base, off + h_offset(sizeof(S), plane)) * scale;
            s0 += gv;
            if constexpr (v.x != 0) sj[0] += double(v.x) * gv;
            if constexpr (v.y != 0) sj[1] += double(v.y) * gv;
            if constexpr (D == 3 && v.z != 0) sj[2] += double(v.z) * gv;
            se += double(V.qn[v.group]) * gv;
            sh += hv;
        });
        const double rho = DEV ? 1.0 + s0 : s0;
        const double rhoE = 0.5 * a.r * a.r * se + sh + (DEV ? a.rest_energy : 0.0);
        tot[0] = rho;
#pragma unroll
        for (int k = 0; k < D; ++k) tot[1 + k] = a.r * sj[k];
        tot[D + 1] = rhoE;
        if (a.rho) a.rho[cell] = rho;
        if (a.u) {
#pragma unroll
            for (int k = 0; k < D; ++k) a.u[k * a.N + cell] = tot[1 + k] / rho;
        }
        if (a.E) a.E[cell] = rhoE / rho;
        if (a.T) {
            // Sec. II: E = |u|^2 / 2 + (D + delta) T / 2
            double uu = 0.0;
#pragma unroll
            for (int k = 0; k < D; ++k) uu += (tot[1 + k] / rho) * (tot[1 + k] / rho);
            a.T[cell] = (2.0 * (rhoE / rho) - uu) * a.inv_dof;
        }
    }
    if (!a.partials) return;
    // wave reduction (fixed butterfly), then across the 4 waves in order
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        double v = tot[k];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
        tot[k] = v;
    }
    __shared__ double wsum[kReadBlock / 64][NT];
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < NT; ++k) wsum[wave][k] = tot[k];
    }
    __syncthreads();
    if (threadIdx.x < NT) {
        double v = 0.0;
        for (int w = 0; w < kReadBlock / 64; ++w) v += wsum[w][threadIdx.x];
        a.partials[(int64_t)tile * NT + threadIdx.x] = v;
    }
}

// Final pass: one workgroup sums the partials in a fixed order.
template <int NT>
__global__ __launch_bounds__(256) void k_final_reduce(const double* __restrict__ partials,
                                                      int blocks, double* out) {
    __shared__ double sm[256][NT];
    double acc[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) acc[k] = 0.0;
    for (int b = threadIdx.x; b < blocks; b += 256) {
#pragma unroll
        for (int k = 0; k < NT; ++k) acc[k] += partials[(int64_t)b * NT + k];
    }
#pragma unroll
    for (int k = 0; k < NT; ++k) sm[threadIdx.x][k] = acc[k];
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if ((int)threadIdx.x < s) {
#pragma unroll
            for (int k = 0; k < NT; ++k) sm[threadIdx.x][k] += sm[threadIdx.x + s][k];
        }
        __syncthreads();
    }
    if (threadIdx.x < NT) out[threadIdx.x] = sm[0][threadIdx.x];
}

// Occupancy hint for the split D3Q107 float kernels: asking for at least
// two waves per SIMD gave 4% more bandwidth than the compiler's own
// choice (three waves at 162 VGPRs).  In double, two waves (256 VGPRs,
// 30 values spilled to scratch, against one wave at 256 + 28 AGPRs) ran
// 2.4% faster in isolated timings but not in the benchmark, and the
// spills added 13% to the HBM bytes; it keeps one.  The other kernels
// run best as compiled.
template <int D, class P>
constexpr int kSplitWaves = (D == 3 && sizeof(typename P::T) == 4) ? 2 : 1;

// Stores of a step (streamed / cached, us, on one allocation in turn): D2Q37 FP32
// 512^2 (155 MB) 32.6 / 26.2, 700^2 (290 MB) 57.0 / 54.5, FP16 1024^2 (310 MB)
// 63.6 / 59.7, D3Q107 FP32 45x40x40 (123 MB) 31.1 / 25.4; beyond, D3Q107 FP32 64^3
// (449 MB) 87.8 / 90.3, 256^3 5552 / 5654 (more apart on some allocations); below,
// FP32 32^3 (56 MB) 13.6 / 14.3, D2Q37 256^2 (39 MB) 12.1 / 12.8.
bool streamed(int dim, size_t elem, int64_t P) {
    const int64_t state = state_bytes(dim, elem, P);
    return state <= (int64_t(64) << 20) || state > (int64_t(304) << 20);
}

template <int D, class P>
hipError_t init_collide_impl(bool split, void* s0, void* p0, const InitFields& f,
                             const Physics& ph, const double* w_group, hipStream_t s) {
    const int tile = split ? 128 : 256;
    const bool nt = streamed(D, sizeof(typename P::S), f.P);
    auto* kernel = split ? (nt ? &k_init_collide<D, P, true, kSplitWaves<D, P>, true>
                               : &k_init_collide<D, P, true, kSplitWaves<D, P>, false>)
                         : (nt ? &k_init_collide<D, P, false, 1, true>
                               : &k_init_collide<D, P, false, 1, false>);
    return launch_kernel(kernel, dim3((unsigned)((f.N + tile - 1) / tile)), dim3(256), s,
                         static_cast<char*>(s0), static_cast<char*>(p0), f, groups_of(w_group),
                         ph);
}

template <int D, class P>
hipError_t step_impl(bool split, const StepArgs& a0, hipStream_t s) {
    StepArgs a = a0;
    a.pull = pull_grid(a.nx, a.ny, a.nz, a.open_end);
    const int L = split ? 32 : 64;  // cells per wave
    // Up to one wave for each SIMD of the chip: workgroups of one wave, which
    // spread over all CUs (us a step, four waves / one: D3Q107 FP64 on 23x9x16,
    // 104 waves, 13.5 / 9.2, D2Q37 FP64 200x4 8.2 / 5.1, 1000x16 9.8 / 7.8).
    a.waves = (a.N + L - 1) / L <= 1024 ? 1 : 4;
    int grid;
    step_tiles(a.N, a.nx, a.waves * L, &a.run, &grid);
    const dim3 block(64 * a.waves);
    const bool nt = streamed(D, sizeof(typename P::S), a.P);
    auto* kernel = split ? (nt ? &k_step_split<D, P, kSplitWaves<D, P>, true>
                               : &k_step_split<D, P, kSplitWaves<D, P>, false>)
                         : (nt ? &k_step<D, P, 1, true> : &k_step<D, P, 1, false>);
    return launch_kernel(kernel, dim3(grid), block, s, a);
}

template <int D, class P>
hipError_t fd_step_impl(bool split, const StepArgs& a0, hipStream_t s) {
    StepArgs a = a0;
    const int L = split ? 32 : 64;
    a.segs = (a.nx + L - 1) / L;
    a.rows = a.ny * a.nz;
    a.items = a.segs * a.rows;
    const int grid = (a.items + 3) / 4;
    if (split) return launch_kernel(&k_fd_step<D, P, true, 1>, dim3(grid), dim3(256), s, a);
    return launch_kernel(&k_fd_step<D, P, false, 1>, dim3(grid), dim3(256), s, a);
}

}  // namespace

// Run `f` with the storage policy of `precision`.
template <class F>
hipError_t with_policy(int precision, F&& f) {
    if (precision == LBM_FP64) return f(F64{});
    if (precision == LBM_FP16_SCALED) return f(F16Dev{});
    return f(F32Dev{});
}

hipError_t launch_init_collide(int dim, int precision, bool split, void* s0, void* p0,
                               const InitFields& f, const Physics& ph, const double* w_group,
                               hipStream_t s) {
    return with_policy(precision, [&](auto pol) {
        using P = decltype(pol);
        return dim == 2 ? init_collide_impl<2, P>(split, s0, p0, f, ph, w_group, s)
                        : init_collide_impl<3, P>(split, s0, p0, f, ph, w_group, s);
    });
}

hipError_t launch_step_lds(int precision, const StepArgs& a0, hipStream_t s) {
    StepArgs a = a0;
    if (a.nx % 128 != 0) return hipErrorInvalidValue;
    a.rows = a.ny * a.nz;
    a.tiles_per_row = a.nx / 128;
    const int grid = 8 * a.tiles_per_row * ((a.rows + 7) / 8);
    return with_policy(precision, [&](auto pol) {
        using P = decltype(pol);
        constexpr int kWaves = sizeof(typename P::T) == 4 ? 2 : 1;
        return launch_kernel(&k_step_split_lds<P, kWaves>, dim3(grid), dim3(256), s, a);
    });
}

hipError_t launch_step(int dim, int precision, bool split, const StepArgs& a, hipStream_t s) {
    return with_policy(precision, [&](auto pol) {
        using P = decltype(pol);
        return dim == 2 ? step_impl<2, P>(split, a, s) : step_impl<3, P>(split, a, s);
    });
}

void step_tiles(int64_t N, int64_t nx, int tile, int32_t* run, int* grid) {
    const int64_t tiles = (N + tile - 1) / tile;
    // a run is about one row, as long as there are runs enough for all XCDs
    int64_t r = (nx + tile - 1) / tile;
    if (tiles < 64 * r) r = 1;
    *run = (int32_t)r;
    *grid = (int)(8 * r * ((tiles + 8 * r - 1) / (8 * r)));
}

hipError_t launch_fd_step(int dim, int precision, bool split, const StepArgs& a, hipStream_t s) {
    // no half storage in the finite-difference form (lbm_create_fd refuses it)
    if (precision == LBM_FP16_SCALED) return hipErrorInvalidValue;
    if (precision == LBM_FP64)
        return dim == 2 ? fd_step_impl<2, F64>(split, a, s) : fd_step_impl<3, F64>(split, a, s);
    return dim == 2 ? fd_step_impl<2, F32Dev>(split, a, s) : fd_step_impl<3, F32Dev>(split, a, s);
}

hipError_t launch_readout(int dim, int precision, const ReadArgs& a0, int blocks, hipStream_t s) {
    ReadArgs a = a0;
    a.pull = pull_grid(a.nx, a.ny, a.nz, a.open_end);
    if (!a.stream)
        for (PullAxis& axis : a.pull.axis)
            for (int32_t& shift : axis.shift) shift = 0;
    a.blocks = blocks;
    int grid;
    step_tiles(a.N, a.nx, kReadBlock, &a.run, &grid);
    return with_policy(precision, [&](auto pol) {
        using P = decltype(pol);
        if (dim == 2) return launch_kernel(&k_readout<2, P>, dim3(grid), dim3(kReadBlock), s, a);
        return launch_kernel(&k_readout<3, P>, dim3(grid), dim3(kReadBlock), s, a);
    });
}

hipError_t launch_final_reduce(int dim, const double* partials, int blocks, double* out,
                               hipStream_t s) {
    if (dim == 2)
        return launch_kernel(&k_final_reduce<4>, dim3(1), dim3(256), s, partials, blocks, out);
    else
        return launch_kernel(&k_final_reduce<5>, dim3(1), dim3(256), s, partials, blocks, out);
}

}  // namespace lbm
