// Internal declarations shared by the host runtime and the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <tuple>
#include <type_traits>
#include <utility>

#include "lbm.h"
#include "velocity_set.h"

namespace lbm {

// Lattice constants derived on the host (lattice.cpp).
struct LatticeTables {
    int dim, q, groups;
    double r;
    double w_group[10];
    double w[107];
    int8_t e[107][3];
    int group[107];
};
const LatticeTables& lattice_tables(int dim);

// Group weights and their reciprocals by value (kernel argument).
struct WGroups {
    double w[10], inv_w[10];
};
inline WGroups groups_of(const double* w_group) {
    WGroups wg;
    for (int k = 0; k < 10; ++k) {
        wg.w[k] = w_group[k];
        wg.inv_w[k] = 1.0 / w_group[k];
    }
    return wg;
}

// Initial fields on the device, and what the equilibrium takes beside them.
struct InitFields {
    const double* rho;  // [N]
    const double* u;    // [D][N]
    const double* T;    // [N]
    int64_t N, P;       // cells; plane stride in cells
    double half_delta, r;
};

// Physical parameters of one solve as the collision uses them.
struct Physics {
    double omega_f, omega_g;  // 1 / tau (lattice scheme), dt / tau (finite differences)
    double half_delta;        // delta / 2
    double inv_dof;           // 1 / (D + delta)
    double r;                 // lattice scale, xi = r e
    double w[10];             // group weights
    float wf[10];             // the same, rounded to float
    float inv_wf[10];         // 1 / w (scaling of half-precision storage)
    double fd_cs;             // finite differences: dt r / 6 (0 for the lattice scheme)
    float fd_csf;             // the same, rounded to float
    double ec;                // energy-conserving collision: 1 - tau_g / tau_f, else 0
    float ecf;                // the same, rounded to float
};

// Division of 0 <= n < 2^31 by a divisor d >= 1 known to the host: with l =
// ceil(log2 d) and mul = ceil(2^(31 + l) / d) < 2^32, n mul / 2^(31 + l) exceeds
// n / d by less than 1 / d, so that (2 n mul) >> (32 + l) is the quotient.
struct Divisor {
    uint32_t mul, shift;
};
inline Divisor divisor_of(int64_t d) {
    uint32_t l = 0;
    while ((int64_t(1) << l) < d) ++l;
    const uint64_t p = uint64_t(1) << (31 + l);
    return {(uint32_t)((p + (uint64_t)d - 1) / (uint64_t)d), l};
}

// Where a pull reads along one axis of n cells: e = 1, 2, 3 cells away, taken
// modulo n on a periodic axis, one turn of n (none at open ends) bringing it
// back.
struct PullAxis {
    int32_t turn;
    int32_t shift[3];
};
struct PullGrid {
    PullAxis axis[3];
    Divisor by_nx, by_nxy;
};
inline PullGrid pull_grid(int64_t nx, int64_t ny, int64_t nz, uint32_t open_end) {
    PullGrid g;
    const int64_t n[3] = {nx, ny, nz};
    for (int k = 0; k < 3; ++k) {
        const bool open = open_end >> k & 1u;
        g.axis[k].turn = open ? 0 : (int32_t)n[k];
        for (int e = 1; e <= 3; ++e)
            g.axis[k].shift[e - 1] = open ? e : (int32_t)(e % n[k]);
    }
    g.by_nx = divisor_of(nx);
    g.by_nxy = divisor_of(nx * ny);
    return g;
}

// Arguments of the fused step kernel (passed by value in the kernarg
// segment, so every field is wave-uniform and lives in SGPRs).
struct StepArgs {
    const void* src;      // one ping-pong side (layout: cell_bytes, h_offset)
    void* dst;            // same layout
    int64_t N;            // cells
    int64_t P;            // plane stride in cells (>= N; see plane_stride)
    int32_t nx, ny, nz;
    int32_t nxy;          // nx * ny
    uint32_t open_end;    // bit k: axis k is zero-gradient, else periodic
    PullGrid pull;        // lattice step
    int32_t run;          // consecutive tiles an XCD serves (step_tiles)
    int32_t waves;        // waves per workgroup (tile)
    int32_t segs;         // fused finite differences: row segments per row (one wave each)
    int32_t rows;         // ny * nz
    int32_t items;        // row segments in the grid
    int32_t tiles_per_row;  // row-tile kernels: tiles per row
    int32_t fd_w;         // finite-difference update sweep: tiles per x-chunk
    int32_t fd_yb;        // finite-difference update sweep: rows per y sub-band
    int32_t fd_tx, fd_ty, fd_tz;  // finite-difference update: tiles per axis
    int32_t fd_bw, fd_bh, fd_bd;  // and per brick (fd.hip)
    Physics ph;
};

// Plane stride (cells) of a solve's population planes for N cells of elem
// bytes each in dim dimensions (lattice.cpp): N rounded up to 128 bytes, and
// for large planes moved off a large power of two bytes apart.
int64_t plane_stride(int64_t N, size_t elem, int dim);

// Storage layout of one ping-pong side.  Population i owns the slab of
// 2 P elem bytes that starts at byte 2 i P elem.  In FP64 and FP32 the slab
// holds the g plane and then the h plane.  In half storage the g and h
// values of a cell share one 32-bit word, g in the low half, so that one
// 4-byte access moves both populations of the cell.  cell_bytes: distance
// from one cell to the next; h_offset: where h sits relative to g.
constexpr uint32_t cell_bytes(size_t elem) { return elem == 2 ? 4u : (uint32_t)elem; }
constexpr uint32_t h_offset(size_t elem, uint32_t plane_bytes) {
    return elem == 2 ? 2u : plane_bytes;
}

// Bytes of both sides of a state together.  A step's stores stream past the
// caches unless that much fits the 256 MiB last-level cache (about, and by
// far not the L2s): then a cached store leaves the state there for the next
// step's reads.
constexpr int64_t state_bytes(int dim, size_t elem, int64_t P) {
    return 4 * (dim == 2 ? 37 : 107) * (int64_t)elem * P;
}

// Register layout the lattice step takes by default.  D3Q107 in float or
// double splits g and h over lane pairs (214 values do not fit one lane);
// half storage keeps one cell per lane in both velocity sets, its 214 halves
// held as 107 g/h words.
constexpr bool default_split(int dim, int precision) {
    return dim == 3 && precision != LBM_FP16_SCALED;
}

// Collision parameters of a solve (lattice.cpp).  dt > 0 selects the
// finite-difference form: relaxation rates dt / tau, convection scale dt r / 6.
// energy_fix selects the energy-conserving collision (see collide_*).
Physics physics_of(int dim, double delta, double tau_f, double tau_g, double dt = 0.0,
                   bool energy_fix = false);

// Arguments of the readout kernel (moments and conservation partials).
struct ReadArgs {
    const void* src;
    int64_t N;
    int64_t P;                // plane stride of src in cells
    int32_t nx, ny, nz, nxy;
    uint32_t open_end;
    int32_t stream;           // 1: the source holds P_{n-1}; pull to get S_n
    PullGrid pull;            // set by launch_readout, as
    int32_t run, blocks;      // are the runs of tiles and their number
    double r;
    double rest_energy;       // (D + delta) / 2, added back in deviation storage
    double inv_dof;           // 1 / (D + delta): T = (2E - |u|^2) / (D + delta)
    double w[10];             // group weights (scaled storage is divided by them)
    double* rho;              // [N] or null
    double* u;                // [D][N] or null
    double* E;                // [N] or null
    double* T;                // [N] or null
    double* partials;         // [blocks][D + 2] or null
};

// Launch with the launch's own status (hipLaunchKernel), so that an error
// left behind by unrelated work in the process is not taken for ours.
template <typename... KArgs, typename... Args>
inline hipError_t launch_kernel(void (*kernel)(KArgs...), dim3 grid, dim3 block, hipStream_t s,
                         Args&&... args) {
    std::tuple<std::decay_t<KArgs>...> vals(std::forward<Args>(args)...);
    void* ptrs[sizeof...(KArgs) > 0 ? sizeof...(KArgs) : 1];
    std::apply([&](auto&... v) {
        int i = 0;
        ((ptrs[i++] = static_cast<void*>(&v)), ...);
    }, vals);
    return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, 0, s);
}

// Kernel launchers (kernels.hip).  `split` selects the layout in which one
// lane holds the g populations of a cell and its partner lane (lane ^ 32)
// the h populations.
// S_0 into one side and P_0 = Collide(S_0) into the other.
hipError_t launch_init_collide(int dim, int precision, bool split, void* s0, void* p0,
                               const InitFields& f, const Physics& ph, const double* w_group,
                               hipStream_t s);
// D3Q107 lattice step with the pulled rows staged in LDS (nx a multiple of
// 128, streaming steps only; hipErrorInvalidValue otherwise).
hipError_t launch_step_lds(int precision, const StepArgs& a, hipStream_t s);
hipError_t launch_step(int dim, int precision, bool split, const StepArgs& a,
                       hipStream_t s);
// One explicit finite-difference step (Sec. III); sets the wave mapping
// fields of a copy of `a`.
hipError_t launch_fd_step(int dim, int precision, bool split, const StepArgs& a,
                          hipStream_t s);
// The same step from a per-cell record of the macroscopic state (fd.hip):
// every population's update also adds to the next step's record
// (record_valid: the record is that of a.src; otherwise a moments pass makes it
// first).  FP64 and FP32 deviation storage.
// Whether AUTO takes the fused step instead (launch_fd_step, one lane per cell).
bool fd_fused_by_default(int dim, int precision, int64_t nx, int64_t ny);
size_t fd_record_bytes(int dim, int precision, int64_t P);
// S_0 of the finite-difference form and, unless `record` is null, its record.
hipError_t launch_fd_init(int dim, int precision, void* dst, void* record, const InitFields& f,
                          const Physics& ph, const double* w_group, hipStream_t s);
hipError_t launch_fd_two_pass(int dim, int precision, const StepArgs& a, void* record,
                              bool record_valid, hipStream_t s);
// Launch shape of a lattice step over N cells in rows of nx, with workgroups
// of `tile` cells: consecutive tiles an XCD serves, and the grid (a multiple
// of 8; tiles past the last cell have no work).
void step_tiles(int64_t N, int64_t nx, int tile, int32_t* run, int* grid);
hipError_t launch_readout(int dim, int precision, const ReadArgs& a,
                          int blocks, hipStream_t s);
hipError_t launch_final_reduce(int dim, const double* partials, int blocks,
                               double* out, hipStream_t s);
constexpr int kReadBlock = 256;

}  // namespace lbm

struct lbm_solver;
namespace lbm {

// Staging of the host-array calls of one solve: a device buffer and, for up to
// kOneCopy bytes, a host block that lets all arrays of a call go as one copy.
// Made on first use; the device buffer is kept up to kKeep bytes and freed with
// the call above (an allocation is small beside those copies).  What bounds the
// small calls is the runtime's time per copy, 6 to 8 us each: moments of D2Q37
// FP64 200x4 55 -> 30 us; from 256 KiB on the copies' own bytes take over
// (1000x16: 68 -> 66 us).  A pinned block gains 1 to 4 us more on a call, but
// costs each solve 0.1 ms to allocate and free.
struct HostStage {
    static constexpr size_t kKeep = size_t(16) << 20;
    static constexpr size_t kOneCopy = size_t(256) << 10;
    double* dev;
    size_t bytes;
    double* host;  // kOneCopy bytes

    hipError_t reserve(size_t need);
    void done();     // after the call's work has ended
    void release();
    // n arrays of sizes[k] values, one after the other in `dev`, to or from
    // host memory on stream s; from the device: waits for s.
    hipError_t to_device(const double* const* src, const size_t* sizes, int n, hipStream_t s);
    hipError_t to_host(double* const* dst, const size_t* sizes, int n, hipStream_t s);
};

// Readout of a solve's S_n into device outputs (any may be null), with the
// FP64 totals into the solve's own buffer when `totals` (api.hip).
int solver_readout(lbm_solver* h, double* rho, double* u, double* E, double* T, bool totals);
}  // namespace lbm

// The opaque handle.
struct lbm_solver {
    int dim, q, precision;
    int64_t nx, ny, nz, N;
    int64_t P;            // plane stride in cells (lbm::plane_stride)
    uint32_t bc;
    double gamma, delta, tau_f, tau_g;
    const lbm::LatticeTables* lat;
    size_t elem;          // bytes per stored value
    size_t buf_bytes;     // bytes of one ping-pong side (2 Q P elem)
    void* buf[2];         // ping-pong sides
    int cur;              // side holding the latest post-collision state
    bool have_state;
    bool initial;         // buf[cur ^ 1] holds S_0 itself (no step yet)
    int64_t steps;
    int scheme;           // 0: lattice (collide, stream), 1: finite differences
    int collision;        // LBM_COLLISION_PAPER or LBM_COLLISION_ENERGY_CONSERVING
    double dt;            // finite-difference time step (grid step 1, speeds r e)
    double* partials;     // readout block partials
    double* totals;       // [D + 2] final totals (device)
    int read_blocks;
    hipStream_t stream;
    hipStream_t own_stream;
    int device;
    bool split;
    bool lds;             // D3Q107 lattice step: pulled rows staged in LDS
    bool fd_fused;        // finite differences: one fused kernel (LANE / SPLIT variants)
    void* fd_record;      // finite differences: per-cell record (TWO_PASS)
    bool fd_record_valid; // the record describes the current state
    lbm::HostStage stage; // fields of host-array calls
    size_t device_bytes;
};
