// The library's device code of offsets and of the initial values' rounding,
// compiled for the host.
#include <cmath>
#include <cstdint>

inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)((uint64_t)a * b >> 32); }
template <typename T> T __shfl_xor(T v, int) { return v; }  // named by code not used here
using std::max;
using std::min;
#include "step_core.h"

using namespace lbm;

extern "C" {

int host_divide(int n, int64_t d) { return core::divide(n, divisor_of(d)); }

void host_stored_half(const double* x, uint16_t* out, int64_t n) {
    for (int64_t k = 0; k < n; ++k)
        out[k] = __builtin_bit_cast(uint16_t, core::stored<_Float16>(x[k]));
}

void host_quotient(const double* x, double w, double* out, int64_t n) {
    for (int64_t k = 0; k < n; ++k) out[k] = core::quotient(x[k], w, 1.0 / w);
}

// Cells whose offsets differ from the plain forms in any of the seven shifts
// of an axis.
int64_t host_offsets_wrong(int dim, int nx, int ny, int nz, uint32_t open_end) {
    const PullGrid g = pull_grid(nx, ny, nz, open_end);
    const int nxy = nx * ny;
    int64_t wrong = 0;
    for (int z = 0; z < nz; ++z)
        for (int y = 0; y < ny; ++y)
            for (int x = 0; x < nx; ++x) {
                const int cell = x + nx * (y + ny * z);
                const uint32_t role = 12u;
                auto check = [&](const auto& o) {
                    bool ok = o.own == (uint32_t)cell * 4u + role;
                    for (int e = -3; e <= 3; ++e) {
                        ok &= o.xo[e + 3] ==
                              (uint32_t)core::pull_coord(x, e, nx, open_end & 1u) * 4u + role;
                        ok &= o.yo[e + 3] ==
                              (uint32_t)(core::pull_coord(y, e, ny, open_end & 2u) * nx) * 4u;
                        if (dim == 3)
                            ok &= o.zo[e + 3] ==
                                  (uint32_t)(core::pull_coord(z, e, nz, open_end & 4u) * nxy) * 4u;
                    }
                    wrong += !ok;
                };
                if (dim == 2) {
                    core::CellOffsets<2, float> o;
                    o.fill(cell, nx, ny, nz, nxy, g, role);
                    check(o);
                } else {
                    core::CellOffsets<3, float> o;
                    o.fill(cell, nx, ny, nz, nxy, g, role);
                    check(o);
                }
            }
    return wrong;
}
}
