// Allocation-free entry point: the liquid volume fractions W_L of one sample
// set (Section 5, Figs. 3-4) straight from a nodal liquid level set, with no
// context, no device allocation and no work space: one kernel from the level set
// to the caller's array, by way of a static one where the two overlap (filling,
// sub-cell, weight and unpack kernels over a work array took 20 us at 64^2).  The
// operation order is that of vfs_assemble, so the result is bit-identical to
// vfs_get_weights(ctx, set, VFS_WEIGHT_LIQUID, out) on a context assembled from
// the same level set.
#include <cmath>
#include <string>

#include "vfs_internal.h"

using namespace vfs;

namespace {

// the grids this call takes, by the bytes of their sub-cell fractions and weights
constexpr long long kMostBytes = 96LL * 1024 * 1024;
// they hold at least 8 (2D: two materials of four sets) arrays of NP values, and a
// set has fewer values than NP
static_assert(kMostSetValues >= kMostBytes / 8 / 8, "the largest set");

// errors are reported through vfs_last_error(NULL)
int nfail(int code, const std::string& m) { return fail_global(code, m); }

// bytes of a grid's sub-cell fractions (two level sets) and padded liquid and
// fluid weights of every set; -1 for invalid sizes
long long grid_bytes(int dim, int nx, int ny, int nz) {
    if ((dim != 2 && dim != 3) || nx < 1 || ny < 1 || (dim == 3 && nz < 1)) return -1;
    if (nx > 16384 || ny > 16384 || (dim == 3 && nz > 2048)) return -1;
    const Geo g = make_geo(dim, nx, ny, nz, 1.0);
    const long long sub = (dim == 2 ? 4LL : 8LL) * nx * ny * (dim == 3 ? nz : 1);
    return (2 * sub + 2LL * g.nsets() * g.NP) * 8;
}

}  // namespace

extern "C" {

int vfs_liquid_weights_noalloc(int dim, int nx, int ny, int nz, double w_min,
                               const double* phi_liquid, int set, double* out, void* hip_stream) {
    const long long need = grid_bytes(dim, nx, ny, nz);
    if (need < 0) return nfail(VFS_EINVAL, "dim must be 2 or 3 and sizes in range");
    if (need > kMostBytes)
        return nfail(VFS_EINVAL, "grid too large: a work space for its fractions and weights is " +
                                     std::to_string(need) + " bytes, " +
                                     std::to_string(kMostBytes) + " at most");
    if (!phi_liquid || !out) return nfail(VFS_EINVAL, "NULL level set or output");
    if (!(w_min >= 0.0) || !(w_min < 0.5)) return nfail(VFS_EINVAL, "w_min must be in [0,0.5)");
    const int nsets = dim == 2 ? 4 : 7;
    // public set numbers: 2D cell, x faces, y faces, nodes (VFS_SET_NODE);
    // 3D the seven sets in their order
    int internal;
    if (dim == 2) {
        if (set == VFS_SET_CELL || set == VFS_SET_FACE_X || set == VFS_SET_FACE_Y)
            internal = set;
        else if (set == VFS_SET_NODE)
            internal = 3;
        else
            return nfail(VFS_EINVAL, "bad sample set for 2D");
    } else {
        if (set < 0 || set >= nsets) return nfail(VFS_EINVAL, "bad sample set for 3D");
        internal = set;
    }
    const Geo g = make_geo(dim, nx, ny, nz, 1.0);
    launch_weights_set(g, internal, phi_liquid, w_min, out, reinterpret_cast<hipStream_t>(hip_stream));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return nfail(VFS_EHIP, std::string("launch: ") + hipGetErrorString(e));
    return VFS_OK;
}

}  // extern "C"
