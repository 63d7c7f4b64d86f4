// Where the tensor-product kernels (fe_tensor.hip) apply, where they are the
// default, and the launch by degree.
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "fe_internal.h"

namespace fe {

// Whether a plane of every block lies within the 31 bits of its buffer requests
// (a byte offset past them is what an absent row requests).  At the Gamma point
// the columns are complex vectors' real and imaginary parts, and the line is
// that of the parts' own blocks with half the leading dimension, or the
// results would not be the parts' bit for bit: so a real block has to leave
// the room for its complex one, 1 GiB a plane (below that line the kernel's
// plane ranges hold either; larger planes run the cell kernels).
static bool planes_in_range(const fe_mesh *m, const StepArgs &a) {
    const bool pairs = a.S || (a.vectors && a.vectors != a.N);
    const int64_t plane = m->nf[0] * m->nf[1], ld = std::max(std::max(a.ldx, a.ldy), a.Ym1 ? a.ldm : (int64_t)0);
    return ld <= (int64_t)0x7FFFFFFF / 16 / plane * (pairs ? 2 : 1);
}

// Whether the tensor-product form applies: no zero-Neumann axis (M^-1/2 of a
// node is then a product of factors of its local indices, the same in every
// cell), planes in range, and a recurrence whose beta / alpha is a number.
bool tensor_applies(const fe_mesh *m, const StepArgs &a) {
    for (int d = 0; d < 3; ++d)
        if (m->bc[d] == FE_BC_NEUMANN) return false;
    if (!planes_in_range(m, a)) return false;
    if (a.N >= (int64_t)1 << 31) return false;
    return a.alpha != 0.0 && std::isfinite(a.beta / a.alpha);
}

// Where it is the default.  The line is not one of speed: it is drawn by what
// else holds, namely that the default of the other degrees on a few cells, and of
// one or two vectors up to a mesh of the size where Lanczos and CG spend time on
// the product, are documented to equal the one-cell kernel (variant 1) bit for
// bit.  At the line (us per product, cell kernels / this one): 64 cells, 16
// vectors 34 / 9 at p = 1 and 2, 148 / 23 at p = 5, 311 / 27 at p = 6, 323 / 32 at
// p = 7; one vector on 1100 cells 42 / 9 (p = 1) to 328 / 44 (p = 7).  Below it the
// cell kernels' times stand.  The rule looks at the number of vectors, not of
// real columns, so that a complex block at the Gamma point takes the kernel of its
// real and imaginary parts; at other k-points (no such equality there) it has no
// line.
bool tensor_default(const fe_mesh *m, const StepArgs &a) {
    if (a.S) return true;
    const int64_t vectors = a.vectors ? a.vectors : a.N;
    if (vectors < 3) return false;
    return m->p == 3 || m->p == 4 || m->ncells >= 64;
}

#define FE_DEGREES(F) \
    switch (m->p) {   \
    case 1: F(1);     \
    case 2: F(2);     \
    case 3: F(3);     \
    case 4: F(4);     \
    case 5: F(5);     \
    case 6: F(6);     \
    case 7: F(7);     \
    default: return hipErrorInvalidValue; \
    }

hipError_t launch_tensor(const fe_mesh *m, const StepArgs &a, hipStream_t s) {
#define FE_STEP(PP) return launch_tensor_degree<PP>(m, a, s)
    FE_DEGREES(FE_STEP)
#undef FE_STEP
}

// One or two vectors, real or (at the Gamma point) complex.  part (not null):
// also the partial sums of x times y over the workgroups, *nparts of them,
// unless *done is nonzero; where the tiles are more than max_parts, *nparts is
// zero and nothing is launched.
bool tensor_vec_applies(const fe_mesh *m, const StepArgs &a) {
    if (a.S || a.N < 1 || (a.vectors ? a.vectors : a.N) > 2) return false;
    if (!planes_in_range(m, a)) return false;
    return a.alpha != 0.0 && std::isfinite(a.beta / a.alpha);
}

hipError_t launch_tensor_vec(const fe_mesh *m, const StepArgs &a, hipStream_t s, const double *done, double *part,
                             int max_parts, int *nparts) {
#define FE_VEC(PP) return launch_vec_degree<PP>(m, a, s, done, part, max_parts, nparts)
    FE_DEGREES(FE_VEC)
#undef FE_VEC
}
#undef FE_DEGREES

}  // namespace fe
