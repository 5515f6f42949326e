// F64 instantiation of the element operator (see ax_impl.h).
#include "ax_impl.h"

namespace semx {
template int launch_ax<double>(const Level &, const double *, const double *, const double *, const double *,
                            double *, double, double, const double *, double *, int64_t *, hipStream_t,
                            const int *);
template int launch_ax_multi<double>(const Level &, const double *, const double *, const double *, const double *,
                                 int64_t, double *, int64_t, const VSet &, double, double, const double *,
                                 double *, int64_t, int64_t *, hipStream_t, const int *, int, const PcgDir &);

int ax_direction_lanes(const Level &L, double h2, const double *k)
{
#define SEM_AX_LANES(NQ) \
    case NQ: return ax_direction_lanes_nq<NQ>(L, h2, k);
    switch (L.nq) {
        SEM_AX_LANES(2) SEM_AX_LANES(3) SEM_AX_LANES(4) SEM_AX_LANES(5) SEM_AX_LANES(6)
        SEM_AX_LANES(7) SEM_AX_LANES(8) SEM_AX_LANES(9) SEM_AX_LANES(10) SEM_AX_LANES(11)
        SEM_AX_LANES(12) SEM_AX_LANES(13) SEM_AX_LANES(14) SEM_AX_LANES(15) SEM_AX_LANES(16)
    }
#undef SEM_AX_LANES
    return 64;
}
}  // namespace semx
