// Instantiations of the register-held (x2, y2)-plane pass (complex128 storage, table form).
#include "plane_regs.hpp"

namespace hom4d_impl {
namespace {
using namespace dev;

template <int NX, int NY>
AxisKernel mk(bool nt, int* threads, size_t* lds) {
    *threads = plane_regs_threads(NX, NY);
    *lds = plane_regs_lds(NX, NY);
    return nt ? k_plane_regs<NX, NY, true> : k_plane_regs<NX, NY, false>;
}
}  // namespace

dev::AxisKernel pick_plane_regs(int nx, int ny, bool nt, int* threads, size_t* lds) {
    if (nx == 128 && ny == 128) return mk<128, 128>(nt, threads, lds);
    if (nx == 128 && ny == 64) return mk<128, 64>(nt, threads, lds);
    if (nx == 64 && ny == 128) return mk<64, 128>(nt, threads, lds);
    return nullptr;
}
}  // namespace hom4d_impl
