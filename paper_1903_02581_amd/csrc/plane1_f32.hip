// Instantiations of the fused (x1, y1)-plane pass for float2 storage.
#include "plane_pass.hpp"

namespace hom4d_impl {
namespace {
using namespace dev;

template <int NX, int NY>
AxisKernel mk(int vk, Plane1Launch* p) {
    constexpr int W = kPlane1W;
    p->threads = plane1_threads(NX, NY, Shape<NX>::t, Shape<NY>::t, W);
    p->w = W;
    p->lds = sizeof(float2) * NX * NY * W + sizeof(double2) * (NX + 2 * NY);
    return vk == 2 ? k_plane1<float2, NX, NY, W, 2> : k_plane1<float2, NX, NY, W, 1>;
}
}  // namespace

dev::AxisKernel pick_plane1_f32(int nx, int ny, int vk, Plane1Launch* p) {
#define HOM4D_PLANE(X, Y) \
    if (nx == X && ny == Y) return mk<X, Y>(vk, p);
    HOM4D_PAIR_SIZES
#undef HOM4D_PLANE
    return nullptr;
}
}  // namespace hom4d_impl
