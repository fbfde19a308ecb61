// kernels.hip -- the fused-step kernels of one storage type and one group of
// stencils, and the dispatcher that maps a launch onto a compiled
// instantiation.  The build compiles this file once per storage type and
// group, with SO2DR_STORAGE set to the so2dr_dtype value (0 F32, 1 F64, 2
// BF16, 3 F16) and SO2DR_GROUP to 0..2, so that the sets of instantiations
// compile in parallel; kMaxDepth (depths.hpp) decides which stencils and
// depths each type gets, stencil_group (launch.hpp) which group a stencil is in.
#include "so2dr.h"

#include "depths.hpp"
#include "launch_impl.hpp"

#if !defined(SO2DR_STORAGE) || !defined(SO2DR_GROUP)
#error "compile with -DSO2DR_STORAGE=<so2dr_dtype value> -DSO2DR_GROUP=<0..2>"
#endif

namespace so2dr {
namespace {

template <int D> struct StorageOf;
template <> struct StorageOf<SO2DR_F32> { using T = float; };
template <> struct StorageOf<SO2DR_F64> { using T = double; };
template <> struct StorageOf<SO2DR_BF16> { using T = __hip_bfloat16; };
template <> struct StorageOf<SO2DR_F16> { using T = __half; };

template <int D>
int dispatch(const LaunchParams &p, hipStream_t s, std::string *msg) {
  using T = typename StorageOf<D>::T;
  switch (p.stencil) {
#define SO2DR_CASE(ID, NDIM, BOX, R)                                          \
  case ID:                                                                  \
    if constexpr (kMaxDepth[D][ID] > 0 && stencil_group(ID) == SO2DR_GROUP)  \
      return launch_depth<T, NDIM, BOX, R, kMaxDepth[D][ID]>(p, s, msg);   \
    break;
    SO2DR_CASE(ST_2D_STAR_R1, 2, false, 1)
    SO2DR_CASE(ST_2D_BOX_R1, 2, true, 1)
    SO2DR_CASE(ST_2D_BOX_R2, 2, true, 2)
    SO2DR_CASE(ST_2D_BOX_R3, 2, true, 3)
    SO2DR_CASE(ST_2D_BOX_R4, 2, true, 4)
    SO2DR_CASE(ST_3D_STAR_R1, 3, false, 1)
    SO2DR_CASE(ST_3D_STAR_R2, 3, false, 2)
    SO2DR_CASE(ST_3D_BOX_R1, 3, true, 1)
#undef SO2DR_CASE
    default:
      break;
  }
  if (msg) *msg = "stencil not built for this storage type";
  return -3;
}

}  // namespace

#define SO2DR_NAME3(A, B, C) A##B##_##C
#define SO2DR_NAME2(A, B, C) SO2DR_NAME3(A, B, C)
int SO2DR_NAME2(launch_tb_, SO2DR_STORAGE, SO2DR_GROUP)(const LaunchParams &p, hipStream_t s, std::string *msg) {
  return dispatch<SO2DR_STORAGE>(p, s, msg);
}

}  // namespace so2dr
