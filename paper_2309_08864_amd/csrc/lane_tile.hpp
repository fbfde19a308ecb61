// lane_tile.hpp -- what the march kernels' tiles are made of: lane shifts for
// the x neighbours, vector access to a lane's consecutive cells, and the tile
// geometry of a 3D workgroup.
#pragma once
#include <type_traits>

#include "tb_kernel.hpp"

namespace so2dr {

// DPP control codes of the whole-wave shifts (GFX9 DPP): lane i receives lane
// i-1 (shift right) or lane i+1 (shift left); the lane without a source gets 0.
constexpr int kDppWaveShr1 = 0x138;
constexpr int kDppWaveShl1 = 0x130;

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_f(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// VX consecutive stored elements <-> VX values of the accumulation type, in
// one vector access.  The address need only be aligned to an element: rows of
// any length start anywhere, and the memory path takes such accesses whole.
template <typename T, int VX> struct VecIO;
template <int VX> struct VecIO<float, VX> {
  using V = typename std::conditional<VX == 4, float4, float2>::type;
  static __device__ __forceinline__ void load(const float *p, float *v) {
    V q;
    __builtin_memcpy(&q, p, sizeof(V));
    __builtin_memcpy(v, &q, sizeof(V));
  }
  static __device__ __forceinline__ void store(float *p, const float *v) {
    V q;
    __builtin_memcpy(&q, v, sizeof(V));
    __builtin_memcpy(p, &q, sizeof(V));
  }
};
template <int VX> struct VecIO<double, VX> {
  static __device__ __forceinline__ void load(const double *p, double *v) {
#pragma unroll
    for (int i = 0; i < VX; i += 2) {
      double2 q;
      __builtin_memcpy(&q, p + i, sizeof(q));
      v[i] = q.x;
      v[i + 1] = q.y;
    }
  }
  static __device__ __forceinline__ void store(double *p, const double *v) {
#pragma unroll
    for (int i = 0; i < VX; i += 2) {
      const double2 q = make_double2(v[i], v[i + 1]);
      __builtin_memcpy(p + i, &q, sizeof(q));
    }
  }
};
template <typename H16, int VX> struct VecIOHalf {
  using V = typename std::conditional<VX == 4, uint2, unsigned>::type;
  static __device__ __forceinline__ void load(const H16 *p, float *v) {
    V q;
    __builtin_memcpy(&q, p, sizeof(V));
    unsigned short bits[VX];
    __builtin_memcpy(bits, &q, sizeof(V));
#pragma unroll
    for (int i = 0; i < VX; ++i) {
      H16 h;
      __builtin_memcpy(&h, &bits[i], 2);
      v[i] = Store<H16>::load(&h);
    }
  }
  static __device__ __forceinline__ void store(H16 *p, const float *v) {
    unsigned short bits[VX];
#pragma unroll
    for (int i = 0; i < VX; ++i) {
      H16 h;
      Store<H16>::store(&h, v[i]);
      __builtin_memcpy(&bits[i], &h, 2);
    }
    V q;
    __builtin_memcpy(&q, bits, sizeof(V));
    __builtin_memcpy(p, &q, sizeof(V));
  }
};
template <int VX> struct VecIO<__hip_bfloat16, VX> : VecIOHalf<__hip_bfloat16, VX> {};
template <int VX> struct VecIO<__half, VX> : VecIOHalf<__half, VX> {};
// one cell per lane: plain scalar accesses
template <> struct VecIO<float, 1> {
  static __device__ __forceinline__ void load(const float *p, float *v) { v[0] = *p; }
  static __device__ __forceinline__ void store(float *p, const float *v) { *p = v[0]; }
};
template <> struct VecIO<double, 1> {
  static __device__ __forceinline__ void load(const double *p, double *v) { v[0] = *p; }
  static __device__ __forceinline__ void store(double *p, const double *v) { *p = v[0]; }
};
template <> struct VecIO<__hip_bfloat16, 1> {
  static __device__ __forceinline__ void load(const __hip_bfloat16 *p, float *v) { v[0] = Store<__hip_bfloat16>::load(p); }
  static __device__ __forceinline__ void store(__hip_bfloat16 *p, const float *v) { Store<__hip_bfloat16>::store(p, v[0]); }
};
template <> struct VecIO<__half, 1> {
  static __device__ __forceinline__ void load(const __half *p, float *v) { v[0] = Store<__half>::load(p); }
  static __device__ __forceinline__ void store(__half *p, const float *v) { Store<__half>::store(p, v[0]); }
};

// HA: the x halo is rounded up to a multiple of HA cells (whole lanes at
// least); with 64-cell-multiple rows and a 64-byte halo the output rows of
// every tile start and end on 128-byte lines.
template <int R, int KL, int NW, int M, int VX_, int HA = VX_>
struct StarTile {
  static constexpr int VX = VX_;                        // x cells per lane
  static constexpr int TX = 64 * VX, TY = NW * M;
  static constexpr int HX = (KL * R + HA - 1) / HA * HA;  // x halo
  static_assert(HA % VX == 0, "the x halo must be whole lanes");
  static constexpr int HY = KL * R;
  static constexpr int OX = TX - 2 * HX, OY = TY - 2 * HY;
  static_assert(M >= R && R <= 2 * VX && OX > 0 && OY > 0, "tile too small for this depth");
};

}  // namespace so2dr
