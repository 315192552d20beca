// Sums, maxima and prefix sums over the 64 lanes of a wave (fp64 mostly).
#pragma once
#include <hip/hip_runtime.h>

// Wave-wide sum through the data-parallel-primitive lane moves (no LDS round trips as with shuffles): quads,
// rows of 16, then the row totals across the four rows; lane 63 ends up with the total, which is handed to every
// lane as a uniform value.  The order of the additions is fixed, so equal inputs give equal bits everywhere.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move_f64(double v) {       // lanes without a source lane read 0.0
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xf, false);
  return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_move_u64(unsigned long long v) {
  const unsigned int lo = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)(unsigned int)v, CTRL, 0xf, 0xf, false);
  const unsigned int hi = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)(unsigned int)(v >> 32), CTRL, 0xf, 0xf, false);
  return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_move_f64<0xB1, 0xf>(v);    // quad_perm [1,0,3,2]
  v += dpp_move_f64<0x4E, 0xf>(v);    // quad_perm [2,3,0,1]
  v += dpp_move_f64<0x124, 0xf>(v);   // row_ror:4
  v += dpp_move_f64<0x128, 0xf>(v);   // row_ror:8: every lane holds the total of its row
  v += dpp_move_f64<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_move_f64<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3: lane 63 holds the total
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}

// The largest of a value over the lanes of a wave, in every lane: rows of 16 by lane moves that pair the lanes
// symmetrically, the rows' results handed on to the rows behind, the last lane's read back as a uniform value.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_other_f32(float v) {          // lanes without a source lane read their own value
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}
__device__ __forceinline__ float wave_max_f32(float v) {
  v = fmaxf(v, dpp_other_f32<0xB1, 0xf>(v));    // quad_perm [1,0,3,2]
  v = fmaxf(v, dpp_other_f32<0x4E, 0xf>(v));    // quad_perm [2,3,0,1]
  v = fmaxf(v, dpp_other_f32<0x141, 0xf>(v));   // row_half_mirror
  v = fmaxf(v, dpp_other_f32<0x140, 0xf>(v));   // row_mirror
  v = fmaxf(v, dpp_other_f32<0x142, 0xa>(v));   // row_bcast:15 into rows 1 and 3
  v = fmaxf(v, dpp_other_f32<0x143, 0xc>(v));   // row_bcast:31 into rows 2 and 3
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// The largest of a value over each quad of lanes, or row of 16, in every lane of it.
__device__ __forceinline__ float quad_max_f32(float v) {
  v = fmaxf(v, dpp_other_f32<0xB1, 0xf>(v));    // quad_perm [1,0,3,2]
  return fmaxf(v, dpp_other_f32<0x4E, 0xf>(v));    // quad_perm [2,3,0,1]
}
__device__ __forceinline__ float row16_max_f32(float v) {
  v = quad_max_f32(v);
  v = fmaxf(v, dpp_other_f32<0x141, 0xf>(v));   // row_half_mirror
  return fmaxf(v, dpp_other_f32<0x140, 0xf>(v));   // row_mirror
}

// The sum in single precision.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_move_f32(float v) {           // lanes without a source lane read 0
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}
__device__ __forceinline__ float wave_sum_f32(float v) {
  v += dpp_move_f32<0xB1, 0xf>(v);    // quad_perm [1,0,3,2]
  v += dpp_move_f32<0x4E, 0xf>(v);    // quad_perm [2,3,0,1]
  v += dpp_move_f32<0x124, 0xf>(v);   // row_ror:4
  v += dpp_move_f32<0x128, 0xf>(v);   // row_ror:8: every lane holds the total of its row
  v += dpp_move_f32<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_move_f32<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3: lane 63 holds the total
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// The maximum for doubles.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_other_f64(double v) {        // lanes without a source lane read their own value
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROW_MASK, 0xf, false),
                          __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROW_MASK, 0xf, false));
}
__device__ __forceinline__ double wave_max_f64(double v) {
  v = fmax(v, dpp_other_f64<0xB1, 0xf>(v));
  v = fmax(v, dpp_other_f64<0x4E, 0xf>(v));
  v = fmax(v, dpp_other_f64<0x141, 0xf>(v));
  v = fmax(v, dpp_other_f64<0x140, 0xf>(v));
  v = fmax(v, dpp_other_f64<0x142, 0xa>(v));
  v = fmax(v, dpp_other_f64<0x143, 0xc>(v));
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63), __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// Inclusive prefix sums over the lanes of a wave by the same kind of lane moves: inside every row of 16 (sources
// outside the row count 0), then the row totals handed on to the rows behind.  Fixed order, equal bits everywhere.
__device__ __forceinline__ double wave_inclusive_scan(double v) {
  v += dpp_move_f64<0x111, 0xf>(v);   // row_shr:1
  v += dpp_move_f64<0x112, 0xf>(v);   // row_shr:2
  v += dpp_move_f64<0x114, 0xf>(v);   // row_shr:4
  v += dpp_move_f64<0x118, 0xf>(v);   // row_shr:8
  v += dpp_move_f64<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_move_f64<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}

// Lanes of one wave handing values to each other through LDS: the hardware executes a wave's LDS instructions
// in order, but the compiler reasons per thread and would otherwise be free to reuse a value it loaded before
// another lane's store (or to forward only its own store).  This fence makes it reload.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
