// Sums of doubles over the lanes of a wave (gfx950, wave64), in the order of
// a tree over lane ^ 32, 16, 8, 4, 2, 1.
#pragma once
#include <hip/hip_runtime.h>

namespace spand {

// v + (v of lane ^ O), every lane active.  The partner comes by lane moves in
// the vector ALU (DPP within rows of 16, permlane swaps across them: 10-15
// cycles) instead of a trip through the LDS crossbar (75 cycles a step, which
// made a wave sum of doubles cost 510 cycles instead of 150).
template <int O>
__device__ inline double add_xor(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  if constexpr (O == 32 || O == 16) {
    // the swap of a value with its copy leaves one row pair in each result
    auto a = O == 32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                     : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    auto b = O == 32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                     : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double(int(b[0]), int(a[0])) + __hiloint2double(int(b[1]), int(a[1]));
  } else {
    int l, h;
    if constexpr (O == 8) {           // row_ror:8
      l = __builtin_amdgcn_update_dpp(0, lo, 0x128, 0xF, 0xF, false);
      h = __builtin_amdgcn_update_dpp(0, hi, 0x128, 0xF, 0xF, false);
    } else if constexpr (O == 4) {    // row_shl:4 into the even banks of 4, row_shr:4 into the odd ones
      l = __builtin_amdgcn_update_dpp(0, lo, 0x104, 0xF, 0x5, false);
      l = __builtin_amdgcn_update_dpp(l, lo, 0x114, 0xF, 0xA, false);
      h = __builtin_amdgcn_update_dpp(0, hi, 0x104, 0xF, 0x5, false);
      h = __builtin_amdgcn_update_dpp(h, hi, 0x114, 0xF, 0xA, false);
    } else {                          // quad_perm
      constexpr int C = O == 2 ? 0x4E : 0xB1;
      l = __builtin_amdgcn_update_dpp(0, lo, C, 0xF, 0xF, false);
      h = __builtin_amdgcn_update_dpp(0, hi, C, 0xF, 0xF, false);
    }
    return v + __hiloint2double(h, l);
  }
}
__device__ inline double wave_sum(double v) {
  v = add_xor<32>(v);
  v = add_xor<16>(v);
  v = add_xor<8>(v);
  v = add_xor<4>(v);
  v = add_xor<2>(v);
  return add_xor<1>(v);
}

// a of lanes 0-31 | b of lanes 32-63, each added to its partner of lane ^ 32
// (O = 32), or the same for the even and odd rows of 16 lanes (O = 16): two
// sums go on in one register.
template <int O>
__device__ inline double add_halves(double a, double b) {
  static_assert(O == 32 || O == 16, "rows or halves of a wave");
  const int al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
  auto l = O == 32 ? __builtin_amdgcn_permlane32_swap(al, bl, false, false)
                   : __builtin_amdgcn_permlane16_swap(al, bl, false, false);
  auto h = O == 32 ? __builtin_amdgcn_permlane32_swap(ah, bh, false, false)
                   : __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
  return __hiloint2double(int(h[0]), int(l[0])) + __hiloint2double(int(h[1]), int(l[1]));
}
// wave_sum of four values at once: lane 16 q gets the sum of v[q]
__device__ inline double wave_sum4(const double (&v)[4]) {
  double s = add_halves<16>(add_halves<32>(v[0], v[2]), add_halves<32>(v[1], v[3]));
  s = add_xor<8>(s);
  s = add_xor<4>(s);
  s = add_xor<2>(s);
  return add_xor<1>(s);
}

}  // namespace spand
