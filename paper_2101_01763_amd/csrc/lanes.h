// Sums of doubles over the lanes of a wave (gfx950, wave64), in the order of
// a tree over lane ^ 32, 16, 8, 4, 2, 1, and multiply-adds with a value of
// another lane.
#pragma once
#include <hip/hip_runtime.h>

namespace spand {

// v + (v of lane ^ O), every lane active.  The partner comes by lane moves in
// the vector ALU (DPP within rows of 16, permlane swaps across them: 10-15
// cycles), not by a trip through the LDS crossbar (75 cycles): a wave sum of
// doubles in 150 cycles, not 510.
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

// s[0..7] += h * p_l for the lanes l = R..R+7 of every row of 16 lanes of p:
// a value that the lanes of a wave hold once per 16 lanes multiplies every
// lane's h without a trip through LDS (DPP row_newbcast).  The wait states
// cover a p that was computed right before.  The sums are early clobbers: the
// first instruction writes one while the later ones still read p and h, which
// must not share its register (they would where they hold the same value).
#define FMAC_ROW(w, i, p, h, l) \
  "v_fmac_f" #w "_dpp %" #i ", %" #p ", %" #h " row_newbcast:" #l " row_mask:0xf bank_mask:0xf\n\t"
#define FMAC_8(w, l0, l1, l2, l3, l4, l5, l6, l7)                                                \
  asm("s_nop 1\n\t" FMAC_ROW(w, 0, 8, 9, l0) FMAC_ROW(w, 1, 8, 9, l1) FMAC_ROW(w, 2, 8, 9, l2)   \
          FMAC_ROW(w, 3, 8, 9, l3) FMAC_ROW(w, 4, 8, 9, l4) FMAC_ROW(w, 5, 8, 9, l5)             \
              FMAC_ROW(w, 6, 8, 9, l6) FMAC_ROW(w, 7, 8, 9, l7)                                  \
      : "+&v"(s[0]), "+&v"(s[1]), "+&v"(s[2]), "+&v"(s[3]), "+&v"(s[4]), "+&v"(s[5]),            \
        "+&v"(s[6]), "+&v"(s[7])                                                                 \
      : "v"(p), "v"(h))
#define FMAC_4(w)                                                                                \
  asm("s_nop 1\n\t" FMAC_ROW(w, 0, 4, 5, 4) FMAC_ROW(w, 1, 4, 5, 5) FMAC_ROW(w, 2, 4, 5, 6)      \
          FMAC_ROW(w, 3, 4, 5, 7)                                                                \
      : "+&v"(s[0]), "+&v"(s[1]), "+&v"(s[2]), "+&v"(s[3])                                       \
      : "v"(p), "v"(h))
template <int R>
__device__ inline void fmac8(float *s, float p, float h) {
  static_assert(R == 0 || R == 8, "half rows");
  if constexpr (R == 0) FMAC_8(32, 0, 1, 2, 3, 4, 5, 6, 7);
  else FMAC_8(32, 8, 9, 10, 11, 12, 13, 14, 15);
}
template <int R>
__device__ inline void fmac8(double *s, double p, double h) {
  static_assert(R == 0 || R == 8, "half rows");
  if constexpr (R == 0) FMAC_8(64, 0, 1, 2, 3, 4, 5, 6, 7);
  else FMAC_8(64, 8, 9, 10, 11, 12, 13, 14, 15);
}
// the same for the four lanes 4..7
__device__ inline void fmac4(float *s, float p, float h) { FMAC_4(32); }
__device__ inline void fmac4(double *s, double p, double h) { FMAC_4(64); }
#undef FMAC_4
#undef FMAC_8
#undef FMAC_ROW

}  // namespace spand
