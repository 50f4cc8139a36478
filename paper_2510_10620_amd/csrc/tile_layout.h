// LDS tiles of bf16 rows for any head dim, and fp32 operands in bf16 parts.
#pragma once
#include "mfma_common.h"

namespace dcp {

// Tiles are [rows][D] bf16 without padding: a 256-byte line of the 64 banks holds 128 / D rows, and the 16-byte chunk c of a row
// sits at chunk ((row % (128 / D)) * (D / 8) + c) ^ swz(line) of its line; 16 consecutive rows at one chunk (row-major reads)
// fall into 16 different chunks, 4 consecutive rows x 64 bytes (transposing reads) into 4 different 64-byte groups.  D = 128 is
// the layout of tile_off().
template <int D>
struct TileLayout {
  static constexpr int KS = D / 16, DT = D / 32;       // MFMA steps over D, 32-column tiles of D
  static constexpr int kRow = 2 * D, kBytes = kTN * kRow;
  static constexpr int RPL = 128 / D, CPR = D / 8;     // rows per 256-byte line, chunks per row
  static constexpr int kORow = kRow + 16;              // pitch of a staged output row
  static __device__ __forceinline__ constexpr int swz(int line) {
    return D == 128 ? ((line & 3) << 2) | ((line >> 2) & 3) : D == 64 ? ((line & 1) << 2) | ((line >> 1) & 3) : line & 3;
  }
  static __device__ __forceinline__ int off(int row, int c) {
    const int line = row / RPL;
    return line * 256 + ((((row % RPL) * CPR + c) ^ swz(line)) << 4);
  }
};

// Fragment addresses from two registers: every other one is an XOR of these with a constant.
template <int D>
struct Frags {
  typedef TileLayout<D> L;
  int rm, tr;
  __device__ __forceinline__ void init(int lane) {
    rm = L::off(lane & 31, lane >> 5);
    const int j = lane & 15, blk = lane >> 4, col = 16 * (blk & 1) + 4 * (j & 3);
    tr = L::off(4 * (blk >> 1) + (j >> 2), col >> 3) + (col & 7) * 2;
  }
  __device__ __forceinline__ bf16x8 rows(const char* tile, int ks) const { return as_frag(*(const uint4*)(tile + (rm ^ (ks << 5)))); }
  // rows 16 c + 8a + 4h + b, columns 32 dt + lane % 32
  __device__ __forceinline__ bf16x8 cols(const char* tile, int c, int dt) const {
    typedef __attribute__((address_space(3))) s16x4* lds_p;
    const int a0 = tr ^ (dt << 6), a1 = a0 ^ (8 / L::RPL * 256 + 0x20);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(tile + c * 16 * L::kRow + a0));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(tile + c * 16 * L::kRow + a1));
    s16x8 v;
    v[0] = lo[0]; v[1] = lo[1]; v[2] = lo[2]; v[3] = lo[3]; v[4] = hi[0]; v[5] = hi[1]; v[6] = hi[2]; v[7] = hi[3];
    return __builtin_bit_cast(bf16x8, v);
  }
};

// Registers 8c .. 8c + 7 of a C tile as three bf16 operands that add up to the values exactly: 8 significant bits each, cut
// off (not rounded: a finite value has finite parts), the remainders being exact in fp32.
__device__ __forceinline__ void pack_split(const f32x16& s, int c, bf16x8 (&part)[3]) {
  uint32_t w[3][4];
#pragma unroll
  for (int e = 0; e < 4; e++) {
    float a = s[8 * c + 2 * e], b = s[8 * c + 2 * e + 1];
#pragma unroll
    for (int k = 0; k < 3; k++) {
      const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
      w[k][e] = __builtin_amdgcn_perm(ub, ua, 0x07060302);   // the upper halves of both
      a -= __uint_as_float(ua & 0xffff0000u);
      b -= __uint_as_float(ub & 0xffff0000u);
    }
  }
#pragma unroll
  for (int k = 0; k < 3; k++) part[k] = as_frag(make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]));
}

}  // namespace dcp
