// Weight fragments of the dual family's matrix kernels: the packed outlier
// half-words of one lane (layout.h, dual section B) as the sparse operand of
// v_smfmac_i32_32x32x64_i8.
//
// The instruction takes the sparse operand as two stored values per four
// positions of K, each with its position in a 2-bit index, and multiplies 64
// dense K in the time the dense instruction takes for 32.  A group of eight
// with one or two outliers always fits: it is two fours of two slots each.
// Lane h*32 + r supplies row r; its stored bytes 4i..4i+3 (i = 0..3) belong
// to the groups K = 16h + 8i (i < 2) and 32 + 16h + 8(i - 2) of the 64-K
// step, which are the half-words the blob keeps for that lane; index bits
// 8i..8i+7 hold the four slots' positions in their fours.  The dense operand's
// lane h*32 + c holds bytes K = 32h .. 32h + 31 of column c.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace sdq {
namespace dual {

typedef int v4i __attribute__((ext_vector_type(4)));

// The value as it stands, so that what is computed from it starts here.
__host__ __device__ __forceinline__ uint32_t opaque(uint32_t x) {
#ifdef __HIP_DEVICE_COMPILE__
  asm("" : "+v"(x));
#endif
  return x;
}

// bytes 0-3 of the selector's table are lo's, 4-7 hi's
__host__ __device__ __forceinline__ uint32_t byte_perm(uint32_t hi, uint32_t lo, uint32_t sel) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_perm(hi, lo, sel);
#else
  const uint64_t t = (uint64_t(hi) << 32) | lo;
  uint32_t r = 0;
  for (int i = 0; i < 4; ++i) r |= uint32_t((t >> (8 * ((sel >> (8 * i)) & 7u))) & 0xFFu) << (8 * i);
  return r;
#endif
}

struct SparseOut {
  uint32_t v[4];  // stored values: byte 4i + slot of group i
  uint32_t idx;   // positions: bits 8i + 2 slot of group i
};

// a[p] and b[p]: half-words of groups 0, 1 and 2, 3 of plane p (bits 0-2 the
// position, bits 8-15 the code).
//
// One outlier per group at position p goes to slot p >> 1 (of the group's
// four slots): slots 0 and 2 hold an even-numbered pair's positions {0, 1} of
// their four, slots 1 and 3 {2, 3}, so the two positions of a four ascend
// whatever the codes are; an empty slot has value 0 at position 0 or 2.  Two
// outliers of a group (ascending) use the same rule unless both lie in one
// such pair: then they take the two slots of that four.
template <int NP>
__host__ __device__ __forceinline__ SparseOut sparse_outliers(const uint32_t (&a)[NP], const uint32_t (&b)[NP]) {
  // positions' index bytes: 0x88 (slots at positions 0, 2, 0, 2) with bit
  // (p & 1) << (p & 6) set
  constexpr uint32_t kIdxLo = 0x8C888988u, kIdxHi = 0xC8889888u;
  SparseOut s;
  const uint32_t p0 = byte_perm(b[0], a[0], 0x06040200u) & 0x07070707u;
  uint32_t sh0 = (p0 & 0x06060606u) << 2;  // 8 * slot, a byte per group
  s.idx = byte_perm(kIdxHi, kIdxLo, p0);
  if constexpr (NP == 1) {
    sh0 = opaque(sh0);  // a shift then takes its amount and its code from bytes in one instruction
    s.v[0] = ((a[0] >> 8) & 0xFFu) << (sh0 & 0xFFu);
    s.v[1] = (a[0] >> 24) << ((sh0 >> 8) & 0xFFu);
    s.v[2] = ((b[0] >> 8) & 0xFFu) << ((sh0 >> 16) & 0xFFu);
    s.v[3] = (b[0] >> 24) << (sh0 >> 24);
  } else {
    const uint32_t p1 = byte_perm(b[1], a[1], 0x06040200u) & 0x07070707u;
    uint32_t sh1 = (p1 & 0x06060606u) << 2;
    // bit 3 of a byte: both positions in one pair
    const uint32_t same = (0x08080808u - ((p0 ^ p1) & 0x06060606u)) & 0x08080808u;
    sh0 &= ~same;
    sh1 |= same;
    // both in one pair {q, q + 1}: the four's slots at q & 3 and (q & 3) + 1
    constexpr uint32_t kBothLo = 0x8E8E8484u, kBothHi = 0xE8E84848u;
    const uint32_t m = (same << 5) - (same >> 3);  // 0xFF where bit 3 is set
    s.idx = ((s.idx | byte_perm(kIdxHi, kIdxLo, p1)) & ~m) | (byte_perm(kBothHi, kBothLo, p0) & m);
    sh0 = opaque(sh0);
    sh1 = opaque(sh1);
    s.v[0] = (((a[0] >> 8) & 0xFFu) << (sh0 & 0xFFu)) | (((a[1] >> 8) & 0xFFu) << (sh1 & 0xFFu));
    s.v[1] = ((a[0] >> 24) << ((sh0 >> 8) & 0xFFu)) | ((a[1] >> 24) << ((sh1 >> 8) & 0xFFu));
    s.v[2] = (((b[0] >> 8) & 0xFFu) << ((sh0 >> 16) & 0xFFu)) | (((b[1] >> 8) & 0xFFu) << ((sh1 >> 16) & 0xFFu));
    s.v[3] = ((b[0] >> 24) << (sh0 >> 24)) | ((b[1] >> 24) << (sh1 >> 24));
  }
  return s;
}

}  // namespace dual
}  // namespace sdq
