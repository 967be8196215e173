// Dual-family decomposed GEMM: Section 5.1's worked configuration, in which
// the outliers (int8) multiply int8 activations A_o and the inliers (fp4)
// multiply fp4 activations A_i:
//   Y[m,n] = s_a[m] * s_o[n] * sum_k A_o[m,k] q_o[n,k]
//          + sum_k A_i[m,k] 2^Ea[m,k/32] * q_i[n,k] 2^Ei[n,k/32].
//
// On gfx950 both branches are matrix-core contractions:
//   * inliers: v_mfma_scale_f32_32x32x64_f8f6f4 with fp4 on both sides and
//     the two e8m0 scales applied inside the instruction.  The packer stores
//     the n_i:8 inliers as dense nibbles (zeros at the other positions) in
//     exactly the operand order, so the B fragment is one 16-byte load per
//     lane and needs no expansion;
//   * outliers: the int8 instructions, exact in int32.  In the split-K form
//     v_mfma_i32_32x32x32_i8: each lane expands its two groups' (position,
//     code) half-words into 16 dense bytes; with 2:8 outliers the second
//     plane's half-words scatter into the same bytes (the two positions of a
//     group differ).  Lane half h covers K [16h, 16h + 16) of the 32-K step
//     for both operands (the K order inside the instruction is free as long
//     as A and B agree).
// The branches accumulate apart (fp32 and int32) and meet in the epilogue.
//
// Tiled form: a workgroup covers 4*TN 32-row tiles of W and 32*MS tokens with
// eight waves, two per SIMD.  Four of them (one per TN tiles) multiply the
// inliers and four the outliers of the same outputs, so that every wave
// holds one set of accumulators: the fp32 sums and the int32 sums of a 128 x
// 64 wave tile together would leave a SIMD one wave, whose vector, LDS and
// memory instructions then add to its matrix time instead of hiding behind
// it (128 x 256 outputs at M = 4096, 11008x4096: 282 us with one wave for
// both branches, 268 with two).  The two sums meet in LDS at the end.
//
// The outliers run on v_smfmac_i32_32x32x64_i8 (dual_frag.h): at most two of
// eight positions are stored, so the 2:4 sparse instruction covers them, 64
// dense K in the time the dense instruction takes for 32 (measured 7.85 PF
// against 4.05).  W is the first operand (the sparse one), tokens are the
// columns.
//
// The activations of a 128-K chunk are staged in LDS once per workgroup in
// three buffers (one barrier per chunk); weights stream into registers a
// chunk and more ahead.  What bounds it, by counters on 11008x4096 at M = 4096
// (128 x 256): a chunk takes a compute unit 2550 cycles, of which the matrix
// cores are busy 1024 (MfmaUtil 37-39%), the LDS 800, the vector memory address
// unit 1690 and its data path 1930 (76%; a request of 64 lanes x 16 bytes takes
// the address unit 17 cycles, one of 4 bytes a lane 9, one that touches 32 rows
// 62).  That layer: 268 us (dense int8 outliers, one wave per SIMD: 390);
// 4096x4096 at M = 256: 14.5 (28).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dual_frag.h"
#include "kernels.h"
#include "tile_out.h"

namespace sdq {
namespace {

constexpr int kDWaves = 4;
constexpr int kDThreads = kDWaves * 64;

using namespace dual;

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

struct DualArgs {
  const uint8_t* Xo;  // [M][K] int8 codes of A_o
  const float* s_a;   // [M] fp32 scales of A_o
  const uint8_t* Xi;  // [M][K/2] e2m1 codes of A_i, the even k in the low nibble
  const uint8_t* Ea;  // [M][K/32] e8m0 scales of A_i
  const uint8_t* blob;
  void* Y;
  int M, N, K, n_chunks, n_tiles;
  int64_t out_off, scale_off, rows_off;
  bool y_bf16 = false;  // Y as bf16
  int groups = 1, m_blocks = 1;  // tiled form: the grid is 1-D over (tile group, token block)
  bool y_vec = false;   // Y 16-byte aligned and N a multiple of 4
};

__device__ __forceinline__ v4i ld16(__amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, v, s, 0);
}
__device__ __forceinline__ int ld8(__amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
  return int(__builtin_amdgcn_raw_buffer_load_b8(r, v, s, 0));
}

// The four e8m0 scales of chunk cs of the A_i row at byte v of ea, block j
// in byte j.  One dword when K is a multiple of 128.  Otherwise a row's K/32
// bytes do not fill whole dwords, and a dword reaching past the end of the
// buffer's range would read as 0 whole: four byte loads, and 127 (2^0) for
// the blocks past K, whose weight codes are zero and add nothing whatever
// their scale.
__device__ __forceinline__ uint32_t ld_ea4(__amdgpu_buffer_rsrc_t ea, uint32_t v, uint32_t cs, uint32_t K) {
  if ((K & 127u) == 0) return __builtin_amdgcn_raw_buffer_load_b32(ea, v, cs * 4, 0);
  uint32_t e = 0;
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j)
    e |= (cs * 4 + j < K / 32 ? uint32_t(__builtin_amdgcn_raw_buffer_load_b8(ea, v + j, cs * 4, 0)) : 127u)
         << (8 * j);
  return e;
}

// Dense int8 bytes of two 8-groups from their half-words (bits 0-2 position,
// bits 8-15 code): group i fills dwords 2i, 2i + 1.
__device__ __forceinline__ v4i outlier_bytes(uint32_t hw2) {
  const uint32_t v0 = hw2 & 0xFFFFu, v1 = hw2 >> 16;
  const uint32_t b0 = (v0 >> 8) << ((v0 & 3u) << 3), b1 = (v1 >> 8) << ((v1 & 3u) << 3);
  const bool u0 = (v0 & 4u) != 0, u1 = (v1 & 4u) != 0;
  const v4i r = {int(u0 ? 0u : b0), int(u0 ? b0 : 0u), int(u1 ? 0u : b1), int(u1 ? b1 : 0u)};
  return r;
}

// Outlier bytes per (tile, chunk) with NP half-word planes.
template <int NP>
constexpr uint32_t out_bytes_tc() { return uint32_t(NP) * kDualOutBytesPerTC; }

// Dense int8 outlier bytes of two groups from NP planes of half-word pairs.
template <int NP>
__device__ __forceinline__ v4i outlier_bytes_np(const uint32_t (&hw)[NP]) {
  v4i b = outlier_bytes(hw[0]);
  if constexpr (NP == 2) b |= outlier_bytes(hw[1]);
  return b;
}

// Physical 16-byte piece of logical piece p of an LDS row: 128-byte rows of
// A_o codes (8 pieces) and 64-byte rows of A_i codes (4), XORed with a
// function of the row so that any aligned group of 8 or 16 rows reads one
// logical piece from distinct banks (32 or 64 banks of 4 bytes).
__device__ __forceinline__ int swz_o(int r) { return (r & 7) ^ ((r >> 3) & 1); }
__device__ __forceinline__ int swz_i(int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); }

template <int MS, int TN, int NP, int KG>
__global__ __launch_bounds__(KG * 2 * kDThreads, KG * 2) void dual_tiled_kernel(DualArgs a) {
  constexpr int BM = 32 * MS;
  // LDS: three chunk buffers of the workgroup's activations (xo_s: codes of
  // A_o, xi_s: of A_i), then the e8m0 scales of A_i as [chunk & 15][row] (the
  // four bytes of a row's chunk); the epilogue stages its outputs over them
  constexpr int kXo = BM * kChunkK, kXi = kXo / 2, kEa = 3 * (kXo + kXi);
  constexpr int kOutW = TN * kTileN, kOutRow = kOutW + 4;  // staged floats per token, padded
  constexpr int kOutBytes = kDWaves * BM * kOutRow * 4;
  constexpr int kGroupBytes = kEa + 16 * BM * 4;  // of one K group's loop
  // KG = 2: the second K group's accumulators, [role][wave][tile][sub-tile][element][lane]
  constexpr int kRedBytes = KG == 1 ? 0 : 2 * kDWaves * TN * MS * 16 * 64 * 4;
  constexpr int kLds = KG * kGroupBytes > kOutBytes + kRedBytes ? KG * kGroupBytes : kOutBytes + kRedBytes;
  __shared__ __align__(16) uint8_t lds[kLds];

  const int tid = int(threadIdx.x) % (2 * kDThreads), lane = tid & 63;  // within the K group
  const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(int(threadIdx.x) / (2 * kDThreads));
  const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave8 & 3;
  uint8_t* const xo_s = lds + kg * kGroupBytes;
  uint8_t* const xi_s = xo_s + 3 * kXo;
  uint32_t* const ea_s = reinterpret_cast<uint32_t*>(xo_s + kEa);
  const int col = lane & 31, h = lane >> 5;
  int group, mblock;
  square_work(blockIdx.x, a.groups, a.m_blocks, group, mblock);
  const int m0 = mblock * BM;
  const int t0 = (group * kDWaves + wave) * TN;  // the wave's first tile (tiles past the last read 0)
  const int KC = a.n_chunks, last = KC - 1;
  // the K group's chunks, cn of them from cb on (a second group's last may
  // lie past the end: its weights read 0)
  const int cn = KG == 1 ? KC : (KC + 1) / 2, cb = kg * cn;
  const uint32_t K = uint32_t(a.K);

  // activations of the workgroup's rows (rows past M read 0)
  const uint32_t rows = uint32_t(min(a.M - m0, BM));
  const __amdgpu_buffer_rsrc_t xo = buffer_rsrc(a.Xo + size_t(m0) * K, rows * K);
  const __amdgpu_buffer_rsrc_t xi = buffer_rsrc(a.Xi + size_t(m0) * (K / 2), rows * (K / 2));
  // (from up to 16 rows before, so that the range holds 16 bytes)
  const uint32_t eback = uint32_t(min(m0, 16)), ebytes = (rows + eback) * (K / 32);
  const __amdgpu_buffer_rsrc_t ea = buffer_rsrc(a.Ea + size_t(m0 - int(eback)) * (K / 32), ebytes);

  // One role's main loop (0: inliers, 1: outliers) and its part of the
  // outputs, which end up in os (kOutRow floats per token) for the stores.
  float* const os = reinterpret_cast<float*>(lds) + wave * (BM * kOutRow);
  auto run = [&](auto role_tag) __attribute__((always_inline)) {
    constexpr int ROLE = decltype(role_tag)::value;
    typedef std::conditional_t<ROLE == 0, v16f, v16i> Acc;

    // ---- the wave's tiles: dense inlier nibbles and their scales, or outlier half-words
    __amdgpu_buffer_rsrc_t w0[TN], w1[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
      const bool ok = t0 + t < a.n_tiles;
      const size_t tc = size_t(ok ? t0 + t : 0) * KC;
      const uint32_t kc = ok ? uint32_t(KC) : 0u;
      if constexpr (ROLE == 0) {
        w0[t] = buffer_rsrc(a.blob + tc * kDualNibBytesPerTC, kc * kDualNibBytesPerTC);
        w1[t] = buffer_rsrc(a.blob + a.scale_off + tc * kDualScaleBytesPerTC, kc * kDualScaleBytesPerTC);
      } else {
        w0[t] = buffer_rsrc(a.blob + a.out_off + tc * out_bytes_tc<NP>(), kc * out_bytes_tc<NP>());
      }
    }

    // ---- activation staging of chunk c, in 16-byte pieces (8 per row of
    //      A_o, 4 per row of A_i; LDS in order, the logical piece by the
    //      row's swizzle).  From 64 tokens all threads move A_o's, with 32
    //      the outlier waves; the inlier waves move A_i's and the scales.
    //      The scales of a row are few bytes a chunk, and a request costs by
    //      the lines it touches, so they come 16 bytes (four chunks) at a
    //      time for a quarter of the rows: with chunk c the rows BM / 4 *
    //      (c & 3) .. of the four chunks after chunk c's, eight lanes of each
    //      wave on eight rows (fewer below 128 tokens, the rest repeat them).
    constexpr bool kMoveO = MS >= 2 || ROLE == 1;
    constexpr int kPo = !kMoveO ? 0 : MS >= 2 ? MS / 2 : 1;
    constexpr int kPi = ROLE == 1 ? 0 : MS >= 2 ? MS / 2 : 1;
    constexpr int kPieces = kPo + kPi + (ROLE == 0 ? 1 : 0);
    struct XRegs { v4i o[kPo + 1]; v4i i[kPi + 1]; v4i e; };
    constexpr int kOThreads = MS >= 2 ? 2 * kDThreads : kDThreads;
    const int otid = tid % kOThreads, itid = tid % kDThreads;
    const uint32_t ro = uint32_t(otid >> 3), ri = uint32_t(itid >> 2) % BM;
    const uint32_t re = uint32_t(wave * 8 + (lane >> 3)) % (BM / 4);
    const uint32_t vo = ro * K + uint32_t(((otid & 7) ^ swz_o(ro)) * 16);
    const uint32_t vi = ri * (K / 2) + uint32_t(((itid & 3) ^ swz_i(ri)) * 16);
    const uint32_t pi = (uint32_t(itid) % (BM * 4)) * 16;
    // A row's request for the four chunks from c & ~3 on is made early by d
    // bytes where it would reach past the row's end, and its bytes move down:
    // the slots of blocks past K then hold bytes of the same row.  The weights
    // there are zero codes, which cancel any finite scale but not a NaN (0xFF),
    // and a NaN of this row makes its outputs NaN anyway, whereas the bytes
    // that follow in memory are the next row's.  (Masks in the loop instead:
    // 4096x4096 at M = 256 in 15.6 us, not 14.2; a branch for the last chunks
    // undid the loop's schedule, 11008x4096 at M = 4096 in 1300 us, not 239.)
    const int eblocks = int(K / 32);
    auto e_start = [&](int c) { return min((cb + (c & ~3)) * 4, eblocks - 16); };
    auto e_row = [&](int c) { return re + uint32_t(c & 3) * (BM / 4); };
    auto load_e = [&](int c, v4i& e) __attribute__((always_inline)) {
      e = ld16(ea, (e_row(c) + eback) * (K / 32) + uint32_t(e_start(c)), 0);
    };
    auto move_down = [](v4i& e, uint32_t d) __attribute__((always_inline)) {
      if (d & 8) { e[0] = e[2]; e[1] = e[3]; }
      if (d & 4) { e[0] = e[1]; e[1] = e[2]; e[2] = e[3]; }
#pragma unroll
      for (int j = 0; j < 4; ++j) e[j] = int(__builtin_amdgcn_alignbyte(e[j < 3 ? j + 1 : 3], e[j], d & 3));
    };
    auto store_e = [&](int c, v4i e) __attribute__((always_inline)) {
      move_down(e, uint32_t((cb + (c & ~3)) * 4 - e_start(c)));
#pragma unroll
      for (int j = 0; j < 4; ++j) ea_s[(((c & ~3) + j) & 15) * BM + e_row(c)] = e[j];
    };
    // The same for the K group's first four chunks, whatever the row's length
    // (a row of fewer than 16 blocks ends within them): early only where the
    // buffer ends, and 2^0 for the blocks past K.
    auto load_e0 = [&](int q, v4i& e) __attribute__((always_inline)) {
      e = ld16(ea, min((e_row(q) + eback) * (K / 32) + uint32_t(cb) * 4, ebytes - 16), 0);
    };
    auto store_e0 = [&](int q, v4i e) __attribute__((always_inline)) {
      const uint32_t off = (e_row(q) + eback) * (K / 32) + uint32_t(cb) * 4;
      move_down(e, off - min(off, ebytes - 16));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int left = min(max(eblocks - 4 * (cb + j), 0), 4);  // blocks of the row in this dword
        const uint32_t own = uint32_t((uint64_t(1) << (8 * left)) - 1);
        ea_s[j * BM + e_row(q)] = (uint32_t(e[j]) & own) | (0x7F7F7F7Fu & ~own);
      }
    };
    auto load_x1 = [&](int c, XRegs& x, int j) __attribute__((always_inline)) {
      const uint32_t cs = uint32_t(min(cb + c, last));
      if (j < kPo) x.o[j] = ld16(xo, vo + uint32_t(j) * (kOThreads / 8) * K, cs * kChunkK);
      else if (j < kPo + kPi) x.i[j - kPo] = ld16(xi, vi + uint32_t(j - kPo) * 32 * K, cs * (kChunkK / 2));
      else load_e(c + 4, x.e);
    };
    auto store_x1 = [&](int buf, int c, const XRegs& x, int j) __attribute__((always_inline)) {
      if (j < kPo) *reinterpret_cast<v4i*>(&xo_s[buf * kXo + (otid + j * kOThreads) * 16]) = x.o[j];
      else if (j < kPo + kPi) *reinterpret_cast<v4i*>(&xi_s[buf * kXi + pi + (j - kPo) * kDThreads * 16]) = x.i[j - kPo];
      else store_e(c + 4, x.e);
    };
    auto load_x = [&](int c, XRegs& x) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < kPieces; ++j) load_x1(c, x, j);
    };
    auto store_x = [&](int buf, int c, const XRegs& x) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < kPieces; ++j) store_x1(buf, c, x, j);
    };

    // ---- the wave's weight stream, one 64-K step per stage
    struct BIn {
      v4i bi[TN];       // fp4 inlier fragments
      uint32_t sb[TN];  // the dword that holds their e8m0 scale (block 2s + h of row col)
    };
    struct BOut {
      uint32_t hw[TN][2][NP];  // outlier half-word pairs of the two 32-K steps, per plane
    };
    typedef std::conditional_t<ROLE == 0, BIn, BOut> BStep;
    constexpr int kLoads = ROLE == 0 ? 2 * TN : 2 * TN * NP;  // requests per step
    auto load_b1 = [&](int c, int s, BStep& st, int j) __attribute__((always_inline)) {
      const uint32_t cs = uint32_t(cb + c);  // past the last chunk: reads 0
      if constexpr (ROLE == 0) {
        const int t = j >> 1;
        if ((j & 1) == 0)
          st.bi[t] = ld16(w0[t], uint32_t(s * 64 + lane) * 16u, cs * kDualNibBytesPerTC);
        else
          // (a byte load would be narrowed to 8 bits across the loop, and its
          // widening waits for the load at the top of the chunk; shifted at use)
          st.sb[t] = __builtin_amdgcn_raw_buffer_load_b32(w1[t], uint32_t(s * 64 + (lane & ~3)),
                                                          cs * kDualScaleBytesPerTC, 0);
      } else {
        const int t = j / (2 * NP), u = (j / NP) & 1, p = j % NP;
        st.hw[t][u][p] = __builtin_amdgcn_raw_buffer_load_b32(
            w0[t], uint32_t(p * kDualOutBytesPerTC) + uint32_t((2 * s + u) * 64 + lane) * 4u, cs * out_bytes_tc<NP>(), 0);
      }
    };
    auto load_b = [&](int c, int s, BStep& st) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < kLoads; ++j) load_b1(c, s, st, j);
    };

    // ---- activation fragments of one (64-K step, 32-token sub-tile)
    struct FIn { v4i i; uint32_t e; };
    struct FOut { v4i o0, o1; };
    typedef std::conditional_t<ROLE == 0, FIn, FOut> Frag;
    uint32_t ai[2], ao[2][2];  // LDS byte offsets of row col
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      ai[s] = uint32_t(col * (kChunkK / 2) + (((2 * s + h) ^ swz_i(col)) << 4));
#pragma unroll
      for (int u = 0; u < 2; ++u) ao[s][u] = uint32_t(col * kChunkK + (((4 * s + 2 * h + u) ^ swz_o(col)) << 4));
    }
    auto read_frag = [&](int buf, int c, int s, int ms, Frag& f) __attribute__((always_inline)) {
      if constexpr (ROLE == 0) {
        f.i = *reinterpret_cast<const v4i*>(&xi_s[buf * kXi + ai[s] + ms * 32 * (kChunkK / 2)]);
        f.e = ea_s[(c & 15) * BM + ms * 32 + col];  // (shifted where it is used, after the wait for the slot's reads)
      } else {
        f.o0 = *reinterpret_cast<const v4i*>(&xo_s[buf * kXo + ao[s][0] + ms * 32 * kChunkK]);
        f.o1 = *reinterpret_cast<const v4i*>(&xo_s[buf * kXo + ao[s][1] + ms * 32 * kChunkK]);
      }
    };

    Acc acc[TN][MS];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][ms][e] = 0;

    XRegs X[2];           // [chunk parity]
    BStep B[2][2];        // [chunk parity][step]
    SparseOut so[2][TN];  // [step]; outliers
    Frag F[2];
    auto expand = [&](const BStep& w, int t, SparseOut& d) __attribute__((always_inline)) {
      if constexpr (ROLE == 1) d = sparse_outliers<NP>(w.hw[t][0], w.hw[t][1]);
    };
    // the prologue's requests in the loop's own order, which the compiler's
    // wait counts at the loop head would otherwise be tightened to
    {
      XRegs P0, P1;
      v4i e0[4];  // the scales of chunks 0..3, every quarter of the rows
      load_x(0, P0);
      load_x(1, P1);
      if constexpr (ROLE == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) load_e0(q, e0[q]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        load_x(2 + p, X[p]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 2 - p; ++s) load_b(p, s, B[p][s]);
        __builtin_amdgcn_sched_barrier(0);
      }
      store_x(0, 0, P0);
      store_x(1, 1, P1);
      if constexpr (ROLE == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) store_e0(q, e0[q]);
      }
    }
    __syncthreads();
    read_frag(0, 0, 0, 0, F[0]);
#pragma unroll
    for (int t = 0; t < TN; ++t) expand(B[0][0], t, so[0][t]);

    // One chunk is 2 MS slots, one per (step, sub-tile).  A slot reads the
    // next slot's activation fragment, multiplies its own by the TN tiles,
    // and carries a share of the other work: the next step's sparse operands,
    // the weights of chunk c + 2 into the registers the previous step freed,
    // and chunk c + 2's activations from registers to LDS and c + 4's into
    // them.  Slots are kept apart for the scheduler, which would otherwise
    // sink products past the barrier.
    int b0 = 0, b1 = 1, b2 = 2;  // LDS buffers of chunks c, c + 1, c + 2
    auto chunk = [&](int c, BStep (&W)[2], BStep (&V)[2], XRegs& x) __attribute__((always_inline)) {
      constexpr int kSlots = 2 * MS;
#pragma unroll
      for (int k = 0; k < kSlots; ++k) {
        const int s = k / MS, ms = k % MS;
        const Frag& f = F[k & 1];
        Frag& nx = F[(k + 1) & 1];
        if (k + 1 < kSlots) read_frag(b0, c, (k + 1) / MS, (k + 1) % MS, nx);
        else read_frag(b1, c + 1, 0, 0, nx);
        // the other step's operands: step 1 of this chunk, or step 0 of the next
#pragma unroll
        for (int t = 0; t < TN; ++t)
          if (ms == (MS >= 4 ? 1 + t : MS - 1)) expand(s == 0 ? W[1] : V[0], t, so[1 - s][t]);
#pragma unroll
        for (int j = k * kPieces / kSlots; j < (k + 1) * kPieces / kSlots; ++j) {
          store_x1(b2, c + 2, x, j);
          load_x1(c + 4, x, j);
        }
#pragma unroll
        for (int t = 0; t < TN; ++t) {
          if constexpr (ROLE == 0) {
            const v8i xa = {f.i[0], f.i[1], f.i[2], f.i[3], 0, 0, 0, 0};
            const v8i wa = {W[s].bi[t][0], W[s].bi[t][1], W[s].bi[t][2], W[s].bi[t][3], 0, 0, 0, 0};
            // fp4 (format 4) on both sides, each lane half with its block's scale
            acc[t][ms] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                wa, xa, acc[t][ms], 4, 4, 0, int(W[s].sb[t] >> (8 * (lane & 3))), 0, int(f.e >> (16 * s + 8 * h)));
          } else {
            const v8i xb = __builtin_shufflevector(f.o0, f.o1, 0, 1, 2, 3, 4, 5, 6, 7);
            const v4i wv = {int(so[s][t].v[0]), int(so[s][t].v[1]), int(so[s][t].v[2]), int(so[s][t].v[3])};
            acc[t][ms] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(wv, xb, acc[t][ms], int(so[s][t].idx), 0, 0);
          }
        }
        // the step that just ended leaves its registers to a later chunk's
#pragma unroll
        for (int j = ms * kLoads / MS; j < (ms + 1) * kLoads / MS; ++j) {
          if (s == 0) load_b1(c + 1, 1, V[1], j);
          else load_b1(c + 2, 0, W[0], j);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
      const int t = b0;
      b0 = b1;
      b1 = b2;
      b2 = t;
    };
    int c = 0;
    for (; c + 1 < cn; c += 2) {  // one exit, so the accumulators stay in place
      chunk(c, B[0], B[1], X[0]);
      chunk(c + 1, B[1], B[0], X[1]);
    }
    if (c < cn) chunk(c, B[0], B[1], X[0]);  // a last chunk of even rank

    // ---- the second K group's accumulators join the first's
    if constexpr (KG == 2) {
      typedef std::conditional_t<ROLE == 0, float, int> Elem;
      Elem* const red = reinterpret_cast<Elem*>(lds + kOutBytes) + (ROLE * kDWaves + wave) * (TN * MS * 16 * 64) + lane;
      if (kg == 1) {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
          for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int e = 0; e < 16; ++e) red[((t * MS + ms) * 16 + e) * 64] = acc[t][ms][e];
      }
      __syncthreads();
      if (kg == 0) {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
          for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][ms][e] += red[((t * MS + ms) * 16 + e) * 64];
      }
    }
    // ---- lane (col, h) holds token 32 ms + col, outputs 8 j + 4 h .. + 3 of
    //      each tile: the outlier waves leave s_o * P in LDS, the inlier
    //      waves turn that into the output in place
    if constexpr (ROLE == 1) {
      if (kg == 0) {
#pragma unroll
        for (int t = 0; t < TN; ++t) {
          const float* sop = reinterpret_cast<const float*>(a.blob + a.rows_off) + min(t0 + t, a.n_tiles - 1) * kTileN + 4 * h;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float4 q = *reinterpret_cast<const float4*>(sop + 8 * j);
#pragma unroll
            for (int ms = 0; ms < MS; ++ms)
              *reinterpret_cast<float4*>(&os[(ms * 32 + col) * kOutRow + t * kTileN + 8 * j + 4 * h]) =
                  make_float4(q.x * float(acc[t][ms][4 * j]), q.y * float(acc[t][ms][4 * j + 1]),
                              q.z * float(acc[t][ms][4 * j + 2]), q.w * float(acc[t][ms][4 * j + 3]));
          }
        }
      }
      __syncthreads();
    } else {
      const __amdgpu_buffer_rsrc_t sr = buffer_rsrc(a.s_a + m0, rows * 4u);
      float sa[MS];
#pragma unroll
      for (int ms = 0; ms < MS; ++ms)
        sa[ms] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(sr, uint32_t(ms * 32 + col) * 4u, 0, 0));
      __syncthreads();
      if (kg == 0) {
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
          for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              float4* p = reinterpret_cast<float4*>(&os[(ms * 32 + col) * kOutRow + t * kTileN + 8 * j + 4 * h]);
              const float4 q = *p;
              *p = make_float4(fmaf(sa[ms], q.x, acc[t][ms][4 * j]), fmaf(sa[ms], q.y, acc[t][ms][4 * j + 1]),
                               fmaf(sa[ms], q.z, acc[t][ms][4 * j + 2]), fmaf(sa[ms], q.w, acc[t][ms][4 * j + 3]));
            }
      }
    }
    __syncthreads();
  };
  if (wave8 < kDWaves) run(std::integral_constant<int, 0>{});
  else run(std::integral_constant<int, 1>{});

  // ---- the waves that share an output group store an equal part of its tokens
  const int nw = t0 * kTileN, n_left = a.N - nw;  // the group's outputs
  constexpr int kRows = BM / (2 * KG);
  const int r_lo = (2 * kg + (wave8 >> 2)) * kRows;
  store_staged<kOutW>(os + r_lo * kOutRow, out_rows(a.Y, a.y_bf16, a.M, a.N, m0, BM), a.y_vec, a.N, r_lo, kRows, nw,
                      n_left, lane);
}

// Split-K form for few tokens (up to 32, more on narrow layers): one 32-row tile per workgroup, its
// NW waves take interleaved 128-K chunks (two in flight per wave) and read
// their activations straight into registers; the wave partials of both
// accumulators are summed through LDS in a fixed-order tree.  This keeps
// n_tiles * NW waves streaming weights where the tiled form above would run
// only n_tiles / 4 workgroups.
template <int NW, int NP>
__global__ __launch_bounds__(NW * 64, 2) void dual_splitk_kernel(DualArgs a) {
  __shared__ float red[NW / 2][2][16][64];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, h = lane >> 5;
  const int m0 = blockIdx.y * 32;
  const int tile = blockIdx.x;
  const int KC = a.n_chunks, last = KC - 1;
  const uint32_t K = uint32_t(a.K);

  const uint32_t rows = uint32_t(min(a.M - m0, 32));
  const __amdgpu_buffer_rsrc_t xo = buffer_rsrc(a.Xo + size_t(m0) * K, rows * K);
  const __amdgpu_buffer_rsrc_t xi = buffer_rsrc(a.Xi + size_t(m0) * (K / 2), rows * (K / 2));
  const __amdgpu_buffer_rsrc_t ea = buffer_rsrc(a.Ea + size_t(m0) * (K / 32), rows * (K / 32));
  const __amdgpu_buffer_rsrc_t wn =
      buffer_rsrc(a.blob + size_t(tile) * KC * kDualNibBytesPerTC, uint32_t(KC) * kDualNibBytesPerTC);
  const __amdgpu_buffer_rsrc_t wo = buffer_rsrc(a.blob + a.out_off + size_t(tile) * KC * out_bytes_tc<NP>(),
                                                uint32_t(KC) * out_bytes_tc<NP>());
  const __amdgpu_buffer_rsrc_t ws = buffer_rsrc(a.blob + a.scale_off + size_t(tile) * KC * kDualScaleBytesPerTC,
                                                uint32_t(KC) * kDualScaleBytesPerTC);

  struct Stage {
    v4i bi[2];
    int sb[2];
    uint32_t hw[4][NP];
    v4i ai[2];
    uint32_t sa;  // the chunk's four e8m0 bytes of token row col
    v4i ao[4];
  };
  auto load = [&](int c, Stage& st) __attribute__((always_inline)) {
    const uint32_t cs = uint32_t(c);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      st.bi[s] = ld16(wn, uint32_t(s * 64 + lane) * 16u, cs * kDualNibBytesPerTC);
      st.sb[s] = ld8(ws, uint32_t(s * 64 + lane), cs * kDualScaleBytesPerTC);
      st.ai[s] = ld16(xi, uint32_t(col) * (K / 2) + uint32_t(s * 32 + h * 16), cs * (kChunkK / 2));
    }
    st.sa = ld_ea4(ea, uint32_t(col) * (K / 32), cs, K);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
      for (int p = 0; p < NP; ++p)
        st.hw[u][p] = __builtin_amdgcn_raw_buffer_load_b32(
            wo, uint32_t(p * kDualOutBytesPerTC) + uint32_t(u * 64 + lane) * 4u, cs * out_bytes_tc<NP>(), 0);
      st.ao[u] = ld16(xo, uint32_t(col) * K + uint32_t(u * 32 + h * 16), cs * kChunkK);
    }
  };

  v16f acc;
  v16i acco;
#pragma unroll
  for (int e = 0; e < 16; ++e) { acc[e] = 0.f; acco[e] = 0; }

  auto compute = [&](const Stage& st) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const v8i b = {st.bi[s][0], st.bi[s][1], st.bi[s][2], st.bi[s][3], 0, 0, 0, 0};
      const v8i av = {st.ai[s][0], st.ai[s][1], st.ai[s][2], st.ai[s][3], 0, 0, 0, 0};
      const int sa = int((st.sa >> (8 * (2 * s + h))) & 0xFFu);
      acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, b, acc, 4, 4, 0, sa, 0, st.sb[s]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      acco = __builtin_amdgcn_mfma_i32_32x32x32_i8(st.ao[u], outlier_bytes_np<NP>(st.hw[u]), acco, 0, 0, 0);
  };

  // wave w takes chunks w, w + NW, ...; stage s0 its even-numbered ones and s1
  // the odd ones, each refilled right after its products; loads past the last
  // chunk re-read it (never used)
  Stage s0, s1;
  load(min(wave, last), s0);
  load(min(wave + NW, last), s1);
  int c = wave;
  for (; c + NW < KC; c += 2 * NW) {  // one exit, so the accumulators stay in place
    compute(s0);
    load(min(c + 2 * NW, last), s0);
    compute(s1);
    load(min(c + 3 * NW, last), s1);
  }
  if (c < KC) compute(s0);

  // ---- tree over the waves: in round r, wave w + 2^r hands its partials to w
#pragma unroll
  for (int stride = NW / 2; stride >= 1; stride >>= 1) {
    if (wave >= stride && wave < 2 * stride) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float x = acc[e];
        const int y = acco[e];
        red[wave - stride][0][e][lane] = x;
        red[wave - stride][1][e][lane] = __int_as_float(y);
      }
    }
    __syncthreads();
    if (wave < stride) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[e] += red[wave][0][e][lane];
        acco[e] += __float_as_int(red[wave][1][e][lane]);
      }
    }
    __syncthreads();
  }
  if (wave > 0) return;
  const int n = tile * kTileN + col;
  if (n >= a.N) return;
  const float so = reinterpret_cast<const float*>(a.blob + a.rows_off)[n];
  const RowScales<1> rs = load_row_scales<1>(a.s_a, a.M, m0, h);
  const OutRows yr = out_rows(a.Y, a.y_bf16, a.M, a.N, m0, 32);
#pragma unroll
  for (int e = 0; e < 16; ++e) store_out(yr, a.N, n, 0, e, h, fmaf(rs.v[0][e], so * float(acco[e]), acc[e]));
}

template <int MS, int TN, int NP, int KG>
hipError_t launch_tiled(DualArgs a, hipStream_t st) {
  a.groups = (a.n_tiles + kDWaves * TN - 1) / (kDWaves * TN);
  a.m_blocks = (a.M + 32 * MS - 1) / (32 * MS);
  const dim3 grid(unsigned(a.groups) * unsigned(a.m_blocks));
  hipLaunchKernelGGL((dual_tiled_kernel<MS, TN, NP, KG>), grid, dim3(KG * 2 * kDThreads), 0, st, a);
  return hipGetLastError();
}

template <int NP>
hipError_t launch_np(DualForm f, const DualArgs& a, hipStream_t st) {
  switch (f) {
    case DualForm::k32x128: return launch_tiled<1, 1, NP, 2>(a, st);
    case DualForm::k64x128: return launch_tiled<2, 1, NP, 1>(a, st);
    case DualForm::k64x256: return launch_tiled<2, 2, NP, 1>(a, st);
    case DualForm::k128x256: return launch_tiled<4, 2, NP, 1>(a, st);
    default: break;
  }
  const dim3 grid(unsigned(a.n_tiles), unsigned((a.M + 31) / 32));
  hipLaunchKernelGGL((dual_splitk_kernel<4, NP>), grid, dim3(4 * 64), 0, st, a);
  return hipGetLastError();
}

}  // namespace

// The split-K form while its grid (one tile x 32 tokens per workgroup) stays
// within one round, and on wider layers up to 12 tokens (16 with two outlier
// planes, whose expansion weighs more in the tiled form): its waves gather
// activation rows themselves, which costs by the row (4096x4096 at M = 16 / 64:
// 9.4 / 12.7 us against 12.2 / 12.6 in tiles; 11008x4096, 344 workgroups, at M =
// 9 / 16 / 32, weights from memory: 15.0 / 17.0 / 24.2 against 16.0 / 16.4 /
// 18.5, with two planes 17.4 / 18.7 / 26.1 against 19.5 / 20.1 / 22.6); and up to
// 24 tokens on rows of up to 768 and 32 on 512, where a tile's prologue is most
// of its time (11008x512 at M = 9 / 16 / 32: 5.6 / 5.9 / 6.8 against 6.6 / 6.6 /
// 7.0; 8224x768 at M = 16 / 24: 6.6 / 7.2 against 7.3 / 7.4; 11008x1024 at M = 9 /
// 16 / 32 8.3 / 9.1 / 11.6 against 8.2 / 8.4 / 9.0).  Else the tiled form
// of least cost, with these costs of a round of 256 workgroups in half
// microseconds at K = 4096 (other K scale alike): 32 tokens x 128 outputs 27;
// 64 x 128 33, and 24 for each further round (two run per CU); 64 x 256 46;
// 128 x 256 66.  Measured (the four in this order): 4096x4096 at M = 256 / 512
// / 1024 / 2048: 14.2, 16.6, 21.2, 29.2 / 26.1, 19.6, 23.8, 30.8 / 53.7, 32.3,
// 28.2, 35.6 / -, 60.7, 55.6, 46.0; 11008x4096 at M = 128 / 256 / 512: 24.9,
// 17.7, 21.9, 29.6 / 37.2, 27.7, 24.4, 31.5 / 71.0, 42.5, 46.3, 36.7;
// 4096x11008 at M = 256 / 768: 28.8, 35.8, 45.9, 63.6 / 81.2, 66.1, 52.8, 68.7.
DualForm dual_form(int64_t M, int64_t N, int64_t K, int planes) {
  if (dual_decode_fits(M, N, K)) return DualForm::kDecode;
  const int64_t tiles = (N + kTileN - 1) / kTileN;
  // (what is left has the 16 bytes of scales that the tiled form's first requests take)
  if (M <= (planes == 2 ? 16 : 12) || (M <= 24 && K <= 768) || (M <= 32 && K <= 512) || tiles * ((M + 31) / 32) <= 256)
    return DualForm::kSplitK;
  const int64_t g4 = (tiles + 3) / 4, g8 = (tiles + 7) / 8;
  const auto rounds = [](int64_t wgs) { return (wgs + 255) / 256; };
  const int64_t c11 = 27 * rounds(g4 * ((M + 31) / 32)), c21 = 9 + 24 * rounds(g4 * ((M + 63) / 64));
  const int64_t c22 = 46 * rounds(g8 * ((M + 63) / 64)), c42 = 66 * rounds(g8 * ((M + 127) / 128));
  if (c11 <= c21 && c11 <= c22 && c11 <= c42) return DualForm::k32x128;
  if (c21 <= c22 && c21 <= c42) return DualForm::k64x128;
  return c22 <= c42 ? DualForm::k64x256 : DualForm::k128x256;
}

hipError_t launch_dual_mfma(const Cfg& c, const uint8_t* Xo, const float* s_a, const uint8_t* Xi,
                            const uint8_t* Ea, int64_t M, const uint8_t* blob, int64_t N, int64_t K,
                            void* Y, hipStream_t st) {
  const DualLayout L = make_dual_layout(N, K, c.n_o);
  DualArgs a{Xo, s_a, Xi, Ea, blob, Y, int(M), int(N), int(K), int(L.n_chunks), int(L.n_tiles),
             L.out_off, L.scale_off, L.rows_off};
  a.y_bf16 = c.y_bf16;
  a.y_vec = out_vec(Y, N);
  const DualForm f = dual_form(M, N, K, L.out_planes);
  if (f == DualForm::kDecode) return launch_dual_decode(c, Xo, s_a, Xi, Ea, M, blob, N, K, Y, st);
  return L.out_planes == 2 ? launch_np<2>(f, a, st) : launch_np<1>(f, a, st);
}

}  // namespace sdq
