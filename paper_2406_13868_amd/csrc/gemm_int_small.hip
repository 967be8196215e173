// INT-family decomposed GEMM for 9 to 64 tokens.  Section 5.1:
// Y = SpMM(A, W_o) + SpMM(A, W_i), one fp32 result per output.
//
// At these sizes the vector work of expanding every packed weight once, not
// the matrix cores, sets the time, so it has to be spread over the whole GPU:
// a workgroup owns 16 rows of W (half a tile; 4096 rows are 256 workgroups,
// one per CU, where a 32-row tile per workgroup would leave half of them
// idle) and 16 or 32 tokens, and its waves take interleaved 128-K chunks.
// The 16x16x32 f16 instruction (weights first, tokens as columns) wastes no
// rows on 16 tokens.  Lane l holds row l % 16 and, by l / 16, the lane half h
// and the half j of the chunk: the four words of its 16 bytes are the groups
// 8j + 2q + h, so one 1 KB request brings the 16 rows' words of a chunk and
// instruction q takes the four lane quarters' groups.
//
// A wave requests its activations as whole lines (a request that touches 32
// rows costs the address unit 62 cycles, one of 8 rows 17), converts them to
// f16 once and reads its fragments back from an LDS region of its own, so
// that no barrier runs inside the loop.  Both branches are exact as in
// gemm_int_mfma.hip (hi and lo fragments; int8 outliers on the int8
// instruction in int32, e4m3 ones on the f16 instruction).  The waves' sums
// meet in LDS in wave order.
//
// What bounds it: the vector instructions of the expansion (about 45 per
// word, 230 per chunk with the activations' conversion: 3.8 us of the 8.1 on
// 4096x4096 at M = 16), then the launch and the chain of the first requests.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "int_frag.h"
#include "kernels.h"
#include "tile_out.h"

namespace sdq {
namespace {

using namespace intfrag;

constexpr int kSmallRows = 16;            // rows of W per workgroup
constexpr int kRowF = kChunkK + 8;        // f16 per token row in LDS
constexpr int kRowB = kChunkK + 16;       // int8 bytes per token row

typedef float f4v __attribute__((ext_vector_type(4)));
typedef int i4v __attribute__((ext_vector_type(4)));

struct SmallArgs {
  const uint8_t* Xq;
  const float* s_a;
  const uint8_t* blob;
  void* Y;
  int M, N, K, n_chunks;
  int64_t scales_off, rows_off, irow_off;
  int qs, srow;  // log2(qv / 16); bytes of a row's scales in a chunk
  bool y_bf16, y_vec;
};

template <int MT, int NI, bool OUT_INT8, int NW, int SF>
__global__ __launch_bounds__(NW * 64) void int_small_kernel(SmallArgs a) {
  constexpr bool SC8 = SF == kScaleE4M3;  // two-level: a power of two per row
  constexpr bool ONE = SF != kScaleF16;   // q * s exact in one fp16 fragment
  constexpr int BM = 16 * MT;
  constexpr int kF = BM * kRowF * 2, kStage = kF + (OUT_INT8 ? BM * kRowB : 0);
  constexpr int kRed = 2 * MT * 4 * 64 * 4;  // a wave's sums: [branch][token tile][element][lane]
  constexpr int kWave = kStage > kRed ? kStage : kRed;
  __shared__ __align__(16) uint8_t lds[NW * kWave];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, quad = lane >> 4, h = quad & 1, j = quad >> 1;
  const int b = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tile = b >> 1, r0 = (b & 1) * kSmallRows;
  const int m0 = blockIdx.y * BM;
  const int KC = a.n_chunks;
  const int kSB = kTileN * a.srow;
  uint8_t* const mine = lds + wave * kWave;
  _Float16* const xf = reinterpret_cast<_Float16*>(mine);
  uint8_t* const xb = mine + kF;

  const __amdgpu_buffer_rsrc_t wr =
      buffer_rsrc(a.blob + size_t(tile) * KC * kWordBytesPerTC, uint32_t(KC) * kWordBytesPerTC);
  // (16 bytes more: a request may take bytes of the next row's scales, or of
  // the row scales that follow in the blob)
  const __amdgpu_buffer_rsrc_t sr =
      buffer_rsrc(a.blob + a.scales_off + size_t(tile) * KC * kSB, uint32_t(KC) * kSB + 16);
  const __amdgpu_buffer_rsrc_t xr =
      buffer_rsrc(a.Xq + size_t(m0) * a.K, uint32_t(min(a.M - m0, BM)) * uint32_t(a.K));
  const uint32_t woff = uint32_t((h * 32 + r0 + r) * 2 + j) * 16;
  // this lane's four blocks' scales: srow / 2 bytes, as the low bytes of 8
  const uint32_t sbyte = uint32_t((r0 + r) * a.srow + j * (a.srow >> 1));
  const uint32_t soff = sbyte & ~3u, sshift = 8 * (sbyte & 3u);
  const uint32_t xoff = uint32_t(lane >> 3) * uint32_t(a.K) + uint32_t(lane & 7) * 16;

  typedef unsigned int u4_ __attribute__((ext_vector_type(4)));
  typedef unsigned int u2_ __attribute__((ext_vector_type(2)));
  struct Stage {
    u4_ w;
    u2_ s;
    u4_ x[2 * MT];
  };
  auto load = [&](int c, Stage& st) __attribute__((always_inline)) {  // chunks past the last read 0 weights
    st.w = __builtin_bit_cast(u4_, __builtin_amdgcn_raw_buffer_load_b128(wr, woff, uint32_t(c) * kWordBytesPerTC, 0));
    st.s = __builtin_bit_cast(u2_, __builtin_amdgcn_raw_buffer_load_b64(sr, soff, uint32_t(c) * kSB, 0));
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i)
      st.x[i] = __builtin_bit_cast(u4_, __builtin_amdgcn_raw_buffer_load_b128(
                                            xr, xoff + uint32_t(8 * i) * uint32_t(a.K), uint32_t(c) * kChunkK, 0));
  };

  using OAcc = std::conditional_t<OUT_INT8, i4v, f4v>;
  f4v acc[MT];
  OAcc acco[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) { acc[t] = f4v{0.f, 0.f, 0.f, 0.f}; acco[t] = OAcc{0, 0, 0, 0}; }

  auto compute = [&](const Stage& st) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) {
      const int row = (lane >> 3) + 8 * i, cp = lane & 7;
      uint32_t o[8];
#pragma unroll
      for (int q = 0; q < 4; ++q) i8x4_to_f16x4(st.x[i][q], o[2 * q], o[2 * q + 1]);
      uint4* dst = reinterpret_cast<uint4*>(&xf[row * kRowF + cp * 16]);
      dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
      dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
      if constexpr (OUT_INT8) *reinterpret_cast<u4_*>(&xb[row * kRowB + cp * 16]) = st.x[i];
    }
    const uint32_t sv[4] = {st.s[0] >> sshift, st.s[1], 0, 0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t w = st.w[q];
      const _Float16 s = block_scale<SF>(sv, q, a.qs);
      h8 bh, bl;
      if constexpr (ONE) {
        const h8 sv8 = {s, s, s, s, s, s, s, s};
        bh = inlier_f16<NI>(w) * sv8;  // exact in fp16 (at most 7 significant bits)
      } else {
        scaled_hi_lo(inlier_f16<NI>(w), s, bh, bl);
      }
      h8 av[MT];
#pragma unroll
      for (int t = 0; t < MT; ++t)
        av[t] = *reinterpret_cast<const h8*>(&xf[(16 * t + r) * kRowF + (8 * j + 2 * q + h) * 8]);
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bh, av[t], acc[t], 0, 0, 0);
        if constexpr (!ONE) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bl, av[t], acc[t], 0, 0, 0);
      }
      if constexpr (OUT_INT8) {
        if ((q & 1) == 0) {  // words q and q + 1 in one int8 instruction over 64 K
          uint32_t o0, o1, o2, o3;
          outlier_i8(w, o0, o1);
          outlier_i8(st.w[q + 1], o2, o3);
          const i4v bo = {int(o0), int(o1), int(o2), int(o3)};
#pragma unroll
          for (int t = 0; t < MT; ++t) {
            const uint8_t* p = &xb[(16 * t + r) * kRowB + (8 * j + 2 * q + h) * 8];
            const u2_ x0 = *reinterpret_cast<const u2_*>(p), x1 = *reinterpret_cast<const u2_*>(p + 16);
            const i4v ax = {int(x0[0]), int(x0[1]), int(x1[0]), int(x1[1])};
            acco[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bo, ax, acco[t], 0, 0, 0);
          }
        }
      } else {
        const h8 bo = outlier_f16(w);
#pragma unroll
        for (int t = 0; t < MT; ++t) acco[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bo, av[t], acco[t], 0, 0, 0);
      }
    }
  };

  // wave w takes chunks w, w + NW, ...: two in flight, each stage refilled
  // right after its products
  Stage s0, s1;
  load(wave, s0);
  load(wave + NW, s1);
  int c = wave;
  for (; c + NW < KC; c += 2 * NW) {  // one exit, so the accumulators stay in place
    compute(s0);
    load(c + 2 * NW, s0);
    compute(s1);
    load(c + 3 * NW, s1);
  }
  if (c < KC) compute(s0);

  // ---- the waves' sums, in wave order (a wave's own region: its reads are over)
  float* const red = reinterpret_cast<float*>(mine);
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const auto o = acco[t][e];
      red[(t * 4 + e) * 64 + lane] = acc[t][e];
      red[((MT + t) * 4 + e) * 64 + lane] = __builtin_bit_cast(float, o);
    }
  __syncthreads();
  if (tid >= MT * 64) return;  // whole waves: wave t finishes token tile t
  const int t = wave;
  f4v va = {0.f, 0.f, 0.f, 0.f};
  OAcc vo = {0, 0, 0, 0};
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float* p = reinterpret_cast<const float*>(lds + w * kWave);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float o = p[((MT + t) * 4 + e) * 64 + lane];
      va[e] += p[(t * 4 + e) * 64 + lane];
      vo[e] += __builtin_bit_cast(std::conditional_t<OUT_INT8, int, float>, o);
    }
  }
  // lane (r, quad): token m0 + 16 t + r, outputs 4 quad .. + 3
  const int m = 16 * t + r, n = tile * kTileN + r0 + 4 * quad;
  if (m0 + m >= a.M || n >= a.N) return;
  const float4 so = *reinterpret_cast<const float4*>(a.blob + a.rows_off + int64_t(n) * 4);
  const float4 gi = SC8 ? *reinterpret_cast<const float4*>(a.blob + a.irow_off + int64_t(n) * 4)
                        : make_float4(1.f, 1.f, 1.f, 1.f);
  const float sa = a.s_a[m0 + m];
  const float4 v = make_float4(sa * fmaf(so.x, float(vo[0]), gi.x * va[0]), sa * fmaf(so.y, float(vo[1]), gi.y * va[1]),
                               sa * fmaf(so.z, float(vo[2]), gi.z * va[2]), sa * fmaf(so.w, float(vo[3]), gi.w * va[3]));
  const OutRows yr = out_rows(a.Y, a.y_bf16, a.M, a.N, m0, BM);
  if (a.y_vec) {
    store_out4(yr, uint32_t(m) * uint32_t(a.N) + uint32_t(n), v);
  } else {
    const float q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (n + i < a.N) store_y(a.Y, a.y_bf16, size_t(m0 + m) * size_t(a.N) + size_t(n + i), q[i]);
  }
}

template <int MT, int NI, int SF>
hipError_t launch_nw(const Cfg& c, const SmallArgs& a, int64_t n_tiles, hipStream_t st) {
  const dim3 grid(unsigned(2 * n_tiles), unsigned((a.M + 16 * MT - 1) / (16 * MT)));
  if (c.fmt_o == SDQ_FMT_INT8)
    hipLaunchKernelGGL((int_small_kernel<MT, NI, true, 8, SF>), grid, dim3(512), 0, st, a);
  else
    hipLaunchKernelGGL((int_small_kernel<MT, NI, false, 8, SF>), grid, dim3(512), 0, st, a);
  return hipGetLastError();
}

template <int MT, int SF>
hipError_t launch_ni(const Cfg& c, const SmallArgs& a, int64_t n_tiles, hipStream_t st) {
  if (c.n_i == 1) return launch_nw<MT, 1, SF>(c, a, n_tiles, st);
  if (c.n_i == 2) return launch_nw<MT, 2, SF>(c, a, n_tiles, st);
  return launch_nw<MT, 3, SF>(c, a, n_tiles, st);
}

template <int MT>
hipError_t launch_sf(const Cfg& c, const SmallArgs& a, int64_t n_tiles, hipStream_t st) {
  if (c.sc8) return launch_ni<MT, kScaleE4M3>(c, a, n_tiles, st);
  if (c.e6m2) return launch_ni<MT, kScaleE6M2>(c, a, n_tiles, st);
  return launch_ni<MT, kScaleF16>(c, a, n_tiles, st);
}

}  // namespace

// Up to 16 tokens always (4096x4096 at M = 16: 8.1 us against 14.1 in 32-row
// tiles, 11008x4096 16.1 against 23.3, 16384x4096 20.6 against 24.4,
// 4096x11008 16.9 against 20.7 on the split-K path); up to 64 while one round
// of workgroups holds the grid (4096x4096 at M = 32: 10.3 against 14.7;
// 1024x4096 at M = 64: 9.1 against 13.6; two rounds, 4096x4096 at M = 48: 15.3
// against 15.1); and up to 32 tokens on up to 12288 rows with e4m3 outliers,
// whose staging leaves room for two workgroups per CU (11008x4096 at M = 32:
// 21.7 against 24.5, with int8 outliers 27.4 against 22.8; 16384x4096 27.8
// against 25.5).
bool int_small_wins(const Cfg& c, int64_t M, int64_t N) {
  if (M <= 16) return true;
  const int64_t tiles = (N + kTileN - 1) / kTileN;
  if (M <= 64 && 2 * tiles * ((M + 31) / 32) <= 256) return true;
  return M <= 32 && c.fmt_o != SDQ_FMT_INT8 && tiles <= 384;
}

hipError_t launch_int_small(const Cfg& c, const uint8_t* Xq, const float* s_a, int64_t M, const uint8_t* blob,
                            int64_t N, int64_t K, void* Y, hipStream_t st) {
  const Layout L = layout_for(c, N, K);
  const SmallArgs a{Xq, s_a, blob, Y, int(M), int(N), int(K), int(L.n_chunks), L.scales_off, L.rows_off, L.irow_off,
                    c.qv == 64 ? 2 : c.qv == 32 ? 1 : 0, int((kChunkK / c.qv) * c.scale_bytes()), c.y_bf16,
                    out_vec(Y, N)};
  return M <= 16 ? launch_sf<1>(c, a, L.n_tiles, st) : launch_sf<2>(c, a, L.n_tiles, st);
}

}  // namespace sdq
