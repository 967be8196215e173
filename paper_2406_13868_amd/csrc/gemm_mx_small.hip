// MX-family decomposed GEMM for few tokens (or few rows of W).  Section 5.1:
// Y = s_a * Xq (W_o + W_i)^T, both branches in one fp32 accumulator.
//
// At these sizes the packed weights are read and expanded once, which sets the
// time, so both have to be spread over the whole GPU without a second pass
// over partial sums: a workgroup owns 16 rows of W (half a tile) and all K of
// 16 * MT tokens, and its waves take interleaved 128-K chunks, whose sums meet
// in LDS in wave order.  The 16x16x128 scaled instruction (weights first,
// tokens as columns) takes a whole chunk and wastes no rows on 16 tokens.
//
// Operand layouts (16x16x128, lane l, r = l % 16 the row or column, quad l / 16):
//   fp8 operand: byte i holds K = 64*(i/16) + 16*quad + i%16
//   fp4 operand: nibble i of the first 4 dwords holds K = 32*quad + i
//   scale:       quad q supplies the scale of K block [32q, 32q + 32)
// So a lane's fp8 weights are two groups of block quad/2 and two of block
// 2 + quad/2, eight bytes of the packed words each, with no exchange between
// lanes.
//
// A wave requests its activations as whole lines (8 rows of 128 bytes; read as
// fragments straight from memory a request touches 16 rows and costs the
// address unit about twice as much) and reads the fragments back from an LDS
// region of its own, so that no barrier runs inside the loop.
//
// What bounds it: the vector instructions of the expansion (about 125 per
// chunk: 4.5 us of the 8.6 on 11008x4096 at M = 16, whose 21 MB stream in 4),
// then the launch and the chain of the first requests; from 64 tokens also the
// LDS traffic of the activations.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "mx_frag.h"
#include "tile_out.h"

namespace sdq {
namespace {

using namespace mx;

constexpr int kSmallRows = 16;  // rows of W per workgroup
constexpr int kNW = 8;          // waves per workgroup

typedef float f4v __attribute__((ext_vector_type(4)));
typedef int i4v __attribute__((ext_vector_type(4)));
typedef int i2v __attribute__((ext_vector_type(2)));

struct SmallArgs {
  const uint8_t* Xq;
  const float* s_a;
  const uint8_t* blob;
  void* Y;
  int M, N, K, n_chunks;
  int64_t scales_off;
  bool y_bf16, y_vec;
};

// 16 * MT tokens per workgroup.
template <int MT, int NI, bool HAS_O>
__global__ __launch_bounds__(kNW * 64) void mx_small_kernel(SmallArgs a) {
  constexpr int BM = 16 * MT;
  // a wave's own region: its chunk's activations (rows of 128 bytes, piece p of
  // row t at p ^ lds_swizzle(t)), then its sums [token tile][element][lane]
  constexpr int kWave = BM * kChunkK;
  static_assert(kWave >= MT * 4 * 64 * 4, "the sums fit the region");
  __shared__ __align__(16) uint8_t lds[kNW * kWave];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, quad = lane >> 4;
  const int b = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tile = b >> 1, r0 = (b & 1) * kSmallRows;
  const int m0 = blockIdx.y * BM;
  const int KC = a.n_chunks;
  const uint8_t* const wbase = a.blob + size_t(tile) * KC * kWordBytesPerTC;
  const uint8_t* const sbase = a.blob + a.scales_off + size_t(tile) * KC * kMxScaleBytesPerTC;
  const uint8_t* const xbase = a.Xq + size_t(m0) * a.K;
  const uint32_t wbytes = uint32_t(KC) * kWordBytesPerTC, sbytes = uint32_t(KC) * kMxScaleBytesPerTC;
  const uint32_t xbytes = uint32_t(min(a.M - m0, BM)) * uint32_t(a.K);
  // fp4 order: block `quad` (step quad / 2, half quad % 2); fp8 order: two
  // words of half quad / 2 of either step
  const uint32_t w4 = uint32_t((quad >> 1) * 1024 + ((quad & 1) * 32 + r0 + r) * 16);
  const uint32_t w8 = uint32_t(((quad >> 1) * 32 + r0 + r) * 16 + (quad & 1) * 8);
  const uint32_t se = uint32_t(((quad & 1) * 32 + r0 + r) * 4);   // word with the scales of block quad
  const uint32_t st = uint32_t(((quad >> 1) * 32 + r0 + r) * 4);  // word with the scales of the fp8 groups' blocks
  const uint32_t xo = uint32_t(lane >> 3) * uint32_t(a.K) + uint32_t(lane & 7) * 16;
  uint8_t* const mine = lds + wave * kWave;
  constexpr uint32_t kOut = 0x80000000u;  // past the end of every buffer here: reads 0

  struct Stage {
    i4v w;
    uint32_t se, st;
    i4v x[2 * MT];
  };
  auto load = [&](int c, Stage& s) __attribute__((always_inline)) {
    // chunks past the last request nothing (empty buffers)
    const bool in = c < KC;
    const uint32_t cc = in ? uint32_t(c) : 0u;
    const __amdgpu_buffer_rsrc_t wr = buffer_rsrc(wbase, in ? wbytes : 0u);
    const __amdgpu_buffer_rsrc_t sr = buffer_rsrc(sbase, in ? sbytes : 0u);
    const __amdgpu_buffer_rsrc_t xr = buffer_rsrc(xbase, in ? xbytes : 0u);
    s.se = __builtin_amdgcn_raw_buffer_load_b32(sr, se, cc * kMxScaleBytesPerTC, 0);
    if constexpr (HAS_O) {
      s.st = __builtin_amdgcn_raw_buffer_load_b32(sr, st, cc * kMxScaleBytesPerTC, 0);
      const i2v a0 = __builtin_bit_cast(i2v, __builtin_amdgcn_raw_buffer_load_b64(wr, w8, cc * kWordBytesPerTC, 0));
      const i2v a1 =
          __builtin_bit_cast(i2v, __builtin_amdgcn_raw_buffer_load_b64(wr, w8 + 1024, cc * kWordBytesPerTC, 0));
      s.w = i4v{a0[0], a0[1], a1[0], a1[1]};
    } else {
      s.w = __builtin_bit_cast(i4v, __builtin_amdgcn_raw_buffer_load_b128(wr, w4, cc * kWordBytesPerTC, 0));
    }
    // a partial last chunk: pieces past the row read 0, not the next row
    const uint32_t xc = int(cc) * kChunkK + 16 * (lane & 7) < a.K ? xo : kOut;
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i)
      s.x[i] = __builtin_bit_cast(i4v, __builtin_amdgcn_raw_buffer_load_b128(
                                           xr, xc + uint32_t(8 * i) * uint32_t(a.K), cc * kChunkK, 0));
  };

  f4v acc[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t] = f4v{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](int c, const Stage& s) __attribute__((always_inline)) {
    i8v xv[MT];
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) {
      const int row = (lane >> 3) + 8 * i;
      *reinterpret_cast<i4v*>(&mine[row * kChunkK + (((lane & 7) ^ lds_swizzle(row)) << 4)]) = s.x[i];
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const uint8_t* row = &mine[(16 * t + r) * kChunkK];
      const i4v x0 = *reinterpret_cast<const i4v*>(&row[(quad ^ lds_swizzle(r)) << 4]);
      const i4v x1 = *reinterpret_cast<const i4v*>(&row[((quad + 4) ^ lds_swizzle(r)) << 4]);
      xv[t] = __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7);
    }
    const uint32_t sb = s.se >> (16 * (quad >> 1));  // Eo, Ei of block quad
    if constexpr (HAS_O) {
      ShiftTable T[2];
      bool ok[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t q = s.st >> (16 * u);
        const int d = int((q >> 8) & 0xFFu) - int(q & 0xFFu);
        ok[u] = d >= -5 && d <= 6;
        T[u] = shift_table(d, ok[u]);
      }
      i8v bw;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t lo, hi;
        merged_e4m3<NI>(uint32_t(s.w[i]), T[i >> 1], lo, hi);
        bw[2 * i] = int(lo);
        bw[2 * i + 1] = int(hi);
      }
      const int e = int(sb & 0xFFu);
#pragma unroll
      for (int t = 0; t < MT; ++t)
        acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(bw, xv[t], acc[t], 0, 0, 0, e, 0, 127);
      if (__any(!(ok[0] && ok[1]))) {  // wave-uniform, rare: the inliers of blocks that did not merge
        const i4v wv = __builtin_bit_cast(
            i4v, __builtin_amdgcn_raw_buffer_load_b128(buffer_rsrc(wbase, wbytes), w4, uint32_t(c) * kWordBytesPerTC, 0));
        i8v bi;
        int ei;
        split_inliers_fp4<NI>(make_uint4(wv[0], wv[1], wv[2], wv[3]), s.se, quad >> 1, bi, ei);
#pragma unroll
        for (int t = 0; t < MT; ++t)
          acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(bi, xv[t], acc[t], 4, 0, 0, ei, 0, 127);
      }
    } else {
      i8v bw;
#pragma unroll
      for (int i = 0; i < 4; ++i) bw[i] = int(inlier_fp4<NI>(uint32_t(s.w[i])));
#pragma unroll
      for (int i = 4; i < 8; ++i) bw[i] = 0;
      const int e = int((sb >> 8) & 0xFFu);
#pragma unroll
      for (int t = 0; t < MT; ++t)
        acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(bw, xv[t], acc[t], 4, 0, 0, e, 0, 127);
    }
  };

  // wave w takes chunks w, w + kNW, ...: two in flight, each stage refilled
  // right after its products (four in flight measured slower: the workgroups
  // of a CU already hide each other's requests, and the registers cost waves)
  Stage s0, s1;
  load(wave, s0);
  load(wave + kNW, s1);
  int c = wave;
  for (; c + kNW < KC; c += 2 * kNW) {  // one exit, so the accumulators stay in place
    compute(c, s0);
    load(c + 2 * kNW, s0);
    compute(c + kNW, s1);
    load(c + 3 * kNW, s1);
  }
  if (c < KC) compute(c, s0);

  // ---- the waves' sums, in wave order (a wave's own region: its reads are over)
  float* const red = reinterpret_cast<float*>(mine);
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[(t * 4 + e) * 64 + lane] = acc[t][e];
  __syncthreads();
  if (wave >= MT) return;  // wave t finishes token tile t
  const int t = wave;
  f4v v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < kNW; ++w)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += reinterpret_cast<const float*>(lds + w * kWave)[(t * 4 + e) * 64 + lane];
  // lane (r, quad): token m0 + 16 t + r, outputs 4 quad .. + 3
  const int m = 16 * t + r, n = tile * kTileN + r0 + 4 * quad;
  if (m0 + m >= a.M || n >= a.N) return;
  const float sa = a.s_a[m0 + m];
  if (a.y_vec) {
    const OutRows yr = out_rows(a.Y, a.y_bf16, a.M, a.N, m0, BM);
    store_out4(yr, uint32_t(m) * uint32_t(a.N) + uint32_t(n), make_float4(sa * v[0], sa * v[1], sa * v[2], sa * v[3]));
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (n + i < a.N) store_y(a.Y, a.y_bf16, size_t(m0 + m) * size_t(a.N) + size_t(n + i), sa * v[i]);
  }
}

template <int MT, int NI>
hipError_t launch_o(const Cfg& c, const SmallArgs& a, int64_t n_tiles, hipStream_t st) {
  const dim3 grid(unsigned(2 * n_tiles), unsigned((a.M + 16 * MT - 1) / (16 * MT)));
  if (c.n_o)
    hipLaunchKernelGGL((mx_small_kernel<MT, NI, true>), grid, dim3(kNW * 64), 0, st, a);
  else
    hipLaunchKernelGGL((mx_small_kernel<MT, NI, false>), grid, dim3(kNW * 64), 0, st, a);
  return hipGetLastError();
}

template <int MT>
hipError_t launch_ni(const Cfg& c, const SmallArgs& a, int64_t n_tiles, hipStream_t st) {
  if (c.n_i == 1) return launch_o<MT, 1>(c, a, n_tiles, st);
  if (c.n_i == 2) return launch_o<MT, 2>(c, a, n_tiles, st);
  return launch_o<MT, 3>(c, a, n_tiles, st);
}

}  // namespace

// On SDQ_PATH_SPLITK alone, against the K ranges with their second pass; AUTO
// takes that path up to 16384 rows on K of 1024 and more (mx_split_wins in
// abi.hip), and the calls without a workspace never do.  Up to 32 tokens always
// (us per call, this kernel against the K ranges: 4096x4096 at M = 1 / 16 /
// 32 / 64: 4.9 / 5.0 / 5.6 / 7.7 against 8.6 / 9.7 / 10.8 / 14.0; 11008x4096
// at M = 1 / 16 / 32 8.4 / 8.6 / 11.0 against 13.2 / 14.8 / 16.4; 4096x11008 at M =
// 16 / 64: 8.6 / 14.6 against 14.9 / 18.8; 4096x1024 at M = 16: 2.8 against
// 7.4).  Up to 64 tokens on up to 12288 rows (22016x4096, a path asked for by
// name, at M = 48 / 64: 37.9 / 39.6 against 28.6 / 29.9) while rows are not
// long: a workgroup walks all of K, so its time follows K alone while the grid
// fits one round, where the K ranges' follows N too (M = 64, this kernel /
// K ranges: 1024 rows at K = 6144 / 8192 / 11008: 10.4, 11.0 / 12.3, 11.7 / 16.1,
// 13.5; 2048 rows at K = 11008 / 13824: 16.7, 18.6 / 19.5, 20.6; 4096 rows at K =
// 11008 / 16000: 17.4, 19.0 / 22.6, 21.1; 8192 rows at K = 4096 / 6144: 15.7, 16.2
// / 20.3, 19.2, 11008 rows at K = 2048 / 4096: 14.9, 17.6 / 21.8, 20.0).
// Above, each 64 tokens expand the weights again, which pays while the
// grid is at most two workgroups per CU on rows of up to 8192 K, or one on
// longer ones (4096x4096 at M = 128: 13.9 against 20.8, M = 256, four per CU,
// 24.5 against 26.7, M = 301 28 against 26; 1024x4096 at M = 256 / 512: 7.4 /
// 12.8 against 14.6 / 19.8; 2048x8192 at M = 128 / 256: 11.8 / 20.0 against
// 20.1 / 22.8; 4096x11008 at M = 128, two per CU: 27.7 against 24.7; 8192x2048
// at M = 128, four: 16.4 against 14.1), and on longer rows while the grid is
// not so small that the K ranges are the fuller one (M = 128: 256 rows, 32
// workgroups, at K = 11008 / 16000: 14.2, 13.4 / 18.8, 15.5; 512 rows 14.5, 14.3
// / 19.2, 17.2; 1024 rows, 128 workgroups, at K = 16000 20.7, 19.1; 2048 rows at
// K = 16000 / 20480: 21.2, 22.7 / 26.3, 25.5).
bool mx_small_wins(int64_t M, int64_t N, int64_t K) {
  if (M <= 32) return true;
  if (M <= 64) return N <= 4096 ? K < 8192 || (K <= (M <= 48 ? 12288 : 14336) && N > 1536)
                             : N <= 12288 && K <= (N <= 8192 ? 5120 : 3072);
  const int64_t wgs = (N + kSmallRows - 1) / kSmallRows * ((M + 63) / 64);
  if (K <= 8192) return wgs <= 512;
  return wgs <= 256 && wgs >= (K <= 14336 ? 64 : K <= 16384 ? 160 : 256);
}

hipError_t launch_mx_small(const Cfg& c, const uint8_t* Xq, const float* s_a, int64_t M, const uint8_t* blob,
                           int64_t N, int64_t K, void* Y, hipStream_t st) {
  const Layout L = make_layout(true, N, K);
  const SmallArgs a{Xq, s_a, blob, Y, int(M), int(N), int(K), int(L.n_chunks), L.scales_off, c.y_bf16, out_vec(Y, N)};
  if (M <= 16) return launch_ni<1>(c, a, L.n_tiles, st);
  if (M <= 32) return launch_ni<2>(c, a, L.n_tiles, st);
  return launch_ni<4>(c, a, L.n_tiles, st);
}

}  // namespace sdq
