// 7x7 stride-2 convolution of a 3-channel (RGB) image batch with ReLU and the
// 3x3 / stride-2 / pad-1 max-pool after it: the stem of the ImageNet ResNets in
// one pass over the image.
//
// Every wave works alone: it walks down a block of 16 stem columns of one
// image, two stem rows (one pooled row) at a time, and nothing but its weights
// passes through LDS.
//  * K is arranged per kernel row: the 7 pixels of one row of the window are 8
//    slots of 4 channels (the fourth channel and the eighth slot zero), one
//    32-wide K step of v_mfma_f32_16x16x32_bf16, so a lane's B operand is two
//    adjacent pixels of an input row.  Nine input rows feed two stem rows; five
//    of them stay in registers for the next two, four are loaded (16 bytes per
//    lane, one pooled row ahead) and widened from 3 to 4 channels there.
//  * All weights are A operands in registers (112 per lane).  Row r of MFMA
//    block cb is output channel 16 (r / 4) + 4 cb + r % 4, so a lane ends with
//    16 consecutive channels of one pixel.
//  * Scale, shift, ReLU and the rounding to bf16 happen in the accumulators'
//    place; the maximum over three rows is taken there too (the last row of a
//    pair is kept for the next one), and the maximum over three columns across
//    lanes.  16 stem columns from 14 b - 1 on hold the windows of 7 pooled
//    pixels, so blocks share 2 columns, and no data.
// The larger of two non-negative bf16 values is the one with the larger bits,
// hence ReLU only, and zero is the identity for rows and columns outside.
//
// What bounds it: a wave's own sequence of 56 MFMAs and 230 vector operations
// per pooled row, on the two waves per SIMD that 224 registers leave (256 images
// of 224 x 224: 2048 waves, the chip exactly; MFMAs alone: 42 us, the 180 MB 36
// us).  Measured for 256 images: 158 -> 102 us.  The form before staged the
// input rows and every stem row in LDS, with five barriers per four stem rows.
#include "conv_dev.hpp"
#include "kernels.hpp"

namespace dycl {
namespace k {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

constexpr int kKS = 7;        // kernel size
constexpr int kPool = 7;      // pooled pixels per block of 16 stem columns

struct StemPoolP {
  const uint16_t* x;   // [n][H][W][3]
  const uint16_t* w;   // [64][Kp], K order (kh, kw, c)
  const float* scale;
  const float* shift;
  uint16_t* y;         // [n][Hp][Wp][64]
  int n, H, W, Ho, Wo, Hp, Wp, pad, Kp;
  int blocks, parts;   // column blocks per image; ranges of pooled rows per image
};

__device__ __forceinline__ uint32_t max2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void stem_pool_kernel(StemPoolP p) {
  __shared__ __align__(16) uint4 wl[kKS * 4 * 64];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, l16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // weights: fragment (kh, block cb, lane) holds its output channel at K
  // values (kw, c) = (2 g + j / 4, j % 4), j < 8 (zero where kw >= 7 or c == 3)
  // (thread tid holds block cb = wave and lane `lane` of each kernel row; all
  // its loads are requested at once)
  {
    const int ch = 16 * (l16 >> 2) + 4 * (tid >> 6) + (l16 & 3);
    const uint16_t* wr = p.w + static_cast<size_t>(ch) * p.Kp + 2 * g * 3;
    uint32_t v[kKS][6];
#pragma unroll
    for (int kh = 0; kh < kKS; ++kh)
#pragma unroll
      for (int j = 0; j < 6; ++j) v[kh][j] = j < 3 || g < 3 ? wr[kh * kKS * 3 + j] : 0u;
#pragma unroll
    for (int kh = 0; kh < kKS; ++kh)
      wl[kh * 256 + tid] = make_uint4(v[kh][0] | (v[kh][1] << 16), v[kh][2], v[kh][3] | (v[kh][4] << 16), v[kh][5]);
  }
  __syncthreads();

  // this wave's unit: image, range of pooled rows, column block.  Workgroups
  // are dealt round robin over the XCDs: consecutive ones of a range to one.
  const int units = p.n * p.parts * p.blocks, T = (units + 3) / 4, T8 = (T >> 3) << 3;
  const int wg = blockIdx.x;
  const int u = (wg < T8 ? (wg & 7) * (T8 >> 3) + (wg >> 3) : wg) * 4 + wave;
  if (u >= units) return;                         // (no barrier follows)
  const int b = u % p.blocks, ip = u / p.blocks, part = ip % p.parts, img = ip / p.parts;
  const int j0 = part * p.Hp / p.parts, j1 = (part + 1) * p.Hp / p.parts;

  bf16x8 wf[kKS][4];
#pragma unroll
  for (int kh = 0; kh < kKS; ++kh)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) wf[kh][cb] = __builtin_bit_cast(bf16x8, wl[(kh * 4 + cb) * 64 + lane]);
  float sc[16], sh[16];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const u32x4 one = {0x3f800000u, 0x3f800000u, 0x3f800000u, 0x3f800000u}, zero = {0u, 0u, 0u, 0u};
    const u32x4 s4 = p.scale ? buffer_load16(p.scale, 256, 64 * g + 16 * q) : one;
    const u32x4 h4 = p.shift ? buffer_load16(p.shift, 256, 64 * g + 16 * q) : zero;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sc[4 * q + e] = __uint_as_float(s4[e]);
      sh[4 * q + e] = __uint_as_float(h4[e]);
    }
  }

  // this lane's stem column, and its two input pixels (iw, iw + 1) of a row;
  // the masks clear pixels outside the row and the eighth slot
  const int ow = 2 * kPool * b - 1 + l16, iw = 2 * ow - p.pad + 2 * g;
  const uint32_t m0 = iw >= 0 && iw < p.W ? ~0u : 0u;
  const uint32_t m1 = iw + 1 >= 0 && iw + 1 < p.W && g < 3 ? ~0u : 0u;
  const uint32_t m0l = m0 & 0xffffu;
  const uint32_t mcol = ow >= 0 && ow < p.Wo ? ~0u : 0u;
  // Byte offset of pixel iw in its row, down to a whole word: an odd pixel's
  // six bytes start in the middle of one.  A row's buffer is the row, and
  // offsets outside it (all of a row outside the image) read zeros, dword by
  // dword.
  const int odd = (p.pad & 1) * 16;               // shift of the words, in bits
  // (An offset before the row's start would lose all four words, and pixel 0
  // can be the second of a lane's two: that lane takes the row's first words
  // in the place of its last.)
  const bool first = iw == -1;
  const uint32_t lofs = first ? 0u : static_cast<uint32_t>(iw * 6 - (p.pad & 1) * 2);
  const int rowb = p.W * 6;
  int j = j0 > 0 ? j0 - 1 : 0;                    // pooled row
  int ih = 4 * j - p.pad;                         // the next input row to load, and its address
  const char* rp = reinterpret_cast<const char*>(p.x) + (static_cast<int64_t>(img) * p.H + ih) * rowb;
  auto load = [&]() __attribute__((always_inline)) {
    const bool in = static_cast<unsigned>(ih) < static_cast<unsigned>(p.H);
    const u32x4 r = buffer_load16(rp, static_cast<uint32_t>(rowb), in ? lofs : 0xC0000000u);
    ++ih;
    rp += rowb;
    return r;
  };
  auto widen = [&](u32x4 r) __attribute__((always_inline)) {
    r[2] = first ? r[0] : r[2];
    r[3] = first ? r[1] : r[3];
    const uint32_t a0 = __builtin_amdgcn_alignbit(r[1], r[0], odd), a1 = __builtin_amdgcn_alignbit(r[2], r[1], odd),
                   a2 = __builtin_amdgcn_alignbit(r[3], r[2], odd);
    return __builtin_bit_cast(
        bf16x8, u32x4{a0 & m0, a1 & m0l, __builtin_amdgcn_alignbit(a2, a1, 16) & m1, (a2 >> 16) & m1});
  };

  // one stem row from its seven input rows: bf16 pairs of channels 16 g + 2 r
  auto stem_row = [&](const bf16x8* f, bool live, uint32_t (&o)[8]) __attribute__((always_inline)) {
    f32x4 acc[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kh = 0; kh < kKS; ++kh)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[kh][cb], f[kh], acc[cb], 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int c = 2 * r;
      const float v0 = act_t<ACT_RELU>(fmaf(acc[c >> 2][c & 3], sc[c], sh[c]));
      const float v1 = act_t<ACT_RELU>(fmaf(acc[c >> 2][(c & 3) + 1], sc[c + 1], sh[c + 1]));
      o[r] = live ? pack_bf16(v0, v1) : 0u;
    }
  };

  // input rows 4 j - pad + k of pooled row j, k = 0 .. 8; a range that starts
  // inside the image first runs the pooled row before it, for the stem row
  // that the two share
  bf16x8 f[9];
#pragma unroll
  for (int k = 0; k < 5; ++k) f[k] = widen(load());
  u32x4 raw[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) raw[k] = load();
  uint32_t carry[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) carry[r] = 0u;
  const int pw = kPool * b + (l16 >> 1);
  // stores through a buffer of one pooled row: a lane without a pixel (and a
  // row that is not this range's) has an offset past it.  Every pass stores, so
  // the wait for its loads can leave the stores before them in flight.
  const uint32_t yofs = (l16 & 1) == 0 && l16 < 2 * kPool && pw < p.Wp ? pw * 128 + g * 32 : 0xC0000000u;
  const uint32_t ybytes = p.Wp * 128;
  uint16_t* yrow = p.y + (static_cast<int64_t>(img) * p.Hp + j) * p.Wp * 64;
  // (two stores to nowhere: every way into the loop then has the same
  // operations in flight behind its loads)
  buffer_store16(yrow, ybytes, 0xC0000000u, u32x4{0u, 0u, 0u, 0u});
  buffer_store16(yrow, ybytes, 0xC0000000u, u32x4{0u, 0u, 0u, 0u});
  for (; j < j1; ++j) {
#pragma unroll
    for (int k = 0; k < 4; ++k) f[5 + k] = widen(raw[k]);
#pragma unroll
    for (int k = 0; k < 4; ++k) raw[k] = load();   // the next pooled row's
    uint32_t a[8], c[8];
    stem_row(f, 2 * j < p.Ho, a);
    stem_row(f + 2, 2 * j + 1 < p.Ho, c);
    uint32_t o[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t m = max2(max2(a[r], c[r]), carry[r]) & mcol;
      carry[r] = c[r];
      const uint32_t s1 = __builtin_amdgcn_update_dpp(0u, m, 0x101, 0xf, 0xf, true);   // the column to the right
      const uint32_t s2 = __builtin_amdgcn_update_dpp(0u, m, 0x102, 0xf, 0xf, true);   // and the one after
      o[r] = max2(max2(m, s1), s2);
    }
    const uint32_t at = j >= j0 ? yofs : 0xC0000000u;
    buffer_store16(yrow, ybytes, at, u32x4{o[0], o[1], o[2], o[3]});
    buffer_store16(yrow, ybytes, at + 16, u32x4{o[4], o[5], o[6], o[7]});
    yrow += p.Wp * 64;
#pragma unroll
    for (int k = 0; k < 5; ++k) f[k] = f[k + 4];
  }
}

}  // namespace

void conv_stem_pool(const ConvArgs& a, hipStream_t s) {
  StemPoolP p;
  p.x = a.src;
  p.w = a.w;
  p.scale = a.scale;
  p.shift = a.shift;
  p.y = static_cast<uint16_t*>(a.dst);
  p.n = a.n;
  p.H = a.H;
  p.W = a.W;
  p.Ho = a.Ho;
  p.Wo = a.Wo;
  p.Hp = (a.Ho - 1) / 2 + 1;
  p.Wp = (a.Wo - 1) / 2 + 1;
  p.pad = a.pad;
  p.Kp = a.Kp;
  p.blocks = (p.Wp + kPool - 1) / kPool;
  // two waves per SIMD (2048) in one go; a range of pooled rows recomputes one
  // more, so none shorter than four
  const long whole = static_cast<long>(a.n) * p.blocks;
  const int most = p.Hp >= 8 ? p.Hp / 4 : 1;
  const long want = (2048 + whole - 1) / whole;
  p.parts = static_cast<int>(want < most ? want : most);
  const long wgs = (whole * p.parts + 3) / 4;
  hipLaunchKernelGGL(stem_pool_kernel, dim3(static_cast<unsigned>(wgs)), dim3(256), 0, s, p);
}

}  // namespace k
}  // namespace dycl
