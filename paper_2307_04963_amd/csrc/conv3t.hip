// 3x3 / stride 1 / pad 1 convolutions with Cin and Cout multiples of 64:
// linear pixel tiles, the input patch and the weights in LDS.
//
// A workgroup of four waves (2 x 2) computes BM consecutive output pixels
// (of the whole batch: a tile may cross rows and images, so only the last
// one is partly empty) times BN output channels.  K runs over 64-channel
// chunks and, inside a chunk, the nine taps; one step is one tap of one
// chunk, 64 of K.
//  * The chunk's input patch is staged in LDS once and read by all nine taps.
//    It lives in a virtual image list in which every image row is preceded by
//    one zero pixel and every image by one zero row: the pixel (img, r, c)
//    has the index ((img (H + 1) + r + 1) (W + 1) + c + 1), whose eight
//    neighbours are at constant distances, and the patch of a tile is one
//    contiguous range of indices.  The zeros of the padding come from the
//    range check of the buffer loads.  A patch pixel is 128 bytes; its eight
//    16-byte chunks are XOR-swizzled by the index, so the 16 lanes of a
//    ds_read_b128 phase fall on distinct bank groups.
//  * The weights of a step (BN rows of 128 bytes, swizzled alike) are loaded
//    straight into one of two LDS stages while the step before runs.
//
// What bounds it: the MFMAs, from 128 x 128 tiles on (the MFMAs and barriers of
// a layer's K loop alone take 73 % of the loop's time; the loads straight into
// LDS 16 %, the operand reads 13 %, measured with either left out), and the
// load latency of a step on few tiles.  Two workgroups share a CU (80 KB of
// LDS each), so the load of a patch, the epilogue and the barriers of one run
// under the other's MFMAs.  Measured, before (persistent workgroups with
// loader waves: four waves computing) and after: 183 images 28x28, 128 -> 128
// channels 61 -> 45 us (950 TFLOP/s); 107 of 14x14, 256 -> 256 38 -> 30 us;
// 774 of 16x16, 128 -> 128 with a residual 90 -> 68 us.  On top of the whole
// tiles' gain it comes from the linear tiles: whole-row tiles of 28- and
// 14-pixel images left 12 and 24 % of the MFMA rows empty.
#include "conv_dev.hpp"
#include "kernels.hpp"

namespace dycl {
namespace k {

namespace {

// x / d for 0 <= x < 2^31, d >= 2: the high half of a product and a shift
struct Div {
  uint32_t mul, sh;
};
Div div_by(uint32_t d) {
  uint32_t l = 1;
  while ((1ull << l) < d) ++l;   // 2^(l - 1) < d <= 2^l
  return {static_cast<uint32_t>((1ull << (31 + l)) / d + 1), l - 1};
}
__device__ __forceinline__ int quot(int x, const Div& d) {
  return static_cast<int>(__umulhi(static_cast<uint32_t>(x), d.mul) >> d.sh);
}

struct Conv3TP {
  const uint16_t* src;
  const uint16_t* w;       // [cout_pad][Kp] packed, K = tap * cin + ci
  const float* scale;
  const float* shift;
  const uint16_t* res;
  uint16_t* dst;
  int n, H, W, cin, cout, Kp;
  int nt;                  // output channel tiles
  Div dHW, dW, dPW, dH1;   // division by H W, W, W + 1 and H + 1
  const int32_t* nc;       // device count of live images (<= n) or null
};

// patch pixels of a tile of bm consecutive pixels: the pixels, a zero pixel
// per row boundary and a zero row per image boundary inside, and a row and a
// pixel on either side
int patch_pixels(int bm, int H, int W) {
  const int b = bm - 1;
  return b + (b + W - 1) / W + (b + H * W - 1) / (H * W) * (W + 1) + 2 * (W + 1) + 3;
}

template <int TA, int TB, int CAP, int NS, int D, bool EARLY, int ACT, bool RES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void conv3t_kernel(Conv3TP p) {
  constexpr int WP = 2, WC = 2;
  constexpr int BM = 32 * TA * WP, BN = 32 * TB * WC, WN = 32 * TB;
  constexpr int JW = BN / 32;                     // weight loads per thread and step
  constexpr int NJ = (CAP + 31) / 32;             // patch loads per thread and chunk
  constexpr int EPW = WN + 4;                     // epilogue staging row (floats)
  constexpr int EPB = 32 * EPW * 4;               // epilogue staging of a wave
  constexpr int WS = BN * 128;                    // bytes of a weight stage
  static_assert(CAP * 128 >= 2 * EPB && NS * WS >= 2 * EPB, "epilogue staging fits");
  // separate objects: reads of one do not wait for loads into another
  __shared__ __align__(128) char patch[CAP * 128];
  __shared__ __align__(128) char wst[NS * BN * 128];

  const int HW = p.H * p.W, PW = p.W + 1, cin = p.cin, Kp = p.Kp;
  const int n = p.nc ? min(*p.nc, p.n) : p.n;
  const int M = n * HW;
  // XCD-aware order: workgroup ids are dealt round robin over the eight
  // XCDs; consecutive tiles (which share halo rows, and the channel tiles of
  // one pixel tile, which share the patch) go to one XCD
  const int T = (M + BM - 1) / BM * p.nt, T8 = (T >> 3) << 3;
  const int wg = blockIdx.x;
  if (wg >= T) return;
  const int t = wg < T8 ? (wg & 7) * (T8 >> 3) + (wg >> 3) : wg;
  const int mt = t / p.nt;
  const int m0 = mt * BM, n0 = (t - mt * p.nt) * BN;

  const int tid = threadIdx.x, lane = tid & 63, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = wave >> 1, wc = wave & 1;

  // loads: thread tid brings 16-byte slot tid of every 32-row group; its
  // chunk of a row is the same in each (rows advance by 32)
  const int lrow = tid >> 3, lch = (tid & 7) ^ ((tid >> 4) & 7);
  const uint16_t* const wlane = p.w + static_cast<size_t>(n0 + lrow) * Kp + lch * 8;
  auto issue_w = [&](char* st, int koff, int j) __attribute__((always_inline)) {
    load_lds16(wlane + koff + static_cast<size_t>(j) * 32 * Kp, st + j * 4096 + wave * 1024);
  };
  static_assert(NS >= 2 && NS <= 9, "the first steps are taps of the first chunk");
#pragma unroll
  for (int g = 0; g < NS - 1; ++g)
#pragma unroll
    for (int j = 0; j < JW; ++j) issue_w(wst + g * WS, g * cin, j);

  auto vidx = [&](int m) __attribute__((always_inline)) {
    const int img = quot(m, p.dHW), rem = m - img * HW, r = quot(rem, p.dW);
    return (img * (p.H + 1) + r + 1) * PW + (rem - r * p.W) + 1;
  };
  const int vf = vidx(m0);                        // index of the tile's first pixel
  const int NP = vidx(min(m0 + BM, M) - 1) - vf + 2 * PW + 3;
  // byte offset of each of this thread's patch slots; zero pixels get one that
  // no buffer reaches.  The buffer starts at the first pixel that the patch can
  // hold (pixel mq of the tile's first image: the one above and to the left of
  // the tile's first), so the offsets span the patch and not the images that it
  // lies in: those may be of any size.
  const int img0 = quot(m0, p.dHW);
  const int mq = max(m0 - img0 * HW - p.W - 1, 0), mp = img0 * HW + mq;
  uint32_t pofs[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int v = vf - PW - 1 + j * 32 + lrow;
    const int vr = quot(v, p.dPW), c = v - vr * PW, img = quot(vr, p.dH1), r = vr - img * (p.H + 1);
    pofs[j] = (c >= 1 && r >= 1 && img < n)
                  ? static_cast<uint32_t>(((img - img0) * HW + (r - 1) * p.W + (c - 1) - mq) * cin * 2 + lch * 16)
                  : 0xC0000000u;
  }
  const uint16_t* const sbase = p.src + static_cast<size_t>(mp) * cin;
  const size_t sleft = static_cast<size_t>(M - mp) * cin * 2;
  const uint32_t sbytes = sleft < 0x7fffffffu ? static_cast<uint32_t>(sleft) : 0x7fffffffu;
  auto issue_patch = [&](int chunk) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      if (j * 32 + lrow < NP)                     // the patch ends inside its last group
        buffer_load_lds16(sbase + chunk * 64, sbytes - chunk * 128, pofs[j],
                          (lds_void_ptr)(patch + j * 4096 + wave * 1024));
  };
  issue_patch(0);

  // this lane's pixels: patch index of tap (0, 0)
  int pq[TA];
#pragma unroll
  for (int a = 0; a < TA; ++a) pq[a] = vidx(min(m0 + wp * 32 * TA + a * 32 + (lane & 31), M - 1)) - vf;
  // scale and shift of the eight channels that this lane finishes
  constexpr int G = WN / 8, RPI = 64 / G, VI = 32 / RPI;   // channel groups, rows per pass, passes
  const int g8 = lane % G, col = n0 + wc * WN + g8 * 8;
  float sc[8], sh[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    sc[e] = 1.0f;
    sh[e] = 0.0f;
  }
  auto load8 = [&](float (&d)[8], const float* g) __attribute__((always_inline)) {
    const u32x4 lo = buffer_load16(g, p.cout * 4, col * 4), hv = buffer_load16(g, p.cout * 4, col * 4 + 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      d[e] = __uint_as_float(lo[e]);
      d[4 + e] = __uint_as_float(hv[e]);
    }
  };
  if (p.scale) load8(sc, p.scale);
  if (p.shift) load8(sh, p.shift);

  f32x16 acc[TB][TA];
#pragma unroll
  for (int b = 0; b < TB; ++b)
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[b][a][r] = 0.f;

  const int nch = cin / 64;

  // MFMA operands: A = weights (32 output channels), B = pixels
  const int wrow = wc * WN + (lane & 31);
  const int wadr = wrow * 128 + ((hi ^ ((wrow >> 1) & 7)) << 4);
  bf16x8 wf[4][TB], pf[4][TA];
  int padr[TA];
  auto fetch_w = [&](const char* st, int s, int b) __attribute__((always_inline)) {
    wf[s][b] = *reinterpret_cast<const bf16x8*>(st + (wadr ^ (s << 5)) + b * 4096);
  };
  auto fetch_p = [&](int s, int a) __attribute__((always_inline)) {
    pf[s][a] = *reinterpret_cast<const bf16x8*>(patch + (padr[a] ^ (s << 5)));
  };
  auto set_tap = [&](int tap, int a) __attribute__((always_inline)) {
    const int dy = tap / 3, q = pq[a] + dy * PW + (tap - dy * 3);
    padr[a] = q * 128 + ((hi ^ ((q >> 1) & 7)) << 4);
  };

#pragma unroll
  for (int a = 0; a < TA; ++a) set_tap(0, a);
  seen_barrier();                                 // the first patch and weights have landed
#pragma unroll
  for (int s = 0; s < D; ++s) {
    if (EARLY)
#pragma unroll
      for (int b = 0; b < TB; ++b) fetch_w(wst, s, b);
#pragma unroll
    for (int a = 0; a < TA; ++a) fetch_p(s, a);
  }
  // One step: the MFMAs of a tap of a chunk from the weight stage at `cur`,
  // while the weights NS - 1 steps ahead (K offset wk) go to the free stage.
  // Loads and LDS reads are spread between the MFMAs: issued together they
  // would hold up the wave (a load straight into LDS takes the load path ~20
  // clocks).  No branch inside a step: past the last step the weights of the
  // last one are loaded again, into a free stage, and the next operands are
  // read for nothing.
  constexpr int NM = TA * TB;
  // loads that may be in flight at the end of a step: those of the stages
  // after the next two (the next step reads the first operands of the one
  // after it)
  constexpr int FLY = (NS - (EARLY ? 3 : 2)) * JW;
  const int S = 9 * nch;
  int wtap = NS - 1, wk = (NS - 1) * cin, cst = 0, lst = (NS - 1) * WS;
  for (int g = 0, tap = 0, chunk = 0; g < S; ++g) {
    const bool turn = tap == 8;
    const int nst = cst + WS == NS * WS ? 0 : cst + WS, tap1 = turn ? 0 : tap + 1;
    if (!EARLY)
#pragma unroll
      for (int s = 0; s < D; ++s)
#pragma unroll
        for (int b = 0; b < TB; ++b) fetch_w(wst + cst, s, b);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        // operands of sub-step s + D in the first half of this one's
        // MFMAs: weights 0, pixels, the other weights
        constexpr int PER = (2 * (TA + TB) + NM - 1) / NM;
#pragma unroll
        for (int f = i * PER; f < (i + 1) * PER && f < TA + TB; ++f) {
          if (f >= 1 && f <= TA) {
            if (s + D == 4) set_tap(tap1, f - 1);
            fetch_p((s + D) & 3, f - 1);
          } else if (s + D < 4 || EARLY) {
            fetch_w(wst + (s + D < 4 ? cst : nst), (s + D) & 3, f ? f - TA : 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        acc[i / TA][i % TA] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[s][i / TA], pf[s][i % TA],
                                                                      acc[i / TA][i % TA], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int JS = (JW + 2) / 3;          // loads per sub-step, in the first three
        const int j = s * JS + i - (NM - JS);
        if (i >= NM - JS && s < 3 && j < JW) issue_w(wst + lst, wk, j);
      }
    }
    cst = nst;
    lst = lst + WS == NS * WS ? 0 : lst + WS;
    if (g + NS < S) {                             // the K offset of the next weights to load
      wk += cin;
      if (++wtap == 9) {
        wtap = 0;
        wk += 64 - 9 * cin;
      }
    }
    tap = tap1;
    if (turn && g + 1 < S) {
      ++chunk;
      lds_barrier();                              // every wave is done with the patch
      issue_patch(chunk);
      seen_barrier();
#pragma unroll
      for (int s = 0; s < D; ++s)
#pragma unroll
        for (int a = 0; a < TA; ++a) fetch_p(s, a);
    } else {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(%1)\n\ts_barrier" ::"n"(FLY), "n"(0) : "memory");
    }
  }

  // epilogue: each wave stages 32 pixels x WN channels of raw sums in its
  // own part of the patch's space, then a lane finishes 8 channels of a pixel
  // (scale / shift, residual, activation, rounding) and stores 16 bytes
  // every residual vector is requested before the first store: loads and
  // stores complete in one order, and a later load would wait for the stores.
  // A wave's LDS operations run in order, so its staging needs no waits of
  // its own, only that the compiler keeps the order.
  const int rw0 = wp * 32 * TA + lane / G;        // this lane's first row in the tile
  u32x4 rv[TA][VI];
  if (RES) {
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
      for (int v = 0; v < VI; ++v)
        rv[a][v] = *reinterpret_cast<const u32x4*>(
            p.res + static_cast<size_t>(min(m0 + rw0 + a * 32 + v * RPI, M - 1)) * p.cout + col);
  }
  seen_barrier();
  float* const ep = reinterpret_cast<float*>((wave & 2 ? wst : patch) + (wave & 1) * EPB);
  // rows past the last one fall outside the store buffer and are dropped
  uint16_t* const dbase = p.dst + static_cast<size_t>(m0) * p.cout;
  const uint32_t dbytes = static_cast<uint32_t>(min(BM, M - m0)) * p.cout * 2;
#pragma unroll
  for (int a = 0; a < TA; ++a) {
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(ep + (lane & 31) * EPW + b * 32 + 8 * q + 4 * hi) =
            make_float4(acc[b][a][4 * q], acc[b][a][4 * q + 1], acc[b][a][4 * q + 2], acc[b][a][4 * q + 3]);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int v = 0; v < VI; ++v) {
      const float* e = ep + (v * RPI + lane / G) * EPW + g8 * 8;
      const float4 lo = *reinterpret_cast<const float4*>(e), hv = *reinterpret_cast<const float4*>(e + 4);
      float x[8] = {lo.x, lo.y, lo.z, lo.w, hv.x, hv.y, hv.z, hv.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = fmaf(x[i], sc[i], sh[i]);
      if (RES) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x[2 * i] += __uint_as_float(rv[a][v][i] << 16);
          x[2 * i + 1] += __uint_as_float(rv[a][v][i] & 0xffff0000u);
        }
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = act_t<ACT>(x[i]);
      u32x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = pack_bf16(x[2 * i], x[2 * i + 1]);
      buffer_store16(dbase, dbytes, static_cast<uint32_t>(((rw0 + a * 32 + v * RPI) * p.cout + col) * 2), o);
    }
    asm volatile("" ::: "memory");
  }
}

template <int TA, int TB, int CAP, int NS, int D, bool EARLY>
void go3t(const Conv3TP& p, int act, hipStream_t s) {
  constexpr int BM = 64 * TA;
  const dim3 grid(static_cast<unsigned>((static_cast<long>(p.n) * p.H * p.W + BM - 1) / BM * p.nt));
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, p); };
  if (p.res) {
    if (act == ACT_RELU) go(conv3t_kernel<TA, TB, CAP, NS, D, EARLY, ACT_RELU, true>);
    else if (act == ACT_GELU) go(conv3t_kernel<TA, TB, CAP, NS, D, EARLY, ACT_GELU, true>);
    else go(conv3t_kernel<TA, TB, CAP, NS, D, EARLY, ACT_NONE, true>);
  } else {
    if (act == ACT_RELU) go(conv3t_kernel<TA, TB, CAP, NS, D, EARLY, ACT_RELU, false>);
    else if (act == ACT_GELU) go(conv3t_kernel<TA, TB, CAP, NS, D, EARLY, ACT_GELU, false>);
    else go(conv3t_kernel<TA, TB, CAP, NS, D, EARLY, ACT_NONE, false>);
  }
}

}  // namespace

bool conv3_tiles_shape(const ConvArgs& a) {
  if (a.k != 3 || a.stride != 1 || a.pad != 1 || a.src2 || a.out_f32 || a.Ho != a.H || a.Wo != a.W || a.cin % 64 ||
      a.cout % 64 || a.Kp != 9 * a.cin || a.src_rows || a.src2_rows || a.res_rows || a.dst_rows || a.pool || a.act > ACT_GELU)
    return false;
  // The smallest images (4 x 4, 3 x 3) go to the implicit GEMM and its K split:
  // faster there up to ~120 of them and slower above (us, 512 -> 512 on 4 x 4, K
  // split | these tiles: 60 images 17.5 | 23.7, 255 40 | 29, 1500 192 | 96).  The
  // two sum in different orders, and a row's bits must not depend on how many
  // rows come with it, so the shape alone decides.
  if (a.H * a.W <= 128 && 2 * a.H * a.W < (a.H + 2) * (a.W + 2)) return false;
  return a.W >= 2 && patch_pixels(128, a.H, a.W) <= 372;   // (the widest images: 79 pixels)
}

bool conv3_tiles(const ConvArgs& a, hipStream_t s) {
  if (!conv3_tiles_shape(a)) return false;
  const int cap = patch_pixels(128, a.H, a.W);
  const long Mh = static_cast<long>(a.nhint > 0 && a.nhint < a.n ? a.nhint : a.n) * a.H * a.W;
  const long mt = (Mh + 127) / 128;
  // 64 input channels on wide images (a patch over 244 pixels: 128 x 64 tiles, 72
  // KB of weights streamed for each): with many tiles, the implicit GEMM's 128 x 128
  // and 128 x 256 ones (us, these | GEMM, 64 -> 256: 4 images of 56x56, 392 tiles,
  // 9.0 | 10.1; 6, 588, 16.7 | 17.6; 8, 784, 19.4 | 17.8; 200, 289 | 204).  Its sums are
  // in the same order.  (Pooling sums are not: see the caller.)
  if (a.cin == 64 && a.cout % 128 == 0 && cap > 244 && mt * (a.cout / 64) > 640) return false;
  Conv3TP p;
  p.src = a.src;
  p.w = a.w;
  p.scale = a.scale;
  p.shift = a.shift;
  p.res = a.res;
  p.dst = static_cast<uint16_t*>(a.dst);
  p.n = a.n;
  p.H = a.H;
  p.W = a.W;
  p.cin = a.cin;
  p.cout = a.cout;
  p.Kp = a.Kp;
  p.nc = a.ncount;
  p.dHW = div_by(a.H * a.W);
  p.dW = div_by(a.W);
  p.dPW = div_by(a.W + 1);
  p.dH1 = div_by(a.H + 1);
  // Tile by the expected number of tiles, measured (us, 128 x 128 | 128 x 64
  // | 64 x 64): 183 images 28x28x128 45 | 51 | 72, 300 of 8x8x256 (300 tiles
  // of 128 x 128) 30 | 34 | 38, 40 of 28x28x128 (245) 12.2 | 12.8 | 17.5, 4 of
  // 28x28x512 (100) 33.2 | 27.5 | 27.1, 10 of 28x28x128 (62) 10.8 | 9.3 | 8.1:
  // with fewer tiles than ~3 of every 4 CUs, the length of a tile's chain
  // counts and not its traffic.  Wide images (a patch over 244 pixels) and
  // other channel counts take 128 x 64.
  if (a.cout % 128 == 0 && cap <= 244 && mt * (a.cout / 128) >= 192) {
    p.nt = a.cout / 128;
    go3t<2, 2, 244, 3, 1, false>(p, a.act, s);
  } else if (cap <= 372 && (mt * (a.cout / 64) >= 256 || patch_pixels(64, a.H, a.W) > 250)) {
    p.nt = a.cout / 64;
    go3t<2, 1, 372, 4, 1, false>(p, a.act, s);
  } else {
    p.nt = a.cout / 64;
    go3t<1, 1, 250, 6, 3, true>(p, a.act, s);
  }
  return true;
}

}  // namespace k
}  // namespace dycl
